"""The batched autotuner's saved choices (MGFEM_TUNE_CACHE)."""
import re

import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_choices_of_earlier_kernels_are_timed_again(tmp_path, monkeypatch):
    """A choice saved under the number of an earlier set of candidates does not
    decide; one saved under the present number does."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    monkeypatch.delenv("MGFEM_BATCH_PATH", raising=False)

    def batch(sizes, path):
        monkeypatch.setenv("MGFEM_TUNE_CACHE", str(path))
        b = mg.BatchedSolver([W.circle(N, radius=0.7) for N in sizes], sizes)
        tile = b.tile
        b.close()
        return tile

    first = tmp_path / "first"
    sizes = [32, 64, 64]
    tile = batch(sizes, first)
    (line,) = first.read_text().splitlines()
    key, choice = line.split()
    assert int(choice) == tile
    version = int(re.search(r"paths=(\d+)", key).group(1))
    # another batch each time: the process remembers its own choices
    for count, earlier in ((5, 2), (6, 1), (7, 0)):
        sizes = [32] * count + [64]
        nodes = sum((n + 1) ** 2 for n in sizes)
        assert version > 2
        name = key.replace(f"paths={version}", f"paths={version - earlier}")
        name = re.sub(r"count=\d+", f"count={len(sizes)}", re.sub(r"nodes=\d+", f"nodes={nodes}", name))
        path = tmp_path / f"saved{count}"
        path.write_text(f"{name} 256\n")
        tile = batch(sizes, path)
        lines = path.read_text().splitlines()
        if earlier:
            assert len(lines) == 2 and f"paths={version}|" in lines[1] and int(lines[1].split()[1]) == tile
        else:
            assert len(lines) == 1 and tile == 256
