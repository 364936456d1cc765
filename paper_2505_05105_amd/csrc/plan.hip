// Setup, part 3 (host side of the runtime): launch plans built once per
// hierarchy from small device arrays copied back.
//
//  * Cut-vertex groups for the extra-smoothing kernel.  One smoothing step
//    applies 4 eta colour phases to the cut vertices; a value after them
//    depends on values at most 4 eta nodes away, so a group owning the cut
//    vertices of one tile and holding every cut vertex within 4 eta of that
//    tile (its closure) computes its own vertices exactly, alone.  A group is
//    one wave with a node of each colour per lane; a tile whose closure has more
//    is split in four.  Levels where that does not help (and eta > 4) take
//    groups of four waves, split until their closure fits in LDS.
//  * The single-workgroup part: the coarsest levels whose arrays (iterate,
//    right-hand side, residual on the bounding box grown by one ring, the
//    stored stencil rows and the cut lists) fit in one workgroup's LDS.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <future>
#include <system_error>

#include "mgfem_internal.h"

namespace mgfem {
namespace {

inline int align16(int v) { return (v + 15) & ~15; }

__global__ void k_cutpos(const int* __restrict__ list, int cnt, int* __restrict__ pos) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < cnt) pos[list[q]] = q;
}

// closure-node coefficients in one contiguous record: 8 off-diagonals, 1/diagonal
__global__ void k_gather_coef(const double* __restrict__ A, int64_t n, const int* __restrict__ node, int cnt,
                              double* __restrict__ out, float* __restrict__ out32) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= cnt) return;
  const int64_t k = node[t];
  const int pl[8] = {0, 1, 2, 3, 5, 6, 7, 8};
  for (int e = 0; e < 8; ++e) {
    const double v = A[pl[e] * n + k];
    out[9 * (int64_t)t + e] = v;
    if (out32) out32[9 * (int64_t)t + e] = (float)v;
  }
  const double d = A[4 * n + k];
  out[9 * (int64_t)t + 8] = 1.0 / d;
  if (out32) out32[9 * (int64_t)t + 8] = 1.0f / (float)d;
}

__global__ void k_fill_i(int* __restrict__ p, int64_t n, int v) {
  const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k < n) p[k] = v;
}

// the same in planes over the slots of each group of one wave
__global__ void k_gather_slots(const double* __restrict__ A, int64_t n, const int* __restrict__ node, int cnt,
                               double* __restrict__ out, float* __restrict__ out32) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= cnt || node[t] < 0) return;
  const int64_t k = node[t];
  const int pl[9] = {0, 1, 2, 3, 5, 6, 7, 8, 4};
  for (int e = 0; e < 9; ++e) {
    const int64_t w = ((int64_t)(t / CutPlan::kSlots) * 9 + e) * CutPlan::kSlots + t % CutPlan::kSlots;
    const double v = A[pl[e] * n + k];
    out[w] = e < 8 ? v : 1.0 / v;
    if (out32) out32[w] = e < 8 ? (float)v : 1.0f / (float)v;
  }
}

struct GroupBuild {
  // groups of one wave: slots, the eight neighbours of each, external sources
  std::vector<int> w_node, w_q, w_ext;
  std::vector<uint16_t> w_nbr;
  std::vector<int> info, node, q, ext;
  std::vector<uint8_t> own;
  std::vector<int16_t> nbr;
  int lds64 = 0, lds32 = 0;
};

// The cut vertices of one level by 16 x 16-node bucket and by tile (the list
// sorted by either, with the runs' starts), and scratch of one group: a grid over
// its box (its closure and one ring) with the position in the level's list, slot
// in the closure and index of the external value, and its lists.
struct GroupLevel {
  const std::vector<uint32_t>& xy;  // column | row << 16 of each cut vertex, in the list's order
  const std::vector<int>&bstart, &bq;
  int N, DX, DY;  // the closure's reach in columns and rows
  size_t lds_cap;
  bool wave;      // one wave per group
  static constexpr int BT = 16;
  int nbx;
  struct Cell {
    int q;
    int16_t slot, ext;
  };
  std::vector<Cell> grid;
  std::vector<int> cl, ext;
  std::vector<int16_t> nbr;
  std::vector<uint16_t> slot;
};

// a list of cut vertices sorted by square of 2^sh nodes (n squares a side)
void by_square(const std::vector<uint32_t>& xy, int sh, int n, std::vector<int>& start, std::vector<int>& list) {
  auto square = [&](uint32_t v) { return ((v & 0xffff) >> sh) + (size_t)(v >> 16 >> sh) * n; };
  start.assign((size_t)n * n + 1, 0);
  for (uint32_t v : xy) ++start[square(v) + 1];
  for (size_t g = 0; g + 1 < start.size(); ++g) start[g + 1] += start[g];
  list.resize(xy.size());
  std::vector<int> at(start.begin(), start.end() - 1);
  for (size_t q = 0; q < xy.size(); ++q) list[at[square(xy[q])]++] = (int)q;
}

// recursively split the rectangle [x0,x1) x [y0,y1) until each closure fits.  The
// host's part of a plan is this: one grid pass per colour instead of a sort, no
// allocation and no division per group (plans of N = 2048 and 1024: 2.7 ms before,
// 2.1 like this).
bool build_groups(GroupLevel& G, int x0, int x1, int y0, int y1, const int* owned_q, int nowned, GroupBuild& gb) {
  if (nowned == 0) return true;
  const std::vector<uint32_t>& xy = G.xy;
  const int N = G.N, DX = G.DX, DY = G.DY, s = N + 1, BT = GroupLevel::BT;
  // closure: cut vertices in the rectangle grown by its reach; the ring around it
  // holds cut vertices whose values are read from the snapshot
  const int bx = x0 - DX - 1, by = y0 - DY - 1, W = x1 - x0 + 2 * DX + 2, H = y1 - y0 + 2 * DY + 2;
  G.grid.assign((size_t)W * H, GroupLevel::Cell{-1, -1, -1});
  const int b0 = std::max(0, bx / BT), b1 = std::min(G.nbx - 1, (bx + W - 1) / BT);
  const int c0 = std::max(0, by / BT), c1 = std::min(G.nbx - 1, (by + H - 1) / BT);
  for (int cy = c0; cy <= c1; ++cy)
    for (int cx = b0; cx <= b1; ++cx) {
      const size_t sq = cx + (size_t)cy * G.nbx;
      for (int w = G.bstart[sq]; w < G.bstart[sq + 1]; ++w) {
        const int q = G.bq[w], i = (int)(xy[q] & 0xffff) - bx, j = (int)(xy[q] >> 16) - by;
        if (i >= 0 && j >= 0 && i < W && j < H) G.grid[i + j * W].q = q;
      }
    }
  // the closure in the order of the level's list: colour, then node index
  std::vector<int>& cl = G.cl;
  cl.clear();
  int col_off[5] = {0, 0, 0, 0, 0}, col_max = 0;
  for (int cc = 0; cc < 4; ++cc) {
    for (int j = 1 + ((by + 1 + (cc >> 1)) & 1); j < H - 1; j += 2)
      for (int i = 1 + ((bx + 1 + (cc & 1)) & 1); i < W - 1; i += 2) {
        GroupLevel::Cell& cell = G.grid[i + j * W];
        if (cell.q < 0) continue;
        cell.slot = (int16_t)std::min<size_t>(cl.size(), 32767);  // (no group keeps as many)
        cl.push_back(cell.q);
      }
    col_off[cc + 1] = (int)cl.size();
    col_max = std::max(col_max, col_off[cc + 1] - col_off[cc]);
  }
  std::vector<int>& ext = G.ext;
  std::vector<int16_t>& nbr = G.nbr;
  ext.clear();
  bool fits = !G.wave || col_max <= CutPlan::kLanes;
  if (fits) {
    nbr.assign(8 * cl.size(), -1);
    const int pl[8] = {0, 1, 2, 3, 5, 6, 7, 8};
    for (size_t t = 0; t < cl.size(); ++t) {
      const int i = (int)(xy[cl[t]] & 0xffff), j = (int)(xy[cl[t]] >> 16);
      for (int e = 0; e < 8; ++e) {
        const int ii = i + pl[e] % 3 - 1, jj = j + pl[e] / 3 - 1;
        if (ii < 0 || jj < 0 || ii > N || jj > N) continue;
        GroupLevel::Cell& cell = G.grid[(ii - bx) + (jj - by) * W];
        if (cell.slot >= 0) {
          nbr[8 * t + e] = cell.slot;
          continue;
        }
        if (cell.ext < 0) {
          cell.ext = (int16_t)std::min<size_t>(ext.size(), 32767);
          ext.push_back(cell.q >= 0 ? -(1 + cell.q) : ii + jj * s);
        }
        nbr[8 * t + e] = (int16_t)std::min<size_t>(cl.size() + cell.ext, 32767);
      }
    }
    const size_t bytes = (size_t)cut_lds_layout((int)cl.size(), (int)ext.size(), (int)sizeof(double)).total;
    fits = G.wave ? ext.size() <= (size_t)CutPlan::kExt : bytes <= G.lds_cap && cl.size() + ext.size() <= 32000;
  }
  if (!fits) {
    if (x1 - x0 <= 4 && y1 - y0 <= 4) return false;
    const int xm = (x0 + x1) / 2, ym = (y0 + y1) / 2;
    const int rx[4][2] = {{x0, xm}, {xm, x1}, {x0, xm}, {xm, x1}};
    const int ry[4][2] = {{y0, ym}, {y0, ym}, {ym, y1}, {ym, y1}};
    for (int h = 0; h < 4; ++h) {
      std::vector<int> sub;
      for (int w = 0; w < nowned; ++w) {
        const int q = owned_q[w], i = (int)(xy[q] & 0xffff), j = (int)(xy[q] >> 16);
        if (i >= rx[h][0] && i < rx[h][1] && j >= ry[h][0] && j < ry[h][1]) sub.push_back(q);
      }
      if (!build_groups(G, rx[h][0], rx[h][1], ry[h][0], ry[h][1], sub.data(), (int)sub.size(), gb)) return false;
    }
    return true;
  }
  if (G.wave) {
    constexpr int NS = CutPlan::kSlots, NL = CutPlan::kLanes, NE = CutPlan::kExt;
    const size_t base = gb.w_node.size(), eb = gb.w_ext.size();
    gb.w_node.resize(base + NS, -1);
    gb.w_q.resize(base + NS, 0);
    gb.w_nbr.resize(8 * (base + NS), 0);
    gb.w_ext.resize(eb + NE, (int)((xy[cl[0]] & 0xffff) + (xy[cl[0]] >> 16) * s));
    std::vector<uint16_t>& slot = G.slot;
    slot.resize(cl.size());
    for (int cc = 0; cc < 4; ++cc)
      for (int t = col_off[cc]; t < col_off[cc + 1]; ++t) slot[t] = (uint16_t)(cc * NL + t - col_off[cc]);
    for (size_t t = 0; t < cl.size(); ++t) {
      const int i = (int)(xy[cl[t]] & 0xffff), j = (int)(xy[cl[t]] >> 16), k = i + j * s;
      const bool own = i >= x0 && i < x1 && j >= y0 && j < y1;
      gb.w_node[base + slot[t]] = k;
      gb.w_q[base + slot[t]] = own ? cl[t] : (int)((unsigned)cl[t] | 0x80000000u);
      for (int e = 0; e < 8; ++e) {
        const int r = nbr[8 * t + e];  // neighbours outside the grid read the zero behind the external values
        gb.w_nbr[8 * (base + slot[t]) + e] =
            r < 0 ? (uint16_t)(NS + NE) : r < (int)cl.size() ? slot[r] : (uint16_t)(NS + r - (int)cl.size());
      }
    }
    for (size_t e = 0; e < ext.size(); ++e) gb.w_ext[eb + e] = ext[e];
    return true;
  }
  const int base = (int)gb.node.size(), ebase = (int)gb.ext.size();
  gb.info.push_back(base);
  gb.info.push_back((int)cl.size());
  gb.info.push_back(ebase);
  gb.info.push_back((int)ext.size());
  for (int cc = 0; cc < 5; ++cc) gb.info.push_back(col_off[cc]);
  for (size_t t = 0; t < cl.size(); ++t) {
    const int i = (int)(xy[cl[t]] & 0xffff), j = (int)(xy[cl[t]] >> 16), k = i + j * s;
    gb.node.push_back(k);
    gb.q.push_back(cl[t]);
    gb.own.push_back((i >= x0 && i < x1 && j >= y0 && j < y1) ? 1 : 0);
  }
  // neighbours outside the grid read the zero slot after the external values
  for (auto& r : nbr)
    if (r < 0) r = (int16_t)(cl.size() + ext.size());
  gb.nbr.insert(gb.nbr.end(), nbr.begin(), nbr.end());
  gb.lds64 = std::max(gb.lds64, cut_lds_layout((int)cl.size(), (int)ext.size(), 8).total);
  gb.lds32 = std::max(gb.lds32, cut_lds_layout((int)cl.size(), (int)ext.size(), 4).total);
  gb.ext.insert(gb.ext.end(), ext.begin(), ext.end());
  return true;
}

template <class V>
int upload(mgfem_ctx* c, V** dst, const std::vector<V>& src) {
  MGFEM_HIP_TRY(ctx_alloc_t(c, dst, std::max<size_t>(1, src.size())));
  if (!src.empty())
    MGFEM_HIP_TRY(hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(V), hipMemcpyHostToDevice, c->s));
  return MGFEM_OK;
}

}  // namespace

namespace {
int lds_cap(mgfem_ctx* c, size_t& cap) {
  int dev = 0, lds_max = 65536;
  MGFEM_HIP_TRY(hipGetDevice(&dev));
  MGFEM_HIP_TRY(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  cap = (size_t)lds_max - 4096;  // room for the kernels' static LDS
  return MGFEM_OK;
}
}  // namespace

// every node's position in its level's cut list (-1: none), built once
int build_cutpos(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  if (L.cutpos) return MGFEM_OK;
  const int cnt = L.cut_off[4];
  MGFEM_HIP_TRY(ctx_alloc_t(c, &L.cutpos, L.n));
  hipLaunchKernelGGL(k_fill_i, dim3((unsigned)((L.n + 255) / 256)), dim3(256), 0, c->s, L.cutpos, L.n, -1);
  if (cnt > 0)
    hipLaunchKernelGGL(k_cutpos, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, c->s, L.cut_list, cnt,
                       L.cutpos);
  MGFEM_HIP_TRY(hipGetLastError());
  return MGFEM_OK;
}

// snapshots and cut groups of one level
int build_cut_groups(mgfem_ctx* c, int l) {
  const bool mixed = c->p.precision == MGFEM_PREC_MIXED;
  size_t cap = 0;
  if (const int e = lds_cap(c, cap)) return e;
  const int D = 4 * c->p.eta;
  // MGFEM_NO_CUT_GROUPS=1: no group plans, so every level takes the list
  // smoother (the path of a level whose groups do not fit in LDS)
  const char* ng_env = std::getenv("MGFEM_NO_CUT_GROUPS");
  const bool no_groups = ng_env && ng_env[0] && ng_env[0] != '0';
  Level& L = c->lv[l];
  const int cnt = L.cut_off[4];
  if (const int e = build_cutpos(c, l)) return e;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &L.snap, std::max(1, cnt)));
  if (mixed) MGFEM_HIP_TRY(ctx_alloc_t(c, &L.snap32, std::max(1, cnt)));
  MGFEM_HIP_TRY(hipGetLastError());
  if (cnt == 0 || c->p.eta == 0 || no_groups) return MGFEM_OK;
  std::vector<int> nodes(cnt);
  MGFEM_HIP_TRY(hipMemcpyAsync(nodes.data(), L.cut_list, cnt * sizeof(int), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  std::vector<uint32_t> xy(cnt);
  for (int q = 0; q < cnt; ++q) xy[q] = (uint32_t)(nodes[q] % L.stride) | (uint32_t)(nodes[q] / L.stride) << 16;
  std::vector<int> bstart, bq;
  GroupLevel G{xy, bstart, bq, L.N, D, D, cap, false, (L.N + GroupLevel::BT) / GroupLevel::BT, {}, {}, {}, {}, {}};
  by_square(xy, 4, G.nbx, bstart, bq);
  const int GT = 32;  // owned tile of one group
  const int ngx = (L.N + GT) / GT;
  std::vector<int> ostart, owned;
  by_square(xy, 5, ngx, ostart, owned);
  std::vector<int> tiles;
  for (int g = 0; g < ngx * ngx; ++g)
    if (ostart[g + 1] > ostart[g]) tiles.push_back(g);
  GroupBuild gb;
  auto build = [&](size_t t0, size_t t1, GroupBuild& out) {
    GroupLevel mine(G);
    bool ok = true;
    for (size_t t = t0; t < t1 && ok; ++t) {
      const int g = tiles[t], x0 = (g % ngx) * GT, y0 = (g / ngx) * GT;
      ok = build_groups(mine, x0, x0 + GT, y0, y0 + GT, owned.data() + ostart[g], ostart[g + 1] - ostart[g], out);
    }
    return ok;
  };
  // Groups of one wave know their own slots only, so runs of tiles are built side
  // by side (a group takes some 5 us, a thread 20 to start) and put together in
  // order.  Plan of N = 2048: 1.34 ms, like this 0.84; mixed set-up of N = 4096
  // 18.7, 16.7.  Below 64 tiles a second thread is not worth its start.
  auto build_waves = [&] {
    const size_t parts = std::min<size_t>(4, tiles.size() / 32);
    if (parts < 2) return build(0, tiles.size(), gb);
    std::vector<GroupBuild> part(parts);
    std::vector<std::future<bool>> run(parts);
    auto at = [&](size_t p) { return tiles.size() * p / parts; };
    bool ok = true;
    for (size_t p = 1; p < parts; ++p) {
      try {
        run[p] = std::async(std::launch::async, [&, p] { return build(at(p), at(p + 1), part[p]); });
      } catch (const std::system_error&) {  // no thread to be had: here, below
      }
    }
    for (size_t p = 0; p < parts; ++p)
      ok = (run[p].valid() ? run[p].get() : build(at(p), at(p + 1), part[p])) && ok;
    if (!ok) return false;
    for (GroupBuild& q : part) {
      gb.w_node.insert(gb.w_node.end(), q.w_node.begin(), q.w_node.end());
      gb.w_q.insert(gb.w_q.end(), q.w_q.begin(), q.w_q.end());
      gb.w_ext.insert(gb.w_ext.end(), q.w_ext.begin(), q.w_ext.end());
      gb.w_nbr.insert(gb.w_nbr.end(), q.w_nbr.begin(), q.w_nbr.end());
    }
    return true;
  };
  // groups of one wave where every one fits (a sweep's four phases reach four
  // columns, but two rows: rows alternate between the even and the odd colours)
  G.wave = true;
  G.DY = D / 2;
  if (c->p.eta <= 4 && build_waves()) {
    CutPlan& P = L.cp;
    const int nslot = (int)gb.w_node.size();
    P.ok = P.wave = true;
    P.ngroups = nslot / CutPlan::kSlots;
    P.units = (P.ngroups + CutPlan::kWaves - 1) / CutPlan::kWaves;
    P.lds64 = CutPlan::kWaves * CutPlan::kVals * (int)sizeof(double);
    P.lds32 = P.lds64 / 2;
    int rc;
    if ((rc = upload(c, &P.w_node, gb.w_node))) return rc;
    if ((rc = upload(c, &P.w_q, gb.w_q))) return rc;
    if ((rc = upload(c, &P.w_ext, gb.w_ext))) return rc;
    MGFEM_HIP_TRY(ctx_alloc_t(c, &P.w_nbr, nslot));
    MGFEM_HIP_TRY(hipMemcpyAsync(P.w_nbr, gb.w_nbr.data(), gb.w_nbr.size() * 2, hipMemcpyHostToDevice, c->s));
    MGFEM_HIP_TRY(ctx_alloc_t(c, &P.w_coef, 9 * (size_t)nslot));
    if (mixed) MGFEM_HIP_TRY(ctx_alloc_t(c, &P.w_coef32, 9 * (size_t)nslot));
    hipLaunchKernelGGL(k_gather_slots, dim3((unsigned)((nslot + 255) / 256)), dim3(256), 0, c->s, L.A, L.n,
                       (const int*)P.w_node, nslot, P.w_coef, P.w_coef32);
    MGFEM_HIP_TRY(hipGetLastError());
    MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
    return MGFEM_OK;
  }
  G.wave = false;
  G.DY = D;
  gb = GroupBuild();
  L.cp.ok = build(0, tiles.size(), gb);
  if (!L.cp.ok) return MGFEM_OK;
  L.cp.ngroups = L.cp.units = (int)gb.info.size() / 9;
  L.cp.lds64 = gb.lds64;
  L.cp.lds32 = gb.lds32;
  int rc;
  if ((rc = upload(c, &L.cp.g_info, gb.info))) return rc;
  if ((rc = upload(c, &L.cp.cl_node, gb.node))) return rc;
  if ((rc = upload(c, &L.cp.cl_q, gb.q))) return rc;
  if ((rc = upload(c, &L.cp.cl_own, gb.own))) return rc;
  if ((rc = upload(c, &L.cp.cl_nbr, gb.nbr))) return rc;
  // entry 0 is read (and not used) by lanes beyond a group's count, so a
  // level whose groups have no external node still gets one (a node index)
  if (gb.ext.empty()) gb.ext.push_back(0);
  if ((rc = upload(c, &L.cp.ext_src, gb.ext))) return rc;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &L.cp.cl_coef, 9 * std::max<size_t>(1, gb.node.size())));
  if (mixed) MGFEM_HIP_TRY(ctx_alloc_t(c, &L.cp.cl_coef32, 9 * std::max<size_t>(1, gb.node.size())));
  if (!gb.node.empty())
    hipLaunchKernelGGL(k_gather_coef, dim3((unsigned)((gb.node.size() + 255) / 256)), dim3(256), 0, c->s, L.A,
                       L.n, L.cp.cl_node, (int)gb.node.size(), L.cp.cl_coef, L.cp.cl_coef32);
  MGFEM_HIP_TRY(hipGetLastError());
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  return MGFEM_OK;
}

int build_coarse_plan(mgfem_ctx* c) {
  const int nl = (int)c->lv.size();
  const bool mixed = c->p.precision == MGFEM_PREC_MIXED;
  size_t cap = 0;
  if (const int e = lds_cap(c, cap)) return e;
  // --- single-workgroup coarse part: as many coarsest levels as fit in LDS
  struct LevHost {
    int W, H, ox, oy, nstored, ncut, nact;
    std::vector<int16_t> slot, cutl, actl;
    std::vector<double> coef;
    int cut_off[5], act_off[5];
  };
  std::vector<LevHost> hosts;
  int total64 = 0;
  int lc = nl;
  for (int l = nl - 1; l >= 1 && nl - l <= 12; --l) {
    Level& L = c->lv[l];
    if (L.N > 256) break;
    LevHost h{};
    h.ox = L.bbox[0] - 1;
    h.oy = L.bbox[2] - 1;
    h.W = L.bbox[1] - L.bbox[0] + 3;
    h.H = L.bbox[3] - L.bbox[2] + 3;
    if (L.empty()) {
      h.ox = h.oy = 0;
      h.W = h.H = 3;
    }
    const int nb = h.W * h.H;
    if (nb > 32000) break;
    std::vector<uint8_t> fl(L.n);
    std::vector<double> A(9 * L.n);
    MGFEM_HIP_TRY(hipMemcpyAsync(fl.data(), L.flags, L.n, hipMemcpyDeviceToHost, c->s));
    MGFEM_HIP_TRY(hipMemcpyAsync(A.data(), L.A, 9 * L.n * sizeof(double), hipMemcpyDeviceToHost, c->s));
    std::vector<int> cl(std::max(1, L.cut_off[4]));
    if (L.cut_off[4] > 0)
      MGFEM_HIP_TRY(hipMemcpyAsync(cl.data(), L.cut_list, L.cut_off[4] * sizeof(int), hipMemcpyDeviceToHost, c->s));
    MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
    const bool coarsest = l == nl - 1;
    h.slot.assign(nb, -2);
    h.nstored = 0;
    std::vector<int16_t> bycol[4];
    const int pl[8] = {0, 1, 2, 3, 5, 6, 7, 8};
    for (int q = 0; q < nb; ++q) {
      const int gi = h.ox + q % h.W, gj = h.oy + q / h.W;
      if (gi < 0 || gj < 0 || gi > L.N || gj > L.N) continue;
      const int64_t k = gi + (int64_t)gj * L.stride;
      const uint8_t f = fl[k];
      if (!(f & kFlagActive)) continue;  // the outer ring of the box is never active
      if (coarsest) bycol[0].push_back((int16_t)q);  // ascending node order (the inverse's order)
      else bycol[(gi & 1) + 2 * (gj & 1)].push_back((int16_t)q);
      if (f & kFlagStored) {
        h.slot[q] = (int16_t)h.nstored++;
        for (int e = 0; e < 8; ++e) h.coef.push_back(A[pl[e] * L.n + k]);
        h.coef.push_back(A[4 * L.n + k]);
        h.coef.push_back(1.0 / A[4 * L.n + k]);
      } else {
        h.slot[q] = -1;
      }
    }
    if (h.nstored > 32000) break;
    h.act_off[0] = 0;
    for (int cc = 0; cc < 4; ++cc) {
      h.actl.insert(h.actl.end(), bycol[cc].begin(), bycol[cc].end());
      h.act_off[cc + 1] = (int)h.actl.size();
    }
    h.nact = (int)h.actl.size();
    h.ncut = coarsest ? 0 : L.cut_off[4];
    for (int cc = 0; cc < 5; ++cc) h.cut_off[cc] = coarsest ? 0 : L.cut_off[cc];
    for (int q = 0; q < h.ncut; ++q) {
      const int k = cl[q], gi = k % L.stride, gj = k / L.stride;
      h.cutl.push_back((int16_t)((gi - h.ox) + (gj - h.oy) * h.W));
    }
    auto bytes = [&](int ts) {
      int bsz = 3 * align16(nb * ts) + align16(h.nact * 2) + align16(nb * 2) + align16(10 * h.nstored * ts) +
                align16(h.ncut * 2);
      if (coarsest) bsz += align16(c->coarse_n * c->coarse_n * 8);
      return bsz;
    };
    if (coarsest && h.nact != c->coarse_n) {
      c->last_error = "coarsest active count mismatch";
      return MGFEM_ERR_HIP;
    }
    if (total64 + bytes(8) > (int)cap) break;
    total64 += bytes(8);
    hosts.insert(hosts.begin(), h);
    lc = l;
  }
  if (hosts.empty() || lc + (int)hosts.size() != nl) {
    c->last_error = "the coarsest grid does not fit in one workgroup's LDS";
    return MGFEM_ERR_UNSUPPORTED;
  }
  // descriptors: a float64 block and a float32 block (same layout, different LDS offsets)
  CoarsePlan& P = c->cplan;
  P.lc = lc;
  P.ndesc = (int)hosts.size();
  std::vector<int> desc;
  std::vector<double> coef;
  std::vector<int16_t> slot, cutl, actl;
  for (int pass = 0; pass < 2; ++pass) {
    const int ts = pass == 0 ? 8 : 4;
    // LDS: first the static block of every level (colour lists, row slots,
    // rows, cut lists, the coarsest inverse), padded to whole 1 KB chunks
    // (copied from the image), then the vectors x, b, r of every level
    // (zeroed in place)
    int off = 0, coef_off = 0, slot_off = 0, cut_off = 0, act_off = 0;
    std::vector<int> lev_desc(kDesc * P.ndesc, 0);
    for (int q = 0; q < P.ndesc; ++q) {
      const LevHost& h = hosts[q];
      const int nb = h.W * h.H;
      int* d = lev_desc.data() + kDesc * q;
      d[0] = c->lv[lc + q].N;
      d[1] = h.W;
      d[2] = h.H;
      d[3] = h.ox;
      d[4] = h.oy;
      d[5] = coef_off;
      d[6] = slot_off;
      for (int cc = 0; cc < 5; ++cc) d[7 + cc] = cut_off + h.cut_off[cc];
      d[15] = off;
      off += align16(h.nact * 2);
      d[16] = off;
      off += align16(nb * 2);
      d[17] = off;
      off += align16(10 * h.nstored * ts);
      d[18] = off;
      off += align16(h.ncut * 2);
      d[19] = h.nstored;
      if (q == P.ndesc - 1) {
        d[20] = off;
        off += align16(c->coarse_n * c->coarse_n * 8);
      }
      for (int cc = 0; cc < 5; ++cc) d[21 + cc] = act_off + h.act_off[cc];
      coef_off += h.nstored;
      slot_off += nb;
      cut_off += h.ncut;
      act_off += h.nact;
      if (pass == 0) {
        coef.insert(coef.end(), h.coef.begin(), h.coef.end());
        slot.insert(slot.end(), h.slot.begin(), h.slot.end());
        cutl.insert(cutl.end(), h.cutl.begin(), h.cutl.end());
        actl.insert(actl.end(), h.actl.begin(), h.actl.end());
      }
    }
    off = (off + 1023) / 1024 * 1024;
    if (pass == 0) P.static64 = off;
    else P.static32 = off;
    for (int q = 0; q < P.ndesc; ++q) {
      const LevHost& h = hosts[q];
      const int nb = h.W * h.H;
      int* d = lev_desc.data() + kDesc * q;
      d[12] = off;
      off += align16(nb * ts);
      d[13] = off;
      off += align16(nb * ts);
      d[14] = off;
      off += align16(nb * ts);
    }
    desc.insert(desc.end(), lev_desc.begin(), lev_desc.end());
    if (pass == 0) P.lds64 = off;
    else P.lds32 = off;
  }
  // LDS images: static parts at their offsets, vectors zero, the inverse
  // copied in on the device below
  std::vector<unsigned char> img[2];
  img[0].assign(P.static64, 0);
  img[1].assign(P.static32, 0);
  for (int pass = 0; pass < 2; ++pass) {
    for (int q = 0; q < P.ndesc; ++q) {
      const LevHost& h = hosts[q];
      const int* d = desc.data() + kDesc * (pass * P.ndesc + q);
      unsigned char* b = img[pass].data();
      std::memcpy(b + d[15], h.actl.data(), h.actl.size() * 2);
      std::memcpy(b + d[16], h.slot.data(), h.slot.size() * 2);
      std::memcpy(b + d[18], h.cutl.data(), h.cutl.size() * 2);
      if (pass == 0) {
        std::memcpy(b + d[17], h.coef.data(), h.coef.size() * 8);
      } else {
        std::vector<float> f32(h.coef.begin(), h.coef.end());
        std::memcpy(b + d[17], f32.data(), f32.size() * 4);
      }
    }
  }
  int rc;
  if ((rc = upload(c, &P.img64, img[0]))) return rc;
  if ((rc = upload(c, &P.img32, img[1]))) return rc;
  {
    const int last64 = desc[kDesc * (P.ndesc - 1) + 20], last32 = desc[kDesc * (2 * P.ndesc - 1) + 20];
    const size_t ib = (size_t)c->coarse_n * c->coarse_n * sizeof(double);
    MGFEM_HIP_TRY(hipMemcpyAsync(P.img64 + last64, P.inv, ib, hipMemcpyDeviceToDevice, c->s));
    MGFEM_HIP_TRY(hipMemcpyAsync(P.img32 + last32, P.inv, ib, hipMemcpyDeviceToDevice, c->s));
  }
  if ((rc = upload(c, &P.desc, desc))) return rc;
  if ((rc = upload(c, &P.coef, coef))) return rc;
  if (mixed) {
    std::vector<float> c32(coef.begin(), coef.end());
    if ((rc = upload(c, &P.coef32, c32))) return rc;
  }
  if ((rc = upload(c, &P.slot, slot))) return rc;
  if ((rc = upload(c, &P.cutl, cutl))) return rc;
  if ((rc = upload(c, &P.actl, actl))) return rc;
  {
    // grid indices of the first coarse level's active nodes in its list order
    // (rows and columns of the coarse map)
    const LevHost& h = hosts[0];
    const int s0 = c->lv[lc].stride;
    std::vector<int> gidx(std::max(1, h.nact));
    for (int q = 0; q < h.nact; ++q)
      gidx[q] = (h.ox + h.actl[q] % h.W) + (h.oy + h.actl[q] / h.W) * s0;
    if ((rc = upload(c, &P.map.idx, gidx))) return rc;
    P.map.n = h.nact;
  }
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  set_kernel_attributes();
  return MGFEM_OK;
}

}  // namespace mgfem
