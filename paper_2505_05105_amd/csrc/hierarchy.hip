// Setup on the device, part 2: the Galerkin hierarchy and its bookkeeping.
//
// Coarse operators A_{l+1} = R A_l P with P the bilinear prolongation of the
// exact shape-function relation (section 5.1) and R = P^T (eq. galerkin,
// read with the operators in the order that makes the product square).  Each
// coarse row is gathered from the nine fine rows in the support of its coarse
// shape function, so the product needs no atomics and is deterministic.
// A coarse node is active when its diagonal is non-zero.  A coarse row is the
// constant interior Q1 stencil when all nine fine rows it is built from are
// (shape functions are nested); such rows are marked as not stored.
// Cut cells of a coarse grid are those containing a cut fine cell; their
// vertices form the extra-smoothing set of that level (every level but the
// coarsest).  The coarsest active block is factored by Cholesky.
#include <algorithm>
#include <cmath>

#include "mgfem_internal.h"

namespace mgfem {
namespace {

__device__ inline double pw(int d) { return d == 0 ? 1.0 : 0.5; }  // 1D prolongation weight

__global__ void k_rap(const double* __restrict__ Af, const uint8_t* __restrict__ flf, int Nf,
                      double* __restrict__ Ac, uint8_t* __restrict__ flc, int Nc) {
  const int sf = Nf + 1, sc = Nc + 1;
  const int64_t nf = (int64_t)sf * sf, nc = (int64_t)sc * sc;
  int64_t kc = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (kc >= nc) return;
  const int I = (int)(kc % sc), J = (int)(kc / sc);
  double acc[9];
  for (int q = 0; q < 9; ++q) acc[q] = 0.0;
  bool regular = true;
  for (int b = -1; b <= 1; ++b)
    for (int a = -1; a <= 1; ++a) {
      const int fi = 2 * I + a, fj = 2 * J + b;
      if (fi < 0 || fj < 0 || fi > Nf || fj > Nf) {
        regular = false;
        continue;
      }
      const int64_t fk = fi + (int64_t)fj * sf;
      const uint8_t fl = flf[fk];
      if ((fl & kFlagStored) || !(fl & kFlagActive)) regular = false;
      if (!(fl & kFlagActive)) continue;
      const double wi = pw(a) * pw(b);
      for (int ey = -1; ey <= 1; ++ey)
        for (int ex = -1; ex <= 1; ++ex) {
          const double aij = Af[((ex + 1) + 3 * (ey + 1)) * nf + fk];
          if (aij == 0.0) continue;
          const int gi = fi + ex, gj = fj + ey;  // column node j
          for (int dy = -1; dy <= 1; ++dy) {
            const int py = gj - 2 * (J + dy);
            if (py < -1 || py > 1 || J + dy < 0 || J + dy > Nc) continue;
            for (int dx = -1; dx <= 1; ++dx) {
              const int px = gi - 2 * (I + dx);
              if (px < -1 || px > 1 || I + dx < 0 || I + dx > Nc) continue;
              acc[(dx + 1) + 3 * (dy + 1)] += wi * aij * (pw(px) * pw(py));
            }
          }
        }
    }
  for (int q = 0; q < 9; ++q) Ac[q * nc + kc] = acc[q];
  uint8_t f = 0;
  if (acc[4] != 0.0) {
    f |= kFlagActive;
    if (!regular) f |= kFlagStored;
  }
  flc[kc] = f;
}

__global__ void k_coarsen_cells(const uint8_t* __restrict__ cf, int Nf, uint8_t* __restrict__ cc,
                                int Nc) {
  int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (c >= (int64_t)Nc * Nc) return;
  int I = (int)(c % Nc), J = (int)(c / Nc);
  int64_t f0 = 2 * I + (int64_t)(2 * J) * Nf;
  cc[c] = (cf[f0] | cf[f0 + 1] | cf[f0 + Nf] | cf[f0 + Nf + 1]) ? 1 : 0;
}

// Marks the vertices of cut cells (active ones), and the level's counts:
// bounding box of the active nodes, active rows, stored rows.  A fixed grid
// strides over the nodes, so that only kCountBlocks blocks touch the five
// shared counters (one atomic per node cost 52 ms at N = 16384).
constexpr int kCountBlocks = 1024;
struct LevelCounts {
  int bbox[4];  // i_lo, i_hi, j_lo, j_hi
  unsigned long long active, stored;
};
__global__ __launch_bounds__(256) void k_mark_count(const uint8_t* __restrict__ cellcut, int N,
                                                    uint8_t* __restrict__ fl, int mark, LevelCounts* __restrict__ out) {
  __shared__ int sb[4], sn[2];
  if (threadIdx.x < 2) {
    sb[2 * threadIdx.x] = 1 << 30;
    sb[2 * threadIdx.x + 1] = -1;
    sn[threadIdx.x] = 0;
  }
  __syncthreads();
  const int s = N + 1;
  int ilo = 1 << 30, ihi = -1, jlo = 1 << 30, jhi = -1, na = 0, ns = 0;
  for (int64_t k = blockIdx.x * 256ll + threadIdx.x; k < (int64_t)s * s; k += 256ll * gridDim.x) {
    const uint8_t f = fl[k];
    if (!(f & kFlagActive)) continue;
    const int i = (int)(k % s), j = (int)(k / s);
    ++na;
    if (f & kFlagStored) {
      ++ns;
      // a vertex of a cut cell is a stored row
      bool cut = false;
      if (mark)
        for (int cy = j - 1; cy <= j; ++cy)
          for (int cx = i - 1; cx <= i; ++cx)
            if (cx >= 0 && cy >= 0 && cx < N && cy < N && cellcut[cx + (int64_t)cy * N]) cut = true;
      if (cut) fl[k] = f | kFlagCut;
    }
    ilo = min(ilo, i);
    ihi = max(ihi, i);
    jlo = min(jlo, j);
    jhi = max(jhi, j);
  }
  for (int o = 32; o > 0; o >>= 1) {
    ilo = min(ilo, __shfl_xor(ilo, o));
    ihi = max(ihi, __shfl_xor(ihi, o));
    jlo = min(jlo, __shfl_xor(jlo, o));
    jhi = max(jhi, __shfl_xor(jhi, o));
    na += __shfl_xor(na, o);
    ns += __shfl_xor(ns, o);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&sb[0], ilo);
    atomicMax(&sb[1], ihi);
    atomicMin(&sb[2], jlo);
    atomicMax(&sb[3], jhi);
    atomicAdd(&sn[0], na);
    atomicAdd(&sn[1], ns);
  }
  __syncthreads();
  if (threadIdx.x == 0 && sn[0]) {
    atomicMin(&out->bbox[0], sb[0]);
    atomicMax(&out->bbox[1], sb[1]);
    atomicMin(&out->bbox[2], sb[2]);
    atomicMax(&out->bbox[3], sb[3]);
    atomicAdd(&out->active, (unsigned long long)sn[0]);
    atomicAdd(&out->stored, (unsigned long long)sn[1]);
  }
}
__global__ void k_counts_init(LevelCounts* c, int n) {
  const int q = threadIdx.x;
  if (q < n) c[q] = LevelCounts{{1 << 30, -1, 1 << 30, -1}, 0, 0};
}

// Ordered compaction of the cut vertices, one list per colour, by rows: one
// wave per grid row counts them (cnt: colour-major, rows ascending), one
// workgroup turns the counts into offsets, one wave per row writes its own.
__global__ __launch_bounds__(256) void k_row_count(const uint8_t* __restrict__ fl, int N, int j0, int j1, int i0,
                                                   int i1, int* __restrict__ cnt /* 4 x (N+1) */) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, s = N + 1;
  if (j > N) return;
  int n0 = 0, n1 = 0;  // even and odd columns
  if (j >= j0 && j <= j1)
    for (int b = i0 & ~1; b <= i1; b += 64) {
      const int i = b + lane;
      const bool on = i >= i0 && i <= i1 && (fl[i + (int64_t)j * s] & kFlagCut);
      const unsigned long long m = __ballot(on);
      n0 += __popcll(m & 0x5555555555555555ull);
      n1 += __popcll(m & 0xaaaaaaaaaaaaaaaaull);
    }
  if (lane < 4) cnt[lane * s + j] = (lane >> 1) == (j & 1) ? ((lane & 1) ? n1 : n0) : 0;
}

__global__ __launch_bounds__(1024) void k_row_scan(int* __restrict__ cnt, int s, int* __restrict__ tot /* 5 */) {
  __shared__ int sa[1024];
  const int t = threadIdx.x, n = 4 * s, per = (n + 1023) / 1024, lo = min(n, t * per), hi = min(n, lo + per);
  int a = 0;
  for (int q = lo; q < hi; ++q) a += cnt[q];
  sa[t] = a;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = t >= o ? sa[t - o] : 0;
    __syncthreads();
    sa[t] += v;
    __syncthreads();
  }
  int x = sa[t] - a;
  for (int q = lo; q < hi; ++q) {
    const int v = cnt[q];
    cnt[q] = x;
    if (q % s == 0) tot[q / s] = x;
    x += v;
  }
  if (t == 1023) tot[4] = sa[1023];
}

__global__ __launch_bounds__(256) void k_row_scatter(const uint8_t* __restrict__ fl, int N, int j0, int j1, int i0,
                                                     int i1, const int* __restrict__ off, int* __restrict__ list) {
  const int j = j0 + blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, s = N + 1;
  if (j > j1) return;
  int p0 = off[2 * (j & 1) * s + j], p1 = off[(2 * (j & 1) + 1) * s + j];
  for (int b = i0 & ~1; b <= i1; b += 64) {
    const int i = b + lane;
    const bool on = i >= i0 && i <= i1 && (fl[i + (int64_t)j * s] & kFlagCut);
    const unsigned long long m = __ballot(on), e = m & 0x5555555555555555ull, o = m & 0xaaaaaaaaaaaaaaaaull;
    const unsigned long long below = (1ull << lane) - 1;
    if (on) list[(lane & 1) ? p1 + __popcll(o & below) : p0 + __popcll(e & below)] = (int)(i + (int64_t)j * s);
    p0 += __popcll(e);
    p1 += __popcll(o);
  }
}

// Gather and factor the coarsest active block, and its explicit inverse
// L^-T L^-1, by one workgroup: right-looking Cholesky (every entry takes its
// subtractions in column order), then a column of the inverse per thread.
// The factor and the columns are kept in LDS where they fit (cn <= kFactorLds:
// 16 to 40 unknowns with 4 x 4 cells; one thread took 0.4 to 1.9 ms).
constexpr int kFactorLds = 64;
__global__ __launch_bounds__(256) void k_coarse_factor(const double* __restrict__ A, const uint8_t* __restrict__ fl,
                                                       int N, double* __restrict__ Lg, double* __restrict__ Xg,
                                                       int* __restrict__ idx, double* __restrict__ inv, Stats* st) {
  __shared__ double sL[kFactorLds * kFactorLds], sX[kFactorLds * kFactorLds];
  __shared__ int scn, bad;
  const int s = N + 1, n = s * s, t = threadIdx.x;
  if (t < 64) {
    int m = 0;
    for (int k0 = 0; k0 < n; k0 += 64) {
      const bool on = k0 + t < n && (fl[k0 + t] & kFlagActive);
      const unsigned long long b = __ballot(on);
      if (on) idx[m + __popcll(b & ((1ull << t) - 1))] = k0 + t;
      m += __popcll(b);
    }
    if (t == 0) {
      scn = m;
      bad = 0;
    }
  }
  __syncthreads();
  const int cn = scn;
  double* Lm = cn <= kFactorLds ? sL : Lg;
  double* X = cn <= kFactorLds ? sX : Xg;  // column col of the inverse: X[i * cn + col]
  for (int r = t; r < cn * cn; r += 256) {
    const int k = idx[r / cn], kk = idx[r % cn], di = kk % s - k % s, dj = kk / s - k / s;
    Lm[r] = abs(di) <= 1 && abs(dj) <= 1 ? A[(int64_t)((di + 1) + 3 * (dj + 1)) * n + k] : 0.0;
  }
  __syncthreads();
  for (int j = 0; j < cn; ++j) {
    const double d = Lm[j * cn + j];
    if (!(d > 0.0)) {  // uniform
      if (t == 0) bad = 1;
      break;
    }
    __syncthreads();
    const double q = sqrt(d);
    for (int i = j + t; i < cn; i += 256) Lm[i * cn + j] = i == j ? q : Lm[i * cn + j] / q;
    __syncthreads();
    const int m = cn - j - 1;
    for (int r = t; r < m * m; r += 256) {
      const int i = j + 1 + r / m, c = j + 1 + r % m;
      if (c <= i) Lm[i * cn + c] -= Lm[i * cn + j] * Lm[c * cn + j];
    }
    __syncthreads();
  }
  __syncthreads();
  if (t == 0) {
    st->coarse_status = bad;
    st->coarse_n = cn;
  }
  if (bad) return;
  for (int col = t; col < cn; col += 256) {
    for (int i = 0; i < cn; ++i) {
      double v = (i == col) ? 1.0 : 0.0;
      for (int q = 0; q < i; ++q) v -= Lm[i * cn + q] * X[q * cn + col];
      X[i * cn + col] = v / Lm[i * cn + i];
    }
    for (int i = cn - 1; i >= 0; --i) {
      double v = X[i * cn + col];
      for (int q = i + 1; q < cn; ++q) v -= Lm[q * cn + i] * X[q * cn + col];
      X[i * cn + col] = v / Lm[i * cn + i];
    }
    for (int i = 0; i < cn; ++i) inv[(int64_t)col * cn + i] = X[i * cn + col];  // stored by rows (symmetric)
  }
}

__global__ void k_to_float(const double* __restrict__ src, float* __restrict__ dst, int64_t n) {
  int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k < n) dst[k] = (float)src[k];
}

inline unsigned nblk(int64_t n, int tb) { return (unsigned)((n + tb - 1) / tb); }

}  // namespace

int setup_hierarchy(mgfem_ctx* c, const double* psi_in, const double* chi_in) {
  const int tb = 256;
  const int nl = (int)c->lv.size();
  const bool mixed = c->p.precision == MGFEM_PREC_MIXED;
  // coarse operators
  for (int l = 0; l + 1 < nl; ++l) {
    Level& F = c->lv[l];
    Level& C = c->lv[l + 1];
    if (c->p.coarse_op == MGFEM_COARSE_REDISCRETISED) {
      const int rc = assemble_level(c, l + 1, psi_in, chi_in);
      if (rc != MGFEM_OK) return rc;
      continue;
    }
    MGFEM_HIP_TRY(ctx_alloc_t(c, &C.A, 9 * C.n));
    MGFEM_HIP_TRY(ctx_alloc_t(c, &C.flags, C.n));
    MGFEM_HIP_TRY(ctx_alloc_t(c, &C.cellcut, (int64_t)C.N * C.N));
    hipLaunchKernelGGL(k_rap, dim3(nblk(C.n, tb)), dim3(tb), 0, c->s, F.A, F.flags, F.N, C.A,
                       C.flags, C.N);
    hipLaunchKernelGGL(k_coarsen_cells, dim3(nblk((int64_t)C.N * C.N, tb)), dim3(tb), 0, c->s,
                       F.cellcut, F.N, C.cellcut, C.N);
  }
  MGFEM_HIP_TRY(hipGetLastError());
  // cut marks, bounding boxes, active and stored row counts
  LevelCounts* cd = nullptr;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &cd, nl));
  hipLaunchKernelGGL(k_counts_init, dim3(1), dim3(64), 0, c->s, cd, nl);
  for (int l = 0; l < nl; ++l) {
    Level& L = c->lv[l];
    hipLaunchKernelGGL(k_mark_count, dim3(std::min(kCountBlocks, (int)nblk(L.n, tb))), dim3(tb), 0, c->s, L.cellcut,
                       L.N, L.flags, (l + 1 < nl) ? 1 : 0, cd + l);
  }
  MGFEM_HIP_TRY(hipGetLastError());
  std::vector<LevelCounts> ch(nl);
  MGFEM_HIP_TRY(hipMemcpyAsync(ch.data(), cd, nl * sizeof(LevelCounts), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  for (int l = 0; l < nl; ++l) {
    Level& L = c->lv[l];
    for (int q = 0; q < 4; ++q) L.bbox[q] = ch[l].bbox[q];
    if (L.bbox[1] < 0) {  // empty level
      L.bbox[0] = 1;
      L.bbox[1] = 0;
      L.bbox[2] = 1;
      L.bbox[3] = 0;
    }
    L.n_active = (int64_t)ch[l].active;
    L.n_stored = (int64_t)ch[l].stored;
  }
  if (c->lv[0].empty()) {
    c->last_error = "no active node: the level set has no point with psi < 0 after snapping";
    return MGFEM_ERR_EMPTY_DOMAIN;
  }
  // cut lists: the offsets of every level in one copy, then the lists
  int *cnt = nullptr, *tot = nullptr;
  size_t rows = 0;
  for (int l = 0; l + 1 < nl; ++l) rows += 4 * (size_t)c->lv[l].stride;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &cnt, rows));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &tot, 5 * nl));
  std::vector<int> toth(5 * nl);
  std::vector<int*> lcnt(nl, cnt);
  for (int l = 0; l + 1 < nl; ++l) {
    const Level& L = c->lv[l];
    if (l > 0) lcnt[l] = lcnt[l - 1] + 4 * c->lv[l - 1].stride;
    hipLaunchKernelGGL(k_row_count, dim3(nblk(L.stride, 4)), dim3(tb), 0, c->s, L.flags, L.N, L.bbox[2], L.bbox[3],
                       L.bbox[0], L.bbox[1], lcnt[l]);
    hipLaunchKernelGGL(k_row_scan, dim3(1), dim3(1024), 0, c->s, lcnt[l], L.stride, tot + 5 * l);
  }
  MGFEM_HIP_TRY(hipMemcpyAsync(toth.data(), tot, 5 * nl * sizeof(int), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  for (int l = 0; l + 1 < nl; ++l) {
    Level& L = c->lv[l];
    for (int q = 0; q < 5; ++q) L.cut_off[q] = toth[5 * l + q];
    MGFEM_HIP_TRY(ctx_alloc_t(c, &L.cut_list, std::max(1, L.cut_off[4])));
    if (L.cut_off[4] > 0)
      hipLaunchKernelGGL(k_row_scatter, dim3(nblk(L.bbox[3] - L.bbox[2] + 1, 4)), dim3(tb), 0, c->s, L.flags, L.N,
                         L.bbox[2], L.bbox[3], L.bbox[0], L.bbox[1], (const int*)lcnt[l], L.cut_list);
  }
  MGFEM_HIP_TRY(hipGetLastError());
  // work vectors (zero-initialised: inactive entries are read but never written)
  for (int l = 0; l < nl; ++l) {
    Level& L = c->lv[l];
    MGFEM_HIP_TRY(ctx_alloc_t(c, &L.X[0], L.n));
    if (l > 0) MGFEM_HIP_TRY(ctx_alloc_t(c, &L.b, L.n));
    MGFEM_HIP_TRY(ctx_alloc_t(c, &L.X[1], L.n));
    if (l == 0) c->x0 = L.X[0];
    if (mixed) {
      MGFEM_HIP_TRY(ctx_alloc_t(c, &L.A32, 9 * L.n));
      hipLaunchKernelGGL(k_to_float, dim3(nblk(9 * L.n, tb)), dim3(tb), 0, c->s, L.A, L.A32,
                         9 * L.n);
      MGFEM_HIP_TRY(ctx_alloc_t(c, &L.X32[0], L.n));
      MGFEM_HIP_TRY(ctx_alloc_t(c, &L.X32[1], L.n));
      MGFEM_HIP_TRY(ctx_alloc_t(c, &L.b32, L.n));
    }
  }
  // coarsest factorisation
  Level& Lc = c->lv[nl - 1];
  const int cmax = (int)Lc.n;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &c->coarse_idx, cmax));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &c->cplan.inv, (int64_t)cmax * cmax));
  double* work = nullptr;  // the factor and the inverse's columns where they do not fit in LDS
  const int64_t block = cmax > kFactorLds ? (int64_t)cmax * cmax : 1;
  MGFEM_HIP_TRY(ctx_alloc_t(c, &work, 2 * block));
  hipLaunchKernelGGL(k_coarse_factor, dim3(1), dim3(256), 0, c->s, Lc.A, Lc.flags, Lc.N, work, work + block,
                     c->coarse_idx, c->cplan.inv, c->stats);
  MGFEM_HIP_TRY(hipGetLastError());
  return MGFEM_OK;
}

}  // namespace mgfem
