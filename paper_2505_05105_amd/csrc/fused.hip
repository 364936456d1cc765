// Smoothing steps of the levels whose launches are bound by latency, not by
// bytes, with the extra cut-vertex smoothing folded into the
// kernel that reads its result.
//
// The eta sweeps over the cut vertices start from an iterate x with residual
// r = b - A x and are linear: they change x at the cut vertices by
// Delta = D r, with r taken at the cut vertices only and D fixed by the level's
// rows.  A sweep carries a value at most 4 nodes along x and 2 along y (colours
// 0, 1 are the even grid rows, 2, 3 the odd ones), so row p of D has its
// columns within (4 eta, 2 eta) nodes of p.  A sweep leaves r at the cut
// vertices of its tile (one more ring of halo pays for it), and whatever
// reads the iterate next (the next sweep, the residual, the prolongation to
// the finer level) adds D r to the cut vertices of its staged region.  The
// iterate in memory is then short of its last cut sweeps ("pending").
//
// Why: on MI355X a dependent launch costs 1.64 us before it does anything,
// and the 16 barrier-separated colour phases of the cut kernel another 2 us;
// a level's step was two launches of 4.6 us each (N = 512).  As a product the
// cut sweeps are one pass over D beside the staging loads.  What bounds these
// kernels is their chain of dependent loads, so a tile's record holds
// everything at addresses that follow from the tile's number: the columns to
// gather r from, the rows, and D cut into segments of 16 values of one row,
// one segment per thread, all its loads in flight together.
//
// Float32 cycles keep the cut sweeps as launches of their own: a mixed solve
// stops where its float32 rounding leaves it (its result moves by 4e-9 when
// that rounding changes), so their arithmetic stays, operation for operation,
// that of the separate kernels, and only the tiles, the staging and the work
// of a thread differ.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "mgfem_internal.h"
#include "reduce.h"

namespace mgfem {
namespace {

constexpr int kCell = 4;  // nodes per side of a block's cell
// Tiles of FT x FT nodes and their staged region: a sweep is exact on the core
// grown by one ring (the ring feeds the residual at the core's cut vertices).
// Colours 0, 1 are the even grid rows and 2, 3 the odd ones, so a sweep needs
// the start iterate only two rows beyond that, but four columns.  The
// prolongation reads the CRW x CRH coarse nodes under the region.
constexpr int kHX = 5, kHY = 3;
template <int FT>
struct Geo {
  static constexpr int RW = FT + 2 * kHX, RH = FT + 2 * kHY, RN = RW * RH;
  static constexpr int CRW = FT / 2 + 7, CRH = FT / 2 + 5, CRN = CRW * CRH;
  static constexpr int rows = FT == 16 ? 256 : FTile::kRows;  // rows, columns of D a tile's threads take
  static constexpr int cols = FT == 16 ? 512 : FTile::kCols;
};

template <class T>
struct FArgs {
  const T* xin;  // null: zero
  T* xout;
  const T* b;
  const uint8_t* fl;
  int N, s;
  const FTile* tiles;
  int ntiles;
  const int* st_idx;   // stored rows of a tile: region index | colour << 11, position + 1 << 13 of a core cut vertex
  const T* st_coef;    // 10 planes per tile: the row, 1/diagonal
  // sweeps, at the core's cut vertices, by position: in float64 the residual
  // the cut sweeps start from, in float32 the values
  T* cut_out;
  // float64: D of the tiles (16-byte groups, 16-bit local columns), the
  // residual it is applied to (null: nothing pending), the values at the cut
  // vertices after the pending sweeps (written by a sweep or a restriction
  // for the core, read by the prolongation)
  const double2* D;
  const uint4* Didx;
  const double* r;
  const int* rows;     // transposed step from zero: r is b at these nodes (i | j << 16 by position)
  int reverse;         // colours 3 .. 0
  double* xs_out;
  const double* xs_in;
  // prolongation from the coarser level, and its pending residual
  const T* xc;
  int sc;
  const double* rc;
  // residual and restriction
  T* bc;
  const uint8_t* flc;
  T* xc_zero;          // coarse iterate to clear (a level smoothed by the separate kernels), or null
  const int* cutposc;
  T* snapc;
  double* part;        // per-tile (max |r|, sum r^2) of the incoming iterate, or null
  Reduce red;          // sweeps: pairs of an earlier launch that one more workgroup reduces
};

__device__ inline double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ inline float fma_t(float a, float b, float c) { return fmaf(a, b, c); }

// lanes of one wave see each other's LDS stores
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// one segment: 16 values of D and their columns, loaded (nothing is used
// before every load is issued), then summed against r in LDS in order
struct Segment {
  double2 v[8];
  uint4 c[2];
  __device__ void load(const double2* D, const uint4* idx, int base, int nseg, int sg) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = D[(int64_t)base * 8 + k * nseg + sg];
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = idx[(int64_t)base * 2 + k * nseg + sg];
  }
  __device__ double sum(const double* sr) const {
    const unsigned w[8] = {c[0].x, c[0].y, c[0].z, c[0].w, c[1].x, c[1].y, c[1].z, c[1].w};
    double x[16];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      x[2 * k] = sr[w[k] & 0xffff];
      x[2 * k + 1] = sr[w[k] >> 16];
    }
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc = fma(v[k].y, x[2 * k + 1], fma(v[k].x, x[2 * k], acc));
    return acc;
  }
};

// phase bounds of colour c inside the region (inclusive), and the number of
// its nodes: the region's origin is odd in x and y (tiles start at multiples
// of FT), so even grid columns are odd region columns
template <int FT>
struct Phase {
  __host__ __device__ static constexpr int lox(int c) { return 1 + c; }
  __host__ __device__ static constexpr int hix(int c) { return Geo<FT>::RW - 2 - c; }
  __host__ __device__ static constexpr int loy(int c) { return 1 + (c >> 1); }
  __host__ __device__ static constexpr int hiy(int c) { return Geo<FT>::RH - 2 - (c >> 1); }
  __host__ __device__ static constexpr int nx(int c) { return (hix(c) - lox(c)) / 2 + 1; }
  __host__ __device__ static constexpr int ny(int c) { return (hiy(c) - loy(c)) / 2 + 1; }
};
static_assert(kHX % 2 == 1 && kHY % 2 == 1, "the region's origin is odd");

template <class T, int RW>
__device__ inline T q1_sum(const T* su, int q) {
  return (su[q - RW - 1] + su[q - RW] + su[q - RW + 1]) + (su[q - 1] + su[q + 1]) +
         (su[q + RW - 1] + su[q + RW] + su[q + RW + 1]);
}
template <class T, int RW>
__device__ inline T row_off(const T* cf, const T* su, int q) {
  T acc = cf[0] * su[q - RW - 1];
  acc += cf[1] * su[q - RW];
  acc += cf[2] * su[q - RW + 1];
  acc += cf[3] * su[q - 1];
  acc += cf[5] * su[q + 1];
  acc += cf[6] * su[q + RW - 1];
  acc += cf[7] * su[q + RW];
  acc += cf[8] * su[q + RW + 1];
  return acc;
}

// 16 x 16 tiles up to N = 512 (256 threads each where two workgroups per CU of
// 512 threads would not hold every tile), 32 x 32 beyond
constexpr int kWideTiles = 512;
inline int tile_nodes(int N) { return N <= 512 ? 16 : 32; }

// kinds of a tile's work
constexpr int kSweepK = 0, kRestrictK = 1, kUpK = 2, kProlongK = 3;

// One tile.  The first threads take the regular rows of a phase (at most 120 of
// one colour in a 16 x 16 tile, 360 in a 32 x 32 one), the stored rows go to
// the threads of the next whole wave on, one each with its row in registers,
// so that neither waits for the other inside a wave.
template <class T, int KIND, int FT, int BS>
__device__ void fused_tile(const FArgs<T>& a, const int t) {
  using GE = Geo<FT>;
  using PH = Phase<FT>;
  constexpr int kRW = GE::RW, kRN = GE::RN, kCRW = GE::CRW, kCRN = GE::CRN;
  static_assert(BS >= GE::rows && BS >= FTile::kCRows && BS >= kCRN, "one row and one coarse node per thread");
  constexpr int NW = BS / 64, NS = (kRN + BS - 1) / BS, NC = GE::cols / BS;
  constexpr int kFree = (PH::nx(0) * PH::ny(0) + 63) / 64 * 64;  // first thread without a regular row
  static_assert(kFree < BS, "threads for the stored rows");
  __shared__ T su[kRN];
  __shared__ uint8_t sfl[kRN];
  constexpr bool kD = sizeof(T) == 8;                            // cut sweeps as a product
  constexpr bool kUp = KIND == kUpK || KIND == kProlongK;        // adds P x_c
  __shared__ double sr[kD ? GE::cols : 1];
  __shared__ double ps[kD ? FTile::kSegs : 1];
  __shared__ T sx[kUp ? kCRN : 1];
  constexpr int RR = FT + 1;  // residual region of a restriction
  constexpr int NRR = (RR * RR + BS - 1) / BS;
  static_assert(NRR <= 4, "residual nodes per thread");
  __shared__ T sres[KIND == kRestrictK ? RR * RR : 1];
  const FTile& R = a.tiles[t];
  const int x0 = R.x0, y0 = R.y0, st = R.st, nst = R.nst;
  const int ox = x0 - kHX, oy = y0 - kHY;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // the pending cut sweeps: this thread's columns, row and segment (entries
  // beyond the counts are zero: position 0, a row that is not used)
  const double* rp = KIND == kUpK ? a.rc : a.r;
  const int base = KIND == kUpK ? R.cseg : R.seg, nseg = kD && rp ? (KIND == kUpK ? R.ncseg : R.nseg) : 0;
  const int nrow = KIND == kUpK ? R.ncrow : R.nrow;
  int colp[NC];
  FRow row{0, 0, 0}, frow{0, 0, 0};
  double pv = 0.0;
  Segment sg;
  if constexpr (kD) {
    if (nseg > 0) {
#pragma unroll
      for (int u = 0; u < NC; ++u) colp[u] = KIND == kUpK ? R.ccols[tid + u * BS] : R.cols[tid + u * BS];
      row = KIND == kUpK ? R.crows[min(tid, FTile::kCRows - 1)] : R.rows[min(tid, GE::rows - 1)];
      sg.load(a.D, a.Didx, base, nseg, min(tid, nseg - 1));
    }
    if (KIND == kUpK && a.xs_in && R.nrow > 0) {
      frow = R.rows[min(tid, GE::rows - 1)];
      pv = a.xs_in[frow.pos];
    }
  }
  // loads of the region (a node off the grid loads a clamped one and drops it)
  T rx[NS];
  uint8_t rf[NS];
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int q = min(tid + u * BS, kRN - 1);
    const int gi = min(max(ox + q % kRW, 0), a.N), gj = min(max(oy + q / kRW, 0), a.N);
    const int64_t k = gi + (int64_t)gj * a.s;
    rx[u] = a.xin ? a.xin[k] : T(0);
    rf[u] = R.inner ? (uint8_t)kFlagActive : a.fl[k];
  }
  // this thread's stored row
  const int e = (tid + BS - kFree) % BS;
  int si = -1;
  T cf[10], sb = T(0);
#pragma unroll
  for (int p = 0; p < 10; ++p) cf[p] = T(0);
  if (e < nst) {
    si = a.st_idx[st + e];
#pragma unroll
    for (int p = 0; p < 10; ++p) cf[p] = a.st_coef[10 * (int64_t)st + p * nst + e];
  }
  const int sq = si >= 0 ? si & 2047 : -1, scol = (si >> 11) & 3, spos = (si >> 13) - 1;
  // regular rows: one node of each phase, or of the residual.  Phase c takes
  // colour c, in a reversed sweep colour 3 - c, whose sub-lattice starts one
  // node further in both directions
  const int rev = KIND == kSweepK && a.reverse ? 1 : 0;
  int pq[4];
  T pb[4];
  if constexpr (KIND != kRestrictK) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int nx = PH::nx(c), ny = PH::ny(c);
      const int ri = PH::lox(c) + rev + 2 * (tid % nx), rj = PH::loy(c) + rev + 2 * (tid / nx);
      const int gi = ox + ri, gj = oy + rj;
      const bool ok = tid < nx * ny && gi >= 0 && gj >= 0 && gi <= a.N && gj <= a.N;
      pq[c] = ok ? ri + rj * kRW : -1;
      pb[c] = ok ? a.b[gi + (int64_t)gj * a.s] : T(0);
    }
  } else {
#pragma unroll
    for (int u = 0; u < NRR; ++u) {
      const int q = tid + u * BS, ri = kHX - 1 + q % RR, rj = kHY - 1 + q / RR;
      const int gi = ox + ri, gj = oy + rj;
      const bool ok = q < RR * RR && gi >= 0 && gj >= 0 && gi <= a.N && gj <= a.N;
      pq[u] = ok ? ri + rj * kRW : -1;
      pb[u] = ok ? a.b[gi + (int64_t)gj * a.s] : T(0);
    }
  }
  T rc = T(0);
  if constexpr (kUp) {
    const int Nc = a.N >> 1, cx = x0 / 2 - 3, cy = y0 / 2 - 2;
    const int I = cx + tid % kCRW, J = cy + tid / kCRW;
    const bool in = tid < kCRN && I >= 0 && J >= 0 && I <= Nc && J <= Nc;
    rc = in ? a.xc[I + (int64_t)J * a.sc] : T(0);
  }
  double rv[NC];
  if constexpr (kD)
    if (nseg > 0) {
#pragma unroll
      for (int u = 0; u < NC; ++u) {
        // from a zero start the residual is the right-hand side
        const int ij = KIND == kSweepK && a.rows ? a.rows[colp[u]] : 0;
        rv[u] = KIND == kSweepK && a.rows ? (double)a.b[(ij & 0xffff) + (int64_t)(ij >> 16) * a.s] : rp[colp[u]];
      }
    }
  if (sq >= 0) sb = a.b[(ox + sq % kRW) + (int64_t)(oy + sq / kRW) * a.s];
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int q = tid + u * BS;
    const int gi = ox + q % kRW, gj = oy + q / kRW;
    const bool in = gi >= 0 && gj >= 0 && gi <= a.N && gj <= a.N;
    if (q < kRN) {
      su[q] = in ? rx[u] : T(0);
      sfl[q] = in ? rf[u] : (uint8_t)0;
    }
  }
  if constexpr (kUp)
    if (tid < kCRN) sx[tid] = rc;
  if constexpr (kD)
    if (nseg > 0) {
#pragma unroll
      for (int u = 0; u < NC; ++u) sr[tid + u * BS] = rv[u];
    }
  __syncthreads();
  if constexpr (kD) {
    if (nseg > 0) {
      if (tid < nseg) ps[tid] = sg.sum(sr);
      for (int w = tid + BS; w < nseg; w += BS) {
        sg.load(a.D, a.Didx, base, nseg, w);
        ps[w] = sg.sum(sr);
      }
      __syncthreads();
      if (tid < nrow) {
        const int s0 = row.seg & 0xffff, n = row.seg >> 16, q = row.at & 0xffff;
        double v = 0.0;
        for (int k = 0; k < n; ++k) v += ps[s0 + k];
        if constexpr (KIND == kUpK) {
          sx[q] += v;
        } else {
          v += su[q];
          su[q] = v;
          if (a.xs_out && (row.at >> 16)) a.xs_out[row.pos] = v;
        }
      }
      if constexpr (KIND != kUpK) __syncthreads();
    }
    if constexpr (KIND == kUpK) {
      if (a.xs_in && tid < R.nrow) su[frow.at & 0xffff] = pv;
      __syncthreads();
    }
  }
  if constexpr (kUp) {
    // + P x_c (for an even index both parents coincide)
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int q = tid + u * BS;
      const int gi = ox + q % kRW, gj = oy + q / kRW;
      if (q < kRN && gi >= 0 && gj >= 0 && gi <= a.N && gj <= a.N) {
        const int cx = x0 / 2 - 3, cy = y0 / 2 - 2;
        const int I0 = (gi >> 1) - cx, I1 = ((gi + 1) >> 1) - cx;
        const int J0 = ((gj >> 1) - cy) * kCRW, J1 = (((gj + 1) >> 1) - cy) * kCRW;
        su[q] += T(0.25) * ((sx[I0 + J0] + sx[I1 + J0]) + (sx[I0 + J1] + sx[I1 + J1]));
      }
    }
    __syncthreads();
  }
  // rows beyond one per thread (a region crowded with stored rows): read again where they are used
  auto extra = [&](auto&& f) {
    for (int w = e + BS; w < nst; w += BS) {
      const int s2 = a.st_idx[st + w], q2 = s2 & 2047;
      T c2[10];
#pragma unroll
      for (int p = 0; p < 10; ++p) c2[p] = a.st_coef[10 * (int64_t)st + p * nst + w];
      f(q2, (s2 >> 11) & 3, (s2 >> 13) - 1, c2, a.b[(ox + q2 % kRW) + (int64_t)(oy + q2 / kRW) * a.s]);
    }
  };
  auto in_core = [](int q) {
    const int ri = q % kRW, rj = q / kRW;
    return ri >= kHX && ri < kHX + FT && rj >= kHY && rj < kHY + FT;
  };
  if constexpr (KIND == kRestrictK) {
#pragma unroll
    for (int u = 0; u < NRR; ++u) {
      const int q = pq[u], w = tid + u * BS;
      if (w >= RR * RR) continue;
      const uint8_t f = q >= 0 ? sfl[q] : 0;
      if (!(f & kFlagActive)) sres[w] = T(0);
      else if (!(f & kFlagStored)) sres[w] = pb[u] - (T(8) / T(3) * su[q] - q1_sum<T, kRW>(su, q) * T(1.0 / 3.0));
    }
    auto put = [&](int qq, const T* c, T bv) {
      const int ri = qq % kRW - (kHX - 1), rj = qq / kRW - (kHY - 1);
      if (ri >= 0 && rj >= 0 && ri < RR && rj < RR) sres[ri + rj * RR] = bv - (c[4] * su[qq] + row_off<T, kRW>(c, su, qq));
    };
    if (sq >= 0) put(sq, cf, sb);
    extra([&](int q2, int, int, const T* c2, T b2) { put(q2, c2, b2); });
    __syncthreads();
    constexpr int CT = FT / 2;
    if (tid < CT * CT) {
      const int Nc = a.N >> 1, I = x0 / 2 + tid % CT, J = y0 / 2 + tid / CT;
      const int64_t kc = min(I, Nc) + (int64_t)min(J, Nc) * a.sc;
      const uint8_t f = (I <= Nc && J <= Nc) ? a.flc[kc] : 0;
      if (f & kFlagActive) {
        const T* r0 = sres + 2 * (tid % CT) + 1 + (2 * (tid / CT) + 1) * RR;
        const T mid = r0[0] + T(0.5) * (r0[-1] + r0[1]);
        const T lo = r0[-RR] + T(0.5) * (r0[-RR - 1] + r0[-RR + 1]);
        const T hi = r0[RR] + T(0.5) * (r0[RR - 1] + r0[RR + 1]);
        a.bc[kc] = mid + T(0.5) * (lo + hi);
        if (a.xc_zero) {
          a.xc_zero[kc] = T(0);
          if (f & kFlagCut) a.snapc[a.cutposc[kc]] = T(0);
        }
      }
    }
  } else {
    if constexpr (KIND == kSweepK && sizeof(T) == 8) {
      if (a.part) {
        __shared__ double smx[NW], ssm[NW];
        double mx = 0.0, sm = 0.0;
        auto add = [&](double r) {
          mx = nanmax2(mx, fabs(r));
          sm += r * r;
        };
        // the regular rows of the core are the phases' nodes: every core node is one of them
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int q = pq[c];
          if (q < 0 || !in_core(q)) continue;
          const uint8_t f = sfl[q];
          if ((f & kFlagActive) && !(f & kFlagStored))
            add((double)(pb[c] - (T(8) / T(3) * su[q] - q1_sum<T, kRW>(su, q) * T(1.0 / 3.0))));
        }
        if (sq >= 0 && in_core(sq)) add((double)(sb - (cf[4] * su[sq] + row_off<T, kRW>(cf, su, sq))));
        extra([&](int q2, int, int, const T* c2, T b2) {
          if (in_core(q2)) add((double)(b2 - (c2[4] * su[q2] + row_off<T, kRW>(c2, su, q2))));
        });
        for (int o = 32; o > 0; o >>= 1) {
          mx = nanmax2(mx, __shfl_xor(mx, o));
          sm += __shfl_xor(sm, o);
        }
        if (lane == 0) {
          smx[wave] = mx;
          ssm[wave] = sm;
        }
        __syncthreads();
        if (tid == 0) {
          for (int w = 1; w < NW; ++w) {
            mx = nanmax2(mx, smx[w]);
            sm += ssm[w];
          }
          a.part[2 * t] = mx;
          a.part[2 * t + 1] = sm;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint8_t f = pq[c] >= 0 ? sfl[pq[c]] : 0;
      if (!(f & kFlagActive) || (f & kFlagStored)) pq[c] = -1;
    }
    if constexpr (KIND != kProlongK)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int colour = rev ? 3 - c : c;
      // (the product is fused here as in the separate kernels, wherever the compiler puts it)
      if (pq[c] >= 0) su[pq[c]] = fma_t(T(3), pb[c], q1_sum<T, kRW>(su, pq[c])) * T(0.125);
      auto update = [&](const T* k, int qq, T bv) {
        const T v = bv - row_off<T, kRW>(k, su, qq);
        su[qq] = kD ? v * k[9] : v / k[4];
      };
      if (sq >= 0 && scol == colour) update(cf, sq, sb);
      extra([&](int q2, int c2, int, const T* k2, T b2) {
        if (c2 == colour) update(k2, q2, b2);
      });
      __syncthreads();
    }
    // what the cut sweeps start from, and the core
    if (a.cut_out) {
      auto put = [&](const T* k, int qq, int pos, T bv) {
        if (pos >= 0) a.cut_out[pos] = kD ? bv - (k[4] * su[qq] + row_off<T, kRW>(k, su, qq)) : su[qq];
      };
      if (sq >= 0) put(cf, sq, spos, sb);
      extra([&](int q2, int, int p2, const T* c2, T b2) { put(c2, q2, p2, b2); });
    }
    for (int c = tid; c < FT * FT; c += BS) {
      const int ri = kHX + c % FT, rj = kHY + c / FT;
      const int q = ri + rj * kRW;
      if (sfl[q] & kFlagActive) a.xout[(ox + ri) + (int64_t)(oy + rj) * a.s] = su[q];
    }
  }
}

// work lists are dealt to the eight XCDs in contiguous eighths (workgroups go
// to the XCDs round robin), so that neighbouring tiles, and a tile's blocks
// of D from one launch to the next, stay in one XCD's L2
__device__ inline int xcd_slot(int per) { return (blockIdx.x & 7) * per + (blockIdx.x >> 3); }

template <class T, int KIND, int FT, int BS>
__global__ __launch_bounds__(BS) void k_fused(FArgs<T> a) {
  if constexpr (KIND == kSweepK && sizeof(T) == 8) {
    if (a.red.part && blockIdx.x == gridDim.x - 1) {
      __shared__ double sh[2 * BS / 64];
      reduce_block<BS, 4>(a.red, sh);
      return;
    }
  }
  const int t = xcd_slot((a.ntiles + 7) >> 3);
  if (t >= a.ntiles) return;  // uniform, before any barrier
  fused_tile<T, KIND, FT, BS>(a, t);
}

// the pending cut sweeps of a tile's core applied to the iterate in place
// (only r and the core's own cut vertices are read)
template <int FT, int BS>
__global__ __launch_bounds__(BS) void k_fused_apply(FArgs<double> a) {
  using GE = Geo<FT>;
  static_assert(BS >= GE::rows, "one row per thread");
  __shared__ double sr[GE::cols];
  __shared__ double ps[FTile::kSegs];
  const int t = xcd_slot((a.ntiles + 7) >> 3);
  if (t >= a.ntiles) return;
  const FTile& R = a.tiles[t];
  const int tid = threadIdx.x, nseg = R.nseg;
  if (nseg == 0) return;  // uniform, before any barrier
  for (int c = tid; c < GE::cols; c += BS) sr[c] = a.r[R.cols[c]];
  const FRow row = R.rows[min(tid, GE::rows - 1)];
  __syncthreads();
  for (int w = tid; w < nseg; w += BS) {
    Segment sg;
    sg.load(a.D, a.Didx, R.seg, nseg, w);
    ps[w] = sg.sum(sr);
  }
  __syncthreads();
  if (tid < R.nrow && (row.at >> 16)) {
    const int s0 = row.seg & 0xffff, n = row.seg >> 16, q = row.at & 0xffff;
    double v = 0.0;
    for (int k = 0; k < n; ++k) v += ps[s0 + k];
    a.xout[(R.x0 - kHX + q % GE::RW) + (int64_t)(R.y0 - kHY + q / GE::RW) * a.s] += v;
  }
}

// float cycles of many problems (16 x 16 tiles): one entry per problem with
// both ping-pong buffers of its level and of the next coarser one
struct FEntry {
  FArgs<float> a;
  float* X[2];
  const float* XC[2];
  int xc_fixed;  // the coarser level's iterate comes from the coarse map: buffer 0
};

template <int KIND, int BS>
__global__ __launch_bounds__(BS) void k_fused_multi(const FEntry* tab, const int2* work, int nwork, int par, int parc,
                                                    int zero) {
  const int i = xcd_slot((nwork + 7) >> 3);
  if (i >= nwork) return;
  const int2 w = work[i];
  const FEntry& E = tab[w.x];
  FArgs<float> a = E.a;
  a.xin = zero ? nullptr : E.X[par];
  a.xout = E.X[1 - par];
  if (KIND == kUpK) a.xc = E.XC[E.xc_fixed ? 0 : parc];
  fused_tile<float, KIND, 16, BS>(a, w.y);
}

// the cut vertices of a dense array from the values by position
__global__ void k_fused_patch(const int* __restrict__ rows, int n, const double* __restrict__ xs,
                              double* __restrict__ x, int s) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) x[(rows[p] & 0xffff) + (int64_t)(rows[p] >> 16) * s] = xs[p];
}

// ---------------------------------------------------------------------------
// set-up
// ---------------------------------------------------------------------------

__global__ void k_zero_int(int* p, int n) {
  for (int q = threadIdx.x; q < n; q += blockDim.x) p[q] = 0;
}

// The set-up kernels take every fused level in one launch: each is a chain of
// dependent loads or phases that one level does not fill the chip with (the
// flower with N = 1024: 2.5 ms level by level, 1.1 ms like this).
struct SetLevel {
  const uint8_t *fl, *flc;  // flags of the level and of the coarser one
  const double* A;
  int64_t n;
  int N, nc, nt, cut;       // cells and tiles per side, cut vertices
  int coarse;               // the coarser level's place in the list, or -1
  int nblk;
  int* sums;                // four arrays over runs of 256 cells (run_sums)
  int *cnt, *pos, *bid, *npos, *rows, *bcell, *ncol, *coff, *nval, *voff, *keep, *slot, *nst, *stoff, *nseg, *segoff;
  FBlock* blocks;
  int* cols;
  double* D;
  int* tot;                 // blocks, cut vertices, columns, values, tiles, stored rows, segments;
                            // [8] columns of the largest block, [9] a record that does not fit
  const int* cutpos;
  FTile* tiles;
  int* st_idx;
  void* st_coef;
  double *fD, *fDT;
  uint16_t* fidx;
  uint8_t* inner;           // levels that stream: tiles that the windows take; else null
};
constexpr int kMaxSet = 12;
struct SetLevels {
  int n;
  SetLevel v[kMaxSet];
};
static_assert(sizeof(SetLevels) <= 3584, "kernel arguments");

__host__ __device__ inline int cell_runs(int nc) { return (nc * nc + 255) / 256; }
// 0 cut vertices, 1 cells with one per run of 256 cells; 2, 3 those before it
__device__ inline int* run_sums(const SetLevel& L, int k) { return L.sums + k * (cell_runs(L.nc) + 1); }

// Cut vertices per cell, their number and that of the cells with one over the
// block's 256 cells (sums of a block fit in 16 bits).
__global__ __launch_bounds__(256) void k_cell_count(SetLevels S) {
  const SetLevel& L = S.v[blockIdx.y];
  const int N = L.N, nc = L.nc;
  const uint8_t* __restrict__ fl = L.fl;
  if (L.cut == 0 || blockIdx.x * 256 >= nc * nc) return;
  const int c = blockIdx.x * 256 + threadIdx.x;
  int n = 0;
  if (c < nc * nc) {
    const int i0 = (c % nc) * kCell, j0 = (c / nc) * kCell;
    for (int q = 0; q < kCell * kCell; ++q) {
      const int i = i0 + q % kCell, j = j0 + q / kCell;
      if (i <= N && j <= N && (fl[i + (int64_t)j * (N + 1)] & kFlagCut)) ++n;
    }
    L.cnt[c] = n;
  }
  __shared__ int wsum[4];
  int x = n | (n != 0) << 16;
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    x = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    run_sums(L, 0)[blockIdx.x] = x & 0xffff;
    run_sums(L, 1)[blockIdx.x] = x >> 16;
  }
}

// exclusive prefix sum over n values by one workgroup of 1024 threads, in runs
// of eight values per thread: out[0..n], the total in *tot too
__device__ void wg_scan(const int* in, int n, int* out, int* tot) {
  constexpr int U = 8;
  __shared__ int wa[16];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  int ca = 0;  // sum of the runs before
  for (int base = 0; base < n; base += 1024 * U) {
    const int q0 = base + t * U;
    int v[U], a = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = in[min(q0 + u, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (q0 + u >= n) v[u] = 0;
      a += v[u];
    }
    int xa = a;  // inclusive over the wave
    for (int o = 1; o < 64; o <<= 1) {
      const int ya = __shfl_up(xa, o);
      if (lane >= o) xa += ya;
    }
    if (lane == 63) wa[wave] = xa;
    __syncthreads();
    xa += ca - a;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) xa += wa[w];
      ca += wa[w];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (q0 + u < n) {
        out[q0 + u] = xa;
        xa += v[u];
      }
    __syncthreads();
  }
  if (t == 0) {
    out[n] = ca;
    *tot = ca;
  }
}
// Positions and blocks in three steps: sums per 256 cells, their scan, the scan
// within 256 cells where they are used.  (One workgroup over all cells: 1.4 ms at
// N = 4096, 22.7 at 16384.  Set-up of the flower: N = 4096 8.1 ms, like this 6.7;
// N = 2048 4.1, 3.75; both without the plans of the separate kernels.)
__global__ __launch_bounds__(1024) void k_scan_cells(SetLevels S) {
  const SetLevel& L = S.v[blockIdx.x];
  const int k = blockIdx.y;
  if (L.cut > 0) wg_scan(run_sums(L, k), cell_runs(L.nc), run_sums(L, 2 + k), L.tot + 1 - k);
}
__global__ __launch_bounds__(1024) void k_scan_blocks(SetLevels S) {
  const SetLevel& L = S.v[blockIdx.x];
  if (L.nblk > 0)
    wg_scan(blockIdx.y ? L.nval : L.ncol, L.nblk, blockIdx.y ? L.voff : L.coff, L.tot + 2 + blockIdx.y);
}
__global__ __launch_bounds__(1024) void k_scan_tiles(SetLevels S) {
  const SetLevel& L = S.v[blockIdx.x];
  const int k = blockIdx.y;
  wg_scan(k == 0 ? L.keep : k == 1 ? L.nst : L.nseg, L.nt * L.nt, k == 0 ? L.slot : k == 1 ? L.stoff : L.segoff,
          L.tot + 4 + k);
}

// rows by position, positions by node, and the cell of every block
__global__ __launch_bounds__(256) void k_cell_fill(SetLevels S) {
  const SetLevel& L = S.v[blockIdx.y];
  const int N = L.N, nc = L.nc;
  const uint8_t* __restrict__ fl = L.fl;
  int *__restrict__ rows = L.rows, *__restrict__ npos = L.npos, *__restrict__ bcell = L.bcell;
  if (L.cut == 0 || blockIdx.x * 256 >= nc * nc) return;
  const int c = blockIdx.x * 256 + threadIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int v = c < nc * nc ? L.cnt[c] : 0, own = v | (v != 0) << 16;
  __shared__ int wsum[4];
  int x = own;  // inclusive over the wave
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  x -= own;
  for (int w = 0; w < wave; ++w) x += wsum[w];
  int p = run_sums(L, 2)[blockIdx.x] + (x & 0xffff);
  const int b = run_sums(L, 3)[blockIdx.x] + (x >> 16);
  if (c >= nc * nc) return;
  L.pos[c] = p;
  L.bid[c] = v != 0 ? b : -1;
  if (c == nc * nc - 1) {
    L.pos[c + 1] = p + v;
    L.bid[c + 1] = b + (v != 0);
  }
  if (v == 0) return;
  bcell[b] = c;
  const int i0 = (c % nc) * kCell, j0 = (c / nc) * kCell;
  for (int q = 0; q < kCell * kCell; ++q) {
    const int i = i0 + q % kCell, j = j0 + q / kCell;
    if (i > N || j > N) continue;
    const int64_t k = i + (int64_t)j * (N + 1);
    if (!(fl[k] & kFlagCut)) continue;
    rows[p] = i | j << 16;
    npos[k] = p++;
  }
}

// columns of every block: the cut vertices of the cells its rows can reach
// (one contiguous run of positions per row of cells), their number and the
// values of its D
__device__ inline int cell_reach_y(int eta) { return (2 * eta + kCell - 1) / kCell; }
__global__ void k_block_size(SetLevels S, int eta) {
  const SetLevel& L = S.v[blockIdx.y];
  const int *__restrict__ bcell = L.bcell, *__restrict__ pos = L.pos;
  int *__restrict__ ncol = L.ncol, *__restrict__ nval = L.nval, *__restrict__ mx = L.tot + 8;
  const int nc = L.nc, b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= L.nblk) return;
  const int c = bcell[b], cx = c % nc, cy = c / nc, ry = cell_reach_y(eta);
  int n = 0;
  for (int y = max(0, cy - ry); y <= min(nc - 1, cy + ry); ++y)
    n += pos[min(nc - 1, cx + eta) + y * nc + 1] - pos[max(0, cx - eta) + y * nc];
  ncol[b] = n;
  nval[b] = n * (pos[c + 1] - pos[c]);
  atomicMax(mx, n);
}

__global__ void k_block_fill(SetLevels S, int eta) {
  const SetLevel& L = S.v[blockIdx.y];
  const int *__restrict__ bcell = L.bcell, *__restrict__ pos = L.pos, *__restrict__ coff = L.coff,
            *__restrict__ voff = L.voff;
  int* __restrict__ cols = L.cols;
  FBlock* __restrict__ blocks = L.blocks;
  const int nc = L.nc, b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= L.nblk || !cols) return;
  const int c = bcell[b], cx = c % nc, cy = c / nc, ry = cell_reach_y(eta);
  int w = coff[b];
  for (int y = max(0, cy - ry); y <= min(nc - 1, cy + ry); ++y)
    for (int p = pos[max(0, cx - eta) + y * nc]; p < pos[min(nc - 1, cx + eta) + y * nc + 1]; ++p) cols[w++] = p;
  blocks[b] = FBlock{voff[b], pos[c], coff[b], (pos[c + 1] - pos[c]) | (w - coff[b]) << 8};
}

// The rows of one block's D, one workgroup, one row at a time per wave: row p
// is the derivative of the swept value at p with respect to the residual, so
// the eta sweeps run backwards over adjoint values w, from w = e_p.  Undoing
// the update of colour c, x_i = (r_i - sum a_ij x_j) / a_ii, takes
// t_i = w_i / a_ii for the nodes of colour c, adds t_i to D[p][i], clears w_i
// and subtracts a_ij t_i from w_j (A is symmetric: gathered by j from its own
// row).  The waves never wait for one another after the staging.
constexpr int kMaxBlockCols = 512, kBuildWaves = 8;
__global__ __launch_bounds__(64 * kBuildWaves) void k_delta_build(SetLevels S, int eta) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SetLevel& L = S.v[blockIdx.y];
  if ((int)blockIdx.x >= L.nblk || !L.D) return;
  const int *__restrict__ cols = L.cols, *__restrict__ rows = L.rows, *__restrict__ npos = L.npos;
  const uint8_t* __restrict__ fl = L.fl;
  const double* __restrict__ A = L.A;
  double* __restrict__ D = L.D;
  const int64_t n = L.n;
  const int N = L.N;
  const FBlock B = L.blocks[blockIdx.x];
  const int nr = B.n & 0xff, nc = B.n >> 8;
  double* sA = reinterpret_cast<double*>(smem);  // 9 planes of nc: the row, 1/diagonal in plane 4
  double* sw = sA + 9 * nc;                      // one vector of nc per wave
  int* scol = reinterpret_cast<int*>(sw + kBuildWaves * nc);
  int16_t* nbr = reinterpret_cast<int16_t*>(scol + nc);  // 8 planes, -1: none
  uint8_t* col = reinterpret_cast<uint8_t*>(nbr + 8 * nc);
  const int s = N + 1;
  for (int c = threadIdx.x; c < nc; c += blockDim.x) scol[c] = cols[B.col + c];
  __syncthreads();
  // a neighbour's column, by its position (the columns ascend)
  auto find = [&](int p) {
    int lo = 0, hi = nc - 1;
    while (lo <= hi) {
      const int m = (lo + hi) >> 1, v = scol[m];
      if (v == p) return m;
      if (v < p) lo = m + 1;
      else hi = m - 1;
    }
    return -1;
  };
  for (int c = threadIdx.x; c < nc; c += blockDim.x) {
    const int ij = rows[scol[c]], i = ij & 0xffff, j = ij >> 16;
    const int64_t k = i + (int64_t)j * s;
    col[c] = (uint8_t)((i & 1) + 2 * (j & 1));
    for (int p = 0; p < 9; ++p) {
      const double v = A[p * n + k];
      sA[p * nc + c] = p == 4 ? 1.0 / v : v;
      if (p == 4) continue;
      const int ii = i + p % 3 - 1, jj = j + p / 3 - 1;
      int16_t m = -1;
      if (ii >= 0 && jj >= 0 && ii <= N && jj <= N) {
        const int64_t kk = ii + (int64_t)jj * s;
        if (fl[kk] & kFlagCut) m = (int16_t)find(npos[kk]);
      }
      nbr[(p > 4 ? p - 1 : p) * nc + c] = m;
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* w = sw + wave * nc;
  for (int r = wave; r < nr; r += kBuildWaves) {
    double* out = D + B.d + r * nc;
    double d[kMaxBlockCols / 64];
    for (int u = 0; u < kMaxBlockCols / 64; ++u) d[u] = 0.0;
    for (int c = lane; c < nc; c += 64) w[c] = scol[c] == B.row + r ? 1.0 : 0.0;
    wave_sync();
    for (int sweep = 0; sweep < eta; ++sweep)
      for (int cc = 3; cc >= 0; --cc) {
#pragma unroll
        for (int u = 0; u < kMaxBlockCols / 64; ++u) {
          const int c = lane + 64 * u;
          if (c < nc && col[c] == cc) {
            const double tv = w[c] * sA[4 * nc + c];
            d[u] += tv;
            w[c] = tv;  // t for the gather below, cleared after it
          }
        }
        wave_sync();
        for (int c = lane; c < nc; c += 64) {
          if (col[c] == cc) continue;
          double v = w[c];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int h = nbr[e * nc + c];
            if (h >= 0 && col[h] == cc) v -= sA[(e >= 4 ? e + 1 : e) * nc + c] * w[h];
          }
          w[c] = v;
        }
        wave_sync();
        for (int c = lane; c < nc; c += 64)
          if (col[c] == cc) w[c] = 0.0;
        wave_sync();
      }
#pragma unroll
    for (int u = 0; u < kMaxBlockCols / 64; ++u) {
      const int c = lane + 64 * u;
      if (c < nc) out[c] = d[u];
    }
  }
}
inline int build_lds(int nc) { return 8 * nc * (9 + kBuildWaves) + 4 * nc + 16 * nc + ((nc + 15) & ~15); }

// region nodes whose stored rows a tile keeps: all but the outer ring (a sweep
// also updates those outside their colour's phase bounds, from values that are
// not exact there; no node inside the bounds reads them afterwards, in either
// direction)
template <int FT>
__device__ inline bool in_region(int ri, int rj) {
  return ri >= 1 && rj >= 1 && ri < Geo<FT>::RW - 1 && rj < Geo<FT>::RH - 1;
}

// One level as the tile plan sees it: flags, cut-vertex positions (null: no
// cut vertex), the blocks of D
struct PlanLevel {
  const uint8_t* fl;
  int N;
  const int* npos;
  const int* bid;
  int ncell;
  const FBlock* blocks;
  const int* cols;
  const int* rows;
  const double* D;
};

__device__ inline PlanLevel plan_view(const SetLevel& L) {
  return PlanLevel{L.fl, L.N, L.nblk > 0 ? L.npos : nullptr, L.bid, L.nc, L.blocks, L.cols, L.rows, L.D};
}
__device__ inline PlanLevel coarse_view(const SetLevels& S, const SetLevel& L) {
  if (L.coarse >= 0 && S.v[L.coarse].nblk > 0) return plan_view(S.v[L.coarse]);
  PlanLevel P{};
  P.fl = L.flc;
  P.N = L.N >> 1;
  return P;
}

// The rows and columns a box of a tile needs, in LDS: the cut vertices of the
// W x H box at (x, y) are its rows, those within reach of it its columns.
constexpr int kMaxReachX = 16, kMaxReachY = 8;
constexpr int kBoxW = Geo<32>::RW + 2 * kMaxReachX, kBoxH = Geo<32>::RH + 2 * kMaxReachY;
struct BoxPlan {
  int16_t local[kBoxW * kBoxH];  // node of the grown box: column, -1 none
  int16_t row[Geo<32>::RN];              // box index of row e
  int16_t len[Geo<32>::RN];              // columns of row e
  int nrow, ncol, nseg;
};
// W x H box of level P at (x, y), reach (ex, ey); all threads of the block
__device__ void plan_box(const PlanLevel& P, int x, int y, int W, int H, int ex, int ey, BoxPlan& B) {
  const int GW = W + 2 * ex, GH = H + 2 * ey, s = P.N + 1;
  for (int q = threadIdx.x; q < GW * GH; q += blockDim.x) {
    const int gi = x - ex + q % GW, gj = y - ey + q / GW;
    const bool in = P.npos && gi >= 0 && gj >= 0 && gi <= P.N && gj <= P.N;
    B.local[q] = in && (P.fl[gi + (int64_t)gj * s] & kFlagCut) ? 0 : -1;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int n = 0;
    for (int q0 = 0; q0 < GW * GH; q0 += 64) {
      const int q = q0 + threadIdx.x;
      const bool on = q < GW * GH && B.local[q] == 0;
      const unsigned long long m = __ballot(on);
      if (on) B.local[q] = (int16_t)(n + __popcll(m & ((1ull << threadIdx.x) - 1)));
      n += __popcll(m);
    }
    if (threadIdx.x == 0) B.ncol = n;
  } else if (threadIdx.x < 128) {
    const int lane = threadIdx.x - 64;
    int n = 0;
    for (int q0 = 0; q0 < W * H; q0 += 64) {
      const int q = q0 + lane;
      const bool on = q < W * H && B.local[(ex + q % W) + (ey + q / W) * GW] >= 0;
      const unsigned long long m = __ballot(on);
      if (on) B.row[n + __popcll(m & ((1ull << lane) - 1))] = (int16_t)q;
      n += __popcll(m);
    }
    if (lane == 0) B.nrow = n;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < B.nrow; e += blockDim.x) {
    const int q = B.row[e], bi = q % W, bj = q / W;  // the row's reach in the grown box starts here
    int n = 0;
    for (int v = 0; v <= 2 * ey; ++v)
      for (int u = 0; u <= 2 * ex; ++u) n += B.local[(bi + u) + (bj + v) * GW] >= 0;
    B.len[e] = (int16_t)n;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int n = 0;
    for (int e = threadIdx.x; e < B.nrow; e += 64) n += (B.len[e] + 15) / 16;
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if (threadIdx.x == 0) B.nseg = n;
  }
  __syncthreads();
}

// tiles: kept when the core holds an active node, or its coarse nodes one;
// the stored rows of the region, the segments of D, and the
// largest counts a record has to hold
template <int FT>
__global__ __launch_bounds__(256) void k_ftile_count(SetLevels S, int first, int eta) {
  const SetLevel& L = S.v[first + blockIdx.y];
  const int nt = L.nt;
  if ((int)blockIdx.x >= nt * nt) return;
  const PlanLevel P = plan_view(L), C = coarse_view(S, L);
  int *__restrict__ keep = L.keep, *__restrict__ nst = L.nst, *__restrict__ nseg = L.nseg, *__restrict__ over = L.tot + 9;
  using GE = Geo<FT>;
  constexpr int kRW = GE::RW, kRH = GE::RH, kRN = GE::RN, kCRW = GE::CRW, kCRH = GE::CRH;
  __shared__ int cnt;
  __shared__ BoxPlan B;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  const int x0 = (blockIdx.x % nt) * FT, y0 = (blockIdx.x / nt) * FT, N = P.N, s = N + 1;
  int act = 0;
  for (int q = threadIdx.x; q < kRN; q += blockDim.x) {
    const int ri = q % kRW, rj = q / kRW, gi = x0 - kHX + ri, gj = y0 - kHY + rj;
    if (gi < 0 || gj < 0 || gi > N || gj > N) continue;
    const uint8_t f = P.fl[gi + (int64_t)gj * s];
    if (!(f & kFlagActive)) continue;
    if (ri >= kHX && ri < kHX + FT && rj >= kHY && rj < kHY + FT) act = 1;
    if ((f & kFlagStored) && in_region<FT>(ri, rj)) atomicAdd(&cnt, 1);
  }
  const int Nc = N >> 1;
  for (int q = threadIdx.x; q < FT * FT / 4; q += blockDim.x) {
    const int I = x0 / 2 + q % (FT / 2), J = y0 / 2 + q / (FT / 2);
    if (I <= Nc && J <= Nc && (C.fl[I + (int64_t)J * (Nc + 1)] & kFlagActive)) act = 1;
  }
  act = __syncthreads_or(act);
  int take = act;
  if (act && L.inner) {
    // a window's reach around the tile: active nodes with the interior row, no
    // cut vertex on this level or among their parents
    constexpr int WX = kStreamHX, WY = kStreamHY, WW = FT + 2 * WX, WH = FT + 2 * WY;
    int bad = 0;
    for (int q = threadIdx.x; q < WW * WH && !bad; q += blockDim.x) {
      const int i = x0 - WX + q % WW, j = y0 - WY + q / WW;
      if (i < 0 || j < 0 || i > N || j > N) {
        bad = 1;
        continue;
      }
      bad = (P.fl[i + (int64_t)j * s] & (kFlagActive | kFlagStored | kFlagCut)) != kFlagActive;
      if (!(i & 1) && !(j & 1)) bad |= (C.fl[(i >> 1) + (int64_t)(j >> 1) * (Nc + 1)] & kFlagCut) != 0;
    }
    take = __syncthreads_or(bad);
    if (threadIdx.x == 0) L.inner[blockIdx.x] = !take;
  }
  if (!take) {
    if (threadIdx.x == 0) keep[blockIdx.x] = nst[blockIdx.x] = nseg[blockIdx.x] = 0;
    return;
  }
  plan_box(P, x0 - kHX, y0 - kHY, kRW, kRH, 4 * eta, 2 * eta, B);
  const int n1 = B.nseg;
  const bool o1 = B.nrow > GE::rows || B.ncol > GE::cols || B.nseg > FTile::kSegs;
  __syncthreads();
  plan_box(C, x0 / 2 - 3, y0 / 2 - 2, kCRW, kCRH, 4 * eta, 2 * eta, B);
  if (threadIdx.x == 0) {
    keep[blockIdx.x] = 1;
    nst[blockIdx.x] = cnt;
    nseg[blockIdx.x] = n1 + B.nseg;
    if (o1 || B.nrow > FTile::kCRows || B.ncol > GE::cols || B.nseg > FTile::kSegs) atomicMax(over, 1);
  }
}

// rows, columns and segments of one box into a tile's record
__device__ void fill_box(const PlanLevel& P, int x, int y, int W, int H, int ex, int ey, BoxPlan& B, int base,
                         int core_lo_x, int core_lo_y, int core, int* cols, FRow* rows, double* D, double* DT, uint16_t* idx) {
  const int GW = W + 2 * ex, GH = H + 2 * ey, s = P.N + 1;
  for (int q = threadIdx.x; q < GW * GH; q += blockDim.x)
    if (B.local[q] >= 0) cols[B.local[q]] = P.npos[(x - ex + q % GW) + (int64_t)(y - ey + q / GW) * s];
  if (threadIdx.x < 64) {
    int n = 0;
    for (int e0 = 0; e0 < B.nrow; e0 += 64) {
      const int e = e0 + threadIdx.x;
      const int ns = e < B.nrow ? (B.len[e] + 15) / 16 : 0;
      int up = ns;
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(up, o);
        if ((int)threadIdx.x >= o) up += v;
      }
      const int at = n + up - ns;
      n += __shfl(up, 63);
      if (e < B.nrow) {
        const int q = B.row[e], ri = q % W, rj = q / W;
        const bool in = ri >= core_lo_x && ri < core_lo_x + core && rj >= core_lo_y && rj < core_lo_y + core;
        rows[e].at = q | (int)in << 16;
        rows[e].seg = at | ns << 16;
        rows[e].pos = P.npos[(x + ri) + (int64_t)(y + rj) * s];
        B.len[e] = (int16_t)at;  // now the row's first segment
      }
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nseg = B.nseg;
  double* Db = D + (int64_t)base * 16;
  double* Tb = DT ? DT + (int64_t)base * 16 : nullptr;
  uint16_t* ib = idx + (int64_t)base * 16;
  auto put = [&](int sg, int k, double v, double vt, int c) {
    const int64_t w = ((int64_t)(k / 2) * nseg + sg) * 2 + k % 2;
    Db[w] = v;
    if (Tb) Tb[w] = vt;
    ib[((int64_t)(k / 8) * nseg + sg) * 8 + k % 8] = (uint16_t)c;
  };
  for (int e = wave; e < B.nrow; e += (int)blockDim.x / 64) {
    const int q = B.row[e], gi = x + q % W, gj = y + q / W;
    const FBlock K = P.blocks[P.bid[gi / kCell + (gj / kCell) * P.ncell]];
    const int nc = K.n >> 8, s0 = B.len[e];
    const int p = P.npos[gi + (int64_t)gj * s] - K.row;
    int n = 0;
    for (int c0 = 0; c0 < nc; c0 += 64) {
      const int c = c0 + lane;
      int l = -1;
      if (c < nc) {
        const int ij = P.rows[P.cols[K.col + c]], di = (ij & 0xffff) - gi, dj = (ij >> 16) - gj;
        if (abs(di) <= ex && abs(dj) <= ey) l = B.local[(gi + di - x + ex) + (gj + dj - y + ey) * GW];
      }
      const unsigned long long m = __ballot(l >= 0);
      if (l >= 0) {
        const int w = n + __popcll(m & ((1ull << lane) - 1));
        double vt = 0.0;
        if (Tb) {
          // the transposed step's D is the transpose: this row's column in the other node's row
          const int pc = P.cols[K.col + c], ij = P.rows[pc];
          const FBlock Q = P.blocks[P.bid[(ij & 0xffff) / kCell + ((ij >> 16) / kCell) * P.ncell]];
          int lo = 0, hi = (Q.n >> 8) - 1;
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (P.cols[Q.col + mid] < K.row + p) lo = mid + 1;
            else hi = mid;
          }
          if (P.cols[Q.col + lo] == K.row + p) vt = P.D[Q.d + (int64_t)(pc - Q.row) * (Q.n >> 8) + lo];
        }
        put(s0 + w / 16, w % 16, P.D[K.d + (int64_t)p * nc + c], vt, l);
      }
      n += __popcll(m);
    }
    const int full = (n + 15) / 16 * 16;
    if (n + lane < full) put(s0 + (n + lane) / 16, (n + lane) % 16, 0.0, 0.0, 0);
  }
  __syncthreads();
}

// one workgroup per tile: stored rows in region order, then the rows, columns
// and segments of its D on this level and of the coarser one under it
// (1024 threads: a row's values cost a few dependent loads and a search, and
// there are up to 300 rows)
template <class T, int FT>
__global__ __launch_bounds__(1024) void k_ftile_fill(SetLevels S, int first, int eta) {
  const SetLevel& L = S.v[first + blockIdx.y];
  const int nt = L.nt;
  if ((int)blockIdx.x >= nt * nt || !L.tiles) return;
  const PlanLevel P = plan_view(L), C = coarse_view(S, L);
  const double* __restrict__ A = L.A;
  const int64_t n = L.n;
  const int *__restrict__ keep = L.keep, *__restrict__ slot = L.slot, *__restrict__ stoff = L.stoff,
            *__restrict__ nstp = L.nst, *__restrict__ segoff = L.segoff, *__restrict__ cutpos = L.cutpos;
  FTile* __restrict__ tiles = L.tiles;
  int* __restrict__ st_idx = L.st_idx;
  T* __restrict__ st_coef = static_cast<T*>(L.st_coef);
  double *__restrict__ D = L.fD, *__restrict__ DT = L.fDT;
  uint16_t* __restrict__ idx = L.fidx;
  using GE = Geo<FT>;
  constexpr int kRW = GE::RW, kRH = GE::RH, kRN = GE::RN, kCRW = GE::CRW, kCRH = GE::CRH;
  __shared__ BoxPlan B;
  if (!keep[blockIdx.x]) return;
  const int N = P.N, x0 = (blockIdx.x % nt) * FT, y0 = (blockIdx.x / nt) * FT, s = N + 1;
  FTile* R = tiles + slot[blockIdx.x];
  const int off = stoff[blockIdx.x], cnt = nstp[blockIdx.x];
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int w = 0;
    bool inner = true;
    for (int q0 = 0; q0 < kRN; q0 += 64) {
      const int q = q0 + lane, ri = q % kRW, rj = q / kRW, gi = x0 - kHX + ri, gj = y0 - kHY + rj;
      bool on = q < kRN && gi >= 0 && gj >= 0 && gi <= N && gj <= N;
      const int64_t k = on ? gi + (int64_t)gj * s : 0;
      const uint8_t f = on ? P.fl[k] : 0;
      inner = inner && (q >= kRN || ((f & kFlagActive) && !(f & kFlagStored)));
      const int c = (gi & 1) + 2 * (gj & 1);
      on = on && (f & kFlagActive) && (f & kFlagStored) && in_region<FT>(ri, rj);
      const unsigned long long m = __ballot(on);
      if (on) {
        const int e = w + __popcll(m & ((1ull << lane) - 1));
        const bool core = ri >= kHX && ri < kHX + FT && rj >= kHY && rj < kHY + FT;
        const int* np = D ? P.npos : cutpos;
        const int pos = core && np && (f & kFlagCut) ? np[k] : -1;
        st_idx[off + e] = q | c << 11 | (pos + 1) << 13;
        for (int p = 0; p < 9; ++p) st_coef[10 * (int64_t)off + p * cnt + e] = (T)A[p * n + k];
        st_coef[10 * (int64_t)off + 9 * cnt + e] = T(1) / (T)A[4 * n + k];
      }
      w += __popcll(m);
    }
    inner = __all(inner);
    if (lane == 0) R->inner = inner;
  }
  if (threadIdx.x == 0) {
    R->x0 = x0;
    R->y0 = y0;
    R->st = off;
    R->nst = cnt;
  }
  if (!D) return;  // float32
  plan_box(P, x0 - kHX, y0 - kHY, kRW, kRH, 4 * eta, 2 * eta, B);
  const int base = segoff[blockIdx.x], nseg = B.nseg;
  if (threadIdx.x == 0) {
    R->seg = base;
    R->nseg = nseg;
    R->nrow = B.nrow;
  }
  fill_box(P, x0 - kHX, y0 - kHY, kRW, kRH, 4 * eta, 2 * eta, B, base, kHX, kHY, FT, R->cols, R->rows, D, DT,
           idx);
  plan_box(C, x0 / 2 - 3, y0 / 2 - 2, kCRW, kCRH, 4 * eta, 2 * eta, B);
  if (threadIdx.x == 0) {
    R->cseg = base + nseg;
    R->ncseg = B.nseg;
    R->ncrow = B.nrow;
  }
  fill_box(C, x0 / 2 - 3, y0 / 2 - 2, kCRW, kCRH, 4 * eta, 2 * eta, B, base + nseg, 0, 0, 0, R->ccols, R->crows, D,
           nullptr, idx);
}

inline unsigned nblk(int64_t n, int tb) { return (unsigned)((n + tb - 1) / tb); }

// typed views of a level
template <class T>
struct Of;
template <>
struct Of<double> {
  static double* X(Level& L, int w) { return L.X[w]; }
  static double* B(Level& L) { return L.b; }
  static double* snap(Level& L) { return L.snap; }
};
template <>
struct Of<float> {
  static float* X(Level& L, int w) { return L.X32[w]; }
  static float* B(Level& L) { return L.b32; }
  static float* snap(Level& L) { return L.snap32; }
};

template <class T>
FArgs<T> fargs(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  FusedPlan& F = L.fp;
  FArgs<T> a{};
  a.b = Of<T>::B(L);
  a.fl = L.flags;
  a.N = L.N;
  a.s = L.stride;
  a.tiles = F.tiles;
  a.ntiles = F.ntiles;
  a.st_idx = F.st_idx;
  a.st_coef = static_cast<const T*>(F.st_coef);
  a.D = F.D;
  a.Didx = F.Didx;
  Level& C = c->lv[l + 1];
  a.sc = C.stride;
  a.flc = C.flags;
  a.bc = Of<T>::B(C);
  return a;
}

template <class T, int KIND>
void launch_tiles(const FArgs<T>& a, hipStream_t st) {
  const dim3 grid(8u * (unsigned)((a.ntiles + 7) / 8) + (a.red.part ? 1 : 0));
  if (tile_nodes(a.N) == 32) hipLaunchKernelGGL((k_fused<T, KIND, 32, 512>), grid, dim3(512), 0, st, a);
  else if (a.ntiles > kWideTiles) hipLaunchKernelGGL((k_fused<T, KIND, 16, 256>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((k_fused<T, KIND, 16, 512>), grid, dim3(512), 0, st, a);
}

template <class T>
void launch_sweep(mgfem_ctx* c, int l, bool norm, bool up, const Reduce* red) {
  Level& L = c->lv[l];
  FusedPlan& F = L.fp;
  FArgs<T> a = fargs<T>(c, l);
  a.xin = L.zero ? nullptr : Of<T>::X(L, L.cur);
  const int to = L.next();
  a.xout = Of<T>::X(L, to);
  if (red) a.red = *red;
  if (up) a.xc = Of<T>::X(c->lv[l + 1], c->lv[l + 1].cur);
  if constexpr (sizeof(T) == 4) {
    a.cut_out = L.snap32;
  } else {
    if (F.ncut > 0) a.cut_out = F.r[to];
    if (up) {
      const Level& C = c->lv[l + 1];
      if (L.pend) a.xs_in = F.xs;
      if (C.pend) a.rc = C.fp.r[C.cur];
    } else if (L.pend) {
      a.r = F.r[L.cur];
      if (norm) a.xs_out = F.xs;
    }
    if (norm) a.part = c->sweep_part + (L.sp.fused ? 2 * L.sp.nwin : 0);
    L.pend = F.ncut > 0;
  }
  auto go = [a, up](hipStream_t st) {
    if (up) launch_tiles<T, kUpK>(a, st);
    else launch_tiles<T, kSweepK>(a, st);
  };
  if (c->prof.on && l == 0 && !L.sp.fused) {
    constexpr double vb = (double)sizeof(T);
    double bytes = 3.0 * vb * L.n_active + 9.0 * vb * L.n_stored;
    if (up) bytes += vb * c->lv[l + 1].n_active;
    prof_launch(c, sizeof(T) == 8 ? 0 : 1, bytes, go);
  } else {
    go(c->s);
  }
  L.cur = to;
  L.zero = false;
}

// transposed cycles (float64): the cut sweeps come first in a step, so a step
// applies them to the residual the sweep or prolongation before it left, and
// nothing is pending behind it (L.pend: that residual exists; else the
// iterate is zero)
void launch_reverse_sweep(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  FusedPlan& F = L.fp;
  FArgs<double> a = fargs<double>(c, l);
  a.xin = L.zero ? nullptr : L.X[L.cur];
  a.xout = L.X[1 - L.cur];
  a.reverse = 1;
  if (F.ncut > 0) {
    a.D = F.DT;
    a.r = F.r[L.cur];
    a.rows = L.pend ? nullptr : F.rows;
    a.cut_out = F.r[1 - L.cur];
  }
  launch_tiles<double, kSweepK>(a, c->s);
  L.cur = 1 - L.cur;
  L.pend = F.ncut > 0;
  L.zero = false;
}
void launch_prolong(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  FusedPlan& F = L.fp;
  FArgs<double> a = fargs<double>(c, l);
  a.xin = L.X[L.cur];
  a.xout = L.X[1 - L.cur];
  a.xc = c->lv[l + 1].X[c->lv[l + 1].cur];
  if (F.ncut > 0) a.cut_out = F.r[1 - L.cur];
  launch_tiles<double, kProlongK>(a, c->s);
  L.cur = 1 - L.cur;
  L.pend = F.ncut > 0;
}

template <class T>
void launch_rr(mgfem_ctx* c, int l, bool clear_coarse, bool reverse) {
  Level& L = c->lv[l];
  Level& C = c->lv[l + 1];
  FArgs<T> a = fargs<T>(c, l);
  a.xin = L.zero ? nullptr : Of<T>::X(L, L.cur);
  if (L.pend && !reverse) {
    a.r = L.fp.r[L.cur];
    a.xs_out = L.fp.xs;
  }
  if (clear_coarse) {
    a.xc_zero = Of<T>::X(C, C.cur);
    a.cutposc = C.cutpos;
    a.snapc = Of<T>::snap(C);
  }
  launch_tiles<T, kRestrictK>(a, c->s);
}

}  // namespace

void fused_sweep(mgfem_ctx* c, int l, bool fp32, bool norm, bool up, const Reduce* red) {
  if (fp32) launch_sweep<float>(c, l, norm, up, nullptr);
  else launch_sweep<double>(c, l, norm, up, red);
}
void fused_restrict(mgfem_ctx* c, int l, bool fp32, bool clear_coarse, bool reverse) {
  if (fp32) launch_rr<float>(c, l, clear_coarse, false);
  else launch_rr<double>(c, l, clear_coarse, reverse);
}
void fused_reverse_sweep(mgfem_ctx* c, int l) { launch_reverse_sweep(c, l); }
void fused_prolong(mgfem_ctx* c, int l) { launch_prolong(c, l); }
void fused_apply(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  FusedPlan& F = L.fp;
  if (!L.pend) return;
  FArgs<double> a = fargs<double>(c, l);
  a.xout = L.X[L.cur];
  a.r = F.r[L.cur];
  const dim3 grid(8u * (unsigned)((F.ntiles + 7) / 8));
  if (tile_nodes(L.N) == 32) hipLaunchKernelGGL((k_fused_apply<32, 512>), grid, dim3(512), 0, c->s, a);
  else hipLaunchKernelGGL((k_fused_apply<16, 256>), grid, dim3(256), 0, c->s, a);
  L.pend = false;
}
void fused_patch(mgfem_ctx* c, double* x) {
  const Level& L = c->lv[0];
  hipLaunchKernelGGL(k_fused_patch, dim3(nblk(L.fp.ncut, 256)), dim3(256), 0, c->s, (const int*)L.fp.rows, L.fp.ncut,
                     (const double*)L.fp.xs, x, L.stride);
}

// ---- batched solves (float cycles): entries, units and launches
size_t fused_entry_bytes() { return sizeof(FEntry); }
void fused_entry(mgfem_ctx* m, int l, void* out) {
  Level& L = m->lv[l];
  Level& C = m->lv[l + 1];
  FEntry e{};
  e.a = fargs<float>(m, l);
  e.a.cut_out = L.snap32;
  for (int q = 0; q < 2; ++q) {
    e.X[q] = L.X32[q];
    e.XC[q] = C.X32[q];
  }
  e.xc_fixed = m->cplan.lc == l + 1;
  std::memcpy(out, &e, sizeof e);
}
int fused_units(mgfem_ctx* m, int l) {
  return m->lv[l].fp.ok && tile_nodes(m->lv[l].N) == 16 ? m->lv[l].fp.ntiles : -1;
}
void fused_launch(hipStream_t s, int kind, const void* tab, const int2* work, int nwork, int par, int parc, bool zero,
                  bool up) {
  if (nwork <= 0) return;
  const dim3 grid(8u * (unsigned)((nwork + 7) / 8)), bs(256);
  const FEntry* T = static_cast<const FEntry*>(tab);
  if (kind == kTeamRR)
    hipLaunchKernelGGL((k_fused_multi<kRestrictK, 256>), grid, bs, 0, s, T, work, nwork, par, parc, zero);
  else if (up)
    hipLaunchKernelGGL((k_fused_multi<kUpK, 256>), grid, bs, 0, s, T, work, nwork, par, parc, zero);
  else
    hipLaunchKernelGGL((k_fused_multi<kSweepK, 256>), grid, bs, 0, s, T, work, nwork, par, parc, zero);
}

// Plans of the levels that take these kernels: forward cycles with at least
// one post-smoothing sweep and at most 4 cut sweeps per step, levels above the
// coarse part that fill the chip about once (2^19 unknowns: 512 tiles of
// 32 x 32, two workgroups per CU).
// Measured per launch on the flower, one step (sweep with the cut sweeps),
// residual and restriction, prolongation with a step, in us, separate | fused:
//   float64  N = 256    9.6, 3.3, 9.6   |  4.9, 4.2, 4.2
//            N = 1024  10.3, 5.7, 11.6  |  6.6, 5.9, 7.0
//            N = 2048  15.1, 9.4, 17.1  | 19.0, 12.1, 22.4
// A level with a tile whose record does not hold its cut vertices keeps the
// separate kernels (as does MGFEM_NO_CUT_GROUPS=1).
// Larger float64 levels, and 1024 to 2048 above that count, take them only for
// the tiles that streaming passes leave (stream.hip), where one sweep goes up
// (the upward pass does one; a second would take a plan of every tile).  Up to
// N = 16384, the largest measured (solves with the band on the separate kernels
// | on the fused steps: N = 4096 3.7 | 3.1 ms, N = 16384 20.9 | 20.0).
constexpr int kMaxPlanN = 2048, kMinStreamFused = 1024, kMaxStreamFused = 16384;
int build_fused(mgfem_ctx* c) {
  const int cl = c->cplan.map.level >= 0 ? c->cplan.map.level : c->cplan.lc;
  const int eta = c->p.eta;
  const bool f32 = c->p.precision == MGFEM_PREC_MIXED;
  const int reach = f32 ? 0 : eta;  // float32 tiles hold no D, whatever eta is
  const char* env = std::getenv("MGFEM_NO_CUT_GROUPS");
  if ((env && env[0] && env[0] != '0') || (!f32 && 4 * eta > kMaxReachX) || c->p.nu2 < 1) return MGFEM_OK;
  std::vector<int> ls;  // the levels, by tile size: 32 x 32 tiles first
  const int64_t max_active = 1 << 19;
  auto whole = [&](int l) { return c->lv[l].N <= kMaxPlanN && c->lv[l].n_active <= max_active; };
  for (int l = 0; l < cl; ++l)
    if (!c->lv[l].empty() && (whole(l) || (!f32 && c->p.nu2 == 1 && c->lv[l].N >= kMinStreamFused &&
                                           c->lv[l].N <= kMaxStreamFused && stream_candidate(c, l))))
      ls.push_back(l);
  if (ls.empty()) return MGFEM_OK;
  if (ls.size() > (size_t)kMaxSet) return MGFEM_OK;  // (N = 16384 has 7 or so)
  SetLevels S{};
  S.n = (int)ls.size();
  int big = 0;
  for (int q = 0; q < S.n; ++q) big += tile_nodes(c->lv[ls[q]].N) == 32;
  auto carve = [](char*& p, size_t bytes) {
    char* q = p;
    p += (bytes + 255) & ~(size_t)255;
    return q;
  };
  int* tot_dev = nullptr;  // kTot ints per level
  constexpr int kTot = 16;
  // scratch of the plan: sizes bounded by the level's counts
  auto layout = [&](char* base) {
    char* p = base;
    auto ints = [&](size_t n) { return reinterpret_cast<int*>(carve(p, n * sizeof(int))); };
    tot_dev = ints(kTot * S.n);
    for (int q = 0; q < S.n; ++q) {
      const Level& L = c->lv[ls[q]];
      SetLevel& t = S.v[q];
      t.fl = L.flags;
      t.flc = c->lv[ls[q] + 1].flags;
      t.A = L.A;
      t.n = L.n;
      t.N = L.N;
      t.nc = L.N / kCell + 1;
      t.nt = L.N / tile_nodes(L.N) + 1;
      t.cut = eta > 0 && !f32 ? L.cut_off[4] : 0;
      t.coarse = q + 1 < S.n && ls[q + 1] == ls[q] + 1 ? q + 1 : -1;
      t.cutpos = L.cutpos;
      t.tot = tot_dev + kTot * q;
      const int ncell = t.nc * t.nc, ntile = t.nt * t.nt, cut = std::max(1, t.cut);
      for (int** w : {&t.cnt, &t.pos, &t.bid}) *w = ints(t.cut > 0 ? ncell + 1 : 1);
      t.sums = ints(t.cut > 0 ? 4 * (size_t)cell_runs(t.nc) + 4 : 1);
      t.npos = ints(t.cut > 0 ? L.n : 1);
      for (int** w : {&t.bcell, &t.rows, &t.ncol, &t.coff, &t.nval, &t.voff}) *w = ints(cut + 1);
      for (int** w : {&t.keep, &t.slot, &t.nst, &t.stoff, &t.nseg, &t.segoff}) *w = ints(ntile + 1);
      t.blocks = reinterpret_cast<FBlock*>(carve(p, (size_t)cut * sizeof(FBlock)));
      t.inner = whole(ls[q]) ? nullptr : reinterpret_cast<uint8_t*>(carve(p, (size_t)ntile));
    }
    return (size_t)(p - base);
  };
  const size_t total = layout(nullptr) + 256;
  TempMem scratch(c);
  MGFEM_HIP_TRY(scratch.alloc(total));
  layout(scratch.get());
  hipStream_t s = c->s;
  for (int q = 0; q < S.n; ++q)  // (tiles without an active node leave theirs)
    if (S.v[q].inner) MGFEM_HIP_TRY(hipMemsetAsync(S.v[q].inner, 0, (size_t)S.v[q].nt * S.v[q].nt, s));
  std::vector<int> tot(kTot * S.n, 0);
  auto totals = [&]() -> int {
    MGFEM_HIP_TRY(hipGetLastError());
    MGFEM_HIP_TRY(hipMemcpyAsync(tot.data(), tot_dev, tot.size() * sizeof(int), hipMemcpyDeviceToHost, s));
    MGFEM_HIP_TRY(hipStreamSynchronize(s));
    return MGFEM_OK;
  };
  int max_cell = 0, max_tile16 = 0, max_tile32 = 0, max_blk = 0, any_cut = 0;
  for (int q = 0; q < S.n; ++q) {
    const SetLevel& t = S.v[q];
    any_cut |= t.cut > 0;
    max_cell = std::max(max_cell, t.nc * t.nc);
    int& m = q < big ? max_tile32 : max_tile16;
    m = std::max(m, t.nt * t.nt);
  }
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(64), 0, s, tot_dev, kTot * S.n);
  if (any_cut) {
    // cells, positions, blocks
    hipLaunchKernelGGL(k_cell_count, dim3(nblk(max_cell, 256), S.n), dim3(256), 0, s, S);
    hipLaunchKernelGGL(k_scan_cells, dim3(S.n, 2), dim3(1024), 0, s, S);
    hipLaunchKernelGGL(k_cell_fill, dim3(nblk(max_cell, 256), S.n), dim3(256), 0, s, S);
    if (const int e = totals()) return e;
    for (int q = 0; q < S.n; ++q) {
      S.v[q].nblk = tot[kTot * q];
      c->lv[ls[q]].fp.ncut = tot[kTot * q + 1];
      max_blk = std::max(max_blk, S.v[q].nblk);
    }
    if (max_blk > 0) {
      hipLaunchKernelGGL(k_block_size, dim3(nblk(max_blk, 256), S.n), dim3(256), 0, s, S, eta);
      hipLaunchKernelGGL(k_scan_blocks, dim3(S.n, 2), dim3(1024), 0, s, S);
    }
  }
  if (big > 0)
    hipLaunchKernelGGL(k_ftile_count<32>, dim3(max_tile32, big), dim3(256), 0, s, S, 0, reach);
  if (big < S.n)
    hipLaunchKernelGGL(k_ftile_count<16>, dim3(max_tile16, S.n - big), dim3(256), 0, s, S, big, reach);
  hipLaunchKernelGGL(k_scan_tiles, dim3(S.n, 3), dim3(1024), 0, s, S);
  if (const int e = totals()) return e;
  // a level whose own plan, or whose coarser level's, does not fit keeps the
  // separate kernels (a stored row's record holds its position in 18 bits)
  for (int q = 0; q < S.n; ++q)
    c->lv[ls[q]].fp.ok = tot[kTot * q + 8] <= kMaxBlockCols && tot[kTot * q + 9] == 0 &&
                         c->lv[ls[q]].cut_off[4] < (1 << 18);
  // the windows of the levels that stream: no window, no plan
  for (int q = 0; q < S.n; ++q) {
    Level& L = c->lv[ls[q]];
    if (!S.v[q].inner) continue;
    if (L.fp.ok) {
      std::vector<uint8_t> inner((size_t)S.v[q].nt * S.v[q].nt);
      MGFEM_HIP_TRY(hipMemcpyAsync(inner.data(), S.v[q].inner, inner.size(), hipMemcpyDeviceToHost, s));
      MGFEM_HIP_TRY(hipStreamSynchronize(s));
      if (const int e = build_stream_fused(c, ls[q], inner, S.v[q].nt, tile_nodes(L.N))) return e;
    }
    L.fp.ok = L.sp.ok;
  }
  for (int q = S.n; q-- > 0;)
    if (S.v[q].coarse >= 0 && !c->lv[ls[q] + 1].fp.ok && S.v[q + 1].nblk > 0) {
      c->lv[ls[q]].fp.ok = false;
      c->lv[ls[q]].sp = StreamPlan{};
    }
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_delta_build), hipFuncAttributeMaxDynamicSharedMemorySize,
                            build_lds(kMaxBlockCols));
  // the blocks' values and columns
  auto block_bytes = [&](int q) {
    return ((size_t)tot[kTot * q + 3] * sizeof(double) + (size_t)tot[kTot * q + 2] * sizeof(int) + 255) & ~(size_t)255;
  };
  size_t all_blocks = 0;
  int max_cols = 0;
  for (int q = 0; q < S.n; ++q)
    if (c->lv[ls[q]].fp.ok && S.v[q].nblk > 0) {
      all_blocks += block_bytes(q);
      max_cols = std::max(max_cols, tot[kTot * q + 8]);
    }
  TempMem blocks(c);
  if (all_blocks > 0) MGFEM_HIP_TRY(blocks.alloc(all_blocks));
  char* next_block = blocks.get();
  for (int q = 0; q < S.n; ++q) {
    const int l = ls[q];
    Level& L = c->lv[l];
    SetLevel& t = S.v[q];
    FusedPlan& F = L.fp;
    if (!F.ok) continue;
    F.ntiles = tot[kTot * q + 4];
    // the second step carries the reduction of the first one's norm
    if (l == 0 && !f32 && c->p.nu1 >= 2) L.X[2] = c->lam;
    const size_t nst = (size_t)tot[kTot * q + 5], nseg = (size_t)tot[kTot * q + 6], v = f32 ? 4 : 8;
    char* buf = nullptr;
    MGFEM_HIP_TRY(ctx_alloc(c, reinterpret_cast<void**>(&buf),
                            (size_t)F.ncut * (sizeof(int) + 4 * v) + (size_t)F.ntiles * sizeof(FTile) +
                                nst * (sizeof(int) + 10 * v) + nseg * 288 + 8192));
    F.tiles = reinterpret_cast<FTile*>(carve(buf, (size_t)F.ntiles * sizeof(FTile)));
    F.st_coef = carve(buf, nst * 10 * v);
    F.st_idx = reinterpret_cast<int*>(carve(buf, nst * sizeof(int)));
    F.rows = reinterpret_cast<int*>(carve(buf, (size_t)F.ncut * sizeof(int)));
    for (double** w : {&F.r[0], &F.r[1], &F.r[2], &F.xs}) *w = reinterpret_cast<double*>(carve(buf, (size_t)F.ncut * v));
    if (!f32) {
      F.D = reinterpret_cast<double2*>(carve(buf, nseg * 128));
      if (!S.v[q].inner) F.DT = reinterpret_cast<double2*>(carve(buf, nseg * 128));  // (forward cycles alone)
    }
    F.Didx = reinterpret_cast<uint4*>(carve(buf, nseg * 32));
    t.tiles = F.tiles;
    t.st_idx = F.st_idx;
    t.st_coef = F.st_coef;
    t.fD = reinterpret_cast<double*>(F.D);
    t.fDT = reinterpret_cast<double*>(F.DT);
    t.fidx = reinterpret_cast<uint16_t*>(F.Didx);
    if (t.nblk == 0) continue;
    MGFEM_HIP_TRY(hipMemcpyAsync(F.rows, t.rows, (size_t)F.ncut * sizeof(int), hipMemcpyDeviceToDevice, s));
    t.D = reinterpret_cast<double*>(next_block);
    t.cols = reinterpret_cast<int*>(next_block + (size_t)tot[kTot * q + 3] * sizeof(double));
    next_block += block_bytes(q);
  }
  if (all_blocks > 0) {
    hipLaunchKernelGGL(k_block_fill, dim3(nblk(max_blk, 256), S.n), dim3(256), 0, s, S, eta);
    hipLaunchKernelGGL(k_delta_build, dim3(max_blk, S.n), dim3(64 * kBuildWaves), build_lds(max_cols), s, S, eta);
  }
  if (big > 0) {
    if (f32) hipLaunchKernelGGL((k_ftile_fill<float, 32>), dim3(max_tile32, big), dim3(1024), 0, s, S, 0, reach);
    else hipLaunchKernelGGL((k_ftile_fill<double, 32>), dim3(max_tile32, big), dim3(1024), 0, s, S, 0, reach);
  }
  if (big < S.n) {
    const dim3 g(max_tile16, S.n - big);
    if (f32) hipLaunchKernelGGL((k_ftile_fill<float, 16>), g, dim3(1024), 0, s, S, big, reach);
    else hipLaunchKernelGGL((k_ftile_fill<double, 16>), g, dim3(1024), 0, s, S, big, reach);
  }
  MGFEM_HIP_TRY(hipGetLastError());
  MGFEM_HIP_TRY(hipStreamSynchronize(s));  // the scratch goes
  return MGFEM_OK;
}

}  // namespace mgfem
