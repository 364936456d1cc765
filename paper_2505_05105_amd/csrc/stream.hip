// The downward half of a cycle on the largest levels: two smoothing sweeps,
// the residual and its restriction in one pass over memory.
//
// These levels are bound by their bytes (at N = 16384 a sweep moves its 24
// bytes per unknown at 8 TB/s), and the separate kernels read the iterate and
// the right-hand side three times on the way down.  Where every row in reach is
// the interior Q1 row a wave can do all of it as it streams down the grid: 64
// lanes of two columns each, rows in registers, the neighbouring columns by
// lane shifts, no LDS and no barrier.  Colours 0 and 1 are the even grid rows
// and 2 and 3 the odd ones, so a sweep takes one pass: even row 2m needs the old
// odd rows beside it, odd row 2m - 1 the new even ones.  The second sweep
// follows a row pair behind, the residual and its restriction another one.
// A window's values are exact on its core; the 10 columns and 6 rows around it
// are computed again by the windows beside it (a third more arithmetic than
// nodes, of which there is plenty).
//
// The windows are runs of sweep tiles away from the boundary.  The other tiles,
// the band, run the separate kernels, cut sweeps included.  The iterate goes
// through three buffers: the band's first sweep, and the windows that touch the
// band, write the second one, the second sweep the third.
//
// Measured (flower, float64, MI355X): at N = 4096 the two sweeps and the
// residual took 22 + 22 + 19 us in three launches; the windows take 21.5, the
// band 10 + 11 + 10.  At N = 16384 the windows take 320 us, the band 22 + 22 +
// 13, a sweep of the whole level alone 400; a solve went from 31.3 to 20.4 ms.
#include <algorithm>

#include "mgfem_internal.h"
#include "reduce.h"

namespace mgfem {
namespace {

constexpr int kHX = 10, kHY = 6;  // columns on either side of a window's core, rows above and below
constexpr int kCore = 128 - 2 * kHX;

struct Row {  // a lane's two columns: even, odd
  double e, o;
};
struct Pair {  // an even and the next odd row: iterate, right-hand side
  Row xe, xo, be, bo;
};
typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));

__device__ inline Row load_row(const double* p) {
  const double2u v = *reinterpret_cast<const double2u*>(p);
  return Row{v.x, v.y};
}
__device__ inline void store_row(double* p, const Row& v) {
  double2u w;
  w.x = v.e;
  w.y = v.o;
  *reinterpret_cast<double2u*>(p) = w;
}

// the value of the lane to the left, to the right (wave shifts; a wave's end
// lanes get 0, which only halo columns see)
__device__ inline double lane_left(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double lane_right(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// sums of three nodes of a row around each column, l and r the values of the
// neighbouring lanes' odd and even columns
__device__ inline Row sum3(const Row& x, double l, double r) { return Row{(l + x.e) + x.o, (x.e + x.o) + r}; }
__device__ inline double gs(double b, double below, double pair, double above) {
  return fma(3.0, b, (below + pair) + above) * 0.125;
}
__device__ inline double resid(double b, double x, double below, double pair, double above) {
  return b - fma(8.0 / 3.0, x, -(((below + pair) + above) * (1.0 / 3.0)));
}

// Gauss-Seidel on both columns of a row between rows with the sums `below` and
// `above`; l: the left lane's odd value before the update.  Returns the row's
// new sums; l and r become the neighbours' new values.
__device__ inline Row sweep_row(Row& x, const Row& b, const Row& below, const Row& above, double& l, double& r) {
  x.e = gs(b.e, below.e, l + x.o, above.e);
  r = lane_right(x.e);
  x.o = gs(b.o, below.o, x.e + r, above.o);
  l = lane_left(x.o);
  return sum3(x, l, r);
}

struct StreamArgs {
  const double* x;  // start iterate (null: zero)
  const double* b;
  double* out1;     // after the first sweep (windows that touch the band)
  double* out;      // after the second
  double* bc;       // restricted residual
  int N, s, sc;
  const int4* win;  // x, y, width | rows << 16, touches the band
  int nwin;
  double* part;     // per window (max |r|, sum r^2) of the start iterate
};

constexpr int kDepth = 3;  // row pairs in flight

// one window per wave, four per workgroup; the list is dealt to the XCDs in
// contiguous eighths (workgroups go to the XCDs round robin)
__device__ inline int window_of_wave(int nwin) {
  const int per = (((nwin + 3) >> 2) + 7) >> 3;
  return ((blockIdx.x & 7) * per + (blockIdx.x >> 3)) * 4 + (threadIdx.x >> 6);
}

// two sweeps, residual, restriction
template <bool ZERO, bool NORM>
__global__ __launch_bounds__(256) void k_stream(StreamArgs a) {
  const int wi = __builtin_amdgcn_readfirstlane(window_of_wave(a.nwin));
  if (wi >= a.nwin) return;  // whole waves; no barriers below
  const int4 W = a.win[wi];
  const int X = W.x, Y = W.y, width = W.z & 0xffff, H = W.z >> 16, lane = threadIdx.x & 63;
  const bool border = W.w != 0;
  const int col = X - kHX + 2 * lane;
  const bool core = lane >= kHX / 2 && lane < (kHX + width) / 2;
  const int lc = min(col, a.N - 1);  // lanes beyond the window's halo read inside the grid
  const int m0 = Y / 2 - kHY / 2, steps = H / 2 + kHY - 1, last = Y + H + kHY - 3;
  auto load = [&](int m) {
    Pair p;
    const int64_t r0 = (int64_t)min(2 * m, last) * a.s + lc, r1 = (int64_t)min(2 * m + 1, last) * a.s + lc;
    if constexpr (!ZERO) {
      p.xe = load_row(a.x + r0);
      p.xo = load_row(a.x + r1);
    } else {
      p.xe = p.xo = Row{0.0, 0.0};
    }
    p.be = load_row(a.b + r0);
    p.bo = load_row(a.b + r1);
    return p;
  };
  Pair q[kDepth];
#pragma unroll
  for (int k = 0; k < kDepth; ++k) q[k] = load(m0 + k);
  const Row z{0.0, 0.0};
  // first sweep: odd row 2m - 1 (values, old sums, right-hand side, left
  // neighbour), new sums of even row 2m - 2; its old sums for the norm
  Row O = z, Ot = z, Ob = z, Et = z, Eold = z;
  double Ol = 0.0, Onr = 0.0;
  // second sweep: even row 2m - 2, odd row 2m - 3 after the first sweep
  Row F = z, Fb = z, P = z, Pb = z, Pt = z;
  double Fl = 0.0, Pl = 0.0;
  // residual: even row 2m - 4 after both sweeps, its pair sums and sums, sums
  // of row 2m - 5, restricted part of row 2m - 5
  Row G = z, Gb = z, Gp = z, Gt = z, Ht = z;
  double lo = 0.0;
  double mx = 0.0, sm = 0.0;
  auto step = [&](const Pair& p, int m) {
    // --- first sweep: row 2m, then row 2m - 1
    Row E = p.xe;
    const Row Nx = p.xo;
    const double Nl = lane_left(Nx.o), Nr = lane_right(Nx.e);
    const Row Nt = sum3(Nx, Nl, Nr);
    double El = lane_left(E.o), Er;
    if constexpr (NORM) {
      // residuals of the start iterate: row 2m, and row 2m - 1 (its
      // neighbours' sums are all old here)
      const double er = lane_right(E.e);
      const Row old = sum3(E, El, er);
      if (core && 2 * m >= Y && 2 * m < Y + H) {
        const double r0 = resid(p.be.e, E.e, Ot.e, El + E.o, Nt.e);
        const double r1 = resid(p.be.o, E.o, Ot.o, E.e + er, Nt.o);
        mx = nanmax2(nanmax2(mx, fabs(r0)), fabs(r1));
        sm += r0 * r0 + r1 * r1;
      }
      if (core && 2 * m - 1 >= Y && 2 * m - 1 < Y + H) {
        const double r0 = resid(Ob.e, O.e, Eold.e, Ol + O.o, old.e);
        const double r1 = resid(Ob.o, O.o, Eold.o, O.e + Onr, old.o);
        mx = nanmax2(nanmax2(mx, fabs(r0)), fabs(r1));
        sm += r0 * r0 + r1 * r1;
      }
      Eold = old;
    }
    const Row Enew = sweep_row(E, p.be, Ot, Nt, El, Er);
    double Or;
    const Row Onew = sweep_row(O, Ob, Et, Enew, Ol, Or);
    if (border && core) {
      if (2 * m >= Y && 2 * m < Y + H) store_row(a.out1 + (int64_t)(2 * m) * a.s + col, E);
      if (2 * m - 1 >= Y && 2 * m - 1 < Y + H) store_row(a.out1 + (int64_t)(2 * m - 1) * a.s + col, O);
    }
    // --- second sweep: row 2m - 2, then row 2m - 3
    double Fr, Pr;
    const Row Ft = sweep_row(F, Fb, Pt, Onew, Fl, Fr);
    const Row Pt2 = sweep_row(P, Pb, Gt, Ft, Pl, Pr);
    if (core) {
      if (2 * m - 2 >= Y && 2 * m - 2 < Y + H) store_row(a.out + (int64_t)(2 * m - 2) * a.s + col, F);
      if (2 * m - 3 >= Y && 2 * m - 3 < Y + H) store_row(a.out + (int64_t)(2 * m - 3) * a.s + col, P);
    }
    // --- residual: rows 2m - 4 and 2m - 3, restriction to coarse row m - 2
    const double g0 = resid(Gb.e, G.e, Ht.e, Gp.e, Pt2.e), g1 = resid(Gb.o, G.o, Ht.o, Gp.o, Pt2.o);
    const double p0 = resid(Pb.e, P.e, Gt.e, Pl + P.o, Ft.e), p1 = resid(Pb.o, P.o, Gt.o, P.e + Pr, Ft.o);
    const double mid = g0 + 0.5 * (lane_left(g1) + g1);
    const double hi = p0 + 0.5 * (lane_left(p1) + p1);
    if (core && 2 * m - 4 >= Y && 2 * m - 4 < Y + H) a.bc[(col >> 1) + (int64_t)(m - 2) * a.sc] = mid + 0.5 * (lo + hi);
    lo = hi;
    // --- shift
    Ht = Pt2;
    G = F;
    Gb = Fb;
    Gp = Row{Fl + F.o, F.e + Fr};
    Gt = Ft;
    P = O;
    Pb = Ob;
    Pt = Onew;
    Pl = Ol;
    F = E;
    Fb = p.be;
    Fl = El;
    Et = Enew;
    O = Nx;
    Ot = Nt;
    Ob = p.bo;
    Ol = Nl;
    Onr = Nr;
  };
  for (int k0 = 0; k0 < steps; k0 += kDepth)
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
      const Pair p = q[k];
      q[k] = load(m0 + k0 + k + kDepth);
      step(p, m0 + k0 + k);
    }
  if constexpr (NORM) {
    for (int o = 32; o > 0; o >>= 1) {
      mx = nanmax2(mx, __shfl_xor(mx, o));
      sm += __shfl_xor(sm, o);
    }
    if (lane == 0) {
      a.part[2 * wi] = mx;
      a.part[2 * wi + 1] = sm;
    }
  }
}

// tiles of a list whose core and halo hold only active nodes with the interior
// row and no cut vertex
__global__ __launch_bounds__(256) void k_tile_inner(const int* __restrict__ tiles, int ntx, int i0, int j0, int TW,
                                                    int TH, const uint8_t* __restrict__ fl, int N,
                                                    int* __restrict__ inner) {
  const int t = tiles[blockIdx.x], x0 = i0 + (t % ntx) * TW - kHX, y0 = j0 + (t / ntx) * TH - kHY;
  const int W = TW + 2 * kHX, H = TH + 2 * kHY;
  int bad = 0;
  for (int q = threadIdx.x; q < W * H && !bad; q += 256) {
    const int i = x0 + q % W, j = y0 + q / W;
    if (i < 0 || j < 0 || i > N || j > N) bad = 1;
    else bad = (fl[i + (int64_t)j * (N + 1)] & (kFlagActive | kFlagStored | kFlagCut)) != kFlagActive;
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) inner[blockIdx.x] = !bad;
}

// coarse tiles that hold an active node no window restricts to
__global__ __launch_bounds__(256) void k_coarse_band(const int* __restrict__ tiles, int ntx, int I0, int J0, int I1,
                                                     int J1, int CW, int CH, const uint8_t* __restrict__ flc, int sc,
                                                     const uint8_t* __restrict__ inner, int fntx, int i0, int j0,
                                                     int i1, int j1, int TW, int TH, int* __restrict__ keep) {
  const int t = tiles[blockIdx.x], x0 = I0 + (t % ntx) * CW, y0 = J0 + (t / ntx) * CH;
  int any = 0;
  for (int q = threadIdx.x; q < CW * CH; q += 256) {
    const int I = x0 + q % CW, J = y0 + q / CW;
    if (I > I1 || J > J1 || !(flc[I + (int64_t)J * sc] & kFlagActive)) continue;
    const int i = 2 * I, j = 2 * J;
    if (i < i0 || j < j0 || i > i1 || j > j1 || !inner[(i - i0) / TW + (j - j0) / TH * fntx]) any = 1;
  }
  any = __syncthreads_or(any);
  if (threadIdx.x == 0) keep[blockIdx.x] = any;
}

}  // namespace

void stream_pass(mgfem_ctx* c, int l, int in, int mid, int out, double* part) {
  Level& L = c->lv[l];
  StreamArgs a{};
  a.x = L.zero ? nullptr : L.X[in];
  a.b = L.b;
  a.out1 = L.X[mid];
  a.out = L.X[out];
  a.bc = c->lv[l + 1].b;
  a.N = L.N;
  a.s = L.stride;
  a.sc = c->lv[l + 1].stride;
  a.win = L.sp.win;
  a.nwin = L.sp.nwin;
  a.part = part;
  const dim3 g(8u * (unsigned)((((a.nwin + 3) / 4) + 7) / 8)), bs(256);
  if (L.zero && part) hipLaunchKernelGGL((k_stream<true, true>), g, bs, 0, c->s, a);
  else if (L.zero) hipLaunchKernelGGL((k_stream<true, false>), g, bs, 0, c->s, a);
  else if (part) hipLaunchKernelGGL((k_stream<false, true>), g, bs, 0, c->s, a);
  else hipLaunchKernelGGL((k_stream<false, false>), g, bs, 0, c->s, a);
}

// Levels that stream: float64 forward cycles with two sweeps down, N >= 4096
// (the same three launches of a smaller level take 34 us at N = 2048).
constexpr int kStreamN = 4096;
bool stream_candidate(const mgfem_ctx* c, int l) {
  const Level& L = c->lv[l];
  return c->p.precision != MGFEM_PREC_MIXED && c->p.nu1 == 2 && L.N >= kStreamN && !L.empty() &&
         l + 1 < (int)c->lv.size() && !c->lv[l + 1].empty();
}

// Windows and band of a level whose tile lists exist.  No window, or no memory
// for the third buffer: the level keeps the separate kernels.
int build_stream(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  Level& C = c->lv[l + 1];
  StreamPlan& S = L.sp;
  if (!stream_candidate(c, l) || L.ntiles == 0) return MGFEM_OK;
  // tiles of the level (64 wide) and of the residual kernel (N >= 1024)
  const int TW = 64, TH = sweep_shape(c, l) == kShapeFinest ? 32 : 16, CW = 32, CH = 16;
  const int ntx = (L.bbox[1] - L.bbox[0] + TW) / TW, nty = (L.bbox[3] - L.bbox[2] + TH) / TH;
  const int cnx = (C.bbox[1] - C.bbox[0] + CW) / CW;
  struct Owner {
    char* p = nullptr;
    ~Owner() { (void)hipFree(p); }
  } tmp;
  const size_t ints = (size_t)L.ntiles + (size_t)std::max(1, L.rr_ntiles);
  MGFEM_HIP_TRY(hipMalloc(&tmp.p, ints * sizeof(int) + (size_t)ntx * nty));
  int* d_inner = reinterpret_cast<int*>(tmp.p);
  int* d_keep = d_inner + L.ntiles;
  uint8_t* d_map = reinterpret_cast<uint8_t*>(tmp.p + ints * sizeof(int));
  hipLaunchKernelGGL(k_tile_inner, dim3(L.ntiles), dim3(256), 0, c->s, (const int*)L.tiles, ntx, L.bbox[0], L.bbox[2],
                     TW, TH, (const uint8_t*)L.flags, L.N, d_inner);
  std::vector<int> inner(L.ntiles), tiles(L.ntiles);
  MGFEM_HIP_TRY(hipGetLastError());
  MGFEM_HIP_TRY(hipMemcpyAsync(inner.data(), d_inner, inner.size() * sizeof(int), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(tiles.data(), L.tiles, tiles.size() * sizeof(int), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  std::vector<uint8_t> map((size_t)ntx * nty, 0), list((size_t)ntx * nty, 0);
  for (int q = 0; q < L.ntiles; ++q) {
    map[tiles[q]] = inner[q] != 0;
    list[tiles[q]] = 1;
  }
  // windows: runs of inner tiles, several tile rows high where they all are
  // (fewer rows computed twice), as long as they give every SIMD a few waves
  std::vector<int4> win;
  for (int rows = 128 / TH; rows >= 1; rows /= 2) {
    std::vector<uint8_t> left = map;
    win.clear();
    for (int g = rows; g >= 1; g /= 2)
      for (int y = 0; y + g <= nty; y += g)
        for (int x = 0; x < ntx;) {
          auto good = [&](int tx) {
            bool on = tx < ntx;
            for (int v = 0; on && v < g; ++v) on = left[tx + (size_t)(y + v) * ntx] != 0;
            return on;
          };
          int e = x;
          for (; good(e); ++e)
            for (int v = 0; v < g; ++v) left[e + (size_t)(y + v) * ntx] = 0;
          if (e == x) {
            ++x;
            continue;
          }
          const int cols = (e - x) * TW, n = (cols + kCore - 1) / kCore, w = (cols / 2 + n - 1) / n * 2;
          for (int at = 0; at < cols; at += w) {
            const int width = std::min(w, cols - at);
            bool touch = false;  // a listed tile around the window is not inner
            for (int ty = std::max(0, y - 1); ty <= std::min(nty - 1, y + g); ++ty)
              for (int tx = std::max(0, x + at / TW - 1); tx <= std::min(ntx - 1, x + (at + width - 1) / TW + 1); ++tx)
                touch = touch || (list[tx + (size_t)ty * ntx] && !map[tx + (size_t)ty * ntx]);
            win.push_back(make_int4(L.bbox[0] + x * TW + at, L.bbox[2] + y * TH, width | g * TH << 16, touch));
          }
          x = e;
        }
    if (win.size() >= 3072) break;
  }
  if (win.empty()) return MGFEM_OK;
  std::vector<int> meta(8 * (size_t)L.ntiles), band;
  MGFEM_HIP_TRY(hipMemcpyAsync(meta.data(), L.tmeta, meta.size() * sizeof(int), hipMemcpyDeviceToHost, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(d_map, map.data(), map.size(), hipMemcpyHostToDevice, c->s));
  std::vector<int> rr(L.rr_ntiles), rr_keep(L.rr_ntiles), rr_band;
  if (L.rr_ntiles > 0) {
    hipLaunchKernelGGL(k_coarse_band, dim3(L.rr_ntiles), dim3(256), 0, c->s, (const int*)L.rr_tiles, cnx, C.bbox[0],
                       C.bbox[2], C.bbox[1], C.bbox[3], CW, CH, (const uint8_t*)C.flags, C.stride,
                       (const uint8_t*)d_map, ntx, L.bbox[0], L.bbox[2], L.bbox[1], L.bbox[3], TW, TH, d_keep);
    MGFEM_HIP_TRY(hipGetLastError());
    MGFEM_HIP_TRY(hipMemcpyAsync(rr.data(), L.rr_tiles, rr.size() * sizeof(int), hipMemcpyDeviceToHost, c->s));
    MGFEM_HIP_TRY(hipMemcpyAsync(rr_keep.data(), d_keep, rr.size() * sizeof(int), hipMemcpyDeviceToHost, c->s));
  }
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  for (int q = 0; q < L.ntiles; ++q)
    if (!inner[q]) band.insert(band.end(), meta.begin() + 8 * (size_t)q, meta.begin() + 8 * (size_t)(q + 1));
  for (int q = 0; q < L.rr_ntiles; ++q)
    if (rr_keep[q]) rr_band.push_back(rr[q]);
  if (l == 0) {
    L.X[2] = c->lam;
  } else if (ctx_alloc_t(c, &L.X[2], L.n) != hipSuccess) {
    (void)hipGetLastError();
    L.X[2] = nullptr;
    return MGFEM_OK;
  }
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.win, win.size()));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.band, std::max<size_t>(8, band.size())));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.rr_band, std::max<size_t>(1, rr_band.size())));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.win, win.data(), win.size() * sizeof(int4), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.band, band.data(), band.size() * sizeof(int), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.rr_band, rr_band.data(), rr_band.size() * sizeof(int), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  S.nwin = (int)win.size();
  S.nband = (int)band.size() / 8;
  S.nrr = (int)rr_band.size();
  S.ok = true;
  return MGFEM_OK;
}

}  // namespace mgfem
