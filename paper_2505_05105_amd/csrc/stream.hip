// Streaming passes of the largest levels: downwards two smoothing sweeps, the
// residual and its restriction in one pass over memory, upwards the
// prolongation and a sweep.
//
// These levels are bound by their bytes, and the separate kernels read the
// iterate and the right-hand side three times on the way down.  Where every row
// in reach is the interior Q1 row a wave can do all of it as it streams down
// the grid: 64 lanes of two columns each, rows in registers, the neighbouring
// columns by lane shifts, no LDS and no barrier.  Colours 0 and 1 are the even
// grid rows and 2 and 3 the odd ones, so a sweep takes one pass: even row 2m
// needs the old odd rows beside it, odd row 2m - 1 the new even ones.  The
// second sweep follows a row pair behind, the residual and its restriction
// another one.  A window's values are exact on its core; the columns and rows
// around it are computed again by the windows beside it.
//
// The windows are runs of tiles away from the boundary.  The other tiles, the
// band, run the fused steps (fused.hip, on 32 x 32 tiles) where the level has
// their plan, float64 with one sweep up, and else the separate kernels, cut
// sweeps included.  The iterate goes through three buffers: the band's first
// sweep, and the windows that touch the band, write the second one, the second
// sweep the third.
//
// Measured (flower, float64, MI355X).  N = 16384 (54 million unknowns, 1.4 GB
// per pass): down 320 us (4.4 TB/s; a large copy reaches 5.2) where two sweeps
// and the residual took 400 + 400 + 300, up 308 (before 386).  N = 4096 (90 MB
// per pass, in the last-level cache): down 20-21 us where the three launches
// took 22 + 22 + 19, up 20.  The table at the rule below has whole solves.
#include <algorithm>

#include "mgfem_internal.h"
#include "reduce.h"

namespace mgfem {
namespace {

constexpr int kHX = kStreamHX, kHY = kStreamHY;  // columns on either side of a window's core, rows above and below
constexpr int kUpX = 6, kUpY = 2;    // of the upward pass (4 columns of the sweep, one of the prolongation)
constexpr int kCore = 128 - 2 * kHX, kUpCore = 128 - 2 * kUpX;

template <class T>
struct Row {  // a lane's two columns: even, odd
  T e, o;
};
template <class T>
struct Pair {  // an even and the next odd row: iterate, right-hand side
  Row<T> xe, xo, be, bo;
};
typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

__device__ inline Row<double> load_row(const double* p) {
  const double2u v = *reinterpret_cast<const double2u*>(p);
  return Row<double>{v.x, v.y};
}
__device__ inline Row<float> load_row(const float* p) {
  const float2u v = *reinterpret_cast<const float2u*>(p);
  return Row<float>{v.x, v.y};
}
// Stores that no branch guards: a lane or row outside a window's core stores
// beyond the buffer's end, where the hardware drops it.  (Loads and stores
// complete in order behind one counter, so a store that may or may not have
// been issued makes the compiler wait for rows it only wants three pairs
// later.  With the copies below, N = 2048 18.4 us before, 14.6 after.)
struct Out {
  __amdgpu_buffer_rsrc_t r;
  __device__ Out(void* base, unsigned bytes) : r(__builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000)) {}
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  __device__ void put(unsigned at, const Row<double>& v) const {
    u4 w;
    w.x = __double2loint(v.e);
    w.y = __double2hiint(v.e);
    w.z = __double2loint(v.o);
    w.w = __double2hiint(v.o);
    __builtin_amdgcn_raw_buffer_store_b128(w, r, at, 0, 0);
  }
  __device__ void put(unsigned at, double v) const {
    u2 w;
    w.x = __double2loint(v);
    w.y = __double2hiint(v);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, at, 0, 0);
  }
  __device__ void put(unsigned at, const Row<float>& v) const {
    u2 w;
    w.x = __float_as_uint(v.e);
    w.y = __float_as_uint(v.o);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, at, 0, 0);
  }
  __device__ void put(unsigned at, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, at, 0, 0);
  }
};

// the value of the lane to the left, to the right (wave shifts; a wave's end
// lanes get 0, which only halo columns see)
template <int CTRL>
__device__ inline float lane_shift(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ inline double lane_shift(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <class T>
__device__ inline T lane_left(T v) {
  return lane_shift<0x138>(v);
}
template <class T>
__device__ inline T lane_right(T v) {
  return lane_shift<0x130>(v);
}

// A copy in registers of its own.  What a step keeps of a loaded row for the
// next steps goes through it, so that the row's registers are free when the row
// three pairs on is loaded into them: left to itself the compiler rotates the
// prefetched rows through copies at the end of its unrolled loop, each of which
// waits for a load just issued.
__device__ inline float own(float v) {
  float w;
  asm("v_mov_b32 %0, %1" : "=v"(w) : "v"(v));
  return w;
}
__device__ inline double own(double v) {
  int lo, hi;
  asm("v_mov_b32 %0, %1" : "=v"(lo) : "v"(__double2loint(v)));
  asm("v_mov_b32 %0, %1" : "=v"(hi) : "v"(__double2hiint(v)));
  return __hiloint2double(hi, lo);
}
template <class T>
__device__ inline Row<T> own(const Row<T>& r) {
  return Row<T>{own(r.e), own(r.o)};
}

// A sweep does not use the old values of its first colour: their half of a
// row load is used here, so that nothing else takes those registers while the
// load is in flight (and waits for it).
template <class T>
__device__ inline void use(T v) {
  asm volatile("" : : "v"(v));
}

__device__ inline double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ inline float fma_t(float a, float b, float c) { return fmaf(a, b, c); }

// sums of three nodes of a row around each column, l and r the values of the
// neighbouring lanes' odd and even columns
template <class T>
__device__ inline Row<T> sum3(const Row<T>& x, T l, T r) {
  return Row<T>{(l + x.e) + x.o, (x.e + x.o) + r};
}
// the tile kernels' expressions, operation for operation (float32 results do
// not depend on which of the two computed a node)
template <class T>
__device__ inline T gs(T b, T below, T pair, T above) {
  return fma_t(T(3), b, (below + pair) + above) * T(0.125);
}
template <class T>
__device__ inline T resid(T b, T x, T below, T pair, T above) {
  return b - fma_t(T(8) / T(3), x, -(((below + pair) + above) * T(1.0 / 3.0)));
}

// Gauss-Seidel on both columns of a row between rows with the sums `below` and
// `above`; l: the left lane's odd value before the update.  Returns the row's
// new sums; l and r become the neighbours' new values.
template <class T>
__device__ inline Row<T> sweep_row(Row<T>& x, const Row<T>& b, const Row<T>& below, const Row<T>& above, T& l, T& r) {
  x.e = gs(b.e, below.e, l + x.o, above.e);
  r = lane_right(x.e);
  x.o = gs(b.o, below.o, x.e + r, above.o);
  l = lane_left(x.o);
  return sum3(x, l, r);
}

template <class T>
struct StreamArgs {
  const T* x;   // start iterate (null: zero)
  const T* b;
  T* out1;      // down: after the first sweep (windows that touch the band)
  T* out;       // after the last
  T* bc;        // down: restricted residual
  const T* xc;  // up: coarse iterate
  int N, s, sc;
  const int4* win;  // x, y, width | rows << 16, touches the band
  int nwin;
  double* part;  // down: per window (max |r|, sum r^2) of the start iterate
};

constexpr int kDepth = 3;  // row pairs in flight

// one window per wave, four per workgroup; the list is dealt to the XCDs in
// contiguous eighths (workgroups go to the XCDs round robin)
__device__ inline int window_of_wave(int nwin) {
  const int per = (((nwin + 3) >> 2) + 7) >> 3;
  return ((blockIdx.x & 7) * per + (blockIdx.x >> 3)) * 4 + (threadIdx.x >> 6);
}

// two sweeps, residual, restriction
template <class T, bool ZERO, bool NORM, bool BORDER>
__device__ inline void stream_window(const StreamArgs<T>& a, const int wi, const int4 W) {
  const int X = W.x, Y = W.y, width = W.z & 0xffff, H = W.z >> 16, lane = threadIdx.x & 63;
  const int col = X - kHX + 2 * lane;
  const bool core = lane >= kHX / 2 && lane < (kHX + width) / 2;
  const int lc = min(col, a.N - 1);  // lanes beyond the window's halo read inside the grid
  const int m0 = Y / 2 - kHY / 2, steps = H / 2 + kHY - 1, last = Y + H + kHY - 3;
  // byte offsets from the core's first row (a row before or behind the core
  // is beyond the end, as is a lane beside it)
  const unsigned rb = (unsigned)(a.s * sizeof(T)), rc = (unsigned)(a.sc * sizeof(T));
  const unsigned at = core ? (unsigned)(col * (int)sizeof(T)) : 0x80000000u, atc = core ? (unsigned)((col >> 1) * (int)sizeof(T)) : 0x80000000u;
  const Out out(a.out + (int64_t)Y * a.s, (unsigned)H * rb);
  const Out out1(a.out1 + (int64_t)Y * a.s, (unsigned)H * rb);
  const Out bc(a.bc + (int64_t)(Y / 2) * a.sc, (unsigned)(H / 2) * rc);
  auto load = [&](int m) {
    Pair<T> p;
    const int64_t r0 = (int64_t)min(2 * m, last) * a.s + lc, r1 = (int64_t)min(2 * m + 1, last) * a.s + lc;
    if constexpr (!ZERO) {
      p.xe = load_row(a.x + r0);
      p.xo = load_row(a.x + r1);
    } else {
      p.xe = p.xo = Row<T>{T(0), T(0)};
    }
    p.be = load_row(a.b + r0);
    p.bo = load_row(a.b + r1);
    return p;
  };
  Pair<T> q[kDepth];
#pragma unroll
  for (int k = 0; k < kDepth; ++k) {
    q[k] = load(m0 + k);
    __builtin_amdgcn_sched_barrier(0);  // oldest first
  }
  const Row<T> z{0.0, 0.0};
  // first sweep: odd row 2m - 1 (values, old sums, right-hand side, left
  // neighbour), new sums of even row 2m - 2; its old sums for the norm
  Row<T> O = z, Ot = z, Ob = z, Et = z, Eold = z;
  T Ol = T(0), Onr = T(0);
  // second sweep: even row 2m - 2, odd row 2m - 3 after the first sweep
  Row<T> F = z, Fb = z, P = z, Pb = z, Pt = z;
  T Fl = T(0), Pl = T(0);
  // residual: even row 2m - 4 after both sweeps, its pair sums and sums, sums
  // of row 2m - 5, restricted part of row 2m - 5
  Row<T> G = z, Gb = z, Gp = z, Gt = z, Ht = z;
  T lo = T(0);
  double mx = 0.0, sm = 0.0;
  auto step = [&](const Pair<T>& p, int m) {
    // --- first sweep: row 2m, then row 2m - 1
    if constexpr (!ZERO) use(p.xe.e);
    Row<T> E = p.xe;
    const Row<T> Nx = own(p.xo);
    const T Nl = lane_left(Nx.o), Nr = lane_right(Nx.e);
    const Row<T> Nt = sum3(Nx, Nl, Nr);
    T El = lane_left(E.o), Er;
    if constexpr (NORM) {
      // residuals of the start iterate: row 2m, and row 2m - 1 (its
      // neighbours' sums are all old here)
      const T er = lane_right(E.e);
      const Row<T> old = sum3(E, El, er);
      const bool in0 = core && 2 * m >= Y && 2 * m < Y + H, in1 = core && 2 * m - 1 >= Y && 2 * m - 1 < Y + H;
      const double r0 = in0 ? (double)resid(p.be.e, E.e, Ot.e, El + E.o, Nt.e) : 0.0;
      const double r1 = in0 ? (double)resid(p.be.o, E.o, Ot.o, E.e + er, Nt.o) : 0.0;
      const double r2 = in1 ? (double)resid(Ob.e, O.e, Eold.e, Ol + O.o, old.e) : 0.0;
      const double r3 = in1 ? (double)resid(Ob.o, O.o, Eold.o, O.e + Onr, old.o) : 0.0;
      mx = nanmax2(nanmax2(nanmax2(nanmax2(mx, fabs(r0)), fabs(r1)), fabs(r2)), fabs(r3));
      sm += (r0 * r0 + r1 * r1) + (r2 * r2 + r3 * r3);
      Eold = old;
    }
    const Row<T> Enew = sweep_row(E, p.be, Ot, Nt, El, Er);
    T Or;
    const Row<T> Onew = sweep_row(O, Ob, Et, Enew, Ol, Or);
    const unsigned rel = (unsigned)(2 * m - Y);
    if constexpr (BORDER) {
      out1.put(at + rel * rb, E);
      out1.put(at + (rel - 1) * rb, O);
    }
    // --- second sweep: row 2m - 2, then row 2m - 3
    T Fr, Pr;
    const Row<T> Ft = sweep_row(F, Fb, Pt, Onew, Fl, Fr);
    const Row<T> Pt2 = sweep_row(P, Pb, Gt, Ft, Pl, Pr);
    out.put(at + (rel - 2) * rb, F);
    out.put(at + (rel - 3) * rb, P);
    // --- residual: rows 2m - 4 and 2m - 3, restriction to coarse row m - 2
    const T g0 = resid(Gb.e, G.e, Ht.e, Gp.e, Pt2.e), g1 = resid(Gb.o, G.o, Ht.o, Gp.o, Pt2.o);
    const T p0 = resid(Pb.e, P.e, Gt.e, Pl + P.o, Ft.e), p1 = resid(Pb.o, P.o, Gt.o, P.e + Pr, Ft.o);
    const T mid = g0 + T(0.5) * (lane_left(g1) + g1);
    const T hi = p0 + T(0.5) * (lane_left(p1) + p1);
    bc.put(atc + (unsigned)(m - 2 - Y / 2) * rc, mid + T(0.5) * (lo + hi));
    lo = hi;
    // --- shift
    Ht = Pt2;
    G = F;
    Gb = Fb;
    Gp = Row<T>{Fl + F.o, F.e + Fr};
    Gt = Ft;
    P = O;
    Pb = Ob;
    Pt = Onew;
    Pl = Ol;
    F = E;
    Fb = own(p.be);
    Fl = El;
    Et = Enew;
    O = Nx;
    Ot = Nt;
    Ob = own(p.bo);
    Ol = Nl;
    Onr = Nr;
  };
  auto round = [&](int k0) {
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
      step(q[k], m0 + k0 + k);
      q[k] = load(m0 + k0 + k + kDepth);
      __builtin_amdgcn_sched_barrier(0);  // no step starts before its turn (it would wait for its rows)
    }
  };
  // the first round apart: what the loop finds in flight is then the same on
  // every way in, and it waits for no more than its own rows
  round(0);
  for (int k0 = kDepth; k0 < steps; k0 += kDepth) round(k0);
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

template <class T, bool ZERO, bool NORM>
__global__ __launch_bounds__(256) void k_stream(StreamArgs<T> a) {
  const int wi = __builtin_amdgcn_readfirstlane(window_of_wave(a.nwin));
  if (wi >= a.nwin) return;  // whole waves; no barriers below
  const int4 W = a.win[wi];
  if (W.w) stream_window<T, ZERO, NORM, true>(a, wi, W);
  else stream_window<T, ZERO, NORM, false>(a, wi, W);
}

// x + P x_c, then one sweep (odd row 2m - 1 once the even row 2m is new)
template <class T>
__global__ __launch_bounds__(256) void k_stream_up(StreamArgs<T> a) {
  const int wi = __builtin_amdgcn_readfirstlane(window_of_wave(a.nwin));
  if (wi >= a.nwin) return;
  const int4 W = a.win[wi];
  const int X = W.x, Y = W.y, width = W.z & 0xffff, H = W.z >> 16, lane = threadIdx.x & 63;
  const int col = X - kUpX + 2 * lane;
  const bool core = lane >= kUpX / 2 && lane < (kUpX + width) / 2;
  const int lc = min(col, a.N - 1), lcc = min(col, a.N) >> 1, Nc = a.N >> 1;
  const int m0 = Y / 2 - kUpY / 2, steps = H / 2 + kUpY, last = Y + H + kUpY - 1;
  const unsigned rb = (unsigned)(a.s * sizeof(T));
  const unsigned at = core ? (unsigned)(col * (int)sizeof(T)) : 0x80000000u;
  const Out out(a.out + (int64_t)Y * a.s, (unsigned)H * rb);
  struct Rows {
    Pair<T> p;
    T c;  // coarse row m + 1
  };
  auto load = [&](int m) {
    Rows u;
    const int64_t r0 = (int64_t)min(2 * m, last) * a.s + lc, r1 = (int64_t)min(2 * m + 1, last) * a.s + lc;
    u.p.xe = load_row(a.x + r0);
    u.p.xo = load_row(a.x + r1);
    u.c = a.xc[lcc + (int64_t)min(m + 1, Nc) * a.sc];
    u.p.be = load_row(a.b + r0);
    u.p.bo = load_row(a.b + r1);
    return u;
  };
  T C = a.xc[lcc + (int64_t)m0 * a.sc];
  Rows q[kDepth];
#pragma unroll
  for (int k = 0; k < kDepth; ++k) {
    q[k] = load(m0 + k);
    __builtin_amdgcn_sched_barrier(0);  // oldest first
  }
  const Row<T> z{T(0), T(0)};
  T Cr = lane_right(C), Ol = T(0);
  Row<T> O = z, Ot = z, Ob = z, Et = z;
  auto step = [&](const Rows& u, int m) {
    use(u.p.xe.e);
    // even columns have one coarse parent in x, odd ones two; rows in y likewise
    const T D = own(u.c), Dr = lane_right(D);
    Row<T> E, Nx;
    E.e = fma_t(T(0.25), (C + C) + (C + C), u.p.xe.e);
    E.o = fma_t(T(0.25), (C + Cr) + (C + Cr), u.p.xe.o);
    Nx.e = fma_t(T(0.25), (C + C) + (D + D), u.p.xo.e);
    Nx.o = fma_t(T(0.25), (C + Cr) + (D + Dr), u.p.xo.o);
    C = D;
    Cr = Dr;
    const T Nl = lane_left(Nx.o), Nr = lane_right(Nx.e);
    const Row<T> Nt = sum3(Nx, Nl, Nr);
    T El = lane_left(E.o), Er, Or;
    const Row<T> Enew = sweep_row(E, u.p.be, Ot, Nt, El, Er);
    sweep_row(O, Ob, Et, Enew, Ol, Or);
    const unsigned rel = (unsigned)(2 * m - Y);
    out.put(at + rel * rb, E);
    out.put(at + (rel - 1) * rb, O);
    Et = Enew;
    O = Nx;
    Ot = Nt;
    Ob = own(u.p.bo);
    Ol = Nl;
  };
  auto round = [&](int k0) {
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
      step(q[k], m0 + k0 + k);
      q[k] = load(m0 + k0 + k + kDepth);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  round(0);  // apart, as in the downward pass
  for (int k0 = kDepth; k0 < steps; k0 += kDepth) round(k0);
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

namespace {
template <class T>
struct Of;
template <>
struct Of<double> {
  static double* X(const Level& L, int w) { return L.X[w]; }
  static double* B(const Level& L) { return L.b; }
};
template <>
struct Of<float> {
  static float* X(const Level& L, int w) { return L.X32[w]; }
  static float* B(const Level& L) { return L.b32; }
};
template <class T>
StreamArgs<T> stream_args(mgfem_ctx* c, int l, int in, int out, const int4* win, int nwin) {
  const Level& L = c->lv[l];
  StreamArgs<T> a{};
  a.x = Of<T>::X(L, in);
  a.b = Of<T>::B(L);
  a.out = Of<T>::X(L, out);
  a.N = L.N;
  a.s = L.stride;
  a.sc = c->lv[l + 1].stride;
  a.win = win;
  a.nwin = nwin;
  return a;
}
// a pass of level 0 in a profiled solve is timed where it runs (it reads one
// buffer and writes others, so that it can be repeated)
template <class F>
void run_pass(mgfem_ctx* c, int l, int kernel_class, double bytes, const F& go) {
  if (c->prof.on && l == 0) prof_launch(c, kernel_class, bytes, go);
  else go(c->s);
}
inline dim3 stream_grid(int nwin) { return dim3(8u * (unsigned)((((nwin + 3) / 4) + 7) / 8)); }
template <class T>
void launch_down(mgfem_ctx* c, int l, int in, int mid, int out, double* part) {
  const Level& L = c->lv[l];
  StreamArgs<T> a = stream_args<T>(c, l, in, out, L.sp.win, L.sp.nwin);
  a.out1 = Of<T>::X(L, mid);
  a.bc = Of<T>::B(c->lv[l + 1]);
  a.part = part;
  const dim3 g = stream_grid(a.nwin), bs(256);
  const bool zero = L.zero;
  run_pass(c, l, 2, sizeof(T) * (zero ? 2.25 : 3.25) * L.sp.down_nodes, [a, g, bs, zero](hipStream_t st) {
    if (zero && a.part) hipLaunchKernelGGL((k_stream<T, true, true>), g, bs, 0, st, a);
    else if (zero) hipLaunchKernelGGL((k_stream<T, true, false>), g, bs, 0, st, a);
    else if (a.part) hipLaunchKernelGGL((k_stream<T, false, true>), g, bs, 0, st, a);
    else hipLaunchKernelGGL((k_stream<T, false, false>), g, bs, 0, st, a);
  });
}
template <class T>
void launch_up(mgfem_ctx* c, int l, int in, int out) {
  const Level& L = c->lv[l];
  const Level& C = c->lv[l + 1];
  StreamArgs<T> a = stream_args<T>(c, l, in, out, L.sp.up, L.sp.nup);
  a.xc = Of<T>::X(C, C.cur);
  run_pass(c, l, 3, sizeof(T) * 3.25 * L.sp.up_nodes, [a](hipStream_t st) {
    hipLaunchKernelGGL(k_stream_up<T>, stream_grid(a.nwin), dim3(256), 0, st, a);
  });
}
}  // namespace

void stream_down_windows(mgfem_ctx* c, int l, bool fp32, int in, int mid, int out, double* part) {
  if (fp32) launch_down<float>(c, l, in, mid, out, part);
  else launch_down<double>(c, l, in, mid, out, part);
}
void stream_up_windows(mgfem_ctx* c, int l, bool fp32, int in, int out) {
  if (fp32) launch_up<float>(c, l, in, out);
  else launch_up<double>(c, l, in, out);
}

// Levels that stream: forward cycles with two sweeps down.  In float64 with one
// sweep up from N = 1024, the band on the fused steps; otherwise (the band on the
// separate kernels) from N = 4096, in float64 also the coarser levels with
// N >= 2048, whose start iterate is zero and is not read.  The upward pass from
// N >= 4096, and with the fused band.  Speed of solves against one fixed earlier
// program, with separate kernels | downward pass | both | both and the fused band:
//   flower, float64, N = 4096     1.12 | 1.19 | 1.19, with the 2048 level 1.22 | 1.43
//   flower, float64, N = 16384           |      | 1.63 | 1.70
//   ellipse, mixed, N = 4096      1.06 | 1.08 | 1.09, with the 2048 level 1.07 |
//   gradient, float64, N = 2048   1.18 to 1.20, if level 0 streams 1.15 to 1.17 | | 1.26
//   annulus, float64, N = 1536    1.20, if level 0 streams 1.20 | | 1.30
constexpr int kStreamN = 4096, kStreamCoarseN = 2048, kStreamFusedN = 1024, kUpN = 4096;
bool stream_candidate(const mgfem_ctx* c, int l) {
  const Level& L = c->lv[l];
  const int n = c->p.precision == MGFEM_PREC_MIXED ? kStreamN : c->p.nu2 == 1 ? kStreamFusedN
                : l > 0                                               ? kStreamCoarseN
                                                                      : kStreamN;
  return c->p.nu1 == 2 && c->p.nu2 >= 1 && L.N >= n && !L.empty() && l + 1 < (int)c->lv.size() &&
         !c->lv[l + 1].empty();
}

namespace {
// Windows of at most `core` columns over the inner tiles of a tile grid: runs
// of them, several tile rows high where they all are (fewer rows computed
// twice) as long as that gives every SIMD a few waves, half a tile row high
// where even one gives too few (a wave's row pairs are one serial chain).
std::vector<int4> build_windows(const std::vector<uint8_t>& map, const std::vector<uint8_t>& list, int ntx, int nty,
                                int x0, int y0, int TW, int TH, int core) {
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
          const int cols = (e - x) * TW, n = (cols + core - 1) / core, w = (cols / 2 + n - 1) / n * 2;
          for (int at = 0; at < cols; at += w) {
            const int width = std::min(w, cols - at);
            bool touch = false;  // a listed tile around the window is not inner
            for (int ty = std::max(0, y - 1); ty <= std::min(nty - 1, y + g); ++ty)
              for (int tx = std::max(0, x + at / TW - 1); tx <= std::min(ntx - 1, x + (at + width - 1) / TW + 1); ++tx)
                touch = touch || (list[tx + (size_t)ty * ntx] && !map[tx + (size_t)ty * ntx]);
            win.push_back(make_int4(x0 + x * TW + at, y0 + y * TH, width | g * TH << 16, touch));
          }
          x = e;
        }
    if (win.size() >= 3072) return win;
  }
  if (win.size() < 1536)
    for (size_t q = 0, n = win.size(); q < n; ++q) {
      int4 w = win[q];
      const int h = w.z >> 17;
      win[q].z = (w.z & 0xffff) | h << 16;
      w.y += h;
      w.z = win[q].z;
      win.push_back(w);
    }
  return win;
}
double core_nodes(const std::vector<int4>& win) {
  double n = 0.0;
  for (const int4& w : win) n += (double)(w.z & 0xffff) * (w.z >> 16);
  return n;
}
}  // namespace

int build_stream_fused(mgfem_ctx* c, int l, const std::vector<uint8_t>& inner, int nt, int TN) {
  Level& L = c->lv[l];
  StreamPlan& S = L.sp;
  const std::vector<uint8_t> all(inner.size(), 1);
  const std::vector<int4> win = build_windows(inner, all, nt, nt, 0, 0, TN, TN, kCore);
  const std::vector<int4> up = build_windows(inner, all, nt, nt, 0, 0, TN, TN, kUpCore);
  if (win.empty()) return MGFEM_OK;
  if (l == 0) {
    L.X[2] = c->lam;
  } else if (ctx_alloc_t(c, &L.X[2], L.n) != hipSuccess) {
    (void)hipGetLastError();
    return MGFEM_OK;
  }
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.win, win.size()));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.up, up.size()));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.win, win.data(), win.size() * sizeof(int4), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.up, up.data(), up.size() * sizeof(int4), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  S.nwin = (int)win.size();
  S.nup = (int)up.size();
  S.down_nodes = core_nodes(win);
  S.up_nodes = core_nodes(up);
  S.ok = S.fused = true;
  return MGFEM_OK;
}

// Windows and band of a level whose tile lists exist.  No window, or no memory
// for the third buffer: the level keeps the separate kernels.
int build_stream(mgfem_ctx* c, int l) {
  Level& L = c->lv[l];
  Level& C = c->lv[l + 1];
  StreamPlan& S = L.sp;
  if (!stream_candidate(c, l) || L.N < kStreamCoarseN || (l == 0 && L.N < kStreamN) || L.ntiles == 0) return MGFEM_OK;
  // tiles of the level (64 wide) and of the residual kernel (N >= 1024)
  const int TW = 64, TH = sweep_shape(c, l) == kShapeFinest ? 32 : 16, CW = 32, CH = 16;
  const int ntx = (L.bbox[1] - L.bbox[0] + TW) / TW, nty = (L.bbox[3] - L.bbox[2] + TH) / TH;
  const int cnx = (C.bbox[1] - C.bbox[0] + CW) / CW;
  TempMem tmp(c);
  const size_t ints = (size_t)L.ntiles + (size_t)std::max(1, L.rr_ntiles);
  MGFEM_HIP_TRY(tmp.alloc(ints * sizeof(int) + (size_t)ntx * nty));
  int* d_inner = reinterpret_cast<int*>(tmp.get());
  int* d_keep = d_inner + L.ntiles;
  uint8_t* d_map = reinterpret_cast<uint8_t*>(tmp.get() + ints * sizeof(int));
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
  const std::vector<int4> win = build_windows(map, list, ntx, nty, L.bbox[0], L.bbox[2], TW, TH, kCore);
  const std::vector<int4> up = build_windows(map, list, ntx, nty, L.bbox[0], L.bbox[2], TW, TH, kUpCore);
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
  hipError_t e = hipSuccess;
  if (c->p.precision == MGFEM_PREC_MIXED) e = ctx_alloc_t(c, &L.X32[2], L.n);
  else if (l == 0) L.X[2] = c->lam;
  else e = ctx_alloc_t(c, &L.X[2], L.n);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return MGFEM_OK;
  }
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.win, win.size()));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.up, up.size()));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.up, up.data(), up.size() * sizeof(int4), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.band, std::max<size_t>(8, band.size())));
  MGFEM_HIP_TRY(ctx_alloc_t(c, &S.rr_band, std::max<size_t>(1, rr_band.size())));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.win, win.data(), win.size() * sizeof(int4), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.band, band.data(), band.size() * sizeof(int), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipMemcpyAsync(S.rr_band, rr_band.data(), rr_band.size() * sizeof(int), hipMemcpyHostToDevice, c->s));
  MGFEM_HIP_TRY(hipStreamSynchronize(c->s));
  S.nwin = (int)win.size();
  S.nup = L.N >= kUpN ? (int)up.size() : 0;
  S.nband = (int)band.size() / 8;
  S.nrr = (int)rr_band.size();
  S.ok = true;
  return MGFEM_OK;
}

}  // namespace mgfem
