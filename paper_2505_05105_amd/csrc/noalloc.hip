// Allocation-free form of the misfit call: J = 1/2 e^T M e and dJ/du = M e
// with e = u - u_t on the active nodes, every scratch value of the call (the
// per-block partial sums) in one static device array instead of memory the
// library allocates, so that callers that must not allocate (code under HIP
// graph capture, tight serving loops) can evaluate the objective.
//
// The array `scratch` exists once per device for the life of the process.
// Host code never passes its name to a kernel: set-up (the first
// mgfem_setup on a device) asks the runtime for its device address with
// hipGetSymbolAddress and keeps it per device; the kernels get that address.
// Every call on one device shares the array, and each call overwrites all of
// it that it reads (one partial per block of its grid), so nothing has to be
// cleared between calls; calls that overlap on one device race.
#include <mutex>

#include "mgfem_internal.h"

namespace {
constexpr size_t kScratchBytes = size_t(2) << 20;  // 2 MiB per device
}  // namespace

// the scratch of mgfem_misfit_noalloc (see the top of this file)
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace mgfem {
namespace {

constexpr int kMaxDevices = 64;

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
bool g_scratch_tried[kMaxDevices] = {};

// a block takes 256 x 8 nodes; e is staged in LDS with a halo of one (zero off
// the grid and at inactive nodes)
constexpr int kMX = 256, kMY = 8, kMW = kMX + 2, kMH = kMY + 2, kMN = kMW * kMH;

// dJ/du = M e at every node of the block (0 at inactive nodes and off the box
// of active nodes) and the block's share of e^T M e in part[stride block]
// (stride 2: in part[2 block + 1], with 0 beside it, for the pair reduction).
// Rows: the gathered M row at a cut-cell vertex (cut_rows, 18 per vertex in
// cut-list order, M first), the stored planes at any other stored row, the
// interior Q1 mass stencil h^2/36 [1 4 1; 4 16 4; 1 4 1] elsewhere.  Bound by
// its bytes: u, u_t and a flag per node of the box, dJ/du on the whole grid;
// every load of a block is issued before the first is used (none under a
// branch: a node off the grid loads a clamped one and drops it).  The stored
// rows of a wave's nodes are listed first and then taken one per lane, with
// all nine coefficients in flight: row by row, each node with its nine loads
// behind branches, N = 2048 took 30 us, like this 17.
__global__ __launch_bounds__(256) void k_misfit_partial(const double* __restrict__ u, const double* __restrict__ ut,
                                                        const uint8_t* __restrict__ fl, const int* __restrict__ cutpos,
                                                        const double* __restrict__ cut_rows,
                                                        const double* __restrict__ M, double* __restrict__ y, int N,
                                                        double hh36, int i0, int j0, int i1, int j1,
                                                        double* __restrict__ part, int stride) {
  constexpr int NU = (kMN + 255) / 256;
  __shared__ double se[NU * 256];
  __shared__ uint8_t sf[NU * 256];
  __shared__ double wsum[4];
  __shared__ uint16_t list[4][64 * kMY];  // a wave's stored nodes, by row, as indices of se
  const int s = N + 1, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t n = (int64_t)s * s;
  const int bi = blockIdx.x * kMX, bj = blockIdx.y * kMY;
  const bool touches = bi <= i1 && bi + kMX - 1 >= i0 && bj <= j1 && bj + kMY - 1 >= j0;  // uniform
  if (touches) {
    double ru[NU], rt[NU];
    uint8_t rf[NU];
#pragma unroll
    for (int w = 0; w < NU; ++w) {
      const int q = min((int)threadIdx.x + w * 256, kMN - 1);
      const int gi = min(max(bi - 1 + q % kMW, 0), N), gj = min(max(bj - 1 + q / kMW, 0), N);
      const int64_t k = gi + (int64_t)gj * s;
      rf[w] = fl[k];
      ru[w] = u[k];
      rt[w] = ut[k];
    }
#pragma unroll
    for (int w = 0; w < NU; ++w) {
      const int q = threadIdx.x + w * 256;
      const int gi = bi - 1 + q % kMW, gj = bj - 1 + q / kMW;
      const bool in = q < kMN && gi >= 0 && gj >= 0 && gi <= N && gj <= N && (rf[w] & kFlagActive);
      se[q] = in ? ru[w] - rt[w] : 0.0;
      sf[q] = in ? rf[w] : (uint8_t)0;
    }
    __syncthreads();
  }
  double sm = 0.0;
  const int i = bi + threadIdx.x;
  int nst = 0;
#pragma unroll
  for (int rep = 0; rep < kMY; ++rep) {
    const int j = bj + rep;
    const bool in = i <= N && j <= N;
    double me = 0.0;
    bool stored = false;
    if (touches) {
      const int q = threadIdx.x + 1 + (rep + 1) * kMW;
      const uint8_t fk = sf[q];  // 0 off the grid
      stored = (fk & kFlagActive) && (fk & kFlagStored);
      const unsigned long long m = __ballot(stored);
      if (stored) list[wave][nst + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)q;
      nst += __popcll(m);
      if ((fk & kFlagActive) && !stored) {
        const double corners = (se[q - kMW - 1] + se[q - kMW + 1]) + (se[q + kMW - 1] + se[q + kMW + 1]);
        const double edges = (se[q - kMW] + se[q + kMW]) + (se[q - 1] + se[q + 1]);
        me = hh36 * (16.0 * se[q] + 4.0 * edges + corners);
        sm += se[q] * me;
      }
    }
    if (y && in && !stored) y[i + (int64_t)j * s] = me;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the wave's own list
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int e = lane; e < nst; e += 64) {
    const int q = list[wave][e];
    const int64_t k = bi - 1 + q % kMW + (int64_t)(bj - 1 + q / kMW) * s;
    const bool cut = (sf[q] & kFlagCut) != 0;
    const double* row = cut ? cut_rows + 18 * (int64_t)cutpos[k] : M + k;
    const int64_t st = cut ? 1 : n;
    double m[9], me = 0.0;
#pragma unroll
    for (int p = 0; p < 9; ++p) m[p] = row[p * st];
    // zero coefficients are skipped, so that a value without a share in the row has none
#pragma unroll
    for (int p = 0; p < 9; ++p) {
      const double v = se[q + (p % 3 - 1) + (p / 3 - 1) * kMW];
      me += m[p] != 0.0 ? m[p] * v : 0.0;
    }
    sm += se[q] * me;
    if (y) y[k] = me;
  }
  for (int o = 32; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  if (lane == 0) wsum[wave] = sm;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int b = blockIdx.x + blockIdx.y * gridDim.x;
    if (stride == 2) part[2 * b] = 0.0;
    part[stride * b + stride - 1] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
  }
}

// sum of the block partials in a fixed order, written to pinned host memory
__global__ __launch_bounds__(1024) void k_misfit_final(const double* __restrict__ part, int nb, double* host_rec) {
  __shared__ double wsum[16];
  double sm = 0.0;
  for (int t = threadIdx.x; t < nb; t += blockDim.x) sm += part[t];
  for (int o = 32; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sm;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += wsum[w];
    host_rec[0] = t;
    __threadfence_system();
  }
}

}  // namespace

int launch_misfit(mgfem_ctx* c, const double* u, const double* ut, double* dJdu, double* part, int stride) {
  const Level& L = c->lv[0];
  const int N = c->N;
  const dim3 grid((unsigned)((N + kMX) / kMX), (unsigned)((N + kMY) / kMY));  // (N+1) nodes per side
  // a gradient over one of its inputs (blocks still read what others would have
  // written) goes through the handle's scratch
  auto meets = [&](const double* p) { return dJdu && dJdu < p + L.n && p < dJdu + L.n; };
  double* y = meets(u) || meets(ut) ? c->F64tmp : dJdu;
  hipLaunchKernelGGL(k_misfit_partial, grid, dim3(256), 0, c->s, u, ut, (const uint8_t*)L.flags,
                     (const int*)L.cutpos, (const double*)c->cut_rows, (const double*)c->M, y, N,
                     c->h * c->h / 36.0, L.bbox[0], L.bbox[2], L.bbox[1], L.bbox[3], part, stride);
  if (y != dJdu) launch_copy(c, dJdu, y, L.n);
  return (int)(grid.x * grid.y);
}

int scratch_init(int* device) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return MGFEM_ERR_HIP;
  }
  *device = dev;
  if (dev < 0 || dev >= kMaxDevices) return MGFEM_OK;  // the no-allocation call reports it
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_tried[dev]) {
    g_scratch_tried[dev] = true;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e == hipSuccess) g_scratch_ptr[dev] = p;
    else (void)hipGetLastError();
  }
  return MGFEM_OK;
}

}  // namespace mgfem

using namespace mgfem;

extern "C" {

int mgfem_misfit_noalloc(mgfem_handle c, const double* u_dev, const double* ut_dev, double* J_host,
                         double* dJdu_dev) {
  if (!c) return MGFEM_ERR_INVALID_ARG;
  if (c->batched_member || !c->members.empty() || c->lv.empty()) {
    c->last_error = "batched handle: use mgfem_solve_batched";
    return MGFEM_ERR_INVALID_ARG;
  }
  if (!u_dev || !ut_dev || !J_host) {
    c->last_error = "u, ut and J must be given";
    return MGFEM_ERR_INVALID_ARG;
  }
  void* base = nullptr;
  if (c->device >= 0 && c->device < kMaxDevices) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    base = g_scratch_ptr[c->device];
  }
  if (!base) {
    c->last_error = "the static scratch array has no device address on device " + std::to_string(c->device);
    return MGFEM_ERR_HIP;
  }
  const int N = c->N;
  // the documented limit: one value per 256 x 4 nodes (the pass takes half of that)
  const int64_t nb = (int64_t)((N + 256) / 256) * ((N + 4) / 4);
  if (nb * (int64_t)sizeof(double) > (int64_t)kScratchBytes) {
    c->last_error = "N = " + std::to_string(N) + ": 8 bytes per 256 x 4 nodes, " +
                    std::to_string(nb * sizeof(double)) + ", are more than the limit of " +
                    std::to_string(kScratchBytes) + " bytes (every N below 16384 is within it)";
    return MGFEM_ERR_INVALID_ARG;
  }
  double* part = static_cast<double*>(base);
  double* rec = c->red_host + 4 * kRedSlots;  // the handle's own pinned record (allocated at set-up)
  rec[0] = 0.0;
  const int blocks = launch_misfit(c, u_dev, ut_dev, dJdu_dev, part, 1);
  hipLaunchKernelGGL(k_misfit_final, dim3(1), dim3(1024), 0, c->s, (const double*)part, blocks, rec);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(c->s);
  if (e != hipSuccess) {
    c->last_error = std::string("mgfem_misfit_noalloc: ") + hipGetErrorString(e);
    return MGFEM_ERR_HIP;
  }
  *J_host = 0.5 * reinterpret_cast<volatile double*>(rec)[0];
  return MGFEM_OK;
}

}  // extern "C"
