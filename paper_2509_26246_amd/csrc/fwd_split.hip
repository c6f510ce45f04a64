// Forward launches whose keys are divided among blocks: when, and the regions for the partial results.
// (FwdSplit in internal.h says why; the forward kernels write the parts and add them up.)
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>

#include "internal.h"

// Who owns each region of the current device (zero at load: nobody), and the regions themselves.  Arrays built into the library, like the
// scratch of slimattn_bwd_static: one set per GPU the library runs on, held until the process ends, so that no handle pays for
// them.  (Allocated with the first handle and freed with the last, create and destroy of a 65536-token handle
// took 502 us, 173 now.)
static __device__ slimattn::SplitState split_state;
static __device__ __align__(256) float split_data[slimattn::kSplitRegions * slimattn::kSplitRegionFloats];

namespace slimattn {
int& last_hip_error();

namespace {

__global__ void split_claim_kernel(SplitState* state, unsigned long long ticket) {
  if (threadIdx.x != 0) return;
  for (int r = 0; r < kSplitRegions; ++r)
    if (atomicCAS(&state->owner[r], 0ull, ticket) == 0ull) {
      atomicExch(&state->done[r], 0u);
      return;
    }
}

__global__ void split_abandon_kernel(SplitState* state, unsigned long long ticket) {
  if (threadIdx.x < kSplitRegions) atomicCAS(&state->owner[threadIdx.x], ticket, 0ull);
}

constexpr int kMaxDevices = 64;
float* g_data[kMaxDevices] = {};
SplitState* g_state[kMaxDevices] = {};
std::mutex g_mutex;
std::atomic<unsigned long long> g_ticket{1};

}  // namespace

int prepare_split_regions() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return 0;             // launches on it are not divided
  std::lock_guard<std::mutex> lock(g_mutex);
  if (g_data[dev]) return 0;
  void *d = nullptr, *s = nullptr;
  e = hipGetSymbolAddress(&s, HIP_SYMBOL(split_state));
  if (e == hipSuccess) e = hipGetSymbolAddress(&d, HIP_SYMBOL(split_data));
  if (e != hipSuccess) {
    (void)hipGetLastError();                               // launches report only their own errors
    return (int)e;
  }
  g_state[dev] = (SplitState*)s;
  g_data[dev] = (float*)d;
  return 0;
}

// As many parts as one round of blocks holds, of at least kMinPartTiles key tiles, if that is the faster way.  A tile takes about
// 1.15 us while most compute units idle and 1.65 us when all work; claim and adding up were taken at 20 us, and up to 25 more for
// writing and reading a full region (they take less since).  Measured, undivided -> divided: 1024 rows of 8/1 heads after 31K keys
// (8 parts) 569 -> 129 us, 256 rows after 7.9K 150 -> 39, after 2.8K (3 parts) 61 -> 35; 512 rows of 32/8 heads after 3.6K (4 parts)
// 82 -> 59.  With 1024 rows of 32/8 heads only two parts fit: after 3K and 7K keys they stay undivided (82, 157 us), after 31K
// 607 -> 459.
int split_begin(const LaunchCtx& c, int n_items, int divide_rows, FwdSplit* sp) {
  constexpr int kMinPartTiles = 16;
  *sp = FwdSplit{nullptr, nullptr, 0, 1, 1};
  if (divide_rows < kSplitMinRows) return 0;
  const int tiles = divide_rows / 64;
  const int64_t fit = kSplitUnits / ((int64_t)n_items * c.p->n_q_heads);
  const int parts = (int)(fit < tiles / kMinPartTiles ? fit : tiles / kMinPartTiles);
  if (parts < 2) return 0;
  const float fill = (float)(n_items * c.p->n_q_heads * parts) / kSplitUnits;
  if (1.15f * tiles <= tiles / parts * (1.15f + 0.5f * fill) + 20.f + 25.f * fill) return 0;
  int dev = -1;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return 0;
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!g_data[dev]) return 0;
    *sp = FwdSplit{g_data[dev], g_state[dev], g_ticket.fetch_add(1), parts, (tiles + parts - 1) / parts};
  }
  hipLaunchKernelGGL(split_claim_kernel, dim3(1), dim3(64), 0, (hipStream_t)c.stream, sp->state, sp->ticket);
  return (int)hipGetLastError();
}

void split_abandon(const LaunchCtx& c, const FwdSplit& sp) {
  if (sp.parts < 2) return;
  hipLaunchKernelGGL(split_abandon_kernel, dim3(1), dim3(64), 0, (hipStream_t)c.stream, sp.state, sp.ticket);
  (void)hipGetLastError();                                 // the caller reports the error that led here
}

}  // namespace slimattn

using namespace slimattn;

extern "C" int slimattn_fwd_divided_counts(int64_t* counts) {
  if (!counts) return SLIMATTN_EINVAL;
  SplitState now;
  hipError_t e = (hipError_t)prepare_split_regions();
  if (e == hipSuccess) e = hipMemcpyFromSymbol(&now, HIP_SYMBOL(split_state), sizeof(now));
  if (e != hipSuccess) {
    last_hip_error() = (int)e;
    return SLIMATTN_EHIP;
  }
  counts[0] = (int64_t)now.launches[0];
  counts[1] = (int64_t)now.launches[1];
  counts[2] = 0;
  for (unsigned long long owner : now.owner) counts[2] += owner != 0;
  return SLIMATTN_OK;
}
