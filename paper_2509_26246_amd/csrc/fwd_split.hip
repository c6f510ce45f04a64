// Forward launches whose keys are divided among blocks: claiming a region for the partial results, and adding them up.
// (FwdSplit in internal.h says when and why; the forward kernels write the parts.)
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>

#include "internal.h"
#include "mfma_utils.h"

// Who owns each region of the current device (zero at load: nobody), and the regions themselves.  Arrays built into the library, like the
// scratch of slimattn_bwd_static: one set per GPU the library runs on, held until the process ends, so that no handle pays for
// them.  (Allocated with the first handle and freed with the last, create and destroy of a 65536-token handle
// took 502 us, 173 now.)
struct SplitState { unsigned long long owner[slimattn::kSplitRegions]; unsigned done[slimattn::kSplitRegions]; };
static __device__ SplitState split_state;
constexpr size_t kRegionFloats = (size_t)slimattn::kSplitUnits * slimattn::kSplitUnitFloats<128>;
static __device__ __align__(256) float split_data[slimattn::kSplitRegions * kRegionFloats];

namespace slimattn {
namespace {

constexpr float kLn2 = 0.6931471805599453f;

__global__ void split_claim_kernel(unsigned long long* owner, unsigned long long ticket) {
  if (threadIdx.x == 0) atomicCAS(owner, 0ull, ticket);
}

// grid = (items, heads, head-dim blocks of 32): a wave owns 32 rows, a lane 16 columns of one row.  Bound by reading the
// partial results once; the head-dim blocks give enough blocks to cover that latency (1024 rows x 8 heads in 8 parts: 256 blocks).
template <int D>
__global__ __launch_bounds__(256) void split_combine_kernel(FwdSplit sp, bf16* __restrict__ o, float* __restrict__ lse,
                                                            const QItem* __restrict__ items, int T, int Hq) {
  if (__hip_atomic_load(sp.owner, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != sp.ticket) return;   // the launch ran undivided
  const QItem it = items[blockIdx.x];
  const int h = blockIdx.y, db = blockIdx.z, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int common = (it.q_row0 - it.kv_start) / 64 + 1, n = min(sp.parts, (common + sp.target - 1) / sp.target);
  const int r = 32 * wave + l32;
  if (n > 1 && r < it.q_rows) {
    auto unit = [&](int part) { return sp.data + (size_t)(((int)blockIdx.x * sp.parts + part) * Hq + h) * kSplitUnitFloats<D>; };
    float m = -INFINITY;
    for (int p = 0; p < n; ++p) m = fmaxf(m, unit(p)[128 * D + wave * 64 + l32]);
    float l = 0.f;
    floatx4 sum[4] = {};
#pragma unroll 2
    for (int p = 0; p < n; ++p) {
      const float* u = unit(p);
      const float w = __builtin_amdgcn_exp2f(u[128 * D + wave * 64 + l32] - m);
      l += w * u[128 * D + wave * 64 + 32 + l32];
      const floatx4* at = reinterpret_cast<const floatx4*>(u + wave * 32 * D) + db * 256 + lane;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) sum[gq] += w * at[gq * 64];
    }
    const float inv = 1.f / l;
    bf16* op = o + ((size_t)(it.q_row0 + r) * Hq + h) * D + 32 * db + 4 * half;
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      bf16x4 w;
#pragma unroll
      for (int x = 0; x < 4; ++x) w[x] = (bf16)(sum[gq][x] * inv);
      *reinterpret_cast<bf16x4*>(op + 8 * gq) = w;
    }
    if (db == 0 && half == 0) lse[(size_t)h * T + it.q_row0 + r] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
  // the last block to get here gives the region back
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    if (atomicAdd(sp.done, 1u) == gridDim.x * gridDim.y * gridDim.z - 1) {
      *sp.done = 0u;
      __threadfence();
      atomicExch(sp.owner, 0ull);
    }
  }
}

constexpr int kMaxDevices = 64;
float* g_data[kMaxDevices] = {};
SplitState* g_state[kMaxDevices] = {};
std::mutex g_mutex;
std::atomic<unsigned long long> g_ticket{1};
void* g_streams[kSplitRegions] = {};     // the streams the first regions were given to, in order of first use
int g_n_streams = 0;

int region_of(void* stream) {            // under g_mutex
  for (int i = 0; i < g_n_streams; ++i)
    if (g_streams[i] == stream) return i;
  if (g_n_streams < kSplitRegions) {
    g_streams[g_n_streams] = stream;
    return g_n_streams++;
  }
  return (int)((reinterpret_cast<uintptr_t>(stream) >> 6) % kSplitRegions);
}

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
// 1.15 us while most compute units idle and 1.65 us when all work; claim and combining take 20 us, and up to 25 more for
// writing and reading a full region.  Measured, undivided -> divided: 1024 rows of 8/1 heads after 31K keys (8 parts) 569 ->
// 132 us, 256 rows after 7.9K 147 -> 43, after 2.8K (3 parts) 61 -> 37; 512 rows of 32/8 heads after 3.6K (4 parts) 80 -> 68.
// With 1024 rows of 32/8 heads only two parts fit: 82 -> 108 after 3K keys, 157 -> 156 after 7K (both stay undivided), 583 -> 441
// after 31K.
int split_begin(const LaunchCtx& c, int n_items, int divide_rows, FwdSplit* sp) {
  constexpr int kMinPartTiles = 16;
  *sp = FwdSplit{nullptr, nullptr, nullptr, 0, 1, 1};
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
  const unsigned long long ticket = g_ticket.fetch_add(1);
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (dev < 0 || dev >= kMaxDevices || !g_data[dev]) return 0;
    const int region = region_of(c.stream);
    *sp = FwdSplit{g_data[dev] + region * kRegionFloats, &g_state[dev]->owner[region], &g_state[dev]->done[region], ticket, parts,
                   (tiles + parts - 1) / parts};
  }
  hipLaunchKernelGGL(split_claim_kernel, dim3(1), dim3(64), 0, (hipStream_t)c.stream, sp->owner, ticket);
  return (int)hipGetLastError();
}

int split_combine(const LaunchCtx& c, const FwdSplit& sp, void* o, float* lse, const QItem* items, int n_items) {
  const slimattn_params& p = *c.p;
  const dim3 grid((unsigned)n_items, (unsigned)p.n_q_heads, (unsigned)(p.head_dim / 32)), block(256);
  if (p.head_dim == 128)
    hipLaunchKernelGGL(split_combine_kernel<128>, grid, block, 0, (hipStream_t)c.stream, sp, (bf16*)o, lse, items, (int)c.T, p.n_q_heads);
  else
    hipLaunchKernelGGL(split_combine_kernel<64>, grid, block, 0, (hipStream_t)c.stream, sp, (bf16*)o, lse, items, (int)c.T, p.n_q_heads);
  return (int)hipGetLastError();
}

}  // namespace slimattn
