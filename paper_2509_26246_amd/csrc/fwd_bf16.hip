// Forward, bf16 inputs, MFMA products with fp32 accumulation, fp32 online softmax: the kernel with one head per block and
// several blocks per compute unit (head dim 64, odd numbers of query heads per KV head, packs of short samples; the rest
// runs the one-wave kernel of fwd_wide_bf16.hip).
//
// What it computes (paper: PackFlow section -- a slice's queries attend to the cached keys and
// values of every earlier slice of the sample and causally to the slice itself): for a query tile
// of 128 rows of one head, walk the sample's keys kv_start .. last row in tiles of 64, keep a
// running reference and row sum, and accumulate O.
//
// Shape of the computation on CDNA4: the block's 4 waves own 32 query rows each; two blocks (head dim 128, 201 registers; 224
// with exact row sums) or three (64, 137) share a compute unit, so one wave's softmax overlaps another's products and one block's loads and stores
// another's tiles.  Scores are produced transposed, S^T = K Q^T (A = K rows from LDS, B = Q held in registers), so that every
// lane owns one query row: row sums need a cross-lane exchange once per item and the
// accumulator registers of S^T are, as they stand, the B operand of O^T += V^T P^T.  V^T is read
// from the row-major V tile with LDS transpose loads.  K and V tiles are double-buffered in LDS and
// filled by direct global->LDS loads issued one tile ahead; operand fragments are read from LDS a
// few products ahead of their use.
//
// Bound by the vector unit (at 64: 16 products of 32 cycles per wave and tile against 32 exponentials and 80 other vector
// instructions), so the tile has none it can do without: the first product of a score accumulator takes minus the reference
// as its C operand, and the reference moves by a test on the row sums instead of a row maximum.  Both together, 32/8 heads at
// head dim 64, 16K-row sample: 1094 -> 1017 us, 4K-row samples 296 -> 278; odd groups at 128: 4K-row samples 594 -> 548.  A fourth
// block per compute unit (128 registers) spills: 1124.  A kernel with two groups of four waves in opposite phases, which
// head dim 64 had before, took 1083 and 328 (and 144 against 93 on 1K-row samples).  Output rows leave through LDS: on a
// short-sample pack of 32/32 heads 184 -> 168.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "mfma_utils.h"

namespace slimattn {
namespace {

constexpr int kFwdBQ = 128;   // query rows per block: 4 waves x 32 rows
constexpr int kFwdBK = 64;    // keys per step
template <int D> constexpr int kFwdLdsBytes = 4 * kFwdBK * D * 2;   // K and V tiles, two buffers of each
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLazySum = 4096.f;   // the reference moves when a lane's sum of the 32 probabilities of a tile exceeds this

// One 64-key tile for this wave's 32 query rows.  MASKED tiles touch the diagonal.
// pk[ks]: this lane's K-fragment address for key block 0 and head-dim step ks; pv[db][0..1]: its
// V^T-fragment address pair for head-dim block db; both already point into the current buffer.
// qf holds q * scale * log2(e), so the products are scores in log2 units; the accumulators start
// at minus the row's reference (every register of negm), so they come out as the exponents directly.
// EXACT: the row sum adds the probabilities before they are rounded to bf16 for the product, in the order of the one-wave kernel
// (packs of short samples at head dim 128, even groups: their rows get the lse that kernel gives).  Otherwise it adds the rounded
// ones with dot products, half the instructions.
template <int D, bool MASKED, bool EXACT, class Side>
__device__ __forceinline__ void fwd_tile(const lds_cptr (&pk)[D / 16], const lds_cptr (&pv)[D / 32][2],
                                         const bf16x8 (&qf)[D / 16], floatx16 (&oacc)[D / 32], floatx16& negm, float& l_run,
                                         int rel, Side&& side) {
  constexpr int NKS = D / 16, NDB = D / 32, kRowBytes = D * 2;
  floatx16 sacc[2];
  // S^T = K Q^T (minus the reference maximum)
  // (the next tile's global->LDS loads are issued one at a time between the products)
  frag_pipeline_side<2 * NKS, 4>([&](int i) { return lds_ld_row(pk[i % NKS], (i / NKS) * 32 * kRowBytes); },
                                 [&](int i, bf16x8 f) { sacc[i / NKS] = mfma32(f, qf[i % NKS], i % NKS == 0 ? negm : sacc[i / NKS]); }, side);
  if (MASKED) {      // key (j0 + 32b + 8(r/4) + 4 half + r%4) > row  <=>  32b + 8(r/4) + r%4 > rel
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (32 * b + 8 * (r >> 2) + (r & 3) > rel) sacc[b][r] = -INFINITY;
  }
  bf16x8 pf[4];
  float lb[2];                                    // row sums of the two key blocks
  // probabilities against the reference as it stands (`shift` below it), their row sums
  auto probabilities = [&](float shift) {
    float ps[4];
#pragma unroll
    for (int ks2 = 0; ks2 < 4; ++ks2) {
      floatx8 e;
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_exp2f(sacc[ks2 >> 1][8 * (ks2 & 1) + i] - shift);
      pf[ks2] = __builtin_convertvector(e, bf16x8);
      if constexpr (EXACT) {
        float& l = lb[ks2 >> 1];
        l = ks2 & 1 ? l + e[0] : e[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) l += e[i];
      } else {
        ps[ks2] = sum8(pf[ks2], 0.f);
      }
    }
    if constexpr (!EXACT) { lb[0] = ps[0] + ps[1]; lb[1] = ps[2] + ps[3]; }
  };
  probabilities(0.f);
  // Lazy rescaling: the reference only moves when some lane's sum of its 32 probabilities exceeds kLazySum (so no single one
  // does; an overflow to inf does; wave-uniform test): the test costs one comparison where a row maximum costs 16 instructions
  // and a cross-lane exchange.  O / l is unaffected.  The reference starts at the row's score against the sample's first key
  // (always visible), so a row's sum cannot underflow (a part of a divided walk may come to a sum of 0).
  if (__builtin_expect(__any(lb[0] + lb[1] > kLazySum), 0)) {
    float mx = sacc[0][0];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[b][r]);
    // (Every row of the wave with a score above its reference moves along, so where references move a row's last bits depend on the
    // rows of its query tile.  Moving only the rows that asked for it takes many more moves where scores climb at different rates:
    // 4096-row samples of 32/8 heads on the one-wave kernel, climbs of up to 20 nats 555 -> 777 us, of 100 641 -> 1055.)
    const float shift = fmaxf(fmaxf(mx, xor32(mx)), 0.f);
    const float alpha = __builtin_amdgcn_exp2f(-shift);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    probabilities(shift);
    const float m = negm[0] - shift;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = m;
    asm volatile("" : "+v"(negm));
  }
  if constexpr (EXACT) { l_run += lb[0]; l_run += lb[1]; }
  else l_run += lb[0] + lb[1];
  // O^T += V^T P^T: one batch of four V^T fragments (the four 16-key steps) per head-dim block
  Tr4 tb[NDB];
  constexpr int kStep = 16 * kRowBytes;
  tr4_issue<0, kStep, 2 * kStep, 3 * kStep>(pv[0][0], pv[0][1], tb[0]);
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    if (db + 1 < NDB) tr4_issue_wait<0, kStep, 2 * kStep, 3 * kStep>(pv[db + 1][0], pv[db + 1][1], tb[db + 1], tb[db]);
    else tr4_wait(tb[db]);
#pragma unroll
    for (int j = 0; j < 4; ++j) oacc[db] = mfma32(tr4_frag(tb[db], j), pf[j], oacc[db]);
  }
}

// The walk of one wave: rows q0w .. min(q0w + 32, q_end) - 1 of head h, over n_tiles key tiles from kv_start on, up to row q_end - 1.
// first_key: of the sample.  Leaves O^T, the reference (log2 units) and the row sum of this thread's row; all of the block's
// threads are behind a barrier and done with the LDS.
template <int D, bool EXACT>
__device__ __forceinline__ void fwd_walk(LDS_PTR(char) lds, const bf16* __restrict__ q, const bf16* __restrict__ k,
                                         const bf16* __restrict__ v, int q0w, int q_end, int first_key, int kv_start, int n_tiles,
                                         int h, int hk, int Hq, int Hkv, float scale, floatx16 (&oacc)[D / 32], float& m_ref, float& l_tot) {
  constexpr int NKS = D / 16;   // contraction steps over the head dimension
  constexpr int NDB = D / 32;   // 32-wide blocks of the head dimension
  constexpr int kTileBytes = kFwdBK * D * 2, kBufBytes = 2 * kTileBytes;   // LDS: [buffer][K tile, V tile]
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int my_row = q0w + l32;                   // the query row this lane owns

  const TileSource srcK = make_tile_source<D, 256>(k, kv_start, Hkv, hk, q_end, tid);
  const TileSource srcV = make_tile_source<D, 256>(v, kv_start, Hkv, hk, q_end, tid);
  stage_tile<D, kFwdBK, 256>(lds, srcK, 0, tid);
  stage_tile<D, kFwdBK, 256>(lds + kTileBytes, srcV, 0, tid);

  bf16x8 qf[NKS];
  {
    const bf16* qp = q + ((size_t)min(my_row, q_end - 1) * Hq + h) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = scale8(*reinterpret_cast<const bf16x8*>(qp + 16 * ks), scale * kLog2e);
  }
  lds_cptr pk[NKS], pv[NDB][2];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) pk[ks] = lds_row_ptr<D>(lds, l32, 16 * ks + 8 * half);
#pragma unroll
  for (int db = 0; db < NDB; ++db) lds_tr_ptrs<D>(lds + kTileBytes, 32 * db, lane, pv[db][0], pv[db][1]);
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  // reference (log2 units): the row's score against the first key of the sample, for every part of a divided walk.  (A part's own
  // first key may be one that takes no part in the softmax, of a score far below the others or -inf: the part's scores would
  // be lost under such a reference.)
  float l_run = 0.f;
  m_ref = 0.f;
  {
    const bf16* kp = k + ((size_t)first_key * Hkv + hk) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const bf16x8 k0 = *reinterpret_cast<const bf16x8*>(kp + 16 * ks);
      if constexpr (EXACT) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {             // (as the one-wave kernel forms it)
          const bf16x2 a2 = {qf[ks][2 * x], qf[ks][2 * x + 1]}, b2 = {k0[2 * x], k0[2 * x + 1]};
          m_ref = __builtin_amdgcn_fdot2_f32_bf16(a2, b2, m_ref, false);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) m_ref = fmaf((float)qf[ks][e], (float)k0[e], m_ref);
      }
    }
    m_ref += xor32(m_ref);
  }
  floatx16 negm;                                  // minus the reference in every register: the C operand of a tile's first products
#pragma unroll
  for (int r = 0; r < 16; ++r) negm[r] = -m_ref;
  asm volatile("" : "+v"(negm));                  // kept in registers, not rebuilt at every use
  __builtin_amdgcn_s_waitcnt(0);                  // tile 0 has landed in LDS
  __syncthreads();

  for (int t = 0; t < n_tiles; ++t) {
    const int j0 = kv_start + t * kFwdBK;
    // next tile straight into the other buffer (its last readers passed the barrier below); past
    // the end of the tensor the loads return zeros that nobody uses.  kPasses loads per tensor,
    // spread over the first products of the tile.
    const int nb = ((t + 1) & 1) * kBufBytes;
    constexpr int kPasses = kFwdBK * D * 2 / 256 / 16;
    auto side = [&](int i) {
      if (i < kPasses) stage_pass<D, 256>(lds + nb, srcK, (t + 1) * kFwdBK, i, tid);
      else if (i < 2 * kPasses) stage_pass<D, 256>(lds + nb + kTileBytes, srcV, (t + 1) * kFwdBK, i - kPasses, tid);
    };
    const int rel = my_row - j0 - 4 * half;
    if (j0 + kFwdBK - 1 <= q0w) {                  // whole tile visible to every row of the wave
      fwd_tile<D, false, EXACT>(pk, pv, qf, oacc, negm, l_run, rel, side);
    } else if (j0 <= q0w + 31) {                   // diagonal region
      fwd_tile<D, true, EXACT>(pk, pv, qf, oacc, negm, l_run, rel, side);
    } else {                                       // nothing visible to this wave: only fetch
#pragma unroll
      for (int i = 0; i < 2 * kPasses; ++i) side(i);
    }
    const int flip = (t & 1) ? -kBufBytes : kBufBytes;   // fragment addresses follow the buffer switch
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) pk[ks] += flip;
#pragma unroll
    for (int db = 0; db < NDB; ++db) { pv[db][0] += flip; pv[db][1] += flip; }
    __builtin_amdgcn_s_waitcnt(0);                // this thread's direct loads have landed
    __syncthreads();
  }

  m_ref = -negm[0];
  l_tot = l_run + xor32(l_run);
}

// Rows of the wave out: O = O^T / l through LDS, lse.
template <int D>
__device__ __forceinline__ void fwd_out(LDS_PTR(char) lds, const floatx16 (&oacc)[D / 32], float m_ref, float l_tot, bf16* __restrict__ o,
                                        float* __restrict__ lse, int q0w, int q_end, int h, int T, int Hq) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, my_row = q0w + (lane & 31);
  // (the tile buffers are free behind the walk's last barrier; each wave uses a part of its own)
  static_assert(4 * kOutAreaBytes<D> <= kFwdLdsBytes<D>, "the transposition areas must fit the tile buffers");
  store_rows<D>(lds + __builtin_amdgcn_readfirstlane(wave) * kOutAreaBytes<D>, oacc, 1.f / l_tot, o, Hq, h, q0w, q_end, lane);
  if (lane < 32 && my_row < q_end) lse[(size_t)h * T + my_row] = (m_ref + __builtin_amdgcn_logf(l_tot)) * kLn2;
}

template <int D, bool EXACT>
__global__ __launch_bounds__(256, 2) void fwd_bf16_kernel(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                          const bf16* __restrict__ v, bf16* __restrict__ o,
                                                          float* __restrict__ lse, const QItem* __restrict__ items,
                                                          QBlocks n_items, int T, int Hq, int Hkv, float scale) {
  __shared__ __attribute__((aligned(1024))) char smem[kFwdLdsBytes<D>];
  const int g = Hq / Hkv;
  int item_idx, hk, hg, share;
  if (!map_shared_block(blockIdx.x, g, Hkv, n_items, &item_idx, &hk, &hg, &share)) return;
  const QItem it = items[item_idx];
  const int wave = threadIdx.x >> 6, h = __builtin_amdgcn_readfirstlane(hk * g + hg + (wave >> (2 - share)));
  const int q0w = it.q_row0 + 32 * (wave & (3 >> share)), q_end = it.q_row0 + it.q_rows;
  floatx16 oacc[D / 32];
  float m, l;
  fwd_walk<D, EXACT>((LDS_PTR(char))smem, q, k, v, q0w, q_end, it.kv_start, it.kv_start,
                     (q_end - it.kv_start + kFwdBK - 1) / kFwdBK, h, hk, Hq, Hkv, scale, oacc, m, l);
  fwd_out<D>((LDS_PTR(char))smem, oacc, m, l, o, lse, q0w, q_end, h, T, Hq);
}

// The launch whose items' keys are divided: one block per (item, head, part), parts innermost, so that an XCD keeps to the same runs
// of keys; then the heads that share them.
template <int D, bool EXACT>
__global__ __launch_bounds__(256, 2) void fwd_bf16_split_kernel(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                                const bf16* __restrict__ v, bf16* __restrict__ o,
                                                                float* __restrict__ lse, const QItem* __restrict__ items, int T,
                                                                int Hq, int Hkv, float scale, FwdSplit sp) {
  __shared__ __attribute__((aligned(1024))) char smem[kFwdLdsBytes<D>];
  const int part = blockIdx.x % sp.parts, g = Hq / Hkv;
  int item_idx, hk, hg;
  split_block(blockIdx.x / sp.parts, g, Hkv, &item_idx, &hk, &hg);
  QItem it = items[item_idx];
  const int first_key = it.kv_start, q_end = it.q_row0 + it.q_rows, h = hk * g + hg, n = split_parts(sp, it);
  if (part >= n) return;
  const int region = n > 1 ? split_region(sp) : 0;
  if (region < 0) return;                         // the finishing kernel walks the parts
  const int n_tiles = split_range(it, part, n), q0w = it.q_row0 + 32 * (int)(threadIdx.x >> 6);
  floatx16 oacc[D / 32];
  float m, l;
  fwd_walk<D, EXACT>((LDS_PTR(char))smem, q, k, v, q0w, q_end, first_key, it.kv_start, n_tiles, h, hk, Hq, Hkv, scale, oacc, m, l);
  if (n > 1)
    split_store<D>(split_unit<D>(sp, region, (item_idx * sp.parts + part) * Hq + h), threadIdx.x >> 6, threadIdx.x & 63, oacc, m, l);
  else
    fwd_out<D>((LDS_PTR(char))smem, oacc, m, l, o, lse, q0w, q_end, h, T, Hq);
}

// Adds the parts up, grid (items, heads, head-dim blocks).  Without a region the blocks of the first head-dim block walk them, with the
// sums of the parts so far in LDS.
template <int D, bool EXACT>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void fwd_bf16_finish_kernel(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                                 const bf16* __restrict__ v, bf16* __restrict__ o,
                                                                 float* __restrict__ lse, const QItem* __restrict__ items, int T,
                                                                 int Hq, int Hkv, float scale, FwdSplit sp) {
  __shared__ __attribute__((aligned(1024))) char smem[kFwdLdsBytes<D> + kFwdBQ * D * 4];
  const QItem it = items[blockIdx.x];
  const int n = split_parts(sp, it), region = split_region(sp);
  if (n > 1 && region >= 0) {
    split_combine<D>(sp, region, n, it, o, lse, T, Hq);
  } else if (n > 1 && blockIdx.z == 0) {
    const int h = blockIdx.y, q_end = it.q_row0 + it.q_rows, q0w = it.q_row0 + 32 * (int)(threadIdx.x >> 6);
    LDS_PTR(floatx4) sum = (LDS_PTR(floatx4))(smem + kFwdLdsBytes<D>) + threadIdx.x;     // D / 8 vectors of a row, 256 apart
    floatx16 oacc[D / 32];
    float m = 0.f, l = 0.f;
    for (int part = 0; part < n; ++part) {
      QItem run = it;
      const int n_tiles = split_range(run, part, n);
      float mp, lp;
      fwd_walk<D, EXACT>((LDS_PTR(char))smem, q, k, v, q0w, q_end, it.kv_start, run.kv_start, n_tiles, h, h / (Hq / Hkv), Hq, Hkv,
                         scale, oacc, mp, lp);
      const bool first = part == 0;
      if (first) m = mp;
      const SplitAdd add(m, l, mp, lp);
      if (first) l = lp;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          floatx4 x = sum[(db * 4 + gq) * 256];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = oacc[db][4 * gq + e] = first ? oacc[db][4 * gq + e] : add(x[e], oacc[db][4 * gq + e]);
          sum[(db * 4 + gq) * 256] = x;
        }
    }
    fwd_out<D>((LDS_PTR(char))smem, oacc, m, l, o, lse, q0w, q_end, h, T, Hq);
  }
  split_release(sp, region);
}

}  // namespace

int fwd_q_tile(int dtype, int) { return dtype == SLIMATTN_F32 ? 64 : kFwdBQ; }

namespace {
template <int D, bool EXACT>
int launch_fwd_one_head(const LaunchCtx& c, const void* q, const void* k, const void* v, void* o, float* lse, const QList& list, const FwdSplit& sp) {
  const slimattn_params& p = *c.p;
  const int g = p.n_q_heads / p.n_kv_heads, n_items = list.n;
  const bool shared = sp.parts == 1 && shares_heads(list, g);
  const QItem* items = shared ? list.grouped : list.items;
  const dim3 block(256);
  if (sp.parts > 1) {
    hipLaunchKernelGGL((fwd_bf16_split_kernel<D, EXACT>), dim3((unsigned)(n_items * p.n_q_heads * sp.parts)), block, 0, (hipStream_t)c.stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, items, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale, sp);
    const int e = (int)hipGetLastError();
    if (e != 0) return e;
    hipLaunchKernelGGL((fwd_bf16_finish_kernel<D, EXACT>), dim3((unsigned)n_items, (unsigned)p.n_q_heads, split_finish_z(n_items, p.n_q_heads, D)), block, 0,
                       (hipStream_t)c.stream, (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, items, (int)c.T, p.n_q_heads,
                       p.n_kv_heads, p.scale, sp);
    return (int)hipGetLastError();
  }
  return in_runs(n_items, p.n_q_heads, [&](int first, int n) {
    const QBlocks run = shared_blocks(shared && n == n_items ? list.groups : QGroups::plain(n), p.n_kv_heads, g);
    hipLaunchKernelGGL((fwd_bf16_kernel<D, EXACT>), dim3((unsigned)run.end[2]), block, 0,
                       (hipStream_t)c.stream, (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, items + first, run, (int)c.T,
                       p.n_q_heads, p.n_kv_heads, p.scale);
    return (int)hipGetLastError();
  });
}
}  // namespace

// Even groups at head dim 128 go to the one-wave kernel, whose tiles are cheaper, unless the pack's samples are short: it
// holds one block per compute unit, and what an item costs beside its tiles (11 us of loads and stores) is hidden by nothing, while
// two blocks of this kernel overlap each other.  Both cost a row about the same amount plus a share per key, so what
// decides over a pack is the keys its rows see on average, whatever the lengths it is mixed from.  32/8 heads, one-wave kernel
// against this one: 16K tokens in equal samples of 128 rows 104 / 84 us, 512 rows 137 / 119, 800 rows (400 keys) 167 / 161, 1024
// rows 175 / 166, 2048 rows 263 / 277; one of 4096 rows among 200 of 100 (390 keys) 245 / 226, of 3000 among 45 of 300 (395) 184 /
// 166; with 8/1 heads these two 98 / 72 and 78 / 55.  By units of 4096 tokens 128 rows 116 / 106, 800 rows 186 / 174; where the units' blocks
// just fill the chip's rounds, 512 rows 140 / 147.  Every launch of a handle takes the same kernel.  (At head dim 64 this
// kernel is bound by the vector unit, where a second head per wave saves nothing.)
constexpr int kShortMeanKeys = 400;

int launch_fwd_bf16(const LaunchCtx& c, const void* q, const void* k, const void* v, void* o, float* lse, const QList& list, int divide_rows) {
  if (list.n == 0) return 0;
  const slimattn_params& p = *c.p;
  const bool even = p.n_q_heads / p.n_kv_heads % 2 == 0;
  FwdSplit sp;
  int e = split_begin(c, list.n, divide_rows, &sp);
  if (e == 0) {
    if (p.head_dim == 64) e = launch_fwd_one_head<64, false>(c, q, k, v, o, lse, list, sp);
    else if (!even) e = launch_fwd_one_head<128, false>(c, q, k, v, o, lse, list, sp);
    else if (c.mean_keys > kShortMeanKeys) e = launch_fwd_wide_bf16(c, q, k, v, o, lse, list.items, list.n, sp);
    else e = launch_fwd_one_head<128, true>(c, q, k, v, o, lse, list, sp);
  }
  if (e != 0) split_abandon(c, sp);
  return e;
}

}  // namespace slimattn
