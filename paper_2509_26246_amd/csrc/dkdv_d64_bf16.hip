// dK/dV for bf16 inputs at head dim 64: 256 key rows per block, two waves per SIMD, 32 key rows per wave.
//
// What it computes is the dK/dV step of the backward (see bwd_bf16.hip), with the work items, the walk and the output paths of
// dkdv_wide_bf16.hip: a block owns key rows of one KV head and walks every query row of the launch scope at or after
// them, for its query heads of the group, in a fixed order; S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.
//
// Why another shape than at 128.  At 64 a score costs the same exponential, product and packing but half the matrix work: a
// wave that is alone on its SIMD issues longer than the matrix unit runs (per 64 keys x 32 rows 36 products of 32
// cycles, 1152; it took about 1850).  The accumulators of 32 keys (64 registers) with both operand fragments (32) leave room
// for two waves per SIMD, whose element-wise work and products overlap.  K and V fragments stay in registers, so that a step
// reads 16 KB of LDS per wave (Q and dO rows, and both transposed): half of what the LDS delivers in the products' time, and what
// two waves per SIMD can have.  A barrier every two steps; tiles are staged one pair of steps ahead, two LDS stages.  A wave skips
// steps before its keys, and all of them if it has none.
// Measured (16K tokens, 32/8 heads, us, the one-wave kernel at 64 -> this one): 128-row samples 109 -> 77, 1024 rows 433 -> 380 (32K
// tokens), samples of 32 to 512 rows 129 -> 98, one 16K sample 2049 -> 2045, one of 32K on 8/1 heads 2251 -> 2237.  On long samples a step
// takes about 1800 cycles, 1152 of them products; its LDS reads (64 KB of rows and 64 KB transposed per compute unit) are worth
// about 620 at the rates they reach alone, so what is left is latency: the first transposed reads are issued in front of the
// element-wise work (behind it, and with the second batch's wait free to move up: 2079 and 2278), the next step's row reads
// behind its last product.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "mfma_utils.h"

namespace slimattn {
namespace {

constexpr int D = 64;
constexpr int kWaves = 8, kKeys = 32 * kWaves;          // key rows per block
constexpr int kQStep = 32;
constexpr int kNKS = D / 16, kNDB = D / 32, kRowBytes = D * 2;
constexpr int kTileBytes = kQStep * kRowBytes;          // one Q or dO tile
constexpr int kStageBytes = 4 * kTileBytes;             // Q, dO of the first step; Q, dO of the second
constexpr float kLog2e = 1.4426950408889634f;

struct Step { int i0, hi, head; };                      // rows [i0, min(i0 + 32, hi)) of one query head

__global__ __launch_bounds__(64 * kWaves, 2) void dkdv_bf16_kernel_d64(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, const bf16* __restrict__ dO,
    const bf16x8* __restrict__ stat3, float* __restrict__ acc_dk, float* __restrict__ acc_dv, bf16* __restrict__ dK,
    bf16* __restrict__ dV, const KvItem* __restrict__ items, int n_items, const Seg* __restrict__ segs, int T, int Hq, int Hkv,
    float scale, float* __restrict__ parts, int head_parts) {
  constexpr int kOutBytes = kWaves * kOutAreaBytes<D>;
  __shared__ __attribute__((aligned(1024))) char smem[2 * kStageBytes > kOutBytes ? 2 * kStageBytes : kOutBytes];

  const int g = Hq / Hkv;
  // head_parts > 1: that many blocks share the item, each with a run of the group's heads; all store partial tiles
  const int item_idx = blockIdx.x / (Hkv * head_parts), hk = blockIdx.x % Hkv, hpart = blockIdx.x / Hkv % head_parts;
  const int h_lo = g * hpart / head_parts, h_hi = g * (hpart + 1) / head_parts;
  if (item_idx >= n_items) return;
  const KvItem it = items[item_idx];
  const int slot = head_parts > 1 ? it.number * head_parts + hpart : it.slot;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int kv0w = it.kv_row0 + 32 * wave, kv_end = it.kv_row0 + it.kv_rows;
  LDS_PTR(char) lds = (LDS_PTR(char))smem;

  // Flattened walk (block-uniform): runs from the last to the first, inside a run steps of 32 rows from the top down, inside a
  // step the block's heads of the group (co-resident blocks then read the same Q/dO rows at the same time).
  int sgi = it.seg_end - 1, hh = h_lo;
  Seg sg = segs[sgi];
  int lo = max(sg.q_lo, it.kv_row0);
  int n = (sg.q_hi - lo + kQStep - 1) / kQStep - 1;
  bool more = true;
  // The next step of the walk; behind its end an empty step (no row counts and none is read: hi = i0).
  auto next_step = [&]() -> Step {
    Step d{lo + n * kQStep, sg.q_hi, hk * g + hh};
    if (!more) {
      d.i0 = d.hi = it.kv_row0;
      d.head = hk * g;
      return d;
    }
    if (++hh == h_hi) {
      hh = h_lo;
      if (--n < 0) {
        if (--sgi < it.seg_begin) {
          more = false;
        } else {
          sg = segs[sgi];
          lo = max(sg.q_lo, it.kv_row0);
          n = (sg.q_hi - lo + kQStep - 1) / kQStep - 1;
        }
      }
    }
    return d;
  };

  // Q and dO rows come through descriptors based at the tile's first key row (head 0) whose range ends with the query run of the
  // step being staged: rows past the end of the run (another unit's, whose dO may not exist yet, or the next
  // sample's) read as zeros, whatever the memory holds.  Waves 0..3 stage the Q tile, waves 4..7 the dO tile: one load per
  // thread and step.
  const bool stages_do = wave >= 4;
  const TileSource src = make_tile_source<D, 256>(q, it.kv_row0, Hq, 0, T, tid & 255);     // (voff, row_bytes)
  const bf16* const src_base = (stages_do ? dO : q) + (size_t)it.kv_row0 * Hq * D;
  auto stage = [&](const Step& d, int at) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)src_base, 0, __builtin_amdgcn_readfirstlane((d.hi - it.kv_row0) * (Hq * kRowBytes)), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, lds + at + (stages_do ? kTileBytes : 0) + (wave & 3) * 1024, 16, src.voff + d.head * kRowBytes,
                                             __builtin_amdgcn_readfirstlane((d.i0 - it.kv_row0) * src.row_bytes), 0, 0);
  };
  // A step's statistics for this lane's row: -lse2 and -delta as bf16 triples.  (A row past the end of the run takes the run's
  // last row: finite numbers of this launch's own scope; its scores are masked.  An empty step takes the tile's first row.)
  const __amdgpu_buffer_rsrc_t stat_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)stat3, 0, (int)((size_t)T * Hq * 16), 0x00020000);
  auto load_stat = [&](const Step& d) -> bf16x8 {
    const int row = max(min(d.i0 + l32, d.hi - 1), it.kv_row0);
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(stat_rsrc, row * 16, __builtin_amdgcn_readfirstlane(d.head * T * 16), 0));
  };

  Step cur[2], nxt[2];
  bf16x8 stat[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    cur[x] = next_step();
    stage(cur[x], x * 2 * kTileBytes);
    stat[x] = load_stat(cur[x]);
  }
  // B operands kept in registers: K (times scale * log2 e) and V rows of the lane's key
  bf16x8 kf[kNKS], vf[kNKS];
  {
    const size_t off = ((size_t)min(kv0w + l32, T - 1) * Hkv + hk) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < kNKS; ++ks) {
      kf[ks] = scale8(*reinterpret_cast<const bf16x8*>(k + off + 16 * ks), scale * kLog2e);
      vf[ks] = *reinterpret_cast<const bf16x8*>(v + off + 16 * ks);
    }
  }
  // a product of a step's statistics with a fragment of ones puts the sum of a triple into every column of the row: the score
  // accumulators start at minus the statistics (lower half-wave only)
  const __bf16 one = half ? (bf16)0.f : (bf16)1.f, zero = (bf16)0.f;
  const bf16x8 ones_l = {one, one, one, zero, zero, zero, zero, zero}, ones_d = {zero, zero, zero, zero, one, one, one, zero};
  lds_cptr pq[kNKS], pqt[kNDB][2];                      // fragment addresses in the first stage's first Q tile
#pragma unroll
  for (int ks = 0; ks < kNKS; ++ks) pq[ks] = lds_row_ptr<D>(lds, l32, 16 * ks + 8 * half);
#pragma unroll
  for (int db = 0; db < kNDB; ++db) lds_tr_ptrs<D>(lds, 32 * db, lane, pqt[db][0], pqt[db][1]);
  floatx16 dk[kNDB], dv[kNDB];
  const floatx16 zeros = {};
#pragma unroll
  for (int db = 0; db < kNDB; ++db) { dk[db] = zeros; dv[db] = zeros; }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // One step: the wave's 32 keys against 32 query rows.  A lane owns a key, its registers the rows 8 (r / 4) + 4 half + r % 4.
  auto compute = [&](const Step& d, const bf16x8& st3, auto xc) {
    constexpr int at = decltype(xc)::value * 2 * kTileBytes;
    // (wave-uniform) no row at or after the wave's first key, or no key of the tile: nothing to add
    if (min(d.i0 + kQStep, d.hi) <= kv0w || kv0w >= kv_end) return;
    floatx16 s = mfma32(st3, ones_l, zeros), dp = mfma32(st3, ones_d, zeros);
    frag_pipeline<2 * kNKS, 4, 1, 1>([&](int i) { return lds_ld_row(pq[i >> 1], at + (i & 1) * kTileBytes); },
                                     [&](int i, bf16x8 f) {
                                       if (i & 1) dp = mfma32(f, vf[i >> 1], dp);
                                       else s = mfma32(f, kf[i >> 1], s);
                                     });
    if (d.i0 < kv0w + 31 || d.i0 + kQStep > d.hi) {     // some pair does not count: a row before the key or past the run
      const int rel_lo = kv0w + l32 - d.i0 - 4 * half, rel_hi = d.hi - d.i0 - 4 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (c < rel_lo || c >= rel_hi) s[r] = -INFINITY;
      }
    }
    // per 16 rows one batch of transposed fragments: dO^T of both head-dim blocks, Q^T of both; the first is on its way while the
    // element-wise work runs
    Tr4 tb[2];
    auto issue = [&](auto ec) {
      constexpr int e = decltype(ec)::value, off = at + e * 16 * kRowBytes;
      static_for<0, kNDB>([&](auto dc) {
        constexpr int db = decltype(dc)::value;
        tr1_issue<off + kTileBytes>(pqt[db][0], tb[e].r[2 * db]);
        tr1_issue<off + kTileBytes>(pqt[db][1], tb[e].r[2 * db + 1]);
        tr1_issue<off>(pqt[db][0], tb[e].r[4 + 2 * db]);
        tr1_issue<off>(pqt[db][1], tb[e].r[4 + 2 * db + 1]);
      });
    };
    issue(IC<0>{});
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 pf[2], ds[2];
    // at raised priority, as in the dQ kernel: 4K-row samples 566 -> 529 us
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(s[r]);
      dp[r] *= s[r];
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) { pf[e] = pack8(s, 8 * e); ds[e] = pack8(dp, 8 * e); }
    __builtin_amdgcn_s_setprio(0);
    static_for<0, 2>([&](auto ec) {
      constexpr int e = decltype(ec)::value;
      if constexpr (e == 0) issue(IC<1>{});
      tr4_wait_n<e == 0 ? 8 : 0>(tb[e]);
#pragma unroll
      for (int db = 0; db < kNDB; ++db) {
        dv[db] = mfma32(tr4_frag(tb[e], db), pf[e], dv[db]);
        dk[db] = mfma32(tr4_frag(tb[e], kNDB + db), ds[e], dk[db]);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  for (int t = 0;; ++t) {
    const bool last = !more;
    bf16x8 stat_n[2];
    if (!last) {                                        // the next two steps, into the stage the iteration before this one read
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        nxt[x] = next_step();
        stage(nxt[x], ((t + 1) & 1) * kStageBytes + x * 2 * kTileBytes);
        stat_n[x] = load_stat(nxt[x]);
      }
    }
    compute(cur[0], stat[0], IC<0>{});
    compute(cur[1], stat[1], IC<1>{});
    if (last) break;
    const int flip = (t & 1) ? -kStageBytes : kStageBytes;
#pragma unroll
    for (int ks = 0; ks < kNKS; ++ks) pq[ks] += flip;
#pragma unroll
    for (int db = 0; db < kNDB; ++db) { pqt[db][0] += flip; pqt[db][1] += flip; }
#pragma unroll
    for (int x = 0; x < 2; ++x) { cur[x] = nxt[x]; stat[x] = stat_n[x]; }
    __builtin_amdgcn_s_waitcnt(0);                      // this thread's direct loads have landed
    __syncthreads();
  }
  __syncthreads();                                      // the stages are free

  const int my_key = kv0w + l32;
  if (slot < 0 && it.final_from <= it.kv_row0 && it.load_until <= it.kv_row0) {
    LDS_PTR(char) ep = lds + wave * kOutAreaBytes<D>;   // the whole list in one launch: bf16 rows
    store_rows<D>(ep, dk, scale, dK, Hkv, hk, kv0w, kv_end, lane);
    store_rows<D>(ep, dv, 1.f, dV, Hkv, hk, kv0w, kv_end, lane);
  } else if (slot >= 0) {                               // partial tile [slot][kv head][dK, dV][256 rows][D]
    store_part_row<D>(parts + ((size_t)slot * Hkv + hk) * (2 * kKeys * D) + (size_t)(32 * wave + l32) * D, kKeys, dk, dv, scale, half);
  } else if (my_key < kv_end) {
    store_key_row<D>(((size_t)my_key * Hkv + hk) * D, my_key < it.load_until, my_key >= it.final_from, dk, dv, scale, half, acc_dk, acc_dv, dK, dV);
  }
}

}  // namespace

int launch_bwd_dkdv_d64_bf16(const LaunchCtx& c, const void* q, const void* k, const void* v, const void* dO, const void* stat3,
                             float* acc_dk, float* acc_dv, void* dK, void* dV, const KvItem* items, int n_items, const Seg* segs,
                             float* parts, int head_parts) {
  if (n_items == 0) return 0;
  const slimattn_params& p = *c.p;
  return in_runs(n_items, (int64_t)p.n_kv_heads * head_parts, [&](int first, int n) {
    hipLaunchKernelGGL(dkdv_bf16_kernel_d64, dim3((unsigned)(n * p.n_kv_heads * head_parts)), dim3(64 * kWaves), 0, (hipStream_t)c.stream,
                       (const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)dO, (const bf16x8*)stat3, acc_dk, acc_dv,
                       (bf16*)dK, (bf16*)dV, items + first, n, segs, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale, parts, head_parts);
    return (int)hipGetLastError();
  });
}

}  // namespace slimattn
