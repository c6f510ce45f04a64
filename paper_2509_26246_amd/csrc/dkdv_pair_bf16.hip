// dK/dV for bf16 inputs: 128 key rows per block, 32 per wave, two blocks per compute unit at head dim 128, three at 64.  Head dim 64, and 128
// where the walks are short (short_walks in internal.h).
//
// What it computes is the dK/dV step of the backward (see bwd_bf16.hip), with the work items, the walk and the output paths of
// dkdv_wide_bf16.hip: a block owns key rows of one KV head and walks every query row of the launch scope at or after
// them, for its query heads of the group, in a fixed order; S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  An item's 256 rows
// are two blocks.
//
// Why beside the one-wave kernel.  That one holds a compute unit to itself, so what an item costs beside its steps (its first loads
// and its last stores, 22 us: all compute units do them at about the same time, at the rate of the memory) is hidden by nothing.
// Blocks of half the keys overlap each other, steps before a wave's keys are skipped, and a sample that ends in a
// tile's first half wastes half as much.  At 128 a step costs more: one product per LDS fragment (1.25 KB of LDS reads per product), and a
// wave alone takes 2500 cycles for a step of 34 products (1088), two on a SIMD 3400 for both.
// Measured at 128, 16K tokens, one-wave kernel / this one, us: 32/32 heads, samples of 64 rows 430 / 165, 256 rows 244 / 164, 512 rows 286 / 210, 1024
// rows 379 / 316; 32/8 heads, 128 rows 161 / 104, 256 rows 144 / 116, 1024 rows 293 / 272, 4096 rows 891 / 1007; 876 rows of
// 8/1 heads, with the reduction, 45 / 27.  (Raised priority for the element-wise work: 2 to 5 % slower.  The next step's bookkeeping
// behind its first LDS reads, the second half of the element-wise work behind the first gradient products: no gain.)
// At 64 a score costs the same exponential, product and packing as at 128 but half the matrix work, and a step is mostly latency: what counts
// are waves, and barriers, of which there is one every two steps.  Against 256 keys in 8 waves, two per SIMD: 16K tokens, 32/8 heads, samples of 128 rows
// 76 / 52, 2048 rows 291 / 275, one sample 1944 / 1890; 32/32 heads, 1024 rows 207 / 163, 4096 rows 587 / 502; a 32K pack of 10 samples, 32/8 heads, 3128 /
// 2644 (matrix unit busy 0.77 of its time, waves waiting on LDS 0.03 of theirs).  (With first halves first throughout, against 64, 276, 1909, 166, 513: V rows in
// LDS 61, 283, 1972, 158, 514; a barrier for each step 62 to 1957.)
//
// Registers: 245 of 256 at 128, 167 of 168 at 64.  The accumulators take D, K fragments D / 4; V rows are in LDS at 128 and in registers at 64; a tile's fragment
// addresses are formed from one, and the row statistics, 16 bytes per row, come through LDS with the tiles (in registers, for this step and the next,
// they took 3 % at 128 and left no room for V at 64).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "mfma_utils.h"

namespace slimattn {
namespace {

constexpr int kWaves = 4, kKeys = 32 * kWaves;          // key rows per block
constexpr int kQStep = 32;
constexpr float kLog2e = 1.4426950408889634f;

struct Step { int i0, hi, head; };                      // rows [i0, min(i0 + 32, hi)) of one query head
struct QdV { bf16x8 q, d, v; };

// The items are heavy-first, and two or three blocks share a compute unit from the start.  The second round of 256 blocks (what there is of
// it) runs backwards, so that the longest walks share theirs with the shortest of the round: one 16K sample of 32/8 heads at 128 3887 -> 3728
// us, 128-row samples, first halves first, 124 -> 117; 32K pack at 64 2925 -> 2783.  (The low three bits, the XCD, stay.)
__device__ __forceinline__ int paired_block(int block) {
  const int end = min((int)gridDim.x, 512) & ~7;
  return block >= 256 && block < end ? 256 + end - 8 - (block & ~7) + (block & 7) : block;
}

// The fragment addresses of a tile differ from the first one's in the swizzled unit alone, by an exclusive or with the unit's number
// (tiles are 256-byte aligned): formed at each use, one register in the place of eight.
template <int X>
__device__ __forceinline__ lds_cptr lds_xor(lds_cptr p) {
  if constexpr (X == 0) return p;
  unsigned x;
  asm volatile("v_xor_b32 %0, %2, %1" : "=v"(x) : "v"((unsigned)(size_t)p), "n"(X));
  return (lds_cptr)(size_t)x;
}

// Bits MASK of tid >> SHIFT, formed where it is used: the kernels are at their register limit, and only the thread's number stays in one.
template <int SHIFT, int MASK>
__device__ __forceinline__ int at_use(int tid) {
  int x;
  if constexpr (SHIFT == 0) asm volatile("v_and_b32 %0, %2, %1" : "=v"(x) : "v"(tid), "n"(MASK));
  else asm volatile("v_bfe_u32 %0, %1, %2, 8\n\tv_and_b32 %0, %3, %0" : "=&v"(x) : "v"(tid), "n"(SHIFT), "n"(MASK));
  return x;
}

template <int D>
__global__ __launch_bounds__(64 * kWaves, D == 128 ? 2 : 3) void dkdv_pair_bf16_kernel(
    const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v, const bf16* __restrict__ dO,
    const bf16x8* __restrict__ stat3, float* __restrict__ acc_dk, float* __restrict__ acc_dv, bf16* __restrict__ dK,
    bf16* __restrict__ dV, const KvItem* __restrict__ items, int n_items, const Seg* __restrict__ segs, int T, int Hq, int Hkv,
    float scale, float* __restrict__ parts, int head_parts, int row_parts) {
  constexpr int kNKS = D / 16, kNDB = D / 32, kRowBytes = D * 2;
  constexpr int kTileBytes = kQStep * kRowBytes;        // one Q or dO tile
  constexpr int kStepBytes = 2 * kTileBytes + 1024;     // Q tile, dO tile, row statistics of a step
  constexpr int kSteps = D == 128 ? 1 : 2;              // steps of a stage, between two barriers
  constexpr bool kVInLds = D == 128;                    // or fragments in registers, where they fit
  constexpr int kVBase = 2 * kSteps * kStepBytes;       // two stages, then the block's V rows
  constexpr int kLoop = kVBase + (kVInLds ? kKeys * kRowBytes : 0), kOut = kWaves * kOutAreaBytes<D>;
  __shared__ __attribute__((aligned(1024))) char smem[kLoop > kOut ? kLoop : kOut];

  const int g = Hq / Hkv;
  // the halves of a 256-row item are blocks of their own, next to each other with the item's heads in between
  int b = paired_block(blockIdx.x);
  const int hk = b % Hkv;
  b /= Hkv;
  const int part = b % (head_parts * row_parts), hpart = part / row_parts, rpart = part % row_parts;
  b /= head_parts * row_parts;
  // Which half of an item comes first.  Blocks go to the XCDs in turn and inside an XCD to its four engines; the second halves have few keys or none
  // where samples, or their tails, end in the first.  With the first halves always first all the work of a launch of 1, 2 or 4 KV heads was on every
  // second XCD, and of 8 on every second engine.  So the order changes with the item's place in groups of eight blocks, in a pattern over eight of them that was the best
  // of six tried (334 launches: 1.5 % behind each with its best; first halves first 8 %).  120-row samples, us: 32K tokens of 8/1 heads of 128 94 -> 57, 16/4 151 -> 101, 5/5 58
  // -> 51, 16K tokens of 32/8 heads of 64 68 -> 52.  (Two rounds of blocks at most, the halves of a round on all XCDs: the reversed second round evens them out.)
  const int item_idx = b >> 1, half_blocks = Hkv * head_parts * row_parts, group8 = item_idx * half_blocks >> 2;
  const bool first_first = gridDim.x <= 512 && half_blocks % 8 == 0;
  const int sub = (first_first ? b : b ^ group8 ^ group8 >> 2 ^ (half_blocks & 1 ? 0 : group8 >> 1)) & 1;
  const int h_lo = g * hpart / head_parts, h_hi = g * (hpart + 1) / head_parts;
  if (item_idx >= n_items) return;
  const KvItem it = items[item_idx];
  const int row0 = it.kv_row0 + kKeys * sub, kv_end = it.kv_row0 + min(it.kv_rows, kKeys * (sub + 1));
  if (row0 >= kv_end) return;
  const int slot = head_parts * row_parts > 1 ? it.number * (head_parts * row_parts) + part : it.slot;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int kv0w = row0 + 32 * wave;
  LDS_PTR(char) lds = (LDS_PTR(char))smem;

  if constexpr (kVInLds) {
    const TileSource srcV = make_tile_source<D, 256>(v, row0, Hkv, hk, kv_end, tid);
    stage_tile<D, kKeys, 256>(lds + kVBase, srcV, 0, tid);
  }
  bf16x8 kf[kNKS], vf[kNKS];
  {
    const size_t off = ((size_t)min(kv0w + l32, T - 1) * Hkv + hk) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < kNKS; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8*>(k + off + 16 * ks);
      if constexpr (!kVInLds) vf[ks] = *reinterpret_cast<const bf16x8*>(v + off + 16 * ks);
    }
  }

  // Flattened walk (block-uniform): runs from the last to the first, inside a run steps of 32 rows from the top down, inside a
  // step the block's heads of the group (co-resident blocks then read the same Q/dO rows at the same time).
  int sgi = it.seg_end - 1, hh = h_lo, lo = 0, n = 0;
  Seg sg;
  bool more = true;
  auto open_run = [&]() {                               // runs that end before the half's first row have no step
    while (true) {
      if (sgi < it.seg_begin) { more = false; return; }
      sg = segs[sgi];
      if (sg.q_hi > row0) break;
      --sgi;
    }
    lo = max(sg.q_lo, row0);
    n = (sg.q_hi - lo + kQStep - 1) / kQStep - 1;
  };
  open_run();
  int todo = 0x7FFFFFFF;                                // steps of 32 rows still to hand out
  if (row_parts > 1) {                                  // this block's share of them
    int total = 0;
    for (int x = it.seg_begin; x < it.seg_end; ++x) total += max(0, segs[x].q_hi - max(segs[x].q_lo, row0) + kQStep - 1) / kQStep;
    total = __builtin_amdgcn_readfirstlane(total);      // (block-uniform anyway: tells the compiler)
    int skip = total * rpart / row_parts;
    todo = total * (rpart + 1) / row_parts - skip;
    if (todo == 0) more = false;
    while (more && skip > n) {
      skip -= n + 1;
      --sgi;
      open_run();
    }
    n -= skip;
  }
  // The next step of the walk; behind its end an empty step (no row counts and none is read: hi = i0).
  auto next_step = [&]() -> Step {
    if (!more) return Step{row0, row0, hk * g};
    Step d{lo + n * kQStep, sg.q_hi, hk * g + hh};
    if (++hh == h_hi) {
      hh = h_lo;
      if (--todo == 0) more = false;
      else if (--n < 0) { --sgi; open_run(); }
    }
    return d;
  };

  const TileSource src = make_tile_source<D, 256>(q, row0, Hq, 0, T, tid);     // (voff, row_bytes)
  const bf16* const q_base = q + (size_t)row0 * Hq * D;
  const bf16* const do_base = dO + (size_t)row0 * Hq * D;
  // A step's statistics (-lse2 and -delta as bf16 triples) come with its tiles, 16 bytes per row.  (A row past the end of the run takes the
  // run's last row: finite numbers of this launch's own scope; its scores are masked.  An empty step takes the tile's first row.)
  const __amdgpu_buffer_rsrc_t stat_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)stat3, 0, (int)((size_t)T * Hq * 16), 0x00020000);
  auto stage = [&](const Step& d, int at) {
    TileSource a = src, b2 = src;
    const int range = __builtin_amdgcn_readfirstlane((d.hi - row0) * (Hq * kRowBytes));
    a.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)q_base, 0, range, 0x00020000);
    b2.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)do_base, 0, range, 0x00020000);
    a.voff += d.head * kRowBytes;
    b2.voff = a.voff;
    stage_tile<D, kQStep, 256>(lds + at, a, d.i0 - row0, tid);
    stage_tile<D, kQStep, 256>(lds + at + kTileBytes, b2, d.i0 - row0, tid);
    if (wave == 0) {
      const int row = max(min(d.i0 + at_use<0, 63>(tid), d.hi - 1), row0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(stat_rsrc, lds + at + 2 * kTileBytes, 16, row * 16, __builtin_amdgcn_readfirstlane(d.head * T * 16), 0, 0);
    }
  };

  Step cur[kSteps], nxt[kSteps];
#pragma unroll
  for (int x = 0; x < kSteps; ++x) {
    cur[x] = next_step();
    stage(cur[x], x * kStepBytes);
  }
#pragma unroll
  for (int ks = 0; ks < kNKS; ++ks) kf[ks] = scale8(kf[ks], scale * kLog2e);
  const __bf16 one = half ? (bf16)0.f : (bf16)1.f, zero = (bf16)0.f;
  const bf16x8 ones_l = {one, one, one, zero, zero, zero, zero, zero}, ones_d = {zero, zero, zero, zero, one, one, one, zero};
  const lds_cptr pq = lds_row_ptr<D>(lds, l32, 8 * half);
  lds_cptr pqt[2];
  lds_tr_ptrs<D>(lds, 0, lane, pqt[0], pqt[1]);
  const lds_cptr pst = keep(lds + 16 * l32);            // a lane's row statistics
  const int v_rel = wave * 32 * kRowBytes;
  floatx16 dk[kNDB], dv[kNDB];
  const floatx16 zeros = {};
#pragma unroll
  for (int db = 0; db < kNDB; ++db) { dk[db] = zeros; dv[db] = zeros; }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  auto compute = [&](const Step& d, auto xc) {
    constexpr int at = decltype(xc)::value * kStepBytes;
    if (min(d.i0 + kQStep, d.hi) <= kv0w || kv0w >= kv_end) return;
    floatx16 s, dp;
    {
      constexpr int kPre = D == 128 ? 2 : 1;            // head-dim steps read ahead (registers)
      QdV f[kNKS];
      auto load = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const lds_cptr p = lds_xor<32 * i>(pq);
        r1_issue<at>(p, f[i].q);
        r1_issue<at + kTileBytes>(p, f[i].d);
        if constexpr (kVInLds) r1_issue<kVBase>(p + v_rel, f[i].v);
      };
      bf16x8 st3;
      r1_issue<at + 2 * kTileBytes>(pst, st3);
      static_for<0, kPre>(load);
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(st3) : "n"((kVInLds ? 3 : 2) * kPre));
      s = mfma32(st3, ones_l, zeros);
      dp = mfma32(st3, ones_d, zeros);
      static_for<0, kNKS>([&](auto ic) {
        constexpr int i = decltype(ic)::value, ahead = (kNKS - 1 - i < kPre - 1 ? kNKS - 1 - i : kPre - 1) + (i + kPre < kNKS ? 1 : 0);
        if constexpr (i + kPre < kNKS) load(IC<i + kPre>{});
        if constexpr (kVInLds) asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(f[i].q), "+v"(f[i].d), "+v"(f[i].v) : "n"(3 * ahead));
        else asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f[i].q), "+v"(f[i].d) : "n"(2 * ahead));
        s = mfma32(f[i].q, kf[i], s);
        if constexpr (kVInLds) dp = mfma32(f[i].d, f[i].v, dp);
        else dp = mfma32(f[i].d, vf[i], dp);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    if (d.i0 < kv0w + 31 || d.i0 + kQStep > d.hi) {
      const int half4 = at_use<3, 4>(tid), rel_lo = kv0w + at_use<0, 31>(tid) - d.i0 - half4, rel_hi = d.hi - d.i0 - half4;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (c < rel_lo || c >= rel_hi) s[r] = -INFINITY;
      }
    }
    constexpr int kPairs = kNDB / 2;                    // of head-dim blocks
    Tr4 tb[2 * kPairs];
    auto issue = [&](auto ec) {
      constexpr int e = decltype(ec)::value, off = at + e / kPairs * 16 * kRowBytes, db0 = 2 * (e % kPairs);
      static_for<0, 2>([&](auto dc) {
        constexpr int x = decltype(dc)::value;
        const lds_cptr p0 = lds_xor<64 * (db0 + x)>(pqt[0]), p1 = lds_xor<64 * (db0 + x)>(pqt[1]);
        tr1_issue<off + kTileBytes>(p0, tb[e].r[2 * x]);
        tr1_issue<off + kTileBytes>(p1, tb[e].r[2 * x + 1]);
        tr1_issue<off>(p0, tb[e].r[4 + 2 * x]);
        tr1_issue<off>(p1, tb[e].r[4 + 2 * x + 1]);
      });
    };
    issue(IC<0>{});
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 pf[2], ds[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(s[r]);
      dp[r] *= s[r];
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) { pf[e] = pack8(s, 8 * e); ds[e] = pack8(dp, 8 * e); }
    static_for<0, 2 * kPairs>([&](auto ec) {
      constexpr int e = decltype(ec)::value, db0 = 2 * (e % kPairs);
      constexpr bool last = e + 1 == 2 * kPairs;
      if constexpr (!last) issue(IC<e + 1>{});
      tr4_wait_n<last ? 0 : 8>(tb[e]);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        dv[db0 + x] = mfma32(tr4_frag(tb[e], x), pf[e / kPairs], dv[db0 + x]);
        dk[db0 + x] = mfma32(tr4_frag(tb[e], 2 + x), ds[e / kPairs], dk[db0 + x]);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  auto iteration = [&](auto xc) -> bool {
    constexpr int x = decltype(xc)::value;
    const bool last = !more;
    if (!last) {                                        // the next steps, into the stage the iteration before this one read
#pragma unroll
      for (int y = 0; y < kSteps; ++y) {
        nxt[y] = next_step();
        stage(nxt[y], ((1 - x) * kSteps + y) * kStepBytes);
      }
    }
    static_for<0, kSteps>([&](auto yc) { compute(cur[decltype(yc)::value], IC<x * kSteps + decltype(yc)::value>{}); });
    if (last) return false;
#pragma unroll
    for (int y = 0; y < kSteps; ++y) cur[y] = nxt[y];
    __builtin_amdgcn_s_waitcnt(0);                      // this thread's direct loads have landed
    __syncthreads();
    return true;
  };
  while (iteration(IC<0>{}) && iteration(IC<1>{})) {}
  __syncthreads();                                      // the stages are free

  const int out_lane = at_use<0, 63>(tid), out_half = out_lane >> 5, out_l32 = out_lane & 31, my_key = kv0w + out_l32;
  if (slot < 0 && it.final_from <= it.kv_row0 && it.load_until <= it.kv_row0) {
    LDS_PTR(char) ep = lds + wave * kOutAreaBytes<D>;   // the whole list in one launch: bf16 rows
    store_rows<D>(ep, dk, scale, dK, Hkv, hk, kv0w, kv_end, out_lane);
    store_rows<D>(ep, dv, 1.f, dV, Hkv, hk, kv0w, kv_end, out_lane);
  } else if (slot >= 0) {                               // partial tile [slot][kv head][dK, dV][256 rows][D]
    if (my_key < kv_end) store_part_row<D>(parts + ((size_t)slot * Hkv + hk) * (2 * 2 * kKeys * D) + (size_t)(sub * kKeys + 32 * wave + out_l32) * D, 2 * kKeys, dk, dv, scale, out_half);
  } else if (my_key < kv_end) {
    store_key_row<D>(((size_t)my_key * Hkv + hk) * D, my_key < it.load_until, my_key >= it.final_from, dk, dv, scale, out_half, acc_dk, acc_dv, dK, dV);
  }
}

}  // namespace

int launch_bwd_dkdv_pair_bf16(const LaunchCtx& c, const void* q, const void* k, const void* v, const void* dO, const void* stat3,
                              float* acc_dk, float* acc_dv, void* dK, void* dV, const KvItem* items, int n_items, const Seg* segs,
                              float* parts, const DkdvParts& by) {
  if (n_items == 0) return 0;
  const slimattn_params& p = *c.p;
  return in_runs(n_items, 2 * (int64_t)p.n_kv_heads * by.total(), [&](int first, int n) {
    hipLaunchKernelGGL(p.head_dim == 128 ? dkdv_pair_bf16_kernel<128> : dkdv_pair_bf16_kernel<64>, dim3((unsigned)(2 * n * p.n_kv_heads * by.total())),
                       dim3(64 * kWaves), 0, (hipStream_t)c.stream, (const bf16*)q, (const bf16*)k, (const bf16*)v, (const bf16*)dO, (const bf16x8*)stat3, acc_dk, acc_dv,
                       (bf16*)dK, (bf16*)dV, items + first, n, segs, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale, parts, by.heads, by.rows);
    return (int)hipGetLastError();
  });
}

}  // namespace slimattn
