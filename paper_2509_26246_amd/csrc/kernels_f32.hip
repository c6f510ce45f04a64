// fp32 kernels: fp32 matrix products (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation, no reduced-precision step
// anywhere), fp32 softmax, fixed summation order.  This is the mode whose results must agree with the fp64 definition to
// 1e-5; it is kept separate from the bf16 kernels on purpose.
//
// Forward (paper: slice-level causal attention with a KV cache): online softmax over the sample's keys kv_start .. row.
// Backward (paper: scores are recomputed in the backward pass): dQ mirrors the forward walk; dK/dV has one owner per key
// row that walks the query rows at or after it, so contributions from later slices are summed in a fixed order without
// atomics.
//
// Shape on CDNA4.  The unit of work is a 32 x 32 tile of scores.  A product takes 64 cycles of the matrix unit for 64 + 64
// operand registers' worth of data, eight times as long per byte as a bf16 product, so operands need no LDS: a wave reads
// its fragments from global memory (the caches) straight into registers, one phase of products ahead of their use, and
// shares nothing with the other waves of its block until the end.  A block owns 32 rows (query rows for the forward and
// dQ, key rows for dK/dV), its 4 waves take the tiles of the walk in turn -- tile w, w + 4, ... -- and their partial sums
// are added up in wave order through LDS.  That keeps blocks small (a pack of a few hundred rows already fills dozens of
// compute units, each with a quarter of the walk's latency) and the loop without barriers.
//
// Operand layout of the product (lane l, half = l / 32, n = l % 32): A[m = n][k = half], B[k = half][n],
// C[i = 8 (r / 4) + 4 half + r % 4][j = n].  The order of a contraction is free, so
//   - "row" fragments (contraction over the head dimension): a lane reads 4 consecutive dims 8 c + 4 half .. + 3 of its row,
//     16 bytes that feed 4 products;
//   - the C registers of a score tile are, as they stand, the B operands of the next products: register r holds the rows
//     8 (r / 4) + r % 4 (lower half-wave) and + 4 (upper);
//   - "column" fragments (contraction over rows) match that: for register r a lane reads D / 32 consecutive dims of row
//     8 (r / 4) + 4 half + r % 4, one per accumulator block, so block b of an accumulator holds the dims (D / 32) i + b.
// What bounds it: the fp32 matrix rate (154 TFLOP/s for a large product here).  A pack of two samples, 1660 and 2436 rows,
// 8 query and 2 KV heads, head dim 128: forward 5803 -> 195 us, dQ with delta 6743 -> 280 us, dK/dV 12757 -> 381 us against
// one lane per row on the vector unit (2.5 -> 77 TFLOP/s, counting 7 products); the tiny pack of 876 rows, 2 heads of 64:
// 1080 -> 55 us.  (The forward at head dim 128 with 256 registers, two blocks per compute unit, 31 spilled registers and 24 reloads
// per tile, and with 356 registers, one block and no spills: the same 195 us.)
#include <hip/hip_runtime.h>

#include "internal.h"
#include "mfma_utils.h"

namespace slimattn {
namespace {

constexpr int kTileF32 = 64;            // rows of a listed query or key tile; a block takes one half of it
constexpr int kSub = 32;                // rows per block
constexpr int kWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <int D> constexpr int kNC = D / 8;                      // row-fragment chunks (4 products each)
template <int D> constexpr int kNB = D >= 32 ? D / 32 : 1;       // accumulator blocks of 32 dims
template <int D> constexpr int kPad = D + 4;                     // floats per row of the LDS areas the waves' sums meet in

template <int N> struct FloatVec { typedef __attribute__((__vector_size__(N * sizeof(float)))) float type; };
template <> struct FloatVec<1> { typedef float type; };
template <int N> __device__ __forceinline__ float elem(const typename FloatVec<N>::type& x, int i) {
  if constexpr (N == 1) return x; else return x[i];
}

__device__ __forceinline__ floatx16 mfma_f32(float a, float b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int c_row(int r) { return 8 * (r >> 2) + (r & 3); }   // + 4 * half: tile row of C register r

// 32 rows of one head of a [T, H, D] tensor through a buffer descriptor that ends with the last row the tile may use:
// rows behind it read as zeros (they belong to other units and may hold anything).
template <int D> struct Rows32 {
  __amdgpu_buffer_rsrc_t rsrc;
  int row_bytes;
  __device__ __forceinline__ Rows32(const float* base, int row0, int n_rows, int H, int h) {
    row_bytes = H * D * 4;
    const int n = min(n_rows, kSub);
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(base + ((size_t)row0 * H + h) * D), 0, n > 0 ? (n - 1) * row_bytes + D * 4 : 0,
                                             0x00020000);
  }
};
// Per-lane offsets of the two kinds of fragments.
template <int D> __device__ __forceinline__ int row_voff(int row_bytes, int l32, int half) { return l32 * row_bytes + 16 * half; }
template <int D> __device__ __forceinline__ int col_voff(int row_bytes, int l32, int half) {
  if constexpr (D < 32) { if (l32 >= D) return 0x7FF00000; }     // lanes without a dim: out of range, zeros
  return 4 * half * row_bytes + l32 * kNB<D> * 4;
}
template <int D> __device__ __forceinline__ floatx4 load_row(const Rows32<D>& t, int voff, int c) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(t.rsrc, voff + 32 * c, 0, 0));
}
template <int D> __device__ __forceinline__ typename FloatVec<kNB<D>>::type load_col(const Rows32<D>& t, int voff, int r) {
  typedef typename FloatVec<kNB<D>>::type V;
  const int soff = c_row(r) * t.row_bytes;
  if constexpr (kNB<D> == 4) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(t.rsrc, voff, soff, 0));
  else if constexpr (kNB<D> == 2) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(t.rsrc, voff, soff, 0));
  else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(t.rsrc, voff, soff, 0));
}

template <int D> struct RowFrag { floatx4 x[kNC<D>]; };
template <int D> struct ColFrag { typename FloatVec<kNB<D>>::type x[16]; };

// acc += rows . b^T over the head dimension; behind the products of chunk c: next(c), the loads of the following phase that
// may go into the registers chunk c gives free.
template <int D, class Next>
__device__ __forceinline__ void row_products(floatx16& acc, const RowFrag<D>& a, const RowFrag<D>& b, Next&& next) {
  static_for<0, kNC<D>>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = mfma_f32(a.x[c][j], b.x[c][j], acc);
    next(cc);
    __builtin_amdgcn_sched_barrier(0);
  });
}
// acc[b] += columns . s over the tile's rows (s: a score tile's C registers)
template <int D, class Next>
__device__ __forceinline__ void col_products(floatx16 (&acc)[kNB<D>], const ColFrag<D>& a, const floatx16& s, Next&& next) {
  static_for<0, 16>([&](auto rc) {
    constexpr int r = decltype(rc)::value;
#pragma unroll
    for (int b = 0; b < kNB<D>; ++b) acc[b] = mfma_f32(elem<kNB<D>>(a.x[r], b), s[r], acc[b]);
    next(rc);
    __builtin_amdgcn_sched_barrier(0);
  });
}
// The loads of one fragment, cut into pieces: piece c of kNC (behind a row phase's chunk) or piece r of 16.
template <int D, int C> __device__ __forceinline__ void cols_by_chunk(ColFrag<D>& f, const Rows32<D>& t, int voff) {
  constexpr int per = 16 / kNC<D>;
  static_for<0, per>([&](auto i) { constexpr int r = C * per + decltype(i)::value; f.x[r] = load_col<D>(t, voff, r); });
}
template <int D, int R> __device__ __forceinline__ void rows_by_reg(RowFrag<D>& f, const Rows32<D>& t, int voff) {
  constexpr int per = 16 / kNC<D>;
  if constexpr (R % per == 0) f.x[R / per] = load_row<D>(t, voff, R / per);
}
template <int D> __device__ __forceinline__ void load_rows(RowFrag<D>& f, const Rows32<D>& t, int voff) {
#pragma unroll
  for (int c = 0; c < kNC<D>; ++c) f.x[c] = load_row<D>(t, voff, c);
}

// Keys of the diagonal's tile with a NaN or an infinity: the product over the tile would carry them, times a probability of 0, into
// the rows in front of them, which do not see them.  If there are any (kr and kc hold the same keys), their values become 0 in kc
// and NaN goes to the rows that do see them, which is what the product would have given those (their scores are NaN or infinite).
template <int D>
__device__ __forceinline__ void unseen_keys(floatx16 (&acc)[kNB<D>], const RowFrag<D>& kr, ColFrag<D>& kc, int rel) {
  float odd = 0.f;
#pragma unroll
  for (int c = 0; c < kNC<D>; ++c)
#pragma unroll
    for (int j = 0; j < 4; ++j) odd = fmaf(kr.x[c][j], 0.f, odd);     // stays 0 unless one is not finite
  if (__builtin_expect(!__any(odd != 0.f), 1)) return;
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) {
    floatx16 seen = {};                                               // how many such keys a row sees, per dim
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = elem<kNB<D>>(kc.x[r], b);
      const bool bad = !(fabsf(x) < INFINITY);
      seen = mfma_f32(bad ? 1.f : 0.f, c_row(r) > rel ? 0.f : 1.f, seen);
      if constexpr (kNB<D> == 1) kc.x[r] = bad ? 0.f : x; else kc.x[r][b] = bad ? 0.f : x;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = seen[r] > 0.f ? __builtin_nanf("") : acc[b][r];
  }
}

// A wave's accumulator (C layout, lane = row l32) into its LDS area, one row of D floats per lane pair.
template <int D>
__device__ __forceinline__ void put_partial(float (*area)[kPad<D>], const floatx16 (&acc)[kNB<D>], int l32, int half) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = c_row(r) + 4 * half;
    if (D >= 32 || i < D)
#pragma unroll
      for (int b = 0; b < kNB<D>; ++b) area[l32][kNB<D> * i + b] = acc[b][r];
  }
}

template <int D>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                         const float* __restrict__ v, float* __restrict__ o,
                                                         float* __restrict__ lse, const QItem* __restrict__ items, int n_items,
                                                         int T, int Hq, int Hkv, float scale) {
  __shared__ __attribute__((aligned(16))) float part[kWaves][kSub][kPad<D>];
  __shared__ float part_m[kWaves][kSub], part_l[kWaves][kSub];
  const int g = Hq / Hkv;
  int idx, hk, hg;
  if (!map_block(blockIdx.x, g, Hkv, 2 * n_items, &idx, &hk, &hg)) return;
  const QItem it = items[idx >> 1];
  const int h = hk * g + hg, q0 = it.q_row0 + kSub * (idx & 1), q_end = it.q_row0 + min(it.q_rows, kSub * ((idx & 1) + 1));
  if (q0 >= q_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int n = (q_end - it.kv_start + kSub - 1) / kSub;         // key tiles of the walk

  auto tile = [&](const float* base, int kb) { return Rows32<D>(base, it.kv_start + kSub * kb, q_end - it.kv_start - kSub * kb, Hkv, hk); };
  const int rvoff = row_voff<D>(Hkv * D * 4, l32, half), cvoff = col_voff<D>(Hkv * D * 4, l32, half);
  RowFrag<D> kr, qf;
  ColFrag<D> vc;
  load_rows<D>(kr, tile(k, wave), rvoff);
  load_rows<D>(qf, Rows32<D>(q, q0, q_end - q0, Hq, h), row_voff<D>(Hq * D * 4, l32, half));
#pragma unroll
  for (int c = 0; c < kNC<D>; ++c) qf.x[c] *= scale * kLog2e;    // scores in log2 units
  floatx16 acc[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) acc[b] = floatx16{};
  float m = -INFINITY, l = 0.f;
  for (int kb = wave; kb < n; kb += kWaves) {
    const int key0 = it.kv_start + kSub * kb;
    floatx16 s = {};
    const Rows32<D> tv = tile(v, kb), tk = tile(k, kb + kWaves);
    row_products<D>(s, kr, qf, [&](auto cc) { cols_by_chunk<D, decltype(cc)::value>(vc, tv, cvoff); });
    if (key0 + kSub - 1 > q0) {                                  // the tile touches the diagonal of some row
      const int rel = q0 + l32 - key0 - 4 * half;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = c_row(r) > rel ? -INFINITY : s[r];
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(m, fmaxf(mx, xor32(mx)));
    const float ref = mx == -INFINITY ? 0.f : mx;                // a row that has seen no key yet
    const float alpha = __builtin_amdgcn_exp2f(m - ref);
    m = mx;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = __builtin_amdgcn_exp2f(s[r] - ref); sum += s[r]; }
    l = l * alpha + sum;
#pragma unroll
    for (int b = 0; b < kNB<D>; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] *= alpha;
    col_products<D>(acc, vc, s, [&](auto rc) { rows_by_reg<D, decltype(rc)::value>(kr, tk, rvoff); });
  }
  l += xor32(l);
  put_partial<D>(part[wave], acc, l32, half);
  if (half == 0) { part_m[wave][l32] = m; part_l[wave][l32] = l; }
  __syncthreads();
  const int row = tid >> 3;
  if (q0 + row >= q_end) return;
  float w[kWaves], top = part_m[0][row], l_tot = 0.f;            // wave 0 has the sample's first keys: finite
#pragma unroll
  for (int x = 1; x < kWaves; ++x) top = fmaxf(top, part_m[x][row]);
#pragma unroll
  for (int x = 0; x < kWaves; ++x) { w[x] = __builtin_amdgcn_exp2f(part_m[x][row] - top); l_tot += w[x] * part_l[x][row]; }
  const float inv = 1.f / l_tot;
  float* out = o + ((size_t)(q0 + row) * Hq + h) * D;
  for (int c = (tid & 7) * 4; c < D; c += 32) {
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) sum += w[x] * *reinterpret_cast<const floatx4*>(&part[x][row][c]);
    *reinterpret_cast<floatx4*>(out + c) = sum * inv;
  }
  if ((tid & 7) == 0) lse[(size_t)h * T + q0 + row] = top * kLn2 + logf(l_tot);
}

// dQ, and delta = rowsum(dO * O) of the block's rows (every (row, head) of the launch scope belongs to one block), stored for
// the dK/dV launch that follows.
template <int D>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void dq_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ o,
    const float* __restrict__ dO, const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dQ,
    const QItem* __restrict__ items, int n_items, int T, int Hq, int Hkv, float scale) {
  __shared__ __attribute__((aligned(16))) float part[kWaves][kSub][kPad<D>];
  const int g = Hq / Hkv;
  int idx, hk, hg;
  if (!map_block(blockIdx.x, g, Hkv, 2 * n_items, &idx, &hk, &hg)) return;
  const QItem it = items[idx >> 1];
  const int h = hk * g + hg, q0 = it.q_row0 + kSub * (idx & 1), q_end = it.q_row0 + min(it.q_rows, kSub * ((idx & 1) + 1));
  if (q0 >= q_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int n = (q_end - it.kv_start + kSub - 1) / kSub;

  auto tile = [&](const float* base, int kb) { return Rows32<D>(base, it.kv_start + kSub * kb, q_end - it.kv_start - kSub * kb, Hkv, hk); };
  const int rvoff = row_voff<D>(Hkv * D * 4, l32, half), cvoff = col_voff<D>(Hkv * D * 4, l32, half);
  RowFrag<D> kr, vr, qf, dof;
  ColFrag<D> kc;
  load_rows<D>(kr, tile(k, wave), rvoff);
  const int qvoff = row_voff<D>(Hq * D * 4, l32, half);
  load_rows<D>(qf, Rows32<D>(q, q0, q_end - q0, Hq, h), qvoff);
  load_rows<D>(dof, Rows32<D>(dO, q0, q_end - q0, Hq, h), qvoff);
  const size_t stat_at = (size_t)h * T + min(q0 + l32, q_end - 1);
  const float row_lse = lse[stat_at];
  float dlt = 0.f;
  {
    const Rows32<D> to(o, q0, q_end - q0, Hq, h);
#pragma unroll
    for (int c = 0; c < kNC<D>; ++c) {
      const floatx4 x = load_row<D>(to, qvoff, c);
#pragma unroll
      for (int j = 0; j < 4; ++j) dlt = fmaf(x[j], dof.x[c][j], dlt);
      qf.x[c] *= scale * kLog2e;
    }
    dlt += xor32(dlt);
    if (wave == 0 && half == 0 && q0 + l32 < q_end) delta[stat_at] = dlt;
  }
  floatx16 acc[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) acc[b] = floatx16{};
  auto step = [&](int kb, auto masked_c) {
    constexpr bool masked = decltype(masked_c)::value != 0;      // the tile touches the diagonal of some row
    const Rows32<D> tk = tile(k, kb), tv = tile(v, kb), tn = tile(k, kb + kWaves);
    floatx16 s = {}, dp = {};
    row_products<D>(s, kr, qf, [&](auto cc) { constexpr int c = decltype(cc)::value; vr.x[c] = load_row<D>(tv, rvoff, c); });
    row_products<D>(dp, vr, dof, [&](auto cc) { cols_by_chunk<D, decltype(cc)::value>(kc, tk, cvoff); });
    const int rel = q0 + l32 - it.kv_start - kSub * kb - 4 * half;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float ds = __builtin_amdgcn_exp2f(fmaf(row_lse, -kLog2e, s[r])) * (dp[r] - dlt);
      s[r] = masked && c_row(r) > rel ? 0.f : ds;
    }
    if constexpr (masked) unseen_keys<D>(acc, kr, kc, rel);
    col_products<D>(acc, kc, s, [&](auto rc) { rows_by_reg<D, decltype(rc)::value>(kr, tn, rvoff); });
  };
  int kb = wave;
  for (const int n_full = (q0 + 1 - it.kv_start) / kSub; kb < n_full; kb += kWaves) step(kb, IC<0>{});
  for (; kb < n; kb += kWaves) step(kb, IC<1>{});
  put_partial<D>(part[wave], acc, l32, half);
  __syncthreads();
  const int row = tid >> 3;
  if (q0 + row >= q_end) return;
  float* out = dQ + ((size_t)(q0 + row) * Hq + h) * D;
  for (int c = (tid & 7) * 4; c < D; c += 32) {
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) sum += *reinterpret_cast<const floatx4*>(&part[x][row][c]);
    *reinterpret_cast<floatx4*>(out + c) = sum * scale;
  }
}

// dK/dV of 32 key rows of one KV head: S = Q K^T - lse and dP = dO V^T - delta (a lane owns a key; the row statistics enter
// as one product each, the statistic in the lower half-wave's contraction slot times a constant), dV^T += dO^T P,
// dK^T += Q^T dS.  The walk: the scope's query runs at or after the tile, in each run steps of 32 rows, in each step the
// heads of the group; with P = gridDim.y parts, step x belongs to wave x % 4 of part (x / 4) % P.  P = 1: the block owns its
// rows' dK/dV.  P = 2 (whole-list scope only): part 0 leaves its sums in dK/dV, part 1 in the accumulators, which that scope
// does not use otherwise, and add_parts_f32_kernel adds the two.
template <int D>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2) void dkdv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dO,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ acc_dk, float* __restrict__ acc_dv,
    float* __restrict__ dK, float* __restrict__ dV, const KvItem* __restrict__ items, const Seg* __restrict__ segs, int T, int Hq,
    int Hkv, float scale) {
  __shared__ __attribute__((aligned(16))) float part[kWaves][kSub][kPad<D>];
  const int idx = blockIdx.x / Hkv, hk = blockIdx.x % Hkv, g = Hq / Hkv;
  const KvItem it = items[idx >> 1];
  const int k0 = it.kv_row0 + kSub * (idx & 1), k_end = it.kv_row0 + min(it.kv_rows, kSub * ((idx & 1) + 1));
  if (k0 >= k_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;

  const int kvoff = row_voff<D>(Hkv * D * 4, l32, half);
  RowFrag<D> kf, vf;
  load_rows<D>(kf, Rows32<D>(k, k0, k_end - k0, Hkv, hk), kvoff);
  load_rows<D>(vf, Rows32<D>(v, k0, k_end - k0, Hkv, hk), kvoff);
#pragma unroll
  for (int c = 0; c < kNC<D>; ++c) kf.x[c] *= scale * kLog2e;

  // this wave's walk: step `pos` of the run sgi (rows [lo, hi), n_run steps), step = 32 rows and a head
  const int n_parts = gridDim.y, part_no = blockIdx.y;
  int sgi = it.seg_begin, pos = kWaves * part_no + wave, lo = 0, hi = 0, n_run = 0;
  auto open_run = [&]() {
    const Seg sg = segs[sgi];
    lo = __builtin_amdgcn_readfirstlane(max(sg.q_lo, k0));
    hi = __builtin_amdgcn_readfirstlane(sg.q_hi);
    n_run = max(0, (hi - lo + kSub - 1) / kSub) * g;
  };
  auto settle = [&]() -> bool {                                  // past the end of a run: on to the next
    while (pos >= n_run) {
      pos -= n_run;
      if (++sgi >= it.seg_end) { n_run = 0; return false; }
      open_run();
    }
    return true;
  };
  open_run();
  bool live = settle();
  int i0 = 0, n_rows = 0, head = 0;                              // the step whose row fragments are loaded
  float nl = 0.f, nd = 0.f;                                      // its lse, delta (lane = row)
  const int qrow = row_voff<D>(Hq * D * 4, l32, half), qcol = col_voff<D>(Hq * D * 4, l32, half);
  auto take = [&]() {                                            // (an ended walk keeps naming its last step, with no rows)
    if (live) { i0 = lo + kSub * (pos / g); head = hk * g + pos % g; }
    n_rows = live ? min(kSub, hi - i0) : 0;
  };
  auto stats = [&]() {
    if (live) {
      const size_t at = (size_t)head * T + min(i0 + l32, hi - 1);
      nl = lse[at];
      nd = delta[at];
    }
  };
  RowFrag<D> qr, dr;
  ColFrag<D> dc, qc;
  floatx16 dk[kNB<D>], dv[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) { dk[b] = floatx16{}; dv[b] = floatx16{}; }
  const float one = half ? 0.f : 1.f;
  take();
  stats();
  load_rows<D>(qr, Rows32<D>(q, i0, n_rows, Hq, head), qrow);
  while (live) {
    const int c_i0 = i0, c_rows = n_rows;
    const Rows32<D> tq(q, i0, n_rows, Hq, head), td(dO, i0, n_rows, Hq, head);
    floatx16 s = {}, dp = {};
    const float c_nl = nl, c_nd = nd;
    pos += kWaves * n_parts;
    live = settle();
    take();
    stats();
    const Rows32<D> tn(q, i0, n_rows, Hq, head);
    row_products<D>(s, qr, kf, [&](auto cc) { constexpr int c = decltype(cc)::value; dr.x[c] = load_row<D>(td, qrow, c); });
    row_products<D>(dp, dr, vf, [&](auto cc) { cols_by_chunk<D, decltype(cc)::value>(dc, td, qcol); });
    s = mfma_f32(c_nl, -one * kLog2e, s);                        // the statistics last: added to the small accumulators they would
    dp = mfma_f32(c_nd, -one, dp);                               // cost every later addition its low bits
    const bool masked = c_i0 < k0 + kSub - 1 || c_rows < kSub;   // rows before the lane's key or past the end of the run
    const int rel_lo = masked ? k0 + l32 - c_i0 - 4 * half : -4 * kSub, rel_hi = masked ? c_rows - 4 * half : kSub;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = c_row(r) >= rel_lo && c_row(r) < rel_hi ? __builtin_amdgcn_exp2f(s[r]) : 0.f;
      s[r] = p;
      dp[r] *= p;
    }
    col_products<D>(dv, dc, s, [&](auto rc) { constexpr int r = decltype(rc)::value; qc.x[r] = load_col<D>(tq, qcol, r); });
    col_products<D>(dk, qc, dp, [&](auto rc) { rows_by_reg<D, decltype(rc)::value>(qr, tn, qrow); });
  }
  // the waves' sums in wave order; an earlier unit's partial sum of a row is added (rows below load_until); rows no later
  // unit reaches (from final_from on) are written as dK/dV, the others into the accumulators
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if (which) __syncthreads();
    put_partial<D>(part[wave], which ? dv : dk, l32, half);
    __syncthreads();
    const int row = k0 + (tid >> 3);
    if (row < k_end) {
      const bool load_acc = row < it.load_until, store_final = row >= it.final_from && part_no == 0;
      const size_t at = ((size_t)row * Hkv + hk) * D;
      const float* in = (which ? acc_dv : acc_dk) + at;
      float* out = (which ? (store_final ? dV : acc_dv) : (store_final ? dK : acc_dk)) + at;
      for (int c = (tid & 7) * 4; c < D; c += 32) {
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < kWaves; ++x) sum += *reinterpret_cast<const floatx4*>(&part[x][tid >> 3][c]);
        if (!which) sum *= scale;
        if (load_acc) sum += *reinterpret_cast<const floatx4*>(in + c);
        *reinterpret_cast<floatx4*>(out + c) = sum;
      }
    }
  }
}

// dK += acc_dk, dV += acc_dv: the second part of a divided whole-list dK/dV launch.
__global__ __launch_bounds__(256) void add_parts_f32_kernel(float* __restrict__ dK, float* __restrict__ dV,
                                                            const float* __restrict__ acc_dk, const float* __restrict__ acc_dv,
                                                            size_t n4) {
  floatx4* out = reinterpret_cast<floatx4*>(blockIdx.y ? dV : dK);
  const floatx4* in = reinterpret_cast<const floatx4*>(blockIdx.y ? acc_dv : acc_dk);
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n4; e += (size_t)gridDim.x * 256) out[e] += in[e];
}

#define DISPATCH_D(D_, BODY)                 \
  switch (D_) {                              \
    case 16: { constexpr int D = 16; BODY; } break;   \
    case 32: { constexpr int D = 32; BODY; } break;   \
    case 64: { constexpr int D = 64; BODY; } break;   \
    case 128: { constexpr int D = 128; BODY; } break; \
    default: return (int)hipErrorInvalidValue;        \
  }

}  // namespace

int launch_fwd_f32(const LaunchCtx& c, const float* q, const float* k, const float* v, float* o, float* lse,
                   const QItem* items, int n_items) {
  if (n_items == 0) return 0;
  const slimattn_params& p = *c.p;
  return in_runs(n_items, 2 * (int64_t)p.n_q_heads, [&](int first, int n) -> int {
    const dim3 grid((unsigned)mapped_grid(2 * n, p.n_kv_heads, p.n_q_heads / p.n_kv_heads)), block(64 * kWaves);
    DISPATCH_D(p.head_dim, hipLaunchKernelGGL(fwd_f32_kernel<D>, grid, block, 0, (hipStream_t)c.stream, q, k, v, o, lse, items + first,
                                              n, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale));
    return (int)hipGetLastError();
  });
}

int launch_bwd_dq_f32(const LaunchCtx& c, const float* q, const float* k, const float* v, const float* o, const float* dO,
                      const float* lse, float* delta, float* dQ, const QItem* items, int n_items) {
  if (n_items == 0) return 0;
  const slimattn_params& p = *c.p;
  return in_runs(n_items, 2 * (int64_t)p.n_q_heads, [&](int first, int n) -> int {
    const dim3 grid((unsigned)mapped_grid(2 * n, p.n_kv_heads, p.n_q_heads / p.n_kv_heads)), block(64 * kWaves);
    DISPATCH_D(p.head_dim, hipLaunchKernelGGL(dq_f32_kernel<D>, grid, block, 0, (hipStream_t)c.stream, q, k, v, o, dO, lse, delta,
                                              dQ, items + first, n, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale));
    return (int)hipGetLastError();
  });
}

int launch_bwd_dkdv_f32(const LaunchCtx& c, const float* q, const float* k, const float* v, const float* dO,
                        const float* lse, const float* delta, float* acc_dk, float* acc_dv, float* dK, float* dV,
                        const KvItem* items, int n_items, const Seg* segs, int longest) {
  if (n_items == 0) return 0;
  const slimattn_params& p = *c.p;
  const int64_t blocks = 2 * (int64_t)n_items * p.n_kv_heads;
  // Few long walks (up to three rounds of the chip's compute units): the first tiles of the longest sample decide the
  // launch, so every walk is divided in two (the pack above: 634 -> 381 us with the addition).  A wave's longest walk has
  // to be worth the second launch (about 7 us): from 16 steps on (a step is 4 to 8 us at head dims 64 to 128).
  const int parts = longest * (p.n_q_heads / p.n_kv_heads) >= 16 * kSub * kWaves && blocks <= 768 ? 2 : 1;
  const int e = in_runs(n_items, 2 * (int64_t)p.n_kv_heads, [&](int first, int n) -> int {
    const dim3 grid((unsigned)(2 * n * p.n_kv_heads), parts), block(64 * kWaves);
    DISPATCH_D(p.head_dim, hipLaunchKernelGGL(dkdv_f32_kernel<D>, grid, block, 0, (hipStream_t)c.stream, q, k, v, dO, lse, delta,
                                              acc_dk, acc_dv, dK, dV, items + first, segs, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale));
    return (int)hipGetLastError();
  });
  if (e != 0) return e;
  if (parts == 2) {
    const size_t n4 = (size_t)c.T * p.n_kv_heads * p.head_dim / 4;
    hipLaunchKernelGGL(add_parts_f32_kernel, dim3((unsigned)(n4 / 256 < 512 ? n4 / 256 + 1 : 512), 2), dim3(256), 0,
                       (hipStream_t)c.stream, dK, dV, acc_dk, acc_dv, n4);
  }
  return (int)hipGetLastError();
}

}  // namespace slimattn
