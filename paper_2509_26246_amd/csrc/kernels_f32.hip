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
// operand registers' worth of data, eight times as long per byte as a bf16 product, so the walk's operands need no LDS: a wave reads
// its fragments from global memory (the caches) straight into registers, eight to ten loads ahead of their use, and shares nothing with
// the other waves of its block until the end.  A block owns 32 rows (query rows for the forward and dQ, key rows for
// dK/dV), its 4 waves take the tiles of the walk in turn -- tile w, w + 4, ... -- and their partial sums
// are added up in wave order through LDS.  That keeps blocks small (a pack of a few hundred rows already fills dozens of
// compute units, each with a quarter of the walk's latency) and the loop without barriers.  The block's own rows, an operand of every
// score product, are in LDS (one read for four products): with them and whole phases of loads in registers a wave was alone
// on its SIMD at head dim 128 and nothing hid a block's first loads and its last additions; now two blocks (forward: three) share a compute
// unit.
//
// Operand layout of the product (lane l, half = l / 32, n = l % 32): A[m = n][k = half], B[k = half][n],
// C[i = 8 (r / 4) + 4 half + r % 4][j = n].  The order of a contraction is free, so
//   - "row" fragments (contraction over the head dimension): a lane reads 4 consecutive dims 8 c + 4 half .. + 3 of its row,
//     16 bytes that feed 4 products;
//   - the C registers of a score tile are, as they stand, the B operands of the next products: register r holds the rows
//     8 (r / 4) + r % 4 (lower half-wave) and + 4 (upper);
//   - "column" fragments (contraction over rows) match that: for register r a lane reads D / 32 consecutive dims of row
//     8 (r / 4) + 4 half + r % 4, one per accumulator block, so block b of an accumulator holds the dims (D / 32) i + b.
// What bounds it: the fp32 matrix rate (153 TFLOP/s for a large product here).  One sample of 4096 rows, 8 query and 2 KV heads, head dim
// 128: forward 313 -> 270 us, dQ with delta 422 -> 398, dK/dV 610 -> 515 (123 to 128 TFLOP/s) against whole phases of loads and the
// block's rows in registers; two samples, 1660 and 2436 rows, 187 -> 169, 264 -> 249, 361 -> 325, as the longest walks still decide; 2000 rows 124 -> 76, 123 -> 111, 268
// -> 249; samples of 300 rows 66 -> 46, 95 -> 75, 92 -> 78.
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

// The fragments of a walk come as a stream of slots, a slot being one load and the products it feeds: kNC row fragments for each score
// product, 16 column fragments for each product over rows.  R slots are under way: behind slot i's products, the load of slot i + R goes into
// the registers slot i gives free (R divides the slots of a tile, so the places are the same in every tile).
constexpr int ring_slots(int slots) {
  for (int r = 10; r > 1; --r) if (slots % r == 0) return r;
  return 1;
}
template <int R> struct Ring { floatx4 x[R]; };
template <int D> __device__ __forceinline__ void put_col(floatx4& f, const Rows32<D>& t, int voff, int r) {
  const typename FloatVec<kNB<D>>::type c = load_col<D>(t, voff, r);
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) f[b] = elem<kNB<D>>(c, b);
}

// The block's own rows (operands of every score product), in LDS as fragments: chunk c of lane l at [c][l].
template <int D> struct OwnRows { floatx4 x[kNC<D>][64]; };
template <int D>
__device__ __forceinline__ void put_own(OwnRows<D>& own, const Rows32<D>& t, int voff, float factor, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < (kNC<D> + kWaves - 1) / kWaves; ++i) {     // the waves share the chunks
    const int c = kWaves * i + wave;
    if (kNC<D> % kWaves == 0 || c < kNC<D>) own.x[c][lane] = load_row<D>(t, voff, c) * factor;
  }
}

// acc += rows . own^T over the head dimension, slots FIRST .. FIRST + kNC - 1 of the stream; next(i) issues the load of slot i + R.
template <int D, int R, int FIRST, class Next>
__device__ __forceinline__ void row_products(floatx16& acc, Ring<R>& ring, const OwnRows<D>& own, int lane, Next&& next) {
  floatx4 o[2];
  o[0] = own.x[0][lane];
  static_for<0, kNC<D>>([&](auto cc) {
    constexpr int c = decltype(cc)::value, at = (FIRST + c) % R;
    if constexpr (c + 1 < kNC<D>) o[(c + 1) & 1] = own.x[c + 1][lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = mfma_f32(ring.x[at][j], o[c & 1][j], acc);
    next(IC<FIRST + c>{});
    __builtin_amdgcn_sched_barrier(0);
  });
}
// acc[b] += columns . s over the tile's rows (s: a score tile's C registers), slots FIRST .. FIRST + 15.  FINITE: columns that are
// not finite count as 0.
template <int D, int R, int FIRST, bool FINITE = false, class Next>
__device__ __forceinline__ void col_products(floatx16 (&acc)[kNB<D>], Ring<R>& ring, const floatx16& s, Next&& next) {
  static_for<0, 16>([&](auto rc) {
    constexpr int r = decltype(rc)::value, at = (FIRST + r) % R;
#pragma unroll
    for (int b = 0; b < kNB<D>; ++b) {
      float x = ring.x[at][b];
      if constexpr (FINITE) x = fabsf(x) < INFINITY ? x : 0.f;
      acc[b] = mfma_f32(x, s[r], acc[b]);
    }
    next(IC<FIRST + r>{});
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Keys of the diagonal's tile with a NaN or an infinity: the product over the tile would carry them, times a probability of 0, into
// the rows in front of them, which do not see them.  Where there are any, the product takes their values as 0 (FINITE above) and NaN
// goes to the rows that do see them, which is what it would have given those (their scores are NaN or infinite).
template <int D>
__device__ __forceinline__ void unseen_keys(floatx16 (&acc)[kNB<D>], const Rows32<D>& tk, int cvoff, int rel) {
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) {
    floatx16 seen = {};                                               // how many such keys a row sees, per dim
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = elem<kNB<D>>(load_col<D>(tk, cvoff, r), b);
      seen = mfma_f32(fabsf(x) < INFINITY ? 0.f : 1.f, c_row(r) > rel ? 0.f : 1.f, seen);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = seen[r] > 0.f ? __builtin_nanf("") : acc[b][r];
  }
}

// The waves' sums meet in LDS, D / kHalves dims at a time, one row of them per lane pair.
template <int D> constexpr int kHalves = D == 128 ? 2 : 1;
template <int D> constexpr int kPad = D / kHalves<D> + 4;
template <int D> struct Partials { float x[kWaves][kSub][kPad<D>]; };
template <int D, int H>
__device__ __forceinline__ void put_partial(float (*area)[kPad<D>], const floatx16 (&acc)[kNB<D>], int l32, int half) {
  constexpr int n = 16 / kHalves<D>;
#pragma unroll
  for (int r = n * H; r < n * H + n; ++r) {
    const int i = c_row(r) + 4 * half - 2 * n * H;
    if (D >= 32 || i < D)
#pragma unroll
      for (int b = 0; b < kNB<D>; ++b) area[l32][kNB<D> * i + b] = acc[b][r];
  }
}
// For each part of the dims: every wave's sums into the area, then take(row of the block, first dim of four, offset in the area's rows).
template <int D, class Take>
__device__ __forceinline__ void meet(Partials<D>& p, const floatx16 (&acc)[kNB<D>], int wave, int l32, int half, Take&& take) {
  static_for<0, kHalves<D>>([&](auto hc) {
    constexpr int h = decltype(hc)::value, dims = D / kHalves<D>;
    __syncthreads();                                             // the area's last readers are through
    put_partial<D, h>(p.x[wave], acc, l32, half);
    __syncthreads();
    for (int c = (threadIdx.x & 7) * 4; c < dims; c += 32) take((int)threadIdx.x >> 3, h * dims + c, c);
  });
}

// The lists are heavy-first, and two or more blocks share a compute unit from the start.  The second round of 256 blocks runs backwards, so
// that the longest walks share theirs with the shortest of the round (one sample of 4096 rows, dK/dV 718 -> 515 us; 2000 rows, forward 100
// -> 76).  Where that round is not full, the longest walks go to the compute units that get no second block (9 samples of 512 rows, 2/2 heads of 128,
// 288 blocks, forward, dQ, dK/dV: 27.8, 43.9, 49.6 with the first 32 blocks beside a second one, now 23.9, 35.2, 41.4).  (The low three bits, the XCD, stay.)
__device__ __forceinline__ int paired(int block) {
  const int end = min((int)gridDim.x, 512) & ~7, second = max(end - 256, 0);
  if (second == 0 || block >= end) return block;
  return block >= 256 ? 256 + end - 8 - (block & ~7) + (block & 7) : block < second ? 256 - second + block : block - second;
}

template <int D>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                         const float* __restrict__ v, float* __restrict__ o,
                                                         float* __restrict__ lse, const QItem* __restrict__ items, int n_items,
                                                         int T, int Hq, int Hkv, float scale) {
  constexpr int kRows = kNC<D>, kSlots = kRows + 16, R = ring_slots(kSlots);       // a tile's slots: K rows, V columns
  __shared__ __attribute__((aligned(16))) union { OwnRows<D> own; Partials<D> part; } sh;
  __shared__ float part_m[kWaves][kSub], part_l[kWaves][kSub];
  const int g = Hq / Hkv;
  int idx, hk, hg;
  if (!map_block(paired(blockIdx.x), g, Hkv, 2 * n_items, &idx, &hk, &hg)) return;
  const QItem it = items[idx >> 1];
  const int h = hk * g + hg, q0 = it.q_row0 + kSub * (idx & 1), q_end = it.q_row0 + min(it.q_rows, kSub * ((idx & 1) + 1));
  if (q0 >= q_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int n = (q_end - it.kv_start + kSub - 1) / kSub;         // key tiles of the walk

  auto tile = [&](const float* base, int kb) { return Rows32<D>(base, it.kv_start + kSub * kb, q_end - it.kv_start - kSub * kb, Hkv, hk); };
  const int rvoff = row_voff<D>(Hkv * D * 4, l32, half), cvoff = col_voff<D>(Hkv * D * 4, l32, half);
  Ring<R> ring;
  auto load = [&](auto ic, const Rows32<D>& tk, const Rows32<D>& tv) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < kRows) ring.x[i % R] = load_row<D>(tk, rvoff, i);
    else put_col<D>(ring.x[i % R], tv, cvoff, i - kRows);
  };
  {
    const Rows32<D> tq(q, q0, q_end - q0, Hq, h);
    const int qvoff = row_voff<D>(Hq * D * 4, l32, half);
    put_own<D>(sh.own, tq, qvoff, scale * kLog2e, wave, lane);   // scores in log2 units
  }
  {
    const Rows32<D> tk = tile(k, wave), tv = tile(v, wave);
    static_for<0, R>([&](auto ic) { load(ic, tk, tv); });
  }
  __syncthreads();
  floatx16 acc[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) acc[b] = floatx16{};
  float m = -INFINITY, l = 0.f;
  for (int kb = wave; kb < n; kb += kWaves) {
    const int key0 = it.kv_start + kSub * kb;
    floatx16 s = {};
    const Rows32<D> tk = tile(k, kb), tv = tile(v, kb), nk = tile(k, kb + kWaves), nv = tile(v, kb + kWaves);
    auto next = [&](auto ic) {
      constexpr int i = decltype(ic)::value + R;
      if constexpr (i < kSlots) load(IC<i>{}, tk, tv); else load(IC<i - kSlots>{}, nk, nv);
    };
    row_products<D, R, 0>(s, ring, sh.own, lane, next);
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
    col_products<D, R, kRows>(acc, ring, s, next);
  }
  l += xor32(l);
  if (half == 0) { part_m[wave][l32] = m; part_l[wave][l32] = l; }
  __syncthreads();
  const int row = tid >> 3;
  float w[kWaves], top = part_m[0][row], l_tot = 0.f;            // wave 0 has the sample's first keys: finite
#pragma unroll
  for (int x = 1; x < kWaves; ++x) top = fmaxf(top, part_m[x][row]);
#pragma unroll
  for (int x = 0; x < kWaves; ++x) { w[x] = __builtin_amdgcn_exp2f(part_m[x][row] - top); l_tot += w[x] * part_l[x][row]; }
  const float inv = 1.f / l_tot;
  meet<D>(sh.part, acc, wave, l32, half, [&](int row, int dim, int c) {
    if (q0 + row >= q_end) return;
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) sum += w[x] * *reinterpret_cast<const floatx4*>(&sh.part.x[x][row][c]);
    *reinterpret_cast<floatx4*>(o + ((size_t)(q0 + row) * Hq + h) * D + dim) = sum * inv;
  });
  if ((tid & 7) == 0 && q0 + row < q_end) lse[(size_t)h * T + q0 + row] = top * kLn2 + logf(l_tot);
}

// dQ, and delta = rowsum(dO * O) of the block's rows (every (row, head) of the launch scope belongs to one block), stored for
// the dK/dV launch that follows.
template <int D>
__global__ __launch_bounds__(256, 2) void dq_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ o,
    const float* __restrict__ dO, const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dQ,
    const QItem* __restrict__ items, int n_items, int T, int Hq, int Hkv, float scale) {
  constexpr int kRows = kNC<D>, kSlots = 2 * kRows + 16, R = ring_slots(kSlots);   // a tile's slots: K rows, V rows, K columns
  __shared__ __attribute__((aligned(16))) union { OwnRows<D> own[2]; Partials<D> part; } sh;     // Q, dO
  const int g = Hq / Hkv;
  int idx, hk, hg;
  if (!map_block(paired(blockIdx.x), g, Hkv, 2 * n_items, &idx, &hk, &hg)) return;
  const QItem it = items[idx >> 1];
  const int h = hk * g + hg, q0 = it.q_row0 + kSub * (idx & 1), q_end = it.q_row0 + min(it.q_rows, kSub * ((idx & 1) + 1));
  if (q0 >= q_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int n = (q_end - it.kv_start + kSub - 1) / kSub;

  auto tile = [&](const float* base, int kb) { return Rows32<D>(base, it.kv_start + kSub * kb, q_end - it.kv_start - kSub * kb, Hkv, hk); };
  const int rvoff = row_voff<D>(Hkv * D * 4, l32, half), cvoff = col_voff<D>(Hkv * D * 4, l32, half);
  Ring<R> ring;
  auto load = [&](auto ic, const Rows32<D>& tk, const Rows32<D>& tv) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < 2 * kRows) ring.x[i % R] = load_row<D>(i < kRows ? tk : tv, rvoff, i % kRows);
    else put_col<D>(ring.x[i % R], tk, cvoff, i - 2 * kRows);
  };
  const size_t stat_at = (size_t)h * T + min(q0 + l32, q_end - 1);
  const float row_lse = lse[stat_at];
  float dlt = 0.f;
  {
    const int qvoff = row_voff<D>(Hq * D * 4, l32, half);
    const Rows32<D> tq(q, q0, q_end - q0, Hq, h), to(o, q0, q_end - q0, Hq, h), td(dO, q0, q_end - q0, Hq, h);
    put_own<D>(sh.own[0], tq, qvoff, scale * kLog2e, wave, lane);
#pragma unroll
    for (int c = 0; c < kRows; ++c) {                            // (every wave needs delta, so each has all of dO and writes the same)
      const floatx4 x = load_row<D>(to, qvoff, c), y = load_row<D>(td, qvoff, c);
#pragma unroll
      for (int j = 0; j < 4; ++j) dlt = fmaf(x[j], y[j], dlt);
      sh.own[1].x[c][lane] = y;
    }
    dlt += xor32(dlt);
    if (wave == 0 && half == 0 && q0 + l32 < q_end) delta[stat_at] = dlt;
  }
  {
    const Rows32<D> tk = tile(k, wave), tv = tile(v, wave);
    static_for<0, R>([&](auto ic) { load(ic, tk, tv); });
  }
  __syncthreads();
  floatx16 acc[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) acc[b] = floatx16{};
  auto step = [&](int kb, auto masked_c) {
    constexpr bool masked = decltype(masked_c)::value != 0;      // the tile touches the diagonal of some row
    const Rows32<D> tk = tile(k, kb), tv = tile(v, kb), nk = tile(k, kb + kWaves), nv = tile(v, kb + kWaves);
    float odd = 0.f;                                             // stays 0 unless a key of the tile is not finite
    auto next = [&](auto ic) {
      constexpr int i = decltype(ic)::value;
      if constexpr (masked && i < kRows)
#pragma unroll
        for (int j = 0; j < 4; ++j) odd = fmaf(ring.x[i % R][j], 0.f, odd);
      if constexpr (i + R < kSlots) load(IC<i + R>{}, tk, tv); else load(IC<i + R - kSlots>{}, nk, nv);
    };
    floatx16 s = {}, dp = {};
    row_products<D, R, 0>(s, ring, sh.own[0], lane, next);
    row_products<D, R, kRows>(dp, ring, sh.own[1], lane, next);
    const int rel = q0 + l32 - it.kv_start - kSub * kb - 4 * half;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float ds = __builtin_amdgcn_exp2f(fmaf(row_lse, -kLog2e, s[r])) * (dp[r] - dlt);
      s[r] = masked && c_row(r) > rel ? 0.f : ds;
    }
    if constexpr (masked) { if (__builtin_expect(__any(odd != 0.f), 0)) unseen_keys<D>(acc, tk, cvoff, rel); }
    col_products<D, R, 2 * kRows, masked>(acc, ring, s, next);
  };
  int kb = wave;
  for (const int n_full = (q0 + 1 - it.kv_start) / kSub; kb < n_full; kb += kWaves) step(kb, IC<0>{});
  for (; kb < n; kb += kWaves) step(kb, IC<1>{});
  meet<D>(sh.part, acc, wave, l32, half, [&](int row, int dim, int c) {
    if (q0 + row >= q_end) return;
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) sum += *reinterpret_cast<const floatx4*>(&sh.part.x[x][row][c]);
    *reinterpret_cast<floatx4*>(dQ + ((size_t)(q0 + row) * Hq + h) * D + dim) = sum * scale;
  });
}

// dK/dV of 32 key rows of one KV head: S = Q K^T - lse and dP = dO V^T - delta (a lane owns a key; the row statistics enter
// as one product each, the statistic in the lower half-wave's contraction slot times a constant), dV^T += dO^T P,
// dK^T += Q^T dS.  The walk: the scope's query runs at or after the tile, in each run steps of 32 rows, in each step the
// heads of the group; with P = n_parts, step x belongs to wave x % 4 of part (x / 4) % P.  P = 1: the block owns its
// rows' dK/dV.  P = 2 (whole-list scope only): part 0 leaves its sums in dK/dV, part 1 in the accumulators, which that scope
// does not use otherwise, and add_parts_f32_kernel adds the two.
template <int D>
__global__ __launch_bounds__(256, 2) void dkdv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dO,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ acc_dk, float* __restrict__ acc_dv,
    float* __restrict__ dK, float* __restrict__ dV, const KvItem* __restrict__ items, const Seg* __restrict__ segs, int T, int Hq,
    int Hkv, float scale, int n_parts) {
  // a step's slots: Q rows, dO rows, dO columns, Q columns
  constexpr int kRows = kNC<D>, kSlots = 2 * kRows + 32, R = ring_slots(kSlots);
  __shared__ __attribute__((aligned(16))) union { OwnRows<D> own[2]; Partials<D> part; } sh;     // K, V
  const int block = paired(blockIdx.x), part_no = block % n_parts, idx = block / n_parts / Hkv, hk = block / n_parts % Hkv, g = Hq / Hkv;
  const KvItem it = items[idx >> 1];
  const int k0 = it.kv_row0 + kSub * (idx & 1), k_end = it.kv_row0 + min(it.kv_rows, kSub * ((idx & 1) + 1));
  if (k0 >= k_end) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;

  {
    const int kvoff = row_voff<D>(Hkv * D * 4, l32, half);
    const Rows32<D> tk(k, k0, k_end - k0, Hkv, hk), tv(v, k0, k_end - k0, Hkv, hk);
    put_own<D>(sh.own[0], tk, kvoff, scale * kLog2e, wave, lane);
    put_own<D>(sh.own[1], tv, kvoff, 1.f, wave, lane);
  }

  // this wave's walk: step `pos` of the run sgi (rows [lo, hi), n_run steps), step = 32 rows and a head
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
  int i0 = 0, n_rows = 0, head = 0;                              // the step whose first slots are under way
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
  Ring<R> ring;
  auto load = [&](auto ic, const Rows32<D>& tq, const Rows32<D>& td) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < 2 * kRows) ring.x[i % R] = load_row<D>(i < kRows ? tq : td, qrow, i % kRows);
    else put_col<D>(ring.x[i % R], i < 2 * kRows + 16 ? td : tq, qcol, (i - 2 * kRows) % 16);
  };
  floatx16 dk[kNB<D>], dv[kNB<D>];
#pragma unroll
  for (int b = 0; b < kNB<D>; ++b) { dk[b] = floatx16{}; dv[b] = floatx16{}; }
  const float one = half ? 0.f : 1.f;
  take();
  stats();
  {
    const Rows32<D> tq(q, i0, n_rows, Hq, head), td(dO, i0, n_rows, Hq, head);
    static_for<0, R>([&](auto ic) { load(ic, tq, td); });
  }
  __syncthreads();
  while (live) {
    const int c_i0 = i0, c_rows = n_rows;
    const Rows32<D> tq(q, i0, n_rows, Hq, head), td(dO, i0, n_rows, Hq, head);
    floatx16 s = {}, dp = {};
    const float c_nl = nl, c_nd = nd;
    pos += kWaves * n_parts;
    live = settle();
    take();
    stats();
    const Rows32<D> nq(q, i0, n_rows, Hq, head), no(dO, i0, n_rows, Hq, head);
    auto next = [&](auto ic) {
      constexpr int i = decltype(ic)::value + R;
      if constexpr (i < kSlots) load(IC<i>{}, tq, td); else load(IC<i - kSlots>{}, nq, no);
    };
    row_products<D, R, 0>(s, ring, sh.own[0], lane, next);
    row_products<D, R, kRows>(dp, ring, sh.own[1], lane, next);
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
    col_products<D, R, 2 * kRows>(dv, ring, s, next);
    col_products<D, R, 2 * kRows + 16>(dk, ring, dp, next);
  }
  // the waves' sums in wave order; an earlier unit's partial sum of a row is added (rows below load_until); rows no later
  // unit reaches (from final_from on) are written as dK/dV, the others into the accumulators
  static_for<0, 2>([&](auto wc) {
    constexpr int which = decltype(wc)::value;
    meet<D>(sh.part, which ? dv : dk, wave, l32, half, [&](int r, int dim, int c) {
      const int row = k0 + r;
      if (row >= k_end) return;
      const bool load_acc = row < it.load_until, store_final = row >= it.final_from && part_no == 0;
      const size_t at = ((size_t)row * Hkv + hk) * D + dim;
      const float* in = (which ? acc_dv : acc_dk) + at;
      float* out = (which ? (store_final ? dV : acc_dv) : (store_final ? dK : acc_dk)) + at;
      floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < kWaves; ++x) sum += *reinterpret_cast<const floatx4*>(&sh.part.x[x][r][c]);
      if (!which) sum *= scale;
      if (load_acc) sum += *reinterpret_cast<const floatx4*>(in);
      *reinterpret_cast<floatx4*>(out) = sum;
    });
  });
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
  // Few blocks: the first tiles of the longest sample decide the launch, so every walk is divided in two where that is worth the second launch (about
  // 5 us; a step of a wave is 2 to 3 us at head dims 16 and 32, 3 to 7 at 64 and 128) and the second parts' blocks.  dK/dV undivided / divided, us:
  //   both parts of all blocks on compute units of their own, from two steps on: 48 blocks, 1 step 7.2 / 9.1 at 16, 15.6 / 18.0 at 128; 2 steps 9.1 / 9.1,
  //   23.7 / 19.4; 4 steps 12.7 / 11.0, 38.5 / 26.2; 876 rows, 2/2 heads of 64, 23.0 / 17.3;
  //   up to 256 blocks, whose second parts share compute units, from four: 136 blocks, 2 steps 9.3 / 11.1, 23.4 / 29.3; 4 steps 13.0 / 11.5, 38.4 / 30.3;
  //   more blocks: where the longest walk stands out from a compute unit's share of all of them, the less the longer it is.  At 128, steps of the longest and of
  //   the share: 264 blocks, 12 and 6.6, 1.37 times as fast; 288 blocks, 4 and 2.2, 42 / 62; 384 blocks, 8 and 6, 72 / 93; 16 and 12, 135 / 147; 64 and 48,
  //   518 / 425; 512 blocks, 16 and 16, 142 / 176; 520 blocks, 22 and 13, 1.10 times as fast; 528 blocks, 12 and 11, 0.89.  852 launches of more than 256
  //   blocks take 0.7 % longer than each with the better choice; by steps alone, from 16 on and up to 768 blocks, 4.4 %.
  const int64_t steps = (int64_t)longest * (p.n_q_heads / p.n_kv_heads) / (kSub * kWaves);
  const double share = (double)c.T * c.mean_keys * p.n_q_heads / (kSub * kSub * kWaves * 256);
  const bool divided = blocks <= 128 ? steps >= 2 : blocks <= 256 ? steps >= 4 : steps >= 6 && steps * steps >= share * (0.6 * steps + 9);
  const int parts = divided ? 2 : 1;
  const int e = in_runs(n_items, 2 * (int64_t)p.n_kv_heads, [&](int first, int n) -> int {
    const dim3 grid((unsigned)(2 * n * p.n_kv_heads * parts)), block(64 * kWaves);
    DISPATCH_D(p.head_dim, hipLaunchKernelGGL(dkdv_f32_kernel<D>, grid, block, 0, (hipStream_t)c.stream, q, k, v, dO, lse, delta,
                                              acc_dk, acc_dv, dK, dV, items + first, segs, (int)c.T, p.n_q_heads, p.n_kv_heads, p.scale, parts));
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
