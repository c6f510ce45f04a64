// Device helpers for the bf16 MFMA kernels (gfx950): vector types, swizzled LDS tiles, fragment
// reads in both orientations, global<->LDS staging.
//
// MFMA 32x32x16 bf16 operand layout (lane l, half = l / 32, n = l % 32):
//   A[m = n][k = 8*half + t], B[k = 8*half + t][n], t = 0..7 (eight consecutive k per lane);
//   C[i = 8*(r/4) + 4*half + (r%4)][j = n], r = 0..15.
// A product's C registers r = 8e .. 8e+7 therefore hold, for a fixed column, the rows
// {16e + 4*half + 0..3} and {16e + 8 + 4*half + 0..3}; used as the next product's B operand they
// fix which row each k-slot stands for, and the A operand of that product is read to match
// (transposed LDS reads below).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace slimattn {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __bf16 bf16;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

// Swizzled LDS tile of ROWS x D bf16 (no padding).  The 16-byte unit index is XORed with a
// function of the row so that (a) 16 consecutive rows at one column and (b) 4 consecutive rows
// x 4 consecutive units both touch 16 distinct units of a 256-byte bank line.
template <int D>
__device__ __forceinline__ int lds_off16(int row, int unit);
template <>
__device__ __forceinline__ int lds_off16<128>(int row, int unit) {
  const int f = ((row & 3) << 2) | ((row >> 2) & 3);
  return row * 256 + ((unit ^ f) << 4);
}
template <>
__device__ __forceinline__ int lds_off16<64>(int row, int unit) {
  const int R = row >> 1;
  const int f = ((R & 1) << 2) | ((R >> 1) & 3);
  const int u = ((row & 1) << 3) | unit;
  return R * 256 + ((u ^ f) << 4);
}

// Pack eight fp32 accumulators (registers r0 .. r0+7 of a C tile) into a bf16 B operand
// (four packed round-to-nearest-even conversions).
typedef __attribute__((__vector_size__(8 * sizeof(float)))) float floatx8;
__device__ __forceinline__ bf16x8 pack8(const floatx16& c, int r0) {
  floatx8 t;
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = c[r0 + i];
  return __builtin_convertvector(t, bf16x8);
}

// Fragment of eight bf16 values times a scalar, rounded back to bf16 (used to fold the softmax
// scale, in log2 units, into one operand of the score product).
__device__ __forceinline__ bf16x8 scale8(bf16x8 a, float c) {
  floatx8 t = __builtin_convertvector(a, floatx8);
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] *= c;
  return __builtin_convertvector(t, bf16x8);
}

// Sum of the eight bf16 values of a fragment, added to acc (four dot-products against ones).
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
__device__ __forceinline__ float sum8(bf16x8 a, float acc) {
  const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bf16x2 pr = {a[2 * i], a[2 * i + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, acc, false);
  }
  return acc;
}

// Software-pipelined operand stream: N fragments, each read from LDS kPre steps before the
// product that consumes it.  `load(i)` returns fragment i, `use(i, frag)` issues its products.
// The trailing scheduling directives pin the order "kPre reads, then (products, read) ...";
// rpf = LDS read instructions per fragment, upf = products per fragment.
template <int N, int kPre, int rpf, int upf, class Load, class Use>
__device__ __forceinline__ void frag_pipeline(Load&& load, Use&& use) {
  decltype(load(0)) fr[N];
#pragma unroll
  for (int i = 0; i < N + kPre; ++i) {
    if (i < N) fr[i] = load(i);
    if (i >= kPre) use(i - kPre, fr[i - kPre]);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, rpf * kPre, 0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, upf, 0);
    if (i + kPre < N) __builtin_amdgcn_sched_group_barrier(0x100, rpf, 0);
  }
}

// ---- LDS fragment pointers kept in registers --------------------------------------------------
// The swizzle makes a fragment's LDS address a non-additive function of (lane, column block), so
// the per-lane addresses are computed once, kept in registers (laundered through an empty asm so
// the compiler does not recompute them at every use) and advanced by adding uniform byte offsets:
// rows are additive, and so is the buffer switch.
typedef LDS_PTR(const char) lds_cptr;

__device__ __forceinline__ lds_cptr keep(lds_cptr p) {
  asm volatile("" : "+v"(p));
  return p;
}
template <int D>
__device__ __forceinline__ lds_cptr lds_row_ptr(lds_cptr tile, int row, int col0) {
  return keep(tile + lds_off16<D>(row, col0 >> 3));
}
// Transposed fragment for an A operand with m = column, k = row: lane l receives, for column
// col0 + (l % 32), the rows {row0 + 4*half + 0..3} and {row0 + 8 + 4*half + 0..3}.  It is built
// from two LDS transpose loads; in each, the 16 lanes of a group supply the addresses of 4 rows x
// 4 chunks of 4 columns, and lane i gets column i of the four rows.  These are the two addresses
// for row0 = 0: p0 serves rows {4*half + 0..3}, p1 rows {8 + 4*half + 0..3}; a fragment at
// row0 = 16*s is read at both pointers + 16*s*(2*D) bytes.
template <int D>
__device__ __forceinline__ void lds_tr_ptrs(lds_cptr tile, int col0, int lane, lds_cptr& p0, lds_cptr& p1) {
  const int i = lane & 15, grp = lane >> 4;
  const int row = 4 * (grp >> 1) + (i >> 2);
  const int col = col0 + 16 * (grp & 1) + 4 * (i & 3);
  p0 = keep(tile + lds_off16<D>(row, col >> 3) + ((col & 4) << 1));
  p1 = keep(tile + lds_off16<D>(row + 8, col >> 3) + ((col & 4) << 1));
}
__device__ __forceinline__ bf16x8 lds_ld_row(lds_cptr p, int byte_off) {
  return *reinterpret_cast<LDS_PTR(const bf16x8)>(p + byte_off);
}
// ---- transposed fragment stream through inline asm ---------------------------------------------
// The compiler's wait-count insertion treats an LDS transpose load as possibly reading what an
// outstanding direct global->LDS load is still writing and puts a full vmcnt(0) wait in front of
// it, which would serialise each tile behind the prefetch of the next one.  The prefetch targets
// the other buffer, so the transpose loads are issued from inline asm, in batches of four
// fragments (eight loads), with the wait counts written by hand: a batch is issued, then
// lgkmcnt(8) waits for everything older than it -- LDS operations complete in order -- which
// makes the previous batch ready while this one is still in flight.  The previous batch is
// passed through the asm as an in/out operand so that its consumers are ordered after the wait.
struct Tr4 { short4v r[8]; };     // four fragments; fragment j = (r[2j], r[2j+1])

__device__ __forceinline__ bf16x8 tr4_frag(const Tr4& t, int j) {
  typedef __attribute__((__vector_size__(8 * sizeof(short)))) short short8v;
  short8v x = __builtin_shufflevector(t.r[2 * j], t.r[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, x);
}
#define SLIMATTN_TR4_READS                                   \
  "ds_read_b64_tr_b16 %0, %[p0] offset:%[o0]\n\t"            \
  "ds_read_b64_tr_b16 %1, %[p1] offset:%[o0]\n\t"            \
  "ds_read_b64_tr_b16 %2, %[p0] offset:%[o1]\n\t"            \
  "ds_read_b64_tr_b16 %3, %[p1] offset:%[o1]\n\t"            \
  "ds_read_b64_tr_b16 %4, %[p0] offset:%[o2]\n\t"            \
  "ds_read_b64_tr_b16 %5, %[p1] offset:%[o2]\n\t"            \
  "ds_read_b64_tr_b16 %6, %[p0] offset:%[o3]\n\t"            \
  "ds_read_b64_tr_b16 %7, %[p1] offset:%[o3]\n\t"
// Issue the four fragments at byte offsets O0..O3 from the fragment address pair (p0, p1).
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void tr4_issue(lds_cptr p0, lds_cptr p1, Tr4& n) {
  asm volatile(SLIMATTN_TR4_READS
               : "=&v"(n.r[0]), "=&v"(n.r[1]), "=&v"(n.r[2]), "=&v"(n.r[3]), "=&v"(n.r[4]), "=&v"(n.r[5]), "=&v"(n.r[6]),
                 "=&v"(n.r[7])
               : [p0] "v"(p0), [p1] "v"(p1), [o0] "n"(O0), [o1] "n"(O1), [o2] "n"(O2), [o3] "n"(O3));
}
// Issue the next batch, then wait until the previous batch `p` has landed.
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void tr4_issue_wait(lds_cptr p0, lds_cptr p1, Tr4& n, Tr4& p) {
  asm volatile(SLIMATTN_TR4_READS "s_waitcnt lgkmcnt(8)"
               : "=&v"(n.r[0]), "=&v"(n.r[1]), "=&v"(n.r[2]), "=&v"(n.r[3]), "=&v"(n.r[4]), "=&v"(n.r[5]), "=&v"(n.r[6]),
                 "=&v"(n.r[7]), "+v"(p.r[0]), "+v"(p.r[1]), "+v"(p.r[2]), "+v"(p.r[3]), "+v"(p.r[4]), "+v"(p.r[5]),
                 "+v"(p.r[6]), "+v"(p.r[7])
               : [p0] "v"(p0), [p1] "v"(p1), [o0] "n"(O0), [o1] "n"(O1), [o2] "n"(O2), [o3] "n"(O3));
}
// Wait until batch `p` (the last one issued) has landed.
__device__ __forceinline__ void tr4_wait(Tr4& p) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(p.r[0]), "+v"(p.r[1]), "+v"(p.r[2]), "+v"(p.r[3]), "+v"(p.r[4]), "+v"(p.r[5]), "+v"(p.r[6]),
                 "+v"(p.r[7]));
}

// Wait until at most N LDS operations issued after batch `p` are outstanding (`p` has then landed).
template <int N>
__device__ __forceinline__ void tr4_wait_n(Tr4& p) {
  asm volatile("s_waitcnt lgkmcnt(%[n])"
               : "+v"(p.r[0]), "+v"(p.r[1]), "+v"(p.r[2]), "+v"(p.r[3]), "+v"(p.r[4]), "+v"(p.r[5]), "+v"(p.r[6]),
                 "+v"(p.r[7])
               : [n] "n"(N));
}

// Two-fragment variant (four loads per batch) for kernels that are short of registers.
struct Tr2 { short4v r[4]; };
__device__ __forceinline__ bf16x8 tr2_frag(const Tr2& t, int j) {
  typedef __attribute__((__vector_size__(8 * sizeof(short)))) short short8v;
  short8v x = __builtin_shufflevector(t.r[2 * j], t.r[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, x);
}
// Four-fragment row batches.
struct R4 { bf16x8 f[4]; };

// One transposed 64-bit read of a Tr2 batch (r[0], r[1]: first fragment from the two addresses of
// the pair; r[2], r[3]: second fragment), for code that spreads the reads between other instructions.
template <int O>
__device__ __forceinline__ void tr1_issue(lds_cptr p, short4v& r) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=&v"(r) : "v"(p), "n"(O));
}

// One row fragment (for code that spreads a batch's reads between other instructions).
template <int O>
__device__ __forceinline__ void r1_issue(lds_cptr a, bf16x8& f) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(f) : "v"(a), "n"(O));
}

// Wait until at most N LDS operations issued by this wave are outstanding; `p` (a batch issued
// before those N) is then complete, and its consumers are ordered after the wait.
template <int N>
__device__ __forceinline__ void lds_wait(R4& p) {
  asm volatile("s_waitcnt lgkmcnt(%[n])" : "+v"(p.f[0]), "+v"(p.f[1]), "+v"(p.f[2]), "+v"(p.f[3]) : [n] "n"(N));
}
template <int N>
__device__ __forceinline__ void lds_wait(Tr2& p) {
  asm volatile("s_waitcnt lgkmcnt(%[n])" : "+v"(p.r[0]), "+v"(p.r[1]), "+v"(p.r[2]), "+v"(p.r[3]) : [n] "n"(N));
}

// Compile-time loop: f(IC<0>{}), ..., f(IC<N-1>{}).
template <int I> struct IC { static constexpr int value = I; constexpr operator int() const { return I; } };
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IC<I>{});
    static_for<I + 1, N>(f);
  }
}

// ---- global -> LDS staging through buffer loads -----------------------------------------------
// A TileSource addresses the rows of one head of a [T, H, D] bf16 tensor starting at row `row_base`
// through a raw buffer descriptor whose range ends with row `row_end` - 1: the hardware checks the
// whole offset (per-lane part plus scalar part) against the range and answers reads of rows from
// `row_end` on with zeros, without touching memory.  Callers put the end of what their launch
// scope may read there -- the query tile's last row for K/V, the query run's last row for Q/dO --
// so rows behind it (other units' rows, which may not have been produced yet, or the end of the
// tensor) never reach a product, and no clamping code is needed; a tile's address is a per-lane
// constant (voff) plus a wave-uniform scalar.  The bytes from row_base to row_end must stay below
// 4 GiB (checked on the host).
struct TileSource {
  __amdgpu_buffer_rsrc_t rsrc;
  int voff;        // this lane's byte offset within one pass of 256-byte lines
  int row_bytes;   // H * D * 2
};
template <int D, int NT>
__device__ __forceinline__ TileSource make_tile_source(const bf16* base, int row_base, int H, int h, int row_end, int tid) {
  TileSource s;
  const size_t first = ((size_t)row_base * H + h) * D;
  const size_t valid = ((size_t)row_end * H * D - first) * 2;
  s.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(base + first), 0, (int)(valid > 0xFFFFFFFFull ? 0xFFFFFFFFull : valid),
                                             0x00020000);
  s.row_bytes = H * D * 2;
  const int wave = tid >> 6, lane = tid & 63, pos = lane & 15;
  const int line = wave * 4 + (lane >> 4);            // line within a pass; the swizzle repeats every pass
  int row, chunk;
  if (D == 128) {
    row = line;
    chunk = pos ^ (((row & 3) << 2) | ((row >> 2) & 3));
  } else {
    const int u = pos ^ (((line & 1) << 2) | ((line >> 1) & 3));
    row = 2 * line + (u >> 3);
    chunk = u & 7;
  }
  s.voff = row * s.row_bytes + chunk * 16;
  return s;
}
// Issues the loads for rows [row_base + row0, +ROWS) into `tile` (swizzled layout).  Completion is
// tracked by vmcnt; a barrier must follow before other waves read the tile.
template <int D, int ROWS, int NT>
__device__ __forceinline__ void stage_tile(LDS_PTR(char) tile, const TileSource& s, int row0, int tid) {
  constexpr int kLines = ROWS * D * 2 / 256, kLinesPerPass = NT / 16, kRowsPerPass = kLinesPerPass * 256 / (D * 2);
  static_assert(kLines % kLinesPerPass == 0, "tile must divide evenly over the block");
  const int wave_off = __builtin_amdgcn_readfirstlane((tid >> 6) * 1024);   // wave-uniform by construction
#pragma unroll
  for (int i = 0; i < kLines / kLinesPerPass; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, tile + i * kLinesPerPass * 256 + wave_off, 16, s.voff,
                                             __builtin_amdgcn_readfirstlane((row0 + i * kRowsPerPass) * s.row_bytes), 0, 0);
}

// One pass (NT / 16 lines of 256 bytes) of stage_tile: pass i of the tile at row offset row0.
template <int D, int NT>
__device__ __forceinline__ void stage_pass(LDS_PTR(char) tile, const TileSource& s, int row0, int i, int tid) {
  constexpr int kLinesPerPass = NT / 16, kRowsPerPass = kLinesPerPass * 256 / (D * 2);
  const int wave_off = __builtin_amdgcn_readfirstlane((tid >> 6) * 1024);   // wave-uniform by construction
  const int soff = __builtin_amdgcn_readfirstlane((row0 + i * kRowsPerPass) * s.row_bytes);   // uniform as well
  __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rsrc, tile + i * kLinesPerPass * 256 + wave_off, 16, s.voff, soff, 0, 0);
}

// frag_pipeline with one extra action per fragment (`side(i)`, e.g. one global->LDS load) issued
// alongside the products, so that the loads are spread over the phase instead of bunched.
template <int N, int kPre, class Load, class Use, class Side>
__device__ __forceinline__ void frag_pipeline_side(Load&& load, Use&& use, Side&& side) {
  decltype(load(0)) fr[N];
#pragma unroll
  for (int i = 0; i < N + kPre; ++i) {
    if (i < N) fr[i] = load(i);
    if (i >= kPre) {
      use(i - kPre, fr[i - kPre]);
      side(i - kPre);
    }
  }
  __builtin_amdgcn_sched_group_barrier(0x100, kPre, 0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i + kPre < N) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
}

__device__ __forceinline__ floatx16 mfma32(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float xor32(float x) { return __shfl_xor(x, 32); }

// Block -> (work item, kv head, head in group) so that the g query heads that share one K/V
// stream run back to back on the same XCD (blocks are dealt round-robin over the 8 XCDs) and
// heavy items come first on every XCD.  Returns false for padding blocks.
__device__ __forceinline__ bool map_block(int block, int g, int Hkv, int n_items, int* item, int* hk, int* hg) {
  const int xcd = block & 7, slot = block >> 3;
  *hg = slot % g;
  const int j = (slot / g) * 8 + xcd;
  if (j >= n_items * Hkv) return false;
  *item = j / Hkv;
  *hk = j % Hkv;
  return true;
}
inline int mapped_grid(int n_items, int Hkv, int g) { return ((n_items * Hkv + 7) / 8) * 8 * g; }

// The same for a launch over groups of items (QGroups): a block takes 1 << *share heads from *hg on.
struct QBlocks { int n[3], share[3], end[3]; };   // per group: items, log 2 of the heads per block, first block behind it
// Whether blocks of a launch with groups of g query heads take several of them: the list to walk is then the grouped one.
inline bool shares_heads(const QList& list, int g) { return g % 2 == 0 && list.groups.total() > 0; }
inline QBlocks shared_blocks(const QGroups& groups, int Hkv, int g) {
  QBlocks b;
  const int most = g % 4 == 0 ? 2 : g % 2 == 0 ? 1 : 0;
  int end = 0;
  for (int i = 0; i < 3; ++i) {
    b.n[i] = groups.n[i];
    b.share[i] = groups.share[i] < most ? groups.share[i] : most;
    b.end[i] = end += mapped_grid(b.n[i], Hkv, g >> b.share[i]);
  }
  return b;
}
__device__ __forceinline__ bool map_shared_block(int block, int g, int Hkv, const QBlocks& b, int* item, int* hk, int* hg, int* share) {
  // (in front of a block's first load: selects between scalars, where branches, or the array indexed in memory, cost up to a microsecond.
  // The empty statement keeps the compiler from making either out of it.)
  int n0 = b.n[0], n1 = b.n[1], n2 = b.n[2], s0 = b.share[0], s1 = b.share[1], s2 = b.share[2], e0 = b.end[0], e1 = b.end[1];
  asm volatile("" : "+s"(n0), "+s"(n1), "+s"(n2), "+s"(s0), "+s"(s1), "+s"(s2), "+s"(e0), "+s"(e1));
  const bool behind0 = block >= e0, behind1 = block >= e1;
  const int n = behind1 ? n2 : behind0 ? n1 : n0, first = behind1 ? n0 + n1 : behind0 ? n0 : 0, start = behind1 ? e1 : behind0 ? e0 : 0;
  *share = behind1 ? s2 : behind0 ? s1 : s0;
  if (!map_block(block - start, g >> *share, Hkv, n, item, hk, hg)) return false;
  *item += first;
  *hg <<= *share;
  return true;
}

// ---- forward launches whose keys are divided (FwdSplit in internal.h) --------------------------------------
// Block (without its part) -> item, KV head, head in group: the blocks that read the same keys are neighbours.
__device__ __forceinline__ void split_block(int j, int g, int Hkv, int* item, int* hk, int* hg) {
  *hg = j % g;
  *hk = j / g % Hkv;
  *item = j / (g * Hkv);
}

// Parts of an item, and part `part` of n: moves the item's first key and returns the tiles to walk.  Tiles whose first key is
// visible to every row of the item are dealt evenly; the last part also takes the (at most two) tiles behind.
__device__ __forceinline__ int split_parts(const FwdSplit& sp, const QItem& it) {
  const int common = (it.q_row0 - it.kv_start) / 64 + 1;
  return min(sp.parts, (common + sp.target - 1) / sp.target);
}
__device__ __forceinline__ int split_range(QItem& it, int part, int n) {
  const int all = (it.q_row0 + it.q_rows - it.kv_start + 63) / 64, common = (it.q_row0 - it.kv_start) / 64 + 1;
  const int a = (int)((long long)common * part / n), b = part + 1 == n ? all : (int)((long long)common * (part + 1) / n);
  it.kv_start += 64 * a;
  return b - a;
}

// The region the launch has claimed; -1: it found none free.
__device__ __forceinline__ int split_region(const FwdSplit& sp) {
  int region = -1;
#pragma unroll
  for (int r = 0; r < kSplitRegions; ++r)
    if (__hip_atomic_load(&sp.state->owner[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == sp.ticket) region = r;
  return __builtin_amdgcn_readfirstlane(region);
}

// Results of one (item, part, head): `unit` counts them as (item * parts + part) * Hq + head.
template <int D>
__device__ __forceinline__ float* split_unit(const FwdSplit& sp, int region, int unit) {
  return sp.data + region * kSplitRegionFloats + (size_t)unit * kSplitUnitFloats<D>;
}

// One wave's 32 rows of one head: O^T accumulators, reference (log2 units) and row sum of the part (stores of 1 KB per instruction).
template <int D>
__device__ __forceinline__ void split_store(float* base, int wave4, int lane, const floatx16 (&o)[D / 32], float m, float l) {
  floatx4* at = reinterpret_cast<floatx4*>(base + wave4 * 32 * D) + lane;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq)
      at[(db * 4 + gq) * 64] = floatx4{o[db][4 * gq], o[db][4 * gq + 1], o[db][4 * gq + 2], o[db][4 * gq + 3]};
  if (lane < 32) {
    float* stat = base + 128 * D + wave4 * 64 + lane;
    stat[0] = m;
    stat[32] = l;
  }
}

// Adds a part to the sum of those before it, each weighted by its reference: constructed from the two references and row sums,
// then called for each value of O.  (One operation for a multiplication and the addition, written out: the two ways a
// launch is finished must round alike.)
struct SplitAdd {
  float a, b;
  __device__ __forceinline__ SplitAdd(float& m, float& l, float m_part, float l_part) {
    const float top = fmaxf(m, m_part);
    a = __builtin_amdgcn_exp2f(m - top);
    b = __builtin_amdgcn_exp2f(m_part - top);
    m = top;
    l = (*this)(l, l_part);
  }
  __device__ __forceinline__ float operator()(float sum, float part) const { return __builtin_fmaf(b, part, a * sum); }
};

// The finishing kernel of a launch that owns a region, grid (items, heads, 1 .. D / 32): a wave adds up the n parts of 32 rows over N
// head-dim blocks of 32, a lane 16 columns of one row in each.  Bound by reading the partial results once; as the walk in the
// same kernel leaves room for few blocks per compute unit, a launch takes as many head-dim blocks per block as keep it to one
// round (split_finish_z; 1024 rows of 32/8 heads after 31K keys, in 2 parts: whole call 506 us with one each, 459 with four; 512 rows after 3.6K,
// in 4 parts: 78 and 59).
template <int D, int N>
__device__ __forceinline__ void split_combine_blocks(const FwdSplit& sp, int region, int n, const QItem& it, bf16* __restrict__ o,
                                                     float* __restrict__ lse, int T, int Hq) {
  const int h = blockIdx.y, db0 = N * blockIdx.z, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int r = 32 * wave + l32;
  if (r >= it.q_rows) return;
  float m = 0.f, l = 0.f;
  floatx4 sum[N][4];
#pragma unroll 2
  for (int p = 0; p < n; ++p) {
    const float* u = split_unit<D>(sp, region, ((int)blockIdx.x * sp.parts + p) * Hq + h);
    const float mp = u[128 * D + wave * 64 + l32], lp = u[128 * D + wave * 64 + 32 + l32];
    const floatx4* at = reinterpret_cast<const floatx4*>(u + wave * 32 * D) + db0 * 256 + lane;
    floatx4 x[N][4];
#pragma unroll
    for (int i = 0; i < 4 * N; ++i) x[i / 4][i % 4] = at[i * 64];
    if (p == 0) {
      m = mp;
      l = lp;
#pragma unroll
      for (int i = 0; i < 4 * N; ++i) sum[i / 4][i % 4] = x[i / 4][i % 4];
    } else {
      const SplitAdd add(m, l, mp, lp);
#pragma unroll
      for (int i = 0; i < 4 * N; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[i / 4][i % 4][e] = add(sum[i / 4][i % 4][e], x[i / 4][i % 4][e]);
    }
  }
  const float inv = 1.f / l;
  bf16* op = o + ((size_t)(it.q_row0 + r) * Hq + h) * D + 32 * db0 + 4 * half;
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) {
    bf16x4 w;
#pragma unroll
    for (int x = 0; x < 4; ++x) w[x] = (bf16)(sum[i / 4][i % 4][x] * inv);
    *reinterpret_cast<bf16x4*>(op + 8 * i) = w;
  }
  if (db0 == 0 && half == 0) lse[(size_t)h * T + it.q_row0 + r] = (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}
template <int D>
__device__ __forceinline__ void split_combine(const FwdSplit& sp, int region, int n, const QItem& it, bf16* __restrict__ o,
                                              float* __restrict__ lse, int T, int Hq) {
  if (gridDim.z == D / 32) split_combine_blocks<D, 1>(sp, region, n, it, o, lse, T, Hq);
  else if (gridDim.z == D / 64) split_combine_blocks<D, 2>(sp, region, n, it, o, lse, T, Hq);
  else split_combine_blocks<D, D / 32>(sp, region, n, it, o, lse, T, Hq);
}
inline unsigned split_finish_z(int n_items, int n_heads, int head_dim) {
  unsigned z = head_dim / 32;
  while (z > 1 && (int64_t)n_items * n_heads * z > 256) z /= 2;
  return z;
}
// The end of a finishing kernel's block: the last one to get here gives the region back.  A block has only read the region, and what
// it read has arrived (its results are made of it), so nothing has to be written back in front of the count: relaxed atomics in the order of one
// thread.  (A fence for the device here writes the L2 back, once per block: 1024 rows of 8/1 heads after 31K keys, 256 blocks, 16.6 us for the kernel against 9.9.)
__device__ __forceinline__ void split_release(const FwdSplit& sp, int region) {
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (region < 0) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) atomicAdd(&sp.state->launches[1], 1ull);
    return;
  }
  const unsigned before = __hip_atomic_fetch_add(&sp.state->done[region], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before == gridDim.x * gridDim.y * gridDim.z - 1) {
    __hip_atomic_fetch_add(&sp.state->launches[0], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sp.state->owner[region], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---- output rows ------------------------------------------------------------------------------
// A wave's 32 rows of one head from its transposed accumulators times `factor`, rows row0 .. min(row0 + 32, row_end), through the wave's LDS area `ep`
// (kOutAreaBytes<D>): a lane owns a row's values in pieces of 4 columns, and written as they stand each store
// instruction would touch 32 rows with 16 bytes each; transposed, a store instruction writes whole rows.
template <int D> constexpr int kOutStride = D * 2 + 16;
template <int D> constexpr int kOutAreaBytes = 32 * kOutStride<D>;
template <int D>
__device__ __forceinline__ void store_rows(LDS_PTR(char) ep, const floatx16 (&acc)[D / 32], float factor, bf16* __restrict__ out, int Hq, int h,
                                           int row0, int row_end, int lane) {
  constexpr int kChunks = D * 2 / 16, kRowsPerStore = 64 / kChunks;      // 16-byte chunks per row; rows per store
  const int half = lane >> 5, l32 = lane & 31, st_row = lane / kChunks, st_chunk = lane % kChunks;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      bf16x4 w;
#pragma unroll
      for (int x = 0; x < 4; ++x) w[x] = (bf16)(acc[db][4 * gq + x] * factor);
      *reinterpret_cast<LDS_PTR(bf16x4)>(ep + l32 * kOutStride<D> + (32 * db + 8 * gq + 4 * half) * 2) = w;
    }
#pragma unroll
  for (int j = 0; j < 32 / kRowsPerStore; ++j) {
    const int r = j * kRowsPerStore + st_row;
    const bf16x8 w = *reinterpret_cast<LDS_PTR(const bf16x8)>(ep + r * kOutStride<D> + st_chunk * 16);
    if (row0 + r < row_end) *reinterpret_cast<bf16x8*>(out + ((size_t)(row0 + r) * Hq + h) * D + st_chunk * 8) = w;
  }
}

// ---- gradient rows of a key --------------------------------------------------------------------
// A lane's key row from its transposed accumulators (dK times `scale`), where it does not leave as a bf16 row of a whole-list
// launch: into a partial tile of `tile_rows` rows at `row` (dK; dV behind the tile's dK rows), fp32 ...
template <int D>
__device__ __forceinline__ void store_part_row(float* row, int tile_rows, const floatx16 (&dk)[D / 32], const floatx16 (&dv)[D / 32], float scale,
                                               int half) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int off = 32 * db + 8 * gq + 4 * half;
      floatx4 a, b;
#pragma unroll
      for (int x = 0; x < 4; ++x) { a[x] = dk[db][4 * gq + x] * scale; b[x] = dv[db][4 * gq + x]; }
      *reinterpret_cast<floatx4*>(row + off) = a;
      *reinterpret_cast<floatx4*>(row + tile_rows * D + off) = b;
    }
}
// ... or to element `base` of the fp32 accumulators or of dK and dV: rows below load_until continue the sum an earlier unit left
// in the accumulators; rows from final_from on get no later contribution and are written in bf16.
template <int D>
__device__ __forceinline__ void store_key_row(size_t base, bool load_acc, bool store_final, const floatx16 (&dk)[D / 32],
                                              const floatx16 (&dv)[D / 32], float scale, int half, float* __restrict__ acc_dk,
                                              float* __restrict__ acc_dv, bf16* __restrict__ dK, bf16* __restrict__ dV) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const size_t off = base + 32 * db + 8 * gq + 4 * half;
      floatx4 a, b;
#pragma unroll
      for (int x = 0; x < 4; ++x) { a[x] = dk[db][4 * gq + x] * scale; b[x] = dv[db][4 * gq + x]; }
      if (load_acc) {
        a += *reinterpret_cast<const floatx4*>(acc_dk + off);
        b += *reinterpret_cast<const floatx4*>(acc_dv + off);
      }
      if (store_final) {
        bf16x4 wa, wb;
#pragma unroll
        for (int x = 0; x < 4; ++x) { wa[x] = (bf16)a[x]; wb[x] = (bf16)b[x]; }
        *reinterpret_cast<bf16x4*>(dK + off) = wa;
        *reinterpret_cast<bf16x4*>(dV + off) = wb;
      } else {
        *reinterpret_cast<floatx4*>(acc_dk + off) = a;
        *reinterpret_cast<floatx4*>(acc_dv + off) = b;
      }
    }
}

}  // namespace slimattn
