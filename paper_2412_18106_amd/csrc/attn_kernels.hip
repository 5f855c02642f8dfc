// Attention meta-kernel for gfx950: a persistent kernel in which every workgroup
// walks its own list of (Q tile x KV block range) work units, plus the merge
// pass for K/V-split units.
//
// What is computed (paper section 4): per unit, S = scale * Q K^T over the KV
// blocks the unit visits, a row softmax restricted to the visible keys
// (causal bound of section 4.2.2, tree corner of section 4.1.2, tail of the
// last block neutralised as in section 5.2) and O = P V, in the K/V-split
// form with running max / sum (the Update stage of section 4.2.1).  The unit's
// origin (prefill, decode, verify) does not change the code path: only its row
// count does.
//
// How it is laid out on CDNA4 (this design, not the paper's):
//  * 256 threads = 4 wavefronts per workgroup, one per SIMD (so each may use all 512
//    registers of its SIMD lane), one workgroup per CU, 128 KB LDS; K and V stream from
//    HBM straight into LDS (no staging registers) while earlier blocks are consumed.
//  * Scores are produced transposed, S^T = K Q^T, with the 32x32x16 bf16 MFMA:
//    a lane then owns ONE query row (max / sum need one cross-lane exchange), the
//    accumulator registers of S^T are already the B operand of O^T += V^T P^T,
//    and rescaling O^T is one scalar per lane.
//  * V^T fragments come from the row-major V tile in LDS through the
//    transposing LDS read (ds_read_b64_tr_b16).
//  * rows = tokens x heads of one KV head (GQA sharing): a unit with more than
//    32 rows gives each wavefront 64 rows and every key, the wavefronts sharing
//    the K/V stream (every fragment read from LDS feeds two MFMAs), or 32 rows in
//    launches that hand out no unit of more than 128; a unit with
//    up to 32 rows (decode, short verify) is processed by a single wavefront
//    streaming 32-key slices through a private LDS ring, so a CU has four such
//    units in flight and no barrier between them; where a launch has fewer of
//    these than wavefronts, two or four wavefronts of a workgroup share one, each
//    with a part of its slices, and their states meet in LDS at its end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "plan_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr int kD = 128;          // head dim
constexpr int kB = 128;          // keys per K/V tile (one or more pages of the block table)
constexpr int kTileBytes = kB * kD * 2;   // one K or V tile of one KV head
constexpr int kThreads = 256;        // 4 wavefronts: one per SIMD
constexpr int kMergeThreads = 256, kMergeRows = kMergeThreads / 32;     // rows of a family merged by one workgroup
// workgroups of one launch (a launch of 2^32 threads or more runs those modulo 2^32, without an error)
constexpr int64_t kMergeGrid = 1 << 22, kAppendGrid = 1 << 22;
constexpr float kPrescaleMaxC = 0.25f;    // largest c = scale * log2(e) that is folded into Q (wide units)
// Dynamic assignment: the cursor of the shared list, kDoneGroups counts of finished workgroups and the
// count of finished groups, kCounterStride ints (one 128-byte line) apart.
constexpr int kDoneGroups = 8;
constexpr int kCounterStride = 32;
constexpr float kLazyRescale = 8.0f;      // log2 units the running max may lag behind
// Placement of the vector work of a wide iteration between its MFMAs: how many of the 32 exponentials, 16 bf16
// packings and 32 row-sum additions are done before each of the 32 gaps (made by gap_tables.py of this package
// from measured issue costs; a unit test compares them with what that module prints).
#define XY_GAP_TABLE_EXP {0, 2, 4, 5, 6, 7, 8, 10, 11, 12, 13, 14, 14, 15, 16, 17, 18, 19, 21, 22, 22, 22, 24, 25, 26, 27, 28, 30, 30, 31, 32, 32, 32}
#define XY_GAP_TABLE_CVT {0, 0, 0, 1, 1, 2, 3, 3, 3, 4, 5, 5, 5, 6, 7, 7, 8, 8, 8, 9, 9, 10, 10, 10, 11, 12, 13, 13, 13, 14, 15, 16, 16}
#define XY_GAP_TABLE_ADD {0, 0, 1, 2, 2, 3, 5, 5, 7, 7, 9, 10, 11, 11, 13, 14, 15, 16, 17, 17, 18, 19, 20, 21, 22, 23, 25, 25, 26, 27, 29, 32, 32}
// the same for a wavefront of one row tile: 16 gaps, 16 exponentials, 8 packings, 16 additions
#define XY_GAP_TABLE_ONE_EXP {0, 3, 4, 6, 7, 8, 8, 10, 10, 12, 12, 13, 14, 16, 16, 16, 16}
#define XY_GAP_TABLE_ONE_CVT {0, 0, 0, 1, 2, 3, 3, 3, 4, 4, 4, 5, 5, 6, 6, 8, 8}
#define XY_GAP_TABLE_ONE_ADD {0, 0, 1, 2, 3, 5, 5, 5, 7, 8, 8, 9, 10, 11, 12, 15, 16}
constexpr float kRowSumLimit = 18446744073709551616.f;      // 2^64: a wide unit whose row sums stay below was computed without overflow

struct RunParams {
  const XyDevUnit* units;
  const int32_t* worker_offsets;
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* block_table;
  const uint32_t* masks;
  uint16_t* out;
  float* ws;
  int64_t q_ts, q_hs, kv_bs, kv_hs, kv_ts, o_ts, o_hs;
  int32_t max_blocks, num_workers;
  int32_t free_workers;              // workers without units of their own, as they are handed out
  int32_t narrow_depth;              // slices a wavefront keeps in flight (see process_solo)
  int32_t num_units;                 // records: all units, second halves and the shared list included
  int32_t* counters;                 // plan with a shared list: its cursor and the finished-workgroup counts (kCounterStride apart); else null
  int32_t page_shift, page_mask;     // log2 of the tokens per block-table entry (page), and that size - 1
  float c;      // softmax_scale * log2(e)
};

// Read-only tables (units, block table, the kernel arguments themselves) are read through
// the constant address space: with a uniform address such a load is a scalar load, which neither
// occupies a vector register nor shares the in-order counter of the LDS-direct K/V stream.
#define XY_CONST __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const XY_CONST T* as_const(const T* ptr) {
  return (const XY_CONST T*)ptr;
}

// Pointers that reach the kernel through memory (the arguments as the narrow phase reads them) are generic ones to the
// compiler: their loads become flat ones, which count with the scalar and LDS requests and were waited for, Q included,
// before a unit's first K/V address was known.
#define XY_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ XY_GLOBAL T* as_global(T* ptr) {
  return (XY_GLOBAL T*)ptr;
}

template <typename T>     // whole-struct copy out of a read-only table, word by word
__device__ __forceinline__ T load_const(const T* ptr) {
  static_assert(sizeof(T) % 4 == 0, "word-sized records only");
  T out;
  const XY_CONST uint32_t* src = (const XY_CONST uint32_t*)ptr;
  uint32_t* dst = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) dst[i] = src[i];
  return out;
}

// The kernel arguments in registers, all of them, behind one wait.  Field by field, as the compiler loads an argument where it is
// first used, a narrow unit starts with four round trips instead of one.
__device__ __forceinline__ RunParams load_args() {
  typedef __attribute__((ext_vector_type(16))) uint32_t u32x16;
  typedef __attribute__((ext_vector_type(8))) uint32_t u32x8;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  static_assert(sizeof(RunParams) == 176, "RunParams is loaded as 16 + 16 + 8 + 4 words");
  const XY_CONST uint32_t* at = (const XY_CONST uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(at));              // not the copy that the wide units use: what they spill would be read back lane by lane
  u32x16 a, b;
  u32x8 c;
  u32x4 d;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    a[i] = at[i];
    b[i] = at[16 + i];
    if (i < 8) c[i] = at[32 + i];
    if (i < 4) d[i] = at[40 + i];
  }
  asm volatile("" : "+s"(a), "+s"(b), "+s"(c), "+s"(d));
  RunParams p;
  uint32_t* to = reinterpret_cast<uint32_t*>(&p);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    to[i] = a[i];
    to[16 + i] = b[i];
    if (i < 8) to[32 + i] = c[i];
    if (i < 4) to[40 + i] = d[i];
  }
  return p;
}

// A unit record in registers, all of it: left to itself the compiler reads it field by field where a field is first
// used, one round trip after another.
__device__ __forceinline__ XyDevUnit load_unit(const XyDevUnit* at) {
  XyDevUnit u = load_const(at);
  asm volatile("" : "+s"(u.seq), "+s"(u.head_begin), "+s"(u.head_count), "+s"(u.q_begin), "+s"(u.q_count), "+s"(u.kv_begin),
                    "+s"(u.kv_end), "+s"(u.flags), "+s"(u.ws_offset), "+s"(u.mask_off), "+s"(u.q_len), "+s"(u.ctx_len),
                    "+s"(u.token_start), "+s"(u.kv_head));
  return u;
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

__device__ __forceinline__ int swap23(int i) {   // exchange bits 2 and 3
  return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
}

// value held by the lane 32 places away
__device__ __forceinline__ float other_half(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // r[0]: lanes < 32 keep own, lanes >= 32 get lane-32's; r[1]: lanes < 32 get lane+32's, lanes >= 32 keep own
  unsigned o = (threadIdx.x & 32) ? r[0] : r[1];
  return __builtin_bit_cast(float, o);
}

// maximum of x over this lane and the lane 32 places away
__device__ __forceinline__ float max_both_halves(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // r[0] = lower half's x, r[1] = upper half's x
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  bf16x2 p = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(unsigned, p);
}

// ---- global -> LDS staging -------------------------------------------------------
// One wavefront instruction moves 64 x 16 bytes straight into 1 KB of LDS (4 rows of a tile)
// without passing through registers.  LDS slot (row, p) of a tile receives the 16-byte chunk
// p ^ swz(row) of that row; K uses swz = swap23(row) & 15, V uses swz = (row & 3) << 2, which
// spreads the fragment reads below over all LDS banks.  Both depend on the low 4 bits of the
// row only, so any 32-row slice of a tile is laid out the same way.
// The global address of lane l in instruction e is (uniform) tile + (row0 + 4e) rows, plus a
// per-lane 32-bit byte offset that depends on e only through e % 4: five registers per lane in all.
struct DmaOffsets {
  unsigned k[4];    // (l / 16) rows + swizzled chunk of K for e % 4
  unsigned v;       // the same for V (its swizzle does not depend on e)
};

__device__ __forceinline__ DmaOffsets make_dma_offsets(int lane, int64_t kv_ts) {
  DmaOffsets d;
  const int sub = lane >> 4, pos = lane & 15;
  const unsigned rowpart = (unsigned)(sub * kv_ts * 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) d.k[j] = rowpart + ((pos ^ (swap23(4 * j + sub) & 15)) << 4);
  d.v = rowpart + ((pos ^ ((sub & 3) << 2)) << 4);
  return d;
}

// Cache policy of the K/V loads of the narrow (bandwidth-bound) units: every byte is read once per launch, so the
// loads carry the non-temporal hint and leave the L2 to data that is used again (measured: decode-heavy steps
// 9-11 % faster, 5.4 -> 5.9 TB/s).  The wide units leave it off: their K/V is shared by the tiles of a sequence
// that run side by side on a chiplet.
constexpr int kReadOnce = 2;      // the nt bit of the instruction's cache-policy field

template <int NGROUPS>   // NGROUPS x 4 rows, starting at row0 (a multiple of 16), into lds_k / lds_v
__device__ __forceinline__ void load_rows_async(const uint16_t* kg, const uint16_t* vg, int64_t kv_ts, int row0,
                                                unsigned char* lds_k, unsigned char* lds_v, const DmaOffsets& dof,
                                                const bool want_k, const bool want_v) {
#pragma unroll
  for (int e = 0; e < NGROUPS; ++e) {
    const int64_t rows = (int64_t)(row0 + 4 * e) * kv_ts;          // uniform
    if (want_k)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(kg + rows) + (size_t)dof.k[e & 3]),
          (__attribute__((address_space(3))) void*)(lds_k + e * 1024), 16, 0, kReadOnce);
    if (want_v)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(vg + rows) + (size_t)dof.v),
          (__attribute__((address_space(3))) void*)(lds_v + e * 1024), 16, 0, kReadOnce);
  }
}

// ---- LDS fragment reads -----------------------------------------------------------
// The fragment reads are issued as inline assembly and waited for by hand.  The compiler cannot
// tell that a read of one LDS buffer does not depend on an LDS-direct load still in flight to
// ANOTHER buffer, and would drain every outstanding K/V load before each read; issued this way
// the K/V stream stays in flight while the current block is consumed.  Every read is waited for
// (lds_wait) before its registers are used and before its buffer is refilled.
__device__ __forceinline__ unsigned lds_addr(const void* ptr) {
  return (unsigned)(size_t)((__attribute__((address_space(3))) const unsigned char*)ptr);
}

template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128(unsigned addr) {
  bf16x8 r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  return r;
}

template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr16_b64(unsigned addr) {
  s16x4 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  return r;
}

// wait until at most N of this wavefront's LDS reads are outstanding; the operands tie the wait
// to the registers it protects, so no use can be scheduled above it
template <int N>
__device__ __forceinline__ void lds_wait(bf16x8& a, bf16x8& b, bf16x8& c, bf16x8& d) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N) : "memory");
}

// Per-lane byte offsets of the fragments inside any 32-row slice of a K / V tile.
struct LaneOffsets {
  unsigned k[8];   // K fragment ks: row swap23(col), 16-byte chunk (2*ks + half) ^ (col & 15)
  unsigned v[4];   // V^T fragment of d tile dt for keys 8*half + (i16 >> 2); add (16*t + 4*hh) * 256
};

__device__ __forceinline__ LaneOffsets make_lane_offsets(int lane) {
  LaneOffsets lo;
  const int col = lane & 31, half = lane >> 5, i16 = lane & 15, dsub = 16 * ((lane >> 4) & 1);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) lo.k[ks] = swap23(col) * 256 + (((2 * ks + half) ^ (col & 15)) << 4);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
    const int key = 8 * half + (i16 >> 2);
    const int d0 = 32 * dt + dsub + 4 * (i16 & 3);
    lo.v[dt] = key * 256 + (((d0 >> 3) ^ ((key & 3) << 2)) << 4) + ((d0 & 7) << 1);
  }
  return lo;
}

// s_waitcnt vmcnt(N) only (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Rows [first_row, 32) of a 32-row V slice in LDS are set to zero.  The last step of a unit may cover slots behind
// the unit's last key (the rest of a page, keys of later rows): their probabilities are exactly zero, but 0 x NaN
// and 0 x Inf are not, and a cache that was never initialised may hold such patterns there.  K needs nothing of
// the kind: a masked score is overwritten, not multiplied.  Every wavefront that reads the slice clears the same
// rows itself before it reads (the writes are idempotent), so no barrier is needed.
__device__ __forceinline__ void zero_tail_rows(unsigned slice_addr, int first_row, int lane) {
  // two registers in all (the units that need this are at their register limit): one address, one zero
  unsigned addr = slice_addr + (unsigned)(first_row + (lane >> 4)) * 256u + (unsigned)(lane & 15) * 16u;
  const unsigned zero = 0u;
  for (int r = first_row + (lane >> 4); r < 32; r += 4) {
    asm volatile("ds_write_b32 %0, %1 offset:0\n\tds_write_b32 %0, %1 offset:4\n\t"
                 "ds_write_b32 %0, %1 offset:8\n\tds_write_b32 %0, %1 offset:12"
                 :: "v"(addr), "v"(zero) : "memory");
    addr += 1024u;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // before the hand-issued fragment reads that follow
}

// ---- per-lane description of the query rows a wavefront owns -------------------------
template <int NT>
struct Rows {
  int lim[NT];                // causal: number of visible keys; 0 for padding rows
  int tok[NT];                // token index inside the sequence
  bool valid[NT];
  uint32_t mw0[NT], mw1[NT];  // tree corner bits 0..63 of this lane's row (a tree has at most 64 tokens)
};

struct UnitCtx {
  int hc, rows, kvh, ctx, wpr, key_end;
  bool tree;
};

__device__ __forceinline__ UnitCtx make_ctx(const RunParams& p, const XyDevUnit& u) {
  UnitCtx c;
  c.hc = u.head_count;
  c.rows = u.q_count * u.head_count;
  c.kvh = u.kv_head;
  c.ctx = u.ctx_len;
  c.wpr = (u.q_len + 31) >> 5;
  c.tree = (u.flags >> 2) & 1;
  c.key_end = c.tree ? u.ctx_len + u.q_len : u.ctx_len + u.q_begin + u.q_count;   // exclusive
  return c;
}

// Token and head of row rho of a unit (rho = token * hc + head, fewer than 256 of them).  An integer division is some
// forty instructions; the reciprocal is exact enough here: (rho + 1/2) / hc is at least 1 / (2 hc) >= 2^-9 away from an
// integer and is computed to within 2^-14.
struct RowIndex {
  int tl, hl;
};
__device__ __forceinline__ RowIndex row_index(int rho, int hc, float inv_hc) {
  RowIndex r;
  r.tl = (int)(((float)rho + 0.5f) * inv_hc);
  r.hl = rho - r.tl * hc;
  return r;
}

// Byte offset of row (tl, hl) of a Q or O tensor from the unit's first row.  SMALL: strides below kSmallStride
// elements, so that a row of a unit lies within 2^31 bytes of it (24-bit multiplies, 32-bit offsets).
constexpr int64_t kSmallStride = 1 << 21;
template <bool SMALL>
__device__ __forceinline__ int64_t row_bytes(const RowIndex& r, int64_t ts, int64_t hs) {
  if (SMALL) return (int64_t)(uint32_t)(__umul24(r.tl, 2 * (unsigned)ts) + __umul24(r.hl, 2 * (unsigned)hs));
  return 2 * (r.tl * ts + r.hl * hs);
}

// Row bookkeeping of a unit of at most 32 rows: what a lane has to know of its row.
__device__ __forceinline__ void setup_rows(const RunParams& p, const XyDevUnit& u, const UnitCtx& c, int col, float inv_hc, Rows<1>& r) {
  r.valid[0] = col < c.rows;
  r.tok[0] = u.q_begin + row_index(min(col, c.rows - 1), c.hc, inv_hc).tl;
  r.lim[0] = r.valid[0] ? c.ctx + r.tok[0] + 1 : 0;
  r.mw0[0] = r.mw1[0] = 0;
  if (c.tree && r.valid[0]) {
    const XY_GLOBAL uint32_t* mrow = as_global(p.masks + u.mask_off + (int64_t)r.tok[0] * c.wpr);
    r.mw0[0] = mrow[0];
    if (c.wpr > 1) r.mw1[0] = mrow[1];
  }
}

// ---- S^T = K Q^T for 32 keys x (32 * NT) rows -------------------------------------
// kaddr: LDS byte address of the first of the 32 key rows.  Register v of s[rt] is key
// 16*(v>>3) + 8*half + (v&7) of those 32 for this lane's row.
template <int NT>
__device__ __forceinline__ void qk_step(unsigned kaddr, const LaneOffsets& lo, const bf16x8 (&qf)[NT][8],
                                        f32x16 (&s)[NT]) {
  bf16x8 ka[4], kb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) ka[ks] = lds_read_b128<0>(kaddr + lo.k[ks]);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) kb[ks] = lds_read_b128<0>(kaddr + lo.k[4 + ks]);
#pragma unroll
  for (int rt = 0; rt < NT; ++rt)
#pragma unroll
    for (int v = 0; v < 16; ++v) s[rt][v] = 0.f;
  lds_wait<4>(ka[0], ka[1], ka[2], ka[3]);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) s[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[rt][ks], s[rt], 0, 0, 0);
  lds_wait<0>(kb[0], kb[1], kb[2], kb[3]);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt)
      s[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[ks], qf[rt][4 + ks], s[rt], 0, 0, 0);
}

// ---- visibility: causal bound (section 4.2.2) or tree corner (section 4.1.2) ----------
template <int NT>
__device__ __forceinline__ void mask_step(const RunParams& p, const UnitCtx& c,
                                          const Rows<NT>& r, int jbase /* key of register 0 */, f32x16 (&s)[NT]) {
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    if (!c.tree) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int j = jbase + 16 * (v >> 3) + (v & 7);
        if (j >= r.lim[rt]) s[rt][v] = -INFINITY;
      }
    } else {                  // at most 64 speculative tokens: both mask words of the row are in registers
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int sidx = jbase + 16 * (v >> 3) + (v & 7) - c.ctx;   // corner column when >= 0
        const uint32_t w = (sidx & 32) ? r.mw1[rt] : r.mw0[rt];
        const bool bit = sidx < 64 && ((w >> (sidx & 31)) & 1u);
        if (!(r.valid[rt] && (sidx < 0 || bit))) s[rt][v] = -INFINITY;
      }
    }
  }
}

// ---- softmax + Update (section 4.2.1) with a lazily raised reference max -------------
// On return s holds the un-normalised probabilities 2^((score - m_ref) * c) <= 2^kLazyRescale.
template <int NT>
__device__ __forceinline__ void softmax_step(float cs, f32x16 (&s)[NT], float (&m_ref)[NT], float (&l_part)[NT],
                                             f32x16 (&oacc)[NT][4], const bool first /* step: the accumulators are zero */) {
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    float mx = fmaxf(s[rt][0], s[rt][1]);
#pragma unroll
    for (int v = 2; v < 16; ++v) mx = fmaxf(mx, s[rt][v]);
    mx = fmaxf(mx, other_half(mx));
    const bool bump = mx * cs > m_ref[rt] * cs + kLazyRescale;   // also true when m_ref is -inf and mx is not
    if (__any(bump)) {
      // only the rows that asked move their reference: a row's arithmetic does not depend on its neighbours' keys
      const float m_new = bump ? fmaxf(m_ref[rt], mx) : m_ref[rt];
      const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((m_ref[rt] - m_new) * cs);
      l_part[rt] *= alpha;
      if (!first) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[rt][dt][v] *= alpha;
      }
      m_ref[rt] = m_new;
    }
    const float mc = (m_ref[rt] == -INFINITY) ? 0.f : m_ref[rt] * cs;
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = __builtin_amdgcn_exp2f(s[rt][v] * cs - mc);
      s[rt][v] = e;
      sum += e;
    }
    l_part[rt] += sum;
  }
}

// ---- O^T += V^T P^T for the same 32 keys ---------------------------------------------
// The transposing read serves a 16-lane group with 4 keys x 16 d: lane i16 supplies the address
// of key (i16 / 4), d (4 * (i16 % 4)) and receives the 4 keys of d (i16).  v_fetch issues the
// sixteen reads of a step (it may run ahead of the softmax), pv_step waits for them.
struct VFrags {
  bf16x8 f[4];        // [32-wide d tile] for one 16-key half
};

template <int T>      // T = which 16-key half of the step
__device__ __forceinline__ void v_fetch(unsigned vaddr, const LaneOffsets& lo, VFrags& vf) {
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
    const unsigned a = vaddr + lo.v[dt];
    const s16x4 r0 = lds_read_tr16_b64<T * 16 * 256>(a);
    const s16x4 r1 = lds_read_tr16_b64<T * 16 * 256 + 4 * 256>(a);
    s16x8 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      w[e] = r0[e];
      w[4 + e] = r1[e];
    }
    vf.f[dt] = __builtin_bit_cast(bf16x8, w);
  }
}

template <int NT>
__device__ __forceinline__ bf16x8 pack_p(const f32x16& s, int t) {
  uint4 w;
  w.x = pack_bf16(s[8 * t + 0], s[8 * t + 1]);
  w.y = pack_bf16(s[8 * t + 2], s[8 * t + 3]);
  w.z = pack_bf16(s[8 * t + 4], s[8 * t + 5]);
  w.w = pack_bf16(s[8 * t + 6], s[8 * t + 7]);
  return __builtin_bit_cast(bf16x8, w);
}

// O^T accumulators are updated strictly in place.  Written as assembly with the accumulator tied to
// the destination: through the builtin the register allocator keeps migrating the 64 accumulator
// registers between two homes and pays 64 register moves per step.  The compiler does not know this
// is an MFMA, so the wait states it would insert before the result is read are provided by hand:
// inside the loop the next reader is hundreds of cycles away (after the next step's QK MFMAs), and
// after the loop mfma_results_ready() pads before the epilogue reads the accumulators.
template <bool FIRST_OF_GROUP>
__device__ __forceinline__ void mfma_acc(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  // Wait states between a vector-ALU write of an operand (the packed P fragment, a rescaled
  // accumulator) and the MFMA reading it: five before the first MFMA of a group of four, two before
  // the others.  volatile keeps the issue order of the group, so two MFMAs on one accumulator stay
  // four instructions apart.
  if (FIRST_OF_GROUP)
    asm volatile("s_nop 4\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
  else
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_results_ready(f32x16& a, f32x16& b, f32x16& c, f32x16& d) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// vf0 (keys 0..15 of the step) was fetched before the softmax; the fragments of keys 16..31 are
// fetched here, while the first four MFMAs run.
template <int NT>
__device__ __forceinline__ void pv_step(unsigned vaddr, const LaneOffsets& lo, VFrags& vf0, const f32x16 (&s)[NT],
                                        f32x16 (&oacc)[NT][4]) {
  VFrags vf1;
  v_fetch<1>(vaddr, lo, vf1);
  bf16x8 pf0[NT], pf1[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    pf0[rt] = pack_p<NT>(s[rt], 0);
    pf1[rt] = pack_p<NT>(s[rt], 1);
  }
  lds_wait<8>(vf0.f[0], vf0.f[1], vf0.f[2], vf0.f[3]);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      if (dt == 0) mfma_acc<true>(oacc[rt][dt], vf0.f[dt], pf0[rt]);
      else mfma_acc<false>(oacc[rt][dt], vf0.f[dt], pf0[rt]);
    }
  lds_wait<0>(vf1.f[0], vf1.f[1], vf1.f[2], vf1.f[3]);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      if (dt == 0) mfma_acc<true>(oacc[rt][dt], vf1.f[dt], pf1[rt]);
      else mfma_acc<false>(oacc[rt][dt], vf1.f[dt], pf1[rt]);
    }
}


template <int NT>
__device__ __forceinline__ void zero_state(f32x16 (&oacc)[NT][4], float (&m_ref)[NT], float (&l_part)[NT]) {
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[rt][dt][v] = 0.f;
    m_ref[rt] = -INFINITY;
    l_part[rt] = 0.f;
  }
}

// ---- work units ---------------------------------------------------------------------------
// A unit is consumed in steps of 32 keys; step t covers keys [128 kv_begin + 32 t, +32), i.e. slice
// t % 4 of block kv_begin + t / 4, and every slice has the same layout in LDS.

struct UnitState {
  f32x16 oacc[1][4];
  float m_ref[1], l_part[1];
};

// The un-normalised state of 32 rows of a K/V-split unit, handed to the merge pass: [32 groups of four d][rows][4]
// floats, then the rows' references (log2 units), then their sums.  The order is the one the accumulators have: a
// store instruction writes the same four d of 32 consecutive rows, 512 contiguous bytes per half wavefront.
__device__ __forceinline__ void store_partial(const RunParams& p, const XyDevUnit& u, int rows, int rho, bool valid, int half,
                                              const f32x16 (&oacc)[4], float m2, float l_tot) {
  if (!valid) return;
  char* w = reinterpret_cast<char*>(p.ws + u.ws_offset);
  const unsigned lane_off = (unsigned)(half * rows + rho) * 16u;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 x = {oacc[dt][4 * a], oacc[dt][4 * a + 1], oacc[dt][4 * a + 2], oacc[dt][4 * a + 3]};
      *as_global(reinterpret_cast<f32x4*>(w + (size_t)((8 * dt + 2 * a) * rows * 16) + lane_off)) = x;
    }
  if (half == 0) {
    XY_GLOBAL float* ml = as_global(reinterpret_cast<float*>(w) + (int64_t)rows * kD + rho);
    ml[0] = m2;
    ml[rows] = l_tot;
  }
}

// Normalise and store the rows of a finished narrow unit, or hand its un-normalised state to the merge pass.
__device__ __forceinline__ void finish_unit(const RunParams& p, const XyDevUnit& u, const UnitCtx& c, const Rows<1>& r,
                                            UnitState& st, int col, int half) {
  mfma_results_ready(st.oacc[0][0], st.oacc[0][1], st.oacc[0][2], st.oacc[0][3]);
  const float l_tot = st.l_part[0] + other_half(st.l_part[0]);
  if (u.ws_offset >= 0) {   // K/V-split unit
    const float m2 = (st.m_ref[0] == -INFINITY) ? -INFINITY : st.m_ref[0] * p.c;     // running max, log2 units
    store_partial(p, u, c.rows, col, r.valid[0], half, st.oacc[0], m2, l_tot);
    return;
  }
  if (!r.valid[0]) return;
  const int tl = r.tok[0] - u.q_begin, hl = col - tl * c.hc;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  uint16_t* o = p.out + (int64_t)(u.token_start + u.q_begin + tl) * p.o_ts + (int64_t)(u.head_begin + hl) * p.o_hs;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const u32x2 w2 = {pack_bf16(st.oacc[0][dt][4 * a] * inv, st.oacc[0][dt][4 * a + 1] * inv),
                        pack_bf16(st.oacc[0][dt][4 * a + 2] * inv, st.oacc[0][dt][4 * a + 3] * inv)};
      *as_global(reinterpret_cast<u32x2*>(o + 32 * dt + 8 * a + 4 * half)) = w2;
    }
}

// The wavefronts of a team have each seen some of the keys of one unit: their states meet in LDS (each in its own part
// of the ring, 16-byte groups in register order) and every wavefront puts a share of the d tiles together, in the order of
// the members whatever the order they arrive in.  Every wavefront of the workgroup comes here once.
template <int TEAM>
__device__ __forceinline__ void finish_team(const RunParams& p, const XyDevUnit& u, const UnitCtx& c, const Rows<1>& r, UnitState& st,
                                            unsigned char* smem, const bool exists) {
  constexpr int kTiles = 4 / TEAM;            // d tiles of a wavefront
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5, wave = wave_id(), member = wave & (TEAM - 1);
  mfma_results_ready(st.oacc[0][0], st.oacc[0][1], st.oacc[0][2], st.oacc[0][3]);
  f32x4* const mine = reinterpret_cast<f32x4*>(smem + wave * 32768) + lane;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      mine[64 * (4 * dt + a)] = f32x4{st.oacc[0][dt][4 * a], st.oacc[0][dt][4 * a + 1], st.oacc[0][dt][4 * a + 2], st.oacc[0][dt][4 * a + 3]};
  mine[64 * 16] = f32x4{st.m_ref[0], st.l_part[0] + other_half(st.l_part[0]), 0.f, 0.f};
  __syncthreads();
  if (!exists || !r.valid[0]) return;
  const f32x4* const first = reinterpret_cast<const f32x4*>(smem + (wave - member) * 32768) + lane;      // of member 0
  constexpr int kNext = 32768 / 16;
  float m[TEAM], l[TEAM], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int i = 0; i < TEAM; ++i) {
    const f32x4 ml = first[i * kNext + 64 * 16];
    m[i] = ml[0];
    l[i] = ml[1];
    m_all = fmaxf(m_all, m[i]);
  }
  f32x4 o[kTiles][4] = {};
#pragma unroll
  for (int i = 0; i < TEAM; ++i) {
    const float f = m[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[i] - m_all) * p.c);
    l_all += f * l[i];
#pragma unroll
    for (int k = 0; k < kTiles; ++k)
#pragma unroll
      for (int a = 0; a < 4; ++a) o[k][a] += f * first[i * kNext + 64 * (4 * (kTiles * member + k) + a)];
  }
  if (u.ws_offset >= 0) {                     // as store_partial
    char* w = reinterpret_cast<char*>(p.ws + u.ws_offset) + (unsigned)(half * c.rows + col) * 16u;
#pragma unroll
    for (int k = 0; k < kTiles; ++k)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *as_global(reinterpret_cast<f32x4*>(w + (8 * (kTiles * member + k) + 2 * a) * c.rows * 16)) = o[k][a];
    if (half == 0 && member == 0) {
      XY_GLOBAL float* ml = as_global(p.ws + u.ws_offset + (int64_t)c.rows * kD + col);
      ml[0] = m_all == -INFINITY ? -INFINITY : m_all * p.c;
      ml[c.rows] = l_all;
    }
    return;
  }
  const int tl = r.tok[0] - u.q_begin, hl = col - tl * c.hc;
  const float inv = l_all > 0.f ? 1.f / l_all : 0.f;
  uint16_t* out = p.out + (int64_t)(u.token_start + u.q_begin + tl) * p.o_ts + (int64_t)(u.head_begin + hl) * p.o_hs;
#pragma unroll
  for (int k = 0; k < kTiles; ++k)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const u32x2 w2 = {pack_bf16(o[k][a][0] * inv, o[k][a][1] * inv), pack_bf16(o[k][a][2] * inv, o[k][a][3] * inv)};
      *as_global(reinterpret_cast<u32x2*>(out + 32 * (kTiles * member + k) + 8 * a + 4 * half)) = w2;
    }
}

// ---- wide units (more than 32 rows, MFMA-bound) -------------------------------------------------------
// One wavefront per SIMD, 64 rows (two 32-row tiles) per wavefront: every K or V fragment read from LDS
// feeds two MFMAs, which halves the LDS read traffic per MFMA against one tile per wavefront.  The price is
// registers: the O^T accumulators (2 x 4 x 16) and the Q fragments (2 x 8 x 4) live in AGPRs, S^T, P and the
// K / V fragments in VGPRs, about 450 of the 512 a lone wavefront may use.  With nobody else on the SIMD
// there is nothing to hide a stall behind, so the MFMAs and the LDS reads are issued by hand in a fixed
// interleave, every wait is for exactly the fragment that is needed next, and the compiler's output is
// checked at build time for what it cannot know about such instructions (no spills, no use of a result
// or an operand inside the wait states the hardware needs).

template <int T>      // one 32-wide d tile of v_fetch
__device__ __forceinline__ void v_fetch_one(unsigned vaddr, const LaneOffsets& lo, int dt, bf16x8& f) {
  const unsigned a = vaddr + lo.v[dt];
  const s16x4 r0 = lds_read_tr16_b64<T * 16 * 256>(a);
  const s16x4 r1 = lds_read_tr16_b64<T * 16 * 256 + 4 * 256>(a);
  s16x8 w;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    w[e] = r0[e];
    w[4 + e] = r1[e];
  }
  f = __builtin_bit_cast(bf16x8, w);
}

// O^T tile += V^T fragment x P fragment, accumulator in AGPRs
__device__ __forceinline__ void mfma_pv(f32x16& acc, const bf16x8& vfrag, const bf16x8& pfrag) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(vfrag), "v"(pfrag));
}
// wait states between a vector-ALU write of an MFMA operand and a hand-issued MFMA
__device__ __forceinline__ void valu_to_mfma_gap() { asm volatile("s_nop 4"); }
// The compiler does not know that the registers written by a hand-issued MFMA are not valid yet: where
// control flow merges it may copy them right behind the MFMA.  These statements sit directly behind the
// last MFMA of a sequence (volatile keeps the order, the operands keep every use of the results
// behind them) and pad the wait states a vector-ALU access of an MFMA result needs: settle covers a copy
// the compiler may place there, ready covers a read of the values.  No branch comes between: the copy may stand on either
// side of it.  (The build's check of the assembly follows the branches and reports one that does.)
__device__ __forceinline__ void mfma_settle(f32x16& a) { asm volatile("s_nop 7\n\ts_nop 4" : "+v"(a)); }
__device__ __forceinline__ void settle_a(f32x16& a, f32x16& b, f32x16& c, f32x16& d) {
  asm volatile("s_nop 7\n\ts_nop 4" : "+a"(a), "+a"(b), "+a"(c), "+a"(d));
}
__device__ __forceinline__ void ready_a(f32x16& a, f32x16& b, f32x16& c, f32x16& d) {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(a), "+a"(b), "+a"(c), "+a"(d));
}

template <int N>      // wait until at most N LDS requests are outstanding; tied to the fragment it protects
__device__ __forceinline__ void lds_wait1(bf16x8& a) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(N) : "memory");
}

template <int N>      // the same for the two fragments of a pair of chunks
__device__ __forceinline__ void lds_wait2(bf16x8& a, bf16x8& b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N) : "memory");
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
// the same as one instruction on values that are known to be numbers (MFMA results: the compiler would first
// quiet each of them with a v_max of its own)
__device__ __forceinline__ float max3_raw(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// acc *= alpha without the accumulator leaving the AGPR file for good: the product is forced back into
// an AGPR tuple here, in the rare branch, so the loop-carried value keeps one register class and the
// pipelined path sees no copies.
__device__ __forceinline__ void scale_acc(f32x16& acc, const float alpha) {
  f32x16 t = acc * alpha;
  asm volatile("; rescaled accumulator back in the AGPR file" : "+a"(t));
  acc = t;
}

// A unit with more than 32 rows.  Wavefront w owns rows [32 NT w, 32 NT (w + 1)) as NT 32-row tiles and sees every
// key.  K and V stream through a ring of four 64-key half blocks (32 KB each: 16 KB of K, 16 KB of V);
// a "step" is 32 keys, a "trip" two steps = one half block.
// Iteration t works on three steps at once (the paper's cube / vector overlap of section 4.2.1, at
// instruction level inside one wavefront): the QK^T MFMAs of step t + 1, the softmax arithmetic of step t
// and the PV MFMAs of step t - 1, as sixteen chunks of NT MFMAs (one per row tile, sharing the chunk's
// K or V fragment) with a few vector instructions behind each MFMA and the LDS request of a later chunk behind the first.
// PRESCALE: Q carries the factor c = scale x log2(e), see the softmax notes inside.
// NT: row tiles of a wavefront, two as described, or one, where no unit of the launch has more than 128 rows: with two
// such a unit leaves two of the four wavefronts without rows.  One tile means half the MFMAs, exponentials and rows to
// load and store per wavefront and the same LDS requests.  Eight units alone, K/V in the caches, the whole launch fitted over
// 8 to 32 tiles, us around the loop + a step of 32 keys: 124 rows 9.1 + 0.582 on two tiles, 6.9 + 0.402 on one; 256 rows
// 9.2 + 0.592 on two, as halves (kHalfRows in layout.cpp) 6.9 + 0.400.  248 units of 124 rows on 1 / 4 / 16 tiles
// 13.1 / 23.1 / 54.7 -> 11.1 / 19.3 / 44.4 us: 2.1 us a tile there, the memory's rate; four trees of 31 tokens on 10-20k
// keys, with merge pass, 64.1 -> 61.3 us.
// K fragments asked for eight chunks ahead instead of four changed nothing.
template <int NT>
struct GapTables;
template <>
struct GapTables<2> {
  static constexpr int kExp[33] = XY_GAP_TABLE_EXP, kCvt[33] = XY_GAP_TABLE_CVT, kAdd[33] = XY_GAP_TABLE_ADD;
};
template <>
struct GapTables<1> {
  static constexpr int kExp[17] = XY_GAP_TABLE_ONE_EXP, kCvt[17] = XY_GAP_TABLE_ONE_CVT, kAdd[17] = XY_GAP_TABLE_ONE_ADD;
};
template <bool PRESCALE, bool ROWS_CONTIGUOUS, int NT>
// force: the second pass over a unit whose optimistic pass overflowed (exact prefix in every iteration).  Returns
// whether the unit has to be run again that way (only when force is false; nothing has been written then).
__device__ __forceinline__ bool process_wide(const RunParams& p, const XyDevUnit& u,
                                             unsigned char* smem, int* overflow_flags, const bool force,
                                             const LaneOffsets& lo, const DmaOffsets& dof) {
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const UnitCtx c = make_ctx(p, u);
  const int row_base = 32 * NT * wave;
  const bool active = row_base < c.rows;
  const float inv_hc = __builtin_amdgcn_rcpf((float)c.hc);
  bf16x8 qf[NT][8];
  const int mask_from = c.tree ? c.ctx : c.ctx + u.q_begin + row_base / c.hc + 1;
  const int last_page = (u.ctx_len + u.q_len - 1) >> p.page_shift;
  const int64_t head_off = (int64_t)c.kvh * p.kv_hs;
  const int jfirst = u.kv_begin * kB;
  // (the first half of a unit's tokens may see nothing of the last piece: one step then, in which nothing is visible)
  const int key_end = NT == 1 ? max(c.key_end, jfirst + 1) : c.key_end;
  const int nsteps = (min(u.kv_end * kB, key_end) - jfirst + 31) >> 5;
  const float cs = p.c;

  // ---- softmax with the reference folded into the MFMA ------------------------------------------------
  // The wavefront is bound by the number of instructions it can issue, so the common path of the softmax
  // is cut to exp2, pack and row sum.  The first QK^T MFMA of a step starts from -m_ref (the row's running
  // reference, one value per lane, kept in sixteen registers) instead of zero, so S^T arrives already
  // relative to the reference; with PRESCALE, Q is pre-multiplied by c and S^T is the exponent itself.
  // No row maximum is taken on the common path, and none is looked for either: a row gets its reference from
  // the exact prefix below on the first step in which it sees a key (the true maximum of that step), and keeps
  // it.  Floating point does not care how far later scores lie above the reference as long as nothing
  // overflows - the probabilities, the row sums and the accumulators all carry the same power of two, which
  // the final division removes - so the unit is run optimistically and checked once, at its end: if a row
  // sum has left the range [0, 2^64) (an exponent beyond 2^127 makes it infinite, a mix of infinities NaN),
  // the whole unit is run again (the caller's next turn) with the exact prefix in every iteration, which keeps every probability
  // below 2^8 as the lazy rescale of the narrow path does.  That takes a score 64 log2 units (44 nats) above
  // the largest score of the row's first step: inputs made for it (the needle tests), not attention scores.
  // S^T is kept in "score units": log2 units when Q carries the factor c, raw q.k otherwise.
  const float u2l = PRESCALE ? 1.f : cs;                                   // score units -> log2 units
  const float lazy = PRESCALE ? kLazyRescale : kLazyRescale / cs;         // the lazy-rescale margin in score units
  // ---- the K/V stream (paged cache of section 4.1.1) ---------------------------------------------------
  // Half block h lives in ring slot h & 3; wavefronts 0-1 fetch 32 rows of K each, wavefronts 2-3 32 rows
  // of V.  K and V take the same straight-line path (base pointer and swizzle offsets selected once per unit).
  const uint16_t* kv_base = (wave < 2 ? p.k : p.v) + head_off;
  unsigned dsel[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) dsel[e] = wave < 2 ? dof.k[e] : dof.v;
  const int row_sel = 32 * (wave & 1);
  // After the first half blocks, the eight loads of a request are issued one by one during the trip
  // that follows its set-up, so that their data reaches LDS a kilobyte at a time, between the fragment
  // reads, instead of as one burst.
  // Where the two sixteen-row runs of a request come from (page-table entry, page stride, row in the page) is 64-bit
  // arithmetic on scalars, some thirty scalar instructions per trip, which a lone wavefront can hide behind nothing.
  // The lanes work the addresses out instead, 64 half blocks at a time - lane l holds those of half block
  // 64 * window + l - and a trip reads its four words out of that table.
  const uint16_t* rsrc0 = kv_base;
  const uint16_t* rsrc1 = kv_base;
  unsigned char* rdst = smem;
  unsigned src_lo[2] = {0u, 0u}, src_hi[2] = {0u, 0u};
  int window = 0;
  // (64-bit: lanes far behind the unit's last half block look past any sequence length; they are clamped to
  // the last page like every row behind the sequence's end)
  auto table_row = [&](const int w, const int g) { return (int64_t)jfirst + 64 * (64 * (int64_t)w + lane) + row_sel + 16 * g; };
  auto table_entry = [&](const int w, const int g) {
    const int page = (int)min(table_row(w, g) >> p.page_shift, (int64_t)last_page);
    return p.block_table[(int64_t)u.seq * p.max_blocks + page];
  };
  auto fill_table = [&](const int w, const int entry0, const int entry1) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const uint64_t a = (uint64_t)(kv_base + (int64_t)(g ? entry1 : entry0) * p.kv_bs + (table_row(w, g) & p.page_mask) * p.kv_ts);
      src_lo[g] = (unsigned)a;
      src_hi[g] = (unsigned)(a >> 32);
    }
  };
  auto setup_request = [&](const int h) {
    rdst = smem + (h & 3) * 32768 + (wave >> 1) * 16384 + (wave & 1) * 8192;
    if ((h >> 6) != window) {         // once per 64 trips
      window = h >> 6;
      fill_table(window, table_entry(window, 0), table_entry(window, 1));
    }
    const int l = h & 63;
    // (the lane read returns a signed int: widened through unsigned, or a low word with its top bit set would
    // smear over the high word)
    rsrc0 = reinterpret_cast<const uint16_t*>(((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)src_hi[0], l) << 32) |
                                              (uint64_t)(unsigned)__builtin_amdgcn_readlane((int)src_lo[0], l));
    rsrc1 = reinterpret_cast<const uint16_t*>(((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)src_hi[1], l) << 32) |
                                              (uint64_t)(unsigned)__builtin_amdgcn_readlane((int)src_lo[1], l));
  };
  auto issue = [&](const int idx) {
    const int g = idx >> 2, e = idx & 3;
    const uint16_t* src = g ? rsrc1 : rsrc0;
    if (ROWS_CONTIGUOUS) {
      // rows of 256 bytes back to back: four rows further is 1 KB further in the cache and in LDS alike, so the
      // instruction's offset field moves both and the four loads of a page share their scalar operands
      asm volatile("" : "+v"(dsel[e]));      // keeps it a 32-bit lane offset on a scalar base, not a 64-bit address per lane
      const __attribute__((address_space(1))) void* from =
          (const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(src) + (size_t)dsel[e]);
      __attribute__((address_space(3))) void* to = (__attribute__((address_space(3))) void*)(rdst + 4096 * g);
      switch (e) {      // the offset field is part of the instruction
        case 0: __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0); break;
        case 1: __builtin_amdgcn_global_load_lds(from, to, 16, 1024, 0); break;
        case 2: __builtin_amdgcn_global_load_lds(from, to, 16, 2048, 0); break;
        default: __builtin_amdgcn_global_load_lds(from, to, 16, 3072, 0); break;
      }
    } else {
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(src + (int64_t)(4 * e) * p.kv_ts) + (size_t)dsel[e]),
          (__attribute__((address_space(3))) void*)(rdst + 4096 * g + 1024 * e), 16, 0, 0);
    }
  };
  auto k_slice = [&](const int t) { return lds_addr(smem) + ((t >> 1) & 3) * 32768 + (t & 1) * 8192; };

  // ---- start of a unit -----------------------------------------------------------------------------------
  // What stands around the loop is paid once per unit and by nobody else's time (a short prompt's units spend more
  // here than in the loop), so it is laid out for latency: the page-table entries, then the first two half blocks of K and
  // V and Q are in flight together (what bounds them is the 64 bytes a cycle that LDS-direct loads deliver to a CU, 2000
  // cycles for 128 KB, under which the addresses of Q's rows are worked out), and Q goes through LDS.  Read straight into fragments, a Q load touches
  // 32 rows for 32 bytes each, and the address path of the CU takes about a line per cycle; through LDS an
  // instruction moves four whole rows.  The rows (256 bytes, 16-byte chunks swizzled by the low four bits of the
  // row) wait in ring slots 2 and 3, which are requested when every wavefront has its Q.
  // With the way the results leave (below), the first reference taken without rescaling what is still zero and the
  // last V fragments requested together, a unit of 256 rows alone takes 2.9 us less (what is left: GapTables).
  // K and V stand in front of Q: the compiler waits for the page-table entries together with every LDS-direct load behind
  // them, so behind Q they were asked for when it had landed.  All three have landed at one barrier, and the scaling of Q, the first
  // scores' MFMAs and the requests of half block 2 then share one stretch of code instead of following each other.  With
  // the record read as a whole, us before / after: a suffix of 160 tokens beside 24 decodes, planned, appended and merged,
  // eight layers 247.7 / 241.0; eight prompts of 60-4000 tokens 121.7 / 117.8; a chunk of 128 tokens beside three narrow sequences 10.4 / 10.2.
  const int entry0 = table_entry(0, 0), entry1 = table_entry(0, 1);
  __syncthreads();                                          // the ring is free
  fill_table(0, entry0, entry1);
  auto request_now = [&](const int h) {
    setup_request(h);
#pragma unroll
    for (int idx = 0; idx < 8; ++idx) issue(idx);
  };
  request_now(0);
  request_now(1);
  unsigned char* const wave_buf = smem + 65536 + wave * (8192 * NT);        // 32 NT rows of 256 bytes
  const int sub = lane >> 4, pos = lane & 15;               // a load or store of four rows: row, 16-byte chunk
  auto rows_in_order = [&](const int e) { return row_index(min(row_base + 4 * e + sub, c.rows - 1), c.hc, inv_hc); };
  auto chunk_of = [&](const int e) { return (pos ^ ((4 * e + sub) & 15)) << 4; };
  if (active) {
    const char* q0 = reinterpret_cast<const char*>(p.q + (int64_t)(u.token_start + u.q_begin) * p.q_ts + (int64_t)u.head_begin * p.q_hs);
    auto q_load = [&](const char* from, const int e) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                       (__attribute__((address_space(3))) void*)(wave_buf + 1024 * e), 16, 0, 0);
    };
    if (p.q_ts < kSmallStride && p.q_hs < kSmallStride) {
#pragma unroll
      for (int e = 0; e < 8 * NT; ++e) q_load(q0 + row_bytes<true>(rows_in_order(e), p.q_ts, p.q_hs) + chunk_of(e), e);
    } else {
#pragma unroll 1
      for (int e = 0; e < 8 * NT; ++e) q_load(q0 + row_bytes<false>(rows_in_order(e), p.q_ts, p.q_hs) + chunk_of(e), e);
    }
  }
  // the rows a lane owns, while the loads are in flight
  Rows<NT> r;
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    const int rho = row_base + 32 * rt + col;
    r.valid[rt] = rho < c.rows;
    r.tok[rt] = u.q_begin + row_index(min(rho, c.rows - 1), c.hc, inv_hc).tl;
    r.lim[rt] = r.valid[rt] ? c.ctx + r.tok[rt] + 1 : 0;
    r.mw0[rt] = r.mw1[rt] = 0;
    if (c.tree && r.valid[rt]) {
      const uint32_t* mrow = p.masks + u.mask_off + (int64_t)r.tok[rt] * c.wpr;
      r.mw0[rt] = mrow[0];
      if (c.wpr > 1) r.mw1[rt] = mrow[1];
    }
  }
  f32x16 oacc[NT][4];
  float m_ref[NT], l_part[NT][4];      // four running partial row sums per tile, added to in place (plain additions:
                                        // the bf16 dot-product instruction would hold the matrix pipe for 16 cycles)
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[rt][dt][v] = 0.f;
    m_ref[rt] = -INFINITY;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) asm volatile("" : "+a"(oacc[rt][dt]));      // zeros written here, not next to the first MFMA
#pragma unroll
    for (int i = 0; i < 4; ++i) l_part[rt][i] = 0.f;
  }
  f32x16 negm[NT];          // -m_ref of the lane's row in all sixteen registers (0 while the row has no reference)
#pragma unroll
  for (int rt = 0; rt < NT; ++rt)
#pragma unroll
    for (int v = 0; v < 16; ++v) negm[rt][v] = 0.f;
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) asm volatile("" : "+v"(negm[rt]));
  wait_vmcnt<0>();                                          // this wavefront's part of half blocks 0 and 1, and Q
  if (active) {
    const unsigned qaddr = lds_addr(wave_buf) + col * 256;
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        qf[rt][ks] = lds_read_b128<0>(qaddr + rt * 8192 + (((2 * ks + half) ^ (col & 15)) << 4));
      lds_wait<4>(qf[rt][0], qf[rt][1], qf[rt][2], qf[rt][3]);
      lds_wait<0>(qf[rt][4], qf[rt][5], qf[rt][6], qf[rt][7]);
    }
  }
  __builtin_amdgcn_s_barrier();                             // half blocks 0 and 1 are there for everybody, slots 2 and 3 are free
  auto scale_q = [&](const int ks) {
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      if (PRESCALE) {
        uint4 w = __builtin_bit_cast(uint4, qf[rt][ks]);
        unsigned* wp = reinterpret_cast<unsigned*>(&w);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          wp[i] = pack_bf16(__uint_as_float(wp[i] << 16) * cs, __uint_as_float(wp[i] & 0xffff0000u) * cs);
        qf[rt][ks] = __builtin_bit_cast(bf16x8, w);
      }
      asm volatile("; Q fragment lives in the AGPR file from here on" : "+a"(qf[rt][ks]));
    }
  };

  f32x16 sa[NT], sb[NT];
  bf16x8 pa[NT][2], pb[NT][2];
  bf16x8 kf[8], vf[8];
  auto request_k = [&](const unsigned kaddr, const int i) { kf[i] = lds_read_b128<0>(kaddr + lo.k[i]); };
  auto request_v = [&](const unsigned vaddr, const int i) {
    if (i < 4) v_fetch_one<0>(vaddr, lo, i, vf[i]);
    else v_fetch_one<1>(vaddr, lo, i - 4, vf[i]);
  };
  auto mfma_qk = [&](const int i, f32x16& s, const int rt) {     // chunk i of S^T(rt) = -m_ref + K Q^T
    if (i == 0)
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(s) : "v"(kf[0]), "a"(qf[rt][0]), "v"(negm[rt]));
    else
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(kf[i]), "a"(qf[rt][i]));
  };
  auto lane_max = [&](const f32x16& s) {
    const float a0 = max3(s[0], s[1], s[2]), a1 = max3(s[3], s[4], s[5]), a2 = max3(s[6], s[7], s[8]);
    const float a3 = max3(s[9], s[10], s[11]), a4 = max3(s[12], s[13], s[14]);
    return fmaxf(max3(a0, a1, a2), max3(a3, a4, s[15]));
  };
  // whether some valid row of this wavefront has no reference yet (it has not seen a key so far): the next
  // iteration then starts with the exact prefix too.  Wavefront-uniform; changes only where the references change.
  bool pending = true;

  // Exact prefix of an iteration (always in iteration 0, where it gives every row that sees a key its first
  // reference; after that only while some row is still waiting for its first key, or in the second pass over
  // a unit): the true row maximum of the masked s_in moves the reference, and everything
  // that was built against the old one follows it (the scores of this step, the row sums, the
  // accumulators, the packed probabilities of the previous step whose PV product is still to come), so
  // that the pipelined iteration runs unchanged afterwards.  A row that has a reference moves it by a
  // whole number of log2 units, which makes the factor a power of two: the packed probabilities are
  // rescaled without rounding.
  // first: iteration 0, in which nothing has been built against a reference yet.
  auto exact_prefix = [&](const bool first, f32x16 (&s_in)[NT], bf16x8 (&p_in)[NT][2]) {
    if (!first) {
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) ready_a(oacc[rt][0], oacc[rt][1], oacc[rt][2], oacc[rt][3]);
    }
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      const float mx = max_both_halves(lane_max(s_in[rt]));       // relative to the reference
      const bool set = !first && m_ref[rt] != -INFINITY;
      float delta, alpha;
      if (set) {
        const float d2 = mx >= lazy ? ceilf(mx * u2l) : 0.f;      // whole number of log2 units
        delta = PRESCALE ? d2 : d2 / cs;
        alpha = __builtin_amdgcn_exp2f(-d2);
        m_ref[rt] += delta;
      } else {
        delta = mx != -INFINITY ? mx : 0.f;
        alpha = 1.f;
        if (mx != -INFINITY) m_ref[rt] = mx;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) s_in[rt][v] -= delta;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (!first) l_part[rt][i] *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        if (!first) scale_acc(oacc[rt][dt], alpha);
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        if (first) break;
        uint4 w = __builtin_bit_cast(uint4, p_in[rt][h2]);
        unsigned* wp = reinterpret_cast<unsigned*>(&w);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          wp[i] = pack_bf16(__uint_as_float(wp[i] << 16) * alpha, __uint_as_float(wp[i] & 0xffff0000u) * alpha);
        p_in[rt][h2] = __builtin_bit_cast(bf16x8, w);
      }
      const float nm = m_ref[rt] == -INFINITY ? 0.f : -m_ref[rt];
#pragma unroll
      for (int v = 0; v < 16; ++v) negm[rt][v] = nm;
      asm volatile("" : "+v"(negm[rt]));      // sixteen real registers from here on, nothing rebuilt next to the MFMA
    }
    bool waiting = false;
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) waiting = waiting || (r.valid[rt] && m_ref[rt] == -INFINITY);
    pending = __builtin_amdgcn_ballot_w64(waiting) != 0;
  };

  // Iteration t: QK^T of step t + 1 (chunks 0-7), exp2 / pack / row sum of step t (one pair of scores per
  // chunk), PV of step t - 1 (chunks 8-15).  The LDS request issued in a chunk is the fragment needed four
  // chunks later; par >= 0 numbers the iteration inside its trip for the K/V loads it issues.  Returns
  // whether the next iteration starts with the exact prefix; par == -1 marks iteration 0, par == -2 the iteration
  // after which no other follows (its look-ahead scores are never read).
  // kaddr, vaddr, knext: LDS addresses of K of step t + 1, V of step t - 1 and K of step t + 2 (worked out
  // once per trip by the caller).
  auto iterate = [&](const bool exact, const int par, const int t, const unsigned kaddr, const unsigned vaddr,
                     const unsigned knext, f32x16 (&s_in)[NT], f32x16 (&s_out)[NT], bf16x8 (&p_in)[NT][2],
                     bf16x8 (&p_out)[NT][2]) -> bool {
    {
      const int j = jfirst + 32 * t;
      if (j + 32 > mask_from) mask_step<NT>(p, c, r, j + 8 * half, s_in);
    }
    if (exact) {
      exact_prefix(par == -1, s_in, p_in);
      valu_to_mfma_gap();       // the prefix rewrote the reference registers the first MFMA reads
    }
    lds_wait<0>(kf[0], kf[1], kf[2], kf[3]);
    unsigned packed[8 * NT];
    float e[16 * NT];
    // A lone wavefront issues in order: an MFMA that finds the matrix pipe busy holds up everything behind
    // it, and a gap with more than about 26 cycles of other instructions leaves the pipe idle.  So the
    // vector work of the iteration is dealt out over the 32 gaps behind its MFMAs (two per chunk) by a table
    // made offline from the issue costs measured for a lone wavefront (exp2 8.5 cycles, other vector
    // instructions 5, an LDS request 5.7, a scalar instruction 8.5, a wait 4.7), next to what a gap holds
    // anyway (LDS requests, waits, the K/V loads): about 24 cycles in every gap.  Scheduling barriers keep the
    // compiler from moving work between gaps.  The tables count, gap by gap, how many of the 32 exponentials,
    // 16 packings and 32 row-sum additions are done before that gap.
    typedef GapTables<NT> Gaps;
    auto exp_one = [&](const int j) {          // score j & 15 of row tile j >> 4
      e[j] = __builtin_amdgcn_exp2f(PRESCALE ? s_in[j >> 4][j & 15] : s_in[j >> 4][j & 15] * cs);
    };
    auto cvt_one = [&](const int g) {
      packed[g] = pack_bf16(e[2 * g], e[2 * g + 1]);
      asm volatile("" : "+v"(packed[g]));       // stays in this gap
    };
    auto add_one = [&](const int j) {
      l_part[j >> 4][j & 3] += e[j];
      asm volatile("" : "+v"(l_part[j >> 4][j & 3]));
    };
    auto gap_work = [&](const int k) {
#pragma unroll
      for (int j = Gaps::kExp[k]; j < Gaps::kExp[k + 1]; ++j) exp_one(j);
#pragma unroll
      for (int g = Gaps::kCvt[k]; g < Gaps::kCvt[k + 1]; ++g) cvt_one(g);
#pragma unroll
      for (int j = Gaps::kAdd[k]; j < Gaps::kAdd[k + 1]; ++j) add_one(j);
    };
#pragma unroll
    for (int ch = 0; ch < 16; ++ch) {
      // one wait per pair of chunks: before an even chunk, for its own fragment and the next one.  The
      // number allowed to stay outstanding is what has been requested behind those two (K fragments are
      // one request each, V fragments two).
      if (ch == 4) lds_wait2<2>(kf[4], kf[5]);        // behind them: kf6 kf7
      if (ch == 6) lds_wait2<4>(kf[6], kf[7]);        // vf0 vf1
      if (ch == 8) lds_wait2<4>(vf[0], vf[1]);        // vf2 vf3
      if (ch == 10) lds_wait2<4>(vf[2], vf[3]);       // vf4 vf5
      if (ch == 12) lds_wait2<4>(vf[4], vf[5]);       // vf6 vf7
      if (ch == 14) lds_wait2<2>(vf[6], vf[7]);       // kf0 kf1 of the next step
      auto mfma_of = [&](const int rt) {
        if (ch < 8) mfma_qk(ch, s_out[rt], rt);
        else mfma_pv(oacc[rt][(ch - 8) & 3], vf[ch - 8], p_in[rt][(ch - 8) >> 2]);
      };
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) {
        __builtin_amdgcn_sched_barrier(0);
        mfma_of(rt);
        __builtin_amdgcn_sched_barrier(0);
        if (rt == 0) {                                  // the LDS request of the chunk: the fragment needed four chunks on
          if (ch < 4) request_k(kaddr, 4 + ch);
          else if (ch < 12) request_v(vaddr, ch - 4);
          else request_k(knext, ch - 12);
        }
        gap_work(NT * ch + rt);
      }
      if (par >= 0 && (ch & 3) == 1) issue(4 * par + (ch >> 2));      // this trip's share of the K/V stream
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      p_out[rt][0] = __builtin_bit_cast(bf16x8, uint4{packed[8 * rt + 0], packed[8 * rt + 1], packed[8 * rt + 2], packed[8 * rt + 3]});
      p_out[rt][1] = __builtin_bit_cast(bf16x8, uint4{packed[8 * rt + 4], packed[8 * rt + 5], packed[8 * rt + 6], packed[8 * rt + 7]});
    }
    // S^T of the next step stays allocated until its MFMAs have long retired, also when nobody reads it.
    // (Only then: where the next iteration reads it, the same statement makes the allocator copy all 32
    // registers behind every iteration.)
    if (par == -2) {
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) asm volatile("" : "+v"(s_out[rt]));
      return false;
    }
    return force || pending;      // wavefront-uniform
  };
  bool exact = true;
  if (active) {
    // iteration 0 multiplies V of step 0 already (by zeros, see below): cleared first where that is the last step
    if (nsteps == 1) zero_tail_rows(k_slice(0) + 16384, min(u.kv_end * kB, key_end) - jfirst, lane);
    // S^T of step 0 against reference 0 under the scaling of Q, with the requests of half block 2 (K(0..3), V(0..2) in all)
    // in between; then iteration 0 (exact prefix, no previous step)
#pragma unroll
    for (int i = 0; i < 8; ++i) request_k(k_slice(0), i);
    setup_request(2);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      if (i < 8) {
        scale_q(i);
        issue(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i == 1) lds_wait<4>(kf[0], kf[1], kf[2], kf[3]);
      if (i == 5) lds_wait<0>(kf[4], kf[5], kf[6], kf[7]);
      if (i == 8) valu_to_mfma_gap();
      if (i > 0) {
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) mfma_qk(i - 1, sa[rt], rt);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) mfma_settle(sa[rt]);      // ahead of the branch
    if (wave < 2) request_now(3);
#pragma unroll
    for (int i = 0; i < 4; ++i) request_k(k_slice(1), i);
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      pb[rt][0] = pb[rt][1] = bf16x8{};
      asm volatile("" : "+v"(pb[rt][0]), "+v"(pb[rt][1]));
    }
    // iteration 0 has no previous step: its probabilities are zero and meet V of step 0 (keys of the unit, or zeros)
    exact = iterate(true, -1, 0, k_slice(1), k_slice(0) + 16384, k_slice(2), sa, sb, pb, pa);
  } else {
    request_now(2);
    if (wave < 2) request_now(3);
  }
  const int hshift = wave < 2 ? 5 : 4;
  auto hreq = [&](const int j) { return j + hshift; };
  auto end_trip = [&](const int j) {
    // K is consumed one trip ahead of V, so K(j + 5) and V(j + 4) replace what trip j has finished with;
    // they are issued during trip j + 1.  Only the eight loads issued during trip j may still be in flight.
    wait_vmcnt<8>();
    __builtin_amdgcn_s_barrier();
    setup_request(hreq(j));
  };
  end_trip(-1);
  int j = 0;
#pragma unroll 1
  for (; 2 * j + 2 < nsteps; ++j) {
    if (active) {
      // ring slots of half blocks j (V of this trip), j + 1 (K of this trip) and j + 2 (K fragments ahead)
      const unsigned s0 = lds_addr(smem) + (j & 3) * 32768, s1 = lds_addr(smem) + ((j + 1) & 3) * 32768,
                     s2 = lds_addr(smem) + ((j + 2) & 3) * 32768;
      exact = iterate(exact, 0, 2 * j + 1, s1, s0 + 16384, s1 + 8192, sb, sa, pa, pb);
      exact = iterate(exact, 1, 2 * j + 2, s1 + 8192, s0 + 16384 + 8192, s2, sa, sb, pb, pa);
      // no padding behind the last PV MFMAs here: the end of the trip (wait, barrier, next request) stands between
      // them and the next iteration, and the build-time check of the assembly would report a copy placed earlier
    } else {
#pragma unroll
      for (int idx = 0; idx < 8; ++idx) issue(idx);
    }
    end_trip(j);
  }
  if (2 * j + 1 < nsteps) {     // one more step: no refill (the last PV below still reads V of half block j)
    if (active) {
      iterate(exact, -2, 2 * j + 1, k_slice(2 * j + 2), k_slice(2 * j) + 16384, k_slice(2 * j + 3), sb, sa, pa, pb);
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) settle_a(oacc[rt][0], oacc[rt][1], oacc[rt][2], oacc[rt][3]);
    }
  }
  if (active) {                 // PV of the last step
    lds_wait1<0>(kf[0]); lds_wait1<0>(kf[1]); lds_wait1<0>(kf[2]); lds_wait1<0>(kf[3]);
    const unsigned vaddr = k_slice(nsteps - 1) + 16384;
    const int last_keys = min(u.kv_end * kB, key_end) - jfirst - 32 * (nsteps - 1);     // keys of the last step: 1 .. 32
    if (last_keys < 32) zero_tail_rows(vaddr, last_keys, lane);
    bf16x8 p_last[NT][2];
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      p_last[rt][0] = (nsteps & 1) ? pa[rt][0] : pb[rt][0];
      p_last[rt][1] = (nsteps & 1) ? pa[rt][1] : pb[rt][1];
      asm volatile("" : "+v"(p_last[rt][0]), "+v"(p_last[rt][1]));     // selected here, not next to the MFMAs
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) request_v(vaddr, i);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i == 0) lds_wait<8>(vf[0], vf[1], vf[2], vf[3]);          // two requests a fragment
      if (i == 4) lds_wait<0>(vf[4], vf[5], vf[6], vf[7]);
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) mfma_pv(oacc[rt][i & 3], vf[i], p_last[rt][i >> 2]);
    }
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) ready_a(oacc[rt][0], oacc[rt][1], oacc[rt][2], oacc[rt][3]);
  }
  // The check of the optimistic pass.  All four wavefronts stream K/V together, so they repeat the unit together.
  bool bad = false;
  if (active) {
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      const float l_lane = (l_part[rt][0] + l_part[rt][1]) + (l_part[rt][2] + l_part[rt][3]);
      bad = bad || (r.valid[rt] && !(l_lane < kRowSumLimit));      // also true for NaN
    }
  }
  const bool wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
  if (lane == 0) overflow_flags[wave] = wave_bad ? 1 : 0;
  wait_vmcnt<0>();            // no load of the stream lands in the ring after the barrier
  __syncthreads();
  const int any_bad = overflow_flags[0] | overflow_flags[1] | overflow_flags[2] | overflow_flags[3];
  // The second pass is the caller's next turn of its loop over the units, not a loop in here: what a loop around
  // this function would keep alive across the main loop costs more registers than the wide units have to spare.
  if (__builtin_amdgcn_readfirstlane(any_bad) != 0 && !force) return true;
  if (!active) return false;
  float l_tot[NT];
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    const float l_lane = (l_part[rt][0] + l_part[rt][1]) + (l_part[rt][2] + l_part[rt][3]);
    l_tot[rt] = l_lane + other_half(l_lane);
  }
  if (u.ws_offset >= 0) {
#pragma unroll
    for (int rt = 0; rt < NT; ++rt)
      store_partial(p, u, NT == 1 ? (u.flags >> kSlabRowsShift) & 0xfff : c.rows,       // the unit may be a half of its family
                    (NT == 1 ? u.flags >> kSlabFirstShift : 0) + row_base + 32 * rt + col, r.valid[rt], half, oacc[rt],
                    m_ref[rt] == -INFINITY ? -INFINITY : m_ref[rt] * u2l, l_tot[rt]);
    return false;
  }
  // A lane holds four consecutive d of a row at a time; stored as they are, an instruction writes sixteen bytes of each
  // of 32 rows.  Through the wavefront's part of the ring (nobody reads it any more: the barrier of the check above
  // stands behind the last use and behind the last load) it writes four whole rows.
#pragma unroll
  for (int rt = 0; rt < NT; ++rt) {
    const float inv = l_tot[rt] > 0.f ? 1.f / l_tot[rt] : 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        uint2 w2;
        w2.x = pack_bf16(oacc[rt][dt][4 * a] * inv, oacc[rt][dt][4 * a + 1] * inv);
        w2.y = pack_bf16(oacc[rt][dt][4 * a + 2] * inv, oacc[rt][dt][4 * a + 3] * inv);
        *reinterpret_cast<uint2*>(wave_buf + (32 * rt + col) * 256 + (((4 * dt + a) ^ (col & 15)) << 4) + 8 * half) = w2;
      }
  }
  char* o0 = reinterpret_cast<char*>(p.out + (int64_t)(u.token_start + u.q_begin) * p.o_ts + (int64_t)u.head_begin * p.o_hs);
  auto o_store = [&](const int e, const int64_t off) {
    const uint4 w = *reinterpret_cast<const uint4*>(wave_buf + 1024 * e + 16 * lane);
    if (row_base + 4 * e + sub < c.rows) *reinterpret_cast<uint4*>(o0 + off + chunk_of(e)) = w;
  };
  // With heads that divide sixteen and every row there, sixteen rows further is so many tokens further, and all but the first
  // four offsets follow by one addition instead of some sixteen instructions a store.  us without / with it, append and merge
  // included, both in turn, on two boxes: eight prompts of 60-4000 tokens 118.3 / 117.1, eight suffixes of 1024 on 4-16k 810.5 / 804.2,
  // a chunk of 128 tokens beside three narrow sequences 10.15 / 10.01, a chunk of 1024 on 20-24k 321.8 / 320.1.  The other way
  // round: eight layers of a suffix of 160 tokens beside 24 decodes 243.5 / 245.2, though its wide units are all cut and leave above,
  // as those of the chunk do.  A cut unit runs the same blocks but for a few lane reads of spilled scalars, and fewer spilled ones
  // (132 -> 114, with the strides read afresh here), a loop around the stores or hints on the branches left the loss at 0.5 to 1 %:
  // what remains is where the code lies in a kernel of 221 KB.  Other head groups keep the general way: with one of 64-bit offsets
  // in a loop for them short prompts of 3, 5, 6 and 12 heads a group were 1 to 4 % slower.
  const bool small_o = p.o_ts < kSmallStride && p.o_hs < kSmallStride;
  int hc = c.hc;
  asm volatile("" : "+s"(hc));      // what follows from it is worked out here, not kept from the start of the unit
  // whether sixteen rows further is so many tokens further, for all rows of the wavefront, and how many bytes that are (as
  // functions: written into the branch the kernel for short units on two row tiles takes 8 bytes of scratch memory)
  auto in_step = [&](const int hc) { return hc <= 16 && (hc & (hc - 1)) == 0 && row_base + 32 * NT <= c.rows; };
  auto step16 = [&](const int hc, const int64_t ts) { return (32u >> (__builtin_ctz(hc) & 31)) * (unsigned)ts; };
  if (small_o && in_step(hc)) {
    unsigned off[4];
    const unsigned step = step16(hc, p.o_ts);
#pragma unroll
    for (int e = 0; e < 4; ++e) off[e] = (unsigned)row_bytes<true>(rows_in_order(e), p.o_ts, p.o_hs) + chunk_of(e);
#pragma unroll
    for (int e = 0; e < 8 * NT; ++e) {
      *reinterpret_cast<uint4*>(o0 + (size_t)off[e & 3]) = *reinterpret_cast<const uint4*>(wave_buf + 1024 * e + 16 * lane);
      off[e & 3] += step;
    }
  } else if (small_o) {
#pragma unroll
    for (int e = 0; e < 8 * NT; ++e) o_store(e, row_bytes<true>(rows_in_order(e), p.o_ts, p.o_hs));
  } else {
#pragma unroll 1
    for (int e = 0; e < 8 * NT; ++e) o_store(e, row_bytes<false>(rows_in_order(e), p.o_ts, p.o_hs));
  }
  return false;
}

// A unit with at most 32 rows (decode, short verify; bandwidth-bound).  TEAM = 1: one wavefront processes the
// whole unit on its own, streaming 32-key slices through a private ring of one or two slices (K and V slots, each
// refilled as soon as it has been consumed).  No barrier, no cross-wavefront merge: four such
// units are in flight per CU and hide each other's latencies.
// TEAM = 2, 4: so many wavefronts share the unit, each with every TEAM-th slice from its place in the team on, and finish_team
// puts their states together behind a barrier of the workgroup; exists: whether the team has a unit at all.
// Two slices (narrow_depth) with teams and where a launch has at most kDeepTiles tiles per wavefront: with every wavefront at work
// the card's bandwidth is the bound and 16 KB each are enough, but a wavefront whose neighbours have run out of work waits
// for memory in every slice, and that is the end of every launch.  8 decodes x 32 KV heads on 2-6k tokens (7.5 tiles per
// wavefront), this kernel alone, 83.9 -> 82.4 us with two; 128 trees on 512-4096 tokens (14 tiles) 148.2 -> 150.7 us, so those keep one;
// 128 decodes on 2-16k (54 tiles) are level, 552.8 / 552.1.  Launches of short units take process_short instead.
template <int TEAM>
__device__ __forceinline__ void process_solo(const RunParams& p, const XyDevUnit& u, unsigned char* smem, const LaneOffsets& lo,
                                             const DmaOffsets& dof, const bool exists = true) {
  constexpr int NT = 1;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const UnitCtx c = make_ctx(p, u);
  const int mask_from = c.tree ? c.ctx : c.ctx + u.q_begin + 1;
  const XY_CONST int32_t* table = as_const(p.block_table) + (int64_t)u.seq * p.max_blocks;
  const int last_page = (u.ctx_len + u.q_len - 1) >> p.page_shift;
  const int64_t head_off = (int64_t)c.kvh * p.kv_hs;
  const int jfirst = u.kv_begin * kB;
  const int slices = (min(u.kv_end * kB, c.key_end) - jfirst + 31) >> 5, member = wave & (TEAM - 1);
  const int nsteps = TEAM == 1 ? slices : exists ? (slices - member + TEAM - 1) / TEAM : 0;      // of this wavefront
  auto key_of = [&](const int t) { return jfirst + 32 * (TEAM * t + member); };                 // first key of its step t
  unsigned char* ring = smem + wave * 32768;        // one or two slices of [K 8 KB | V 8 KB]
  const int depth = p.narrow_depth;
  const unsigned ring_addr = lds_addr(ring);
  // a 32-key slice starting at key j: two runs of sixteen rows, each inside one page (page j / page size of the sequence, slot
  // j % page size, paper section 4.1.1; pages hold 16, 32, 64 or 128 tokens); eight
  // instructions per tensor, which is what the waits below count
  struct Slice {
    int64_t run[2];
  };
  // page-table entries of the two runs of slice t: asked for early (entries), turned into addresses later (locate)
  struct Entries {
    int e[2];
  };
  auto entries = [&](const int t) {
    Entries n;
#pragma unroll
    for (int g = 0; g < 2; ++g) n.e[g] = table[min((key_of(t) + 16 * g) >> p.page_shift, last_page)];
    return n;
  };
  Entries entries0 = {}, entries1 = {};
  if (TEAM == 1 || nsteps > 0) {
    entries0 = entries(0);
    entries1 = entries(1);
  }
  Rows<NT> r;
  bf16x8 qf[NT][8];
  const float inv_hc = __builtin_amdgcn_rcpf((float)c.hc);
  setup_rows(p, u, c, col, inv_hc, r);
  UnitState st;
  zero_state<NT>(st.oacc, st.m_ref, st.l_part);
  auto locate = [&](const int t, const Entries& n) {
    Slice at;
#pragma unroll
    for (int g = 0; g < 2; ++g)
      at.run[g] = (int64_t)n.e[g] * p.kv_bs + (int64_t)((key_of(t) + 16 * g) & p.page_mask) * p.kv_ts + head_off;
    return at;
  };
  auto load_slice = [&](const Slice& at, const int t, const bool want_k, const bool want_v) {
    unsigned char* slot = ring + (t & (depth - 1)) * 16384;
#pragma unroll
    for (int g = 0; g < 2; ++g)
      load_rows_async<4>(p.k + at.run[g], p.v + at.run[g], p.kv_ts, 0, slot + 4096 * g, slot + 8192 + 4096 * g, dof, want_k, want_v);
  };
  // Q goes through LDS as in the wide units (whole rows, 16-byte chunks swizzled by the low four bits of the row), and
  // not only for that: a load whose result the compiler sees would be waited for with everything that is in flight.
  // It waits where V of the second slice comes to lie, which is asked for when Q has been read.
  unsigned char* const q_buf = ring + 16384 + 8192;
  if (TEAM == 1 || nsteps > 0) {
    const int sub = lane >> 4, pos = lane & 15;             // a load moves four rows: row, 16-byte chunk
    const char* q0 = reinterpret_cast<const char*>(p.q + (int64_t)(u.token_start + u.q_begin) * p.q_ts + (int64_t)u.head_begin * p.q_hs);
    auto load_q = [&](const char* from, const int e) {
      __builtin_amdgcn_global_load_lds((const XY_GLOBAL void*)from, (__attribute__((address_space(3))) void*)(q_buf + 1024 * e), 16, 0, 0);
    };
    auto q_row = [&](const int e) { return q0 + row_bytes<false>(row_index(min(4 * e + sub, c.rows - 1), c.hc, inv_hc), p.q_ts, p.q_hs); };
    // the mask words are waited for here: behind a load to LDS the compiler can only wait for everything in flight
    if (c.tree) asm volatile("" : "+v"(r.mw0[0]), "+v"(r.mw1[0]));
    if ((c.hc == 4 || c.hc <= 2) && (c.rows & 3) == 0) {                 // whole groups of four, 4 / hc tokens further each
      const char* from = q_row(0);
      const int64_t step = (c.hc == 4 ? 2 : c.hc == 2 ? 4 : 8) * p.q_ts;      // bytes
      const int chunk = (pos ^ sub) << 4;
      for (int e = 0; 4 * e < c.rows; ++e, from += step) load_q(from + (chunk ^ ((e & 3) << 6)), e);
    } else {
      for (int e = 0; 4 * e < c.rows; ++e) load_q(q_row(e) + ((pos ^ ((4 * e + sub) & 15)) << 4), e);
    }
    // all four here, behind Q: left to itself the compiler widens each entry as soon as it is asked for, and a unit
    // starts with four round trips one after the other
    asm volatile("" : "+s"(entries0.e[0]), "+s"(entries0.e[1]), "+s"(entries1.e[0]), "+s"(entries1.e[1]));
    const Slice first = locate(0, entries0), second = locate(1, entries1);
    load_slice(first, 0, true, false);          // issue order K, V
    load_slice(first, 0, false, true);
    const bool two = depth == 2 && nsteps > 1;
    if (two) {
      load_slice(second, 1, true, false);
      wait_vmcnt<24>();                         // Q has landed
    } else {
      wait_vmcnt<16>();
    }
    const int row = min(col, c.rows - 1);
    const unsigned qaddr = lds_addr(q_buf) + row * 256;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[0][ks] = lds_read_b128<0>(qaddr + (((2 * ks + half) ^ (row & 15)) << 4));
    lds_wait<4>(qf[0][0], qf[0][1], qf[0][2], qf[0][3]);
    lds_wait<0>(qf[0][4], qf[0][5], qf[0][6], qf[0][7]);
    if (two) load_slice(second, 1, false, true);
  }
#pragma unroll 1
  for (int t = 0; t < nsteps; ++t) {
    const unsigned kaddr = ring_addr + (t & (depth - 1)) * 16384, vaddr = kaddr + 8192;
    const int left = nsteps - 1 - t;          // slices behind this one: depth - 1 of them in flight
    Entries ahead = entries(t + depth);       // arrive while K is waited for
    if (depth == 2 && left > 0) wait_vmcnt<24>();      // K(t) has landed
    else wait_vmcnt<8>();
    asm volatile("" : "+s"(ahead.e[0]), "+s"(ahead.e[1]));      // here, not among the fragment reads that follow
    const Slice next = locate(t + depth, ahead);
    f32x16 s[NT];
    VFrags vf;
    qk_step<NT>(kaddr, lo, qf, s);            // all K reads have completed when this returns
    if (left >= depth) {      // the K slot is free again
      load_slice(next, t, true, false);
      if (depth == 2) wait_vmcnt<24>();       // V(t) has landed
      else wait_vmcnt<8>();
    } else if (left > 0) {
      wait_vmcnt<16>();
    } else {
      wait_vmcnt<0>();
      const int last_keys = min(u.kv_end * kB, c.key_end) - key_of(t);      // keys of the last step: 1 .. 32
      if (last_keys < 32) zero_tail_rows(vaddr, last_keys, lane);
    }
    v_fetch<0>(vaddr, lo, vf);                // the first V fragments arrive while the softmax runs
    const int j = key_of(t);
    if (j + 32 > mask_from) mask_step<NT>(p, c, r, j + 8 * half, s);
    softmax_step<NT>(p.c, s, st.m_ref, st.l_part, st.oacc, t == 0);
    pv_step<NT>(vaddr, lo, vf, s, st.oacc);   // all V reads have completed when this returns
    if (left >= depth) load_slice(next, t, false, true);
  }
  if constexpr (TEAM == 1) finish_unit(p, u, c, r, st, col, half);
  else finish_team<TEAM>(p, u, c, r, st, smem, exists);
}

// A unit of at most 32 rows in a launch of short ones (kShortSlices): one slice at a time, Q straight into registers and
// no address worked out before its turn.  Such a unit is bound by the instructions of a lone wavefront and by the three
// round trips to memory that follow each other (record, page table, K/V); what process_solo does on top pays off from the
// fifth slice on.  512 decodes on 31 keys x 8 KV heads (one slice each) 21.8 -> 20.3 us.
__device__ __forceinline__ void process_short(const RunParams& p, const XyDevUnit& u,
                                              unsigned char* smem, const LaneOffsets& lo, const DmaOffsets& dof) {
  constexpr int NT = 1;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const UnitCtx c = make_ctx(p, u);
  Rows<NT> r;
  bf16x8 qf[NT][8];
  const int rc = min(col, c.rows - 1), tl = rc / c.hc, hl = rc - tl * c.hc;
  r.valid[0] = col < c.rows;
  r.tok[0] = u.q_begin + tl;
  r.lim[0] = r.valid[0] ? c.ctx + r.tok[0] + 1 : 0;
  const uint16_t* qrow = p.q + (int64_t)(u.token_start + r.tok[0]) * p.q_ts + (int64_t)(u.head_begin + hl) * p.q_hs + 8 * half;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) qf[0][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qrow + 16 * ks));
  r.mw0[0] = r.mw1[0] = 0;
  if (c.tree && r.valid[0]) {
    const uint32_t* mrow = p.masks + u.mask_off + (int64_t)r.tok[0] * c.wpr;
    r.mw0[0] = mrow[0];
    if (c.wpr > 1) r.mw1[0] = mrow[1];
  }
  const int mask_from = c.tree ? c.ctx : c.ctx + u.q_begin + 1;
  UnitState st;
  zero_state<NT>(st.oacc, st.m_ref, st.l_part);
  const XY_CONST int32_t* table = as_const(p.block_table) + (int64_t)u.seq * p.max_blocks;
  const int last_page = (u.ctx_len + u.q_len - 1) >> p.page_shift;
  const int64_t head_off = (int64_t)c.kvh * p.kv_hs;
  const int jfirst = u.kv_begin * kB;
  const int nsteps = (min(u.kv_end * kB, c.key_end) - jfirst + 31) >> 5;
  unsigned char* ring = smem + wave * 32768;        // [K slot | V slot]
  const unsigned kaddr = lds_addr(ring), vaddr = kaddr + 8192;
  // as in process_solo: two runs of sixteen rows, each inside one page (rows past the sequence's last page are never visible and
  // redirected to that page, so that what lands in LDS for them is ordinary finite cache content)
  struct Slice {
    int64_t run[2];
  };
  auto locate = [&](const int j) {          // both page-table entries asked for before either is waited for
    int e0 = table[min(j >> p.page_shift, last_page)], e1 = table[min((j + 16) >> p.page_shift, last_page)];
    asm volatile("" : "+s"(e0), "+s"(e1));
    return Slice{{(int64_t)e0 * p.kv_bs + (int64_t)(j & p.page_mask) * p.kv_ts + head_off,
                  (int64_t)e1 * p.kv_bs + (int64_t)((j + 16) & p.page_mask) * p.kv_ts + head_off}};
  };
  auto load_slice = [&](const Slice& at, const bool want_k, const bool want_v) {      // eight instructions per tensor
#pragma unroll
    for (int g = 0; g < 2; ++g)
      load_rows_async<4>(p.k + at.run[g], p.v + at.run[g], p.kv_ts, 0, ring + 4096 * g, ring + 8192 + 4096 * g, dof, want_k, want_v);
  };
  Slice at = locate(jfirst);
  load_slice(at, true, false);          // issue order K, V
  load_slice(at, false, true);
#pragma unroll 1
  for (int t = 0; t < nsteps; ++t) {
    const int tn = t + 1;
    if (tn < nsteps) at = locate(jfirst + 32 * tn);      // while K is waited for
    wait_vmcnt<8>();                          // K(t) has landed; only V(t) may still be in flight
    f32x16 s[NT];
    VFrags vf;
    qk_step<NT>(kaddr, lo, qf, s);            // all K reads have completed when this returns
    if (tn < nsteps) {        // K slot is free again: refill it with the next slice
      load_slice(at, true, false);
      wait_vmcnt<8>();        // V(t) has landed; the K refill stays in flight
    } else {
      wait_vmcnt<0>();
      const int last_keys = min(u.kv_end * kB, c.key_end) - jfirst - 32 * t;      // keys of the last step: 1 .. 32
      if (last_keys < 32) zero_tail_rows(vaddr, last_keys, lane);
    }
    v_fetch<0>(vaddr, lo, vf);                // the first V fragments arrive while the softmax runs
    const int j = jfirst + 32 * t;
    if (j + 32 > mask_from) mask_step<NT>(p, c, r, j + 8 * half, s);
    softmax_step<NT>(p.c, s, st.m_ref, st.l_part, st.oacc, t == 0);
    pv_step<NT>(vaddr, lo, vf, s, st.oacc);   // all V reads have completed when this returns
    if (tn < nsteps) load_slice(at, false, true);
  }
  finish_unit(p, u, c, r, st, col, half);
}

// NARROW: how the units of at most 32 rows are processed (kSolo, kShort: kShortSlices in layout.cpp; 2 or 4: by a team of so many
// wavefronts each, kTeamOf4Slices in layout.cpp); a kernel for each, since the ways in one disturb each other's registers (short units
// 3 to 5 %, launches on two slices up to 2 %).
constexpr int kSolo = 0, kShort = 1;
template <int NARROW>
__device__ __forceinline__ void process_narrow(const RunParams& p, const XyDevUnit& u, unsigned char* smem, const LaneOffsets& lo,
                                               const DmaOffsets& dof) {
  if constexpr (NARROW == kShort) process_short(p, u, smem, lo, dof);
  else process_solo<1>(p, u, smem, lo, dof);
}

// consecutive workgroup ids land on different XCDs; each XCD gets a contiguous range of workers
__device__ __forceinline__ int worker_of(int workgroup, int num_workers) {
  return (num_workers & 7) == 0 ? (workgroup & 7) * (num_workers >> 3) + (workgroup >> 3) : workgroup;
}

// Teams: one unit for every team of the workers without wide units, none drawn; consecutive ones on different chiplets.
// rank: of this worker among them.
template <int TEAM>
__device__ __forceinline__ void team_unit(const RunParams& p, int teams_begin, int rank, unsigned char* smem, const LaneOffsets& lo,
                                          const DmaOffsets& dof) {
  const int i = teams_begin + rank + p.free_workers * (wave_id() / TEAM);
  const bool exists = i < p.num_units;
  const XyDevUnit u = load_unit(p.units + (exists ? i : teams_begin));
  process_solo<TEAM>(p, u, smem, lo, dof, exists);
}

// The narrow units of a worker's own list [begin, end): its wavefronts draw them from a cursor in LDS.
template <int NARROW>
__device__ __forceinline__ void own_units(const RunParams& p, int begin, int end, int& cursor, unsigned char* smem, const LaneOffsets& lo,
                                          const DmaOffsets& dof) {
  if (threadIdx.x == 0) cursor = begin + kThreads / 64;
  __syncthreads();            // the cursor is initialised (and the tiles of the wide units are free)
  int i = begin + wave_id();
#pragma unroll 1
  while (i < end) {
    const XyDevUnit u = load_unit(p.units + i);
    if (u.q_count * u.head_count <= 32) process_narrow<NARROW>(p, u, smem, lo, dof);
    int got = 0;
    if ((threadIdx.x & 63) == 0) got = atomicAdd(&cursor, 1);
    i = __builtin_amdgcn_readfirstlane(got);
  }
}

// The shared list of narrow units (dynamic assignment): every wavefront of every workgroup draws the
// next unit of the list, largest first, until it is empty.  The last workgroup to leave puts the
// counters back to zero for the next launch (a plan runs one launch at a time, as its workspace does).
// First draw: a thousand wavefronts asking one counter at the same moment cost 15 us, so a worker without units
// of its own has four entries reserved for it (numbered wavefront-major over such workers: a short list still
// reaches every one of them).  A worker that comes here from wide units has none - an entry reserved for it
// would wait for those to end while other CUs are idle (4 wide units and a dozen small ones: 25.8 -> 16.4 us, a chunk of 200 tokens beside 24 short decodes
// 46.7 -> 36.3 us, a chunk of 512 beside 64 decodes 161 -> 153 us) -
// and draws four at once, one atomic for the workgroup.  rank: of this worker among those without units of their own, or -1.
template <int NARROW>
__device__ __forceinline__ void shared_units(const RunParams& p, int worker, int shared_begin, int rank, int& first_draw,
                                             unsigned char* smem, const LaneOffsets& lo, const DmaOffsets& dof) {
  const int slots = p.free_workers * (kThreads / 64);
  const bool any_left = shared_begin + slots < p.num_units;                        // behind the reserved entries
  int next = wave_id() * p.free_workers + rank;
  if (rank < 0) {
    if (any_left && threadIdx.x == 0) first_draw = slots + atomicAdd(p.counters, kThreads / 64);
    __syncthreads();          // the tiles of the wide units are free too
    next = any_left ? __builtin_amdgcn_readfirstlane(first_draw) + wave_id() : p.num_units;
  }
#pragma unroll 1
  while (true) {
    const int i = shared_begin + next;
    if (i >= p.num_units) break;
    const XyDevUnit u = load_unit(p.units + i);
    process_narrow<NARROW>(p, u, smem, lo, dof);
    if (!any_left) break;
    int got = 0;
    if ((threadIdx.x & 63) == 0) got = slots + atomicAdd(p.counters, 1);
    next = __builtin_amdgcn_readfirstlane(got);
  }
  if (!any_left) return;      // nothing was drawn: the counters are as they were
  __syncthreads();            // all four wavefronts are done with the cursor
  // No fence: every cursor draw above has returned its value, so it was performed at the
  // memory side before this count is; a device-wide fence here would write back and drop
  // this chiplet's L2 under the workgroups that are still streaming K/V through it.
  // The count of workgroups that have left is kept in two levels (eight groups of workgroups, each
  // on a cache line of its own, then one count of finished groups): 256 atomics on one address
  // would take several microseconds, which a short decode step cannot hide.
  if (threadIdx.x == 0) {
    const int groups = p.num_workers < kDoneGroups ? p.num_workers : kDoneGroups;
    const int g = worker % kDoneGroups;
    const int members = (p.num_workers - g + kDoneGroups - 1) / kDoneGroups;
    int* done = p.counters + kCounterStride * (1 + g);
    int* top = p.counters + kCounterStride * (1 + kDoneGroups);
    if (atomicAdd(done, 1) == members - 1) {
      __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (atomicAdd(top, 1) == groups - 1) {
        __hip_atomic_store(top, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p.counters, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// Launches with units of more than 32 rows.  Every workgroup is one worker of the Task-Table (paper section 3.3).  It first
// works through the wide units of its list together, then its four wavefronts draw the remaining (bandwidth-bound)
// units of the same list one by one from a shared cursor, each wavefront finishing whole units
// on its own.
// NT: row tiles of a wavefront on its wide units (process_wide).
template <int NARROW, int NT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void xy_attn_units_kernel(RunParams p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kTileBytes];
  __shared__ int cursor, first_draw;
  __shared__ int overflow_flags[kThreads / 64];
  const int worker = worker_of(blockIdx.x, p.num_workers);
  const int begin = as_const(p.worker_offsets)[worker], end = as_const(p.worker_offsets)[worker + 1];
  const LaneOffsets lo = make_lane_offsets(threadIdx.x & 63);
  const DmaOffsets dof = make_dma_offsets(threadIdx.x & 63, p.kv_ts);
  bool force = false;         // the unit at hand is run a second time, with exact references (see process_wide)
#pragma unroll 1
  for (int i = begin; i < end;) {
    const XyDevUnit u = load_unit(p.units + i);
    if (u.q_count * u.head_count <= 32) {
      ++i;
      continue;
    }
    // Folding c into Q rounds q * c to bf16 once more; with the usual 1/sqrt(d) scale that is far inside the
    // tolerance, with a scale so large that scores reach tens of log2 units it is not, and c stays in fp32.
    bool again;
    if (p.kv_ts == kD) {
      if (p.c <= kPrescaleMaxC) again = process_wide<true, true, NT>(p, u, smem, overflow_flags, force, lo, dof);
      else again = process_wide<false, true, NT>(p, u, smem, overflow_flags, force, lo, dof);
    } else {
      if (p.c <= kPrescaleMaxC) again = process_wide<true, false, NT>(p, u, smem, overflow_flags, force, lo, dof);
      else again = process_wide<false, false, NT>(p, u, smem, overflow_flags, force, lo, dof);
    }
    force = again;              // wavefront- and workgroup-uniform
    if (!again) ++i;
  }
  // The narrow phase reads the kernel arguments afresh
  // instead of keeping the copies of the wide phase alive: what that phase had to spill to make room for
  // its own scalars would otherwise be reloaded lane by lane in every step of every narrow unit.
  const RunParams pn = load_args();
  if constexpr (NARROW > 1) {
    if (begin < end) return;
    team_unit<NARROW>(pn, as_const(pn.worker_offsets)[pn.num_workers], as_const(pn.worker_offsets)[pn.num_workers + 1 + worker], smem, lo, dof);
    return;
  }
  if (!pn.counters) {
    if (begin < end) own_units<NARROW>(pn, begin, end, cursor, smem, lo, dof);
  } else {                    // all narrow units are on the shared list
    shared_units<NARROW>(pn, worker, as_const(pn.worker_offsets)[pn.num_workers], as_const(pn.worker_offsets)[pn.num_workers + 1 + worker],
                         first_draw, smem, lo, dof);
  }
}

// Launches without: the workers' lists are either all there is, or empty (one shared list, or teams), and there is nothing to
// look up then.  Short ones are bound by the chain of loads in front of a unit's first keys: arguments, record, page-table
// entries, K, each asked for as a whole before anything waits (but in process_short, whose entries are waited for together
// with its Q).  With the lists, a barrier, the arguments read twice and the entries one after the other, as in the kernel above
// until this one was split off, us: one decode of 1000 tokens on teams (8 families in 64 pieces, this kernel alone) 7.07 -> 6.22,
// where a call from Python is bound by the host and level; 24 decodes beside a suffix of 200 tokens (the entries alone)
// 31.8 -> 31.0 a layer, 8 decodes x 32 KV heads on 2-6k tokens 87.8 -> 86.4, 128 trees on 512-4096 tokens 153.1 -> 152.4.
// Teams spill no scalars.  The other two hold a body for the shared list and one for the workers' lists, of which a launch runs one,
// and spill 43 (two of them read back in every slice of one body; else around a unit's loop) and 16.
template <int NARROW>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void xy_attn_narrow_kernel(RunParams) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kTileBytes];
  __shared__ int cursor, first_draw;
  const RunParams p = load_args();
  const LaneOffsets lo = make_lane_offsets(threadIdx.x & 63);
  const DmaOffsets dof = make_dma_offsets(threadIdx.x & 63, p.kv_ts);
  if constexpr (NARROW > 1) {
    team_unit<NARROW>(p, 0, blockIdx.x, smem, lo, dof);
  } else {
    const int worker = worker_of(blockIdx.x, p.num_workers);
    if (p.counters) shared_units<NARROW>(p, worker, 0, worker, first_draw, smem, lo, dof);
    else own_units<NARROW>(p, as_const(p.worker_offsets)[worker], as_const(p.worker_offsets)[worker + 1], cursor, smem, lo, dof);
  }
}

// Merge the partial states of a K/V-split family: O = sum_p 2^(m_p - m*) acc_p / sum_p 2^(m_p - m*) l_p.
// Bound by memory latency on short steps, by the bytes of the partial results on a cut prefill chunk.  One record
// of XyDevMergeRows per workgroup holds all a workgroup has to know (one scalar load, no chain of item, sequence
// and row), eight rows side by side read the partials in the order they are stored in (128 contiguous bytes per
// group of four d), and the loads of up to eight pieces are issued together before any of them is used: a row of eight pieces or fewer
// costs two round trips to memory, the record and the data.  Against one workgroup of 128 threads per row that
// walked item, sequence and pieces one after another: 5.6 -> 2.9 us for one decode on 1300 tokens (8 families of
// 4 rows), 9.5 -> 4.6 us for 24 short decodes, 20 -> 9.2 us for a cut chunk of 1024 tokens x 32 heads.
template <int N>      // pieces [s0, s0 + N), those from num_splits on counted as empty
__device__ __forceinline__ void merge_pieces(const float* acc_row, const float* m_row, const float* l_row, int64_t slab,
                                             int s0, int num_splits, float& m_run, float& den, f32x4& num) {
  constexpr int kCertain = N / 2 + (N > 2);      // more pieces than half a batch, or the next smaller one would do
  float m[N], l[N];
  f32x4 acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t at = (int64_t)min(s0 + i, num_splits - 1) * slab;
    m[i] = m_row[at];
    l[i] = l_row[at];
    acc[i] = *reinterpret_cast<const f32x4*>(acc_row + at);
  }
  float m_new = m_run;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (s0 + i >= num_splits) m[i] = -INFINITY;
    m_new = fmaxf(m_new, m[i]);
  }
  const float keep = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
  den *= keep;
  num *= keep;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i >= kCertain) {    // may be empty: all of it is zero then, a factor of zero would not remove an infinity
      asm volatile("" : "+v"(l[i]), "+v"(acc[i]));      // (the loads stay where they are, not in a branch of their own)
      if (s0 + i >= num_splits) {
        l[i] = 0.f;
        acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    const float f = m[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[i] - m_new);
    num += f * acc[i];
    den += f * l[i];
  }
  m_run = m_new;
}

__global__ __launch_bounds__(kMergeThreads) void xy_attn_merge_kernel(const XyDevMergeRows* items, const float* ws,
                                                                      uint16_t* out, int64_t o_ts, int64_t o_hs) {
  const XyDevMergeRows it = load_const(items + blockIdx.x);
  const int r = it.row_begin + (threadIdx.x & (kMergeRows - 1)), d4 = threadIdx.x / kMergeRows;      // row, group of four d
  if (r >= it.rows) return;
  const int64_t slab = ((int64_t)it.rows * (kD + 2) + 3) & ~(int64_t)3;
  const float* base = ws + it.ws_offset;
  const float* acc_row = base + ((int64_t)d4 * it.rows + r) * 4;
  const float* m_row = base + (int64_t)it.rows * kD + r;
  const float* l_row = m_row + it.rows;
  float m_run = -INFINITY, den = 0.f;
  f32x4 num = {0.f, 0.f, 0.f, 0.f};
  int s = 0;
  for (; it.num_splits - s > 4; s += 8) merge_pieces<8>(acc_row, m_row, l_row, slab, s, it.num_splits, m_run, den, num);
  if (it.num_splits - s > 2) merge_pieces<4>(acc_row, m_row, l_row, slab, s, it.num_splits, m_run, den, num);
  else if (it.num_splits - s > 0) merge_pieces<2>(acc_row, m_row, l_row, slab, s, it.num_splits, m_run, den, num);
  const float inv = den > 0.f ? 1.f / den : 0.f;
  const int tl = r / it.head_count, hl = r - tl * it.head_count;
  uint2 w;
  w.x = pack_bf16(num[0] * inv, num[1] * inv);
  w.y = pack_bf16(num[2] * inv, num[3] * inv);
  *reinterpret_cast<uint2*>(out + (int64_t)(it.token_begin + tl) * o_ts + (int64_t)(it.head_begin + hl) * o_hs + 4 * d4) = w;
}

}  // namespace

// ---- the plan's tables on the GPU ---------------------------------------------------------------------
// One device arena and one pinned staging buffer per plan object, allocated when first needed, grown only when a
// rebuilt plan does not fit, freed with the plan.  A copy packs the tables into the staging buffer and enqueues
// ONE small copy kernel on the caller's stream; an event behind it says when the staging buffer
// may be written again.
void xy_plan_free_device(xy_attn_plan* plan) {
  if (!plan || plan->device < 0) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(plan->device);
  if (plan->copied) {
    (void)hipEventSynchronize(static_cast<hipEvent_t>(plan->copied));
    (void)hipEventDestroy(static_cast<hipEvent_t>(plan->copied));
  }
  if (plan->d_arena) (void)hipFree(plan->d_arena);
  if (plan->h_stage) (void)hipHostFree(plan->h_stage);
  plan->d_arena = plan->h_stage = plan->h_stage_dev = plan->copied = nullptr;
  plan->d_units = plan->d_offsets = plan->d_seqs = plan->d_merges = plan->d_counters = nullptr;
  plan->arena_capacity = 0;
  plan->device = -1;
  plan->device_stale = true;
  (void)hipSetDevice(cur);
}

// 16 bytes per thread from the pinned staging buffer (read over the host link) to the arena
__global__ __launch_bounds__(256) void xy_plan_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                           unsigned chunks) {
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < chunks) dst[i] = src[i];
}

static int plan_copy_to_device(xy_attn_plan* plan, hipStream_t stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return XY_ERR_HIP;
  if (plan->device >= 0 && plan->device != dev) return XY_ERR_ARG;      // the plan lives on another device
  auto round_up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const bool shared_list = plan->worker_offsets.back() < (int64_t)plan->units.size();
  const XyLayout layout = xy_plan_layout(plan);
  const size_t off_units = 0;
  const size_t off_offsets = off_units + round_up((size_t)layout.records * sizeof(XyDevUnit));
  const size_t off_seqs = off_offsets + round_up(2 * plan->worker_offsets.size() * sizeof(int32_t));
  const size_t off_merges = off_seqs + round_up((size_t)plan->num_seqs * sizeof(XyDevSeq));
  int64_t merge_groups = 0;       // workgroups of the merge pass
  for (const xy_merge_item& m : plan->merges) merge_groups += (m.q_count * m.head_count + kMergeRows - 1) / kMergeRows;
  const size_t off_counters = off_merges + round_up((size_t)merge_groups * sizeof(XyDevMergeRows));
  const size_t need = off_counters + round_up(sizeof(int32_t) * kCounterStride * (kDoneGroups + 2));
  if (need > plan->arena_capacity) {
    xy_plan_free_device(plan);
    const size_t cap = std::max<size_t>(round_up(2 * need), (size_t)1 << 20);      // allocations are slow (milliseconds): grow rarely
    hipEvent_t ev = nullptr;
    if (hipMalloc(&plan->d_arena, cap) != hipSuccess || hipHostMalloc(&plan->h_stage, cap, hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
      plan->device = dev;           // so that what was allocated is freed
      plan->copied = ev;
      xy_plan_free_device(plan);
      return XY_ERR_HIP;
    }
    plan->copied = ev;
    plan->arena_capacity = cap;
    plan->device = dev;
    if (hipHostGetDevicePointer(&plan->h_stage_dev, plan->h_stage, 0) != hipSuccess) {
      xy_plan_free_device(plan);
      return XY_ERR_HIP;
    }
  } else if (hipEventSynchronize(static_cast<hipEvent_t>(plan->copied)) != hipSuccess) {
    return XY_ERR_HIP;              // (the copy before this one has long finished in any sensible use)
  }
  unsigned char* h = static_cast<unsigned char*>(plan->h_stage);
  plan->layout = layout;
  plan->free_workers = xy_plan_hand_out(plan, layout, reinterpret_cast<XyDevUnit*>(h + off_units), reinterpret_cast<int32_t*>(h + off_offsets));
  XyDevSeq* ds = reinterpret_cast<XyDevSeq*>(h + off_seqs);
  for (int32_t i = 0; i < plan->num_seqs; ++i) {
    const xy_seq_desc& s = plan->descs[i];
    ds[i] = XyDevSeq{s.context_len, plan->token_start[i]};
  }
  XyDevMergeRows* dm = reinterpret_cast<XyDevMergeRows*>(h + off_merges);
  for (const xy_merge_item& m : plan->merges) {
    const int32_t rows = m.q_count * m.head_count;
    for (int32_t r = 0; r < rows; r += kMergeRows)
      *dm++ = XyDevMergeRows{m.ws_offset, rows, r, m.num_splits, plan->token_start[m.seq] + m.q_begin, m.head_begin, m.head_count};
  }
  plan->merge_groups = merge_groups;
  memset(h + off_counters, 0, need - off_counters);       // cursor and finished-workgroup counts start at zero
  // The tables go over by a small kernel that reads the pinned buffer through its device mapping, not by the copy
  // engine: a copy-engine transfer in front of a kernel on the same stream costs about 0.15 ms of hand-over between
  // the two queues (measured: a serving step of 0.06 ms of kernels took 0.22 ms), a kernel-to-kernel order nothing.
  const unsigned chunks = (unsigned)(need / 16);
  hipLaunchKernelGGL(xy_plan_copy_kernel, dim3((chunks + 255) / 256), dim3(256), 0, stream,
                     static_cast<const uint4*>(plan->h_stage_dev), static_cast<uint4*>(plan->d_arena), chunks);
  if (hipGetLastError() != hipSuccess) return XY_ERR_HIP;
  if (hipEventRecord(static_cast<hipEvent_t>(plan->copied), stream) != hipSuccess) return XY_ERR_HIP;
  unsigned char* d = static_cast<unsigned char*>(plan->d_arena);
  plan->d_units = d + off_units;
  plan->d_offsets = d + off_offsets;
  plan->d_seqs = d + off_seqs;
  plan->d_merges = d + off_merges;
  plan->d_counters = shared_list ? d + off_counters : nullptr;
  plan->device_stale = false;
  return XY_OK;
}

extern "C" int xy_attn_plan_upload_async(xy_attn_plan* plan, void* hip_stream) {
  if (!plan) return XY_ERR_ARG;
  if (plan->device >= 0 && !plan->device_stale) return XY_OK;
  return plan_copy_to_device(plan, static_cast<hipStream_t>(hip_stream));
}

extern "C" int xy_attn_plan_upload(xy_attn_plan* plan) {
  if (!plan) return XY_ERR_ARG;
  if (plan->device >= 0 && !plan->device_stale) return XY_OK;
  if (int rc = plan_copy_to_device(plan, nullptr)) return rc;
  return hipStreamSynchronize(nullptr) == hipSuccess ? XY_OK : XY_ERR_HIP;
}

// Argument checks of a run (everything that can fail before device work is enqueued).
static int check_run_args(xy_attn_plan* plan, const void* q, int64_t q_ts, int64_t q_hs, const void* k_cache,
                          const void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                          const int32_t* block_table, const uint32_t* tree_masks, void* out, int64_t o_ts,
                          int64_t o_hs, void* workspace, size_t workspace_bytes, float softmax_scale,
                          hipStream_t stream) {
  if (!q || !k_cache || !v_cache || !block_table || !out) return XY_ERR_ARG;
  if (plan->has_tree && !tree_masks) return XY_ERR_ARG;
  if (!(softmax_scale > 0.f) || !std::isfinite(softmax_scale)) return XY_ERR_ARG;
  // 16-byte vector accesses: every stride a multiple of 8 elements, every base 16-byte aligned
  const int64_t strides[] = {q_ts, q_hs, kv_bs, kv_hs, kv_ts, o_ts, o_hs};
  for (int64_t s : strides)
    if (s < 0 || (s & 7)) return XY_ERR_ARG;
  if (q_hs < kD || kv_ts < kD || o_hs < kD) return XY_ERR_ARG;
  const uintptr_t ptrs[] = {(uintptr_t)q, (uintptr_t)k_cache, (uintptr_t)v_cache, (uintptr_t)out};
  for (uintptr_t a : ptrs)
    if (a & 15) return XY_ERR_ARG;
  const size_t need = (size_t)plan->workspace_floats * sizeof(float);
  if (need && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15))) return XY_ERR_WORKSPACE;
  if (int rc = xy_attn_plan_upload_async(plan, stream)) return rc;      // first use, or the plan was rebuilt since
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev != plan->device) return XY_ERR_ARG;
  return XY_OK;
}

static int run_impl(int phases, xy_attn_plan* plan, const void* q, int64_t q_ts, int64_t q_hs, const void* k_cache,
                    const void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                    const int32_t* block_table, const uint32_t* tree_masks, void* out, int64_t o_ts,
                    int64_t o_hs, void* workspace, size_t workspace_bytes, float softmax_scale,
                    void* hip_stream) {
  if (!plan || !(phases & (XY_PHASE_UNITS | XY_PHASE_MERGE)) || (phases & ~(XY_PHASE_UNITS | XY_PHASE_MERGE)))
    return XY_ERR_ARG;
  if (plan->units.empty()) return XY_OK;
  if (int rc = check_run_args(plan, q, q_ts, q_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts, block_table, tree_masks,
                              out, o_ts, o_hs, workspace, workspace_bytes, softmax_scale,
                              static_cast<hipStream_t>(hip_stream)))
    return rc;

  RunParams p;
  p.units = static_cast<const XyDevUnit*>(plan->d_units);
  p.worker_offsets = static_cast<const int32_t*>(plan->d_offsets);
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k_cache);
  p.v = static_cast<const uint16_t*>(v_cache);
  p.block_table = block_table;
  p.masks = tree_masks;
  p.out = static_cast<uint16_t*>(out);
  p.ws = static_cast<float*>(workspace);
  p.q_ts = q_ts; p.q_hs = q_hs; p.kv_bs = kv_bs; p.kv_hs = kv_hs; p.kv_ts = kv_ts; p.o_ts = o_ts; p.o_hs = o_hs;
  p.max_blocks = plan->cfg.max_blocks_per_seq;
  p.page_mask = plan->cfg.block_size - 1;
  p.page_shift = plan->cfg.block_size == 16 ? 4 : plan->cfg.block_size == 32 ? 5 : plan->cfg.block_size == 64 ? 6 : 7;
  p.num_workers = plan->cfg.num_workers;
  p.free_workers = plan->free_workers;
  p.num_units = plan->layout.records;
  p.narrow_depth = plan->layout.depth;
  p.counters = static_cast<int32_t*>(plan->d_counters);
  p.c = softmax_scale * 1.4426950408889634f;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (phases & XY_PHASE_UNITS) {
    const XyLayout& l = plan->layout;
    // without wide units either the workers' lists hold everything or none of them holds anything: narrow units have a list of
    // their own as a whole
    const bool narrow_only = plan->narrow_units == (int64_t)plan->units.size();
    const auto kernel = narrow_only ? (l.team == 4 ? xy_attn_narrow_kernel<4> : l.team == 2 ? xy_attn_narrow_kernel<2>
                                       : l.short_units ? xy_attn_narrow_kernel<kShort> : xy_attn_narrow_kernel<kSolo>)
                        : l.team == 4 ? xy_attn_units_kernel<4, 1>
                        : l.team == 2 ? xy_attn_units_kernel<2, 1>
                        : l.row_tiles == 2 ? (l.short_units ? xy_attn_units_kernel<kShort, 2> : xy_attn_units_kernel<kSolo, 2>)
                                           : (l.short_units ? xy_attn_units_kernel<kShort, 1> : xy_attn_units_kernel<kSolo, 1>);
    // teams without wide units need no workgroup more than there are units
    const int32_t workgroups = l.team && narrow_only ? std::min(p.num_workers, p.num_units) : p.num_workers;
    hipLaunchKernelGGL(kernel, dim3(workgroups), dim3(kThreads), 0, stream, p);
    if (hipGetLastError() != hipSuccess) return XY_ERR_HIP;
  }
  if ((phases & XY_PHASE_MERGE) && !plan->merges.empty()) {
    for (int64_t first = 0; first < plan->merge_groups; first += kMergeGrid) {
      const int64_t groups = std::min(kMergeGrid, plan->merge_groups - first);
      hipLaunchKernelGGL(xy_attn_merge_kernel, dim3((unsigned)groups), dim3(kMergeThreads), 0, stream,
                         static_cast<const XyDevMergeRows*>(plan->d_merges) + first, static_cast<const float*>(workspace),
                         p.out, o_ts, o_hs);
      if (hipGetLastError() != hipSuccess) return XY_ERR_HIP;
    }
  }
  return XY_OK;
}

// ---- K/V append (section 4.1.1: the cache holds historical and newly generated tokens) --------
// One thread moves one 16-byte chunk: thread index = ((token * Hkv + kv head) * 2 + (K | V)) * 16 + chunk.
// The sixteen threads of a row read 256 contiguous bytes and write 256 contiguous bytes.  What a small step pays for is
// the chain of dependent loads in front of the copy, and the code that has to be fetched for it, so a wavefront finds
// the sequence of its token among the packed start positions with one load for up to 64 sequences (two up to 4096), one
// lane each, instead of one per halving; the lane that holds it is uniform and read as a scalar, and so is its neighbour for
// a second token of the wavefront.  One or two sequences are walked with scalar loads.  us, bisection / this:
//   one token each of 1 / 2 / 24 / 100 sequences, 8 KV heads   1.37 / 1.79 / 2.82 / 3.08 -> 1.41 / 1.75 / 2.59 / 2.78
//   of 2 / 7 / 24 / 100 sequences, 1 KV head                   1.44 / 1.67 / 2.20 / 3.02 -> 1.43 / 1.63 / 1.97 / 2.71
//   a suffix of 200 tokens beside 24 decodes, 8 KV heads       2.97 -> 2.70
//   8192 x 1 / 4000 x 2 / 1000 x 8 / 50 x 128 tokens           11.7 / 12.6 / 14.0 / 14.8 -> 12.0 / 12.3 / 12.4 / 10.9
// The neighbour by a load costs 0.2 us with one KV head.  The row asked for in front of the
// search changed small steps by nothing and made large ones slower (13.2 / 13.6 / 13.7 / 12.0); four probes a lane and 32-bit
// divisions changed nothing.
__global__ __launch_bounds__(256) void xy_attn_append_kernel(const XyDevSeq* __restrict__ seqs, int num_seqs,
                                                             int64_t total_tokens, int num_kv_heads,
                                                             const uint16_t* __restrict__ k_new,
                                                             const uint16_t* __restrict__ v_new, int64_t n_ts,
                                                             int64_t n_hs, uint16_t* __restrict__ k_cache,
                                                             uint16_t* __restrict__ v_cache, int64_t kv_bs,
                                                             int64_t kv_hs, int64_t kv_ts,
                                                             const int32_t* __restrict__ block_table,
                                                             int max_blocks, int page_shift, int64_t first) {
  const int64_t idx = first + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int chunk = (int)(idx & 15), is_v = (int)((idx >> 4) & 1), lane = threadIdx.x & 63;
  const int64_t row = idx >> 5;                     // token * Hkv + kv head
  const int64_t t = row / num_kv_heads;
  const int g = (int)(row - t * num_kv_heads);
  // the wavefront's first token (with an odd number of KV heads it may have two: a token is 32 Hkv threads)
  const int64_t t0 = (int64_t)__builtin_amdgcn_readfirstlane((int)(t >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)t);
  if (t0 >= total_tokens) return;
  int lo = 0;                                       // the last sequence whose token_start <= t0
  XyDevSeq sq, next = {0, INT32_MAX};               // that one, and the one behind it where the wavefront's second token may be
  if (num_seqs <= 2) {
    sq = seqs[0];
    while (lo + 1 < num_seqs) {
      next = seqs[lo + 1];
      if (next.token_start > t0) break;
      sq = next;
      ++lo;
      next.token_start = INT32_MAX;
    }
  } else {
    int left = num_seqs, step;                      // it is one of [lo, lo + left)
    do {
      step = (left + 63) >> 6;
      const XyDevSeq probe = seqs[lo + min(lane * step, left - 1)];
      const int hit = __popcll(__builtin_amdgcn_ballot_w64(lane * step < left && probe.token_start <= t0)) - 1;
      lo += hit * step;
      if (step == 1 && (num_kv_heads & 1)) {
        if (hit + 1 < left) next = XyDevSeq{__builtin_amdgcn_readlane(probe.ctx_len, hit + 1), __builtin_amdgcn_readlane(probe.token_start, hit + 1)};
        else if (lo + 1 < num_seqs) next = seqs[lo + 1];
      }
      left = min(step, left - hit * step);
      sq = XyDevSeq{__builtin_amdgcn_readlane(probe.ctx_len, hit), __builtin_amdgcn_readlane(probe.token_start, hit)};
    } while (step > 1);
  }
  if (t >= total_tokens) return;
  if (next.token_start <= t) {                      // (no sequence is empty: the second token is in one of the two)
    sq = next;
    ++lo;
  }
  const int j = sq.ctx_len + (int)(t - sq.token_start);          // key position of this token
  const int64_t block = block_table[(int64_t)lo * max_blocks + (j >> page_shift)];
  const uint16_t* src = (is_v ? v_new : k_new) + t * n_ts + (int64_t)g * n_hs + chunk * 8;
  uint16_t* dst = (is_v ? v_cache : k_cache) + block * kv_bs + (int64_t)g * kv_hs + (int64_t)(j & ((1 << page_shift) - 1)) * kv_ts + chunk * 8;
  *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
}

extern "C" int xy_attn_append_kv(xy_attn_plan* plan, const void* k_new, const void* v_new, int64_t n_ts,
                                 int64_t n_hs, void* k_cache, void* v_cache, int64_t kv_bs, int64_t kv_hs,
                                 int64_t kv_ts, const int32_t* block_table, void* hip_stream) {
  if (!plan) return XY_ERR_ARG;
  if (plan->total_tokens == 0) return XY_OK;
  if (!k_new || !v_new || !k_cache || !v_cache || !block_table) return XY_ERR_ARG;
  const int64_t strides[] = {n_ts, n_hs, kv_bs, kv_hs, kv_ts};
  for (int64_t s : strides)
    if (s < 0 || (s & 7)) return XY_ERR_ARG;
  if (n_hs < kD || kv_ts < kD) return XY_ERR_ARG;
  const uintptr_t ptrs[] = {(uintptr_t)k_new, (uintptr_t)v_new, (uintptr_t)k_cache, (uintptr_t)v_cache};
  for (uintptr_t a : ptrs)
    if (a & 15) return XY_ERR_ARG;
  if (int rc = xy_attn_plan_upload_async(plan, hip_stream)) return rc;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev != plan->device) return XY_ERR_ARG;
  const int64_t threads = plan->total_tokens * plan->cfg.num_kv_heads * 32;
  for (int64_t first = 0; first < threads; first += kAppendGrid * 256) {
    const int64_t blocks = std::min(kAppendGrid, (threads - first + 255) / 256);
    hipLaunchKernelGGL(xy_attn_append_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const XyDevSeq*>(plan->d_seqs), plan->num_seqs, plan->total_tokens,
                       plan->cfg.num_kv_heads, static_cast<const uint16_t*>(k_new),
                       static_cast<const uint16_t*>(v_new), n_ts, n_hs, static_cast<uint16_t*>(k_cache),
                       static_cast<uint16_t*>(v_cache), kv_bs, kv_hs, kv_ts, block_table,
                       plan->cfg.max_blocks_per_seq,
                       plan->cfg.block_size == 16 ? 4 : plan->cfg.block_size == 32 ? 5 : plan->cfg.block_size == 64 ? 6 : 7, first);
    if (hipGetLastError() != hipSuccess) return XY_ERR_HIP;
  }
  return XY_OK;
}

// ---- copy-on-write of partly reused blocks (section 4.1.1) ------------------------------------
struct CopyBatch {
  xy_kv_copy c[32];
};

// Workgroup (copy, KV head, K | V) moves rows x 256 bytes in 16-byte chunks.
__global__ __launch_bounds__(256) void xy_attn_copy_rows_kernel(CopyBatch batch, int num_kv_heads,
                                                                uint16_t* __restrict__ k_cache,
                                                                uint16_t* __restrict__ v_cache, int64_t kv_bs,
                                                                int64_t kv_hs, int64_t kv_ts) {
  const int is_v = blockIdx.x & 1;
  const int g = (blockIdx.x >> 1) % num_kv_heads;
  const xy_kv_copy cp = batch.c[(blockIdx.x >> 1) / num_kv_heads];
  uint16_t* cache = is_v ? v_cache : k_cache;
  const uint16_t* src = cache + (int64_t)cp.src_block * kv_bs + (int64_t)g * kv_hs;
  uint16_t* dst = cache + (int64_t)cp.dst_block * kv_bs + (int64_t)g * kv_hs;
  for (int i = threadIdx.x; i < cp.rows * 16; i += blockDim.x) {
    const int64_t off = (int64_t)(i >> 4) * kv_ts + (i & 15) * 8;
    *reinterpret_cast<uint4*>(dst + off) = *reinterpret_cast<const uint4*>(src + off);
  }
}

extern "C" int xy_attn_copy_block_rows(const xy_kv_copy* copies, int32_t n, int32_t num_kv_heads, void* k_cache,
                                       void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                                       void* hip_stream) {
  if (n < 0 || num_kv_heads < 1) return XY_ERR_ARG;
  if (n == 0) return XY_OK;
  if (!copies || !k_cache || !v_cache) return XY_ERR_ARG;
  const int64_t strides[] = {kv_bs, kv_hs, kv_ts};
  for (int64_t st : strides)
    if (st < 0 || (st & 7)) return XY_ERR_ARG;
  if (kv_ts < kD || ((uintptr_t)k_cache & 15) || ((uintptr_t)v_cache & 15)) return XY_ERR_ARG;
  for (int32_t i = 0; i < n; ++i)
    if (copies[i].rows < 0 || copies[i].src_block < 0 || copies[i].dst_block < 0) return XY_ERR_ARG;
  for (int32_t first = 0; first < n; first += 32) {
    CopyBatch batch;
    const int32_t cnt = std::min(32, n - first);
    for (int32_t i = 0; i < cnt; ++i) batch.c[i] = copies[first + i];
    hipLaunchKernelGGL(xy_attn_copy_rows_kernel, dim3((unsigned)(cnt * num_kv_heads * 2)), dim3(256), 0,
                       static_cast<hipStream_t>(hip_stream), batch, num_kv_heads, static_cast<uint16_t*>(k_cache),
                       static_cast<uint16_t*>(v_cache), kv_bs, kv_hs, kv_ts);
    if (hipGetLastError() != hipSuccess) return XY_ERR_HIP;
  }
  return XY_OK;
}

extern "C" int xy_attn_run(xy_attn_plan* plan, const void* q, int64_t q_ts, int64_t q_hs, const void* k_cache,
                           const void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                           const int32_t* block_table, const uint32_t* tree_masks, void* out, int64_t o_ts,
                           int64_t o_hs, void* workspace, size_t workspace_bytes, float softmax_scale,
                           void* hip_stream) {
  return run_impl(XY_PHASE_UNITS | XY_PHASE_MERGE, plan, q, q_ts, q_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts,
                  block_table, tree_masks, out, o_ts, o_hs, workspace, workspace_bytes, softmax_scale, hip_stream);
}

extern "C" int xy_attn_run_phase(int phases, xy_attn_plan* plan, const void* q, int64_t q_ts, int64_t q_hs,
                                 const void* k_cache, const void* v_cache, int64_t kv_bs, int64_t kv_hs,
                                 int64_t kv_ts, const int32_t* block_table, const uint32_t* tree_masks,
                                 void* out, int64_t o_ts, int64_t o_hs, void* workspace, size_t workspace_bytes,
                                 float softmax_scale, void* hip_stream) {
  return run_impl(phases, plan, q, q_ts, q_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts, block_table, tree_masks,
                  out, o_ts, o_hs, workspace, workspace_bytes, softmax_scale, hip_stream);
}

// ---- a run that allocates nothing -----------------------------------------------------------------------
// For callers that cannot allocate (a region under graph capture, a serving loop, a harness that forbids it):
// the partial results of K/V-split units go to a fixed array in device memory instead of a caller's workspace.
// Every GPU the library runs on holds its own copy of the array until the process ends.  In host code the
// array's name stands for the symbol, not for an address a kernel could use: the address on a device is asked
// for once, with that device current, and only that pointer is handed to the kernels.
constexpr size_t kScratchBytes = (size_t)XY_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices] = {};      // per device, resolved on the first call there

int scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return XY_ERR_HIP;
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return XY_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return XY_OK;
}
}  // namespace

extern "C" int xy_attn_run_static(xy_attn_plan* plan, const void* q, int64_t q_ts, int64_t q_hs, const void* k_cache,
                                  const void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                                  const int32_t* block_table, const uint32_t* tree_masks, void* out, int64_t o_ts,
                                  int64_t o_hs, float softmax_scale, void* hip_stream) {
  if (!plan) return XY_ERR_ARG;
  if ((size_t)plan->workspace_floats * sizeof(float) > kScratchBytes) return XY_ERR_WORKSPACE;
  if (plan->units.empty()) return XY_OK;
  if (plan->device < 0 || plan->device_stale) return XY_ERR_ARG;      // copying the plan to the GPU may allocate: xy_attn_plan_upload comes first
  void* ws = nullptr;
  if (int rc = scratch_of_current_device(&ws)) return rc;
  // The partial results need no initialisation: every split unit writes its whole partial before the merge reads it.
  return run_impl(XY_PHASE_UNITS | XY_PHASE_MERGE, plan, q, q_ts, q_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts,
                  block_table, tree_masks, out, o_ts, o_hs, ws, kScratchBytes, softmax_scale, hip_stream);
}

extern "C" int xy_attn_run_fused_qkv(xy_attn_plan* plan, const void* qkv, int64_t qkv_ts, int64_t qkv_hs,
                                     void* k_cache, void* v_cache, int64_t kv_bs, int64_t kv_hs, int64_t kv_ts,
                                     const int32_t* block_table, const uint32_t* tree_masks, void* out,
                                     int64_t o_ts, int64_t o_hs, void* workspace, size_t workspace_bytes,
                                     float softmax_scale, void* hip_stream) {
  if (!plan) return XY_ERR_ARG;
  if (plan->units.empty()) return XY_OK;
  if (!qkv || qkv_hs < kD || (qkv_hs & 7)) return XY_ERR_ARG;
  const uint16_t* base = static_cast<const uint16_t*>(qkv);
  const uint16_t* k_new = base + (int64_t)plan->cfg.num_q_heads * qkv_hs;
  const uint16_t* v_new = k_new + (int64_t)plan->cfg.num_kv_heads * qkv_hs;
  // validate the attention arguments first: a call that fails enqueues no device work
  if (int rc = check_run_args(plan, qkv, qkv_ts, qkv_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts, block_table,
                              tree_masks, out, o_ts, o_hs, workspace, workspace_bytes, softmax_scale,
                              static_cast<hipStream_t>(hip_stream)))
    return rc;
  if (int rc = xy_attn_append_kv(plan, k_new, v_new, qkv_ts, qkv_hs, k_cache, v_cache, kv_bs, kv_hs, kv_ts,
                                 block_table, hip_stream))
    return rc;
  return run_impl(XY_PHASE_UNITS | XY_PHASE_MERGE, plan, qkv, qkv_ts, qkv_hs, k_cache, v_cache, kv_bs, kv_hs,
                  kv_ts, block_table, tree_masks, out, o_ts, o_hs, workspace, workspace_bytes, softmax_scale,
                  hip_stream);
}
