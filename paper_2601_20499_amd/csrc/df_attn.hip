// df_attn_fwd / df_head_score: varlen-per-head flash-style attention for gfx950.
//
// Work decomposition.  A unit is one (head, 256-query tile): 8 wavefronts of 32
// queries each stream the head's visible keys - sink region, window region,
// current chunk, in this order (the concatenation order of Eq. 2) - in tiles of
// 64 keys.  A dummy head has an empty history, so its units iterate the current
// chunk only: no masked tile is ever issued.  Heads differ in length by the ratio
// of their contexts (3x between full and dummy heads, 20x with packed long
// contexts), so heads are not dealt out whole.  The key tiles of all heads,
// longest head first, are the "columns"; query tiles are taken in groups of
// team_size, and the line of (group, column) positions is cut into equal spans,
// one per TEAM of workgroups.  A team has one workgroup per query tile of a
// group: its members walk the same columns at the same time, each for its own
// 256 queries, so they share every K/V tile in L2 while it is hot, and every
// team does the same amount of work.  A unit that lies inside one span is
// finished in place.  A unit cut by span boundaries is put together by the
// workgroup that holds its last piece (the pieces lie with the same member of
// consecutive teams): every workgroup walks its span from the END, so a piece
// that does not end its unit is done early - its sums (m, l, region sums,
// unnormalised O in fp32) go to the workspace and a flag goes up - and the
// piece that ends a unit is the last thing a workgroup does: it waits for the
// flags of the earlier pieces, folds their sums into its own from the nearest
// piece back to the unit's first and writes the result.  This
// needs every workgroup of the launch on the device at once; when the device
// cannot hold them all, the pieces are left in the workspace and a second kernel
// puts them together in the same order with the same arithmetic.  Teams are laid
// out XCD-major (workgroup id mod 8 selects the XCD), so a team sits on one or
// two XCDs.
//
// Launches of few tiles are cut in another way where that costs less (cut_units): into units of 128
// or 256 queries, each head's units into a number of pieces of its own, one workgroup to a
// piece (of about equal length: see UnitCost).  With 128 the two groups of waves (see the schedule)
// have the same queries and take half of every tile's keys each, and a workgroup puts the two together through LDS (exchange_halves).  What such
// launches pay for is not tiles: a second piece in a span cost a workgroup 7 us besides its tiles, and those that
// waited for its sums with it; a piece of 256 queries hands on 136 KB, one of 128 queries 72, and a unit needs
// half as many pieces for the same number of workgroups; and the first load goes out 0.2 us earlier.  One box, spans -> units: 64
// queries 14.4 -> 10.0 us, 1170 queries 38.1 -> 35.3 (with what came after 9.4 and 27.8), 393 queries and 5 heads 29.0 -> 20.0, 266 queries and long histories
// 50.0 -> 31.9, 478 sampled queries 21.1 -> 18.1; 80 random launches 14 % less on average, the worst 1.2 % more.
//
// MFMA mapping.  Scores are computed transposed, S^T = K Q^T, with
// v_mfma_f32_16x16x32_bf16: 16 keys of the K tile are the A operand (ds_read_b128 from a
// row-major LDS tile), 16 queries of the wave's Q the B operand (registers, loaded
// once per unit); an A operand feeds the wave's two blocks of 16 queries.  In the
// 16x16 accumulator layout a lane owns TWO queries (lane%16 of each block) and 4 of the 16
// keys of a block, so the softmax row reductions are in-lane except for the exchange between
// the four lanes of a query at the end, and the probabilities are already in the register
// layout the second product needs as its B operand: O^T += V^T P^T.  V^T is the A operand
// and is read from a row-major V tile in LDS with the transposing ds_read_b64_tr_b16.
//
// Schedule.  The 8 waves form two groups of 4 (one wave of each group per
// SIMD).  Every tile iteration of a wave has an MFMA phase (S = K Q^T of tile t
// and O += V^T P^T of tile t-1) and a VALU/memory phase (online softmax of tile
// t, issue of the global loads of a later tile).  The workgroup meets at one
// barrier per iteration, which group 0 takes after its VALU phase and group 1
// after its MFMA phase: between two barriers group 0 runs MFMA(t), VALU(t) and
// group 1 runs VALU(t-1), MFMA(t), so on every SIMD one wave is in its MFMA
// phase while the other is in its VALU phase: the matrix core and the vector
// ALU overlap without relying on instruction scheduling.  The loop over the tiles of a
// piece is one generated asm statement (gen_attn_phase.py has the schedule and its reasons).
//
// Staging.  K and V tiles go from global memory straight into LDS with
// buffer_load_dwordx4 ... lds (no registers, no LDS store instructions); rows
// past the end of a head's buffer read as zero through the buffer range check.
// One such instruction fills 1 KB of LDS contiguously, so a tile is stored as
// groups of rows {g, g+NG, g+2NG, ...} (NG = 16 groups for d = 128), each group
// 1 KB plus a small pad, and every operand address is still "lane base + compile-time
// offset".  Tiles rotate through four LDS buffers each; loads are issued two to three
// iterations before their first use.
//
// Online softmax keeps a reference exponent per row (in units of log2) and per-lane partial row
// sums l in fp32.  The reference is the maximum of the row's first tile and is NOT raised
// tile by tile: exp2 of a logit above it simply exceeds one, which fp32 holds
// with room to spare.  Only when a row's sum passes 2^100 (or is no longer
// finite) is it raised to the row's current maximum or the logarithm of the
// sum and O, l rescaled, so the per-tile work has no row maximum, no
// comparison against the old one and no rescaling; P is rounded to bf16 (RNE)
// before the second product; l sums the unrounded fp32 values.  The output is
// divided by l and rounded to bf16 once at the end.
//
// The frame attention score of Eq. 3 falls out of the same statistics: with the
// keys ordered sink | window | current, the sums l1 after the sink region and l2 after the window region,
// rescaled with l where the reference goes up, give a row's region masses as l1/l, (l2 - l1)/l and the remainder.  Each unit
// leaves the sums of its rows; the first workgroup adds them up per head when all
// workgroups are on the device at once, else (and for a single team of several
// workgroups) the second kernel does, in the same order.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <numeric>
#include <type_traits>
#include <vector>

#include "df_internal.h"

namespace df {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kBQ = kWaves * 32;   // queries per workgroup ...
constexpr int kHalfBQ = kBQ / 2;   // ... and where its two groups of waves share the queries and halve every tile's keys
constexpr int kKT = 64;            // keys per LDS tile
constexpr int kNBuf = 4;           // LDS buffers per operand
constexpr float kSumLimit = 0x1p100f; // the references are raised when the running sums of a lane's two rows pass this
constexpr int kXcd = 8;            // XCDs per device: consecutive workgroup ids go to consecutive XCDs
constexpr int kNumCU = 256;        // MI355X: one workgroup per CU (LDS-bound occupancy)
constexpr int kMinSpan = 8;        // do not cut the work finer than this many key tiles per team ...
constexpr int kMinSmallSpan = 4;   // ... nor, where the spans are chosen by their cost, finer than this;
constexpr int kMaxCostSpan = 64;   // which they are where all of them together would be shorter than this
constexpr int kSpinLimit = 1 << 22; // polls of a hand-over flag before a workgroup gives up (seconds; normally one poll)

// One head as the kernels read it.  The table is sorted by descending key count.
struct HeadRec {
  int64_t off;         // first history row
  int32_t len;         // history rows that hold keys (a prefix of the head's rows)
  int32_t sink;        // of these, sink rows
  int32_t head;        // index of the head
  uint32_t cut;        // a launch that cuts unit by unit (see cut_units): span behind the head's last one; UnitPieces::length << 16
};

struct AttnParams {
  const u16 *q, *k_cur, *v_cur, *k_hist, *v_hist;
  u16 *out;
  float *lse;          // [H, Nq] or null
  float *part;         // workspace: [H, n_qtiles, 4] partial score sums, or null
  int32_t *tickets;    // workspace: [H] counters of the merged units of a head (zeroed by the main kernel), or null
  unsigned long long *flags;   // workspace: one word per workgroup, = epoch once its hand-over sum is in memory
  unsigned long long epoch;    // this launch's flag value: random, so that memory never holds it by chance
  int32_t handoff;     // cut units are put together inside the main kernel (needs all workgroups on the device at once);
                       // 2 + n: and the reader of flag n gives up on it without a poll (see lost_flag(); a parameter of
                       // its own cost a scored launch 0.4 us, by the scalar register that it holds)
  float *slots;        // workspace: 2 partial-result slots per workgroup (see Slot)
  float *score;        // [H, 3] frame attention scores, or null
  unsigned long long *done;    // one word per workgroup, = epoch once its units' score sums are in memory; null: the
                               // second kernel sums the scores
  int64_t q_st, q_sh, kc_st, kc_sh, o_st, o_sh;
  int32_t Nq, Nc, H, n_qtiles;
  int32_t team_size, n_teams, n_groups;   // members of a team, teams (= spans), groups of team_size query tiles
  int32_t total_cols;          // key tiles of all heads
  int64_t line_len;            // n_groups * total_cols: positions of the line the teams share out
  int16_t n_cut_units[kMaxHeads];   // units of a head that span boundaries cut (put together by the merge kernel)
  int64_t span_base;           // positions per span: line_len / n_teams ...
  int32_t span_rem;            // ... and line_len % n_teams, spread evenly over the spans
  uint32_t by_n_teams, by_team_size;   // reciprocals: see divide_small
  int32_t cum[kMaxHeads + 1];  // first column of the hh-th longest head
  uint32_t cur_bytes;  // addressable bytes of one head's current-chunk rows: ((Nc-1)*kc_st + d) * 2
  float c;             // softmax_scale * log2(e)
  float lse_unit;      // softmax_scale / c: natural logarithm of one unit of the references
  HeadRec rec[kMaxHeads];      // heads sorted by descending key count
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ unsigned pack_bf16x2(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 h = __builtin_convertvector(f, bf16x2);
  return __builtin_bit_cast(unsigned, h);
}

// Sum over the four lanes (lane % 16 + 0, 16, 32, 48) that share a query.
__device__ __forceinline__ float quad_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// A lane's value for query block g % 2 (by value: an address that depends on the lane would put the pair into memory).
__device__ __forceinline__ float of_block(int g, const float (&x)[2]) {
  const float x0 = x[0], x1 = x[1];
  return (g & 1) ? x1 : x0;
}
__device__ __forceinline__ float of_block(int, const float (&x)[1]) { return x[0]; }

// Workgroup barrier that waits for this wave's LDS traffic only: global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Key, inside a block of 16, of row i of a product's A operand (row i of the first product's result, k index i of the
// second's): rows 4..11 are the keys 0, 1, 4, 5, 8, 9, 12, 13, so that the reads of the operands are free of bank
// conflicts (see TileLayout).  key_of_row(4 g + v) = key_of_row(4 g) + key_of_row(4 + v) for v < 4.
__host__ __device__ constexpr int key_of_row(int i) {
  return (i & 1) | ((i & 2) << 1) | ((((i >> 2) + 1) & 2) ? 0 : 2) | (i & 8);
}
// The tile loop adds the keys of rows 4..7 to that of a lane's first row when it masks a region's end, and takes the 16 rows
// of a block as 16 keys.
constexpr bool rows_are_as_the_tile_loop_masks_them() {
  unsigned keys = 0;
  for (int i = 0; i < 16; ++i) {
    if (key_of_row(i) != key_of_row(i & ~3) + key_of_row(4 + (i & 3))) return false;
    keys |= 1u << key_of_row(i);
  }
  return keys == 0xffffu;
}
static_assert(rows_are_as_the_tile_loop_masks_them(), "the tile loop's masks follow key_of_row");

// LDS layout of one 64-key tile (all sizes in bytes).  Row r lives in group r % NG at position
// r / NG; a group is the 1 KB one buffer_load ... lds instruction writes, followed by a pad.
template <int D>
struct TileLayout {
  static constexpr int ROWB = D * 2;            // bytes per row
  static constexpr int RPG = 1024 / ROWB;       // rows per group
  static constexpr int NG = kKT / RPG;          // groups per tile
  static constexpr int KGS = 1024 + 16;         // K group stride
  static constexpr int VGS = 1024 + 32;         // V group stride
  static constexpr int KTILE = NG * KGS, VTILE = NG * VGS;
  static_assert(kNBuf * KTILE >= kBQ * ROWB, "a unit's output rows pass through the K buffers");
  // A lane of quarter g reads the 16-byte chunks first_chunk(g) + ks of its K row, ks = 0 .. D/32 - 1.  The hardware
  // takes the lanes of a ds_read_b128 in the groups {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31} and the same + 32;
  // row r begins at bank slot (16 bytes) r, so a group reads slots {r of its rows in quarter 0 or 2} and
  // {r + 4 of its rows in quarter 1 or 3}: with rows 4..11 on keys 0, 1 mod 4 and the others on 2, 3 mod 4 all 16
  // differ.
  static constexpr int first_chunk(int g) { return 4 * (g & 1) + (D == 128 ? 8 : 2) * (g >> 1); }
  // The four quarters' D / 32 chunks in a row are all chunks of the row: the tile loop reads first_chunk(g) + ks at offset 16 ks.
  static constexpr bool quarters_share_a_row() {
    unsigned chunks = 0;
    for (int g = 0; g < 4; ++g)
      for (int ks = 0; ks < D / 32; ++ks) chunks |= 1u << (first_chunk(g) + ks);
    return chunks == (1u << (D / 8)) - 1u;
  }
  // A wave's rows of Q pass through LDS with chunk c of row r at place c ^ q_swizzle(r): the reads of the fragments are then free of bank
  // conflicts (rows 4 to 11 of 16 are read by another quarter of the wave than rows 0 to 3 and 12 to 15, four chunks on).
  __host__ __device__ static constexpr int q_swizzle(int r) { return (D == 128 ? r & 15 : (r >> 1) & 7) ^ (((r + 4) & 8) >> 1); }
  static constexpr int k_row(int r) { return (r % NG) * KGS + (r / NG) * ROWB; }
  static constexpr int v_row(int r) { return (r % NG) * VGS + (r / NG) * ROWB; }
};

__device__ __forceinline__ unsigned lds_address(const void *ptr) {
  return unsigned(reinterpret_cast<uintptr_t>(ptr));     // low half of a flat LDS address = LDS offset
}

static_assert(TileLayout<128>::quarters_share_a_row() && TileLayout<64>::quarters_share_a_row(), "the tile loop's K operands");

// Buffer descriptor of `bytes` bytes from `base` on (loads past its end return zeros), as the four words themselves.
__device__ __forceinline__ u32x4 buffer_descriptor(const u16 *base, uint32_t bytes) {
  const uint64_t addr = reinterpret_cast<uint64_t>(base);
  return u32x4{uint32_t(addr), uint32_t(addr >> 32) & 0xffffu, bytes, 0x00020000u};
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t as_buffer(const u32x4 &words) {
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(uint64_t(words[0]) | uint64_t(words[1]) << 32), 0,
                                           int(words[2]), int(words[3]));
}

// What the tile loop of a piece needs besides the queries (uniform, or one value per lane where it says so) ...
struct TileLoopArgs {
  int t_begin, te;             // first tile of the piece, tile behind its last
  int nt0, nt1;                // tile behind the sink region, tile behind the window region
  int sink, win, nc;           // keys of the sink region, the window region, the current chunk
  unsigned cs;                 // bytes between rows of the current chunk
  int grp;                     // group of the wave
  unsigned ldsk, ldsv;         // LDS addresses of the wave's first row group in the K and V buffers
  float c, lim;                // scale of the logits in units of log2; row sum beyond which the reference is raised
  unsigned ka, va;             // per lane: LDS addresses of the first K and V operand in buffer 0
  unsigned offh, offc;         // per lane: byte offset of the lane's 16 bytes in the first tile, history and current chunk
  int key0;                    // per lane: key of the first of the lane's four rows of a block
  u32x4 kh, kc, vh, vc;        // buffer descriptors: history and current chunk of K and V
};
// ... and what it leaves for the lane's two queries besides O: reference of the exponentials in units of log2 (its
// negative), the lane's share of the row sum relative to it, and of the sums up to the end of the sink and window region.
struct RowSums {
  float neg_ref[2], l[2], l_sink[2], l_hist[2];
};
template <int D, bool SCORE_ONLY, bool LIVE>
__device__ __forceinline__ void tile_loop(const TileLoopArgs &a, const bf16x8 (&qf)[D / 32][2], f32x4 (&o)[D / 16][2], RowSums &r);
// The same for 32 keys of every tile, from the addresses and keys in `a` on.
template <int D, bool SCORE_ONLY>
__device__ __forceinline__ void half_tile_loop(const TileLoopArgs &a, const bf16x8 (&qf)[D / 32][2], f32x4 (&o)[D / 16][2], RowSums &r);
#include "df_attn_phase.inc"

typedef __attribute__((address_space(3))) void lds_void;

// First of the rows that a wave finishes: 32, or where the two groups share a workgroup's queries, the first or second 16 of the 32 it has
// in common with a wave of the other group.
template <int NQB>
__device__ __forceinline__ int first_row(int qt, int wave) {
  return NQB == 2 ? qt * kBQ + 32 * wave : qt * kHalfBQ + 32 * (wave & 3) + 16 * (wave >> 2);
}

// Partial result of one piece of a unit, as the main kernel leaves it in the workspace and the
// merge kernel reads it back.  Both kernels use the same thread <-> element mapping, so the layout
// is simply "in register order": per thread 4 statistics (reference, l, l_sink, l_sink+window) and D/8 vectors of
// 4 consecutive output elements.  A thread holds the same statistics as three other lanes for each of its two
// queries: it writes those of query block (lane / 16) % 2 and reads its blocks' from lanes lane % 16 and
// 16 + lane % 16 of its wave.  Where a workgroup has half the queries (NQB = 1) a wave ends up with one block of 16.
template <int D, int NQB = 2>
struct Slot {
  static constexpr int kStats = kThreads * 4;                   // floats
  static constexpr int kFloats = kStats + kThreads * (D / 16 * NQB) * 4;
  __device__ static float *stats(float *slot, int tid) { return slot + 4 * tid; }
  __device__ static int stats_reader(int tid, int qb) { return (tid & ~63) + 16 * qb + (tid & 15); }
  __device__ static float *ovec(float *slot, int tid, int i) { return slot + kStats + (i * kThreads + tid) * 4; }
};

// A partial result may be handed from one workgroup to another while the kernel runs (see the piece
// loop).  The L2 caches of the eight XCDs are not kept coherent with each other for ordinary accesses,
// so this data is written and read with the cache-control bits of a system-scope atomic access (sc0
// sc1: stores write through to memory, loads are served from memory) - the same bits the compiler puts
// on a relaxed system-scope atomic, here on 16-byte accesses - instead of cache maintenance, which
// would also throw the K/V tiles the team shares out of L2.
// The idle cycles keep the next instruction off the data registers while the store still reads them (a store of more
// than 8 bytes needs one wait state, which the compiler does not add to inline asm: without it the next address went
// into the first statistics of the last four lanes of every 16).
template <class T, class V>
__device__ __forceinline__ void store4_through(T *ptr, const V &v) {
  static_assert(sizeof(V) == 16, "four registers");
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(ptr), "v"(v) : "memory");
}
// The loads below take their base from scalar registers.  A vector instruction that writes one - the compiler keeps scalars
// in lanes of vector registers and reads them back with v_readlane - must lie five wait states before a vector memory
// instruction that reads it, and the compiler does not look into asm for such an instruction: the statements begin with them.
// The statistics of the thread's two queries from four slots, all loads in flight at once and one wait; `reader` is the
// lane that wrote those of the first query (Slot::stats_reader), the second's lie 16 lanes on.
__device__ __forceinline__ void load_stats_through(const float *s0, const float *s1, const float *s2, const float *s3,
                                                   int reader, f32x4 (&st)[4][2]) {
  asm volatile(
      "s_nop 4\n\t"
      "global_load_dwordx4 %0, %8, %9 sc0 sc1\n\t"
      "global_load_dwordx4 %1, %8, %9 offset:256 sc0 sc1\n\t"
      "global_load_dwordx4 %2, %8, %10 sc0 sc1\n\t"
      "global_load_dwordx4 %3, %8, %10 offset:256 sc0 sc1\n\t"
      "global_load_dwordx4 %4, %8, %11 sc0 sc1\n\t"
      "global_load_dwordx4 %5, %8, %11 offset:256 sc0 sc1\n\t"
      "global_load_dwordx4 %6, %8, %12 sc0 sc1\n\t"
      "global_load_dwordx4 %7, %8, %12 offset:256 sc0 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : "=&v"(st[0][0]), "=&v"(st[0][1]), "=&v"(st[1][0]), "=&v"(st[1][1]), "=&v"(st[2][0]), "=&v"(st[2][1]),
        "=&v"(st[3][0]), "=&v"(st[3][1])
      : "v"(unsigned(reader) * 16u), "s"(s0), "s"(s1), "s"(s2), "s"(s3)
      : "memory");
}

// A whole slot (the statistics of the thread's two queries and its N = D/8 vectors of O) with every load in flight at
// once and one wait: the slot's address is uniform, the thread's part of it is tid * 16 bytes, vectors are 8 KB apart.
template <int N>
__device__ __forceinline__ void load_slot_through(const float *slot, int tid, f32x4 (&st)[2], f32x4 (&v)[N]);
template <>
__device__ __forceinline__ void load_slot_through<16>(const float *slot, int tid, f32x4 (&st)[2], f32x4 (&v)[16]) {
  static_assert(Slot<128>::kStats * 4 == 0x2000 && kThreads * 16 == 0x2000, "offsets of the asm below");
  const unsigned vo = unsigned(tid) * 16u, so = unsigned(Slot<128>::stats_reader(tid, 0)) * 16u;
  unsigned t0, t1;
  asm volatile(
      "s_nop 4\n\t"
      "global_load_dwordx4 %[s0], %[so], %[sb] sc0 sc1\n\t"
      "global_load_dwordx4 %[s1], %[so], %[sb] offset:256 sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x2000, %[vo]\n\t"
      "global_load_dwordx4 %[v0], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x4000, %[vo]\n\t"
      "global_load_dwordx4 %[v1], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x6000, %[vo]\n\t"
      "global_load_dwordx4 %[v2], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x8000, %[vo]\n\t"
      "global_load_dwordx4 %[v3], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0xa000, %[vo]\n\t"
      "global_load_dwordx4 %[v4], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0xc000, %[vo]\n\t"
      "global_load_dwordx4 %[v5], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0xe000, %[vo]\n\t"
      "global_load_dwordx4 %[v6], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x10000, %[vo]\n\t"
      "global_load_dwordx4 %[v7], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x12000, %[vo]\n\t"
      "global_load_dwordx4 %[v8], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x14000, %[vo]\n\t"
      "global_load_dwordx4 %[v9], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x16000, %[vo]\n\t"
      "global_load_dwordx4 %[v10], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x18000, %[vo]\n\t"
      "global_load_dwordx4 %[v11], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x1a000, %[vo]\n\t"
      "global_load_dwordx4 %[v12], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x1c000, %[vo]\n\t"
      "global_load_dwordx4 %[v13], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x1e000, %[vo]\n\t"
      "global_load_dwordx4 %[v14], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x20000, %[vo]\n\t"
      "global_load_dwordx4 %[v15], %[t1], %[sb] sc0 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : [s0] "=&v"(st[0]), [s1] "=&v"(st[1]), [v0] "=&v"(v[0]), [v1] "=&v"(v[1]), [v2] "=&v"(v[2]), [v3] "=&v"(v[3]), [v4] "=&v"(v[4]), [v5] "=&v"(v[5]), [v6] "=&v"(v[6]), [v7] "=&v"(v[7]), [v8] "=&v"(v[8]), [v9] "=&v"(v[9]), [v10] "=&v"(v[10]), [v11] "=&v"(v[11]), [v12] "=&v"(v[12]), [v13] "=&v"(v[13]), [v14] "=&v"(v[14]), [v15] "=&v"(v[15]), [t0] "=&v"(t0), [t1] "=&v"(t1)
      : [vo] "v"(vo), [so] "v"(so), [sb] "s"(slot)
      : "memory");
}
template <>
__device__ __forceinline__ void load_slot_through<8>(const float *slot, int tid, f32x4 (&st)[2], f32x4 (&v)[8]) {
  static_assert(Slot<64>::kStats * 4 == 0x2000 && kThreads * 16 == 0x2000, "offsets of the asm below");
  const unsigned vo = unsigned(tid) * 16u, so = unsigned(Slot<64>::stats_reader(tid, 0)) * 16u;
  unsigned t0, t1;
  asm volatile(
      "s_nop 4\n\t"
      "global_load_dwordx4 %[s0], %[so], %[sb] sc0 sc1\n\t"
      "global_load_dwordx4 %[s1], %[so], %[sb] offset:256 sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x2000, %[vo]\n\t"
      "global_load_dwordx4 %[v0], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x4000, %[vo]\n\t"
      "global_load_dwordx4 %[v1], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0x6000, %[vo]\n\t"
      "global_load_dwordx4 %[v2], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x8000, %[vo]\n\t"
      "global_load_dwordx4 %[v3], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0xa000, %[vo]\n\t"
      "global_load_dwordx4 %[v4], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0xc000, %[vo]\n\t"
      "global_load_dwordx4 %[v5], %[t1], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t0], 0xe000, %[vo]\n\t"
      "global_load_dwordx4 %[v6], %[t0], %[sb] sc0 sc1\n\t"
      "v_add_u32 %[t1], 0x10000, %[vo]\n\t"
      "global_load_dwordx4 %[v7], %[t1], %[sb] sc0 sc1\n\t"
      "s_waitcnt vmcnt(0)"
      : [s0] "=&v"(st[0]), [s1] "=&v"(st[1]), [v0] "=&v"(v[0]), [v1] "=&v"(v[1]), [v2] "=&v"(v[2]), [v3] "=&v"(v[3]), [v4] "=&v"(v[4]), [v5] "=&v"(v[5]), [v6] "=&v"(v[6]), [v7] "=&v"(v[7]), [t0] "=&v"(t0), [t1] "=&v"(t1)
      : [vo] "v"(vo), [so] "v"(so), [sb] "s"(slot)
      : "memory");
}

// Weighted sum of an earlier piece's value and the later pieces', written out so that both places that
// put pieces together (in the main kernel and in the merge kernel) round in the same way.
__device__ __forceinline__ float fold(float earlier, float w_earlier, float later, float w_later) {
  return __fmaf_rn(earlier, w_earlier, __fmul_rn(later, w_later));
}

// Partial-result slot of (span, first or later piece of the span, member of the team).
__host__ __device__ __forceinline__ int64_t slot_index(const AttnParams &p, int span, int which, int member) {
  return int64_t(2 * span + which) * p.team_size + member;
}

// x / n for x < 2^16 and n <= 2^8 with the reciprocal 2^32 / n, rounded up (2^32 - 1 for n = 1): it is too large by less
// than n / 2^32 of itself, and x times that is less than 1 / n.
__host__ __device__ __forceinline__ int divide_small(uint32_t x, uint32_t reciprocal) {
  return int(uint32_t((uint64_t(x) * reciprocal + (reciprocal == UINT32_MAX ? x : 0u)) >> 32));
}
static uint32_t reciprocal_of(int n) { return n == 1 ? UINT32_MAX : uint32_t(((uint64_t(1) << 32) + n - 1) / n); }

// Where the work is cut.  The line has one position per (group of query tiles, column); span s covers
// positions [span_begin(s), span_begin(s+1)), span_begin(s) = floor(s * line_len / n_teams).  Host and device
// use the same arithmetic: with line_len = n_teams * span_base + span_rem only s * span_rem is left to divide,
// which is less than kNumCU^2 (a workgroup needs several of them before it can issue its first load).
__host__ __device__ __forceinline__ int64_t span_begin(const AttnParams &p, int s) {
  return s * p.span_base + divide_small(unsigned(s * p.span_rem), p.by_n_teams);
}

// One piece of a span: the part of a unit (group of query tiles x head) that the span holds.  The same
// walk - from the span's end to its start - is taken by the kernel and by the host check of a plan.
struct Piece {
  int grp, hh;          // group of query tiles; head (index into the length-sorted order)
  int n_tiles;          // key tiles of the unit
  int t_begin, t_end;   // the piece: tiles [t_begin, t_end) of the unit
  int64_t unit_lo;      // line position of the unit's first tile
  int64_t pos;          // line position of the piece's first tile
};
// Head (index into the length-sorted order) that owns column `col`.
__host__ __device__ __forceinline__ int head_of_column(const AttnParams &p, int col) {
  int hh = 0;
  while (col >= p.cum[hh + 1]) ++hh;
  return hh;
}
// The two ways to look a column up: one after the other in the parameters (host, merge kernel) ...
struct ColumnsInParams {
  const AttnParams &p;
  __host__ __device__ __forceinline__ int head_of(int col) const { return head_of_column(p, col); }
  __host__ __device__ __forceinline__ int first(int hh) const { return p.cum[hh]; }
};
// ... or one head per lane in the main kernel's copy in LDS.
struct ColumnsInLds {
  const int *cum;      // [kMaxHeads + 1], INT32_MAX past the last head
  __device__ __forceinline__ int head_of(int col) const {
    return __popcll(__ballot(col >= cum[(threadIdx.x & 63) + 1]));
  }
  __device__ __forceinline__ int first(int hh) const { return __builtin_amdgcn_readfirstlane(cum[hh]); }
};

// The piece of span [span_lo, ...) that ends at line position pos_end (span_lo < pos_end <= the span's end).
template <class Columns>
__host__ __device__ __forceinline__ Piece piece_ending_at(const AttnParams &p, const Columns &columns, int64_t span_lo,
                                                          int64_t pos_end) {
  Piece c;
  const int64_t last = pos_end - 1;
  c.grp = p.n_groups == 1 ? 0 : (p.line_len <= int64_t(UINT32_MAX) ? int(uint32_t(last) / uint32_t(p.total_cols))
                                                                   : int(last / p.total_cols));
  const int col = int(last - int64_t(c.grp) * p.total_cols);
  c.hh = columns.head_of(col);
  c.n_tiles = columns.first(c.hh + 1) - columns.first(c.hh);
  c.unit_lo = int64_t(c.grp) * p.total_cols + columns.first(c.hh);
  c.pos = span_lo > c.unit_lo ? span_lo : c.unit_lo;
  c.t_begin = int(c.pos - c.unit_lo);
  c.t_end = int(pos_end - c.unit_lo);
  return c;
}

// Normalise and round four consecutive output elements.
__device__ __forceinline__ uint2 output4(const f32x4 &o, float inv) {
  uint2 w;
  w.x = pack_bf16x2(o[0] * inv, o[1] * inv);
  w.y = pack_bf16x2(o[2] * inv, o[3] * inv);
  return w;
}
// A wave's 32 (16 * NQB) finished rows (first row row0) go through LDS, `buf` being the wave's own 32 * D bf16 there, and out with
// 16 bytes per lane and whole rows side by side.  In the accumulator layout a lane holds 8-byte bits of two rows, and
// a store of those touches 32 rows: with the 32x32 products of an earlier version, which held 8-byte bits of one row,
// issuing 16 of them and draining them took 5 to 6 us a unit.  Both ways on one box at that time, direct -> through LDS:
// 1170 queries 44.1 -> 42.1 us, 832x480 308.0 -> 305.0, packed-dummy step 234.8 -> 230.7, histories of 3 to 60 frames
// 610.0 -> 601.9; a launch of 64 queries 15.1 -> 15.8.
// 16-byte chunk c of row r lies at position c ^ (r mod chunks per row).  The reads are then free of bank conflicts; the
// 8-byte writes are not: 4 cycles each (264,192 in a 1280x720 launch, 0.03 % of the CU-busy cycles).
// Units of 256 queries write them through to memory, so that a launch does not end with writing its rows back from L2.  In L2 -> through, medians of
// 40 turns on one box: 909 queries of 40 heads 38.6 -> 37.8 us, with an elementwise kernel that reads the rows behind it 43.9 -> 43.3; 2340 of 12
// heads 82.1 -> 81.6; 832x480 258.5 -> 257.1 and 261.5 -> 261.0, which the turns' own spread (quartiles 0.8 apart) hardly tells apart.
// The rows of units of 128, the smaller launches, stay in L2, where the next kernel finds them: 200 queries and that kernel 13.0 us, through 13.15.
template <int D, int NQB>
__device__ __forceinline__ void store_output(const AttnParams &p, int h, int row0, unsigned char *buf, int lane,
                                             const f32x4 (&o)[D / 16][NQB], const float (&inv)[NQB]) {
  constexpr int kChunks = D / 8;                   // 16-byte chunks per row
  const int g = lane >> 4;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int r = 16 * qb + (lane & 15);
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
      *reinterpret_cast<uint2 *>(buf + r * 2 * D + 16 * ((2 * db + (g >> 1)) ^ (r % kChunks)) + 8 * (g & 1)) =
          output4(o[db][qb], inv[qb]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // lanes read what other lanes of the wave wrote
  const int c = lane % kChunks;
#pragma unroll
  for (int i = 0; i < kChunks * NQB / 4; ++i) {
    const int r = i * (64 / kChunks) + lane / kChunks;
    const u32x4 v = *reinterpret_cast<const u32x4 *>(buf + r * 2 * D + 16 * (c ^ (r % kChunks)));
    if (row0 + r < p.Nq) {
      u16 *to = p.out + (row0 + r) * p.o_st + h * p.o_sh + 8 * c;
      if constexpr (NQB == 2) store4_through(to, v);
      else *reinterpret_cast<u32x4 *>(to) = v;
    }
  }
}

// Log-sum-exp of a wave's 16 * NQB finished rows: quarter qb of the wave writes those of query block qb.
template <int NQB>
__device__ __forceinline__ void store_lse(const AttnParams &p, int h, int row0, int lane, const float (&ref)[NQB],
                                          const float (&lt)[NQB]) {
  const int row = row0 + lane;
  if (p.lse != nullptr && lane < 16 * NQB && row < p.Nq) {
    // The parts are added in 64 bits, so that the sum is rounded once; the logarithm is that of l's mantissa, whose error is small.  Relative error
    // over 20 launches, sum and logarithm in 32 bits -> so: 4.7e-8 -> 2.7e-8.
    const float l = of_block(lane >> 4, lt);
    const double parts = double(of_block(lane >> 4, ref)) * double(p.lse_unit) + double(__builtin_amdgcn_frexp_expf(l)) * 0.6931471805599453;
    p.lse[int64_t(h) * p.Nq + row] = float(parts + double(__logf(__builtin_amdgcn_frexp_mantf(l))));
  }
}

// Region masses (sink, sink + window) of a lane's rows `row` and, of a second block, row + 16.
template <int NQB>
__device__ __forceinline__ void unit_masses(const AttnParams &p, int row, const float (&lt)[NQB], const float (&l1)[NQB],
                                            const float (&l2)[NQB], float &mass_a, float &mass_b) {
  const float inv0 = 1.f / lt[0], inv1 = 1.f / lt[NQB - 1];
  const bool in0 = row < p.Nq, in1 = NQB == 2 && row + 16 < p.Nq;
  mass_a = (in0 ? l1[0] * inv0 : 0.f) + (in1 ? l1[NQB - 1] * inv1 : 0.f);
  mass_b = (in0 ? l2[0] * inv0 : 0.f) + (in1 ? l2[NQB - 1] * inv1 : 0.f);
}
// Sum of the two region masses over the 256 (128) rows of a unit, in a fixed order (deterministic): a
// butterfly over the 32 rows of every wave, two to a lane (16, one to a lane), then the 8 waves in order.  The four lanes of a query hold
// the same masses, so the butterfly stays inside 16 lanes.
__device__ __forceinline__ void reduce_masses(const AttnParams &p, float *lds_red, int h, int qt, int tid,
                                              float mass_a, float mass_b) {
  const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    mass_a += __shfl_xor(mass_a, m);
    mass_b += __shfl_xor(mass_b, m);
  }
  if (lane == 0) {
    lds_red[2 * wave] = mass_a;
    lds_red[2 * wave + 1] = mass_b;
  }
  lds_barrier();
  if (tid < 2) {
    double acc = 0.0;
    for (int w = 0; w < kWaves; ++w) acc += double(lds_red[2 * w + tid]);
    // written through: the sums of all units may be read by another workgroup of this launch
    __hip_atomic_store(p.part + (int64_t(h) * p.n_qtiles + qt) * 4 + tid, float(acc), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  lds_barrier();
}

// F[h] = (sum_a, sum_b - sum_a, n - sum_b) / n over the head's query tiles, in tile order: in 64 bits, so that all of it is rounded once.
__device__ __forceinline__ void store_score(const AttnParams &p, int h, double a, double b) {
  const double n = double(p.Nq), inv = 1.0 / n;
  p.score[3 * h] = float(a * inv);
  p.score[3 * h + 1] = float((b - a) * inv);
  p.score[3 * h + 2] = float((n - b) * inv);
}
__device__ __forceinline__ void finish_score(const AttnParams &p, int h) {
  double a = 0.0, b = 0.0;
  for (int t = 0; t < p.n_qtiles; ++t) {
    a += double(p.part[(int64_t(h) * p.n_qtiles + t) * 4]);
    b += double(p.part[(int64_t(h) * p.n_qtiles + t) * 4 + 1]);
  }
  store_score(p, h, a, b);
}

template <int D>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t all_slots(const AttnParams &p) {
  return __builtin_amdgcn_make_buffer_rsrc(p.slots, 0, int(2u * kNumCU * unsigned(sizeof(float) * Slot<D>::kFloats)), 0x00020000);
}
// A system-scope load (sc0 sc1, see store4_through) that the compiler waits for where it is used.
__device__ __forceinline__ f32x4 slot_load4(const __amdgpu_buffer_rsrc_t &slots, unsigned lane_offset, unsigned offset) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slots, int(lane_offset), int(offset), 1 | 16));
}

// Wait, for a bounded time, until a flag word holds this launch's value.  `number` is the flag's in lost_flag()'s numbering.
__device__ __forceinline__ int await_flag(const AttnParams &p, unsigned long long *flag, int number) {
  int up = 0;
  for (int spin = number == p.handoff - 2 ? kSpinLimit : 0; spin < kSpinLimit && !up; ++spin) {
    up = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == p.epoch;
    if (!up) __builtin_amdgcn_s_sleep(16);
  }
  return up;
}
// Put it back: a flag is read by one workgroup, and a replay of the launch (same value) has to start clean.
__device__ __forceinline__ void reset_flag(unsigned long long *flag) {
  __hip_atomic_store(flag, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ int take_flag(const AttnParams &p, unsigned long long *flag, int number) {
  const int up = await_flag(p, flag, number);
  reset_flag(flag);
  return up;
}

// The frame attention scores of all heads, by the first workgroup at the end of its span: when every workgroup has
// raised its flag, the units' sums come into LDS (`buf`, room for PAIRS of them) with all threads loading, and
// one thread per head adds its tiles up in finish_score's order, so that both ways give the same bits.  A second
// launch for these few sums took 4 to 6 us by the kernel trace; this costs two trips to memory (1170 queries 44.7 ->
// 43.4 us, 832x480 sampled scores 67.4 -> 65.6).  An atomic counter per head instead of the flags puts a trip on every
// unit's path.
template <int PAIRS>
__device__ __forceinline__ void finish_all_scores(const AttnParams &p, float2 *buf, int *all_up, int tid) {
  const int n_wg = p.n_teams * p.team_size;
  if (tid == 0) *all_up = 1;
  __syncthreads();
  if (tid < n_wg && !take_flag(p, p.done + tid, kNumCU + tid)) *all_up = 0;
  __syncthreads();
  const double poison = *all_up ? 0.0 : double(NAN);
  static_assert(PAIRS >= kMaxHeads, "one tile of every head");
  const int tiles_at_once = PAIRS / p.H;
  double a = 0.0, b = 0.0;
  for (int t0 = 0; t0 < p.n_qtiles; t0 += tiles_at_once) {
    const int n = min(tiles_at_once, p.n_qtiles - t0);
    for (int i = tid; i < p.H * n; i += kThreads) {
      const int h = i / n, t = i - h * n;
      const unsigned long long both =
          __hip_atomic_load(reinterpret_cast<unsigned long long *>(p.part + (int64_t(h) * p.n_qtiles + t0 + t) * 4),
                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      buf[i] = __builtin_bit_cast(float2, both);
    }
    __syncthreads();
    if (tid < p.H)
      for (int t = 0; t < n; ++t) {
        a += double(buf[tid * n + t].x);
        b += double(buf[tid * n + t].y);
      }
    __syncthreads();
  }
  if (tid < p.H) store_score(p, tid, a + poison, b + poison);
}

template <bool FIRST, class A, class B>
__device__ __forceinline__ auto &either(A &a, B &b) {
  if constexpr (FIRST) return a;
  else return b;
}

// Where the two groups of waves hold sums of the same queries over different keys: wave w of group 0 finishes the first block of 16 of their 32
// queries and wave w + 4 of group 1 the second.  Each leaves the other's block in LDS (statistics, then O) and returns what it finds of its own.
template <int D, bool SCORE_ONLY>
__device__ __forceinline__ f32x4 exchange_halves(f32x4 *from_group0, f32x4 *from_group1, int group, int wave, int lane, const f32x4 &stats,
                                                 const f32x4 (&o)[D / 16][2], f32x4 (&theirs)[D / 16][1]) {
  constexpr int kVectors = SCORE_ONLY ? 1 : 1 + D / 16;
  static_assert(SCORE_ONLY || 4 * kVectors * 1024 <= kNBuf * TileLayout<D>::KTILE, "four waves' vectors in the K or the V buffers");
  f32x4 *mine = (group ? from_group1 : from_group0) + (wave & 3) * kVectors * 64 + lane;
  const f32x4 *other = (group ? from_group0 : from_group1) + (wave & 3) * kVectors * 64 + lane;
  mine[0] = stats;
  if (!SCORE_ONLY) {
#pragma unroll
    for (int db = 0; db < D / 16; ++db) mine[(1 + db) * 64] = group ? o[db][0] : o[db][1];
  }
  lds_barrier();
  const f32x4 st = other[0];
  if (!SCORE_ONLY) {
#pragma unroll
    for (int db = 0; db < D / 16; ++db) theirs[db][0] = other[(1 + db) * 64];
  }
  lds_barrier();                                   // what follows goes where these lie
  return st;
}
// A whole slot of a workgroup with half the queries, all loads in flight at once (as load_slot_through).  Nothing in the loads says that
// they may not go out before the look at the flag that the sums are there; the empty statement does.
template <int D>
__device__ __forceinline__ void load_half_slot(const AttnParams &p, int64_t slot, int tid, f32x4 &st, f32x4 (&v)[D / 16]) {
  asm volatile("" ::: "memory");
  const __amdgpu_buffer_rsrc_t slots = all_slots<D>(p);
  const unsigned at = unsigned(slot) * unsigned(sizeof(float) * Slot<D, 1>::kFloats);
  st = slot_load4(slots, unsigned(Slot<D, 1>::stats_reader(tid, 0)) * 16u, at);
#pragma unroll
  for (int i = 0; i < D / 16; ++i) v[i] = slot_load4(slots, unsigned(tid) * 16u, at + unsigned((Slot<D, 1>::kStats + i * kThreads * 4) * 4));
  asm volatile("" : "+v"(st));
#pragma unroll
  for (int i = 0; i < D / 16; ++i) asm volatile("" : "+v"(v[i]));
}

// Where a wave's 32 rows of Q lie between their loads and the reads of the fragments: in the tile buffers that a piece's first tiles do
// not use (K's fourth, V's third and fourth), as far as they go.
template <int D, bool SCORE_ONLY>
constexpr int kQBytes = (SCORE_ONLY ? kWaves : 2) * 32 * 2 * D;
template <int D, bool SCORE_ONLY>
__device__ __forceinline__ unsigned char *q_area(unsigned char *lds_k, unsigned char *lds_v, unsigned char *lds_q, int wave) {
  using L = TileLayout<D>;
  constexpr int kWaveBytes = 32 * L::ROWB;
  static_assert(4 * kWaveBytes <= 2 * L::VTILE && 2 * kWaveBytes <= L::KTILE, "rows of Q in the tile buffers");
  if (SCORE_ONLY) return lds_q + wave * kWaveBytes;
  return wave < 4 ? lds_v + 2 * L::VTILE + wave * kWaveBytes
                  : wave < 6 ? lds_k + 3 * L::KTILE + (wave - 4) * kWaveBytes : lds_q + (wave - 6) * kWaveBytes;
}
// The fragments of a wave's 32 rows, once all but the PENDING latest of its loads have landed; `at`: LDS addresses of the lane's chunks of
// the first 16 rows.
template <int D, int PENDING>
__device__ __forceinline__ void read_q(const unsigned (&at)[D / 32], bf16x8 (&qf)[D / 32][2]) {
  if constexpr (D == 128)
    asm volatile(
        "s_waitcnt vmcnt(%12)\n\t"
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:4096\n\t"
        "ds_read_b128 %2, %9\n\t"
        "ds_read_b128 %3, %9 offset:4096\n\t"
        "ds_read_b128 %4, %10\n\t"
        "ds_read_b128 %5, %10 offset:4096\n\t"
        "ds_read_b128 %6, %11\n\t"
        "ds_read_b128 %7, %11 offset:4096\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(qf[0][0]), "=&v"(qf[0][1]), "=&v"(qf[1][0]), "=&v"(qf[1][1]), "=&v"(qf[2][0]), "=&v"(qf[2][1]), "=&v"(qf[3][0]),
          "=&v"(qf[3][1])
        : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "n"(PENDING)
        : "memory");
  else
    asm volatile(
        "s_waitcnt vmcnt(%6)\n\t"
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:2048\n\t"
        "ds_read_b128 %2, %5\n\t"
        "ds_read_b128 %3, %5 offset:2048\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(qf[0][0]), "=&v"(qf[0][1]), "=&v"(qf[1][0]), "=&v"(qf[1][1])
        : "v"(at[0]), "v"(at[1]), "n"(PENDING)
        : "memory");
}

// The other way to cut a launch: unit by unit, each head's into a number of pieces of its own, one workgroup to a piece.
// No workgroup then pays for a second piece, nor waits for one that does, and a short unit is left whole; it takes few
// enough units to go round.  The fewest pieces go with units of kHalfBQ queries, the fewest tiles for the machine with
// units of kBQ.  UnitCost is the time in us of a launch that is cut so: `start`, `wg` for each workgroup, and for its slowest unit
// `tile` for each tile of its longest piece (`crowd` of it more for each workgroup, `few` of it where half of the waves have no rows and the others
// a SIMD to themselves, or, of units of kHalfBQ, half of its waves), and where it is cut `cut` and for each piece that is
// handed on `fold`.  SpanCost is that of equal spans: `start`, `cost` times span_cost, `tile` for each tile of a span and `wg` for each
// workgroup.  Fitted to 420 launches (1 to 6 000 queries, 2 to 61 heads, up to 100 GFLOP) with the spans that span_cost chooses and up to 14
// cuts by units of either kind measured on each; they meet the times to 3 % by units and 3 to 6 % in spans.  By units if that
// takes units_margin of the spans' time: of the 420, attention then takes 27 % less time on average and scores 10 %, four of them up to
// 4 % more; the cheapest of all cuts measured would be another 1.3 % less.
struct UnitCost {
  float start, wg, tile, crowd, few, cut, fold;
  int ahead, lag;
  // `ahead`: tiles that the last piece of a unit has more than the one before it, done while the others' sums are on the way.  Equal
  // pieces -> so, one box: 1170 queries, every output 29.9 -> 26.8 us, 1170 sampled ones 54.7 -> 53.8; 60 random launches 1.6 % less.
  // `lag`: sixteenths of a tile that each of the pieces before that has more than the next, about `fold`: while the last
  // piece's workgroup folds one, the one before is on its way.  One wait for all flags -> each wave for each piece on its own -> the latter with
  // lag: 46 random attention launches 3.3 and 6.2 % less (half of the lag 4.5, three quarters 5.2; 5/4 and 6/4 as the whole), 290
  // queries and 10 pieces 20.5 -> 18.9 us, 720 queries and 14 pieces 33.9 -> 27.7.  While scoring a fold is a sixth of
  // that, and four go in one trip: no lag there.
};
// The pieces of a unit: all but the last `count` - 1 have `length` tiles and what `lag` adds; where the j-th begins.
struct UnitPieces {
  int count, length, lag;
  __host__ __device__ __forceinline__ int begin(int j) const { return j * length + ((j * (2 * count - 3 - j) / 2 * lag) >> 4); }
};
struct SpanCost {
  float start, cost, tile, wg;
};
struct LaunchCost {
  UnitCost half, whole;        // units of kHalfBQ and of kBQ queries
  SpanCost spans;
};
template <int D, bool SCORE_ONLY>
constexpr LaunchCost kLaunchCost =
    D == 128 ? (SCORE_ONLY ? LaunchCost{{8.26f, 0.0059f, 0.394f, 0.00076f, 0.96f, 1.76f, 0.147f, 3, 0}, {7.63f, 0.0062f, 0.706f, 0.00056f, 0.78f, 1.44f, 0.200f, 1, 0}, {5.83f, 0.371f, 0.600f, 0.f}}
                           : LaunchCost{{8.01f, 0.0117f, 0.576f, 0.00054f, 0.86f, 1.83f, 0.667f, 3, 18}, {7.86f, 0.0169f, 1.048f, 0.00030f, 0.65f, 2.05f, 1.403f, 1, 19}, {1.10f, 1.213f, 0.297f, 0.0148f}})
             : (SCORE_ONLY ? LaunchCost{{7.97f, 0.0079f, 0.342f, 0.00022f, 0.91f, 1.78f, 0.141f, 4, 0}, {7.07f, 0.0084f, 0.613f, 0.00017f, 0.73f, 1.59f, 0.199f, 2, 0}, {5.78f, 0.437f, 0.263f, 0.f}}
                           : LaunchCost{{6.81f, 0.0094f, 0.419f, 0.00030f, 0.90f, 1.59f, 0.489f, 4, 16}, {6.45f, 0.0117f, 0.763f, 0.00023f, 0.71f, 1.58f, 0.800f, 2, 14}, {4.51f, 0.709f, 0.262f, 0.0112f}});

template <int D, bool SCORE_ONLY, bool UNITS, bool HALF>
__global__ __launch_bounds__(kThreads) void df_attn_kernel(const AttnParams p) {
  constexpr int NQB = HALF ? 1 : 2;     // blocks of 16 finished queries per wave
  constexpr bool PIECEWISE = UNITS && !SCORE_ONLY;   // earlier pieces are waited for one by one
  constexpr int KS = D / 32;            // k-steps of the first product
  constexpr int DB = D / 16;            // 16-row blocks of O^T
  using L = TileLayout<D>;
  constexpr int GPW = L::NG / kWaves;   // row groups each wave loads per tile (2 for d=128, 1 for d=64)
  constexpr int kDmaPerPhase = GPW * (SCORE_ONLY ? 1 : 2);   // buffer loads a wave issues per VALU phase
  __shared__ __attribute__((aligned(16))) unsigned char lds_k[kNBuf * L::KTILE];
  __shared__ __attribute__((aligned(16))) unsigned char lds_v[SCORE_ONLY ? 16 : kNBuf * L::VTILE];
  __shared__ __attribute__((aligned(16))) unsigned char lds_q[kQBytes<D, SCORE_ONLY>];
  __shared__ float lds_red[kWaves * 2];
  __shared__ int lds_ok;
  __shared__ int lds_cum[kMaxHeads + 1];
  __shared__ HeadRec lds_rec[kMaxHeads];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int group = wave >> 2;
  const int j = lane & 15, g = lane >> 4;  // the lane's query in a block of 16; its quarter of the wave

  // The head tables, one head per thread: a single trip to memory, and a column is then found with one ballot.
  // (Read where they are needed they were a chain of scalar loads, one per head up to the one sought and three
  // more behind it, each a miss to memory at the start of a launch.)  The loads go out before anything else is
  // known, and one scalar load from each line of the other parameters goes out beside them: the loads that follow
  // where a value is needed then hit the scalar cache (64 queries 16.9 -> 15.9 us, 1170 queries 43.4 -> 41.5,
  // 832x480 1.5 % less).
  // (By units there is one piece, whose head every wave finds in its own copy of the table, in registers.)
  HeadRec lane_rec;
  int lane_cum;
  {
    const int i = UNITS ? lane : tid < kMaxHeads ? tid : 0;
    const HeadRec rec = p.rec[i];
    const int cum = p.cum[i + 1];
    lane_rec = rec;
    lane_cum = cum;
    asm volatile("" ::"s"(p.q), "s"(p.lse_unit), "s"(p.part), "s"(p.slots), "s"(p.q_st), "s"(p.o_sh), "s"(p.n_teams), "s"(p.span_base),
                 "s"(p.H), "v"(cum), "v"(rec.off), "v"(rec.len), "v"(rec.sink), "v"(rec.head), "v"(rec.cut));
    if (!UNITS && tid < kMaxHeads) {
      lds_rec[tid] = rec;
      lds_cum[tid + 1] = tid < p.H ? cum : INT32_MAX;
      if (tid == 0) lds_cum[0] = 0;
    }
  }
  if (!UNITS) __syncthreads();

  // the merge kernel, where there is one, counts the merged units of a head: its counters start at zero (this kernel
  // ends before that one begins)
  if (blockIdx.x == 0 && p.tickets != nullptr && tid < p.H) p.tickets[tid] = 0;

  // ---- this workgroup's team (span of the line) and member index (query tile inside a group); XCD-major numbering
  // (a grid of kXcd workgroups or more is rounded up to a multiple of kXcd; gridDim lies in another line of the
  // kernel's arguments, a miss of its own)
  const int n_wg = p.n_teams * p.team_size;
  const int wg = n_wg >= kXcd ? (blockIdx.x % kXcd) * ((n_wg + kXcd - 1) / kXcd) + blockIdx.x / kXcd : blockIdx.x;
  const int span = divide_small(wg, p.by_team_size), member = wg - span * p.team_size;
  if (span >= p.n_teams) return;
  const int64_t span_lo = UNITS ? 0 : span_begin(p, span);       // by units: one piece, whatever its place
  const int64_t span_hi = UNITS ? 1 : span_begin(p, span + 1);

  // per-lane LDS byte addresses of the MFMA A operands (buffer 0); see TileLayout for the row placement
  const int krow = key_of_row(j), vrow = key_of_row(4 * g + (j >> 2));
  const unsigned k_lane_addr = lds_address(lds_k) + (krow % L::NG) * L::KGS + (krow / L::NG) * L::ROWB + 16 * L::first_chunk(g);
  const unsigned v_lane_addr = lds_address(lds_v) + (vrow % L::NG) * L::VGS + (vrow / L::NG) * L::ROWB + 8 * (j & 3);
  // lane -> (row position inside the group, 16-byte chunk of the row) in the 1 KB a load writes
  const int dma_pos = (16 * lane) / L::ROWB, dma_chunk = (16 * lane) % L::ROWB;
  const uint32_t cur_stride_b = uint32_t(p.kc_st) * 2u;
  const int voff_hist = dma_pos * L::NG * L::ROWB + dma_chunk;
  const int voff_cur = dma_pos * L::NG * int(cur_stride_b) + dma_chunk;
  constexpr uint32_t kNoTile = 0x7ff00000u;      // beyond every descriptor (plus any lane offset): the load writes zeros
  const uint32_t lane_vo_hist = uint32_t(voff_hist) + uint32_t(wave) * L::ROWB;      // lane offset + this wave's first row group
  const uint32_t lane_vo_cur = uint32_t(voff_cur) + uint32_t(wave) * cur_stride_b;

  // The pieces of the span are taken from its end to its start.  A head that a span boundary cuts in two
  // is then begun by the workgroup that has it at the end of its span as the FIRST thing it does, and
  // completed by the workgroup that has the rest at the start of its span as the LAST thing it does: by
  // then the first part has long been in memory, and the second workgroup finishes the unit itself
  // (hand-over) instead of leaving a partial result to a second kernel.
  int s_unit = 0;                                  // by units: span of the unit's first piece
#pragma unroll 1
  for (int64_t pos_end = span_hi; pos_end > span_lo;) {
    // ---- the piece that ends at `pos_end`: group of query tiles, head, first and last tile of this team's share
    Piece piece;
    int h, len_h, sink;
    int64_t hoff;
    if constexpr (UNITS) {
      auto of_head = [](int x, int hh) { return __builtin_amdgcn_readlane(x, hh); };
      const int lane_end = lane < p.H ? int(lane_rec.cut & 0xffffu) : INT32_MAX;
      const int hh = __popcll(__ballot(span >= lane_end));
      const int before = max(hh - 1, 0), first_span = hh ? of_head(lane_end, before) : 0;
      const int n = of_head(lane_cum, hh) - (hh ? of_head(lane_cum, before) : 0), nth = span - first_span;
      const unsigned cut = unsigned(of_head(int(lane_rec.cut), hh));
      constexpr int kLag = (HALF ? kLaunchCost<D, SCORE_ONLY>.half : kLaunchCost<D, SCORE_ONLY>.whole).lag;
      const UnitPieces u{int(cut & 0xffffu) - first_span, int(cut >> 16), kLag};
      piece = {0, hh, n, u.begin(nth), 0, 0, 0};
      piece.t_end = nth + 1 < u.count ? u.begin(nth + 1) : n;
      h = of_head(lane_rec.head, hh);
      len_h = of_head(lane_rec.len, hh);
      sink = of_head(lane_rec.sink, hh);
      hoff = int64_t(uint64_t(uint32_t(of_head(int(lane_rec.off), hh))) | uint64_t(uint32_t(of_head(int(lane_rec.off >> 32), hh))) << 32);
      s_unit = first_span;
    } else {
      piece = piece_ending_at(p, ColumnsInLds{lds_cum}, span_lo, pos_end);
      const HeadRec &rec = lds_rec[piece.hh];
      h = __builtin_amdgcn_readfirstlane(rec.head);
      hoff = int64_t(uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(rec.off)))) |
                     uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(rec.off >> 32)))) << 32);
      len_h = __builtin_amdgcn_readfirstlane(rec.len);
      sink = __builtin_amdgcn_readfirstlane(rec.sink);
    }
    const int grp = piece.grp;
    const int nt0 = (sink + kKT - 1) / kKT;
    const int nt1 = (len_h - sink + kKT - 1) / kKT;
    const int nt2 = (p.Nc + kKT - 1) / kKT;
    const int n_tiles = piece.n_tiles;             // = nt0 + nt1 + nt2
    const int64_t unit_lo = piece.unit_lo;         // line position of the unit's first tile
    const int64_t piece_pos = piece.pos;
    const int t_begin = piece.t_begin, t_end = piece.t_end;
    pos_end = piece_pos;
    // Hand-over: a piece that does not end its unit leaves its partial sums in the workspace and raises a
    // flag; the piece that ends the unit (always the last thing its workgroup does) collects the sums of
    // all earlier pieces - they lie with the same member of the preceding teams - and finishes the unit.
    const bool give = p.handoff && t_end < n_tiles;
    const bool take = p.handoff && t_begin > 0 && t_end == n_tiles;
    const int qt = grp * p.team_size + member;     // this workgroup's query tile in this group
    if (qt >= p.n_qtiles) continue;                // the last group may have fewer tiles than the team has members
    const int q0 = HALF ? qt * kHalfBQ + (wave & 3) * 32 : qt * kBQ + wave * 32;
    // a wave whose 32 rows all lie past the last query (tail of the last query tile) moves tiles and keeps
    // the barriers, but computes nothing
    const bool wave_live = q0 < p.Nq;

    // ---- global -> LDS: buffer descriptors of this head's history and current-chunk rows.  A load
    // past the end of the descriptor returns zeros, which is how partial and absent tiles are padded.
    const uint32_t hist_bytes = uint32_t(len_h) * L::ROWB;
    const u32x4 rs_kh = buffer_descriptor(p.k_hist + hoff * D, hist_bytes);
    const u32x4 rs_kc = buffer_descriptor(p.k_cur + h * p.kc_sh, p.cur_bytes);
    const u32x4 rs_vh = buffer_descriptor((SCORE_ONLY ? p.k_hist : p.v_hist) + hoff * D, hist_bytes);
    const u32x4 rs_vc = buffer_descriptor((SCORE_ONLY ? p.k_cur : p.v_cur) + h * p.kc_sh, p.cur_bytes);
    // Issue this wave's share of tile t (zeros if the piece does not reach it) into LDS buffer `slot`.
    // The whole byte offset travels in the VGPR offset, the only part of a buffer address that the
    // hardware checks against the descriptor's size (the SGPR offset is not range-checked).
    auto dma_tile = [&](int t, int slot, bool is_v) {
      bool cur = false;
      uint32_t toff = kNoTile;
      uint32_t stride_b = L::ROWB;
      if (t >= t_end) toff = kNoTile;
      else if (t < nt0) toff = uint32_t(t * kKT) * L::ROWB;
      else if (t < nt0 + nt1) toff = uint32_t(sink + (t - nt0) * kKT) * L::ROWB;
      else { cur = true; stride_b = cur_stride_b; toff = uint32_t((t - nt0 - nt1) * kKT) * cur_stride_b; }
      unsigned char *dst = is_v ? lds_v + slot * L::VTILE : lds_k + slot * L::KTILE;
      const int gs = is_v ? L::VGS : L::KGS;
#pragma unroll
      for (int i = 0; i < GPW; ++i) {
        const int g = wave + kWaves * i;
        lds_void *d = (lds_void *)(dst + g * gs);
        const int vo = int(toff + uint32_t(g) * stride_b + uint32_t(cur ? voff_cur : voff_hist));
        if (cur) __builtin_amdgcn_raw_ptr_buffer_load_lds(as_buffer(is_v ? rs_vc : rs_kc), d, 16, vo, 0, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(as_buffer(is_v ? rs_vh : rs_kh), d, 16, vo, 0, 0, 0);
      }
    };

    // ---- Q: the wave's 32 rows go into LDS first, whole rows side by side, 1 KB a load.  (In the order of the fragments a load touches 16
    // rows, four 64-byte parts of each: the eight of a wave took the address unit four times as long as whole rows do.  Direct ->
    // through LDS, one box: 1170 queries 34.6 -> 32.2 us, 698 queries 24.2 -> 22.4, 832x480 0.6 % less.)
    const unsigned q_lds = lds_address(q_area<D, SCORE_ONLY>(lds_k, lds_v, lds_q, wave));
    if (wave_live) {
      constexpr int kChunks = L::ROWB / 16;
      const int lane_row = lane / kChunks, lane_chunk = lane % kChunks;
      const u16 *row = p.q + q0 * p.q_st + h * p.q_sh, *last = row + (p.Nq - 1 - q0) * p.q_st;
      row += lane_row * p.q_st;
      const int64_t step = L::RPG * p.q_st;
#pragma unroll
      for (int i = 0; i < 32 / L::RPG; ++i, row += step) {
        const u16 *src = row < last ? row : last;  // tail rows re-read the last query; never stored
        src += 8 * (lane_chunk ^ L::q_swizzle(i * L::RPG + lane_row));
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                         (lds_void *)(uintptr_t)(q_lds + 1024 * i), 16, 0, 0);
      }
    }

    // ---- piece prologue: the first three K tiles and first two V tiles go on their way into LDS in the order in
    // which they are read.  Only Q and the first K tile are waited for: the rest are what two VALU phases leave in
    // flight, so the waits of the tile loop cover them.  (All workgroups of a launch start here at once, and five
    // tiles and Q for each are 37 MB: waiting for all of it took 2.5 to 3.7 us a piece.)
    dma_tile(t_begin, 0, false);
    dma_tile(t_begin + 1, 1, false);
    if (!SCORE_ONLY) dma_tile(t_begin, 0, true);
    dma_tile(t_begin + 2, 2, false);
    if (!SCORE_ONLY) dma_tile(t_begin + 1, 1, true);
    // Q fragments: B operands of S^T = K Q^T.  Lane (j, g) holds, for queries j and 16 + j,
    // chunk (8 elements) first_chunk(g) + ks of every k-step.
    bf16x8 qf[KS][2];
    if (wave_live) {
      unsigned at[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) at[ks] = q_lds + j * L::ROWB + 16 * ((L::first_chunk(g) + ks) ^ L::q_swizzle(j));
      read_q<D, (SCORE_ONLY ? 3 : 5) * GPW>(at, qf);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kDmaPerPhase) : "memory");
    lds_barrier();

    // ---- the tiles.  One workgroup barrier per iteration, taken by group 1 before its VALU phase and by group 0 after
    // its: between two barriers group 0 runs MFMA(t), VALU(t) and group 1 runs VALU(t-1), MFMA(t), MFMA(t) being the
    // products S(t) = K(t) Q and O += V(t-1) P(t-1), so the two waves of a SIMD are in opposite phases without
    // being locked phase by phase.
    // Barrier n is the one group 0 takes after VALU(n) and group 1 before it, so behind barrier n both have finished MFMA(n),
    // and group 0 its VALU(n).
    // The loads of VALU phase t, K(t+3) and V(t+2), go where K(t-1) and V(t-2) were, which MFMA(t-1) reads last.  Behind
    // barrier t-1 every wave has finished that: group 0 issues the loads between barriers t-1 and t, group 1 behind barrier t.
    // They are first read in MFMA(t+3), which both groups run between barriers t+2 and t+3.  Before a barrier a wave waits for those of
    // its loads that the MFMA phases behind it read, here before barrier t+2: group 0 has by then issued the loads of phases up to t+2 and
    // may leave those of its latest two in flight, group 1, which issues phase t+2 behind that barrier, those of its latest one.  Either
    // way a load has about two iterations to land.  Every wave issues the same number of loads in every VALU phase (absent
    // tiles load zeros), so the counts hold.
    TileLoopArgs a;
    a.t_begin = t_begin; a.te = t_end;
    a.nt0 = nt0; a.nt1 = nt0 + nt1;
    a.sink = sink; a.win = len_h - sink; a.nc = p.Nc;
    a.cs = cur_stride_b;
    a.grp = group;
    a.ldsk = lds_address(lds_k) + wave * L::KGS; a.ldsv = lds_address(lds_v) + wave * L::VGS;
    a.c = p.c; a.lim = kSumLimit;
    // where the groups halve the keys, group 1 begins 32 rows into the tile: 32 / NG row positions on
    const unsigned half = HALF ? group * (kKT / 2 / L::NG * L::ROWB) : 0;
    a.ka = k_lane_addr + half; a.va = v_lane_addr + half;
    a.offh = lane_vo_hist; a.offc = lane_vo_cur;
    a.key0 = key_of_row(4 * g) + (HALF ? group * (kKT / 2) : 0);
    a.kh = rs_kh; a.kc = rs_kc; a.vh = rs_vh; a.vc = rs_vc;
    f32x4 o[DB][2];
    RowSums sums;
    if (wave_live) {
      if constexpr (HALF) half_tile_loop<D, SCORE_ONLY>(a, qf, o, sums);
      else tile_loop<D, SCORE_ONLY, true>(a, qf, o, sums);
    } else {
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        sums.neg_ref[qb] = INFINITY;
        sums.l[qb] = sums.l_sink[qb] = sums.l_hist[qb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      tile_loop<D, SCORE_ONLY, false>(a, qf, o, sums);
    }
    int s_first = span;                            // span that holds the unit's first tile
    unsigned long long next_flag = 0;
    if (take) {
      // The earlier pieces were written when their workgroups began their spans (a piece that fills a whole
      // span: when that workgroup ended), i.e. long ago or at about this time.  Wait until every flag says
      // its piece is in memory; the wait is bounded so that a workgroup that never runs cannot hang the
      // device: the unit's rows, and through them the head's scores, then come out as NaN.  The first wave looks as soon
      // as its own tiles are done: the other waves are up to half an iteration behind it.
      if (UNITS) s_first = s_unit;
      else do --s_first; while (s_first > 0 && span_begin(p, s_first) > unit_lo);
      if (PIECEWISE) {
        // Each wave waits for each piece on its own, before it folds it, and looks first while it still waits for its tiles.
        next_flag = __hip_atomic_load(p.flags + (span - 1) * p.team_size + member, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      } else if (wave == 0) {
        // one flag per lane: a poll is a round trip to memory, and a unit can have many pieces
        int ok = 1;
        for (int sp = s_first + lane; sp < span; sp += 64) {
          const int number = sp * p.team_size + member;
          ok &= take_flag(p, p.flags + number, number);
        }
        const int all_ok = __all(ok);              // the whole wave votes: inside `lane == 0` only that lane would
        if (lane == 0) lds_ok = all_ok;
      }
    }
    // no load of this piece may land in the next one's tiles, and no wave may still be reading them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    // What follows is worked out from here on: hoisted out of the loop over the pieces its addresses stood before a
    // workgroup's first load, and in registers (2 spilled at d = 128, none now).
    int tid_ = tid;
    asm volatile("" : "+v"(tid_));
    const int lane_ = tid_ & 63, g_ = lane_ >> 4, j_ = lane_ & 15;
    // ---- piece epilogue.  Region sums of this piece: a region that ended before the piece began contributes
    // nothing, a region the piece ends in (or before) contains everything the piece has summed.
    float ref_w[2], lt_w[2], l1_w[2], l2_w[2];     // reference; sums of all keys, the sink region, sink + window
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      ref_w[qb] = -sums.neg_ref[qb];
      lt_w[qb] = quad_sum(sums.l[qb]);
      l1_w[qb] = nt0 >= t_end ? lt_w[qb] : quad_sum(sums.l_sink[qb]);
      l2_w[qb] = nt0 + nt1 >= t_end ? lt_w[qb] : quad_sum(sums.l_hist[qb]);
    }
    // What the wave finishes: its two blocks, or, where the groups halve the keys, block `group` of its own and its partner's sums.
    float ref_h[1], lt_h[1], l1_h[1], l2_h[1];
    f32x4 out_h[DB][1];
    auto &ref_u = either<HALF>(ref_h, ref_w), &lt_u = either<HALF>(lt_h, lt_w);
    auto &l1_u = either<HALF>(l1_h, l1_w), &l2_u = either<HALF>(l2_h, l2_w);
    auto &out = either<HALF>(out_h, o);
    if constexpr (HALF) {
      const f32x4 theirs = exchange_halves<D, SCORE_ONLY>(
          reinterpret_cast<f32x4 *>(lds_k), reinterpret_cast<f32x4 *>(SCORE_ONLY ? lds_k + 4 * 1024 : lds_v), group, wave, lane_,
          group ? f32x4{ref_w[0], lt_w[0], l1_w[0], l2_w[0]} : f32x4{ref_w[1], lt_w[1], l1_w[1], l2_w[1]}, o, out);
      const float mine_ref = group ? ref_w[1] : ref_w[0];
      const float ref_new = fmaxf(theirs[0], mine_ref);
      const float w_t = theirs[0] == ref_new ? 1.f : fast_exp2(theirs[0] - ref_new);
      const float w_m = mine_ref == ref_new ? 1.f : fast_exp2(mine_ref - ref_new);
      ref_u[0] = ref_new;
      lt_u[0] = fold(theirs[1], w_t, group ? lt_w[1] : lt_w[0], w_m);
      l1_u[0] = fold(theirs[2], w_t, group ? l1_w[1] : l1_w[0], w_m);
      l2_u[0] = fold(theirs[3], w_t, group ? l2_w[1] : l2_w[0], w_m);
      if (!SCORE_ONLY) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int e = 0; e < 4; ++e) out[db][0][e] = fold(out[db][0][e], w_t, (group ? o[db][1] : o[db][0])[e], w_m);
      }
    }
    if (take) {
      float poison = PIECEWISE || lds_ok ? 0.f : NAN;
      // From this piece back to the unit's first, the order and arithmetic of the merge kernel: every earlier piece is
      // folded into this one's registers, all of it loaded with one wait.  (Front to back the sum so far needs
      // registers of its own, and the loads had to go out four at a time: 1170 queries, 6 pieces to a unit, 54.8 us
      // against 47.1.)
      auto slot_of_piece = [&](int sp) { return slot_index(p, sp, !UNITS && unit_lo > span_begin(p, sp) ? 1 : 0, member); };
      auto slot_of = [&](int sp) {
        return p.slots + slot_of_piece(sp) * Slot<D, NQB>::kFloats;
      };
      auto fold_sums = [&](int qb, const f32x4 &st, float &w_h, float &w_t) {
        const float ref_new = fmaxf(st[0], ref_u[qb]);
        w_h = (st[0] == ref_new) ? 1.f : fast_exp2(st[0] - ref_new);
        w_t = (ref_u[qb] == ref_new) ? 1.f : fast_exp2(ref_u[qb] - ref_new);
        ref_u[qb] = ref_new;
        lt_u[qb] = fold(st[1], w_h, lt_u[qb], w_t);
        l1_u[qb] = fold(st[2], w_h, l1_u[qb], w_t);
        l2_u[qb] = fold(st[3], w_h, l2_u[qb], w_t);
      };
      if constexpr (SCORE_ONLY) {
        // four pieces a trip (past the unit's first piece that one again, not looked at): 2.8 -> 1.2 us for 832x480
        // sampled scores, whose units are cut four times
#pragma unroll 1
        for (int sp = span - 1; sp >= s_first; sp -= 4) {
          f32x4 st[4][2];
          load_stats_through(slot_of(sp), slot_of(max(sp - 1, s_first)), slot_of(max(sp - 2, s_first)),
                             slot_of(max(sp - 3, s_first)), Slot<D>::stats_reader(tid_, 0), st);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (sp - i >= s_first) {
              float w_h, w_t;
              fold_sums(0, st[i][0], w_h, w_t);
              if (NQB == 2) fold_sums(NQB - 1, st[i][1], w_h, w_t);
            }
        }
      } else {
#pragma unroll 1
        for (int sp = span - 1; sp >= s_first; --sp) {
          f32x4 st[2], v[DB * NQB];
          if constexpr (PIECEWISE) {
            const int number = sp * p.team_size + member;
            unsigned long long *flag = p.flags + number;
            if (poison == 0.f && (next_flag != p.epoch || number == p.handoff - 2) && !await_flag(p, flag, number)) poison = NAN;
            // seen when these sums are in, and so for nothing if the piece is
            if (sp > s_first) next_flag = __hip_atomic_load(flag - p.team_size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
          if constexpr (HALF) load_half_slot<D>(p, slot_of_piece(sp), tid_, st[0], v);
          else load_slot_through<D / 8>(slot_of(sp), tid_, st, v);
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            float w_h, w_t;
            fold_sums(qb, st[qb], w_h, w_t);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
              for (int e = 0; e < 4; ++e) out[db][qb][e] = fold(v[NQB * db + qb][e], w_h, out[db][qb][e], w_t);
          }
        }
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) lt_u[qb] += poison;   // every result divides by it: rows, log-sum-exp, score sums
    }
    if (t_end == n_tiles && (t_begin == 0 || take)) {
      // the unit is complete
      const int row0 = first_row<NQB>(qt, wave);
      if (!SCORE_ONLY) {
        float inv[NQB];
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) inv[qb] = 1.f / lt_u[qb];
        store_output<D, NQB>(p, h, row0, lds_k + wave * (32 * 2 * D), lane_, out, inv);
        store_lse(p, h, row0, lane_, ref_u, lt_u);
      }
      if (p.part != nullptr) {
        float mass_a, mass_b;
        unit_masses(p, row0 + j_, lt_u, l1_u, l2_u, mass_a, mass_b);
        reduce_masses(p, lds_red, h, qt, tid_, mass_a, mass_b);
      }
      else if (!SCORE_ONLY) lds_barrier();         // the next piece's tiles go where the rows were
      if (PIECEWISE && take && wave == kWaves - 1)   // every wave has seen all flags
        for (int sp = s_first + lane; sp < span; sp += 64) reset_flag(p.flags + sp * p.team_size + member);
    } else {
      // a piece that starts at the span's first position uses the span's slot 0, a later one slot 1
      float *slot = p.slots + slot_index(p, span, piece_pos == span_lo ? 0 : 1, member) * Slot<D, NQB>::kFloats;
      store4_through(Slot<D, NQB>::stats(slot, tid_),
                     f32x4{of_block(g_, ref_u), of_block(g_, lt_u), of_block(g_, l1_u), of_block(g_, l2_u)});
      if (!SCORE_ONLY) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) store4_through(Slot<D, NQB>::ovec(slot, tid_, NQB * db + qb), out[db][qb]);
      }
      if (give) {
        // each thread's stores are in memory when its counter reaches zero; after the barrier all are
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
          __hip_atomic_store(p.flags + span * p.team_size + member, p.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
  if (p.done != nullptr) {
    if (wave == 0) {                               // the wave that wrote the units' sums: they are in memory, then the flag
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) __hip_atomic_store(p.done + span * p.team_size + member, p.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (span == 0 && member == 0) finish_all_scores<kNBuf * L::KTILE / 8>(p, reinterpret_cast<float2 *>(lds_k), &lds_ok, tid);
  }
}

// Second kernel.  Workgroup (k, member; db) looks at the boundary between spans k-1 and k: if it falls
// inside a head (not on its first column), the unit (group, head, member's query tile) was cut there
// and is put together from the partial results of its pieces, last to first, with the usual
// log-sum-exp weights; a unit cut by several boundaries is handled at the first of them.  blockIdx.y
// = db selects 32 of the D output columns, so that a unit is spread over D/32 workgroups (the kernel
// is a pure data mover and wants many loads in flight).  When scores are wanted, the db = 0 workgroup
// that completes the last unit of a head (counted per head) sums the head's per-tile masses in tile
// order; heads that were not cut anywhere get a workgroup of their own for that
// (blockIdx.x >= (n_teams - 1) * team_size).
template <int D, bool SCORE_ONLY, bool UNITS, bool HALF>
__global__ __launch_bounds__(kThreads) void df_attn_merge_kernel(const AttnParams p) {
  constexpr int NQB = HALF ? 1 : 2;
  __shared__ float lds_red[kWaves * 2];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, j = lane & 15;
  const int dq = int(blockIdx.y);                  // quarter (half at d = 64) of the output columns
  const int n_merge = (p.n_teams - 1) * p.team_size;
  if (int(blockIdx.x) >= n_merge) {                // score of a head no boundary cuts
    const int h = int(blockIdx.x) - n_merge;
    if (dq == 0 && tid == 0 && p.n_cut_units[h] == 0) finish_score(p, h);
    return;
  }
  const int k = int(blockIdx.x) / p.team_size + 1, member = int(blockIdx.x) % p.team_size;
  int h, qt, s_lo, s_hi;                           // head, query tile, spans that hold the unit's first and last column
  int64_t u_lo = 0;
  if constexpr (UNITS) {
    int hh = 0, first = 0;
    for (int end = int(p.rec[0].cut & 0xffffu); k >= end; end = int(p.rec[hh].cut & 0xffffu)) { first = end; ++hh; }
    if (k != first + 1) return;                    // not the first boundary inside a unit
    h = p.rec[hh].head;
    qt = member;
    s_lo = first;
    s_hi = int(p.rec[hh].cut & 0xffffu) - 1;
  } else {
    const int64_t cut = span_begin(p, k);
    const int grp = int(cut / p.total_cols);
    const int col = int(cut - int64_t(grp) * p.total_cols);
    const int hh = head_of_column(p, col);
    if (col == p.cum[hh]) return;                  // the boundary coincides with the head's first column
    u_lo = int64_t(grp) * p.total_cols + p.cum[hh];
    const int64_t u_hi = u_lo + (p.cum[hh + 1] - p.cum[hh]);
    if (k >= 2 && span_begin(p, k - 1) > u_lo) return;   // an earlier boundary cuts the same unit
    qt = grp * p.team_size + member;
    if (qt >= p.n_qtiles) return;
    h = p.rec[hh].head;
    s_lo = k - 1;
    s_hi = k;
    while (span_begin(p, s_hi + 1) < u_hi) ++s_hi;
  }

  float M[NQB], Lt[NQB] = {}, La[NQB] = {}, Lb[NQB] = {};
  f32x4 o[2][NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    M[qb] = -INFINITY;
    o[0][qb] = o[1][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll 1
  for (int sp = s_hi; sp >= s_lo; --sp) {          // last piece first, as in the main kernel
    float *slot = p.slots + slot_index(p, sp, !UNITS && u_lo > span_begin(p, sp) ? 1 : 0, member) * Slot<D, NQB>::kFloats;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const f32x4 st = *reinterpret_cast<const f32x4 *>(Slot<D, NQB>::stats(slot, Slot<D, NQB>::stats_reader(tid, qb)));
      const float m_new = fmaxf(st[0], M[qb]);
      // a piece of a wave that computes nothing (rows past the last query) has a reference of -inf throughout
      const float w_h = (st[0] == m_new) ? 1.f : fast_exp2(st[0] - m_new);
      const float w_t = (M[qb] == m_new) ? 1.f : fast_exp2(M[qb] - m_new);
      M[qb] = m_new;
      Lt[qb] = fold(st[1], w_h, Lt[qb], w_t);
      La[qb] = fold(st[2], w_h, La[qb], w_t);
      Lb[qb] = fold(st[3], w_h, Lb[qb], w_t);
      if (!SCORE_ONLY) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(Slot<D, NQB>::ovec(slot, tid, NQB * (2 * dq + i) + qb));
#pragma unroll
          for (int e = 0; e < 4; ++e) o[i][qb][e] = fold(v[e], w_h, o[i][qb][e], w_t);
        }
      }
    }
  }
  const int row0 = first_row<NQB>(qt, wave);
  if (!SCORE_ONLY) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (row0 + 16 * qb + j < p.Nq)
          *reinterpret_cast<uint2 *>(p.out + (row0 + 16 * qb + j) * p.o_st + h * p.o_sh + 32 * dq + 16 * i +
                                     4 * (lane >> 4)) = output4(o[i][qb], 1.f / Lt[qb]);
    if (dq == 0) store_lse(p, h, row0, lane, M, Lt);
  }
  if (dq == 0 && p.part != nullptr) {
    float mass_a, mass_b;
    unit_masses(p, row0 + j, Lt, La, Lb, mass_a, mass_b);
    reduce_masses(p, lds_red, h, qt, tid, mass_a, mass_b);
    // the unit's masses are out; whoever completes the head's last merged unit sums the head
    if (tid == 0) {
      __threadfence();
      const int done = __hip_atomic_fetch_add(p.tickets + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (done == p.n_cut_units[h] - 1) {
        __threadfence();
        finish_score(p, h);
      }
    }
  }
}

constexpr int64_t kMaxBufferBytes = 0x7ff00000;   // one head's rows must stay below the "no tile" offset
constexpr int kMinQTile = 128;   // smallest query tile any kernel variant uses (sizes the workspace)

// Workspace layout: [score partials: H * ceil(Nq/128) * 4 floats, rounded up to 256 B]
//                   [unit counters of the merge kernel: 256 B]
//                   [hand-over flags: one 8-byte word per workgroup]
//                   [partial-result slots: 2 per workgroup, kNumCU workgroups at most; the flags of the score sums, one
//                    8-byte word per workgroup, lie in the last span's slot for later pieces, which stays empty]
static size_t part_bytes(int H, int Nq) {
  const size_t tiles = (size_t(Nq) + kMinQTile - 1) / kMinQTile;
  return ((size_t(H) * tiles * 4 * sizeof(float) + 255) / 256) * 256;
}
constexpr size_t kTicketBytes = 256;
static_assert(kMaxHeads * sizeof(int32_t) <= kTicketBytes, "one counter per head");
static size_t slot_bytes(int d) {
  return size_t(d == 128 ? Slot<128>::kFloats : Slot<64>::kFloats) * sizeof(float);
}
constexpr size_t kFlagBytes = kNumCU * sizeof(unsigned long long);
static size_t workspace_bytes(int H, int d, int Nq) {
  return part_bytes(H, Nq) + kTicketBytes + kFlagBytes + 2 * size_t(kNumCU) * slot_bytes(d);
}

// Spans for a launch that cannot give every compute unit a long one.  There, what a piece costs besides its tiles
// decides: a workgroup that holds the end of one unit and the start of the next pays for two, and every
// earlier piece of a unit is another trip to memory for the workgroup that finishes it.  span_cost is the time of
// the slowest workgroup, counted in tile iterations: a piece's start and end, leaving its sums behind, and the flags and sums
// of earlier pieces; kSpanCost is what each span more slows all of them.  The five numbers are fitted to up to 50
// numbers of spans measured on each of 193 launches (64 to 8 000 queries, 1 to 40 heads, spans of 4 to 63 tiles, d = 64 and
// 128, attention and scores): above the best number measured the launches take 1.1 % on average, where all spans that a device
// holds (and for short ones the numbers that stamps inside the kernel had given) take 2.6 %.  Of 302 other launches (one query to 3 000,
// 2 to 64 heads, 0.3 to 150 GFLOP) 216 get another number than all spans and take 7.5 % less on average, from 31 % less to 10 %
// more.  d = 64 and scoring use the same numbers.  Choosing the spans (not planning by units: see cheapest_units) takes the host 1.6 us on average and 6 at most (3 000 launches of
// 2 to 64 heads, 64 to 2048 tokens a frame, a 2.7 GHz Xeon; walked span by span and without kMaxWalk 3.5 and 16; 64 heads of a few
// tiles each 7 against 42).
constexpr float kPieceCost = 2.9f, kGiveCost = 0.7f, kPollCost = 2.6f, kFoldCost = 0.9f, kSpanCost = 0.00024f;
constexpr float kSurelyCheaper = 0.92f;
constexpr int kMaxWalk = 1024;
// The walk goes from unit to unit (the spans that lie inside one differ by a tile at most) and ends with infinity where the cost
// reaches `limit`.
static float span_cost(const AttnParams &p, int n, float limit, int &units_walked) {
  const int line = int(p.line_len), base = line / n, rem = line % n;
  const uint32_t by_n = reciprocal_of(n);
  const uint64_t by_line = (uint64_t(1) << 40) / unsigned(line) + 1;   // of numbers below 2^22: line * n
  auto begin_of = [&](int span) { return span * base + divide_small(unsigned(span * rem), by_n); };
  float worst = 0.f, ready = 0.f;          // ready: when the last of the current unit's pieces so far is in memory
  float t = 0.f, fold = 0.f;               // the current span: time of its pieces so far; of the earlier pieces it collects
  bool takes = false;                      // ... if it does
  int span = 0, hi = begin_of(1);          // the current span and its end
  auto end_span = [&] {
    worst = std::max(worst, takes ? std::max(t, ready) + fold : t);
    t = 0.f;
    takes = false;
  };
  for (int group = 0; group < line; group += p.total_cols)
    for (int hh = 0; hh < p.H; ++hh) {
      const int lo = group + p.cum[hh], end = group + p.cum[hh + 1];
      ++units_walked;
      if (end > hi) {                        // handed on: the first thing the workgroup does
        const float give_at = kPieceCost + float(hi - lo) + kGiveCost;
        t += kPieceCost + float(hi - lo);
        t += kGiveCost;
        end_span();
        // the spans that the unit fills (`inside` of them, positions hi .. last), and the one that holds its end
        const int last_span = int((uint64_t(unsigned(end) * unsigned(n) - 1u) * by_line) >> 40), inside = last_span - span - 1;
        const int last = begin_of(last_span);
        ready = give_at;
        if (inside > 0) {
          const float filled = kPieceCost + float(base + (last - hi > inside * base)) + kGiveCost;
          worst = std::max(worst, filled);
          ready = std::max(ready, filled);
        }
        if (worst >= limit) return INFINITY;
        span = last_span;
        hi = begin_of(span + 1);
        takes = true;
        fold = kPollCost + kFoldCost * float(inside + 1);
        t = kPieceCost + float(end - last);
      } else {
        t += kPieceCost + float(end - lo);
      }
      if (end == hi) {
        end_span();
        if (worst >= limit) return INFINITY;
        hi = begin_of(++span + 1);
      }
    }
  return worst < limit ? worst : INFINITY;
}
// The cheapest number of spans up to n_max.  A few first, so that the walks of the others give up early; the largest that cut the
// units of equally long heads into equal parts; then every number down to those whose spans alone cost more (every second, third, ... of
// more than 90) until kMaxWalk units have been walked.  Numbers that must be dearer than the best are not walked.
static int cheapest_spans(const AttnParams &p, int n_max) {
  const int line = int(p.line_len), units = p.H * p.n_groups;
  int best = n_max, walked = 0;
  float best_cost = INFINITY;
  auto consider = [&](int n, float share = 1.f) {
    const float slower = 1.f + kSpanCost * float(n), limit = share * best_cost;
    const int span = line / n, longest = span + 1, n_before = (p.cum[1] - 1) / longest;
    // no less than this where the longest unit fills a span and lies in two more
    if (n_before > 1 && slower * (float(span) + kPieceCost + kGiveCost + kPollCost + kFoldCost * float(n_before)) > limit) return;
    const float c = slower * span_cost(p, n, limit / slower, walked);
    if (c < limit) { best_cost = c; best = n; }
  };
  for (int eighths = 8; eighths >= 4; --eighths) consider(std::max(1, n_max * eighths / 8));
  for (int n = n_max / units * units, i = 0; n >= 1 && i < 8; n -= units, ++i) consider(n);
  const int step = std::max(1, n_max * n_max / 8192);
  for (int n = n_max - 1; n >= 1 && float(line) / float(n) < best_cost && walked < kMaxWalk; n -= step) consider(n);
  // The fewest spans that are one to six tiles longer, which a step may have passed over: spans of even length cost less than their
  // neighbours.  They have to be cheaper by more than the cost is wrong by.  92 launches that take one of them: 9 % less on
  // average, from 16 % less to 6 % more.
  for (int longer : {1, 2, 4, 6}) consider(std::max(1, line / (line / n_max + longer)), kSurelyCheaper);
  return best;
}

static void set_spans(AttnParams &p, int n_teams) {
  p.n_teams = n_teams;
  p.span_base = p.line_len / p.n_teams;
  p.span_rem = int32_t(p.line_len % p.n_teams);
  p.by_n_teams = reciprocal_of(p.n_teams);
  p.by_team_size = reciprocal_of(p.team_size);
}

// The decomposition of a launch (A4).  Columns = key tiles of all heads, longest head first.  Query tiles
// are taken in groups of `team_size`; the line has one position per (group, column) and is cut into
// equal spans, one per team.  A team has one workgroup per query tile of a group; its members walk the
// same columns at the same time.  team_size is chosen so that as many of the kNumCU workgroups as
// possible have a query tile in every group: when the number of query tiles does not divide the
// number of compute units, smaller teams (more groups) fill the machine better than one team member per
// query tile.
static df_status plan(AttnParams &p, float *spans_cost) {
  p.n_qtiles = (p.Nq + kBQ - 1) / kBQ;
  int64_t total = 0;
  for (int hh = 0; hh < p.H; ++hh) {
    const int64_t len = p.rec[hh].len;
    const int64_t sink = p.rec[hh].sink;
    p.cum[hh] = int32_t(total);
    total += (sink + kKT - 1) / kKT + (len - sink + kKT - 1) / kKT + (p.Nc + kKT - 1) / kKT;
    if (total > INT32_MAX / 2) return DF_ERR_RANGE;
  }
  p.cum[p.H] = int32_t(total);
  p.total_cols = int32_t(total);
  // busy share of the machine for a team size s: workgroups launched x tiles present in the average group
  auto teams_of = [&](int s) {
    const int64_t groups = (p.n_qtiles + s - 1) / s;
    return int64_t(std::max<int64_t>(1, std::min<int64_t>(kNumCU / s, groups * total / kMinSpan)));
  };
  auto busy = [&](int s) {
    const int64_t groups = (p.n_qtiles + s - 1) / s;
    return double(teams_of(s) * s) / kNumCU * double(p.n_qtiles) / double(groups * s);
  };
  const int s_max = std::min(p.n_qtiles, kNumCU);
  double best = 0.0;
  for (int s = 1; s <= s_max; ++s) best = std::max(best, busy(s));
  // Larger teams share every K/V tile among more workgroups while it is hot in L2, so the largest team
  // that keeps 95 % of the machine busy (or the best there is) wins.
  const double want = std::min(best, 0.95);
  int team = s_max;
  while (team > 1 && busy(team) < want) --team;
  p.team_size = team;
  p.n_groups = (p.n_qtiles + team - 1) / team;
  p.line_len = int64_t(p.n_groups) * total;
  p.n_teams = int32_t(teams_of(team));
  // Where all the spans that the machine holds are shorter than kMaxCostSpan tiles their number is chosen by their cost (longer
  // ones lose more by idle compute units than the cut saves: of 19 launches of 66 to 450 tiles a span one gains 1.8 %).
  // All spans -> chosen, us: 1170 sampled queries 56.6 -> 55.0, 825 queries 107.7 -> 98.8, 1104 of two heads 54.3 -> 47.9, 98
  // sampled ones of 24 heads 21.4 -> 18.9.
  if (p.line_len < int64_t(kMaxCostSpan) * (kNumCU / team))
    p.n_teams = cheapest_spans(p, std::max(1, std::min(kNumCU / team, int(p.line_len) / kMinSmallSpan)));
  set_spans(p, p.n_teams);
  if (spans_cost) {
    int walked = 0;
    *spans_cost = p.line_len < int64_t(kMaxCostSpan) * (kNumCU / team)
                      ? (1.f + kSpanCost * float(p.n_teams)) * span_cost(p, p.n_teams, INFINITY, walked) : 0.f;
  }
  return DF_OK;
}

// Share of the spans' time `us` that units may take: less of longer launches, in which the clock under load and not these sums decides
// and equal spans keep all compute units busy to the end; none from kMaxUnitLaunch on.  Scoring, which the issue of instructions bounds, has
// nothing to gain there either: 1170 sampled queries of 12 heads, 8 cached frames (spans of 64 tiles) 65.8 us in spans and 65.1 by units, 12 85.1 and
// 84.3, 21 (139 tiles) 128.8 and 128.1, 32 181.9 and 183.3.
constexpr float kMaxUnitLaunch = 110.f;
static float units_margin(float us) { return us > kMaxUnitLaunch ? 0.f : 0.97f - 0.002f * std::max(0.f, us - 50.f); }
constexpr int kMaxTiles = 0xffff;      // of a unit, for HeadRec::cut

// Heads whose units have the same number of tiles, longest first (heads are sorted by keys: a ragged sink region can make a unit a tile
// longer than the one before).
struct Runs {
  struct { int n, heads; } run[kMaxHeads];
  int n_runs = 0, heads, first_n;        // first_n: tiles of a unit of the head with the most keys
  explicit Runs(const AttnParams &p) : heads(p.H), first_n(p.cum[1]) {
    for (int hh = 0; hh < p.H; ++hh) {
      const int n = p.cum[hh + 1] - p.cum[hh];
      int r = n_runs;
      while (r > 0 && run[r - 1].n < n) --r;
      if (r > 0 && run[r - 1].n == n) {
        ++run[r - 1].heads;
        continue;
      }
      std::copy_backward(run + r, run + n_runs, run + n_runs + 1);
      run[r] = {n, 1};
      ++n_runs;
    }
  }
};
// Tiles of the shortest piece but the last of `count` > 1 that a unit of `n` is cut into (less than one: there are too many).
static int piece_length(int n, int count, const UnitCost &cost) {
  return (n - cost.ahead - UnitPieces{count, 0, cost.lag}.begin(count - 1) + count - 1) / count;
}
// The fewest pieces of a unit of `n` tiles, the shortest but the last of at most `longest`; none if the last would be empty.
// (`from`: a number that is known to be too few or just right.)
static UnitPieces pieces(int n, int longest, const UnitCost &cost, int from = 1) {
  UnitPieces u{from, longest, cost.lag};
  while (u.count <= kNumCU && u.begin(u.count - 1) + longest + cost.ahead < n) ++u.count;
  u.length = u.count == 1 ? std::max(1, n - cost.ahead) : piece_length(n, u.count, cost);
  if (u.count > kNumCU || (u.count > 1 && (u.length < 1 || u.begin(u.count - 1) >= n))) u.count = 0;
  return u;
}
// Most tiles of a piece of the cheapest cut into units of `rows` queries, if that costs less than `best` (which it then replaces), else 0.
// From whole units on, each time with the longest pieces with which the unit that was the slowest can be part of a cheaper cut: what lies in
// between leaves it too slow.  Of the units that are whole only the longest can be the slowest.  Whole units are those of the head with the
// most keys: where others are a tile longer, to leave these whole too is a little cheaper by the model but takes 3 to 5 % longer in launches of
// few tiles (58 queries and 40 heads 14.1 -> 15.7 us; 14 launches of one or two lengths 1.02 on average while attending).
// Walked so, planning by units takes the host 0.8 us with heads of one length, 2.2 with 12 and 5.9 with 64 on average (3, 7 and 17 at most) besides
// the 1.5 to 2.5 for the spans (400 launches each, a 2.7 GHz Xeon); with all heads walked for each length of piece, 3 % apart, and given up after 512
// of them it took 2.1, 16 and 17 (14, 41 and 40), and where heads have 20 to 64 lengths the cuts that it found took 13 to 29 % more time.
static int cheapest_units(const Runs &runs, int Nq, int rows, const UnitCost &cost, float &best) {
  const int m = (Nq + rows - 1) / rows, most = kNumCU / m;
  struct { int count, length; float fold; } cut[kMaxHeads];      // of the first n_cut runs; the others are whole
  int best_longest = 0, n_cut = 0, spans = runs.heads;
  for (int longest = std::max(1, runs.first_n - cost.ahead);;) {
    for (; n_cut < runs.n_runs && runs.run[n_cut].n - cost.ahead > longest; ++n_cut) cut[n_cut] = {1, INT32_MAX, 0.f};
    for (int r = 0; r < n_cut; ++r)
      if (cut[r].length > longest) {
        const UnitPieces u = pieces(runs.run[r].n, longest, cost, cut[r].count);
        if (u.count == 0) return best_longest;
        spans += (u.count - cut[r].count) * runs.run[r].heads;
        cut[r] = {u.count, u.length, cost.cut + cost.fold * float(u.count - 1)};
      }
    if (spans > most) return best_longest;
    const float tile = cost.tile * (1.f + cost.crowd * float(spans * m)) * (2 * Nq <= rows ? cost.few : 1.f);
    const float others = cost.start + cost.wg * float(spans * m);
    int slowest = n_cut;                                         // a run that is cut, or the first one that is not
    float t = n_cut < runs.n_runs ? tile * float(runs.run[n_cut].n) : 0.f;
    for (int r = 0; r < n_cut; ++r) {
      const float t_r = tile * float(cut[r].length) + cut[r].fold;
      if (t_r > t) { t = t_r; slowest = r; }
    }
    if (others + t < best) { best = others + t; best_longest = longest; }
    // the fewest pieces with which that unit alone would leave a cheaper cut possible, and the longest pieces that take as many
    int count = slowest < n_cut ? cut[slowest].count : 1;
    int length = slowest < n_cut ? cut[slowest].length : runs.run[slowest].n - cost.ahead;
    for (float t_slowest = INFINITY; others + t_slowest >= best;) {
      longest = length - 1;
      const float fold = cost.cut + cost.fold * float(count++);
      length = piece_length(runs.run[slowest].n, count, cost);
      if (length < 1 || others + tile + fold >= best) return best_longest;
      t_slowest = tile * float(length) + fold;
    }
  }
}
// Cuts the launch into units of `rows` queries, in pieces of at most `longest` tiles.
static void cut_units(AttnParams &p, int rows, int longest, const UnitCost &cost) {
  int spans = 0;
  for (int hh = 0; hh < p.H; ++hh) {
    const UnitPieces u = pieces(p.cum[hh + 1] - p.cum[hh], longest, cost);
    spans += u.count;
    p.rec[hh].cut = uint32_t(spans) | uint32_t(u.length) << 16;
  }
  p.n_qtiles = p.team_size = (p.Nq + rows - 1) / rows;
  p.n_groups = 1;
  p.line_len = p.total_cols;
  set_spans(p, spans);
}
// For tests of each way to cut a launch at sizes where another would be chosen: DF_ATTN_CUT=spans, 128 or 256 in the environment (looked
// at on every call) cuts into spans, or by units of so many queries where the machine holds them.  0, the queries, or -1: what costs least.
static int forced_cut() {
  const char *e = std::getenv("DF_ATTN_CUT");
  if (!e) return -1;
  return !std::strcmp(e, "spans") ? 0 : !std::strcmp(e, "128") ? kHalfBQ : !std::strcmp(e, "256") ? kBQ : -1;
}
// The plan by units if it costs less than the spans do (`spans_cost` as plan gives it, 0: not known): rows of its units, or 0.
static int plan_units(AttnParams &p, const LaunchCost &cost, float spans_cost) {
  const int forced = forced_cut();
  if (forced == 0 || p.cum[1] > kMaxTiles) return 0;
  if (forced > 0) {
    const UnitCost &unit = forced == kBQ ? cost.whole : cost.half;
    float any = INFINITY;
    const int longest = cheapest_units(Runs(p), p.Nq, forced, unit, any);
    if (longest) cut_units(p, forced, longest, unit);
    return longest ? forced : 0;
  }
  if (spans_cost <= 0.f) return 0;
  const float in_spans = cost.spans.start + cost.spans.cost * spans_cost + cost.spans.tile * float(p.span_base) +
                         cost.spans.wg * float(p.n_teams * p.team_size);
  float best = units_margin(in_spans) * in_spans;
  if (best <= 0.f) return 0;
  const Runs runs(p);
  const int half = cheapest_units(runs, p.Nq, kHalfBQ, cost.half, best), whole = cheapest_units(runs, p.Nq, kBQ, cost.whole, best);
  const int rows = whole ? kBQ : half ? kHalfBQ : 0;
  if (rows) cut_units(p, rows, whole ? whole : half, whole ? cost.whole : cost.half);
  return rows;
}

// The units of each head that span boundaries cut (the same walk as the merge kernel's), for df_attn_plan and for the
// two-kernel path; a launch that puts its units together itself has no use for them.
static void count_cut_units(AttnParams &p, bool by_units = false) {
  if (by_units) {
    for (int hh = 0, first = 0; hh < p.H; ++hh) {
      const int end = int(p.rec[hh].cut & 0xffffu);
      if (end - first > 1) p.n_cut_units[p.rec[hh].head] = int16_t(p.n_qtiles);
      first = end;
    }
    return;
  }
  for (int k = 1; k < p.n_teams; ++k) {
    const int64_t cut = span_begin(p, k);
    const int grp = int(cut / p.total_cols);
    const int col = int(cut - int64_t(grp) * p.total_cols);
    const int hh = head_of_column(p, col);
    if (col == p.cum[hh]) continue;
    const int64_t u_lo = int64_t(grp) * p.total_cols + p.cum[hh];
    if (k >= 2 && span_begin(p, k - 1) > u_lo) continue;
    p.n_cut_units[p.rec[hh].head] += std::min(p.team_size, p.n_qtiles - grp * p.team_size);
  }
}

// Whether the workgroups of a launch can hand partial results and score sums to each other while it runs: every one of
// them must be on the device at the same time, i.e. the device must have a compute unit for each (one
// workgroup fills a compute unit's LDS).  DF_ATTN_HANDOVER=0 in the environment selects the two-kernel
// path regardless (a process whose queues are restricted to a subset of the compute units needs it).
static bool handover_possible(int n_wg) {
  const char *e = std::getenv("DF_ATTN_HANDOVER");   // looked at on every call
  if (e && e[0] == '0') return false;
  static std::mutex mu;
  static int cus[64] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return false;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      n = -1;
    }
    cus[dev] = n > 0 ? n : -1;
  }
  return cus[dev] >= n_wg;
}

// For tests of what a call returns when one of its workgroups never runs: DF_ATTN_LOST_FLAG=n in the environment
// (looked at on every call) lets the reader of flag n give up on it at once, as it would after kSpinLimit polls.  The
// hand-over flags are numbered by workgroup (span * team_size + member; by units a head's pieces are as many spans, longest head
// first, and team_size is the number of query tiles), the flags of the score sums follow from kNumCU on.
static int lost_flag() {
  const char *e = std::getenv("DF_ATTN_LOST_FLAG");
  return e && *e ? std::clamp(std::atoi(e), -1, 2 * kNumCU) : -1;
}

// A flag value that neither stale workspace contents nor an earlier launch hold: a counter run through a
// 64-bit mixer, never zero.
static unsigned long long next_epoch() {
  static std::atomic<unsigned long long> counter{0x9e3779b97f4a7c15ull ^ (unsigned long long)(uintptr_t)&counter};
  unsigned long long z = counter.fetch_add(0x9e3779b97f4a7c15ull) + 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z ? z : 1ull;
}

template <int D, bool SCORE_ONLY, bool UNITS, bool HALF>
static df_status launch_planned(AttnParams &p, void *workspace, float *score_out, hipStream_t st) {
  using S = Slot<D, HALF ? 1 : 2>;
  // One team of several workgroups has no cut unit: it waits for nothing and needs no two compute units at a time.  Its
  // scores are left to the second kernel, so that this stays so: 16.5 against 15.7 us with 2 workgroups, 19.6 against
  // 18.5 with 8.  (A lone workgroup waits for its own flag only.)
  const int n_wg = p.n_teams * p.team_size;
  const bool together = (p.n_teams > 1 || (score_out && n_wg == 1)) && handover_possible(n_wg);
  if (together) {
    p.handoff = 2 + lost_flag();
    p.epoch = next_epoch();
  } else {
    count_cut_units(p, UNITS);
  }
  char *ws = static_cast<char *>(workspace);
  p.part = score_out ? reinterpret_cast<float *>(ws) : nullptr;
  p.tickets = score_out && !together ? reinterpret_cast<int32_t *>(ws + part_bytes(p.H, p.Nq)) : nullptr;
  p.flags = reinterpret_cast<unsigned long long *>(ws + part_bytes(p.H, p.Nq) + kTicketBytes);
  p.slots = reinterpret_cast<float *>(ws + part_bytes(p.H, p.Nq) + kTicketBytes + kFlagBytes);
  p.score = score_out;
  // The last span ends where the line does and hands nothing on, so the slots of its later pieces are free: the
  // flags of the score sums lie there.
  p.done = together && score_out
               ? reinterpret_cast<unsigned long long *>(p.slots + slot_index(p, p.n_teams - 1, 1, 0) * S::kFloats)
               : nullptr;
  const int grid = n_wg >= kXcd ? (n_wg + kXcd - 1) / kXcd * kXcd : n_wg;   // XCD-major numbering needs a multiple of 8
  hipLaunchKernelGGL((df_attn_kernel<D, SCORE_ONLY, UNITS, HALF>), dim3(grid), dim3(kThreads), 0, st, p);
  if (df_status s = launch_status()) return s;
  if (together) return DF_OK;
  // second launch: the units that span boundaries cut, and the per-head score sums
  const int n_merge = (p.n_teams - 1) * p.team_size + (score_out ? p.H : 0);
  if (n_merge > 0) {
    hipLaunchKernelGGL((df_attn_merge_kernel<D, SCORE_ONLY, UNITS, HALF>), dim3(n_merge, SCORE_ONLY ? 1 : D / 32),
                       dim3(kThreads), 0, st, p);
    if (df_status s = launch_status()) return s;
  }
  return DF_OK;
}

template <int D, bool SCORE_ONLY>
static df_status launch(AttnParams &p, void *workspace, float *score_out, hipStream_t st) {
  float spans_cost;
  if (df_status s = plan(p, &spans_cost)) return s;
  switch (plan_units(p, kLaunchCost<D, SCORE_ONLY>, spans_cost)) {
    case kHalfBQ: return launch_planned<D, SCORE_ONLY, true, true>(p, workspace, score_out, st);
    case kBQ: return launch_planned<D, SCORE_ONLY, true, false>(p, workspace, score_out, st);
    default: return launch_planned<D, SCORE_ONLY, false, false>(p, workspace, score_out, st);
  }
}

// The head table: longest history first, heads of equal length in their own order.
static void sort_heads(AttnParams &p, int H, const int64_t *off, const int32_t *len, const int32_t *sink) {
  int idx[kMaxHeads];
  std::iota(idx, idx + H, 0);
  std::stable_sort(idx, idx + H, [&](int a, int b) { return len[a] > len[b]; });
  for (int i = 0; i < H; ++i) {
    const int h = idx[i];
    p.rec[i] = HeadRec{off ? off[h] : 0, len[h], sink ? sink[h] : 0, h, 0};
  }
}

// Checks shared by both entry points; fills the per-head tables of `p`.
static df_status fill_heads(AttnParams &p, int H, int d, int Nq, int Nc, const int64_t *hist_off,
                            const int32_t *sink_len, const int32_t *hist_len, bool need_sink, const void *k_hist,
                            const void *v_hist, bool need_v) {
  if (H <= 0 || Nq <= 0 || Nc <= 0) return DF_ERR_SHAPE;
  if (H > kMaxHeads || (d != 64 && d != 128)) return DF_ERR_UNSUPPORTED;
  if (!hist_off) return DF_ERR_NULL;
  if (need_sink && !sink_len) return DF_ERR_NULL;
  if (hist_off[0] != 0) return DF_ERR_RANGE;
  int64_t any = 0;
  int32_t lens[kMaxHeads], sinks[kMaxHeads];
  for (int h = 0; h < H; ++h) {
    const int64_t rows = hist_off[h + 1] - hist_off[h];
    if (rows < 0 || rows * d * 2 >= kMaxBufferBytes) return DF_ERR_RANGE;
    const int64_t len = hist_len ? hist_len[h] : rows;
    if (len < 0 || len > rows) return DF_ERR_RANGE;
    const int32_t sl = sink_len ? sink_len[h] : 0;
    if (sl < 0 || sl > len) return DF_ERR_RANGE;
    lens[h] = int32_t(len);
    // Without scores nobody asks where the sink region ends, and its rows and the window's lie side by side: one region has up to one
    // ragged tile less than two (98 tokens a frame, one chunk of them, 5 heads of 1 + 21 frames: 18.9 -> 17.8 us).
    sinks[h] = need_sink ? sl : 0;
    any += len;
  }
  if (any > 0) {
    if (!k_hist || (need_v && !v_hist)) return DF_ERR_NULL;
    if (!aligned16(k_hist) || (need_v && !aligned16(v_hist))) return DF_ERR_ALIGN;
  }
  sort_heads(p, H, hist_off, lens, sinks);
  p.H = H;
  p.Nq = Nq;
  p.Nc = Nc;
  return DF_OK;
}

}  // namespace df

using namespace df;

extern "C" size_t df_attn_workspace_bytes(int32_t H, int32_t d, int32_t Nq) {
  if (H <= 0 || Nq <= 0 || (d != 64 && d != 128)) return 0;
  return workspace_bytes(H, d, Nq);
}

// The plan of a launch of which only sizes are given.
static df_status plan_of_sizes(AttnParams &p, int32_t H, int32_t Nq, int32_t Nc, const int32_t *hist_len, const int32_t *hist_sink_len,
                               float *spans_cost) {
  if (H <= 0 || Nq <= 0 || Nc <= 0) return DF_ERR_SHAPE;
  if (H > kMaxHeads) return DF_ERR_UNSUPPORTED;
  for (int h = 0; h < H; ++h) {
    const int32_t sl = hist_sink_len ? hist_sink_len[h] : 0;
    if (hist_len[h] < 0 || sl < 0 || sl > hist_len[h]) return DF_ERR_RANGE;
  }
  sort_heads(p, H, nullptr, hist_len, hist_sink_len);
  p.H = H;
  p.Nq = Nq;
  p.Nc = Nc;
  return plan(p, spans_cost);
}

extern "C" df_status df_attn_units(int32_t H, int32_t d, int32_t score_only, int32_t Nq, int32_t Nc, const int32_t *hist_len,
                                   const int32_t *hist_sink_len, int32_t *unit_rows, int32_t *pieces) {
  if (!hist_len || !unit_rows || !pieces) return DF_ERR_NULL;
  if (d != 64 && d != 128) return DF_ERR_UNSUPPORTED;
  AttnParams p{};
  float spans_cost;
  if (df_status s = plan_of_sizes(p, H, Nq, Nc, hist_len, hist_sink_len, &spans_cost)) return s;
  *unit_rows = plan_units(p, d == 128 ? (score_only ? kLaunchCost<128, true> : kLaunchCost<128, false>)
                                               : (score_only ? kLaunchCost<64, true> : kLaunchCost<64, false>), spans_cost);
  for (int hh = 0; hh < H; ++hh)
    pieces[p.rec[hh].head] = *unit_rows ? int32_t(p.rec[hh].cut & 0xffffu) - (hh ? int32_t(p.rec[hh - 1].cut & 0xffffu) : 0) : 0;
  return DF_OK;
}

extern "C" df_status df_attn_plan(int32_t H, int32_t Nq, int32_t Nc, const int32_t *hist_len,
                                  const int32_t *hist_sink_len, df_attn_plan_info *out) {
  if (!hist_len || !out) return DF_ERR_NULL;
  AttnParams p{};
  if (df_status s = plan_of_sizes(p, H, Nq, Nc, hist_len, hist_sink_len, nullptr)) return s;
  out->n_qtiles = p.n_qtiles;
  out->team_size = p.team_size;
  out->n_groups = p.n_groups;
  out->n_teams = p.n_teams;
  out->workgroups = p.n_teams * p.team_size;
  count_cut_units(p);
  out->cut_units = 0;
  for (int h = 0; h < H; ++h) out->cut_units += p.n_cut_units[h];
  out->total_cols = p.total_cols;
  out->line_len = p.line_len;
  out->span_min = INT64_MAX;
  out->span_max = 0;
  for (int t = 0; t < p.n_teams; ++t) {
    const int64_t len = span_begin(p, t + 1) - span_begin(p, t);
    out->span_min = std::min(out->span_min, len);
    out->span_max = std::max(out->span_max, len);
  }
  out->busy = double(out->workgroups) / kNumCU * double(p.n_qtiles) / double(int64_t(p.n_groups) * p.team_size);
  // Walk every span the way the kernel does and check what the hand-over relies on: the pieces of a span
  // tile it, the pieces of a unit are consecutive, lie in consecutive spans and cover the unit, and a span
  // holds at most one piece that leaves its sums for a later span and at most one that collects earlier ones.
  out->pieces = out->gives = out->takes = out->max_pieces_per_unit = 0;
  out->consistent = 1;
  int64_t expect_unit = -1;        // unit_lo of the unit whose next piece the walk must meet, or -1
  int expect_t = 0, unit_pieces = 0, first_span = 0;
  for (int span = 0; span < p.n_teams; ++span) {
    const int64_t lo = span_begin(p, span), hi = span_begin(p, span + 1);
    // the kernel walks from the end; collect, then check in line order
    std::vector<Piece> list;
    for (int64_t pos_end = hi; pos_end > lo;) {
      const Piece c = piece_ending_at(p, ColumnsInParams{p}, lo, pos_end);
      if (c.pos >= pos_end || c.pos < lo) { out->consistent = 0; break; }
      list.push_back(c);
      pos_end = c.pos;
    }
    const int n = int(list.size());
    int gives = 0, takes = 0;
    int64_t at = lo;
    for (int i = n - 1; i >= 0; --i) {
      const Piece &c = list[i];
      if (c.pos != at || c.t_begin < 0 || c.t_end > c.n_tiles || c.t_begin >= c.t_end) out->consistent = 0;
      at = c.pos + (c.t_end - c.t_begin);
      if (c.t_begin == 0) {
        if (expect_unit != -1) out->consistent = 0;          // the unit before was left unfinished
        unit_pieces = 0;
        first_span = span;
      } else if (expect_unit != c.unit_lo || expect_t != c.t_begin || i != n - 1) {
        out->consistent = 0;                                  // a continued unit is the first piece of its span
      }
      ++unit_pieces;
      if (c.t_end < c.n_tiles) {
        ++gives;
        expect_unit = c.unit_lo;
        expect_t = c.t_end;
        if (i != 0) out->consistent = 0;                      // an unfinished unit is the last piece of its span
      } else {
        expect_unit = -1;
        if (c.t_begin > 0) {
          ++takes;
          // the kernel finds the span of the unit's first piece by stepping back from its own
          int s_first = span - 1;
          while (s_first > 0 && span_begin(p, s_first) > c.unit_lo) --s_first;
          if (s_first != first_span || unit_pieces != span - first_span + 1) out->consistent = 0;
        }
        out->max_pieces_per_unit = std::max(out->max_pieces_per_unit, unit_pieces);
      }
    }
    if (at != hi || gives > 1 || takes > 1) out->consistent = 0;
    out->pieces += n;
    out->gives += gives;
    out->takes += takes;
  }
  if (expect_unit != -1) out->consistent = 0;
  return DF_OK;
}

// df_attn_fwd with the workspace given separately: the caller's (df_attn_fwd) or the library's static
// scratch (df_attn_fwd_static).
static df_status attn_fwd(const df_attn_args *a, void *stream, void *workspace, size_t workspace_size) {
  if (!a) return DF_ERR_NULL;
  if (!a->q || !a->k_cur || !a->v_cur || !a->out) return DF_ERR_NULL;
  AttnParams p{};
  if (df_status s = fill_heads(p, a->H, a->d, a->Nq, a->Nc, a->hist_off, a->hist_sink_len, a->hist_len,
                               a->score_out != nullptr, a->k_hist, a->v_hist, true))
    return s;
  if (!aligned16(a->q) || !aligned16(a->k_cur) || !aligned16(a->v_cur) || !aligned16(a->out))
    return DF_ERR_ALIGN;
  const bool multi = a->H > 1;
  if (!stride_ok(a->q_stride_tok) || !stride_ok(a->kc_stride_tok) || !stride_ok(a->o_stride_tok) ||
      (multi && (!stride_ok(a->q_stride_head) || !stride_ok(a->kc_stride_head) || !stride_ok(a->o_stride_head))))
    return DF_ERR_ALIGN;
  if (!(a->softmax_scale > 0.f) || !std::isfinite(a->softmax_scale)) return DF_ERR_RANGE;
  if (!workspace || workspace_size < workspace_bytes(a->H, a->d, a->Nq)) return DF_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return DF_ERR_ALIGN;
  p.q = static_cast<const u16 *>(a->q);
  p.k_cur = static_cast<const u16 *>(a->k_cur);
  p.v_cur = static_cast<const u16 *>(a->v_cur);
  p.k_hist = static_cast<const u16 *>(a->k_hist);
  p.v_hist = static_cast<const u16 *>(a->v_hist);
  p.out = static_cast<u16 *>(a->out);
  p.lse = a->lse_out;
  p.q_st = a->q_stride_tok; p.q_sh = a->q_stride_head;
  p.kc_st = a->kc_stride_tok; p.kc_sh = a->kc_stride_head;
  p.o_st = a->o_stride_tok; p.o_sh = a->o_stride_head;
  if ((int64_t(a->Nc - 1) * a->kc_stride_tok + a->d) * 2 >= kMaxBufferBytes || a->kc_stride_tok >= (1 << 24))
    return DF_ERR_RANGE;
  p.cur_bytes = uint32_t((int64_t(a->Nc - 1) * a->kc_stride_tok + a->d) * 2);
  p.c = a->softmax_scale * 1.4426950408889634f;
  p.lse_unit = float(double(a->softmax_scale) / double(p.c));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (a->d == 128) return launch<128, false>(p, workspace, a->score_out, st);
  return launch<64, false>(p, workspace, a->score_out, st);
}

extern "C" df_status df_attn_fwd(const df_attn_args *a, void *stream) {
  if (!a) return DF_ERR_NULL;
  return attn_fwd(a, stream, a->workspace, a->workspace_bytes);
}

// ---- df_attn_fwd_static: the same call for callers that cannot allocate (see df.h) -------------------
// The workspace is a file-scope device array.  Its name is only a host-side handle: the device address
// is looked up once per device and kept, and only that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[DF_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, or null if the runtime cannot provide it.
void *static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" df_status df_attn_fwd_static(const df_attn_args *a, void *stream) {
  if (!a) return DF_ERR_NULL;
  // sizes first: nothing else is looked at when the launch cannot fit the static scratch
  if (a->H <= 0 || a->Nq <= 0 || a->Nc <= 0) return DF_ERR_SHAPE;
  if (a->H > kMaxHeads || (a->d != 64 && a->d != 128)) return DF_ERR_UNSUPPORTED;
  if (workspace_bytes(a->H, a->d, a->Nq) > size_t(DF_STATIC_SCRATCH_BYTES)) return DF_ERR_WORKSPACE;
  void *ws = static_scratch();
  if (!ws) return DF_ERR_LAUNCH;
  return attn_fwd(a, stream, ws, size_t(DF_STATIC_SCRATCH_BYTES));
}

extern "C" df_status df_head_score(const df_score_args *a, void *stream) {
  if (!a) return DF_ERR_NULL;
  if (!a->q || !a->k_cur || !a->score_out) return DF_ERR_NULL;
  AttnParams p{};
  if (df_status s = fill_heads(p, a->H, a->d, a->Nq, a->Nc, a->hist_off, a->hist_sink_len, a->hist_len, true,
                               a->k_hist, nullptr, false))
    return s;
  if (a->q_sample_stride < 1 || a->q_offset < 0 || a->q_offset >= a->q_sample_stride || a->q_offset >= a->Nq)
    return DF_ERR_RANGE;
  if (!aligned16(a->q) || !aligned16(a->k_cur)) return DF_ERR_ALIGN;
  const bool multi = a->H > 1;
  if (!stride_ok(a->q_stride_tok) || !stride_ok(a->kc_stride_tok) ||
      (multi && (!stride_ok(a->q_stride_head) || !stride_ok(a->kc_stride_head))))
    return DF_ERR_ALIGN;
  if (!(a->softmax_scale > 0.f) || !std::isfinite(a->softmax_scale)) return DF_ERR_RANGE;
  if (!a->workspace || a->workspace_bytes < workspace_bytes(a->H, a->d, a->Nq)) return DF_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(a->workspace) & 255u) return DF_ERR_ALIGN;
  // the sampled queries are a strided view of Q
  const int n_samp = (a->Nq - a->q_offset + a->q_sample_stride - 1) / a->q_sample_stride;
  p.q = static_cast<const u16 *>(a->q) + int64_t(a->q_offset) * a->q_stride_tok;
  p.q_st = a->q_stride_tok * a->q_sample_stride;
  p.q_sh = a->q_stride_head;
  p.Nq = n_samp;
  p.k_cur = static_cast<const u16 *>(a->k_cur);
  p.v_cur = nullptr;
  p.k_hist = static_cast<const u16 *>(a->k_hist);
  p.v_hist = nullptr;
  p.out = nullptr;
  p.lse = nullptr;
  p.kc_st = a->kc_stride_tok; p.kc_sh = a->kc_stride_head;
  if ((int64_t(a->Nc - 1) * a->kc_stride_tok + a->d) * 2 >= kMaxBufferBytes || a->kc_stride_tok >= (1 << 24))
    return DF_ERR_RANGE;
  p.cur_bytes = uint32_t((int64_t(a->Nc - 1) * a->kc_stride_tok + a->d) * 2);
  p.c = a->softmax_scale * 1.4426950408889634f;
  p.lse_unit = float(double(a->softmax_scale) / double(p.c));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (a->d == 128) return launch<128, true>(p, a->workspace, a->score_out, st);
  return launch<64, true>(p, a->workspace, a->score_out, st);
}
