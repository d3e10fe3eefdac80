// Device body of the causal prefill attention (one work-group of it), shared
// by the prefill kernel and the fused prefill + decode kernel.
//
// Prefill is compute-bound (paper Sec. 2.2; Sec. 3.3, Table
// "tab:theory_cost": O(n d^2 + L n d) with L = r + n), so both contractions
// run on the bf16 matrix cores (fp32 accumulate).
//
// The queries of a (sequence, kv head) are its n positions x `group` query
// heads, laid end to end as rows position * group + head.  A query block is
// 256 consecutive rows (8 waves; 128 with 4), wave w its rows 32w .. 32w + 31,
// so every K/V tile staged in LDS serves all of them whatever the group: 64
// positions of a group of 4, 256 of a group of 1, 16 of a group of 16.  (Four
// waves of four heads each, the earlier layout, left 3 of 4 waves idle with
// one query head per kv head: a 1000-token chunk over 1003 cached tokens with
// 32 query and 32 kv heads took 76 us.)  Which block a work-group runs is the
// kernel's choice (work_item below); it may run two, one after the other.
// Each wave's state (Q^T, S, P, O) stays in registers.
//
// Per key tile t of a wave:
//     S(t)^T = K(t) Q^T;  mask, online softmax of S(t) -> P(t) (bf16);
//     O^T += V(t)^T P(t)^T
// Three bodies share these steps: 8 waves on 256 rows, two wave groups half a
// period apart on the same tiles; kDual, 8 waves on 128 rows, the two groups on
// alternate tiles, each with its own buffers; and 4 waves on 128 rows, two
// work-groups per CU.  The first needs the fewest K/V loads per flop.  The
// second halves a block's time when there are too few blocks for the CUs: a
// 4-wave work-group takes 1.2 us per tile alone on its CU and 1.5 beside another,
// so the longest block of a 2048-token prompt (32 tiles) bounded the launch at
// 46 us of a 54 us call; a dual one takes 0.7 us per tile on few CUs and 0.85 on
// all (1.7 us for the two groups' tiles, 1270 TFLOP/s over 256 CUs, near the 1337
// of a 16384^3 library product) and the call 46 us.  The third keeps the plain
// entry point's results the same bits on any CU count (the groups' merge of
// the second reorders sums).
// Key tiles of 64 keys = 4 pages go from HBM straight into LDS with the direct
// buffer-to-LDS loads, double-buffered; the first tile of a block is requested
// before Q and the block-table copy are waited for.
// Rows are 256 B with their 16-byte chunks permuted by XOR with
// swz(r) = 4(r%4) ^ (r/4)%4, which makes both the 16-byte K operand reads and
// the transposing V reads bank-conflict free; the permutation is applied on
// the HBM side of each load.  The 16 MFMAs of each product issue in a fixed
// order with the LDS operands of the next few already in flight.
//   S^T[key][q] = K Q^T      32x32x16 MFMA; A = K rows from LDS, B = Q^T
//   O^T[d][q] += V^T P^T     32x32x16 MFMA; A = V^T gathered by the LDS
//                            transposing read (ds_read_b64_tr_b16), B = P^T
//                            taken straight from the S^T accumulators as bf16
// Online softmax in base 2 (scores scaled by scale*log2 e inside one FMA); the
// causal mask is applied only on tiles that cross the diagonal; row sums are
// taken in fp32 over the probabilities before they are rounded to bf16 for PV.
// The running maximum moves only when a column's tile maximum exceeds it by more than 2^8
// (O and l are then rescaled); O / l does not depend on the reference maximum.
// O is staged through LDS so that each store writes whole 256-byte rows.
// Causal position: query row i of a sequence with prefix r sees keys
// 0 .. r + i (bottom-right alignment; a chunk reads every earlier chunk's KV).
#pragma once
#include <type_traits>

#include "mw_internal.h"
#include "prefill_layout.h"
#include "prefill_schedule.h"

namespace {
namespace pf {

using namespace mw;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int BN = 64;                       // keys per tile
constexpr int ROW = kHeadDim;                // tile row = one key, 128 bf16 (256 B)
constexpr int TILE = BN * ROW;               // one K or V tile, bf16 elements
constexpr int kBtCache = 4096;               // block-table entries staged in LDS
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRescaleLog2 = 8.f;          // lazy-rescale threshold (log2 units)

typedef __attribute__((address_space(3))) void lds_void;
constexpr int kBufferFormat = 0x00020000;    // buffer descriptor word 3: 32-bit data format

constexpr int kAhead = 4;                    // MFMA operands kept in flight

template <bool B>
using flag = std::integral_constant<bool, B>;

// Where a piece of a key-range-split query block leaves its partial result:
// the unnormalised output O~ = sum_j 2^(s_j - m) v_j and (m, l = sum_j
// 2^(s_j - m)) over the piece's keys (s in log2 units), for every row and
// query head, in slot `piece`.
struct SplitOut {
    float *o;     // [max_pieces][rows][hq][128] fp32
    float2 *ml;   // [max_pieces][rows][hq]
    int64_t rows; // rows of the call (sum of the new lengths)
    int piece_tiles, max_pieces, piece;
};

__device__ inline int swz(int row) { return ((row & 3) << 2) ^ ((row >> 2) & 3); }

__device__ inline uint32_t cvt2(float a, float b) {
    bf16x2 v;
    v[0] = static_cast<__bf16>(a);
    v[1] = static_cast<__bf16>(b);
    return __builtin_bit_cast(uint32_t, v);
}

// NaN-propagating maximum: a single v_maximum3_f32 on gfx950, with no
// canonicalisation of the MFMA results it reads.
__device__ inline float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// max(x, x of lane l ^ 32).  v_permlane32_swap exchanges lanes 32..63 of its
// first operand with lanes 0..31 of its second, so with x in both operands
// one result holds the lower half's values in every lane and the other the
// upper half's.  Inline assembly because this compiler takes the builtin's
// second result to be its first (the maximum would then cover only half the
// keys); the s_nop covers the two wait states the swap needs after a vector
// instruction writes its operands.
__device__ inline float max_xor32(float x) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return vmax(a, b);
}

// Transposing LDS read: within each 16-lane group, lane s points at 4
// consecutive elements of a row; lane 4a+b receives element b of the chunks of
// lanes a, a+4, a+8, a+12.  The address-space cast keeps the pointer's origin
// visible to the compiler.
__device__ inline i16x4 lds_read_tr(const char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(p));
}

// Work-group barrier without the memory fence of __syncthreads: LDS reads are
// consumed before every barrier, and the tile loads are waited for explicitly.
__device__ inline void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Inclusive scan over the wave's lanes: lane i receives the sum of x over
// lanes 0 .. i (lane 63 the total).
__device__ inline int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// The query block(s) one work-group runs: block blk, then blk2 if >= 0, of
// sequence b (first row row0 of Q, n new tokens over a prefix of r) and kv
// head kvh.
struct Item {
    int b, kvh, row0, n, r, blk, blk2;
};

// How the work-groups of a launch are mapped to query blocks.  x counts kv
// heads fastest: work-groups go round-robin over the 8 XCDs, so with 8 kv heads
// each XCD's L2 holds the K/V of one.  j = x / hkv is then:
//   kPerSequence  the j-th heaviest block of sequence blockIdx.y
//   kPairs        blocks nqb-1-j and j of sequence blockIdx.y (equal cost)
//   kSorted       the j-th heaviest block of the whole batch (at most 64
//                 sequences): the blocks of one call are dispatched longest
//                 first whatever their sequence, and no work-group is empty
enum { kPerSequence = 0, kPairs = 1, kSorted = 2 };

// Fills `it` for work-group (x, y); false if there is no block for it.
// kBR: query rows per block.  Uniform over the work-group.
template <int kBR>
__device__ __forceinline__ bool work_item(const int32_t *__restrict__ qo_indptr,
                                          const int32_t *__restrict__ prefix_lens, int batch, Divisor hkv, Divisor group,
                                          int order, int x, int y, Item &it) {
    int j = x / hkv;
    it.kvh = x - j * hkv;
    it.blk2 = -1;
    if (order == kSorted && batch > 1) {
        // lane i: sequence i
        const int lane = threadIdx.x & 63;
        const bool in = lane < batch;
        const int first = in ? qo_indptr[lane] : 0;
        const int n = in ? qo_indptr[lane + 1] - first : 0;
        const int r = in ? prefix_lens[lane] : 0;
        const int nqb = (n * group + kBR - 1) / kBR;
        auto at_least = [&](int t) __attribute__((always_inline)) {
            return prefill_blocks_at_least(nqb, n, r, group, kBR, t);
        };
        auto total = [&](int v) __attribute__((always_inline)) {
            return __builtin_amdgcn_readlane(wave_scan(v), 63);
        };
        if (j >= total(nqb)) return false;
        // the j-th heaviest block has t tiles, t the largest with more than j
        // blocks of t or more
        int t = 1, step = 1;
        while (total(at_least(t + step)) > j) step <<= 1;
        for (; step > 0; step >>= 1)
            if (total(at_least(t + step)) > j) t += step;
        const int above = at_least(t + 1), same = at_least(t) - above;
        j -= total(above);
        const int incl = wave_scan(same);
        const uint64_t hit = __builtin_amdgcn_ballot_w64(j >= incl - same && j < incl);
        if (!hit) return false;
        const int src = __builtin_ctzll(hit);
        it.b = src;
        it.blk = __builtin_amdgcn_readlane(nqb - above - 1 + incl - same, src) - j;
        it.row0 = __builtin_amdgcn_readlane(first, src);
        it.n = __builtin_amdgcn_readlane(n, src);
        it.r = __builtin_amdgcn_readlane(r, src);
        return true;
    }
    it.b = y;
    it.row0 = qo_indptr[y];
    it.n = qo_indptr[y + 1] - it.row0;
    it.r = prefix_lens[y];
    const int nqb = (it.n * group + kBR - 1) / kBR;
    if (j >= (order == kPairs ? (nqb + 1) / 2 : nqb)) return false;
    it.blk = nqb - 1 - j;
    if (order == kPairs && j != it.blk) it.blk2 = j;
    return true;
}

// kTableInLds: every block-table entry the work-group needs fits the LDS copy.
// The other instantiation reads entries past it with scalar loads, which makes
// the compiler wait for all outstanding LDS reads wherever it needs one.
// NW: waves per work-group.  8 (query blocks of 256 rows; waves w and
// w+4 share a SIMD) or 4 (blocks of 128 rows, two work-groups per CU):
// the same per-wave work, for grids that would leave CUs idle with 8.
// kDual (8 waves): a block of 128 rows run by both wave groups, group 0 on the
// key tiles 0, 2, 4 .. and group 1 on 1, 3, 5 .. of its range, merged through
// LDS at the end; for one block (no blk2).
// kSplit (kDual only): the work-group computes piece sp.piece of its query
// block's key range (prefill_pieces), writing partials to sp when the block
// has more than one piece and the normalised output otherwise.
template <bool kTableInLds, int NW, bool kDual = false, bool kSplit = false>
__device__ __forceinline__ void
prefill_block(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
              const uint16_t *__restrict__ q, uint16_t *__restrict__ out, const int32_t *__restrict__ bt,
              int bt_stride, Divisor hkv, Divisor group, int num_pages, float scale_log2,
              // the block(s) to run, and the LDS buffers: K and V tiles
              // (2 * TILE each, or 4 * TILE with kDual, 1024-byte aligned) and
              // the block-table copy (kBtCache entries)
              const Item item, uint16_t *s_k, uint16_t *s_v, int32_t *s_bt, const SplitOut sp = {}) {
    static_assert(NW == 8 || NW == 4, "8 or 4 waves");
    static_assert(!kDual || NW == 8, "two groups of four waves");
    static_assert(!kSplit || kDual, "the key-range split runs dual blocks");
    static_assert(kDualBufBytes == 2 * TILE * sizeof(uint16_t) && kDualTableBytes == kBtCache * sizeof(int32_t),
                  "buffers of a dual block");
    constexpr int kBR = kDual ? 128 : 32 * NW;  // query rows per block
    constexpr int kNT = 64 * NW;        // threads
    constexpr bool kStageQ = kDual || NW == 4;  // Q through LDS: 256 rows do not fit beside the first tile
    constexpr int kRows = 64 / NW;      // tile rows (keys) each wave loads
    constexpr int kJ = kRows / 4;       // 1-KB loads per wave per K (or V) tile
    constexpr int kEvery = 8 / kJ;      // QK MFMAs between two of this wave's loads
    const int b = item.b, kvh = item.kvh, row0 = item.row0, n = item.n, r = item.r;
    const int rows = n * group;
    // key tiles of block qb: those of its last row's position
    auto block_tiles = [&](int qb) __attribute__((always_inline)) {
        return (r + (min((qb + 1) * kBR, rows) + group - 1) / group + BN - 1) / BN;
    };
    const int nt_a = block_tiles(item.blk);  // the heavier block's
    // key tiles [t_lo, t_hi) of this work-group's (single) block and its
    // number of pieces (1 without the split); tile t_lo is loaded first and
    // page p of the sequence sits at s_bt[p - 4 t_lo] in the table copy
    int t_lo = 0, t_hi = nt_a, n_pieces = 1;
    if constexpr (kSplit) {
        n_pieces = prefill_pieces(nt_a, sp.piece_tiles, sp.max_pieces);
        if (sp.piece >= n_pieces) return;
        t_lo = sp.piece * nt_a / n_pieces;
        t_hi = (sp.piece + 1) * nt_a / n_pieces;
    }
    const int pbase = 4 * t_lo;
    const int32_t *btrow = bt + static_cast<size_t>(b) * bt_stride;
    const int np_seq = min((r + n + kPageSize - 1) / kPageSize, bt_stride);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform per wave
    const int hq = hkv * group;
    const int l32 = lane & 31, g = lane >> 5;
    // quotient of a row offset o < group + 32 by group: a product with the
    // rounded-up reciprocal is exact while o * group < 2^16
    // (groups of up to 32; for larger ones the quotient is 0 or 1)
    const int recip = group <= 32 ? 65536 / group + 1 : 0;
    const int one_at = group <= 32 ? 1 << 30 : group;
    auto over_group = [&](int o) __attribute__((always_inline)) { return ((o * recip) >> 16) + (o >= one_at); };

    // Block-table entries of this work-group's keys (the heavier block's): two
    // per thread are requested here, ahead of the first tile and Q, and stored
    // to LDS behind them, so that the three latencies overlap (waiting for
    // each in turn made a work-group's start 3.4 us of ~20).
    const int np_wg = min(4 * t_hi, np_seq), bt_end = min(np_wg, pbase + kBtCache);
    int32_t bt_first[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) bt_first[k] = btrow[min(pbase + static_cast<int>(threadIdx.x) + k * kNT, bt_end - 1)];
    const int seq_len = r + n;

    // ---- per-lane byte offsets, computed once
    // K operand: row l32 (+32 rows for the second key block), logical chunk
    // 2kb+g; since 2kb+g = 2kb ^ g, dim-step kb is at koff ^ 32kb
    const int koff = l32 * 256 + 16 * (g ^ swz(l32));
    // V transposing reads: lane s of 16-lane group q reads row 8hh + 4(q/2) + s/4
    // (+16 ks) at dims 32db + 16(q%2) + 4(s%4): logical chunk 4db + 2(q%2) + (s%4)/2,
    // so dim block db is at voff[hh] ^ 64db
    int voff[2];
    {
        const int q16 = lane >> 4, s16 = lane & 15;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int row = 8 * hh + 4 * (q16 >> 1) + (s16 >> 2);
            const int chunk = (2 * (q16 & 1) + ((s16 & 3) >> 1)) ^ swz(row);
            voff[hh] = row * 256 + 16 * chunk + 8 * (s16 & 1);
        }
    }
    // direct loads: wave w moves rows kRows w + 4j + lane/16 (j < kJ) of every
    // K and V tile, all in page kRows w / 16 of the tile; lane i lands in
    // physical chunk i%16.  Byte offsets within the page:
    int goff[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int row = (kRows * wave) % 16 + 4 * j + (lane >> 4);
        goff[j] = 2 * (row * kHeadDim + 8 * ((lane & 15) ^ swz(row)));
    }
    const int lpage = kRows * wave / 16;  // page of the tile this wave loads
    const int grp = NW == 8 ? wave >> 2 : 0;  // wave group of the 8-wave bodies
    uint16_t *const sk = s_k + (kDual ? grp * 2 * TILE : 0);  // the tile buffers the wave reads
    uint16_t *const sv = s_v + (kDual ? grp * 2 * TILE : 0);
    // whole-page loads of the 8-wave bodies: 4 KB of K or V in four loads
    const int lw = wave & 3;  // page of the tile
    int goffp[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 4 * j + (lane >> 4);
        goffp[j] = 2 * (row * kHeadDim + 8 * ((lane & 15) ^ swz(row)));
    }

    // per-item state
    int nt = 0, qabs = 0, diag = 0;
    // Key tiles that some row of the wave sees, from tile 0.  For the others of its
    // block (past all of its rows) it only loads its pages and takes the barriers:
    // their probabilities are 0, but 0 times a value that is not finite is not.
    // A wave past the sequence's rows has none: computing there on zeros only
    // slowed the others down (14 sequences of 8 to 53 tokens over 12549 with 32/32
    // heads took 732 us, now 558; 15 of 8 to 20 over 198 with 32/8 on 64 CUs 22.3,
    // now 18.7).
    int nt_w = 0;
    int pos0 = 0, head0 = 0;   // position and head of the wave's first row
    uint4 qop[8];
    f32x16 oacc[4];
    f32x16 sacc[2];
    uint4 pop[4];
    // With kDual a row may see no key of a group's first tiles (they lie past
    // its position): starting from the lowest finite value instead of -inf
    // keeps its probabilities there at 2^(-inf) = 0 (and not at NaN), and any
    // real score still raises it.
    constexpr float kNoMax = kDual ? -__FLT_MAX__ : -INFINITY;
    float m_run = kNoMax;
    float l_run = 0.f;

    // The (page, kv head) block of sequence page p (uniform per wave): its pool
    // element offset and the bytes of it that hold the sequence's tokens.  A
    // page past the sequence or outside the pool has 0 bytes, and the last page
    // only its rows below r + n: the buffer loads return zeros past that, so
    // slack slots and absent pages are never read, whatever bits they hold
    // (zero keys and values past the sequence are also discarded by the causal
    // mask: they lie after every query).
    struct PageRef {
        size_t base;
        int bytes;
    };
    auto page_ref = [&](int p, int page) __attribute__((always_inline)) {
        const bool ok = p < np_seq && page >= 0 && page < num_pages;
        PageRef ref;
        ref.base = ok ? (static_cast<size_t>(page) * hkv + kvh) * (kPageSize * kHeadDim) : 0;
        ref.bytes = ok ? min(seq_len - kPageSize * p, kPageSize) * (kHeadDim * 2) : 0;
        return ref;
    };
    // Page `lpage` of key tile `it`, its entry read from the LDS copy of the table.
    auto tile_page = [&](int it) __attribute__((always_inline)) {
        const int p = 4 * it + lpage;
        int page = -1;
        if (p < np_seq) {
            if constexpr (kTableInLds)
                page = __builtin_amdgcn_readfirstlane(s_bt[p - pbase]);
            else
                page = p - pbase < kBtCache ? __builtin_amdgcn_readfirstlane(s_bt[p - pbase]) : btrow[p];
        }
        return page_ref(p, page);
    };
    // Loads (1 KB each) of this wave's half page of one tile: buffer loads over
    // a descriptor of the page's valid rows (the hardware returns zeros past
    // them).  Buffer rather than global loads: the compiler counts a global
    // load into LDS as an outstanding LDS access too, which would make every
    // operand read wait for all LDS reads in flight.  The LDS destination goes
    // through an integer, so the compiler does not tie later LDS reads to these
    // loads; the loop waits for them explicitly.
    auto page_rsrc = [&](const uint16_t *pool, PageRef ref) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(pool + ref.base), 0, ref.bytes,
                                                 kBufferFormat);
    };
    auto page_load = [&](__amdgpu_buffer_rsrc_t rsrc, uint16_t *dst, int j) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc, reinterpret_cast<lds_void *>(reinterpret_cast<uintptr_t>(dst + (kRows * wave + 4 * j) * ROW)), 16,
            goff[j], 0, 0, 0);
    };

    auto page_load_full = [&](__amdgpu_buffer_rsrc_t rsrc, uint16_t *dst, int j) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc, reinterpret_cast<lds_void *>(reinterpret_cast<uintptr_t>(dst + (16 * lw + 4 * j) * ROW)), 16,
            goffp[j], 0, 0, 0);
    };

    // Matrix work: O^T += V^T P^T with V from tile buffer vbuf (if PV), then
    // S^T = K Q^T with K from tile buffer kbuf (if QK); `load(j)` is called
    // after every kEvery-th MFMA of a QK-only phase.  Operation i < npv is PV
    // key-step i/4, dim block i%4; the rest are QK dim-step j/2, key block j%2.
    auto mfma_phase = [&](auto pv_flag, auto qk_flag, int kbuf, int vbuf, auto load) __attribute__((always_inline)) {
        constexpr bool PV = decltype(pv_flag)::value, QK = decltype(qk_flag)::value;
        constexpr int npv = PV ? 16 : 0;
        constexpr int nop = npv + (QK ? 16 : 0);
        const char *vb_ = reinterpret_cast<const char *>(sv + vbuf * TILE);
        const char *kb_ = reinterpret_cast<const char *>(sk + kbuf * TILE);
        // per-read offsets are recomputed here (one XOR each) rather than held
        // in registers across the loop
        int ko = koff, vo0 = voff[0], vo1 = voff[1];
        asm volatile("" : "+v"(ko), "+v"(vo0), "+v"(vo1));
        auto fetch = [&](int i) __attribute__((always_inline)) -> bf16x8 {
            if (i < npv) {
                const int off = (i >> 2) * 16 * 256;
                const i16x4 lo = lds_read_tr(vb_ + off + (vo0 ^ (64 * (i & 3))));
                const i16x4 hi = lds_read_tr(vb_ + off + (vo1 ^ (64 * (i & 3))));
                return __builtin_bit_cast(
                    bf16x8, make_uint4(__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y,
                                       __builtin_bit_cast(uint2, hi).x, __builtin_bit_cast(uint2, hi).y));
            }
            const int j = i - npv;
            return *reinterpret_cast<const bf16x8 *>(kb_ + (j & 1) * 32 * 256 + (ko ^ (32 * (j >> 1))));
        };
        __builtin_amdgcn_s_setprio(2);  // a wave issuing MFMAs wins issue conflicts on the SIMD
        bf16x8 opnd[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) opnd[i] = fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < nop; ++i) {
            const bf16x8 a = opnd[i % kAhead];
            if (i < npv) {
                oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    a, __builtin_bit_cast(bf16x8, pop[i >> 2]), oacc[i & 3], 0, 0, 0);
            } else {
                // the first step of each key block starts from zero, so the
                // score registers are free until the QK half of the phase
                const int j = i - npv;
                const f32x16 zero = {};
                sacc[j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    a, __builtin_bit_cast(bf16x8, qop[j >> 1]), j < 2 ? zero : sacc[j & 1], 0, 0, 0);
            }
            if (i + kAhead < nop) opnd[i % kAhead] = fetch(i + kAhead);
            if (!PV && i % kEvery == kEvery - 1) load(i / kEvery);
            if (PV && kDual && i % 8 == 3) load(i / 8);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };

    // Causal mask and online softmax of S(t) into P(t).
    auto softmax_phase = [&](int t, auto load) __attribute__((always_inline)) {
        const int k0 = t * BN;
        load(0);
        load(1);
        if (k0 + BN - 1 > diag) {
#pragma unroll
            for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = k0 + 32 * blk + 8 * (i >> 2) + 4 * g + (i & 3);
                    if (key > qabs) sacc[blk][i] = -INFINITY;
                }
        }
        // column maximum as a tree of 3-way maxima (short dependency chain)
        float m8[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            m8[j] = vmax(vmax(sacc[j >> 2][4 * (j & 3)], sacc[j >> 2][4 * (j & 3) + 1]),
                         vmax(sacc[j >> 2][4 * (j & 3) + 2], sacc[j >> 2][4 * (j & 3) + 3]));
        float mx = vmax(vmax(vmax(m8[0], m8[1]), vmax(m8[2], m8[3])), vmax(vmax(m8[4], m8[5]), vmax(m8[6], m8[7])));
        mx = max_xor32(mx);  // lanes l and l^32 hold the same query
        const float m_tile = mx * scale_log2;
        if (__builtin_amdgcn_ballot_w64(m_tile > m_run + kRescaleLog2) != 0) {
            const float m_new = vmax(m_run, m_tile);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
        }
        load(2);
        load(3);
        // key-step ks covers registers 8a..8a+7 of block ks/2, i.e. keys
        // 16ks + 8(e/4) + 4g + e%4 for operand element e
        float lsum[4];
#pragma unroll
        for (int kstep = 0; kstep < 4; ++kstep) {
            const int blk = kstep >> 1, a8 = (kstep & 1) * 8;
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[blk][a8 + e], scale_log2, -m_run));
            pop[kstep] = make_uint4(cvt2(p[0], p[1]), cvt2(p[2], p[3]), cvt2(p[4], p[5]), cvt2(p[6], p[7]));
            // row sums in fp32 with plain adds: a dot product over the bf16
            // values would wait behind the other wave's MFMAs on this SIMD
            load(4 + kstep);
            lsum[kstep] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        }
        l_run += (lsum[0] + lsum[1]) + (lsum[2] + lsum[3]);
    };

    // The first tile of an item: its pages straight from the block table in
    // HBM, so the loads can start before the table copy in LDS is complete
    // (its K and, with 4 waves, its V; the 8-wave body loads V(0) in its
    // first period).
    auto first_tile = [&](auto with_v) __attribute__((always_inline)) {
        const int p0 = pbase + lpage;
        const PageRef ref = page_ref(p0, p0 < np_seq ? btrow[p0] : -1);
        const __amdgpu_buffer_rsrc_t rk = page_rsrc(kpool, ref), rv = page_rsrc(vpool, ref);
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            page_load(rk, s_k, j);
            if constexpr (decltype(with_v)::value) page_load(rv, s_v, j);
        }
    };

    for (int pass = 0; pass < (item.blk2 >= 0 ? 2 : 1); ++pass) {
        const int qblk = pass == 0 ? item.blk : item.blk2;
        nt = block_tiles(qblk);
        const int wrow = qblk * kBR + (kDual ? lw : wave) * 32;  // the wave's first row
        pos0 = wrow / group;
        head0 = wrow - pos0 * group;
        const int o = head0 + l32, dpos = over_group(o);
        const int pos = pos0 + dpos;        // this lane's query column
        const int hrow = o - dpos * group;  // and its head in the group
        qabs = r + pos;
        diag = r + pos0;                    // smallest query of the wave
        // (kept from the compiler, and the branches of the 8-wave loop hinted below:
        // telling a wave without rows apart, it laid that loop out with jumps that
        // made full blocks take up to 4% longer)
        int last_key = wrow < rows ? r + pos0 + over_group(head0 + 31) : -BN;
        asm volatile("" : "+s"(last_key));
        nt_w = min(nt, last_key / BN + 1);
        if (pass > 0) wg_barrier();  // the previous block's output staging is done
        PageRef ref_0{0, 0}, ref_1{0, 0};  // kDual: page lw of the group's first two tiles
        if constexpr (kDual) {
            // pages straight from the block table in HBM (the LDS copy is not
            // complete yet)
            const int p0 = pbase + 4 * grp + lw, p1 = p0 + 8;
            ref_0 = page_ref(p0, p0 < min(4 * t_hi, np_seq) ? btrow[p0] : -1);
            ref_1 = page_ref(p1, p1 < min(4 * t_hi, np_seq) ? btrow[p1] : -1);
            const __amdgpu_buffer_rsrc_t rk = page_rsrc(kpool, ref_0);
#pragma unroll
            for (int j = 0; j < 4; ++j) page_load_full(rk, sk, j);
        } else {
            first_tile(flag<NW == 4>());
        }
        // Q^T operand, all 8 dim-steps (k = 16*kb + 8*g + e).  The rows go
        // through tile buffers that are free until tile 1, a wave's 8 KiB in
        // the K operand's layout, and rows past the sequence's end are zeros
        // (their results are not stored).  Loaded straight into registers every
        // lane's 16 bytes lie in another row, so a request touches 32 rows and
        // both groups of a dual block ask for the same ones: the CU's 64
        // requests took about 1 us of a work-group's start; whole rows, once
        // each, are 32 requests of four rows.  Kernel time, direct / through
        // LDS: one prompt of 256 tokens (32/8 heads) 9.7 / 8.6 us, of 768
        // 15.8 / 14.6, of 2048 41.6 / 40.0; 2048 tokens of 8/1 heads on 96 CUs
        // 28.6 / 26.9.  The 8-wave body keeps the direct loads: staging what
        // fits (six waves' rows) was 1% slower on 16384-token prompts.
        [[maybe_unused]] uint16_t *const sq = kDual ? s_v + (lw < 2 ? 1 : 3) * TILE + (lw & 1) * (TILE / 2)
                                                    : (wave < 2 ? s_k : s_v) + TILE + (wave & 1) * (TILE / 2);
        if constexpr (kStageQ) {
            const uint16_t *qp = q + (static_cast<size_t>(row0 + min(pos0, n - 1)) * hq + kvh * group) * kHeadDim;
            // bytes from head 0 of the group at position pos0 to the sequence's
            // end (a wave's rows lie within 33 positions)
            const int bytes = 2 * kHeadDim * max(min(n - pos0, 33) * hq - kvh * group, 0);
            const __amdgpu_buffer_rsrc_t rq =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(qp), 0, bytes, kBufferFormat);
            const int first = kDual ? 16 * grp : 0;  // each group loads half of the rows both use
#pragma unroll
            for (int j = 0; j < (kDual ? 4 : 8); ++j) {
                const int row = first + 4 * j + (lane >> 4), oo = head0 + row, dp = over_group(oo);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rq, reinterpret_cast<lds_void *>(reinterpret_cast<uintptr_t>(sq + (first + 4 * j) * ROW)), 16,
                    2 * ((dp * hq + oo - dp * group) * kHeadDim + 8 * ((lane & 15) ^ swz(row))), 0, 0, 0);
            }
        } else {  // (here rows past the end take the last position's)
            const uint16_t *qp =
                q + (static_cast<size_t>(row0 + min(pos, n - 1)) * hq + kvh * group + hrow) * kHeadDim + 8 * g;
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) qop[kb] = *reinterpret_cast<const uint4 *>(qp + 16 * kb);
        }
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
        m_run = kNoMax;
        l_run = 0.f;
        if (pass == 0) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = pbase + static_cast<int>(threadIdx.x) + k * kNT;
                if (i < bt_end) s_bt[i - pbase] = bt_first[k];
            }
            for (int i = pbase + static_cast<int>(threadIdx.x) + 2 * kNT; i < bt_end; i += kNT)
                s_bt[i - pbase] = btrow[i];
            __syncthreads();
        }
        if constexpr (kStageQ)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        [[maybe_unused]] auto read_q = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int kb = 0; kb < 8; ++kb)
                qop[kb] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(sq) + (koff ^ (32 * kb)));
        };
        if constexpr (!kDual) {
            // the wave's own rows, out of the buffers before tile 1's loads
            if constexpr (kStageQ) {
                read_q();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            wg_barrier();
        }

        if constexpr (kDual) {
            // Two wave groups on alternate tiles (dual_schedule has the order of
            // their steps, and why no buffer is written while it is read).
            const int total = t_hi - t_lo;
            const int own = (total + 1 - grp) / 2;  // tiles of this group
            const int mine = min(own, max(0, (nt_w - t_lo - grp + 1) / 2));  // of them the wave's rows see
            const auto tile = [&](int u) __attribute__((always_inline)) { return t_lo + 2 * u + grp; };
            // page lw of the group's tile u, its entry read a period ahead
            auto table_entry = [&](int u) __attribute__((always_inline)) {
                const int p = 4 * tile(u) + lw;
                const bool ok = u < own && p < np_seq;
                if constexpr (kTableInLds)
                    return s_bt[ok ? p - pbase : 0];
                else
                    return ok ? (p - pbase < kBtCache ? s_bt[p - pbase] : btrow[p]) : -1;
            };
            int pg_n = 0;
            PageRef ref_v = ref_1;  // page lw of tile u + 1, whose V is loaded in M(u + 1)
            PageRef ref_k{0, 0};    // page lw of tile u + 2, whose K is loaded in S(u)
            // page lw of tile u + 2 (no bytes past the group's last tile: the loads
            // return zeros)
            const auto next_k = [&](int u) __attribute__((always_inline)) {
                if constexpr (kTableInLds) {
                    ref_k = page_ref(4 * tile(u + 2) + lw, __builtin_amdgcn_readfirstlane(pg_n));
                    pg_n = table_entry(u + 3);
                } else {
                    ref_k = page_ref(4 * tile(u + 2) + lw, __builtin_amdgcn_readfirstlane(table_entry(u + 2)));
                }
                return page_rsrc(kpool, u + 2 < own ? ref_k : PageRef{0, 0});
            };
            dual_schedule(grp, total, mine, [&](auto kind, int u) __attribute__((always_inline)) {
                constexpr DualStep what = decltype(kind)::value;
                if constexpr (what == kDualFirstLoads) {
                    const __amdgpu_buffer_rsrc_t rv = page_rsrc(vpool, ref_0), rk = page_rsrc(kpool, ref_1);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        page_load_full(rv, sv, j);
                        page_load_full(rk, sk + TILE, j);
                    }
                } else if constexpr (what == kDualReadQ) {
                    read_q();
                    if constexpr (kTableInLds) pg_n = table_entry(2);
                } else if constexpr (what == kDualBarrier) {
                    wg_barrier();
                } else if constexpr (what == kDualWaitAll) {
                    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                } else if constexpr (what == kDualWaitOlder) {
                    __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
                } else if constexpr (what == kDualScores) {
                    mfma_phase(flag<false>(), flag<true>(), 0, 0, [](int) {});
                } else if constexpr (what == kDualSoftmax) {
                    const __amdgpu_buffer_rsrc_t rk = next_k(u);
                    softmax_phase(tile(u), [&](int j) __attribute__((always_inline)) {
                        if (j >= 4) page_load_full(rk, sk + (u & 1) * TILE, j - 4);
                    });
                } else if constexpr (what == kDualMatrix) {
                    const __amdgpu_buffer_rsrc_t rv = page_rsrc(vpool, ref_v);
                    mfma_phase(flag<true>(), flag<true>(), (u + 1) & 1, u & 1,
                               [&](int j) __attribute__((always_inline)) {
                                   page_load_full(rv, sv + ((u + 1) & 1) * TILE, j);
                               });
                    ref_v = ref_k;
                } else if constexpr (what == kDualLoadK) {
                    const __amdgpu_buffer_rsrc_t rk = next_k(u);
#pragma unroll
                    for (int j = 0; j < 4; ++j) page_load_full(rk, sk + (u & 1) * TILE, j);
                } else if constexpr (what == kDualLoadV) {
                    const __amdgpu_buffer_rsrc_t rv = page_rsrc(vpool, ref_v);
#pragma unroll
                    for (int j = 0; j < 4; ++j) page_load_full(rv, sv + ((u + 1) & 1) * TILE, j);
                    ref_v = ref_k;
                } else if constexpr (what == kDualLastSoftmax) {
                    softmax_phase(tile(u), [](int) {});
                } else if constexpr (what == kDualLastMatrix) {
                    mfma_phase(flag<true>(), flag<false>(), 0, u & 1, [](int) {});
                }
            });
        } else if constexpr (NW == 8) {
            // Two groups of four waves (one wave of each on every SIMD), half a
            // period apart: while one group runs its matrix phase M(t) =
            // O += V(t-1)^T P(t-1)^T, S(t) = K(t) Q^T, the other runs the
            // softmax of its previous scores on the vector ALU, so the matrix
            // cores of a SIMD stay busy through both waves' softmax.  Period t
            // (t = 0 .. nt):
            //   phase 2t:   group 0 M(t)        | group 1 softmax(t-1)
            //   phase 2t+1: group 0 softmax(t)  | group 1 M(t)
            // with a work-group barrier after each phase.  K(t+1) and V(t) are
            // loaded during period t (into the buffers K(t-1) and V(t-2) used)
            // and waited for at its end.  Row sums are plain fp32 adds: a dot
            // product instruction would wait behind the other group's MFMAs.
            // Each wave runs its own sequence M(0) S(0) M(1) .. S(nt-1) M(nt),
            // group 1 one phase after group 0 (a barrier ends every phase, 2nt+2
            // in all for both groups).  Group 1 issues all loads of period t
            // (K(t+1) and V(t), one page of each per wave) at the start of
            // phase 2t, its softmax phase, and waits for them at the end of
            // phase 2t+1: group 0's matrix phases issue only MFMAs and their
            // operand reads.
            // Block-table entry of page lw of tile it.  With the whole table in
            // LDS it is read one period before its loads (pg_n), so they never
            // wait for an LDS read, and taken as read (entry 0 past the
            // sequence): page_ref gives pages past the sequence no bytes and
            // tiles past the block are not loaded, so no select waits for it.
            auto table_entry = [&](int it) __attribute__((always_inline)) {
                const int p = 4 * it + lw;
                const bool ok = it < nt && p < np_seq;
                if constexpr (kTableInLds)
                    return s_bt[ok ? p - pbase : 0];
                else
                    return ok ? (p - pbase < kBtCache ? s_bt[p - pbase] : btrow[p]) : -1;
            };
            int pg_n = 0;
            PageRef ref_v{0, 0};  // page lw of tile t, whose V is loaded in period t
            auto period_loads = [&](int t) __attribute__((always_inline)) {
                PageRef ref_k;
                if constexpr (kTableInLds) {
                    ref_k = page_ref(4 * (t + 1) + lw, __builtin_amdgcn_readfirstlane(pg_n));
                    pg_n = table_entry(t + 2);
                } else {
                    ref_k = page_ref(4 * (t + 1) + lw, __builtin_amdgcn_readfirstlane(table_entry(t + 1)));
                }
                if (__builtin_expect(t + 1 < nt, 1)) {
                    const __amdgpu_buffer_rsrc_t rk = page_rsrc(kpool, ref_k);
#pragma unroll
                    for (int j = 0; j < 4; ++j) page_load_full(rk, s_k + ((t + 1) & 1) * TILE, j);
                }
                const __amdgpu_buffer_rsrc_t rv = page_rsrc(vpool, ref_v);
#pragma unroll
                for (int j = 0; j < 4; ++j) page_load_full(rv, s_v + (t & 1) * TILE, j);
                ref_v = ref_k;
            };
            auto vm_wait = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0x0F70); };
            if (grp == 1) {  // group 1's first phase: the loads of period 0
                ref_v = page_ref(lw, __builtin_amdgcn_readfirstlane(table_entry(0)));
                if constexpr (kTableInLds) pg_n = table_entry(1);
                period_loads(0);
                wg_barrier();
            }
            int t = 0;
            if (__builtin_expect(nt_w > 0, 1)) {
                mfma_phase(flag<false>(), flag<true>(), 0, 0, [](int) {});  // M(0): S(0) = K(0) Q^T
                if (grp == 1) vm_wait();
                wg_barrier();
                for (; __builtin_expect(t + 1 < nt_w, 1); ++t) {
                    // (a 64-byte line: where other code moved the head off it, the 70B
                    // layer's chunk on 96 CUs took 860 us instead of 837)
                    asm volatile(".p2align 6");
                    if (grp == 1) period_loads(t + 1);
                    softmax_phase(t, [](int) {});
                    wg_barrier();
                    // M(t+1): O += V(t)^T P(t)^T, S(t+1) = K(t+1) Q^T
                    mfma_phase(flag<true>(), flag<true>(), (t + 1) & 1, t & 1, [](int) {});
                    if (grp == 1) vm_wait();
                    wg_barrier();
                }
                // the wave's last tile: softmax(t), then O += V(t)^T P(t)^T
                if (grp == 1 && t + 1 < nt) period_loads(t + 1);
                softmax_phase(t, [](int) {});
                wg_barrier();
                mfma_phase(flag<true>(), flag<false>(), 0, t & 1, [](int) {});
                if (grp == 1) vm_wait();
                wg_barrier();
                ++t;
            } else {
                if (grp == 1) vm_wait();
                wg_barrier();
            }
            // tiles that only other waves see
            for (; t < nt; ++t) {
                if (grp == 1 && t + 1 < nt) period_loads(t + 1);
                wg_barrier();
                if (grp == 1) vm_wait();
                wg_barrier();
            }
            if (grp == 0) wg_barrier();  // group 0's last phase: none of its own work
        } else
        // Tile t+1 is loaded (into the other buffer) while tile t is processed;
        // the K and V pages of a tile are the same pages of the pool.
        for (int t = 0; t < nt; ++t) {
            const bool more = t + 1 < nt;
            const PageRef ref = more ? tile_page(t + 1) : PageRef{0, 0};
            const __amdgpu_buffer_rsrc_t rk = page_rsrc(kpool, ref), rv = page_rsrc(vpool, ref);
            uint16_t *dk = s_k + ((t + 1) & 1) * TILE;
            uint16_t *dv = s_v + ((t + 1) & 1) * TILE;
            auto load = [&](int j) __attribute__((always_inline)) {
                if (more) {
                    if (j < kJ)
                        page_load(rk, dk, j);
                    else
                        page_load(rv, dv, j - kJ);
                }
            };
            if (t < nt_w) {
                mfma_phase(flag<false>(), flag<true>(), t & 1, t & 1, load);
                softmax_phase(t, [](int) {});
                mfma_phase(flag<true>(), flag<false>(), t & 1, t & 1, [](int) {});
            } else {
#pragma unroll
                for (int j = 0; j < 2 * kJ; ++j) load(j);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's direct loads landed
            wg_barrier();
        }

        if constexpr (kDual) {
            // ---- merge the groups: waves w and w + 4 hold the same rows over
            // different keys.  Group 0 finishes dims 0..63 and group 1 dims
            // 64..127: each hands the other half of its O (in its own K
            // buffers, as float4 per lane) with its (m, l) (in the table copy,
            // which no wave reads past the loop's last barrier).
            const float lt = l_run + __shfl_xor(l_run, 32);
            f32x16 keep[2];
            {
                float4 *give = reinterpret_cast<float4 *>(reinterpret_cast<char *>(sk) + dual_hand_over(lw));
#pragma unroll
                for (int db = 0; db < 2; ++db) {
                    const f32x16 gv = grp == 0 ? oacc[2 + db] : oacc[db];
                    keep[db] = grp == 0 ? oacc[db] : oacc[2 + db];
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
                        give[(4 * db + i4) * 64 + lane] =
                            make_float4(gv[4 * i4], gv[4 * i4 + 1], gv[4 * i4 + 2], gv[4 * i4 + 3]);
                }
                if (g == 0)
                    *reinterpret_cast<float2 *>(reinterpret_cast<char *>(s_bt) + dual_ml(grp, lw * 32 + l32)) =
                        make_float2(m_run, lt);
            }
            __syncthreads();
            float inv, m_all, l_all;
            {
                const char *pk = reinterpret_cast<const char *>(s_k + (1 - grp) * 2 * TILE);
                const float2 ml = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(s_bt) +
                                                                    dual_ml(1 - grp, lw * 32 + l32));
                m_all = vmax(m_run, ml.x);
                const float wa = __builtin_amdgcn_exp2f(m_run - m_all), wb = __builtin_amdgcn_exp2f(ml.x - m_all);
                l_all = wa * lt + wb * ml.y;
                inv = 1.f / l_all;
                const float4 *got = reinterpret_cast<const float4 *>(pk + dual_hand_over(lw));
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const float4 v = got[(4 * db + i4) * 64 + lane];
                        keep[db][4 * i4 + 0] = wa * keep[db][4 * i4 + 0] + wb * v.x;
                        keep[db][4 * i4 + 1] = wa * keep[db][4 * i4 + 1] + wb * v.y;
                        keep[db][4 * i4 + 2] = wa * keep[db][4 * i4 + 2] + wb * v.z;
                        keep[db][4 * i4 + 3] = wa * keep[db][4 * i4 + 3] + wb * v.w;
                    }
            }
            // the wave's 32 x 64 half tile, staged in its group's V buffers so
            // that stores write whole half rows.  Nothing else of the merge lies
            // there, so no barrier is needed: the waves still merging read the
            // other group's K buffers and the table copy.
            char *st = reinterpret_cast<char *>(sv) + dual_stage(lw);
            if (kSplit && n_pieces > 1) {
                // this piece's partial: (m, l) and the unnormalised O, fp32
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const int c = 8 * db + 2 * i4 + g;
                        *reinterpret_cast<float4 *>(st + dual_stage_f32(l32, c)) =
                            make_float4(keep[db][4 * i4], keep[db][4 * i4 + 1], keep[db][4 * i4 + 2],
                                        keep[db][4 * i4 + 3]);
                    }
                const size_t slot = static_cast<size_t>(sp.piece) * sp.rows + row0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int row = 4 * j + (lane >> 4), c = lane & 15;
                    const float4 v = *reinterpret_cast<const float4 *>(st + dual_stage_f32(row, c));
                    const int oo = head0 + row, dp = over_group(oo);
                    const int h = kvh * group + oo - dp * group;
                    if (pos0 + dp < n)
                        *reinterpret_cast<float4 *>(sp.o + ((slot + pos0 + dp) * hq + h) * kHeadDim + 64 * grp +
                                                    4 * c) = v;
                }
                if (grp == 0 && g == 0 && pos < n)
                    sp.ml[(slot + pos) * hq + kvh * group + hrow] = make_float2(m_all, l_all);
            } else {
                // normalised bf16
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const int c = 4 * db + i4;
                        *reinterpret_cast<uint2 *>(st + dual_stage_bf16(l32, c) + 8 * g) =
                            make_uint2(cvt2(keep[db][4 * i4 + 0] * inv, keep[db][4 * i4 + 1] * inv),
                                       cvt2(keep[db][4 * i4 + 2] * inv, keep[db][4 * i4 + 3] * inv));
                    }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = 8 * j + (lane >> 3), c = lane & 7;
                    const uint4 v = *reinterpret_cast<const uint4 *>(st + dual_stage_bf16(row, c));
                    const int oo = head0 + row, dp = over_group(oo);
                    const int h = kvh * group + oo - dp * group;
                    if (pos0 + dp < n)
                        *reinterpret_cast<uint4 *>(out + (static_cast<size_t>(row0 + pos0 + dp) * hq + h) * kHeadDim +
                                                   64 * grp + 8 * c) = v;
                }
            }
            return;
        }
        // ---- normalise and write O[pos][h][d].  The wave's 32 x 128 tile is
        // staged in LDS (the K/V buffers are free now) so that every store
        // writes 16 bytes per lane and four whole 256-byte rows per
        // instruction.  Row q of the staged tile holds its 16-byte chunk c at
        // chunk c ^ (q % 16).
        if (nt_w == 0) continue;  // (of no rows)
        const float lt = l_run + __shfl_xor(l_run, 32);
        const float inv = 1.f / lt;
        char *st = reinterpret_cast<char *>((wave < 4 ? s_k : s_v) + (wave & 3) * (32 * ROW));
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const int c = 4 * db + i4;
                *reinterpret_cast<uint2 *>(st + l32 * 256 + 16 * (c ^ (l32 & 15)) + 8 * g) =
                    make_uint2(cvt2(oacc[db][4 * i4 + 0] * inv, oacc[db][4 * i4 + 1] * inv),
                               cvt2(oacc[db][4 * i4 + 2] * inv, oacc[db][4 * i4 + 3] * inv));
            }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = 4 * j + (lane >> 4), c = lane & 15;
            const uint4 v = *reinterpret_cast<const uint4 *>(st + row * 256 + 16 * (c ^ (row & 15)));
            const int oo = head0 + row, dp = over_group(oo);
            const int h = kvh * group + oo - dp * group;
            if (pos0 + dp < n)
                *reinterpret_cast<uint4 *>(out + (static_cast<size_t>(row0 + pos0 + dp) * hq + h) * kHeadDim +
                                           8 * c) = v;
        }
    }
}


}  // namespace pf
}  // namespace
