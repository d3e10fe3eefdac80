// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdint>
#include <deque>
#include <vector>

#include "mw.h"

namespace mw {

constexpr int kHeadDim = 128;
constexpr int kPageSize = 16;
constexpr int kMaxTimingEvents = 8;

// Records `msg` as the calling thread's last error and returns `st`.
mw_status fail(mw_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// A divisor known on the host with its reciprocal, for the divisions of a prefill
// work-group's start: four scalar operations each instead of some twenty vector
// ones in a row.  m = floor((2^32 - 1) / d) makes the product's high half the
// quotient or one less for 0 <= n < 2^31.  Kernel time of calls of one tile 5.43
// -> 5.27 us, of a one-kv-head chunk of 2048 tokens over 4096 on 96 CUs 112.7 ->
// 109.6.
struct Divisor {
    int d;
    uint32_t m;
    __host__ explicit Divisor(int x) : d(x), m(0xffffffffu / static_cast<uint32_t>(x)) {}
    __host__ __device__ operator int() const { return d; }
};
__host__ __device__ inline int operator/(int n, Divisor by) {
    const int q = static_cast<int>((static_cast<uint64_t>(static_cast<uint32_t>(n)) * by.m) >> 32);
    return q + (n - q * by.d >= by.d ? 1 : 0);
}

// Key-range split of the prefill query blocks of the dual kernel: a block
// whose causal key range spans nt tiles of 64 keys is cut into this many
// pieces, piece i covering tiles [i nt / k, (i + 1) nt / k).  With
// piece_tiles >= 4 every cut lies at least three tiles before the block's end,
// so the first tile of every piece holds a key that every query of the block
// sees (a block of at most 128 positions has its diagonal in its last three
// tiles).
constexpr int kPrefillMaxPieces = 8;
constexpr int kPrefillMinPieceTiles = 4;
__host__ __device__ inline int prefill_pieces(int nt, int piece_tiles, int max_pieces) {
    const int k = (nt + piece_tiles - 1) / piece_tiles;
    return k < 1 ? 1 : (k > max_pieces ? max_pieces : k);
}
// Key tiles (64 keys) of query block q of a sequence with prefix r and n new
// tokens: blocks of `block_rows` rows of its n x group queries.  T: the type of
// the row counts; 32 bits hold those of a call that fits the device's memory, but
// not of every length a caller may ask a size for.
template <class T = int>
__host__ __device__ inline int prefill_block_tiles(T r, T n, T q, T block_rows, T group) {
    const T end = (q + 1) * block_rows < n * group ? (q + 1) * block_rows : n * group;
    return static_cast<int>((r + (end + group - 1) / group + 63) / 64);
}

// Blocks of t or more key tiles among the nqb blocks of `block_rows` rows of a
// sequence.  A block that ends with row e reads r + ceil(e / group) keys, so it has
// t tiles of 64 or more when e > (64 (t - 1) - r) group: the sequence's last blocks,
// counted without dividing by the group.
__host__ __device__ inline int prefill_blocks_at_least(int nqb, int n, int r, int group, int block_rows, int t) {
    const int c = 64 * (t - 1) - r;
    return c < 0 ? nqb : c >= n ? 0 : nqb - static_cast<int>(static_cast<unsigned>(c * group) / static_cast<unsigned>(block_rows));
}

// Number of CUs a stream's kernels may run on (its CU mask; all CUs of the
// current device for a stream without one).
int stream_cus(hipStream_t s);

}  // namespace mw

#define MW_HIP_TRY(expr)                                                                  \
    do {                                                                                  \
        hipError_t mw_e_ = (expr);                                                        \
        if (mw_e_ != hipSuccess)                                                          \
            return mw::fail(MW_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(mw_e_)); \
    } while (0)

struct mw_kv_pool {
    mw_kv_pool_desc desc;
    uint16_t *k;
    uint16_t *v;
    std::deque<int32_t> free_list;
    std::vector<uint8_t> is_free;
};

struct mw_timing {
    hipEvent_t ev[mw::kMaxTimingEvents];
    int n_events;          // events recorded by the last call (start + one per kernel)
    bool created;
    double host_ms;        // host time spent enqueueing
    std::chrono::steady_clock::time_point t0;
};

struct mw_partition {
    int device;
    hipStream_t prefill;
    hipStream_t decode;
    uint32_t prefill_mask[8];
    uint32_t decode_mask[8];
};

namespace mw {

// Timing helpers: begin() records the start event, kernel_done() one event per
// kernel, end() the host-side duration.  All are no-ops for a NULL handle.
mw_status timing_begin(mw_timing *t, hipStream_t s);
mw_status timing_kernel_done(mw_timing *t, hipStream_t s);
void timing_end(mw_timing *t);

// Reports a failed kernel launch (bad configuration) as MW_ERR_HIP.
mw_status check_launch(const char *what);

}  // namespace mw

namespace mw {

// Checked launch parameters of one decode call (shared by mw_decode_attn and
// the fused kernel's launcher).
struct DecodePlan {
    int64_t units;        // work-groups of the split kernel
    int chunk_pages;      // fixed chunks: resolved chunk length; 0 with the balanced split
    int64_t per_unit;     // balanced split: pages per unit (0 with fixed chunks)
    int64_t total;        // balanced split: pages of all (sequence, kv head) segments, in the split's numbering
    bool aligned;         // balanced split: each segment padded to a multiple of per_unit pages
    int64_t slots;        // partial slots in the workspace
    // workspace layout: partial O, (m, l), then per-sequence chunk bases (fixed
    // chunks) or per-slot done flags (balanced split)
    size_t off_ml, off_meta, bytes;
    int hkv, group;
    float scale_log2;
};
// Validates a decode call's arguments (workspace size included) and plans it.
// cus > 0 with chunk_pages = 0: the balanced split over that many CUs;
// cus = 0: fixed chunks only (chunk_pages 0 then means automatic chunks).
mw_status decode_prepare(const mw_decode_args *a, int64_t cus, DecodePlan *p, const char *who);
// Launches the kernel that merges the chunk partials of every (sequence, kv
// head) of a fixed-chunk split (the balanced split merges its own).
mw_status decode_combine_launch(const mw_decode_args *a, const DecodePlan &p, hipStream_t s);

// Checked launch parameters of one prefill call.
struct PrefillPlan {
    int hkv, group, batch;
    // the launch: waves of a work-group (8: 256-row query blocks; 4: 128-row
    // blocks, or the halves of dual blocks), grid (gx 0: nothing to do) and order
    // of the blocks (prefill_block.h)
    int waves, order;
    int64_t gx;
    int gy;
    bool table_in_lds;    // every block-table entry a work-group needs fits its LDS copy
    float scale_log2;
    // calls that may split key ranges (planned by prefill_split_plan)
    bool dual;            // dual blocks
    int64_t big_units;    // 256-row units of a launch whose last round runs as dual halves; 0: not such a launch
    int pieces;           // most pieces of any block; 1: no split
    int piece_tiles;      // target key tiles per piece
    int64_t rows;         // sum of the new lengths (rows of the workspace partials)
    size_t split_bytes;   // workspace the split needs
};
// Validates a prefill call's arguments and plans it for a stream that may use
// `cus` CUs: one launch of 8-wave blocks (with allow_small, or of 4-wave ones),
// or with split whatever prefill_split_plan finds best.
mw_status prefill_prepare(const mw_prefill_args *a, int64_t cus, bool allow_small, PrefillPlan *p, const char *who,
                          bool split = false);
// Plans body, order and key-range split of a call on `cus` CUs from its lengths
// (cus = 0: only the largest split any stream could take), with no more pieces
// than fit workspace_bytes; hkv and group must be set, lengths must have been
// validated.
void prefill_split_plan(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int hq,
                        int64_t cus, PrefillPlan *p, size_t workspace_bytes = ~size_t{0});
// Plans again if the caller's workspace is short of what the plan wants, with as
// many pieces as it holds, or none.  MW_ERR_INVALID_ARG where it is also short of
// what callers have always brought: prefill_base_pieces.
mw_status prefill_fit_workspace(const mw_prefill_args *a, int64_t cus, PrefillPlan *p, const void *ws, size_t bytes,
                                const char *who);
// Pieces of a call on blocks of 32 positions x up to four query heads (1: none):
// with fewer of them than CUs, so many that two work-groups come on a CU; with
// fewer than two per CU, three for blocks of 96 tiles and more.  A caller that
// plans for those knows no other calls to need a workspace.  (estimator.cpp,
// whose modelled launch they belong to.)
int prefill_base_pieces(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int hkv, int group,
                        int64_t cus);

}  // namespace mw
