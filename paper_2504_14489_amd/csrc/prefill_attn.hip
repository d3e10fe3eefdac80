// Causal prefill attention of a chunk of new tokens over its cached prefix:
// the kernel (its work-group body is in prefill_block.h) and its launch.
#include <algorithm>
#include <vector>

#include "prefill_block.h"

using namespace mw;

namespace {

using namespace pf;

template <bool kTableInLds, int NW>
__global__ void __launch_bounds__(64 * NW, NW == 4 ? 2 : 1)
k_prefill_attn(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
               const uint16_t *__restrict__ q, uint16_t *__restrict__ out,
               const int32_t *__restrict__ qo_indptr, const int32_t *__restrict__ prefix_lens,
               const int32_t *__restrict__ bt, int bt_stride, int batch, int hkv, int group, int num_pages,
               float scale_log2, int order) {
    __shared__ __attribute__((aligned(1024))) uint16_t s_k[2 * TILE];
    __shared__ __attribute__((aligned(1024))) uint16_t s_v[2 * TILE];
    __shared__ int32_t s_bt[kBtCache];
    Item item;
    if (!work_item<32 * NW>(qo_indptr, prefix_lens, batch, hkv, group, order, blockIdx.x, blockIdx.y, item))
        return;
    prefill_block<kTableInLds, NW>(kpool, vpool, q, out, bt, bt_stride, hkv, group, num_pages, scale_log2, item, s_k,
                                   s_v, s_bt);
}

// Launches of fewer pairs of 256-row blocks than CUs, through the entry point
// that may split key ranges: 128-row blocks whose keys the two wave groups
// share (kDual), one work-group per CU.  With kSplit, work-group (x, y) runs
// piece x % max_pieces of block unit x / max_pieces (nothing when the block has
// fewer pieces), so the pieces of a block are dispatched together, heaviest
// blocks first.
template <bool kTableInLds, bool kSplit>
__global__ void __launch_bounds__(512, 1)
k_prefill_dual(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
               const uint16_t *__restrict__ q, uint16_t *__restrict__ out,
               const int32_t *__restrict__ qo_indptr, const int32_t *__restrict__ prefix_lens,
               const int32_t *__restrict__ bt, int bt_stride, int batch, int hkv, int group, int num_pages,
               float scale_log2, int order, float *__restrict__ ws_o, float2 *__restrict__ ws_ml,
               int64_t rows, int piece_tiles, int max_pieces) {
    __shared__ __attribute__((aligned(1024))) uint16_t s_k[4 * TILE];
    __shared__ __attribute__((aligned(1024))) uint16_t s_v[4 * TILE];
    __shared__ int32_t s_bt[kBtCache];
    const int unit = kSplit ? static_cast<int>(blockIdx.x) / max_pieces : static_cast<int>(blockIdx.x);
    const SplitOut sp{ws_o, ws_ml, rows, piece_tiles, max_pieces, static_cast<int>(blockIdx.x) - unit * max_pieces};
    Item item;
    if (!work_item<128>(qo_indptr, prefix_lens, batch, hkv, group, order, unit, blockIdx.y, item)) return;
    prefill_block<kTableInLds, 8, true, kSplit>(kpool, vpool, q, out, bt, bt_stride, hkv, group, num_pages, scale_log2,
                                                item, s_k, s_v, s_bt, sp);
}

// Launches of 256-row blocks whose last round would leave most CUs idle: the
// n_big heaviest (block, kv head) units run as 256-row blocks and the rest,
// which fill at most half a round, as two 128-row dual blocks each, which end in
// about half the time.
template <bool kTableInLds>
__global__ void __launch_bounds__(512, 1)
k_prefill_mixed(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
                const uint16_t *__restrict__ q, uint16_t *__restrict__ out,
                const int32_t *__restrict__ qo_indptr, const int32_t *__restrict__ prefix_lens,
                const int32_t *__restrict__ bt, int bt_stride, int batch, int hkv, int group, int num_pages,
                float scale_log2, int order, int n_big) {
#ifdef __HIP_DEVICE_COMPILE__  // the host pass refuses a second use of one prefill_block instantiation
    __shared__ __attribute__((aligned(1024))) uint16_t s_k[4 * TILE];
    __shared__ __attribute__((aligned(1024))) uint16_t s_v[4 * TILE];
    __shared__ int32_t s_bt[kBtCache];
    // past n_big, kv heads fastest, then the unit's two halves
    const int x = blockIdx.x, over = x - n_big;
    const bool big = over < 0;
    const int half = big ? 0 : over / hkv % 2;
    const int unit = big ? x : n_big + over / (2 * hkv) * hkv + over % hkv;
    Item item;
    if (!work_item<256>(qo_indptr, prefix_lens, batch, hkv, group, order, unit, 0, item)) return;
    if (big) {
        prefill_block<kTableInLds, 8>(kpool, vpool, q, out, bt, bt_stride, hkv, group, num_pages, scale_log2, item, s_k,
                                      s_v, s_bt);
    } else {
        item.blk = 2 * item.blk + 1 - half;  // the heavier half first
        if (item.blk * 128 >= item.n * group) return;
        prefill_block<kTableInLds, 8, true>(kpool, vpool, q, out, bt, bt_stride, hkv, group, num_pages, scale_log2,
                                            item, s_k, s_v, s_bt);
    }
#endif
}

// Merge of the pieces of every split block: work-group (x, b) takes 32 of the
// n x hq output rows of sequence b (8 threads per row, 16 dims each): with M
// the largest reference maximum of the pieces,
// O = sum_i 2^(m_i - M) O~_i / sum_i 2^(m_i - M) l_i, written as bf16.
// Rows of blocks with one piece were written by the split kernel itself.
__global__ void __launch_bounds__(256)
k_prefill_merge(const float *__restrict__ ws_o, const float2 *__restrict__ ws_ml, uint16_t *__restrict__ out,
                const int32_t *__restrict__ qo_indptr, const int32_t *__restrict__ prefix_lens, int hq, int group,
                int64_t rows, int piece_tiles, int max_pieces) {
    const int b = blockIdx.y;
    const int row0 = qo_indptr[b];
    const int n = qo_indptr[b + 1] - row0;
    const unsigned at = 32u * blockIdx.x + (threadIdx.x >> 3);
    const int i = static_cast<int>(at / static_cast<unsigned>(hq)), h = static_cast<int>(at) - i * hq;
    if (i >= n) return;
    const int k = prefill_pieces(prefill_block_tiles(prefix_lens[b], n, (i * group + h % group) / 128, 128, group),
                                 piece_tiles, max_pieces);
    if (k < 2) return;
    const int d0 = 16 * (threadIdx.x & 7);
    const size_t row = static_cast<size_t>(row0 + i) * hq + h;
    const size_t stride = static_cast<size_t>(rows) * hq;  // one piece's slot
    // every piece's (m, l) and four pieces' O~ are requested together (one
    // piece at a time, 4 pieces of 2048 rows x 8 heads took 8.6 us)
    float2 ml[kPrefillMaxPieces];
#pragma unroll
    for (int p = 0; p < kPrefillMaxPieces; ++p)
        ml[p] = p < k ? ws_ml[p * stride + row] : make_float2(-INFINITY, 0.f);
    float m = -INFINITY;
#pragma unroll
    for (int p = 0; p < kPrefillMaxPieces; ++p) m = fmaxf(m, ml[p].x);
    float l = 0.f, o[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] = 0.f;
#pragma unroll
    for (int p0 = 0; p0 < kPrefillMaxPieces; p0 += 4) {
        if (p0 >= k) break;
        float4 v[4][4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float4 *src = reinterpret_cast<const float4 *>(
                ws_o + ((p0 + p < k ? p0 + p : 0) * stride + row) * kHeadDim + d0);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[p][e] = src[e];
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            // a piece without keys contributes nothing (nor does one past k)
            const bool in = ml[p0 + p].y > 0.f;
            const float w = in ? exp2f(ml[p0 + p].x - m) : 0.f;
            l += w * ml[p0 + p].y;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[4 * e + 0] += in ? w * v[p][e].x : 0.f;
                o[4 * e + 1] += in ? w * v[p][e].y : 0.f;
                o[4 * e + 2] += in ? w * v[p][e].z : 0.f;
                o[4 * e + 3] += in ? w * v[p][e].w : 0.f;
            }
        }
    }
    const float inv = 1.f / l;
    uint32_t packed[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) packed[e] = cvt2(o[2 * e] * inv, o[2 * e + 1] * inv);
    uint4 *dst = reinterpret_cast<uint4 *>(out + row * kHeadDim + d0);
    dst[0] = make_uint4(packed[0], packed[1], packed[2], packed[3]);
    dst[1] = make_uint4(packed[4], packed[5], packed[6], packed[7]);
}

// Sequences of a call whose blocks are ordered over the whole batch (one lane
// of a wave each).
constexpr int kMaxSorted = 64;

}  // namespace

namespace mw {

void prefill_split_plan(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int hq,
                        int64_t cus, PrefillPlan *p) {
    p->pieces = 1;
    p->piece_tiles = 0;
    p->split_bytes = 0;
    p->rows = 0;
    p->body = kBodyPlain;
    int max_nt = 0, min_nt = INT32_MAX;
    int64_t units = 0, tiles = 0, units8 = 0, tiles8 = 0;  // 128- and 256-row query blocks x kv heads, their key tiles
    for (int32_t b = 0; b < batch; ++b) {
        const int n = h_new_lens[b], r = h_prefix_lens[b];
        p->rows += n;
        const int64_t blocks = (static_cast<int64_t>(n) * p->group + 127) / 128, blocks8 = (blocks + 1) / 2;
        if (blocks == 0) continue;
        const int first = prefill_block_tiles<int64_t>(r, n, 0, 128, p->group), last = static_cast<int>((static_cast<int64_t>(r) + n + 63) / 64);
        max_nt = std::max(max_nt, last);
        min_nt = std::min(min_nt, first);
        units += blocks;
        tiles += blocks * (first + last) / 2;
        units8 += blocks8;
        tiles8 += blocks8 * (prefill_block_tiles<int64_t>(r, n, 0, 256, p->group) + last) / 2;
    }
    units *= p->hkv;
    tiles *= p->hkv;
    units8 *= p->hkv;
    tiles8 *= p->hkv;
    if (p->waves != 4 || units == 0) return;
    const auto bytes_for = [&](int pieces) {
        return pieces > 1 ? static_cast<size_t>(pieces) * p->rows * hq * (kHeadDim * 4 + 8) : 0;
    };
    if (cus <= 0) {  // sizing: the most pieces any stream's plan can take
        p->piece_tiles = kPrefillMinPieceTiles;
        p->pieces = prefill_pieces(max_nt, kPrefillMinPieceTiles, kPrefillMaxPieces);
        p->split_bytes = bytes_for(p->pieces);
        return;
    }
    // The cheapest body, and for dual blocks number of pieces of the longest
    // block, by their time in microseconds, fitted to 40 calls of 1 to 16
    // sequences, 1 to 4096 new tokens over 0 to 8000, groups of 1 to 8, on 96
    // to 256 CUs (each body and 1, 2 and 4 pieces measured on each; the choice
    // is within 8% of the best measured on all of them).  The fit dates from
    // before the 128-row bodies took Q through LDS, which made both alike 0.5
    // to 1.1 us faster.  A work-group takes `around` and `per` for each key
    // tile.  With no more work-groups than slots the call lasts as long as its
    // longest one; past that as the even share of the work and half the
    // lightest one, dispatched last.
    struct Cost {
        double around, per;
    };
    const Cost kAlone4{5.1, units <= cus ? 1.2 : 1.35}, kShared4{5.1, 2.0}, kDual{6.8, 0.75}, kFullDual{7.0, 0.79},
        kAlone8{6.5, 1.45}, kFull8{7.0, 1.6};
    const auto time_of = [&](int64_t n, double n_tiles, double longest, double lightest, int64_t slots, Cost alone,
                             Cost full) {
        const double one = alone.around + alone.per * longest;
        if (n <= cus) return one;
        return std::max(one, (full.around * n + full.per * n_tiles) / slots +
                                 0.5 * (full.around + full.per * lightest) * (n > slots));
    };
    const double us4 = time_of(units, tiles, max_nt, min_nt, 2 * cus, kAlone4, kShared4);
    const double us8 = time_of(units8, tiles8, max_nt, min_nt, cus, kAlone8, kFull8);
    // Pieces: partials are written and read at about 4 TB/s for the rows of
    // blocks longer than a piece, in a second launch (2 us).  Two blocks per CU
    // and more even out by themselves and are never cut; fewer, of 96 tiles and
    // more, always.
    const bool must_cut = units < 2 * cus && max_nt >= 96;
    double best = INFINITY;
    int best_pt = 0;
    for (int k = must_cut ? 2 : 1; k <= (units < 2 * cus ? kPrefillMaxPieces : 1); ++k) {
        const int pt = std::max(kPrefillMinPieceTiles, (max_nt + k - 1) / k);
        if (k > 1 && pt >= max_nt) break;
        const double cut = k == 1 ? 0.0 : std::min(1.0, static_cast<double>(max_nt - pt) / (max_nt - min_nt + 1));
        double us = time_of(units * k, tiles, pt, k == 1 ? min_nt : 0.5 * pt, cus, kDual, kFullDual);
        if (k > 1) us += 2.0 + cut * 2.0 * bytes_for(k) / 4e6;
        if (us < best) {
            best = us;
            best_pt = k > 1 ? pt : 0;
        }
    }
    if (!must_cut && us8 < std::min(best, us4)) {
        p->body = kBodyEight;
        return;
    }
    if (!must_cut && us4 < best) return;
    p->body = kBodyDual;
    if (best_pt == 0) return;
    p->piece_tiles = best_pt;
    p->pieces = prefill_pieces(max_nt, best_pt, kPrefillMaxPieces);
    p->split_bytes = bytes_for(p->pieces);
}

// Units (block, kv head) that a call of 256-row blocks on `cus` CUs runs as such
// when the rest, its last and partial round, goes to dual blocks; 0: all of
// them, one launch of k_prefill_attn.  Blocks taken longest first fill CUs
// evenly when they differ much in length (a prompt without a prefix), so only
// calls whose lightest block has at least half the tiles of the heaviest are
// treated.  There the last round costs a whole block's time for any fraction f
// of a round; as dual blocks it costs a little over half a block's while
// f <= 1/2.  Simulated over 2.3 to 5.3 rounds the launch gets 5-17% shorter,
// and past f = 1/2 longer.  Measured: the 70B layer's 2048-token chunk over 6144
// cached tokens on 96 CUs (5.33 rounds) next to its decode, 958 -> 911 us a
// step.
static int64_t prefill_big_units(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int64_t cus,
                                 const PrefillPlan &p) {
    if (p.waves != 8 || p.grid_y != 1 || p.order == kPairs) return 0;
    const int64_t units = p.blocks * p.hkv, whole = units / cus * cus;
    if (whole < 2 * cus || whole == units || 2 * (units - whole) > cus) return 0;
    int most = 0, least = INT32_MAX;
    for (int32_t b = 0; b < batch; ++b) {
        if (h_new_lens[b] == 0) continue;
        most = std::max(most, static_cast<int>((static_cast<int64_t>(h_prefix_lens[b]) + h_new_lens[b] + 63) / 64));
        least = std::min(least, prefill_block_tiles<int64_t>(h_prefix_lens[b], h_new_lens[b], 0, 256, p.group));
    }
    if (2 * least < most) return 0;
    return whole / p.hkv * p.hkv;
}

// Pairs of query blocks of `block_rows` rows over a batch's sequences.
static int64_t prefill_pairs(int32_t batch, const int32_t *h_new_lens, int group, int64_t block_rows) {
    int64_t n_pairs = 0;
    for (int32_t b = 0; b < batch; ++b)
        n_pairs += ((static_cast<int64_t>(h_new_lens[b]) * group + block_rows - 1) / block_rows + 1) / 2;
    return n_pairs;
}

mw_status prefill_prepare(const mw_prefill_args *a, int64_t cus, bool allow_small, PrefillPlan *p, const char *who) {
    if (!a || !a->pool || a->batch < 0 || a->batch > 65535 || a->bt_stride < 1 ||
        (a->batch > 0 && (!a->h_new_lens || !a->h_prefix_lens)))
        return fail(MW_ERR_INVALID_ARG, "%s: bad arguments", who);
    const mw_attn_shape *shape = &a->shape;
    const mw_kv_pool *pool = a->pool;
    if (shape->head_dim != kHeadDim) return fail(MW_ERR_UNSUPPORTED, "%s: head_dim must be 128", who);
    if (!(shape->scale > 0.f) || !(shape->scale < INFINITY))
        return fail(MW_ERR_INVALID_ARG, "%s: scale must be positive and finite", who);
    if (shape->num_kv_heads != pool->desc.num_kv_heads || shape->num_q_heads < 1 ||
        shape->num_q_heads % shape->num_kv_heads)
        return fail(MW_ERR_INVALID_ARG, "%s: num_q_heads must be a multiple of the pool's %d kv heads", who,
                    pool->desc.num_kv_heads);
    int64_t max_n = 0, max_pages = 0;
    for (int32_t b = 0; b < a->batch; ++b) {
        const int32_t n = a->h_new_lens[b], r = a->h_prefix_lens[b];
        if (n < 0 || r < 0 || static_cast<int64_t>(n) + r > static_cast<int64_t>(a->bt_stride) * kPageSize)
            return fail(MW_ERR_INVALID_ARG, "%s: sequence %d: prefix %d + new %d exceeds %d table pages", who, b, r,
                        n, a->bt_stride);
        max_n = n > max_n ? n : max_n;
        const int64_t pages = (static_cast<int64_t>(n) + r + kPageSize - 1) / kPageSize;
        max_pages = pages > max_pages ? pages : max_pages;
    }
    if (max_n > 0 && (!a->d_qo_indptr || !a->d_prefix_lens || !a->d_block_table || !a->d_q || !a->d_out))
        return fail(MW_ERR_INVALID_ARG, "%s: NULL device pointer", who);
    if (max_n > 0 && (!aligned16(a->d_q) || !aligned16(a->d_out)))
        return fail(MW_ERR_INVALID_ARG, "%s: Q and O must be 16-byte aligned", who);
    prefill_plan_lengths(a->batch, a->h_new_lens, shape->num_kv_heads, shape->num_q_heads / shape->num_kv_heads, cus,
                         allow_small, p);
    p->table_in_lds = max_pages <= kBtCache;
    p->scale_log2 = shape->scale * kLog2e;
    // Ordering over the batch costs a work-group 1.3 us to find its block: worth
    // it when blocks are long against the rounds of work-groups (an eighth of
    // the longest one's time), not for a launch that is resident at once.
    if (p->order == kSorted) {
        int64_t max_n_rows = 0, longest = 0;
        for (int32_t b = 0; b < a->batch; ++b) {
            max_n_rows = std::max<int64_t>(max_n_rows, static_cast<int64_t>(a->h_new_lens[b]) * p->group);
            if (a->h_new_lens[b] > 0)
                longest = std::max<int64_t>(longest, (static_cast<int64_t>(a->h_prefix_lens[b]) + a->h_new_lens[b] + 63) / 64);
        }
        const int64_t rows = 32 * p->waves, slots = p->waves == 8 ? cus : 2 * cus;
        const int64_t grid = (max_n_rows + rows - 1) / rows * p->hkv * a->batch;
        if (grid <= slots || 1.6 * longest * slots < 8 * 1.3 * grid) {
            p->order = p->paired ? kPairs : kPerSequence;
            p->grid_x = p->gx;
            p->grid_y = a->batch;
        }
    }
    if (p->grid_x > 0x7fffffff) return fail(MW_ERR_UNSUPPORTED, "%s: grid too large", who);
    return MW_OK;
}

void prefill_plan_lengths(int32_t batch, const int32_t *h_new_lens, int hkv, int group, int64_t cus,
                          bool allow_small, PrefillPlan *p) {
    p->hkv = hkv;
    p->group = group;
    p->batch = batch;
    p->table_in_lds = true;
    p->scale_log2 = 0.f;
    p->paired = 0;
    p->gx = p->grid_x = p->blocks = 0;
    p->grid_y = 1;
    p->order = kPerSequence;
    p->pieces = 1;
    p->piece_tiles = 0;
    p->rows = 0;
    p->split_bytes = 0;
    p->waves = 8;
    int64_t max_n = 0;
    for (int32_t b = 0; b < batch; ++b) max_n = std::max<int64_t>(max_n, h_new_lens[b]);
    if (max_n == 0) return;
    auto pairs_of = [&](int64_t rows) { return prefill_pairs(batch, h_new_lens, group, rows) * hkv; };
    // Eight waves (256-row blocks, one work-group per CU) unless their pairs
    // would not even give every CU one: then four waves (128-row blocks,
    // two work-groups per CU), which doubles the work-groups.
    int64_t rows = 256, slots = cus;
    if (allow_small && pairs_of(rows) < cus) {
        p->waves = 4;
        rows = 128;
        slots = 2 * cus;
    }
    // Pair blocks only when the pairs fill whole rounds of the work-group slots
    // of the stream's CUs: equal-cost pairs then finish together.  Otherwise
    // single blocks, heaviest first, fill the last round better.
    const int64_t max_blocks = (max_n * group + rows - 1) / rows;
    const int64_t n_pairs = pairs_of(rows);
    const int64_t rounds = (n_pairs + slots - 1) / slots;
    p->paired = n_pairs >= slots && rounds * slots * 20 <= n_pairs * 21;
    p->gx = (p->paired ? (max_blocks + 1) / 2 : max_blocks) * hkv;
    for (int32_t b = 0; b < batch; ++b) p->blocks += (static_cast<int64_t>(h_new_lens[b]) * group + rows - 1) / rows;
    // Up to 64 sequences: blocks ordered over the whole batch (a sequence at a
    // time leaves the last one's long blocks to the end of the launch, and
    // gives every sequence as many work-groups as the longest needs)
    if (batch > 1 && batch <= kMaxSorted) {
        p->order = kSorted;
        p->grid_x = p->blocks * hkv;
    } else {
        p->order = p->paired ? kPairs : kPerSequence;
        p->grid_x = p->gx;
        p->grid_y = batch;
    }
}

}  // namespace mw

// One launch of 8- or 4-wave blocks as planned by prefill_prepare.
static mw_status launch_plain(const mw_prefill_args &a, const PrefillPlan &pl, hipStream_t s, mw_timing *timing) {
    mw_status st = timing_begin(timing, s);
    if (st != MW_OK) return st;
    if (pl.grid_x > 0) {
        auto kernel = pl.waves == 4 ? (pl.table_in_lds ? k_prefill_attn<true, 4> : k_prefill_attn<false, 4>)
                                    : (pl.table_in_lds ? k_prefill_attn<true, 8> : k_prefill_attn<false, 8>);
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(pl.grid_x), pl.grid_y), dim3(64 * pl.waves), 0, s,
                           a.pool->k, a.pool->v, static_cast<const uint16_t *>(a.d_q),
                           static_cast<uint16_t *>(a.d_out), a.d_qo_indptr, a.d_prefix_lens, a.d_block_table,
                           a.bt_stride, a.batch, pl.hkv, pl.group, a.pool->desc.num_pages, pl.scale_log2, pl.order);
        st = check_launch("k_prefill_attn");
        if (st != MW_OK) return st;
    }
    st = timing_kernel_done(timing, s);
    timing_end(timing);
    return st;
}

extern "C" mw_status mw_prefill_attn(const mw_kv_pool *pool, const mw_attn_shape *shape, int32_t batch,
                                     const int32_t *h_new_lens, const int32_t *h_prefix_lens,
                                     const int32_t *d_qo_indptr, const int32_t *d_prefix_lens,
                                     const int32_t *d_block_table, int32_t bt_stride, const void *d_q,
                                     void *d_out, mw_stream stream, mw_timing *timing) {
    const char *who = "mw_prefill_attn";
    if (!shape) return fail(MW_ERR_INVALID_ARG, "%s: bad arguments", who);
    const mw_prefill_args a{pool,          *shape,        batch,     h_new_lens, h_prefix_lens, d_qo_indptr,
                            d_prefix_lens, d_block_table, bt_stride, d_q,        d_out};
    hipStream_t s = static_cast<hipStream_t>(stream);
    PrefillPlan pl;
    mw_status st = prefill_prepare(&a, stream_cus(s), true, &pl, who);
    if (st != MW_OK) return st;
    return launch_plain(a, pl, s, timing);
}

extern "C" mw_status mw_prefill_workspace_size(const mw_attn_shape *shape, int32_t batch, const int32_t *h_new_lens,
                                               const int32_t *h_prefix_lens, int32_t num_cus, size_t *bytes) {
    const char *who = "mw_prefill_workspace_size";
    if (!shape || !bytes || batch < 0 || batch > 65535 || num_cus < 0 || (batch > 0 && (!h_new_lens || !h_prefix_lens)))
        return fail(MW_ERR_INVALID_ARG, "%s: bad arguments", who);
    if (shape->head_dim != kHeadDim) return fail(MW_ERR_UNSUPPORTED, "%s: head_dim must be 128", who);
    if (shape->num_kv_heads < 1 || shape->num_q_heads < 1 || shape->num_q_heads % shape->num_kv_heads)
        return fail(MW_ERR_INVALID_ARG, "%s: num_q_heads must be a multiple of num_kv_heads", who);
    for (int32_t b = 0; b < batch; ++b)
        if (h_new_lens[b] < 0 || h_prefix_lens[b] < 0 ||
            static_cast<int64_t>(h_new_lens[b]) + h_prefix_lens[b] > INT32_MAX - 64)
            return fail(MW_ERR_INVALID_ARG, "%s: sequence %d: bad lengths", who, b);
    PrefillPlan pl{};
    pl.hkv = shape->num_kv_heads;
    pl.group = shape->num_q_heads / pl.hkv;
    // the split runs where the launch takes 4-wave blocks (as in prefill_prepare);
    // without a CU count, size for any stream
    pl.waves = num_cus == 0 || prefill_pairs(batch, h_new_lens, pl.group, 256) * pl.hkv < num_cus ? 4 : 8;
    prefill_split_plan(batch, h_new_lens, h_prefix_lens, shape->num_q_heads, num_cus, &pl);
    *bytes = pl.split_bytes;
    return MW_OK;
}

extern "C" mw_status mw_prefill_attn_ws(const mw_kv_pool *pool, const mw_attn_shape *shape, int32_t batch,
                                        const int32_t *h_new_lens, const int32_t *h_prefix_lens,
                                        const int32_t *d_qo_indptr, const int32_t *d_prefix_lens,
                                        const int32_t *d_block_table, int32_t bt_stride, const void *d_q,
                                        void *d_out, void *d_workspace, size_t workspace_bytes, mw_stream stream,
                                        mw_timing *timing) {
    const char *who = "mw_prefill_attn_ws";
    if (!shape) return fail(MW_ERR_INVALID_ARG, "%s: bad arguments", who);
    const mw_prefill_args a{pool,          *shape,        batch,     h_new_lens, h_prefix_lens, d_qo_indptr,
                            d_prefix_lens, d_block_table, bt_stride, d_q,        d_out};
    hipStream_t s = static_cast<hipStream_t>(stream);
    PrefillPlan pl;
    const int64_t cus = stream_cus(s);
    mw_status st = prefill_prepare(&a, cus, true, &pl, who);
    if (st != MW_OK) return st;
    const int64_t n_big = prefill_big_units(batch, h_new_lens, h_prefix_lens, cus, pl);
    if ((pl.waves == 8 && n_big == 0) || pl.gx == 0)
        return launch_plain(a, pl, s, timing);
    if (n_big > 0) {
        const int64_t units = pl.blocks * pl.hkv;
        st = timing_begin(timing, s);
        if (st != MW_OK) return st;
        auto kernel = pl.table_in_lds ? k_prefill_mixed<true> : k_prefill_mixed<false>;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_big + 2 * (units - n_big))), dim3(512), 0, s, pool->k,
                           pool->v, static_cast<const uint16_t *>(d_q), static_cast<uint16_t *>(d_out), d_qo_indptr,
                           d_prefix_lens, d_block_table, bt_stride, batch, pl.hkv, pl.group, pool->desc.num_pages,
                           pl.scale_log2, pl.order, static_cast<int>(n_big));
        st = check_launch("k_prefill_mixed");
        if (st != MW_OK) return st;
        st = timing_kernel_done(timing, s);
        timing_end(timing);
        return st;
    }
    prefill_split_plan(batch, h_new_lens, h_prefix_lens, shape->num_q_heads, cus, &pl);
    if (pl.body != kBodyDual) {
        if (pl.body == kBodyEight) {
            st = prefill_prepare(&a, cus, false, &pl, who);
            if (st != MW_OK) return st;
        }
        return launch_plain(a, pl, s, timing);
    }
    const bool cut = pl.pieces > 1;
    if (cut && (!d_workspace || !aligned16(d_workspace) || workspace_bytes < pl.split_bytes))
        return fail(MW_ERR_INVALID_ARG, "%s: the split needs a 16-byte aligned workspace of %zu bytes (got %zu)",
                    who, pl.split_bytes, workspace_bytes);
    int64_t max_n = 0;
    for (int32_t b = 0; b < batch; ++b) max_n = std::max<int64_t>(max_n, h_new_lens[b]);
    // single blocks, over the whole batch or a sequence at a time
    const int64_t gx = (pl.order == kSorted ? pl.blocks : (max_n * pl.group + 127) / 128) * pl.hkv;
    const int order = pl.order == kSorted ? kSorted : kPerSequence;
    if (gx * pl.pieces > 0x7fffffff) return fail(MW_ERR_UNSUPPORTED, "%s: grid too large", who);
    st = timing_begin(timing, s);
    if (st != MW_OK) return st;
    float *ws_o = static_cast<float *>(d_workspace);
    float2 *ws_ml = reinterpret_cast<float2 *>(static_cast<char *>(d_workspace) +
                                               static_cast<size_t>(pl.pieces) * pl.rows * shape->num_q_heads *
                                                   kHeadDim * 4);
    auto kernel = cut ? (pl.table_in_lds ? k_prefill_dual<true, true> : k_prefill_dual<false, true>)
                      : (pl.table_in_lds ? k_prefill_dual<true, false> : k_prefill_dual<false, false>);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(gx * pl.pieces), pl.grid_y), dim3(512), 0, s, pool->k,
                       pool->v, static_cast<const uint16_t *>(d_q), static_cast<uint16_t *>(d_out), d_qo_indptr,
                       d_prefix_lens, d_block_table, bt_stride, batch, pl.hkv, pl.group, pool->desc.num_pages,
                       pl.scale_log2, order, ws_o, ws_ml, pl.rows, pl.piece_tiles, pl.pieces);
    st = check_launch("k_prefill_dual");
    if (st != MW_OK) return st;
    st = timing_kernel_done(timing, s);
    if (st != MW_OK) return st;
    if (!cut) {
        timing_end(timing);
        return MW_OK;
    }
    const int64_t gm = (max_n * shape->num_q_heads + 31) / 32;
    hipLaunchKernelGGL(k_prefill_merge, dim3(static_cast<unsigned>(gm), batch), dim3(256), 0, s, ws_o, ws_ml,
                       static_cast<uint16_t *>(d_out), d_qo_indptr, d_prefix_lens, shape->num_q_heads,
                       pl.group, pl.rows, pl.piece_tiles, pl.pieces);
    st = check_launch("k_prefill_merge");
    if (st != MW_OK) return st;
    st = timing_kernel_done(timing, s);
    timing_end(timing);
    return st;
}
