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
               const int32_t *__restrict__ bt, int bt_stride, int batch, Divisor hkv, Divisor group, int num_pages,
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
               const int32_t *__restrict__ bt, int bt_stride, int batch, Divisor hkv, Divisor group, int num_pages,
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
                const int32_t *__restrict__ bt, int bt_stride, int batch, Divisor hkv, Divisor group, int num_pages,
                float scale_log2, int order, int n_big) {
    // Device pass only: clang's host pass, whose code for a kernel is a stub in any
    // case, refuses the second use of an instantiation that k_prefill_attn has used
    // ("no matching function for call to 'prefill_block' ... candidate template
    // ignored: substitution failure", with no reason given).
#ifdef __HIP_DEVICE_COMPILE__
    __shared__ __attribute__((aligned(1024))) uint16_t s_k[4 * TILE];
    __shared__ __attribute__((aligned(1024))) uint16_t s_v[4 * TILE];
    __shared__ int32_t s_bt[kBtCache];
    // past n_big, kv heads fastest, then the unit's two halves
    const int x = blockIdx.x, over = x - n_big;
    const bool big = over < 0;
    const int row = big ? 0 : over / hkv, half = row & 1;
    const int unit = big ? x : n_big + over - (row + 1) / 2 * hkv;
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

// The work-groups of one way to launch a call, from its lengths: `n` of them in
// a grid of `grid`, or `sorted_grid` in length order (the rest find no work), of
// `tiles` key tiles in all; tiles of the longest, of the lightest and of the last
// sequence's longest.
struct Jobs {
    int64_t n = 0, grid = 0, sorted_grid = 0;
    double tiles = 0, longest = 0, lightest = 1e30, last = 0;
};

// What a work-group takes (us): around its tiles and per tile, alone on its CU
// and on a full partition, on 256 busy CUs; `clock`: the share of the time per
// tile that the clock takes off it as fewer CUs are busy; to find its block in a
// batch in length order; a work-group without work.  How a launch of more
// work-groups than slots ends: shares of the lightest one (end_lightest), of the
// last round's idle part, in lightest (end_round) and in what the mean has more
// (end_mean), of how much the last sequence's longest block exceeds the lightest
// (end_last); `uneven`: by the times of launches of several rounds, work-groups go
// to groups of CUs (8 dies, 4 groups each) in turn and not to the CU that is free
// first, so that with the heaviest first the first group gets 16 x (longest -
// lightest) / cus more tiles a CU than the mean; the share of twice that which
// shows (`uneven_batch`: of sequences one after the other).
struct BodyCost {
    double around_alone, per_alone, around, per, clock, empty, search, end_lightest, end_round, end_mean, end_last, late,
        uneven, uneven_batch;
};
// Fitted by least squares of the log error to 5000 calls (1 to 16 sequences of 1
// to 8192 new tokens over 0 to 131072, groups of 1 to 16, 32 to 256 CUs, each
// body, order and number of pieces measured on each: 57000 launches, 4%, 4% and
// 6% off in the median).  The cheapest by these is 1.8% slower than the fastest
// measured of each call (geometric mean, calls of 8 us and more).  Fitted to
// prefixes up to 28672 only, without the clock, the empty work-groups' places and
// the uneven groups it was 2.6%, and 2048 tokens over 16384 on 192 CUs took 734
// us, now 615.
constexpr BodyCost kCost4{4.5, 1.285, 4.25, 1.6, 0.144, 1.04, 1.03, 0.326, 0.229, 0.325, 0.234, 0.17, 0.39, 0.04};    // 2 work-groups per CU
constexpr BodyCost kCost8{6.2, 1.48, 5.5, 1.49, 0.188, 1.6, 1.1, 0.01, 0.8, 0.0, 0.18, 0.04, 0.57, 0.635};
constexpr BodyCost kCostDual{5.55, 0.804, 5.8, 0.838, 0.215, 1.6, 1.56, 0.0, 0.723, 0.253, 0.0, 0.48, 0.15, 0.6};
constexpr double kMergeUs = 5.6, kMergeBytesPerUs = 8.7e6;  // the second launch, and its partials' way out and back

double at_clock(double clock, int64_t busy) {
    return 1.0 - clock * (1.0 - static_cast<double>(std::min<int64_t>(busy, 256)) / 256);
}

// Time of a launch (us, without what is common to all), for CUs that hold
// per_cu work-groups each.  Work-groups without work take a place all the same:
// 62 work-groups among 76 on 64 CUs take two rounds (554 us; in length order,
// which leaves the empty ones out, 292).
double launch_us(const BodyCost &c, const Jobs &j, int64_t cus, int per_cu, bool sorted, bool one_sequence) {
    if (j.n == 0) return 0.0;
    const int64_t slots = per_cu * cus, grid = sorted ? j.sorted_grid : j.grid;
    const double search = sorted ? c.search : 0.0;
    const double empty = c.empty * (grid - j.n) / slots;
    const double full = c.per * at_clock(c.clock, cus), alone = c.per_alone * at_clock(c.clock, std::min(j.n, cus));
    // the longest work-group, alone on its CU or beside the heaviest of those
    // that no longer find an empty CU
    double us = c.around_alone + search + alone * j.longest;
    if (grid <= cus) return us + empty;
    if (per_cu == 2 && j.n > cus) {
        const double beside = std::max(j.lightest, j.longest - (j.longest - j.lightest) * cus / j.n);
        us = std::max(us, c.around + search + full * beside + alone * (j.longest - beside));
    }
    // the even share, and past one round what the last one leaves idle
    double share = ((c.around + search) * j.n + full * j.tiles) / slots + empty;
    if (grid > slots) {
        const double lightest = c.around + full * j.lightest, spread = full * (j.longest - j.lightest);
        const double idle = std::clamp(std::ceil(static_cast<double>(grid) / slots) - static_cast<double>(j.n) / slots, 0.0, 1.0);
        const bool batch_order = !sorted && !one_sequence;
        share += c.end_lightest * lightest +
                 idle * (c.end_round * lightest + c.end_mean * full * (j.tiles / j.n - j.lightest)) +
                 (batch_order ? c.uneven_batch : c.uneven) * spread * 32 / slots;
        if (batch_order) share += c.end_last * (c.around + full * (j.last - j.lightest));
    }
    return std::max(us, share) + (grid > j.n && grid > slots ? c.late : 0.0);
}

// Time of a launch of 8-wave pairs (blocks nqb-1-i and i).  Taken only where they
// are alike (to 12%) and fill the rounds of the CUs (to 5%): every CU then gets the
// same, where single blocks, heaviest first, leave uneven CUs (2048 tokens of
// 32/8 heads on 64 CUs 107.7 us, single blocks 116.8; 4096 on 32 750 and 787);
// elsewhere a pair's length makes the last round (4096 on 96, 2.7 rounds: 282 and
// 267).  With these constants the choice is 0.8% slower than the faster one on
// the 273 measured calls that have such pairs.
double pairs_us(const Jobs &j, int64_t cus) {
    const int64_t rounds = (j.n + cus - 1) / cus;
    if (j.n < cus || rounds * cus * 20 > j.n * 21 || j.longest - j.lightest > 0.12 * j.longest) return INFINITY;
    const double per = 1.46 * at_clock(kCost8.clock, cus);
    return std::max(11.0 + per * j.longest, (11.0 * j.n + per * j.tiles) / cus);
}

// A call's work-groups on blocks of 256 rows, one each (one8) and two each, nqb-1-i
// and i (two8), and on blocks of 128 rows (one4); most8, most4: blocks of the
// sequence with the most.
struct CallJobs {
    Jobs one8, two8, one4;
    int64_t most8 = 0, most4 = 0;
};

CallJobs count_jobs(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int hkv, int group) {
    CallJobs c;
    const auto add = [](Jobs *j, int64_t n, double tiles, double longest, double lightest) {
        j->n += n;
        j->tiles += tiles;
        j->longest = std::max(j->longest, longest);
        j->lightest = std::min(j->lightest, lightest);
        j->last = longest;
    };
    for (int32_t b = 0; b < batch; ++b) {
        const int64_t n = h_new_lens[b], r = h_prefix_lens[b];
        if (n == 0) continue;
        const double last = static_cast<double>((r + n + 63) / 64);
        const int64_t n8 = (n * group + 255) / 256, n4 = (n * group + 127) / 128;
        const double first8 = prefill_block_tiles<int64_t>(r, n, 0, 256, group);
        const double first4 = prefill_block_tiles<int64_t>(r, n, 0, 128, group);
        const double pair = n8 > 1 ? first8 + last : last;
        add(&c.one8, n8 * hkv, n8 * hkv * (first8 + last) / 2, last, first8);
        add(&c.two8, (n8 + 1) / 2 * hkv, n8 * hkv * (first8 + last) / 2, pair, n8 % 2 == 0 ? pair : (first8 + last) / 2);
        add(&c.one4, n4 * hkv, n4 * hkv * (first4 + last) / 2, last, first4);
        c.most8 = std::max(c.most8, n8);
        c.most4 = std::max(c.most4, n4);
    }
    c.one8.grid = c.most8 * hkv * batch;
    c.one4.grid = c.most4 * hkv * batch;
    c.one8.sorted_grid = c.one8.n;
    c.one4.sorted_grid = c.one4.n;
    return c;
}

void set_launch(PrefillPlan *p, int waves, int order, const CallJobs &c) {
    const Jobs &j = waves == 8 ? c.one8 : c.one4;
    const int64_t most = waves == 8 ? c.most8 : c.most4;
    p->waves = waves;
    p->order = order;
    p->gx = order == kSorted ? j.n : (order == kPairs ? (most + 1) / 2 : most) * p->hkv;
    p->gy = order == kSorted ? 1 : p->batch;
}

bool sortable(int32_t batch) { return batch > 1 && batch <= kMaxSorted; }

// Plans a call as one launch of 8- or, if allowed, 4-wave blocks, the cheapest of
// their orders; returns its time.
double choose_plain(const CallJobs &c, int64_t cus, bool allow_small, PrefillPlan *p) {
    double best = INFINITY;
    const auto take = [&](double us, int waves, int order) {
        if (us >= best) return;
        best = us;
        set_launch(p, waves, order, c);
    };
    const bool one = p->batch == 1;
    take(launch_us(kCost8, c.one8, cus, 1, false, one), 8, kPerSequence);
    take(pairs_us(c.two8, cus), 8, kPairs);
    if (sortable(p->batch)) take(launch_us(kCost8, c.one8, cus, 1, true, one), 8, kSorted);
    if (!allow_small) return best;
    take(launch_us(kCost4, c.one4, cus, 2, false, one), 4, kPerSequence);
    if (sortable(p->batch)) take(launch_us(kCost4, c.one4, cus, 2, true, one), 4, kSorted);
    return best;
}

// Units (block, kv head) that a call of 256-row blocks on `cus` CUs runs as such
// when the rest, its last and partial round, goes to dual blocks; 0: not such a
// call, which takes `plain` us as one launch of one body.  Blocks taken longest
// first fill CUs evenly when they differ much in length (a prompt without a
// prefix), so only calls whose lightest block has at least half the tiles of the
// heaviest are treated.  There the last round costs a whole block's time for any
// fraction f of a round; as dual blocks it costs a little over half a block's while
// f <= 1/2.  Simulated over 2.3 to 5.3 rounds the launch gets 5-17% shorter, and
// past f = 1/2 longer.  Measured: the 70B layer's 2048-token chunk over 6144 cached
// tokens on 96 CUs (5.33 rounds) next to its decode, 958 -> 911 us a step; on blocks
// of 2 tiles, where starts are all, 4-wave blocks 13.8 us and this 20.8.
int64_t big_units(const CallJobs &c, int64_t cus, const PrefillPlan &p, double plain) {
    const int64_t units = c.one8.n, whole = units / cus * cus;
    if (whole < 2 * cus || whole == units || 2 * (units - whole) > cus) return 0;
    if (2 * c.one8.lightest < c.one8.longest) return 0;
    // more than one sequence: in length order, where that pays by itself
    if (p.batch > 1 && (!sortable(p.batch) || launch_us(kCost8, c.one8, cus, 1, true, false) >
                                                  launch_us(kCost8, c.one8, cus, 1, false, false)))
        return 0;
    const double rest = c.one8.lightest + (c.one8.longest - c.one8.lightest) * (units - whole) / units;
    const double us = whole / cus * (kCost8.around + (p.batch > 1 ? kCost8.search : 0.0) +
                                     kCost8.per * at_clock(kCost8.clock, cus) * c.one8.tiles / units) +
                      kCostDual.around_alone + kCostDual.per_alone * at_clock(kCostDual.clock, cus) * rest;
    return us < plain ? whole / p.hkv * p.hkv : 0;
}

}  // namespace

namespace mw {

void prefill_split_plan(int32_t batch, const int32_t *h_new_lens, const int32_t *h_prefix_lens, int hq,
                        int64_t cus, PrefillPlan *p, size_t workspace_bytes) {
    p->pieces = 1;
    p->piece_tiles = 0;
    p->split_bytes = 0;
    p->rows = 0;
    p->big_units = 0;
    p->dual = false;
    p->batch = batch;
    for (int32_t b = 0; b < batch; ++b) p->rows += h_new_lens[b];
    const CallJobs c = count_jobs(batch, h_new_lens, h_prefix_lens, p->hkv, p->group);
    const Jobs &j = c.one4;
    if (j.n == 0) {
        set_launch(p, 8, kPerSequence, c);
        return;
    }
    const int max_nt = static_cast<int>(j.longest), min_nt = static_cast<int>(j.lightest);
    const auto bytes_for = [&](int pieces) {
        return pieces > 1 ? static_cast<size_t>(pieces) * p->rows * hq * (kHeadDim * 4 + 8) : 0;
    };
    if (cus <= 0) {  // sizing: the most pieces any stream's plan can take
        p->piece_tiles = kPrefillMinPieceTiles;
        p->pieces = prefill_pieces(max_nt, kPrefillMinPieceTiles, kPrefillMaxPieces);
        p->split_bytes = bytes_for(p->pieces);
        return;
    }
    const double plain = choose_plain(c, cus, true, p);
    p->big_units = big_units(c, cus, *p, plain);
    if (p->big_units > 0) {
        set_launch(p, 8, batch == 1 ? kPerSequence : kSorted, c);
        return;
    }
    // Dual blocks, whole or in pieces.  Only launches of few blocks are cut: two
    // blocks per CU and more even out by themselves.  Two kinds always are, as
    // every caller's workspace provides for: fewer than two blocks per CU of 96
    // tiles and more, and blocks of 10 tiles and more of which four pieces each
    // fit the CUs at once (whole ones are up to 2 us faster at 10 to 13 tiles, and
    // 1 to 5 us slower from 15).
    const bool cuttable = c.two8.n < cus && j.n < 2 * cus && bytes_for(2) <= workspace_bytes;
    const bool must_cut = cuttable && (max_nt >= 96 || (4 * j.n <= cus && max_nt >= 10));
    double best = must_cut ? INFINITY : plain;
    // the blocks' tiles and how many blocks have them, from up to 64 blocks of a
    // sequence, the lightest and the longest among them.  512 hold every cuttable
    // call of 256 CUs; what a larger one has beyond counts with the last
    struct Length {
        int tiles;
        double blocks;
    } lengths[512];
    int kinds = 0;
    for (int32_t b = 0; cuttable && b < batch; ++b) {
        const int64_t n = h_new_lens[b], r = h_prefix_lens[b], nqb = (n * p->group + 127) / 128;
        const int64_t taken = std::min<int64_t>(nqb, 64);
        for (int64_t i = 0; i < taken; ++i) {
            const int64_t q = taken > 1 ? i * (nqb - 1) / (taken - 1) : 0;
            const int nt = prefill_block_tiles<int64_t>(r, n, q, 128, p->group);
            if (kinds == 0 || (lengths[kinds - 1].tiles != nt && kinds < 512)) lengths[kinds++] = {nt, 0.0};
            lengths[kinds - 1].blocks += static_cast<double>(nqb * p->hkv) / taken;
        }
    }
    for (int k = must_cut ? 2 : 1; k <= (cuttable ? kPrefillMaxPieces : 1); ++k) {
        const int pt = std::max(kPrefillMinPieceTiles, (max_nt + k - 1) / k);
        if (k > 1 && (pt >= max_nt || bytes_for(prefill_pieces(max_nt, pt, kPrefillMaxPieces)) > workspace_bytes)) break;
        Jobs jk = j;
        double merge = 0.0;
        if (k > 1) {
            jk.grid *= k;
            jk.sorted_grid *= k;
            jk.longest = 0;
            jk.lightest = max_nt;
            double found = 0.0;
            for (int i = 0; i < kinds; ++i) {
                const int nt = lengths[i].tiles, np = prefill_pieces(nt, pt, k);
                found += np * lengths[i].blocks;
                jk.longest = std::max<double>(jk.longest, (nt + np - 1) / np);
                jk.lightest = std::min<double>(jk.lightest, nt / np);
            }
            jk.n = static_cast<int64_t>(found + 0.5);
            jk.last = std::min(j.last, jk.longest);
            const double cut = std::min(1.0, static_cast<double>(max_nt - pt) / (max_nt - min_nt + 1));
            merge = kMergeUs + cut * 2.0 * bytes_for(prefill_pieces(max_nt, pt, k)) / kMergeBytesPerUs;
        }
        for (int sorted = 0; sorted <= (sortable(batch) ? 1 : 0); ++sorted) {
            const double us = launch_us(kCostDual, jk, cus, 1, sorted != 0, batch == 1) + merge;
            if (us >= best) continue;
            best = us;
            p->dual = true;
            p->piece_tiles = k > 1 ? pt : 0;
            set_launch(p, 4, sorted ? kSorted : kPerSequence, c);
        }
    }
    if (!p->dual || p->piece_tiles == 0) return;
    p->pieces = prefill_pieces(max_nt, p->piece_tiles, kPrefillMaxPieces);
    p->split_bytes = bytes_for(p->pieces);
}

mw_status prefill_fit_workspace(const mw_prefill_args *a, int64_t cus, PrefillPlan *p, const void *ws, size_t bytes,
                                const char *who) {
    const size_t usable = ws && aligned16(ws) ? bytes : 0;
    if (usable >= p->split_bytes) return MW_OK;
    const int hq = p->hkv * p->group;
    const int pieces = prefill_base_pieces(a->batch, a->h_new_lens, a->h_prefix_lens, p->hkv, p->group, cus);
    const size_t least =
        pieces > 1 ? static_cast<size_t>(pieces) * p->rows * hq * (kHeadDim * 4 + 8) : 0;
    if (usable < std::min(least, p->split_bytes))
        return fail(MW_ERR_INVALID_ARG, "%s: the split needs a 16-byte aligned workspace of %zu bytes (got %zu)", who,
                    p->split_bytes, ws && !aligned16(ws) ? size_t{0} : bytes);
    prefill_split_plan(a->batch, a->h_new_lens, a->h_prefix_lens, hq, cus, p, usable);
    return MW_OK;
}

mw_status prefill_prepare(const mw_prefill_args *a, int64_t cus, bool allow_small, PrefillPlan *p, const char *who,
                          bool split) {
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
    *p = PrefillPlan{};
    p->hkv = shape->num_kv_heads;
    p->group = shape->num_q_heads / shape->num_kv_heads;
    p->batch = a->batch;
    p->pieces = 1;
    p->table_in_lds = max_pages <= kBtCache;
    p->scale_log2 = shape->scale * kLog2e;
    if (split)
        prefill_split_plan(a->batch, a->h_new_lens, a->h_prefix_lens, shape->num_q_heads, cus, p);
    else
        choose_plain(count_jobs(a->batch, a->h_new_lens, a->h_prefix_lens, p->hkv, p->group), cus, allow_small, p);
    if (p->gx * p->pieces > 0x7fffffff) return fail(MW_ERR_UNSUPPORTED, "%s: grid too large", who);
    return MW_OK;
}

}  // namespace mw

// One launch of 8- or 4-wave blocks as planned by prefill_prepare.
static mw_status launch_plain(const mw_prefill_args &a, const PrefillPlan &pl, hipStream_t s, mw_timing *timing) {
    mw_status st = timing_begin(timing, s);
    if (st != MW_OK) return st;
    if (pl.gx > 0) {
        auto kernel = pl.waves == 4 ? (pl.table_in_lds ? k_prefill_attn<true, 4> : k_prefill_attn<false, 4>)
                                    : (pl.table_in_lds ? k_prefill_attn<true, 8> : k_prefill_attn<false, 8>);
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(pl.gx), pl.gy), dim3(64 * pl.waves), 0, s,
                           a.pool->k, a.pool->v, static_cast<const uint16_t *>(a.d_q),
                           static_cast<uint16_t *>(a.d_out), a.d_qo_indptr, a.d_prefix_lens, a.d_block_table,
                           a.bt_stride, a.batch, Divisor(pl.hkv), Divisor(pl.group), a.pool->desc.num_pages, pl.scale_log2, pl.order);
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
    mw_status st = prefill_prepare(&a, cus, true, &pl, who, true);
    if (st == MW_OK) st = prefill_fit_workspace(&a, cus, &pl, d_workspace, workspace_bytes, who);
    if (st != MW_OK) return st;
    if (pl.big_units > 0) {
        const int64_t n_big = pl.big_units, units = pl.gx;
        st = timing_begin(timing, s);
        if (st != MW_OK) return st;
        auto kernel = pl.table_in_lds ? k_prefill_mixed<true> : k_prefill_mixed<false>;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_big + 2 * (units - n_big))), dim3(512), 0, s, pool->k,
                           pool->v, static_cast<const uint16_t *>(d_q), static_cast<uint16_t *>(d_out), d_qo_indptr,
                           d_prefix_lens, d_block_table, bt_stride, batch, Divisor(pl.hkv), Divisor(pl.group), pool->desc.num_pages,
                           pl.scale_log2, pl.order, static_cast<int>(n_big));
        st = check_launch("k_prefill_mixed");
        if (st != MW_OK) return st;
        st = timing_kernel_done(timing, s);
        timing_end(timing);
        return st;
    }
    if (!pl.dual) return launch_plain(a, pl, s, timing);
    const bool cut = pl.pieces > 1;
    int64_t max_n = 0;
    for (int32_t b = 0; b < batch; ++b) max_n = std::max<int64_t>(max_n, h_new_lens[b]);
    st = timing_begin(timing, s);
    if (st != MW_OK) return st;
    float *ws_o = static_cast<float *>(d_workspace);
    float2 *ws_ml = reinterpret_cast<float2 *>(static_cast<char *>(d_workspace) +
                                               static_cast<size_t>(pl.pieces) * pl.rows * shape->num_q_heads *
                                                   kHeadDim * 4);
    auto kernel = cut ? (pl.table_in_lds ? k_prefill_dual<true, true> : k_prefill_dual<false, true>)
                      : (pl.table_in_lds ? k_prefill_dual<true, false> : k_prefill_dual<false, false>);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(pl.gx * pl.pieces), pl.gy), dim3(512), 0, s, pool->k,
                       pool->v, static_cast<const uint16_t *>(d_q), static_cast<uint16_t *>(d_out), d_qo_indptr,
                       d_prefix_lens, d_block_table, bt_stride, batch, Divisor(pl.hkv), Divisor(pl.group), pool->desc.num_pages,
                       pl.scale_log2, pl.order, ws_o, ws_ml, pl.rows, pl.piece_tiles, pl.pieces);
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
