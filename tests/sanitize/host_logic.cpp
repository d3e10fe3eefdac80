// The library's host logic on randomised inputs, for a build with
// AddressSanitizer and UndefinedBehaviorSanitizer: the decode and prefill
// launch planners, the dual prefill blocks' step order and the LDS regions of
// their merge, the page allocator and the estimator (with the prefill launch
// simulation).  Nothing here launches a kernel or touches a GPU: the device pointers are host addresses
// the planners only check for alignment.  Prints "ok" when every check holds.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "mw_internal.h"
#include "prefill_layout.h"
#include "prefill_schedule.h"

namespace {

uint64_t g_state = 0x9E3779B97F4A7C15ull;
uint32_t next_u32() {  // xorshift64*
    g_state ^= g_state >> 12;
    g_state ^= g_state << 25;
    g_state ^= g_state >> 27;
    return static_cast<uint32_t>((g_state * 0x2545F4914F6CDD1Dull) >> 32);
}
int uniform(int lo, int hi) { return lo + static_cast<int>(next_u32() % static_cast<uint32_t>(hi - lo + 1)); }

int g_fail = 0;
void check(bool ok, const char *what, int it) {
    if (!ok) {
        std::fprintf(stderr, "check failed at iteration %d: %s (%s)\n", it, what, mw_last_error());
        ++g_fail;
    }
}

alignas(256) unsigned char g_fake[4096];  // stands in for device buffers: never dereferenced

void planners() {
    const int hkvs[4] = {1, 2, 4, 8};
    const int chunks[10] = {0, -1, 8, 16, 32, 64, 128, 256, 5, 300};
    for (int it = 0; it < 3000; ++it) {
        const int hkv = hkvs[uniform(0, 3)];
        const int group = uniform(1, 17);
        mw_kv_pool_desc desc{uniform(1, 1 << 14), 16, hkv, 128};
        mw_kv_pool *pool = nullptr;
        check(mw_kv_pool_create(&desc, g_fake, g_fake, &pool) == MW_OK, "pool create", it);
        const mw_attn_shape shape{hkv * group, hkv, 128, 0.0883883f};
        // decode: lengths on page edges, long and short, occasionally invalid;
        // a quarter of the batches are a few long sequences (equal or not),
        // whose segments the balanced split may pad to whole ranges
        const bool few_long = uniform(0, 3) == 0;
        const int batch = few_long ? uniform(1, 6) : uniform(0, 300);
        const bool equal = few_long && uniform(0, 1) == 0;
        std::vector<int32_t> lens(batch);
        int max_len = 1;
        for (int b = 0; b < batch; ++b) {
            const int kind = uniform(0, 9);
            if (few_long)
                lens[b] = equal && b > 0 ? lens[0] : uniform(2000, 70000);
            else
                lens[b] = kind == 0 ? 16 * uniform(1, 64) : kind == 1 ? uniform(1, 17) : uniform(1, 70000);
            max_len = lens[b] > max_len ? lens[b] : max_len;
        }
        if (batch > 0 && uniform(0, 49) == 0) lens[uniform(0, batch - 1)] = uniform(-3, 0);
        const int chunk = chunks[uniform(0, 9)];
        size_t bytes = 0;
        const mw_status st = mw_decode_workspace_size(&shape, batch, lens.data(), chunk, &bytes);
        const int stride = (max_len + 15) / 16 + uniform(-1, 3);
        mw_decode_args a{pool, shape, batch, lens.data(), reinterpret_cast<int32_t *>(g_fake),
                         reinterpret_cast<int32_t *>(g_fake), stride, g_fake, g_fake, g_fake, bytes, chunk};
        const int cus = uniform(0, 1) ? 8 * uniform(1, 32) : 0;
        mw::DecodePlan dp;
        const mw_status st2 = mw::decode_prepare(&a, cus, &dp, "decode_prepare");
        if (st == MW_OK && st2 == MW_OK) {
            check(dp.bytes <= bytes, "the workspace size covers the split of every CU count", it);
            check(dp.units >= 0 && dp.slots >= dp.units, "plan counts", it);
            check(dp.off_ml <= dp.off_meta && dp.off_meta <= dp.bytes, "workspace layout", it);
            // per-sequence chunk bases, or the balanced split's per-slot done flags
            const size_t meta = dp.per_unit > 0 ? static_cast<size_t>(dp.slots) * 4 : static_cast<size_t>(batch) * 4;
            check(dp.off_meta + meta <= dp.bytes, "workspace holds the flags", it);
            if (dp.aligned) {  // segments padded to whole ranges: one piece of one segment per unit
                int64_t padded = 0;
                for (int b = 0; b < batch; ++b)
                    padded += (static_cast<int64_t>(lens[b] + 15) / 16 + dp.per_unit - 1) / dp.per_unit * dp.per_unit;
                check(dp.per_unit >= 16 && dp.total == padded * hkv && dp.units * dp.per_unit == dp.total,
                      "aligned split covers every padded segment in whole ranges", it);
                check(cus > 0 && dp.units <= std::min<int64_t>(cus, 256), "aligned split within a unit per CU", it);
            }
        }
        if (st != MW_OK) check(st2 != MW_OK, "a refused size is refused by the plan too", it);
        // prefill: varlen batches, prefixes, tables that are too short
        const int pb = uniform(0, 8);
        std::vector<int32_t> nl(pb), pl(pb);
        int max_tok = 1;
        for (int b = 0; b < pb; ++b) {
            nl[b] = uniform(0, 9) == 0 ? 0 : uniform(1, 5000);
            pl[b] = uniform(0, 3) == 0 ? 0 : uniform(0, 80000);
            max_tok = nl[b] + pl[b] > max_tok ? nl[b] + pl[b] : max_tok;
        }
        const int pstride = (max_tok + 15) / 16 + uniform(-1, 2);
        mw_prefill_args p{pool, shape, pb, nl.data(), pl.data(), reinterpret_cast<int32_t *>(g_fake),
                          reinterpret_cast<int32_t *>(g_fake), reinterpret_cast<int32_t *>(g_fake), pstride,
                          g_fake, g_fake};
        mw::PrefillPlan pp;
        const int pcus = 8 * uniform(1, 32);
        if (mw::prefill_prepare(&p, pcus, uniform(0, 1), &pp, "prefill_prepare") == MW_OK) {
            check(pp.gx >= 0 && (pp.waves == 4 || pp.waves == 8) && pp.group == group, "prefill plan", it);
            // the key-range split: at most the pieces the size call with no CU
            // count allows, pieces of at least 4 tiles, only of dual blocks
            mw::prefill_split_plan(pb, nl.data(), pl.data(), shape.num_q_heads, pcus, &pp);
            size_t most = 0;
            check(mw_prefill_workspace_size(&shape, pb, nl.data(), pl.data(), 0, &most) == MW_OK, "size call", it);
            check(pp.split_bytes <= most, "the size with no CU count covers the plan", it);
            check(pp.pieces >= 1 && pp.pieces <= mw::kPrefillMaxPieces, "pieces", it);
            check(pp.pieces == 1 || (pp.dual && pp.waves == 4 && pp.piece_tiles >= mw::kPrefillMinPieceTiles), "cuts", it);
            for (int b = 0; b < pb; ++b)
                for (int qb = 0; 128 * qb < nl[b] * group && pp.pieces > 1; ++qb) {
                    const int nt = mw::prefill_block_tiles(pl[b], nl[b], qb, 128, group);
                    const int k = mw::prefill_pieces(nt, pp.piece_tiles, pp.pieces);
                    // equal pieces of two tiles or more, in order, up to the block's end
                    for (int i = 0; i < k && k > 1; ++i)
                        check((i + 1) * nt / k - i * nt / k >= 2, "a tile for each wave group of a piece", it);
                    check(k * nt / k == nt, "pieces reach the block's end", it);
                    // the last piece has three tiles or more, so every row of the block
                    // (at most 128 positions) sees a key of every piece's first tile
                    check(k == 1 || (k - 1) * nt / k <= nt - 3, "cut before the diagonal", it);
                    check(k == 1 || (k - 1) * nt / k <= (pl[b] + 128 * qb / group) / 64, "first tile of each piece visible", it);
                }
            // the grid has a work-group for every block, in an order that it allows
            int64_t blocks = 0, most_blocks = 0;
            for (int b = 0; b < pb; ++b) {
                const int64_t nb = (static_cast<int64_t>(nl[b]) * group + 32 * pp.waves - 1) / (32 * pp.waves);
                blocks += nb;
                most_blocks = std::max(most_blocks, nb);
            }
            check(pp.order >= 0 && pp.order <= 2 && (pp.order != 2 || (pb > 1 && pb <= 64)), "order", it);
            check(pp.order == 2 ? pp.gy == 1 && pp.gx == blocks * hkv
                                : pp.gy == pb && pp.gx == (pp.order == 1 ? (most_blocks + 1) / 2 : most_blocks) * hkv,
                  "grid covers the blocks", it);
            check(pp.big_units >= 0 && pp.big_units <= pp.gx && pp.big_units % hkv == 0 &&
                      (pp.big_units == 0 || (pp.waves == 8 && pp.gy == 1 && !pp.dual)), "units of the mixed launch", it);
        }
        mw_kv_pool_destroy(pool);
    }
}

// The order over a batch: the counts that the kernel's search adds up against a
// count block by block, and the blocks it gives work-groups 0, 1, ..: every block
// once, no lighter one before a heavier one.  (The search is restated; sequences
// take the place of lanes.)
void batch_order() {
    for (int it = 0; it < 300; ++it) {
        const int batch = uniform(2, 64), group = uniform(1, 40), rows = uniform(0, 1) ? 128 : 256;
        std::vector<int> n(batch), r(batch), nqb(batch);
        std::vector<std::vector<int>> taken(batch);
        int blocks = 0;
        for (int b = 0; b < batch; ++b) {
            n[b] = uniform(0, 5) == 0 ? 0 : uniform(1, it % 3 ? 100 : 2000);
            r[b] = uniform(0, 3) == 0 ? 0 : uniform(0, 5000);
            if (b > 0 && uniform(0, 4) == 0) n[b] = n[b - 1], r[b] = r[b - 1];
            nqb[b] = (n[b] * group + rows - 1) / rows;
            taken[b].assign(nqb[b], 0);
            blocks += nqb[b];
        }
        const auto at_least = [&](int b, int t) { return mw::prefill_blocks_at_least(nqb[b], n[b], r[b], group, rows, t); };
        const auto total = [&](int t) {
            int s = 0;
            for (int b = 0; b < batch; ++b) s += at_least(b, t);
            return s;
        };
        for (int b = 0; b < batch; ++b)
            for (int t = 1; t < 120; ++t) {
                int count = 0;
                for (int q = 0; q < nqb[b]; ++q) count += mw::prefill_block_tiles(r[b], n[b], q, rows, group) >= t;
                check(at_least(b, t) == count, "blocks of t tiles or more", it);
            }
        int last_tiles = INT32_MAX;
        for (int x = 0; x < blocks; ++x) {
            int j = x, t = 1, step = 1;
            while (total(t + step) > j) step <<= 1;
            for (; step > 0; step >>= 1)
                if (total(t + step) > j) t += step;
            j -= total(t + 1);
            bool found = false;
            for (int b = 0, incl = 0; b < batch && !found; ++b) {
                const int above = at_least(b, t + 1), same = at_least(b, t) - above;
                incl += same;
                if (j < incl - same || j >= incl) continue;
                const int blk = nqb[b] - above - 1 + incl - same - j;
                found = blk >= 0 && blk < nqb[b] && taken[b][blk]++ == 0;
                const int tiles = found ? mw::prefill_block_tiles(r[b], n[b], blk, rows, group) : 0;
                check(found && tiles == t && tiles <= last_tiles, "a block of its own, none lighter before", it);
                last_tiles = tiles;
            }
            check(found, "a block for every work-group", it);
        }
    }
    // the batches of the GPU test of this order are planned in it
    for (int batch : {2, 63, 64, 65})
        for (int cus : {8, 256}) {
            std::vector<int32_t> n(batch), r(batch);
            for (int b = 0; b < batch; ++b) r[b] = 53 * b % 1201, n[b] = 1 + 29 * b % 97;
            r[0] = 300, n[0] = 700;
            if (batch == 2) {
                r = {2000, 1900}, n = {759, 61};
            } else {
                n[3] = n[batch - 1] = 0;
                for (int b = 10; b < 20; ++b) r[b] = 600, n[b] = 33;
            }
            mw::PrefillPlan p{};
            p.hkv = 2, p.group = 4;
            mw::prefill_split_plan(batch, n.data(), r.data(), 8, cus, &p);
            check((p.order == 2) == (batch <= 64), "the order test's batches are ordered", batch);
        }
    // heavy-light pairs where they are alike and fill the rounds, and only there
    const struct { int hq, hkv, cus; std::vector<int32_t> n, r; bool pairs; } calls[] = {
        {32, 8, 64, {2048}, {0}, true},        {32, 8, 32, {1024}, {0}, true},
        {32, 8, 32, {4096}, {0}, true},        {32, 8, 64, {4096}, {0}, true},
        {32, 8, 128, {4096}, {0}, true},       {32, 8, 256, {4096}, {0}, true},
        {32, 8, 96, {4096}, {0}, false},       {32, 8, 192, {4096}, {0}, false},
        {32, 8, 64, {4096, 1024}, {0, 0}, false},
    };
    for (const auto &c : calls) {
        mw::PrefillPlan p{};
        p.hkv = c.hkv, p.group = c.hq / c.hkv;
        mw::prefill_split_plan(static_cast<int>(c.n.size()), c.n.data(), c.r.data(), 8, c.cus, &p);
        check((p.order == 1) == c.pairs, "pairs where they fill the rounds", c.cus);
    }
    // equal long blocks just past a round of 256-row ones: dual blocks, whose rounds
    // are half as long; pieces that fill the CUs' rounds; and two sequences of
    // which the shorter one's missing blocks would take the places of a second round
    // (in length order they are left out)
    mw::PrefillPlan p{};
    p.hkv = 8, p.group = 4;
    const int32_t n[2] = {2048, 256}, r[2] = {16384, 131072};
    for (int cus : {192, 224}) {
        mw::prefill_split_plan(1, n, r, 32, cus, &p);
        check(p.dual && p.pieces == 1, "dual blocks past a round", cus);
    }
    mw::prefill_split_plan(1, n + 1, r + 1, 32, 160, &p);
    check(p.dual && p.pieces == 5, "pieces in whole rounds", p.pieces);
    p.hkv = 1, p.group = 16;
    const int32_t n2[2] = {89, 146}, r2[2] = {51576, 53735};
    mw::prefill_split_plan(2, n2, r2, 16, 64, &p);
    check(p.dual && (p.order == 2 || p.gx * p.gy * p.pieces <= 64), "places of empty work-groups", p.pieces);
}

// A prefill workspace short of the plan's pieces: fewer pieces that fit, or none;
// refused only if short of what blocks of 32 positions need as well.
void short_workspaces() {
    mw_kv_pool_desc desc{1 << 14, 16, 1, 128};
    int fewer = 0, none = 0, refused = 0;
    for (int it = 0; it < 3000; ++it) {
        const int hkv = 1 << uniform(0, 3), group = uniform(1, 16), batch = uniform(1, 16);
        desc.num_kv_heads = hkv;
        mw_kv_pool *pool = nullptr;
        check(mw_kv_pool_create(&desc, g_fake, g_fake, &pool) == MW_OK, "pool create", it);
        std::vector<int32_t> n(batch), r(batch);
        const int n_hi = 1 << uniform(0, 11), r_hi = 1 << uniform(0, 14);
        for (int b = 0; b < batch; ++b) n[b] = uniform(1, n_hi), r[b] = uniform(0, r_hi);
        const mw_prefill_args a{pool, {hkv * group, hkv, 128, 0.0883883f}, batch, n.data(), r.data(),
                                reinterpret_cast<int32_t *>(g_fake), reinterpret_cast<int32_t *>(g_fake),
                                reinterpret_cast<int32_t *>(g_fake), (n_hi + r_hi + 15) / 16, g_fake, g_fake};
        const int cus = 8 * uniform(1, 32);
        mw::PrefillPlan want;
        check(mw::prefill_prepare(&a, cus, true, &want, "prepare", true) == MW_OK, "plan", it);
        const int base = mw::prefill_base_pieces(batch, n.data(), r.data(), hkv, group, cus);
        const size_t piece = static_cast<size_t>(want.rows) * hkv * group * (mw::kHeadDim * 4 + 8);
        check(base >= 1 && base <= mw::kPrefillMaxPieces, "base pieces", it);
        for (int given = 0; given <= mw::kPrefillMaxPieces; ++given) {
            mw::PrefillPlan p = want;
            // with no pieces: a missing, a misaligned or an empty workspace
            const void *ws = given ? g_fake : it % 3 == 0 ? nullptr : g_fake + (it % 3 == 1 ? 8 : 0);
            const size_t bytes = given ? given * piece : it % 3 == 1 ? 100 * piece : 0;
            const mw_status st = mw::prefill_fit_workspace(&a, cus, &p, ws, bytes, "fit");
            const int wanted = want.pieces > 1 ? want.pieces : 0, least = std::min(wanted, base > 1 ? base : 0);
            check((st == MW_OK) == (given >= least), "accepted with what callers bring", it);
            if (st != MW_OK) {
                ++refused;
                continue;
            }
            check(p.split_bytes <= given * piece || (given >= wanted && p.split_bytes == want.split_bytes),
                  "pieces fit the workspace", it);
            check(p.pieces == 1 || (p.dual && p.pieces * piece == p.split_bytes), "pieces and bytes", it);
            check(p.gx > 0 && p.gy >= 1 && (given < wanted || p.pieces == want.pieces), "launch", it);
            if (given < wanted) ++(p.pieces > 1 ? fewer : none);
        }
        mw_kv_pool_destroy(pool);
    }
    check(fewer > 10 && none > 10 && refused > 100, "short workspaces of every kind", fewer);
}

// Three segments whose padding would leave a quarter of the units idle and make
// ranges 1.8 (32 CUs) and 1.3 times as long: balanced there, where a CU's stream is
// the bound; padded on the whole GPU, where the memory is and padding is free.
void padding() {
    mw_kv_pool_desc desc{1 << 14, 16, 8, 128};
    mw_kv_pool *pool = nullptr;
    check(mw_kv_pool_create(&desc, g_fake, g_fake, &pool) == MW_OK, "pool create", -1);
    const mw_attn_shape shape{32, 8, 128, 0.0883883f};
    const int32_t lens[3] = {16000, 16000, 4000};
    mw_decode_args a{pool, shape, 3, lens, reinterpret_cast<int32_t *>(g_fake), reinterpret_cast<int32_t *>(g_fake),
                     1000, g_fake, g_fake, g_fake, ~size_t{0}, 0};
    mw::DecodePlan dp;
    for (int cus : {32, 64, 256}) {
        check(mw::decode_prepare(&a, cus, &dp, "decode_prepare") == MW_OK, "plan", cus);
        check(dp.aligned == (cus == 256), "padding by time", cus);
        check(dp.aligned || dp.units == cus, "a unit per CU", cus);
    }
    mw_kv_pool_destroy(pool);
}

// Sizes of calls far past any pool: every length that the size call accepts, with
// groups whose rows no longer fit 32 bits.
void prefill_sizes() {
    const int32_t most = INT32_MAX - 64;
    for (int it = 0; it < 200; ++it) {
        const int group = uniform(1, 64);
        const mw_attn_shape shape{group, 1, 128, 0.0883883f};
        const int32_t n = it < 8 ? most : uniform(1 << 24, most);
        const int32_t r = n == most ? 0 : uniform(0, most - n);
        const int32_t cus = it % 2 ? INT32_MAX : uniform(0, 1 << 30);
        size_t bytes = 0;
        check(mw_prefill_workspace_size(&shape, 1, &n, &r, cus, &bytes) == MW_OK, "size of a large call", it);
        const size_t piece = static_cast<size_t>(n) * group * (mw::kHeadDim * 4 + 8);
        check(bytes % piece == 0 && bytes / piece <= mw::kPrefillMaxPieces, "whole pieces of a large call", it);
    }
}

// Quotients by a divisor with a precomputed reciprocal: every divisor up to 4096 and
// random ones, at multiples, next to them and at the ends of the range.
void divisors() {
    for (int it = 0; it < 6000; ++it) {
        const int d = it < 4096 ? it + 1 : uniform(1, INT32_MAX - 1);
        const mw::Divisor by(d);
        for (int k = 0; k < 60; ++k) {
            const int64_t at = k < 30 ? static_cast<int64_t>(uniform(0, (INT32_MAX - 1) / d)) * d + k % 3 - 1
                                      : k < 32 ? INT32_MAX - (k - 30) : k < 34 ? k - 32 : uniform(0, INT32_MAX - 1);
            const int n = static_cast<int>(std::min<int64_t>(std::max<int64_t>(at, 0), INT32_MAX));
            check(n / by == n / d, "quotient by a reciprocal", it);
        }
    }
}

// The merge of a dual block's two wave groups: no two of the O halves handed
// over, the (m, l) words and the staged rows (fp32 and bf16) may share a byte or
// leave their buffers, for there is no barrier between one wave's staging and
// another's reads.  Counts the bytes that do; ml_at and stage_at place the words
// (in the group's V buffers if ml_in_v, else in the table copy) and the rows.
template <class Ml, class Stage>
int dual_merge_clashes(bool ml_in_v, Ml ml_at, Stage stage_at) {
    int bad = 0;
    std::vector<uint8_t> k[2], v[2], table(mw::kDualTableBytes, 0);
    for (int g = 0; g < 2; ++g) k[g].assign(mw::kDualBufBytes, 0), v[g].assign(mw::kDualBufBytes, 0);
    // bytes past a group's buffers lie in the next group's, or outside
    auto take = [&](std::vector<uint8_t>(&buf)[2], int g, int at, int n, int mark) {
        for (int i = at; i < at + n; ++i) {
            const int gg = g + i / mw::kDualBufBytes;
            if (gg > 1) {
                ++bad;
                continue;
            }
            uint8_t &b = buf[gg][i % mw::kDualBufBytes];
            if ((b && b != mark) || gg != g) ++bad;
            b = static_cast<uint8_t>(mark);
        }
    };
    for (int g = 0; g < 2; ++g)
        for (int w = 0; w < 4; ++w) {
            const int mark = 1 + 4 * g + w;
            for (int lane = 0; lane < 64; ++lane)
                for (int j = 0; j < 8; ++j) take(k, g, mw::dual_hand_over(w) + (j * 64 + lane) * 16, 16, mark);
            for (int row = 0; row < 32; ++row) {
                for (int c = 0; c < 16; ++c) take(v, g, stage_at(w) + mw::dual_stage_f32(row, c), 16, mark);
                for (int c = 0; c < 8; ++c) take(v, g, stage_at(w) + mw::dual_stage_bf16(row, c), 16, mark);
                const int at = ml_at(g, 32 * w + row);
                for (int i = at; i < at + 8; ++i) {
                    if (ml_in_v) {
                        if (v[g][i]) ++bad;
                        v[g][i] = 255;
                    } else {
                        if (i < 0 || i >= mw::kDualTableBytes || table[i]) ++bad;
                        else table[i] = 1;
                    }
                }
            }
        }
    return bad;
}

void dual_merge() {
    check(dual_merge_clashes(false, mw::dual_ml, mw::dual_stage) == 0, "LDS regions of the dual merge", -1);
    // the check finds the words at the start of the V buffers and the rows
    // 1 KiB behind them, whose last fp32 rows run over the end
    check(dual_merge_clashes(true, [](int, int row) { return 8 * row; }, [](int w) { return 1024 + 8192 * w; }) > 0,
          "a clash planted in the dual merge's regions", -1);
}

// The step order of a dual block's two wave groups, run with recording steps.
// Time is counted in barriers passed; the waves of a work-group are unordered
// between two of them, and those of a group may see different numbers of its
// tiles.  Each tile buffer has its requests (content, when requested, when waited
// for) and reads (content expected, from when to when).
struct DualTrace {
    struct Request {
        int buffer, what, at, landed;  // landed: -1 while in flight
    };
    struct Read {
        int buffer, what, from, to;
    };
    std::vector<Request> requests;
    std::vector<Read> reads;
    std::vector<int> barriers;  // of each wave
    bool all_tiles = true;      // every wave computed on just the tiles it sees
};
enum { kBufK = 0, kBufV = 2, kQ = -1 };  // buffer ids: 4 group + kBufK/V + index; content: tile, or kQ

// skip_wait: a wait to leave out (-1: none), counted over all waves in *waits
// (not counted: those with nothing to wait for, and the first of a group with
// tiles, which the next one stands in for)
DualTrace trace_dual(int total, int skip_wait, int *waits = nullptr) {
    DualTrace t;
    int n_waits = 0;
    // before the first step: K(0) and Q requested, waited for
    for (int g = 0; g < 2; ++g) {
        t.requests.push_back({4 * g + kBufK, 0, 0, 0});
        t.requests.push_back({4 * g + kBufV + 1, kQ, 0, 0});
    }
    for (int g = 0; g < 2; ++g) {
        const int own = (total + 1 - g) / 2;
        for (int mine = std::max(0, own - 3); mine <= own; ++mine) {
            int now = 0, scores = 0, outputs = 0, waited = 0;
            std::vector<size_t> flying;  // the wave's requests, oldest first
            std::vector<size_t> q_reads;
            const auto request = [&](int kv, int u) {
                flying.push_back(t.requests.size());
                t.requests.push_back({4 * g + kv + u % 2, u, now, -1});
            };
            const auto read = [&](int kv, int u) { t.reads.push_back({4 * g + kv + u % 2, u, now, now}); };
            mw::dual_schedule(g, total, mine, [&](auto kind, int u) {
                constexpr mw::DualStep what = decltype(kind)::value;
                if constexpr (what == mw::kDualFirstLoads) request(kBufV, 0), request(kBufK, 1);
                if constexpr (what == mw::kDualBarrier) ++now;
                if constexpr (what == mw::kDualReadQ)
                    for (int og = 0; og < 2; ++og) {  // half of the waves from either group's V(1)
                        q_reads.push_back(t.reads.size());
                        t.reads.push_back({4 * og + kBufV + 1, kQ, now, now});
                    }
                if constexpr (what == mw::kDualScores) {
                    for (size_t i : q_reads) t.reads[i].to = now;  // used here
                    read(kBufK, 0);
                    t.all_tiles &= scores++ == 0;
                }
                if constexpr (what == mw::kDualSoftmax || what == mw::kDualLoadK) request(kBufK, u + 2);
                if constexpr (what == mw::kDualMatrix || what == mw::kDualLastMatrix) {
                    read(kBufV, u);
                    t.all_tiles &= outputs++ == u && scores == outputs;
                }
                if constexpr (what == mw::kDualMatrix) read(kBufK, u + 1), ++scores;
                if constexpr (what == mw::kDualMatrix || what == mw::kDualLoadV) request(kBufV, u + 1);
                if constexpr (what == mw::kDualWaitAll || what == mw::kDualWaitOlder) {
                    const size_t keep = what == mw::kDualWaitAll ? 0 : 1;
                    const bool spare = flying.size() <= keep || (waited++ == 0 && own > 0);
                    if (spare || n_waits++ != skip_wait)
                        while (flying.size() > keep) {
                            t.requests[flying.front()].landed = now;
                            flying.erase(flying.begin());
                        }
                }
            });
            t.all_tiles &= scores == mine && outputs == mine;
            t.barriers.push_back(now);
        }
    }
    if (waits) *waits = n_waits;
    return t;
}

// Counts what is wrong with a trace: a barrier too few, a tile left out, a read
// of a buffer that may not hold the tile yet or no longer, a request that may
// overtake an earlier one of its buffer, one in flight at the merge.
int dual_trace_faults(const DualTrace &t) {
    int bad = !t.all_tiles;
    for (int n : t.barriers) bad += n != t.barriers[0];
    for (const auto &rq : t.requests) {
        bad += rq.landed < 0 || (rq.at > 0 && rq.landed >= t.barriers[0]);
        for (const auto &rd : t.reads)
            if (rd.buffer == rq.buffer && rd.what != rq.what && rd.from <= rq.at && rd.to >= rq.at) ++bad;
        for (const auto &other : t.requests)
            if (other.buffer == rq.buffer &&
                (other.at < rq.at ? other.landed >= rq.at : other.at == rq.at && other.what != rq.what))
                ++bad;
    }
    for (const auto &rd : t.reads) {
        int last = -1;  // when the buffer was last requested before the read
        for (const auto &rq : t.requests)
            if (rq.buffer == rd.buffer && rq.at <= rd.to) last = std::max(last, rq.at);
        for (const auto &rq : t.requests)
            if (rq.buffer == rd.buffer && rq.at == last)
                bad += rq.what != rd.what || rq.landed < 0 || (last > 0 && rq.landed >= rd.from);
        bad += last < 0;
    }
    return bad;
}

void dual_order() {
    for (int total = 1; total <= 24; ++total) {
        int waits = 0;
        check(dual_trace_faults(trace_dual(total, -1, &waits)) == 0, "step order of a dual block", total);
        check(waits > 0 || total == 2, "waits that count", total);
        // (with one tile, the only such wait is that of the group without tiles)
        for (int w = 0; w < waits; ++w)
            check(dual_trace_faults(trace_dual(total, w)) > 0, "a wait left out of the step order", total);
    }
}

void allocator() {
    mw_kv_pool_desc desc{1000, 16, 2, 128};
    mw_kv_pool *pool = nullptr;
    check(mw_kv_pool_create(&desc, g_fake, g_fake, &pool) == MW_OK, "pool create", -1);
    std::vector<int32_t> held;
    for (int it = 0; it < 20000; ++it) {
        const int op = uniform(0, 9);
        int32_t n_free = 0;
        mw_kv_pool_num_free(pool, &n_free);
        check(n_free + static_cast<int>(held.size()) == 1000, "pages are conserved", it);
        if (op < 5) {
            const int n = uniform(0, 40);
            std::vector<int32_t> got(n);
            const mw_status st = mw_kv_pool_alloc(pool, n, got.data());
            if (st == MW_OK) held.insert(held.end(), got.begin(), got.end());
            else check(st == MW_ERR_OUT_OF_PAGES && n > n_free, "alloc refuses only when short", it);
        } else if (op < 9 && !held.empty()) {
            const int n = uniform(1, static_cast<int>(held.size()));
            std::vector<int32_t> back(held.end() - n, held.end());
            check(mw_kv_pool_free(pool, back.data(), n) == MW_OK, "free", it);
            held.resize(held.size() - n);
            if (uniform(0, 3) == 0) check(mw_kv_pool_free(pool, back.data(), 1) != MW_OK, "double free refused", it);
        } else {
            // renumber the free list: a permutation of the pages not held
            std::vector<uint8_t> is_held(1000, 0);
            for (int32_t x : held) is_held[x] = 1;
            std::vector<int32_t> order;
            for (int32_t x = 0; x < 1000; ++x)
                if (!is_held[x]) order.push_back(x);
            for (size_t i = order.size(); i > 1; --i) std::swap(order[i - 1], order[next_u32() % i]);
            check(mw_kv_pool_set_free_order(pool, order.data(), static_cast<int32_t>(order.size())) == MW_OK,
                  "set free order", it);
        }
    }
    mw_kv_pool_destroy(pool);
}

void estimator() {
    mw_predictor *p = nullptr;
    mw_guard *g = nullptr;
    check(mw_predictor_create(&p) == MW_OK && mw_guard_create(&g) == MW_OK, "estimator create", -1);
    for (int it = 0; it < 400; ++it) {
        const int cus = 8 * uniform(1, 32), batch = uniform(1, 12);
        std::vector<int32_t> n(batch), r(batch), L(batch);
        for (int b = 0; b < batch; ++b) {
            n[b] = uniform(1, 20000);
            r[b] = uniform(0, 100000);
            L[b] = uniform(1, 100000);
        }
        const double ms = 0.01 + uniform(0, 100000) * 1e-3;
        mw_predictor_add_prefill(p, cus, batch, n.data(), r.data(), ms);
        mw_predictor_add_decode(p, cus, batch, L.data(), ms);
        const mw_guard_key key{uniform(0, 1 << 20), uniform(0, 1 << 20), uniform(1, 512), uniform(0, 1 << 24), cus};
        mw_guard_add(g, &key, 1.0 + uniform(0, 1000) * 1e-3);
        double s = 0.0;
        check(mw_guard_lookup(g, &key, &s) == MW_OK && s >= 1.0, "guard lookup", it);
        if (it % 50 == 49) {
            mw_predictor_fit(p);
            double out = 0.0, th[4];
            mw_predictor_prefill_ms(p, cus, batch, n.data(), r.data(), &out);
            mw_predictor_decode_ms(p, cus, batch, L.data(), &out);
            mw_predictor_coefficients(p, uniform(0, 1), cus, th);
        }
        int32_t npl = 0;
        check(mw_prefill_layers(0.01 + ms, 0.02 + 2 * ms, uniform(1, 128), &npl) == MW_OK && npl >= 1,
              "prefill layers", it);
    }
    mw_predictor_destroy(p);
    mw_guard_destroy(g);
    // prefill models over the simulated launch: random shapes, batches and
    // partitions; every prediction of a fitted model is finite
    const int hkvs[4] = {1, 2, 4, 8};
    for (int shape = 0; shape < 6; ++shape) {
        mw_predictor *q = nullptr;
        check(mw_predictor_create(&q) == MW_OK, "launch-shape predictor create", shape);
        const int hkv = hkvs[uniform(0, 3)], group = uniform(1, 16);
        check(mw_predictor_set_launch_shape(q, hkv * group, hkv) == MW_OK, "set launch shape", shape);
        for (int it = 0; it < 60; ++it) {
            const int cus = 8 * uniform(1, 32), batch = uniform(1, 6);
            std::vector<int32_t> n(batch), r(batch);
            for (int b = 0; b < batch; ++b) {
                n[b] = uniform(1, 6000);
                r[b] = uniform(0, 70000);
            }
            mw_predictor_add_prefill(q, cus, batch, n.data(), r.data(), 0.01 + uniform(0, 100000) * 1e-4);
            if (it % 20 == 19) {
                mw_predictor_fit(q);
                double out = 0.0, th[4];
                if (mw_predictor_prefill_ms(q, cus, batch, n.data(), r.data(), &out) == MW_OK)
                    check(out == out && out < 1e30 && out > -1e30, "launch-shape prediction finite", it);
                mw_predictor_coefficients(q, 2 * uniform(0, 1), cus, th);
            }
        }
        mw_predictor_destroy(q);
    }
}

}  // namespace

int main() {
    planners();
    batch_order();
    short_workspaces();
    padding();
    prefill_sizes();
    divisors();
    dual_merge();
    dual_order();
    allocator();
    estimator();
    if (g_fail) return 1;
    std::printf("ok\n");
    return 0;
}
