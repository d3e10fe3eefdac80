// Device bodies of the split-K decode attention: one unit of the fixed-chunk
// split (shared by its kernel and the fused prefill + decode kernel), and one
// unit of the balanced split.
//
// Decode is memory-bound (paper Sec. 2.2: the decode phase is
// memory-intensive; Sec. 3.3, Table "tab:theory_cost": O(d^2 + (r+1) d)), so
// the design goal is streaming every K/V byte of the batch from HBM exactly
// once with enough bytes in flight; arithmetic is kept off the vector ALU.
// A split depends only on the sequence lengths (never on page ids), so a
// result does not change when pages are renumbered.
//
// In both, a wave streams pages two at a time (a "pair"), with the next pair's
// loads in flight while the current pair is computed.  K and V rows are loaded
// whole (each instruction reads four 256-byte rows, so no cache line is
// requested twice: K loaded straight in its operand layout, 64 bytes of 16 rows
// per instruction, took 507 us instead of 473 on 32 sequences of 16K-32K tokens
// and 139 instead of 118 on 64 of 512-4096) with streaming loads that leave
// nothing in the caches for the other partition's kernel to lose, and go to
// per-wave LDS buffers as loaded (16-byte row-major stores):
//   * K comes back in the A-operand layout of a 16x16x32 bf16 MFMA (one page
//     = 16 tokens x 32 dims per step), B = Q^T of the kv head's G query heads
//     (columns >= G are zero): S^T[token][head].
//   * V comes back through the transposing LDS read as the A operand of a
//     second MFMA, O^T[d][head] += V^T[d][token] P^T[token][head]; P^T is the
//     S^T accumulator itself, converted to bf16.
//   * online softmax per pair in base 2; the reference maximum moves only
//     when a column's maximum grows by more than 2^8 (O and l are then
//     rescaled), which the result O / l does not depend on.
// The waves' (m, l, O) are merged in LDS at the end; a sequence held whole
// writes its bf16 output directly, otherwise the partial goes to the workspace
// and the pieces of each (sequence, kv head) are merged with the log-sum-exp
// identity
//   M = max m_s,  O = sum 2^(m_s - M) o_s / sum 2^(m_s - M) l_s
// by the work-group that finishes the segment's last piece (balanced split)
// or by the combine kernel (fixed chunks).
#pragma once
#include "mw_internal.h"

namespace {
namespace dk {

using namespace mw;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kPair = 2;                      // pages per wave step
constexpr int VSTR = 144;                     // LDS V row stride (bf16): conflict-free transposing reads
constexpr int KSTR = 136;                     // LDS K row stride (bf16): conflict-free 16-byte reads
constexpr int kVBufElems = 16 * kPair * VSTR; // one wave's V buffer
constexpr int kKBufElems = 16 * kPair * KSTR; // one wave's K buffer
constexpr int kWaveBufElems = kVBufElems + kKBufElems;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRescaleLog2 = 8.f;
// chunk_pages = 0: the largest of 128, 64, 32 pages that still gives at least
// kAutoMinUnits work-groups (longer chunks amortise each work-group's set-up
// and merge; enough work-groups keep every CU of a partition streaming)
constexpr int kAutoChunks[3] = {128, 64, 32};
constexpr int64_t kAutoMinUnits = 1024;

__device__ inline uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }
__device__ inline uint32_t cvt2(float a, float b) {
    bf16x2 v;
    v[0] = static_cast<__bf16>(a);
    v[1] = static_cast<__bf16>(b);
    return __builtin_bit_cast(uint32_t, v);
}
__device__ inline uint4 sel4(bool ok, uint4 v) {
    return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}
__device__ inline i16x4 lds_read_tr(const uint16_t *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) i16x4 *>(reinterpret_cast<uintptr_t>(p)));
}

__device__ inline int chunks_of(int L, int ch_pages, int bt_stride) {
    if (L <= 0) return 0;
    int np = (L + kPageSize - 1) / kPageSize;
    np = np < bt_stride ? np : bt_stride;
    return (np + ch_pages - 1) / ch_pages;
}

// Wave-level search for the sequence b and chunk c holding global chunk ci
// (every wave runs it; no barrier).  Returns false if ci is past the end.
__device__ bool locate_chunk(const int32_t *__restrict__ seq_lens, int batch, int ch_pages, int bt_stride,
                             int ci, int &b_out, int &c_out, int &nch_out, int &first_out) {
    const int lane = threadIdx.x & 63;
    int running = 0;
    for (int base = 0; base < batch; base += 64) {
        const int bb = base + lane;
        const int n = bb < batch ? chunks_of(seq_lens[bb], ch_pages, bt_stride) : 0;
        int x = n;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        const int incl = running + x, excl = incl - n;
        const uint64_t hit = __builtin_amdgcn_ballot_w64(bb < batch && ci >= excl && ci < incl);
        if (hit) {
            const int src = __builtin_ctzll(hit);
            first_out = __shfl(excl, src);
            b_out = base + src;
            c_out = ci - first_out;
            nch_out = __shfl(n, src);
            return true;
        }
        running = __shfl(incl, 63);
    }
    return false;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Streaming load: the line is not kept in the caches (decode reads each byte
// of K/V once), so the other partition's working set stays there.
__device__ inline uint4 load_stream(const uint16_t *p) {
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p)));
}

struct PairRegs {
    uint4 k[kPair][4];  // K rows as loaded: token 4i + lane/16, dims 8(lane%16) + 0..7
    uint4 v[kPair][4];  // V rows: token 4i + lane/16, dims 8(lane%16) + 0..7
    bool ok[kPair];
};

__device__ inline void pair_load(PairRegs &pr, const uint16_t *__restrict__ kpool,
                                 const uint16_t *__restrict__ vpool, const int32_t *__restrict__ btrow,
                                 int p0, int p_end, int hkv, int kvh, int num_pages) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < kPair; ++j) {
        const int p = p0 + j;
        const int page = btrow[p < p_end ? p : p0];
        pr.ok[j] = p < p_end && page >= 0 && page < num_pages;
        const size_t base = (static_cast<size_t>(pr.ok[j] ? page : 0) * hkv + kvh) * (kPageSize * kHeadDim);
        // whole 256-byte rows per instruction (four rows each), so no cache
        // line is requested by two instructions
#pragma unroll
        for (int i = 0; i < 4; ++i)
            pr.k[j][i] = load_stream(kpool + base + (4 * i + (lane >> 4)) * kHeadDim + 8 * (lane & 15));
#pragma unroll
        for (int i = 0; i < 4; ++i)
            pr.v[j][i] = load_stream(vpool + base + (4 * i + (lane >> 4)) * kHeadDim + 8 * (lane & 15));
    }
}

// Pages [p_begin, p_end) of sequence b (length L, block-table row btrow),
// kv head kvh, on 4 waves; tid = thread index within them (0..255); s_v,
// s_m, s_l are their LDS.  The merged result is written as the bf16 output
// (direct) or as the fp32 partial (O, (m, l)) of workspace slot `slot`.
// active = false (uniform): nothing is read or written, but both work-group
// barriers are still taken.
__device__ __forceinline__ void
decode_pages(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
             const uint16_t *__restrict__ q, uint16_t *__restrict__ out, const int32_t *__restrict__ btrow,
             float *__restrict__ ws_o, float2 *__restrict__ ws_ml, int b, int L, int hkv, int kvh, int group,
             int num_pages, float scale_log2, int p_begin, int p_end, bool active, bool direct, int64_t slot,
             int tid, uint16_t *s_v, float (*s_m)[16], float (*s_l)[16]) {
    const int lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    if (!active) p_end = p_begin;
    const int hq = hkv * group;

    // Q^T operand: column `col` is query head kvh*group + col
    uint4 qop[4];
    {
        const bool hv = col < group;
        const uint16_t *qp = q + (static_cast<size_t>(b) * hq + kvh * group + (hv ? col : 0)) * kHeadDim + 8 * grp;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
            qop[kb] = hv ? *reinterpret_cast<const uint4 *>(qp + 32 * kb) : make_uint4(0, 0, 0, 0);
    }

    f32x4 oacc[8];  // O^T[d = 16db + 4grp + i][head = col]
#pragma unroll
    for (int db = 0; db < 8; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    uint16_t *vbuf = s_v + wave * kWaveBufElems;
    uint16_t *kbuf = vbuf + kVBufElems;
    // K operand reads: lane l reads row l%16 of each page, 16-byte chunk 4kb + l/16
    const uint16_t *krd = kbuf + col * KSTR + 8 * grp;
    // transposing-read source: lane s of 16-lane group g -> row 4g + s/4 (+16 for
    // the second page), dims 4(s%4) (+16 db)
    const uint16_t *vtr = vbuf + (4 * grp + (col >> 2)) * VSTR + 4 * (col & 3);

    // this wave's pairs: pages p_begin + 2*(wave + 4*j) + {0, 1}
    const int pstart = p_begin + kPair * wave;
    const int pstep = kPair * kWaves;
    PairRegs pr;
    if (pstart < p_end) pair_load(pr, kpool, vpool, btrow, pstart, p_end, hkv, kvh, num_pages);
    for (int p0 = pstart; p0 < p_end; p0 += pstep) {
        bool ok[kPair];
#pragma unroll
        for (int j = 0; j < kPair; ++j) ok[j] = pr.ok[j];
        // K and V of this pair -> LDS as loaded, with V rows of an absent page
        // or past the sequence's end as zeros (a masked key has p = 0, but 0
        // times a NaN or Inf in a slack slot would not be 0); the scores of
        // those keys are masked below
#pragma unroll
        for (int j = 0; j < kPair; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *reinterpret_cast<uint4 *>(kbuf + (16 * j + 4 * i + grp) * KSTR + 8 * col) = pr.k[j][i];
                *reinterpret_cast<uint4 *>(vbuf + (16 * j + 4 * i + grp) * VSTR + 8 * col) =
                    sel4(pr.ok[j] && (p0 + j) * kPageSize + 4 * i + grp < L, pr.v[j][i]);
            }
        // next pair's loads go out while this pair is computed
        const int pn = p0 + pstep;
        if (pn < p_end) pair_load(pr, kpool, vpool, btrow, pn, p_end, hkv, kvh, num_pages);
        // S^T = K Q^T on the matrix core, K read back in the operand layout
        f32x4 sc[kPair];
#pragma unroll
        for (int j = 0; j < kPair; ++j) {
            sc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const uint4 a = *reinterpret_cast<const uint4 *>(krd + 16 * j * KSTR + 32 * kb);
                sc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                                __builtin_bit_cast(bf16x8, qop[kb]), sc[j], 0, 0, 0);
            }
        }

        // mask keys past the sequence or on an absent page, then the pair's
        // maximum per head
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < kPair; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int tok = (p0 + j) * kPageSize + 4 * grp + i;
                const float v = (ok[j] && tok < L) ? sc[j][i] * scale_log2 : -INFINITY;
                sc[j][i] = v;
                mx = fmaxf(mx, v);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleLog2) != 0) {
            const float m_new = fmaxf(m_run, mx);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 8; ++db) oacc[db] *= alpha;
        }
        float p[kPair][4];
#pragma unroll
        for (int j = 0; j < kPair; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                p[j][i] = __builtin_amdgcn_exp2f(sc[j][i] - m_run);
                l_run += p[j][i];
            }
        // P^T operand: k-slot e < 4 is token 4grp+e of page 0, e >= 4 token
        // 16 + 4grp + e-4 of page 1 -- the V^T reads below use the same order
        const uint4 pop = make_uint4(cvt2(p[0][0], p[0][1]), cvt2(p[0][2], p[0][3]),
                                     cvt2(p[1][0], p[1][1]), cvt2(p[1][2], p[1][3]));
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            const i16x4 lo = lds_read_tr(vtr + 16 * db);
            const i16x4 hi = lds_read_tr(vtr + 16 * VSTR + 16 * db);
            const bf16x8 a = __builtin_bit_cast(
                bf16x8, make_uint4(__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y,
                                   __builtin_bit_cast(uint2, hi).x, __builtin_bit_cast(uint2, hi).y));
            oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pop), oacc[db], 0, 0, 0);
        }
    }

    // ---- merge the 4 waves: per-head (m, l) and O^T through LDS
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (grp == 0) {
        s_m[wave][col] = m_run;
        s_l[wave][col] = l_run;
    }
    __syncthreads();  // every wave is done with its V buffer: reuse it for O^T
    float *s_o = reinterpret_cast<float *>(s_v);  // [kWaves][128 d][16 heads]
#pragma unroll
    for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) s_o[(wave * kHeadDim + 16 * db + 4 * grp + i) * 16 + col] = oacc[db][i];
    __syncthreads();
    for (int idx = tid; active && idx < group * kHeadDim; idx += kThreads) {
        const int h = idx / kHeadDim, d = idx % kHeadDim;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, s_m[w][h]);
        float lsum = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = s_m[w][h];
            const float wt = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);  // waves without pages
            lsum += wt * s_l[w][h];
            o += wt * s_o[(w * kHeadDim + d) * 16 + h];
        }
        if (direct) {
            out[(static_cast<size_t>(b) * hq + kvh * group + h) * kHeadDim + d] = to_bf16(o / lsum);
        } else {
            // device-scope stores (through the L2 of this XCD): the piece may be
            // merged by a work-group on another XCD without a cache writeback
            __hip_atomic_store(&ws_o[(static_cast<size_t>(slot) * group + h) * kHeadDim + d], o, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            if (d == 0)
                __hip_atomic_store(reinterpret_cast<unsigned long long *>(&ws_ml[static_cast<size_t>(slot) * group + h]),
                                   __builtin_bit_cast(unsigned long long, make_float2(M, lsum)), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// One (sequence, kv head, chunk) work unit of the fixed-chunk split: unit u
// is chunk u / hkv of the batch's chunks in order, kv head u % hkv.  A
// sequence of one chunk is written directly; otherwise the chunk's partial
// goes to slot u and the sequence's first chunk index to ws_cbase[b].
// kGuarded: the caller runs other work in the same work-group, so a unit
// past the end does nothing but still takes the two work-group barriers.
template <bool kGuarded>
__device__ __forceinline__ void
decode_unit(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
            const uint16_t *__restrict__ q, uint16_t *__restrict__ out, const int32_t *__restrict__ seq_lens,
            const int32_t *__restrict__ bt, int bt_stride, float *__restrict__ ws_o, float2 *__restrict__ ws_ml,
            int32_t *__restrict__ ws_cbase, int batch, int hkv, int group, int num_pages, float scale_log2,
            int ch_pages, int u, int tid, uint16_t *s_v, float (*s_m)[16], float (*s_l)[16]) {
    const int kvh = u % hkv;
    int b = 0, c = 0, nch = 0, first = 0;
    const bool found = locate_chunk(seq_lens, batch, ch_pages, bt_stride, u / hkv, b, c, nch, first);
    // more units than the device lengths give (uniform over the 4 waves): a
    // kernel of its own returns; a fused work-group still takes both barriers
    if constexpr (!kGuarded) {
        if (!found) return;
    }
    const int L = min(seq_lens[b], bt_stride * kPageSize);
    const int np_b = (L + kPageSize - 1) / kPageSize;
    decode_pages(kpool, vpool, q, out, bt + static_cast<size_t>(b) * bt_stride, ws_o, ws_ml, b, L, hkv, kvh,
                 group, num_pages, scale_log2, c * ch_pages, min((c + 1) * ch_pages, np_b), found, nch == 1, u,
                 tid, s_v, s_m, s_l);
    if (found && c == 0 && kvh == 0 && tid == 0) ws_cbase[b] = first;
}

// Merges the pieces j = 0 .. nch-1 of segment (b, kv head), piece j's partial
// in workspace slot first + j * stride, into the bf16 output (the combine
// kernel).  One pass over the pieces with a running maximum; each thread
// merges two outputs (h, d), and the (m, l) and o of 8 pieces of both are
// loaded together, so a short segment costs one round of loads.
__device__ __forceinline__ void
merge_pieces(uint16_t *__restrict__ out, const float *__restrict__ ws_o, const float2 *__restrict__ ws_ml,
             int64_t first, int64_t stride, int nch, int b, int hkv, int kvh, int group, int tid) {
    const int hq = hkv * group;
    const int n_out = group * kHeadDim;
    for (int i0 = tid; i0 < n_out; i0 += 2 * kThreads) {
        const int idx[2] = {i0, i0 + kThreads};
        float M[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f}, osum[2] = {0.f, 0.f};
        for (int s0 = 0; s0 < nch; s0 += 8) {
            float2 ml[2][8];
            float o[2][8];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool in = s0 + j < nch && idx[k] < n_out;
                    const int h = in ? idx[k] / kHeadDim : 0, d = idx[k] % kHeadDim;
                    const size_t uu = static_cast<size_t>(first + (s0 + j) * stride) * group + h;
                    ml[k][j] = in ? ws_ml[uu] : make_float2(-INFINITY, 0.f);
                    o[k][j] = in ? ws_o[uu * kHeadDim + d] : 0.f;
                }
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (!(ml[k][j].y > 0.f)) continue;  // a piece without keys contributes nothing
                    const float mn = fmaxf(M[k], ml[k][j].x);
                    const float a = __builtin_amdgcn_exp2f(M[k] - mn), w = __builtin_amdgcn_exp2f(ml[k][j].x - mn);
                    lsum[k] = lsum[k] * a + w * ml[k][j].y;
                    osum[k] = osum[k] * a + w * o[k][j];
                    M[k] = mn;
                }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (idx[k] < n_out) {
                const int h = idx[k] / kHeadDim, d = idx[k] % kHeadDim;
                out[(static_cast<size_t>(b) * hq + kvh * group + h) * kHeadDim + d] = to_bf16(osum[k] / lsum[k]);
            }
    }
}

// ---------------------------------------------------------------- balanced
// The balanced split: 8 waves per work-group, one work-group per CU.
constexpr int kSpanWaves = 8;
constexpr int kSpanThreads = 64 * kSpanWaves;
constexpr int OSTR = kHeadDim + 4;                       // LDS row stride of a staged O (fp32): conflict-free
constexpr int kSpanBufBytes = 16 * kPair * VSTR * 2;     // one wave's K/V buffer (K, then V of a pair)
constexpr int kSpanHeadBytes = 16 * OSTR * 4;            // one wave's first fragment: up to 16 heads
static_assert(kSpanHeadBytes <= kSpanBufBytes && 16 * kPair * KSTR * 2 <= kSpanBufBytes, "buffer of a wave");

// A fragment: consecutive pages of one segment streamed by one wave, as left
// in LDS when the wave does not hold the whole segment.
struct alignas(16) Fragment {
    int seg;      // b * hkv + kv head; -1: none
    int b, kvh;
    int starts;   // holds the segment's first page
    int ends;     // holds its last page
    int u0, nch;  // the segment's first unit and its units
    int pad;
};

struct SpanLds {
    char buf[kSpanWaves][kSpanBufBytes];    // K/V of the pair in work; at the end the wave's last fragment's O
    char head[kSpanWaves][kSpanHeadBytes];  // the wave's first fragment's O
    float m[kSpanWaves][2][16], l[kSpanWaves][2][16];  // [first, last fragment]
    Fragment frag[kSpanWaves * 2];          // [2 wave + (0: first, 1: last)]
    int done[2];                            // the pending segments' pieces are all done
};

// Inclusive scan over the wave's lanes.
__device__ inline int lane_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

__device__ inline float lane63(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
template <int kCtrl, int kRows>
__device__ inline float dpp_or(float other, float x) {  // the lane's source, `other` where it has none
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, other),
                                                                 __builtin_bit_cast(int, x), kCtrl, kRows, 0xf, false));
}
// Maximum and sum over the wave's lanes, in every lane.
__device__ inline float wave_max(float x) {
    x = fmaxf(x, dpp_or<0x111, 0xf>(-INFINITY, x));
    x = fmaxf(x, dpp_or<0x112, 0xf>(-INFINITY, x));
    x = fmaxf(x, dpp_or<0x114, 0xf>(-INFINITY, x));
    x = fmaxf(x, dpp_or<0x118, 0xf>(-INFINITY, x));
    x = fmaxf(x, dpp_or<0x142, 0xa>(-INFINITY, x));
    x = fmaxf(x, dpp_or<0x143, 0xc>(-INFINITY, x));
    return lane63(x);
}
__device__ inline float wave_sum(float x) {
    x += dpp_or<0x111, 0xf>(0.f, x);
    x += dpp_or<0x112, 0xf>(0.f, x);
    x += dpp_or<0x114, 0xf>(0.f, x);
    x += dpp_or<0x118, 0xf>(0.f, x);
    x += dpp_or<0x142, 0xa>(0.f, x);
    x += dpp_or<0x143, 0xc>(0.f, x);
    return lane63(x);
}

// The lengths of 64 consecutive sequences, one per lane, so that walking from
// one sequence to the next waits for no memory.
struct Lengths {
    const int32_t *seq_lens;
    int batch, bt_stride, group0, v;  // v: length of sequence group0 + lane (0 past the batch)
    __device__ __forceinline__ void load(int b) {
        group0 = b & ~63;
        const int bb = group0 + static_cast<int>(threadIdx.x & 63);
        v = bb < batch ? max(0, min(seq_lens[bb], bt_stride * kPageSize)) : 0;
    }
    __device__ __forceinline__ int at(int b) {
        if ((b & ~63) != group0) load(b);
        return __builtin_amdgcn_readlane(v, b & 63);
    }
    __device__ __forceinline__ static int pages(int len) { return (len + kPageSize - 1) / kPageSize; }
};

// Wave-level search for the sequence b whose kv-head segments hold global
// page g of the balanced split (segments in the order (b, kv head), each of
// the sequence's page count, rounded up to a multiple of `align` when it is
// not 0); base = hkv * (such counts of the sequences < b).  Returns false if g
// is past the end.  Page numbers fit 31 bits (the host refuses calls that do
// not).
__device__ __forceinline__ bool locate_page(Lengths &len, int hkv, int align, int g, int &b_out, int &base_out) {
    int running = 0;
    for (int b0 = 0; b0 < len.batch; b0 += 64) {
        len.load(b0);
        int np = Lengths::pages(len.v);
        if (align > 0) np = (np + align - 1) / align * align;
        const int n = hkv * np;
        const int incl = running + lane_scan(n);
        const uint64_t hit = __builtin_amdgcn_ballot_w64(g >= incl - n && g < incl);
        if (hit) {
            const int src = __builtin_ctzll(hit);
            base_out = __builtin_amdgcn_readlane(incl - n, src);
            b_out = b0 + src;
            return true;
        }
        running = __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}

// Merge of one balanced-split segment in the work-group that finished its
// last piece; pieces j = 0 .. nch-1 in slots first + j, read at device scope
// (they were written in this kernel, possibly on other XCDs).  The waves share
// the heads, and with fewer than 8 heads also the pieces of a head.  A wave
// holds the (m, l) of up to 64 pieces of its head one per lane, which gives
// every piece's weight 2^(m - M) and the denominator within the wave, while the
// partial O of 16 pieces of its share are on their way, two outputs per lane;
// shares of one head are added through LDS.  One round of loads up to 16
// pieces per share (reading (m, l) and then O took 4.2 us for 16 pieces of 4
// heads, and one head per wave of 4 with 8 pieces in flight 24 us for 43
// pieces of 8 heads).
constexpr int kMergeAhead = 16;
__device__ __forceinline__ void
merge_segment(uint16_t *__restrict__ out, const float *__restrict__ ws_o, const float2 *__restrict__ ws_ml,
              int64_t first, int nch, int b, int hkv, int kvh, int group, int tid, SpanLds &lds) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float2 *s_acc = reinterpret_cast<float2 *>(lds.buf);  // [wave][lane]
    const int per_head = group == 1 ? 8 : group == 2 ? 4 : group <= 4 ? 2 : 1;  // waves
    const int share = wave % per_head;
    unsigned long long *ml_src = reinterpret_cast<unsigned long long *>(const_cast<float2 *>(ws_ml)) + first * group;
    unsigned long long *o_src = reinterpret_cast<unsigned long long *>(const_cast<float *>(ws_o)) +
                                static_cast<size_t>(first) * group * (kHeadDim / 2) + lane;
    auto write = [&](int h, float2 acc, float L) __attribute__((always_inline)) {
        const float inv = 1.f / L;
        reinterpret_cast<uint32_t *>(out + (static_cast<size_t>(b) * hkv * group + kvh * group + h) * kHeadDim)[lane] =
            cvt2(acc.x * inv, acc.y * inv);
    };
    float L = 0.f;
    for (int h = wave / per_head; h < group; h += kSpanWaves / per_head) {
        float M = -INFINITY;
        float2 acc = make_float2(0.f, 0.f);
        L = 0.f;
        for (int jb = 0; jb < nch; jb += 64) {
            const int n = min(nch - jb, 64);
            const float2 ml = __builtin_bit_cast(
                float2, __hip_atomic_load(ml_src + (jb + min(lane, n - 1)) * group + h, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT));
            float w = 0.f;
            // (every share takes part in the denominator, so at least one turn)
            for (int j0 = share; j0 < n || j0 == share; j0 += kMergeAhead * per_head) {
                float2 o[kMergeAhead];
#pragma unroll
                for (int k = 0; k < kMergeAhead; ++k)
                    o[k] = __builtin_bit_cast(
                        float2, __hip_atomic_load(o_src + ((jb + min(j0 + k * per_head, n - 1)) * group + h) *
                                                              (kHeadDim / 2),
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (j0 == share) {
                    // (a piece without keys contributes nothing)
                    const bool in = lane < n && ml.y > 0.f;
                    const float M_new = fmaxf(M, wave_max(in ? ml.x : -INFINITY));
                    const float old = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - M_new);
                    w = in ? __builtin_amdgcn_exp2f(ml.x - M_new) : 0.f;
                    L = L * old + wave_sum(in ? w * ml.y : 0.f);
                    acc.x *= old;
                    acc.y *= old;
                    M = M_new;
                }
#pragma unroll
                for (int k = 0; k < kMergeAhead; ++k) {
                    const int j = j0 + k * per_head;
                    const float wj =
                        j < n ? __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), j)) : 0.f;
                    acc.x += wj != 0.f ? wj * o[k].x : 0.f;
                    acc.y += wj != 0.f ? wj * o[k].y : 0.f;
                }
            }
        }
        if (per_head > 1)
            s_acc[wave * 64 + lane] = acc;  // one head per wave here
        else
            write(h, acc, L);
    }
    if (per_head > 1) {
        __syncthreads();
        const int h = wave / per_head;
        if (share == 0 && h < group) {
            float2 acc = s_acc[wave * 64 + lane];
            for (int k = 1; k < per_head; ++k) {
                const float2 v = s_acc[(wave + k) * 64 + lane];
                acc.x += v.x;
                acc.y += v.y;
            }
            write(h, acc, L);
        }
    }
}

// A work-group that has written its pieces of split segments (at most two:
// the unit's first and last) marks them done in their flags (this call's
// tag) and reads the segments' other flags, both segments in one round; a
// work-group that finds every piece of a segment done merges the segment and
// clears its flags.  The work-group that marks last always finds them all;
// two that finish together may both merge, writing the same bits.  Pieces
// and flags are written and read with device-scope stores and loads
// (coherent across the XCDs' L2 caches), and each wave waits for its stores
// to complete before the next step; release/acquire fences would instead
// write back and invalidate the whole L2 of the XCD for every work-group, and
// one counter per segment would serialise the pieces' atomics.  A flag from an
// earlier call shows another tag (tags are never 0, the cleared value), so
// the workspace needs no initialisation, and a replay of the same launch (same
// tag) finds the flags cleared.  No work-group waits for another.
struct Pending {
    struct Piece {
        int b, kvh, nch;      // the segment and its pieces
        int64_t first, self;  // workspace slots of its first piece and of this one
    };
    int n;  // pieces: 0, 1 or 2
    Piece p0, p1;
};
__device__ __forceinline__ void
finish_segments(uint16_t *__restrict__ out, const float *__restrict__ ws_o, const float2 *__restrict__ ws_ml,
                uint32_t *__restrict__ flags, uint32_t tag, const Pending &pend, int64_t slots, int hkv, int group,
                int tid, SpanLds &lds) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's piece stores are complete
    __syncthreads();
    const auto in_workspace = [&](const Pending::Piece &p) {
        return p.first >= 0 && p.first + p.nch - 1 < slots && p.self < slots;
    };
    // device lengths that disagree with the host's must not lead outside the
    // workspace
    const bool ok0 = pend.n > 0 && in_workspace(pend.p0), ok1 = pend.n > 1 && in_workspace(pend.p1);
    if (tid == 0) {
        if (ok0) __hip_atomic_store(flags + pend.p0.self, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ok1) __hip_atomic_store(flags + pend.p1.self, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds.done[0] = ok0;
        lds.done[1] = ok1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    // both segments' flags in one round of loads
    for (int j = tid; j < max(ok0 ? pend.p0.nch : 0, ok1 ? pend.p1.nch : 0); j += kSpanThreads) {
        uint32_t f0 = tag, f1 = tag;
        if (ok0 && j < pend.p0.nch)
            f0 = __hip_atomic_load(flags + pend.p0.first + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ok1 && j < pend.p1.nch)
            f1 = __hip_atomic_load(flags + pend.p1.first + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (f0 != tag) lds.done[0] = 0;
        if (f1 != tag) lds.done[1] = 0;
    }
    __syncthreads();
    const bool all0 = lds.done[0] != 0, all1 = lds.done[1] != 0;
    for (int i = 0; i < 2; ++i) {
        if (!(i == 0 ? all0 : all1)) continue;
        const Pending::Piece p = i == 0 ? pend.p0 : pend.p1;
        for (int j = tid; j < p.nch; j += kSpanThreads)
            __hip_atomic_store(flags + p.first + j, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (i == 1 && all0) __syncthreads();  // the first merge is done with the LDS
        merge_segment(out, ws_o, ws_ml, p.first, p.nch, p.b, hkv, p.kvh, group, tid, lds);
    }
}

// One unit (work-group) of the balanced split: global pages [u R, min((u + 1) R,
// total)) of the (sequence, kv head) segments in order, which may cross segment
// boundaries; with `aligned`, every segment is padded to a multiple of R pages
// (the padding holds no pages), so a unit holds one piece of one segment.
//
// The unit's pages are cut into 8 consecutive shares, one per wave, and a wave
// streams its share pair by pair without meeting the others: it walks from one
// segment's fragment into the next with the next pair's loads already in
// flight (its block-table entries read up to 64 at a time a chunk ahead, its Q
// behind the last scores of the old fragment).  A segment that lies whole in
// the share is written out from the registers; the share's first and last
// fragments of others wait in LDS.  After one barrier the work-group adds up
// the fragments of each such segment, writes it out if the unit holds all of
// it, and otherwise leaves the sum as the piece of unit u of segment s in slot
// u + s (u when aligned), to be merged by the work-group that finds every piece
// done (those of units P / R .. (P + pages(b) - 1) / R, P the segment's first
// global page).
//
// Bound by latency on short calls and by HBM on long ones.  Before, a unit was
// 4 waves (two units per CU) that all met for every segment's piece in it, each
// piece with its own cold start: a shard's batch of 128 sequences of one kv head
// (100 MB) took 54 us a step with its append, now 27; 64 sequences of 512-4096
// tokens (645 MB) 118 and 113; one of 4003 tokens 18.3 and 15.5; a whole tiny
// call (4 sequences of up to 512) 19.4 and 7.2 us of kernel time.
//
// K and V of a pair go through one buffer of the wave's, one after the other:
// V waits in its registers until the scores are done.
__device__ __forceinline__ void
decode_span(const uint16_t *__restrict__ kpool, const uint16_t *__restrict__ vpool,
            const uint16_t *__restrict__ q, uint16_t *__restrict__ out, const int32_t *__restrict__ seq_lens,
            const int32_t *__restrict__ bt, int bt_stride, float *__restrict__ ws_o, float2 *__restrict__ ws_ml,
            uint32_t *__restrict__ flags, uint32_t tag, int64_t slots, int batch, int hkv, int group,
            int num_pages, float scale_log2, int per_unit, int total, bool aligned, int u, int tid, SpanLds &lds) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int hq = hkv * group;
    const int align = aligned ? per_unit : 0;
    Lengths len{seq_lens, batch, bt_stride, 0, 0};

    // this wave's share [g, g_end) and where it starts
    const int u0 = u * per_unit;
    int u1 = min(u0 + per_unit, total);
    int b = 0, base = 0, np = 0, nv = 1, kvh = 0, off = 0, seg_len = 0, seg_first = 0;
    auto at_page = [&](int g) __attribute__((always_inline)) {
        if (!locate_page(len, hkv, align, g, b, base)) return false;
        seg_len = len.at(b);
        np = Lengths::pages(seg_len);
        nv = aligned ? (np + align - 1) / align * align : np;
        kvh = (g - base) / nv;
        seg_first = base + kvh * nv;
        off = g - seg_first;
        return true;
    };
    bool live = u0 < u1;
    if (aligned && live) {
        live = at_page(u0);
        u1 = u0 + min(per_unit, np - off);  // the padding holds no pages
    }
    const int share = (u1 - u0 + kSpanWaves - 1) / kSpanWaves;
    const int g = u0 + wave * share;
    int left = live ? min(share, u1 - g) : 0;  // pages of the share not yet given to a chunk
    if (aligned)
        off += wave * share;
    else if (left > 0 && !at_page(g))
        left = 0;

    // ---- the wave's chunks: up to 64 consecutive pages of one segment
    struct Chunk {
        int b, kvh, p, p_end, np, len, first;
        bool valid;
    };
    auto next_chunk = [&]() __attribute__((always_inline)) {
        Chunk c{b, kvh, off, off, np, seg_len, seg_first, left > 0};
        if (!c.valid) return c;
        const int n = min(min(left, np - off), 64);
        c.p_end = off + n;
        left -= n;
        off += n;
        if (off == np && left > 0) {  // on to the next segment
            off = 0;
            seg_first += np;
            if (++kvh == hkv) {
                kvh = 0;
                if (++b < batch) {
                    seg_len = len.at(b);
                    np = Lengths::pages(seg_len);
                } else {
                    np = 0;
                }
                if (np == 0) left = 0;  // device lengths that disagree with the host's
            }
        }
        return c;
    };
    auto table = [&](const Chunk &c) __attribute__((always_inline)) {  // lane i: page of c.p + i
        return bt[static_cast<size_t>(c.b) * bt_stride + min(c.p + lane, c.np - 1)];
    };
    // Q^T operand: column `col` is query head kvh*group + col.  Columns past
    // the group are zero here, and their reference maximum of +inf makes their
    // probabilities zero too: multiplying zeros draws less power, which the
    // prefill on the other CUs gets as clock.
    const bool in_group = col < group;
    uint4 qop[4];
    auto load_q = [&](const Chunk &c) __attribute__((always_inline)) {
        const uint16_t *qp = q + (static_cast<size_t>(c.b) * hq + c.kvh * group + (in_group ? col : 0)) * kHeadDim + 8 * grp;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) qop[kb] = sel4(in_group, *reinterpret_cast<const uint4 *>(qp + 32 * kb));
    };

    char *buf = lds.buf[wave];
    uint16_t *wbuf = reinterpret_cast<uint16_t *>(buf);
    // K operand reads: lane l reads row l%16 of each page, 16-byte chunk 4kb + l/16
    const uint16_t *krd = wbuf + col * KSTR + 8 * grp;
    // transposing-read source: lane s of 16-lane group g -> row 4g + s/4 (+16 for
    // the second page), dims 4(s%4) (+16 db)
    const uint16_t *vtr = wbuf + (4 * grp + (col >> 2)) * VSTR + 4 * (col & 3);
    const int loff = grp * kHeadDim + 8 * col;  // this lane's place in four whole rows of a page

    uint4 kr[kPair][4], vr[kPair][4];
    const uint16_t *kp[kPair], *vp[kPair];  // the pair being loaded
    int pair_ok = 0;                        // bit j: page j of it exists
    auto pair_pages = [&](const Chunk &c, int tbl, int p) __attribute__((always_inline)) {
        pair_ok = 0;
#pragma unroll
        for (int j = 0; j < kPair; ++j) {
            const int page = __builtin_amdgcn_readlane(tbl, min(p + j, c.p_end - 1) - c.p);
            const bool ok = p + j < c.p_end && page >= 0 && page < num_pages;
            pair_ok |= ok ? 1 << j : 0;
            const size_t at = (static_cast<size_t>(ok ? page : 0) * hkv + c.kvh) * (kPageSize * kHeadDim);
            kp[j] = kpool + at;
            vp[j] = vpool + at;
        }
    };
    auto load_pair = [&](uint4(&r)[kPair][4], const uint16_t *const(&src)[kPair], int ok) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kPair; ++j)
            if (ok >> j & 1) {
                // whole 256-byte rows per instruction (four rows each), so no
                // cache line is requested by two instructions
#pragma unroll
                for (int i = 0; i < 4; ++i) r[j][i] = load_stream(src[j] + loff + 4 * i * kHeadDim);
            }
    };

    f32x4 oacc[8];  // O^T[d = 16db + 4grp + i][head = col]
    float m_run = -INFINITY, l_run = 0.f;
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < 8; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run = in_group ? -INFINITY : INFINITY;
        l_run = 0.f;
    };
    if (lane < 2) lds.frag[2 * wave + lane].seg = -1;

    Chunk cur = next_chunk();
    if (cur.valid) {
        int tbl = table(cur);
        load_q(cur);
        reset();
        int frag_p = cur.p;  // first page of the fragment
        Chunk nxt = next_chunk();
        int tbl_n = nxt.valid ? table(nxt) : 0;
        pair_pages(cur, tbl, cur.p);
        load_pair(kr, kp, pair_ok);
        load_pair(vr, vp, pair_ok);
        for (;;) {
            const bool frag_end = !nxt.valid || nxt.b != cur.b || nxt.kvh != cur.kvh;
            for (int p = cur.p; p < cur.p_end; p += kPair) {
                const int ok = pair_ok;
                // a pair with a missing page, or past the sequence's end
                const bool edge = ok != (1 << kPair) - 1 || (p + kPair) * kPageSize > cur.len;
#pragma unroll
                for (int j = 0; j < kPair; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *reinterpret_cast<uint4 *>(wbuf + (16 * j + 4 * i + grp) * KSTR + 8 * col) = kr[j][i];
                // the next pair's K loads go out while this pair is computed,
                // its V loads once this pair's V is in LDS
                const bool last = p + kPair >= cur.p_end;
                const bool more = !last || nxt.valid;
                if (more) {
                    if (last)
                        pair_pages(nxt, tbl_n, nxt.p);
                    else
                        pair_pages(cur, tbl, p + kPair);
                    load_pair(kr, kp, pair_ok);
                }
                // S^T = K Q^T on the matrix core, K read back in the operand layout
                f32x4 sc[kPair];
#pragma unroll
                for (int j = 0; j < kPair; ++j) {
                    sc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) {
                        const uint4 a = *reinterpret_cast<const uint4 *>(krd + 16 * j * KSTR + 32 * kb);
                        sc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, qop[kb]), sc[j], 0, 0, 0);
                    }
                }
                if (last && frag_end && nxt.valid) load_q(nxt);
                // V rows of an absent page or past the sequence's end are zeros (a
                // masked key has p = 0, but 0 times a NaN or Inf in a slack slot
                // would not be 0), and their scores are masked
#pragma unroll
                for (int j = 0; j < kPair; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[j][i] *= scale_log2;
                if (edge) {
#pragma unroll
                    for (int j = 0; j < kPair; ++j)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int tok = (p + j) * kPageSize;
                            vr[j][i] = sel4((ok >> j & 1) && tok + 4 * i + grp < cur.len, vr[j][i]);
                            if (!(ok >> j & 1) || tok + 4 * grp + i >= cur.len) sc[j][i] = -INFINITY;
                        }
                }
                // the pair's maximum per head
                float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                                 fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleLog2) != 0) {
                    const float m_new = fmaxf(m_run, mx);
                    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                    m_run = m_new;
                    l_run *= alpha;
#pragma unroll
                    for (int db = 0; db < 8; ++db) oacc[db] *= alpha;
                }
                float pr[kPair][4];
#pragma unroll
                for (int j = 0; j < kPair; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        pr[j][i] = __builtin_amdgcn_exp2f(sc[j][i] - m_run);
                        l_run += pr[j][i];
                    }
                // P^T operand: k-slot e < 4 is token 4grp+e of page 0, e >= 4 token
                // 16 + 4grp + e-4 of page 1 -- the V^T reads below use the same order
                const uint4 pop = make_uint4(cvt2(pr[0][0], pr[0][1]), cvt2(pr[0][2], pr[0][3]),
                                             cvt2(pr[1][0], pr[1][1]), cvt2(pr[1][2], pr[1][3]));
#pragma unroll
                for (int j = 0; j < kPair; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *reinterpret_cast<uint4 *>(wbuf + (16 * j + 4 * i + grp) * VSTR + 8 * col) = vr[j][i];
                if (more) load_pair(vr, vp, pair_ok);
#pragma unroll
                for (int db = 0; db < 8; ++db) {
                    const i16x4 lo = lds_read_tr(vtr + 16 * db);
                    const i16x4 hi = lds_read_tr(vtr + 16 * VSTR + 16 * db);
                    const bf16x8 a = __builtin_bit_cast(
                        bf16x8, make_uint4(__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y,
                                           __builtin_bit_cast(uint2, hi).x, __builtin_bit_cast(uint2, hi).y));
                    oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, pop), oacc[db], 0, 0, 0);
                }
            }
            if (frag_end) {
                l_run += __shfl_xor(l_run, 16);
                l_run += __shfl_xor(l_run, 32);
                const bool starts = frag_p == 0, ends = cur.p_end == cur.np;
                if (starts && ends) {
                    if (col < group) {
                        const float inv = 1.f / l_run;
                        uint16_t *orow = out + (static_cast<size_t>(cur.b) * hq + cur.kvh * group + col) * kHeadDim + 4 * grp;
#pragma unroll
                        for (int db = 0; db < 8; ++db)
                            *reinterpret_cast<uint2 *>(orow + 16 * db) =
                                make_uint2(cvt2(oacc[db][0] * inv, oacc[db][1] * inv),
                                           cvt2(oacc[db][2] * inv, oacc[db][3] * inv));
                    }
                } else {
                    // only the share's first fragment continues an earlier page
                    const int slot = starts ? 1 : 0;
                    float *so = reinterpret_cast<float *>(starts ? buf : lds.head[wave]);
                    if (col < group) {
#pragma unroll
                        for (int db = 0; db < 8; ++db)
                            *reinterpret_cast<f32x4 *>(so + col * OSTR + 16 * db + 4 * grp) = oacc[db];
                    }
                    if (grp == 0) {
                        lds.m[wave][slot][col] = m_run;
                        lds.l[wave][slot][col] = l_run;
                    }
                    const int extent = aligned ? (cur.np + align - 1) / align * align : cur.np;
                    const int f0 = cur.first / per_unit, f1 = (cur.first + extent - 1) / per_unit;
                    if (lane == 0)
                        lds.frag[2 * wave + slot] =
                            Fragment{cur.b * hkv + cur.kvh, cur.b, cur.kvh, starts, ends, f0, f1 - f0 + 1, 0};
                }
                if (!nxt.valid) break;
                reset();
                frag_p = nxt.p;
            }
            cur = nxt;
            tbl = tbl_n;
            nxt = next_chunk();
            if (nxt.valid) tbl_n = table(nxt);
        }
    }
    __syncthreads();

    // ---- add up the fragments of each segment (in wave order, each wave's
    // first before its last; those of one segment are neighbours).  Lane i
    // holds record i, so finding them is scalar work
    const Fragment fr = lds.frag[lane & (2 * kSpanWaves - 1)];
    const bool mine = lane < 2 * kSpanWaves && fr.seg >= 0;
    uint32_t todo = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(mine));
    const uint32_t valid = todo, starts_at = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(mine && fr.starts)),
                   ends_at = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(mine && fr.ends));
    Pending pend{};
    while (todo) {
        // the run: record i and the first fragments of the waves after it
        const int i = __builtin_ctz(todo), w = i >> 1;
        int j = i, n = 1;
        while (!(ends_at >> j & 1) && (j | 1) + 1 < 2 * kSpanWaves && (valid >> ((j | 1) + 1) & 1)) {
            j = (j | 1) + 1;
            ++n;
        }
        todo &= ~((2u << j) - 1);
        const bool whole = (starts_at >> i & 1) && (ends_at >> j & 1);
        const int seg = __builtin_amdgcn_readlane(fr.seg, i);
        const int sb = __builtin_amdgcn_readlane(fr.b, i), skvh = __builtin_amdgcn_readlane(fr.kvh, i);
        const int64_t shift = aligned ? 0 : seg;  // of the workspace slots
        const int64_t piece = u + shift;
        for (int idx = tid; idx < group * kHeadDim; idx += kSpanThreads) {
            const int h = idx / kHeadDim, d = idx % kHeadDim;
            float mk[kSpanWaves], lk[kSpanWaves], ok[kSpanWaves];
#pragma unroll
            for (int k = 0; k < kSpanWaves; ++k) {
                mk[k] = -INFINITY;
                lk[k] = ok[k] = 0.f;
                if (k < n) {
                    const int s = k == 0 ? i & 1 : 0;
                    mk[k] = lds.m[w + k][s][h];
                    lk[k] = lds.l[w + k][s][h];
                    ok[k] = reinterpret_cast<const float *>(s ? lds.buf[w + k] : lds.head[w + k])[h * OSTR + d];
                }
            }
            float M = mk[0];
#pragma unroll
            for (int k = 1; k < kSpanWaves; ++k) M = fmaxf(M, mk[k]);
            float lsum = 0.f, o = 0.f;
#pragma unroll
            for (int k = 0; k < kSpanWaves; ++k) {
                const float wt = mk[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk[k] - M);  // no keys on valid pages
                lsum += wt * lk[k];
                o += wt * ok[k];
            }
            if (whole) {
                out[(static_cast<size_t>(sb) * hq + skvh * group + h) * kHeadDim + d] = to_bf16(o / lsum);
            } else if (piece < slots) {
                // device-scope stores (through the L2 of this XCD): the piece may be
                // merged by a work-group on another XCD without a cache writeback
                __hip_atomic_store(&ws_o[(static_cast<size_t>(piece) * group + h) * kHeadDim + d], o, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                if (d == 0)
                    __hip_atomic_store(reinterpret_cast<unsigned long long *>(&ws_ml[static_cast<size_t>(piece) * group + h]),
                                       __builtin_bit_cast(unsigned long long, make_float2(M, lsum)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (!whole) {
            const int64_t f0 = __builtin_amdgcn_readlane(fr.u0, i);
            const Pending::Piece pc{sb, skvh, __builtin_amdgcn_readlane(fr.nch, i), f0 + shift, piece};
            if (pend.n == 0)
                pend.p0 = pc;
            else
                pend.p1 = pc;
            pend.n = pend.n == 0 ? 1 : 2;
        }
    }
    if (pend.n > 0)
        finish_segments(out, ws_o, ws_ml, flags, tag, pend, slots, hkv, group, tid, lds);
}

}  // namespace dk
}  // namespace
