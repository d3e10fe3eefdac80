// Where a dual prefill block's two wave groups leave their results in LDS when
// they merge (host code checks the regions against each other).
//
// A group owns its K buffers and its V buffers (two tiles of 64 keys each); the
// block-table copy is shared.  At the merge no wave reads any of them as keys,
// values or table entries any more.  Offsets are in bytes:
//   group's K buffers   the half of its O that the other group finishes
//   table copy          both groups' (m, l) words
//   group's V buffers   the output half rows on their way to whole-row stores
// A wave stages as soon as it has read the other group's words, while others
// may still be reading theirs, so the staged rows must not share a byte with
// what those read.  (With the words at the start of the V buffers and the rows
// behind them, the last wave's fp32 rows ended 1 KiB past the buffers, on the
// other group's words.)
#pragma once
#include "mw_internal.h"

namespace mw {

constexpr int kDualBufBytes = 2 * 64 * kHeadDim * 2;  // one group's K (or V) buffers
constexpr int kDualTableBytes = 4096 * 4;             // the block-table copy
constexpr int kDualWaveBytes = 32 * 64 * 4;           // 32 rows x 64 dims of fp32

// Of wave `wave` (0..3) of a group: in its group's K buffers, float4 per lane.
__host__ __device__ constexpr int dual_hand_over(int wave) { return wave * kDualWaveBytes; }
// (m, l) of row 0..127 of the block as group `grp` left it, in the table copy.
__host__ __device__ constexpr int dual_ml(int grp, int row) { return (grp * 128 + row) * 8; }
// Of wave `wave`, in its group's V buffers; within it 16-byte chunk c of row q
// (0..31) of the half tile in fp32 (16 chunks) or bf16 (8 chunks), permuted so
// that neither the writes nor the reads conflict.
__host__ __device__ constexpr int dual_stage(int wave) { return wave * kDualWaveBytes; }
__host__ __device__ constexpr int dual_stage_f32(int row, int c) { return row * 256 + 16 * (c ^ (row & 15)); }
__host__ __device__ constexpr int dual_stage_bf16(int row, int c) { return row * 128 + 16 * (c ^ (row & 7)); }

static_assert(dual_hand_over(4) <= kDualBufBytes, "the hand-over of four waves fits the K buffers");
static_assert(dual_stage(4) <= kDualBufBytes, "the staged rows of four waves fit the V buffers");
static_assert(dual_ml(2, 0) <= kDualTableBytes, "both groups' (m, l) fit the table copy");

}  // namespace mw
