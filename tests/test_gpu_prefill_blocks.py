"""Prefill query blocks on the GPU against the CPU oracle: rows of every GQA
grouping laid end to end (block edges at 128 and 256 rows), the blocks whose
keys two wave groups share, their key-range pieces, and the order of the blocks
over a whole batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_14489_amd import mw
from paper_2504_14489_amd.device import Partition, to_bits
from tests.helpers import assert_close, say
from tests.test_gpu_prefill import _varlen_setup

pytestmark = pytest.mark.gpu


def _run(hq, hkv, seqs, cus, seed, bad_from=None, ws_pieces=None):
    """The batch through the split-enabled and the plain entry point on the
    prefill stream of `cus` CUs (0: the whole GPU); every row of both against
    the oracle.  ws_pieces: the workspace holds this many pieces (0: none is
    passed) instead of the most any stream can need.  bad_from: the one sequence's values from this token on are NaN or
    infinite, and only rows that may not depend on them are compared."""
    wls, k, v, bt, stride, q = _varlen_setup(seqs, hq, hkv, seed)
    if bad_from is not None:
        v = v.copy()
        for tok in range(bad_from, sum(seqs[0])):
            v[bt[0, tok // 16], :, tok % 16] = (0x7FC0, 0x7F80, 0xFF80)[tok % 3]  # bf16 NaN, inf, -inf
    dev = torch.device("cuda:0")
    t16 = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).to(dev)
    t32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(dev)
    dk, dv, dq, dbt = t16(k), t16(v), t16(q), t32(bt)
    ns, rs = [n for _, n in seqs], [r for r, _ in seqs]
    indptr, pref = t32(np.cumsum([0] + ns)), t32(rs)
    pool = mw.mw_kv_pool_create(k.shape[0], 16, hkv, 128, dk.data_ptr(), dv.data_ptr())
    part = Partition(cus, 256 - cus) if cus else None
    outs = []
    try:
        stream = part.prefill_stream if part else 0
        nbytes = mw.mw_prefill_workspace_size(hq, hkv, 128, ns, rs, 0)
        if ws_pieces is not None:
            nbytes = ws_pieces * sum(ns) * hq * 520
        ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=dev)
        ws_args = (ws.data_ptr() if nbytes else 0, nbytes)
        for split in (True, False):
            do = torch.zeros_like(dq)
            args = (pool, hq, hkv, 128, 1 / np.sqrt(128), ns, rs, indptr.data_ptr(), pref.data_ptr(), dbt.data_ptr(),
                    stride, dq.data_ptr(), do.data_ptr())
            if split:
                mw.mw_prefill_attn_ws(*args, *ws_args, stream)
            else:
                mw.mw_prefill_attn(*args, stream)
            torch.cuda.synchronize()
            outs.append(to_bits(do))
    finally:
        if part:
            part.close()
        mw.mw_kv_pool_destroy(pool)
    for got, what in zip(outs, ("split-enabled", "plain")):
        row = 0
        for w, (r, n) in zip(wls, seqs):
            if bad_from is not None:
                # whole 64-position groups whose last key tile of 64 ends by bad_from
                seen = max(i for i in range(0, n, 64) if -(-(r + i) // 64) * 64 <= bad_from)
                assert seen > 0
                ref = oracle.prefill(w.q_pre[r:r + seen], w.k_pool, w.v_pool, w.pre_bt, r)
                assert_close(got[row:row + seen], ref, f"{what} hq={hq} hkv={hkv} r={r} n={n} cus={cus} bad values")
            elif n:
                ref = oracle.prefill(w.q_pre[r:r + n], w.k_pool, w.v_pool, w.pre_bt, r)
                assert_close(got[row:row + n], ref, f"{what} hq={hq} hkv={hkv} r={r} n={n} cus={cus}")
            row += n


# one sequence, groups 1 .. 40 (above 32 a row offset holds one head change at
# most): the last block full, one row short of it and one row over it; prefixes
# that leave the diagonal inside one tile, across two and across three; on the
# whole GPU and on 8 CUs (256-row blocks for the larger calls)
@pytest.mark.parametrize("hq,hkv", [(2, 2), (3, 1), (10, 2), (7, 1), (24, 2), (16, 1), (40, 1)])
@pytest.mark.parametrize("cus", [0, 8])
def test_prefill_row_blocks(hq, hkv, cus):
    g = hq // hkv
    for r, rows in ((0, 128), (63, 127), (64, 129), (130, 257), (1, 640)):
        n = max(1, rows // g)
        for nn in sorted({n, n + 1}):
            say(f"prefill row blocks hq={hq} hkv={hkv} r={r} n={nn} cus={cus}")
            _run(hq, hkv, [(r, nn)], cus, 500 + 7 * hq + nn)


# (prefix, new): one to five key tiles (an odd count leaves a wave group without
# its last tile, one tile leaves it without any; rows that see none of a
# group's keys), and ranges long enough to be cut into several pieces
@pytest.mark.parametrize("r,n", [(0, 1), (0, 64), (0, 65), (0, 128), (63, 66), (0, 200), (190, 127), (1500, 1),
                                 (3000, 257), (9000, 40)])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (1, 1)])
def test_prefill_shared_keys(r, n, hq, hkv):
    say(f"prefill shared keys r={r} n={n} hq={hq} hkv={hkv}")
    _run(hq, hkv, [(r, n)], 0, 900 + n)


# batches at the limit of the ordering over the whole batch (64 sequences) and
# past it, with empty sequences, equal ones and one much longer than the rest
# (the host check of the launch planners, batch_order, holds that these very
# batches are planned in that order, on 8 CUs as on 256, up to 64 sequences)
@pytest.mark.parametrize("batch", [2, 63, 64, 65])
@pytest.mark.parametrize("cus", [0, 8])
def test_prefill_batch_order(batch, cus):
    seqs = [(53 * b % 1201, 1 + 29 * b % 97) for b in range(batch)]
    seqs[0] = (300, 700)
    if batch == 2:
        seqs = [(2000, 759), (1900, 61)]
    else:
        seqs[3], seqs[batch - 1] = (seqs[3][0], 0), (seqs[-1][0], 0)
        seqs[10:20] = [(600, 33)] * 10
    say(f"prefill batch order {batch} sequences on {cus or 'all'} CUs")
    _run(8, 2, seqs, cus, 77)


# more than two rounds of 256-row blocks on 8 CUs, the last of at most half a
# round (run as dual halves): one sequence of 17 and of 20 blocks (the heaviest
# block one row long or full, so that a half may be empty), a batch whose
# lightest block is long enough, groups of 4, 3 and 1
@pytest.mark.parametrize("hq,hkv,seqs", [(4, 1, [(1500, 64 * 16 + 1)]), (4, 1, [(1500, 64 * 20)]),
                                         (6, 2, [(1203, 85 * 8 + 7)]), (2, 2, [(3000, 9 * 256 + 130)]),
                                         (4, 1, [(1400, 500), (1501, 513), (1333, 100)])])
def test_prefill_last_round_in_halves(hq, hkv, seqs):
    say(f"prefill last round in halves hq={hq} hkv={hkv} {seqs}")
    _run(hq, hkv, seqs, 8, 1300)


# values that are not finite from the second, third or last key tile on, which
# lie past every position of the rows compared: a row's softmax gives them no
# weight, and 0 times them must not reach the row through the other rows of its
# block (up to 256 positions with one query head per kv head)
@pytest.mark.parametrize("hq,hkv", [(2, 2), (3, 1), (4, 2), (10, 2), (8, 2), (16, 1)])
@pytest.mark.parametrize("r,n,bad_from", [(0, 256, 64), (64, 250, 192), (130, 300, 384), (0, 500, 448)])
@pytest.mark.parametrize("cus", [0, 8])
def test_prefill_later_values_not_finite(hq, hkv, r, n, bad_from, cus):
    say(f"prefill later values not finite hq={hq} hkv={hkv} r={r} n={n} from {bad_from} cus={cus}")
    _run(hq, hkv, [(r, n)], cus, 1700 + n, bad_from)


# workspaces short of the pieces the plan would take: none where blocks of 32
# positions x four heads are more than the CUs (the call runs uncut), three pieces
# of four; and none for a call that has always been cut, which is refused
@pytest.mark.parametrize("hq,hkv,seqs,cus,wanted,given", [
    (16, 1, [(3314, 181), (1958, 168), (3991, 269), (4818, 125), (3609, 73), (5154, 229), (7218, 221), (3371, 200),
             (3815, 106), (5246, 118), (7240, 170), (6627, 73)], 128, 2, 0),
    (32, 8, [(10732, 3), (8417, 4), (4165, 3)], 32, 4, 3)])
def test_prefill_short_workspace(hq, hkv, seqs, cus, wanted, given):
    say(f"prefill short workspace hq={hq} hkv={hkv} {seqs} cus={cus}")
    ns, rs = [n for _, n in seqs], [r for r, _ in seqs]
    assert mw.mw_prefill_workspace_size(hq, hkv, 128, ns, rs, cus) == wanted * sum(ns) * hq * 520
    _run(hq, hkv, seqs, cus, 2100, ws_pieces=given)


def test_prefill_missing_workspace_is_refused():
    with pytest.raises(mw.MWError) as e:
        _run(8, 1, [(6144, 2048)], 96, 2200, ws_pieces=0)
    assert e.value.status == mw.MW_ERR_INVALID_ARG
