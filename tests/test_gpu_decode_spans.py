"""The balanced decode split on the GPU against the CPU oracle, at the sizes
where its pieces change shape: segments held whole by a work-group, by a wave
or by neither, waves whose share starts or ends inside a segment, and segments
cut into more pieces than a wave has lanes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_14489_amd import workloads as W
from paper_2504_14489_amd.device import DeviceWorkload, Partition, to_bits
from tests.helpers import assert_close, say

pytestmark = pytest.mark.gpu


def _check(hq, hkv, lens, cus, seed, q_scale=1.0):
    say(f"decode spans hq={hq} hkv={hkv} {len(lens)} sequences of {min(lens)}..{max(lens)} on {cus or 'all'} CUs")
    cfg = W.custom_config(hq=hq, hkv=hkv, pre_chunks=((0, 1),), dec_batch=len(lens), seed=seed)
    wl = W.make_workload(cfg, dec_lens=np.array(lens), q_scale=q_scale)
    dw = DeviceWorkload(wl)
    part = Partition(256 - cus, cus) if cus else None
    try:
        outs = []
        for _ in range(2):
            dw.o_dec.zero_()
            torch.cuda.synchronize()
            o = dw.decode(part.decode_stream if part else 0)
            torch.cuda.synchronize()
            outs.append(to_bits(o).copy())
    finally:
        if part:
            part.close()
        dw.close()
    assert np.array_equal(outs[0], outs[1]), "run-to-run results differ"
    ref = oracle.decode(wl.q_dec, wl.k_pool, wl.v_pool, wl.dec_bt, wl.dec_lens)
    assert_close(outs[0], ref, f"decode spans hq={hq} hkv={hkv} cus={cus}")


# segments whole in a work-group (up to three pairs per wave) and just past
# that; a single token, a full page, one token over it; an odd page in a pair
@pytest.mark.parametrize("pages", [1, 2, 3, 15, 16, 17, 33, 47, 48, 49, 64, 65])
def test_decode_whole_segments(pages):
    for tail in (1, 16):
        _check(8, 2, [16 * (pages - 1) + tail] * 3, 0, 40 + pages)


# a wave's share holds many whole segments, the ends of two others, or none;
# more sequences than a wave has lanes, and empty shares at the last unit's end
@pytest.mark.parametrize("cus", [8, 64, 0])
@pytest.mark.parametrize("lo,hi,batch", [(1, 16, 130), (1, 60, 200), (100, 700, 67), (1, 3000, 65)])
def test_decode_shares_across_segments(lo, hi, batch, cus):
    rng = np.random.default_rng(batch)
    _check(6, 2, [int(x) for x in rng.integers(lo, hi + 1, batch)], cus, 60 + batch, q_scale=4.0)


# one sequence cut into 244 pieces of 18 pages on the whole GPU (four blocks of 64
# in the merge's lanes), for every number of waves per head and heads per wave
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5, 8, 9, 16])
def test_decode_many_pieces(group):
    _check(group, 1, [70001], 0, 80 + group, q_scale=4.0)
    _check(2 * group, 2, [16385, 9000, 20011], 96, 90 + group)
