"""The attention calls that a user of this library makes, as measured cases.

Every case is one attention layer's step through the C ABI's binding: the KV
append of the new tokens and the attention over the paged cache, for a prefill
batch, for a decode batch, or for both at once on the two CU partitions of one
GPU.  Shapes are those of the workload table in
``paper_2504_14489_amd/workloads.py`` (8B- and 70B-shaped layers, the 70B
layer's share on one GPU at tensor-parallel degree 8, the tiny layer, the long
context layer) and of the GQA groupings its tests run; inputs are N(0, 1) in
bf16 with the query gain that the tests use (1, or 4 for peaked softmaxes).
"""
import math
import random
import weakref

import numpy as np
import torch

from paper_2504_14489_amd import mw
from paper_2504_14489_amd.device import Partition

PAGE = 16
DIM = 128
DEVICE = "cuda"

# (query heads, kv heads) of the layers above and of the groupings 1 .. 16
HEADS = ((32, 8), (64, 8), (8, 1), (8, 2), (32, 32), (4, 4), (2, 1), (12, 2), (6, 2), (16, 1))


def listed():
    return [
        # the smallest step: the tiny layer (256 new tokens, 4 sequences), both
        # phases on half the CUs each; launches and latency are what counts
        dict(name="mux_small", kind="mux", hq=8, hkv=2, pre_batch=1, n_lo=256, n_hi=256, r_lo=0, r_hi=0, dec_batch=4,
             l_lo=128, l_hi=512, dist="uniform", iters=1, pre_cus=128, dec_cus=128, gain=1.0, lens=1),
        # one interactive sequence of a few thousand tokens: decode latency
        dict(name="decode_single", kind="decode", hq=32, hkv=8, dec_batch=1, l_lo=4003, l_hi=4003, dist="uniform",
             gain=1.0, lens=2),
        # an ordinary decode batch: 64 sequences of 512 .. 4096 tokens
        dict(name="decode_8b", kind="decode", hq=32, hkv=8, dec_batch=64, l_lo=512, l_hi=4096, dist="uniform",
             gain=1.0, lens=3),
        # one GPU's share of the 70B layer at TP 8: one kv head, skewed lengths
        dict(name="decode_tp8", kind="decode", hq=8, hkv=1, dec_batch=128, l_lo=64, l_hi=16384, dist="lognormal",
             gain=1.0, lens=4),
        # the largest decode: 32 sequences of 16K .. 32K tokens
        dict(name="decode_long", kind="decode", hq=32, hkv=8, dec_batch=32, l_lo=16384, l_hi=32768, dist="uniform",
             gain=1.0, lens=5),
        # an ordinary prefill: one 2048-token prompt on the whole GPU
        dict(name="prefill_2k", kind="prefill", hq=32, hkv=8, pre_batch=1, n_lo=2048, n_hi=2048, r_lo=0, r_hi=0,
             gain=1.0, lens=6),
        # a later chunk of a long prompt on one GPU of TP 8 (one kv head)
        dict(name="prefill_tp8", kind="prefill", hq=8, hkv=1, pre_batch=1, n_lo=2048, n_hi=2048, r_lo=4096, r_hi=4096,
             gain=1.0, lens=7),
        # the largest prefill: 4096 new tokens over a 28672-token cached prefix
        dict(name="prefill_long", kind="prefill", hq=32, hkv=8, pre_batch=1, n_lo=4096, n_hi=4096, r_lo=28672,
             r_hi=28672, gain=1.0, lens=8),
        # a batch of prompts of ragged lengths, some over a reused prefix
        dict(name="prefill_ragged", kind="prefill", hq=32, hkv=8, pre_batch=12, n_lo=17, n_hi=1500, r_lo=0, r_hi=4000,
             gain=4.0, lens=9),
        # multi-head attention (one query head per kv head), a chunk over a prefix
        dict(name="prefill_mha", kind="prefill", hq=32, hkv=32, pre_batch=1, n_lo=1000, n_hi=1000, r_lo=1003,
             r_hi=1003, gain=1.0, lens=10),
        # both phases at once: the 70B layer's last 2048-token chunk of an 8K
        # prompt on 96 CUs next to its decode batch on 160
        dict(name="mux_70b", kind="mux", hq=64, hkv=8, pre_batch=1, n_lo=2048, n_hi=2048, r_lo=6144, r_hi=6144,
             dec_batch=128, l_lo=64, l_hi=16384, dist="lognormal", iters=3, pre_cus=96, dec_cus=160, gain=1.0, lens=11),
        # both phases at once on the long context layer, five decode iterations
        # next to one prefill chunk
        dict(name="mux_long", kind="mux", hq=32, hkv=8, pre_batch=1, n_lo=4096, n_hi=4096, r_lo=28672, r_hi=28672,
             dec_batch=32, l_lo=16384, l_hi=32768, dist="uniform", iters=5, pre_cus=128, dec_cus=128, gain=1.0,
             lens=12),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same ranges: any grouping, batch and length up to those
    listed, odd sizes included, every kind of step."""
    kind = rng.choice(["decode", "prefill", "prefill", "mux"])
    hq, hkv = rng.choice(HEADS)
    case = dict(kind=kind, hq=hq, hkv=hkv)
    if kind in ("prefill", "mux"):
        batch = _log_int(rng, 1, 16)
        n_hi = _log_int(rng, 1, 4096)
        r_hi = rng.choice([0, _log_int(rng, 1, 28672)])
        # at most the long context layer's work
        while batch * n_hi * (r_hi + n_hi) * hq > 4096 * 32768 * 32 // 2:
            batch, r_hi = max(1, batch // 2), r_hi // 2
            n_hi = n_hi if batch > 1 or r_hi > 0 else n_hi // 2
        case.update(pre_batch=batch, n_lo=max(1, n_hi // rng.choice([1, 2, 16])), n_hi=n_hi,
                    r_lo=r_hi // rng.choice([1, 2, 16]), r_hi=r_hi)
    if kind in ("decode", "mux"):
        l_hi = _log_int(rng, 64, 32768)
        most = (1 << 31) // (512 * hkv * l_hi)  # at most 2 GiB of K and V
        case.update(dec_batch=_log_int(rng, 1, max(1, min(256, most))), l_lo=max(1, l_hi // rng.choice([1, 2, 8])),
                    l_hi=l_hi, dist=rng.choice(["uniform", "lognormal"]))
    if kind == "mux":
        pre_cus = 32 * rng.randint(1, 7)
        case.update(iters=rng.randint(1, 3), pre_cus=pre_cus, dec_cus=256 - pre_cus)
    case.update(gain=rng.choice([1.0, 1.0, 4.0]), lens=rng.randint(100, 1 << 20))
    return case


def _lengths(case):
    """(new tokens, prefixes) of the prefill sequences and the decode lengths:
    part of the case, the same for every seed."""
    rng = random.Random(case["lens"])
    new, prefix, dec = [], [], []
    for _ in range(case.get("pre_batch", 0)):
        new.append(rng.randint(case["n_lo"], case["n_hi"]))
        prefix.append(rng.randint(case["r_lo"], case["r_hi"]))
    for _ in range(case.get("dec_batch", 0)):
        if case["dist"] == "lognormal":
            mid = min(2048, math.sqrt(case["l_lo"] * case["l_hi"]))
            dec.append(min(case["l_hi"], max(case["l_lo"], int(round(math.exp(rng.gauss(math.log(mid), 0.8)))))))
        else:
            dec.append(rng.randint(case["l_lo"], case["l_hi"]))
    return new, prefix, dec


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device=DEVICE)


def _pages(tokens):
    return -(-tokens // PAGE)


class _Inputs:
    """Pool, block tables, queries and new K/V rows of a case, on the GPU."""

    def __init__(self, case, seed):
        gen = torch.Generator(device=DEVICE).manual_seed(int(seed))

        def normal(*shape):
            return torch.randn(*shape, generator=gen, device=DEVICE, dtype=torch.bfloat16)

        self.hq, self.hkv = case["hq"], case["hkv"]
        self.new, self.prefix, self.dec = _lengths(case)
        pages = [_pages(n + r) for n, r in zip(self.new, self.prefix)] + [_pages(length) for length in self.dec]
        total = sum(pages) + 1
        self.num_pages = total
        self.k = normal(total, self.hkv, PAGE, DIM)
        self.v = normal(total, self.hkv, PAGE, DIM)
        # pages dealt from one random permutation; tables padded with the spare page
        order = torch.randperm(total, generator=gen, device=DEVICE).int()
        at, rows = 0, []
        for count in pages:
            rows.append(order[at:at + count])
            at += count

        def table(part):
            width = max(len(row) for row in part)
            out = order[-1].repeat(len(part), width)
            for i, row in enumerate(part):
                out[i, :len(row)] = row
            return out.contiguous()

        split = len(self.new)
        self.rows = rows
        self.pre_table = table(rows[:split]) if self.new else None
        self.dec_table = table(rows[split:]) if self.dec else None
        n_tokens = sum(self.new)
        self.q_pre = normal(n_tokens, self.hq, DIM) * case["gain"]
        self.k_pre, self.v_pre = normal(n_tokens, self.hkv, DIM), normal(n_tokens, self.hkv, DIM)
        self.q_dec = normal(len(self.dec), self.hq, DIM) * case["gain"]
        self.k_dec, self.v_dec = normal(len(self.dec), self.hkv, DIM), normal(len(self.dec), self.hkv, DIM)


_partitions = {}


def _partition(pre_cus, dec_cus):
    """A program makes its partitions once and keeps them."""
    if (pre_cus, dec_cus) not in _partitions:
        part = _partitions[pre_cus, dec_cus] = Partition(pre_cus, dec_cus)
        weakref.finalize(part, mw.mw_partition_destroy, part.h)
    return _partitions[pre_cus, dec_cus]


class _State(_Inputs):
    """What a serving program has in hand: the inputs, its pool handle, host
    and device copies of the lengths, output buffers and workspaces."""

    def __init__(self, case, seed):
        super().__init__(case, seed)
        self.iters = case.get("iters", 1)
        self.scale = 1.0 / math.sqrt(DIM)
        self.pool = mw.mw_kv_pool_create(self.num_pages, PAGE, self.hkv, DIM, self.k.data_ptr(), self.v.data_ptr())
        weakref.finalize(self, mw.mw_kv_pool_destroy, self.pool)
        if case["kind"] == "mux":
            part = _partition(case["pre_cus"], case["dec_cus"])
            self.pre_stream, self.dec_stream = part.prefill_stream, part.decode_stream
        else:
            self.pre_stream = self.dec_stream = torch.cuda.current_stream().cuda_stream
        if self.new:
            self.h_new, self.h_prefix = np.array(self.new, np.int32), np.array(self.prefix, np.int32)
            self.d_indptr = _i32([0] + list(np.cumsum(self.new)))
            self.d_prefix = _i32(self.prefix)
            self.o_pre = torch.zeros_like(self.q_pre)
            size = mw.mw_prefill_workspace_size(self.hq, self.hkv, DIM, self.h_new, self.h_prefix)
            self.pre_ws = torch.empty(max(size, 16), dtype=torch.uint8, device=DEVICE)
        if self.dec:
            self.h_dec, self.h_last = np.array(self.dec, np.int32), np.array(self.dec, np.int32) - 1
            self.h_one = np.ones(len(self.dec), np.int32)
            self.d_dec, self.d_last = _i32(self.dec), _i32([length - 1 for length in self.dec])
            self.d_one = _i32(list(range(len(self.dec) + 1)))
            self.o_dec = torch.zeros_like(self.q_dec)
            size = mw.mw_decode_workspace_size(self.hq, self.hkv, DIM, self.h_dec)
            self.dec_ws = torch.empty(max(size, 16), dtype=torch.uint8, device=DEVICE)

    def decode(self):
        mw.mw_kv_pool_write(self.pool, self.h_one, self.h_last, self.d_one.data_ptr(), self.d_last.data_ptr(),
                            self.dec_table.data_ptr(), self.dec_table.shape[1], self.k_dec.data_ptr(),
                            self.v_dec.data_ptr(), self.dec_stream)
        mw.mw_decode_attn(self.pool, self.hq, self.hkv, DIM, self.scale, self.h_dec, self.d_dec.data_ptr(),
                          self.dec_table.data_ptr(), self.dec_table.shape[1], self.q_dec.data_ptr(),
                          self.o_dec.data_ptr(), self.dec_ws.data_ptr(), self.dec_ws.numel(), 0, self.dec_stream)

    def prefill(self):
        mw.mw_kv_pool_write(self.pool, self.h_new, self.h_prefix, self.d_indptr.data_ptr(), self.d_prefix.data_ptr(),
                            self.pre_table.data_ptr(), self.pre_table.shape[1], self.k_pre.data_ptr(),
                            self.v_pre.data_ptr(), self.pre_stream)
        mw.mw_prefill_attn_ws(self.pool, self.hq, self.hkv, DIM, self.scale, self.h_new, self.h_prefix,
                              self.d_indptr.data_ptr(), self.d_prefix.data_ptr(), self.pre_table.data_ptr(),
                              self.pre_table.shape[1], self.q_pre.data_ptr(), self.o_pre.data_ptr(),
                              self.pre_ws.data_ptr(), self.pre_ws.numel(), self.pre_stream)


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    """One step: decode is enqueued first, as the multiplexing scheduler does."""
    out = {}
    if state.dec:
        for _ in range(state.iters):
            state.decode()
        out["dec"] = state.o_dec
    if state.new:
        state.prefill()
        out["pre"] = state.o_pre
    out["k"], out["v"] = state.k, state.v
    return out


def work(case):
    """K and V of every visible token read once, Q read and O written once, the
    new rows read and written once; QK^T and PV over the visible pairs only."""
    hq, hkv = case["hq"], case["hkv"]
    new, prefix, dec = _lengths(case)
    row = 2 * DIM
    nbytes = flops = 0
    for n, r in zip(new, prefix):
        nbytes += 2 * (n + r) * hkv * row + 2 * n * hq * row + 4 * n * hkv * row + 4 * _pages(n + r)
        flops += 4 * DIM * hq * (n * r + n * (n + 1) // 2)
    iters = case.get("iters", 1)
    for length in dec:
        nbytes += iters * (2 * length * hkv * row + 2 * hq * row + 4 * hkv * row + 4 * _pages(length))
        flops += iters * 4 * DIM * hq * length
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Both phases round the softmax's weights and the outputs to bf16 (a
    relative 2^-9 each): against 64 bits the listed and drawn cases measure
    1.8e-3 to 2.4e-3 off in the 2-norm, and no value by more than 0.03 of the
    result's root mean square (or of itself); four times that is stated."""
    return {"rel": 9e-3, "max": 0.12}


def _attend(q, k, v, prefix):
    """softmax(q k^T / sqrt(DIM)) v in 64 bits for one kv head; q [n][g][DIM],
    k, v [L][DIM]; query i sees keys 0 .. prefix + i."""
    n, g, _ = q.shape
    length = k.shape[0]
    kt, v = k.double().t().contiguous(), v.double()
    out = torch.empty(n, g, DIM, dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 26) // (g * length))
    keys = torch.arange(length, device=DEVICE)
    for i in range(0, n, step):
        rows = q[i:i + step].double()
        m = rows.shape[0]
        s = (rows.reshape(m * g, DIM) @ kt).reshape(m, g, length) / math.sqrt(DIM)
        last = prefix + i + torch.arange(m, device=DEVICE)
        s.masked_fill_((keys[None, :] > last[:, None])[:, None, :], -math.inf)
        out[i:i + step] = (torch.softmax(s, dim=-1).reshape(m * g, length) @ v).reshape(m, g, DIM)
    return out


def exact(case, seed):
    inp = _Inputs(case, seed)
    group = inp.hq // inp.hkv
    k_pool, v_pool = inp.k, inp.v

    def append(pages, first, k_new, v_new):
        pos = torch.arange(first, first + k_new.shape[0], device=DEVICE)
        page, slot = pages.long()[pos // PAGE], pos % PAGE
        k_pool[page, :, slot] = k_new
        v_pool[page, :, slot] = v_new

    def dense(pool, pages, length):
        return pool[pages.long()].permute(1, 0, 2, 3).reshape(inp.hkv, -1, DIM)[:, :length]

    def attention(pages, prefix, q):
        k, v = dense(k_pool, pages, prefix + q.shape[0]), dense(v_pool, pages, prefix + q.shape[0])
        heads = [_attend(q[:, h * group:(h + 1) * group], k[h], v[h], prefix) for h in range(inp.hkv)]
        return torch.cat(heads, dim=1)

    out, row = {}, 0
    o_pre = []
    for n, r, pages in zip(inp.new, inp.prefix, inp.rows):
        append(pages, r, inp.k_pre[row:row + n], inp.v_pre[row:row + n])
        o_pre.append(attention(pages, r, inp.q_pre[row:row + n]))
        row += n
    o_dec = []
    for i, (length, pages) in enumerate(zip(inp.dec, inp.rows[len(inp.new):])):
        append(pages, length - 1, inp.k_dec[i:i + 1], inp.v_dec[i:i + 1])
        o_dec.append(attention(pages, length - 1, inp.q_dec[i:i + 1]))
    if o_dec:
        out["dec"] = torch.cat(o_dec)
    if o_pre:
        out["pre"] = torch.cat(o_pre)
    out["k"], out["v"] = k_pool, v_pool
    return out
