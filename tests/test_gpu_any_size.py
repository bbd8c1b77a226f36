"""Sizes and spd addresses at the edges of the full-width kernels' tiles.

One context-parallel step (forward, then backward with the step's own output)
against the fp64 oracle over: fewer than 16 keys, one key either side of the
16-byte group, the 32-key block and the 64-, 128- and 256-key tiles; query
counts either side of the 64-row wave; head counts that make the launch pick
each split of a workgroup's waves (few heads: the widest split; 128 and 256
heads of 300 rows: two groups and none); and spd slices whose first byte and
row stride fall on every residue mod 4, in a buffer that ends with the last
row's last key."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34420_amd as gt
import synth
from gpu_common import DEV, check_fwd, check_grads, say, tdtype, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [
    # (H, Sq, Sk, d, first byte of the slice, row stride - Sk, n_buckets)
    (2, 1, 1, 64, 3, 0, 9),
    (2, 70, 15, 64, 1, 2, 9),
    (2, 64, 16, 64, 2, 1, 9),
    (2, 65, 17, 64, 0, 0, 9),
    (2, 33, 31, 16, 5, 4, 9),
    (2, 127, 33, 8, 7, 0, 9),
    (2, 129, 63, 64, 4, 1, 9),
    (2, 40, 65, 32, 0, 3, 9),
    (2, 200, 127, 64, 1, 0, 200),
    (2, 100, 128, 64, 3, 1, 9),
    (2, 100, 129, 64, 2, 0, 9),
    (1, 300, 255, 32, 6, 0, 9),
    (1, 300, 257, 16, 0, 1, 9),
    (1, 515, 511, 64, 9, 2, 130),
    (1, 130, 769, 64, 0, 0, 9),
    (1, 130, 1000, 64, 0, 0, 9),          # dword rows, ragged
    (1, 130, 1003, 32, 1, 0, 9),
    (128, 300, 301, 64, 1, 2, 9),
    (128, 300, 300, 32, 4, 0, 9),
    (256, 300, 299, 64, 0, 0, 9),
    (256, 300, 300, 16, 8, 4, 9),
    (256, 260, 448, 64, 4, 4, 9),         # whole key tiles, ragged rows
]


def _slice(spd, first, stride):
    """spd [Sq, Sk] in device memory: row i at byte first + i * stride, the
    last row's last key the buffer's last byte."""
    Sq, Sk = spd.shape
    flat = np.full(first + (Sq - 1) * stride + Sk, 255, np.uint8)
    view = np.lib.stride_tricks.as_strided(flat[first:], (Sq, Sk), (stride, 1))
    view[:] = spd
    buf = to_dev(flat, torch.uint8)
    return torch.as_strided(buf, (Sq, Sk), (stride, 1), first)


def run_case(dt, H, Sq, Sk, d, first, pad, nb):
    g = np.random.default_rng(Sq * 1000 + Sk)
    spd = g.integers(0, min(256, nb + 2), size=(Sq, Sk)).astype(np.uint8)
    q, k, v, do = (g.standard_normal((H, n, d)).astype(np.float32) for n in (Sq, Sk, Sk, Sq))
    if dt == "bf16":
        q, k, v, do = (synth.round_bf16(x) for x in (q, k, v, do))
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    scale = 1.0 / np.sqrt(d)
    td = tdtype(dt)
    tag = f"any size {dt} H={H} Sq={Sq} Sk={Sk} d={d} first={first} pad={pad} nb={nb}"
    say(tag)
    Q, K, V, dO, T = to_dev(q, td), to_dev(k, td), to_dev(v, td), to_dev(do, td), to_dev(table)
    S = _slice(spd, first, Sk + pad)
    o, l = gt.gt_attn_ring_step(Q, K, V, S, 0, 0, T, scale=scale)
    torch.cuda.synchronize()
    o_ref, l_ref = oracle.ring_step(q, k, v, spd, 0, 0, table, scale)
    check_fwd(tag, to_np(o), to_np(l), o_ref, l_ref, dt)
    # the backward as a function of its inputs: both sides get the oracle's
    # output in the input dtype
    o_in = o_ref.astype(np.float32)
    o_in = synth.round_bf16(o_in) if dt == "bf16" else o_in
    l_in = l_ref.astype(np.float32)
    acc = gt.gt_attn_bwd_ring_step(Q, to_dev(o_in, td), to_dev(l_in), dO, K, V, S, 0, 0, T, scale=scale)
    torch.cuda.synchronize()
    ref = oracle.ring_backward_step(q, o_in, l_in, do, k, v, spd, 0, 0, table, scale)
    got = dict(zip(("dq", "dk", "dv", "dtable"), (to_np(x) for x in acc)))
    ref = dict(zip(("dq", "dk", "dv", "dtable"), ref))
    for name in ("dq", "dk", "dtable"):
        # one key: P is 1 and dS the rounding of dO.(V - O), no relative bar
        if Sk == 1:
            assert np.abs(got.pop(name) - ref.pop(name)).max() < 0.05
    check_grads(tag, got, ref, dt)


@pytest.mark.parametrize("H,Sq,Sk,d,first,pad,nb", CASES)
def test_any_size_bf16(H, Sq, Sk, d, first, pad, nb):
    run_case("bf16", H, Sq, Sk, d, first, pad, nb)
