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


# More than 127 buckets in dK/dV: each split of the waves with each of its two
# LDS layouts (d = 64: the four-way split keeps 16 table copies, the others
# have 32), the largest byte value, and bytes past the last bucket.
@pytest.mark.parametrize("H,Sq,Sk,d,first,pad,nb", [
    (1, 130, 300, 64, 0, 0, 256), (1, 130, 300, 32, 1, 0, 256), (1, 70, 100, 8, 0, 0, 128),
    (128, 300, 300, 64, 0, 0, 256), (128, 300, 301, 32, 1, 2, 255), (256, 300, 299, 64, 0, 0, 128),
    (256, 256, 512, 64, 0, 0, 256), (256, 300, 300, 16, 8, 4, 200),
])
def test_many_buckets_bf16(H, Sq, Sk, d, first, pad, nb):
    run_case("bf16", H, Sq, Sk, d, first, pad, nb)


# The histogram is cleared for the table's buckets only: every layout with one,
# two and three buckets, and with bytes far past them.
@pytest.mark.parametrize("H,Sq,Sk,d,nb", [(1, 70, 100, 64, 1), (1, 70, 100, 8, 3), (256, 300, 300, 64, 2),
                                          (128, 300, 300, 64, 1), (1, 130, 300, 64, 128), (256, 300, 300, 64, 129)])
def test_few_buckets_of_many_bytes_bf16(H, Sq, Sk, d, nb):
    g = np.random.default_rng(nb)
    spd = g.integers(0, 256, size=(Sq, Sk)).astype(np.uint8)
    q, k, v, do = (synth.round_bf16(g.standard_normal((H, n, d)).astype(np.float32)) for n in (Sq, Sk, Sk, Sq))
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    scale = 1.0 / np.sqrt(d)
    say(f"few buckets H={H} Sq={Sq} Sk={Sk} d={d} nb={nb}")
    bf = torch.bfloat16
    o, l = oracle.ring_step(q, k, v, spd, 0, 0, table, scale)
    o, l = synth.round_bf16(o.astype(np.float32)), l.astype(np.float32)
    acc = gt.gt_attn_bwd_ring_step(to_dev(q, bf), to_dev(o, bf), to_dev(l), to_dev(do, bf), to_dev(k, bf), to_dev(v, bf),
                                   to_dev(spd, torch.uint8), 0, 0, to_dev(table), scale=scale)
    torch.cuda.synchronize()
    ref = oracle.ring_backward_step(q, o, l, do, k, v, spd, 0, 0, table, scale)
    names = ("dq", "dk", "dv", "dtable")
    check_grads(f"few buckets nb={nb}", dict(zip(names, (to_np(x) for x in acc))), dict(zip(names, ref)), "bf16")


@pytest.mark.parametrize("H,Sq,Sk,d,first,pad,nb", CASES)
def test_any_size_f32(H, Sq, Sk, d, first, pad, nb):
    run_case("f32", H, Sq, Sk, d, first, pad, nb)


def test_f32_nonfinite_gradients():
    """fp32: a NaN dO row reaches every bucket its row holds, and no other; a
    row whose every score is -inf contributes nothing, whatever its dO."""
    H, N, d, nb = 2, 200, 32, 12
    g = np.random.default_rng(3)
    spd = g.integers(1, 8, size=(N, N)).astype(np.uint8)
    spd[5] = g.integers(8, 11, size=N)           # buckets 8..10: row 5 only
    spd[9] = 0                                   # bucket 0 is -inf: row 9 has no score
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    table[:, 0] = -np.inf
    q, k, v, do = (to_dev(g.standard_normal((H, N, d)).astype(np.float32)) for _ in range(4))
    S, T = to_dev(spd, torch.uint8), to_dev(table)
    o, l = gt.gt_attn_fwd(q, k, v, S, T)
    ref = gt.gt_attn_bwd(q, k, v, S, T, o, l, do)
    do[:, 9] = float("nan")
    got = gt.gt_attn_bwd(q, k, v, S, T, o, l, do)
    for a, b in zip(ref[:3], got[:3]):
        assert torch.equal(a, b)
    assert torch.allclose(ref[3], got[3], rtol=1e-5, atol=1e-5) and bool(torch.isfinite(got[3]).all())
    do[:, 5] = float("nan")
    dtab = gt.gt_attn_bwd(q, k, v, S, T, o, l, do)[3]
    assert bool(torch.isnan(dtab[:, 8:11]).all())
    assert torch.allclose(dtab[:, 11], torch.zeros_like(dtab[:, 11]))


@pytest.mark.parametrize("B,H,N,d", [
    (65, 32, 32, 8), (70, 32, 31, 32), (37, 64, 33, 16), (33, 64, 64, 64), (40, 32, 65, 64), (35, 32, 128, 8),
    (259, 8, 17, 64),
])
def test_f32_packed_batch(B, H, N, d):
    """fp32 batches of sequences of at most 128, 64 and 32 rows, of which a
    workgroup takes 2, 4 or 8, the last one a partly filled group."""
    g = np.random.default_rng(B + N)
    nb = 12
    spd = g.integers(0, nb + 2, size=(B, N, N)).astype(np.uint8)
    q, k, v, do = (g.standard_normal((B, H, N, d)).astype(np.float32) for _ in range(4))
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    scale = 1.0 / np.sqrt(d)
    say(f"packed f32 B={B} H={H} N={N} d={d}")
    Q, K, V, dO, S, T = to_dev(q), to_dev(k), to_dev(v), to_dev(do), to_dev(spd, torch.uint8), to_dev(table)
    o, l = gt.gt_attn_fwd_batch(Q, K, V, S, T)
    got = gt.gt_attn_bwd_batch(Q, K, V, S, T, o, l, dO)
    torch.cuda.synchronize()
    dtab = np.zeros((H, nb))
    for b in list(range(0, B, 7)) + [B - 1]:
        o_ref, l_ref = oracle.forward(q[b], k[b], v[b], spd[b], table, scale)
        check_fwd(f"graph {b}", to_np(o[b]), to_np(l[b]), o_ref, l_ref, "f32")
        ref = oracle.backward(q[b], k[b], v[b], spd[b], table, scale, do[b])
        check_grads(f"graph {b}", dict(dq=to_np(got[0][b]), dk=to_np(got[1][b]), dv=to_np(got[2][b])),
                    dict(dq=ref[0], dk=ref[1], dv=ref[2]), "f32")
    for b in range(B):
        dtab += oracle.backward(q[b], k[b], v[b], spd[b], table, scale, do[b])[3]
    check_grads("dtable", dict(dtable=to_np(got[3])), dict(dtable=dtab), "f32")


def run_short_batch(B, H, N, d, first, nb):
    g = np.random.default_rng(N * 10 + d)
    spd = g.integers(0, min(256, nb + 2), size=(B, N, N)).astype(np.uint8)
    q, k, v, do = (synth.round_bf16(g.standard_normal((B, H, N, d)).astype(np.float32)) for _ in range(4))
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    scale = 1.0 / np.sqrt(d)
    say(f"short bf16 B={B} H={H} N={N} d={d} first={first} nb={nb}")
    bf = torch.bfloat16
    Q, K, V, dO, T = to_dev(q, bf), to_dev(k, bf), to_dev(v, bf), to_dev(do, bf), to_dev(table)
    buf = to_dev(np.concatenate([np.zeros(first, np.uint8), spd.ravel()]), torch.uint8)
    S = buf[first:].view(B, N, N)
    o, l = gt.gt_attn_fwd_batch(Q, K, V, S, T)
    torch.cuda.synchronize()
    o_in = np.zeros((B, H, N, d), np.float32)
    l_in = np.zeros((B, H, N), np.float32)
    refs = []
    for b in range(B):
        o_ref, l_ref = oracle.forward(q[b], k[b], v[b], spd[b], table, scale)
        check_fwd(f"graph {b}", to_np(o[b]), to_np(l[b]), o_ref, l_ref, "bf16")
        o_in[b], l_in[b] = synth.round_bf16(o_ref.astype(np.float32)), l_ref.astype(np.float32)
        refs.append(oracle.ring_backward_step(q[b], o_in[b], l_in[b], do[b], k[b], v[b], spd[b], 0, 0, table, scale))
    got = gt.gt_attn_bwd_batch(Q, K, V, S, T, to_dev(o_in, bf), to_dev(l_in), dO)
    torch.cuda.synchronize()
    if N == 1:   # P is 1 and dS the rounding of dO.(V - O): no relative bar
        return
    for b, ref in enumerate(refs):
        check_grads(f"graph {b}", dict(dq=to_np(got[0][b]), dk=to_np(got[1][b]), dv=to_np(got[2][b])),
                    dict(dq=ref[0], dk=ref[1], dv=ref[2]), "bf16")
    check_grads("dtable", dict(dtable=to_np(got[3])), dict(dtable=sum(r[3] for r in refs)), "bf16")


@pytest.mark.parametrize("B,H,N,d,first", [
    (3, 2, 1, 64, 0), (9, 2, 3, 8, 1), (17, 4, 30, 8, 0), (11, 4, 31, 64, 0), (9, 8, 33, 16, 3), (7, 4, 47, 64, 0),
    (5, 8, 63, 32, 0), (5, 2, 65, 64, 2), (5, 2, 129, 16, 0), (3, 2, 203, 32, 0), (3, 2, 255, 64, 1),
    (3, 2, 256, 64, 0), (3, 2, 256, 8, 1), (2, 2, 200, 64, 0), (70, 8, 50, 64, 1),
])
def test_short_batch_any_size(B, H, N, d, first):
    """bf16 batches on the whole-sequence kernels: lengths either side of the
    packing limits, of the 32-key block and of the dword, head dim 64, and spd
    matrices that start at an odd byte; several groups per workgroup."""
    run_short_batch(B, H, N, d, first, 12)


@pytest.mark.parametrize("B,H,N,d,first,nb", [
    (3, 2, 1, 64, 0, 256), (17, 4, 30, 8, 0, 128), (11, 4, 31, 64, 1, 256), (9, 8, 33, 16, 3, 200),
    (9, 4, 32, 32, 0, 256), (5, 8, 63, 32, 0, 129), (5, 4, 64, 8, 0, 256), (5, 2, 100, 16, 0, 256),
    (5, 2, 128, 64, 0, 255), (5, 2, 129, 16, 2, 256),
    (3, 2, 203, 32, 0, 200), (3, 2, 255, 64, 1, 256), (3, 2, 256, 64, 0, 256), (3, 2, 256, 8, 0, 200),
    (70, 8, 50, 64, 1, 256),
])
def test_short_batch_many_buckets(B, H, N, d, first, nb):
    """The same with 128 to 256 buckets: a table entry for every byte value, the
    keys past N masked in the sequence's last block."""
    run_short_batch(B, H, N, d, first, nb)


def test_f32_more_heads_than_a_grid_row():
    """fp32, one node and more heads than a launch has workgroups of 512 threads
    in one dimension: O = V and LSE = the score; dV = dO and no other gradient."""
    H, d = (1 << 23) + 5, 8
    say(f"heads {H}")
    g = torch.Generator(device=DEV)
    g.manual_seed(0)
    q, k, v, do = (torch.randn((H, 1, d), device=DEV, generator=g) for _ in range(4))
    T = torch.randn((H, 2), device=DEV, generator=g)
    S = torch.ones((1, 1), device=DEV, dtype=torch.uint8)
    o, l = gt.gt_attn_fwd(q, k, v, S, T, scale=0.5)
    assert torch.equal(o, v)
    ref = 0.5 * (q.double() * k.double()).sum(2) + T[:, 1:]
    assert float((l.double() - ref).abs().max()) <= 1e-5
    dq, dk, dv, dt = gt.gt_attn_bwd(q, k, v, S, T, o, l, do, scale=0.5)
    # P is 1 up to the rounding of the score against LSE, dS the rounding of dO.(V - O)
    assert float((dv - do).abs().max()) <= 1e-4
    assert max(float(x.abs().max()) for x in (dq, dk, dt)) <= 1e-3
