"""Non-finite inputs reach the results they belong to and no others."""
import numpy as np
import pytest
import torch

import paper_2609_34420_amd as gt
from gpu_common import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("N", [7, 30, 32, 33, 64, 100])
@pytest.mark.parametrize("d", [8, 16, 32, 64])
def test_short_batch_neighbours_of_a_nonfinite_graph(d, N, first, bad):
    """bf16 batches of short sequences, several of which share a workgroup: a
    graph with a NaN or infinity in its K or V leaves every other graph's O and
    LSE, and dQ, dK and dV, the bits they are without it."""
    B, H, nb, p = 9, 4, 12, 3
    say(f"neighbours B={B} H={H} N={N} d={d} first={first} bad={bad}")
    g = np.random.default_rng(N + d)
    bf = torch.bfloat16
    q, k, v, do = (to_dev(g.standard_normal((B, H, N, d)).astype(np.float32), bf) for _ in range(4))
    T = to_dev((g.standard_normal((H, nb)) * 0.5).astype(np.float32))
    spd = g.integers(0, nb, size=(B, N, N)).astype(np.uint8)
    S = to_dev(np.concatenate([np.zeros(first, np.uint8), spd.ravel()]), torch.uint8)[first:].view(B, N, N)
    others = [b for b in range(B) if b != p]

    def run(k, v, o=None, l=None):
        if o is None:
            o, l = gt.gt_attn_fwd_batch(q, k, v, S, T)
        dq, dk, dv, _ = gt.gt_attn_bwd_batch(q, k, v, S, T, o, l, do)
        return o, l, dq, dk, dv

    ref = run(k, v)
    for name in ("k", "v"):
        k2, v2 = k.clone(), v.clone()
        (k2 if name == "k" else v2)[p, :, N // 2, d // 2] = bad
        got = run(k2, v2)
        torch.cuda.synchronize()
        assert not bool(torch.isfinite(got[0][p].float()).all()), name      # it reaches its own graph
        for x, y, what in zip(ref, got, ("O", "LSE", "dQ", "dK", "dV")):
            assert torch.equal(x[others], y[others]), (name, what)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("B,H,N,d", [(1, 2, 200, 64), (1, 2, 300, 32), (1, 256, 257, 8), (40, 32, 100, 16),
                                     (70, 32, 31, 32), (40, 32, 65, 64)])
def test_f32_rows_without_a_score(B, H, N, d, bad):
    """fp32: a row whose every score is -inf gets O = 0 and LSE = -inf whatever
    V holds, and a 32-key block without a score of a row adds nothing to it; a
    NaN score still shows. Key splits and packed sequences."""
    say(f"rows without a score B={B} H={H} N={N} d={d} bad={bad}")
    g = np.random.default_rng(N + d)
    spd = g.integers(1, 12, size=(B, N, N)).astype(np.uint8)
    spd[:, 5] = 0                                 # bucket 0 is -inf: row 5 has no score
    if N > 64:
        spd[:, 7, 32:64] = 0                      # row 7: none in the second block
    table = (g.standard_normal((H, 12)) * 0.5).astype(np.float32)
    table[:, 0] = -np.inf
    q, k, v = (to_dev(g.standard_normal((B, H, N, d)).astype(np.float32)) for _ in range(3))
    S, T = to_dev(spd, torch.uint8), to_dev(table)
    ref, _ = gt.gt_attn_fwd_batch(q, k, v, S, T)
    key = 40 if N > 64 else 3
    v[:, :, key, d // 2] = bad
    q[:, :, 9, 0] = float("nan")
    o, l = gt.gt_attn_fwd_batch(q, k, v, S, T)
    torch.cuda.synchronize()
    assert bool((o[:, :, 5] == 0).all()) and bool(torch.isneginf(l[:, :, 5]).all())
    if N > 64:
        assert torch.equal(o[:, :, 7], ref[:, :, 7])
    assert not bool(torch.isfinite(o[:, :, 6, d // 2]).any())
    assert bool(torch.isnan(o[:, :, 9]).all())
    if B == 1:                                    # merged into a running state that has no block yet
        st = (torch.zeros(H, N, d, device=q.device), torch.full((H, N), -float("inf"), device=q.device))
        gt.gt_attn_ring_step_acc(q[0], k[0], v[0], S[0], 0, 0, T, st)
        assert bool((st[0][:, 5] == 0).all()) and bool(torch.isneginf(st[1][:, 5]).all())
