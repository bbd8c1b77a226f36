"""The fp32 table gradient where a head's bound on dS says little about its
terms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_34420_amd as gt
from gpu_common import rel_l2, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _inputs(H, N, d, nb, seed):
    g = np.random.default_rng(seed)
    q, k, v, do = (g.standard_normal((H, N, d)).astype(np.float32) for _ in range(4))
    spd = g.integers(0, nb, size=(N, N)).astype(np.uint8)
    table = (g.standard_normal((H, nb)) * 0.5).astype(np.float32)
    return q, k, v, do, spd, table


def _dtable(q, k, v, spd, table, o, lse, do):
    o, lse = np.asarray(o, np.float32), np.asarray(lse, np.float32)
    return to_np(gt.gt_attn_bwd(*(to_dev(x) for x in (q, k, v)), to_dev(spd, torch.uint8), to_dev(table), to_dev(o),
                                to_dev(lse), to_dev(do))[3])


@pytest.mark.parametrize("d,big_do,big_v", [(64, 1e4, 1e4), (64, 1e6, 10.0), (16, 1e5, 1e3)])
def test_one_large_row(d, big_do, big_v):
    """One row of dO, with buckets of its own, and one of V are large: they set
    the bound, and the terms of the other buckets, small against it, keep their
    value and have no bias. The 1e-5 bar of the fp32 gradients."""
    q, k, v, do, spd, table = _inputs(2, 1500, d, 16, d)
    spd %= 12
    spd[3] = 12 + spd[3] % 4
    do[:, 3] *= big_do
    v[:, 7] *= big_v
    scale = 1 / np.sqrt(d)
    o, l = oracle.forward(q, k, v, spd, table, scale)
    o, l = o.astype(np.float32), l.astype(np.float32)
    ref = oracle.ring_backward_step(q, o, l, do, k, v, spd, 0, 0, table, scale)[3]
    got = _dtable(q, k, v, spd, table, o, l, do)
    e, e_own = rel_l2(got[:, :12], ref[:, :12]), rel_l2(got[:, 12:], ref[:, 12:])
    say(f"one large row d={d} dO {big_do} V {big_v}: dtable rel-L2 {e:.3e}, the row's own buckets {e_own:.3e}")
    assert max(e, e_own) <= 1e-5


def test_lse_of_other_inputs():
    """An LSE that is not the inputs' (every P e^6 or e^12 times larger): the
    terms pass the bound that the fixed-point sums rely on, and arrive."""
    q, k, v, do, spd, table = _inputs(2, 700, 32, 16, 1)
    scale = 1 / np.sqrt(32)
    o, l = oracle.forward(q, k, v, spd, table, scale)
    for off in (6.0, 12.0):
        o1, l1 = o.astype(np.float32), (l - off).astype(np.float32)
        ref = oracle.ring_backward_step(q, o1, l1, do, k, v, spd, 0, 0, table, scale)[3]
        e = rel_l2(_dtable(q, k, v, spd, table, o1, l1, do), ref)
        say(f"LSE lower by {off}: dtable rel-L2 {e:.3e}")
        # float adds of terms of one sign and the other, some 6e4 a bucket
        assert e <= 1e-4


@pytest.mark.parametrize("N", [200, 700])
def test_norm_that_overflows(N):
    """A finite dO row whose squared norm is infinite has no part in the bound:
    the buckets the other rows hold are right, and its own are."""
    q, k, v, do, spd, table = _inputs(2, N, 32, 16, N)
    spd %= 12
    spd[3] = 12 + spd[3] % 4
    do[:, 3] *= 1e20
    scale = 1 / np.sqrt(32)
    o, l = oracle.forward(q, k, v, spd, table, scale)
    o, l = o.astype(np.float32), l.astype(np.float32)
    ref = oracle.ring_backward_step(q, o, l, do, k, v, spd, 0, 0, table, scale)[3]
    got = _dtable(q, k, v, spd, table, o, l, do)
    e, e_own = rel_l2(got[:, :12], ref[:, :12]), rel_l2(got[:, 12:], ref[:, 12:])
    say(f"norm that overflows N={N}: dtable rel-L2 {e:.3e}, the row's own buckets {e_own:.3e}")
    assert max(e, e_own) <= 1e-5
