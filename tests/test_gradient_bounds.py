"""What the bounds of gradient_bounds.py see, on the CPU: mistakes planted in the oracle's sums, on the inputs of the GPU tests that use them."""
import numpy as np
import pytest

import workloads as W
from gradient_bounds import REL_BF16, worst_block
from oracle import attention as A

L = [1100, 290]


def _inputs(hq, hkv, d):
    r = np.random.default_rng(5)
    q, k, v, dO = (W.bf16_round(r.standard_normal((sum(L), h, d), dtype=np.float32) * np.float32(x)) for h, x in ((hq, .5), (hkv, .5), (hkv, .5), (hq, .1)))
    cu = np.concatenate([[0], np.cumsum(L)])
    o, lse = A.fwd_packed(q, k, v, cu, d ** -0.5)
    return q, k, v, dO, o, lse


def _contribution(q, k, v, dO, o, lse, rows, keys, head, hk, scale):
    """dK, dV of `keys` (rows of the first sample) from the query rows `rows` of one head."""
    i, j = np.arange(*rows), np.arange(*keys)
    s = scale * (q[i, head].astype(np.float64) @ k[j, hk].astype(np.float64).T)
    p = np.where(j[None, :] <= i[:, None], np.exp(s - lse[head, i][:, None]), 0.0)
    d = dO[i, head].astype(np.float64)
    ds = p * (d @ v[j, hk].astype(np.float64).T - (d * o[i, head]).sum(1, keepdims=True))
    return scale * ds.T @ q[i, head], p.T @ d


# one step of 32 rows of one head lost or counted twice for 128 keys, early, in the middle, the last one; a part's rows
@pytest.mark.parametrize("hq,hkv,d", [(3, 1, 128), (8, 2, 64), (1, 1, 128)])
@pytest.mark.parametrize("rows,keys", [((256, 288), (128, 256)), ((544, 576), (0, 128)), ((1056, 1088), (0, 128)), ((1068, 1100), (896, 1024)), ((544, 832), (256, 384))])
def test_a_lost_step_breaks_the_bound(hq, hkv, d, rows, keys):
    q, k, v, dO, o, lse = _inputs(hq, hkv, d)
    scale = d ** -0.5
    _, dk, dv = A.bwd_packed(q, k, v, o, lse, dO, np.concatenate([[0], np.cumsum(L)]), scale)
    assert worst_block(W.bf16_round(dk.astype(np.float32)), dk) <= REL_BF16 / 4 and worst_block(W.bf16_round(dv.astype(np.float32)), dv) <= REL_BF16 / 4
    lost_k, lost_v = _contribution(q, k, v, dO, o, lse, rows, keys, 0, 0, scale)
    for sign in (-1, 1):
        for name, x, part in (("dK", dk, lost_k), ("dV", dv, lost_v)):
            got = x.copy()
            got[keys[0]:keys[1], 0] += sign * part
            assert worst_block(got, x) > REL_BF16, f"{name}: step lost or counted twice"
