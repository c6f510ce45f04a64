"""The two bf16 forward kernels on either side of the rule that chooses between them (keys a row of the pack sees on average),
with ragged samples, references that have to move, and the whole list against one launch per unit (of the same query tiles) bit for
bit.  Against the CPU
fp64 oracle (tolerance as in test_gpu_parity.py: 2e-2 max-abs on O, and on lse relative to 1 + |lse|, as the scaled query is
rounded to bf16 once)."""
import numpy as np
import pytest
import torch

import paper_2509_26246_amd as S
import workloads as W
from oracle import attention as A
from paper_2509_26246_amd import harness as H

pytestmark = pytest.mark.gpu
TOL = 2e-2


# mean keys 400 (last of the short side) and 401, ragged tiles on both sides, samples shorter than a wave's rows
@pytest.mark.parametrize("L", [[800], [801], [511, 37, 200, 128, 1], [1, 1390, 37, 129, 64]], ids=["400", "401", "short", "long"])
@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (8, 1, 128), (3, 1, 128), (4, 1, 64), (3, 1, 64)])
@pytest.mark.parametrize("jump", [0.0, 200.0])
def test_forward_routes(L, hq, hkv, d, jump):
    r = np.random.default_rng(5)
    T, scale = sum(L), d ** -0.5
    arrs = [r.standard_normal((T, h, d), dtype=np.float32) * np.float32(f) for h, f in ((hq, 0.5), (hkv, 0.5), (hkv, 0.5), (hq, 0.1))]
    if jump:                                               # scores climb by `jump` inside each sample, from a key on that moves about
        arrs[0][:, :, 0] = 4.0
        st = 0
        for n in L:
            arrs[1][st:st + n, :, 0] = -jump / (8 * scale)
            arrs[1][st + n * 2 // 3:st + n, :, 0] = jump / (8 * scale)
            st += n
    arrs = [W.bf16_round(a) for a in arrs]
    cu, sl = S.build_slices(L, 192)
    fu = S.build_units(cu, sl, "PER_SAMPLE")
    prob = H.make_problem(*arrs, cu, sl, fu, fu, bf16=True, scale=scale)
    want_o, want_lse = A.fwd_packed(*arrs[:3], cu, scale)
    got = []
    for flags in (0, S.FLAG_PER_UNIT_LAUNCH):
        prob.o.fill_(float("nan"))
        prob.lse.fill_(float("nan"))
        prob.forward(flags=flags)
        torch.cuda.synchronize()
        got.append((prob.o.clone(), prob.lse.clone()))
    o, lse = H.device_to_f32(prob.o), prob.lse.cpu().numpy()
    assert float(np.max(np.abs(o - want_o))) <= TOL
    assert float(np.max(np.abs(lse - want_lse) / (1.0 + np.abs(want_lse)))) <= TOL
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1])


# Even groups at head dim 128 run the one-wave kernel or, in packs of short samples, the one-head kernel: both add probabilities in
# fp32 before they are rounded for the product, so a row's o and lse do not depend on which it is.
@pytest.mark.parametrize("L", [[128] * 9, [511, 37, 200, 128, 1], [400, 399, 65]])
@pytest.mark.parametrize("hq,hkv", [(8, 1), (4, 2)])
def test_short_samples_keep_the_precision_of_lse(L, hq, hkv):
    d, r = 128, np.random.default_rng(11)
    T, scale = sum(L), d ** -0.5
    arrs = [W.bf16_round(r.standard_normal((T + 2000, h, d), dtype=np.float32) * np.float32(f)) for h, f in ((hq, 0.5), (hkv, 0.5), (hkv, 0.5), (hq, 0.1))]
    got = []
    for lengths in (L, L + [2000]):                         # with the long sample a row of the pack sees more than 400 keys on average
        n = sum(lengths)
        cu, sl = S.build_slices(lengths, 4096)
        one = S.build_units(cu, sl, "ALL")
        prob = H.make_problem(*[a[:n] for a in arrs], cu, sl, one, one, bf16=True, scale=scale)
        prob.forward()
        torch.cuda.synchronize()
        got.append((prob.o[:T].clone(), prob.lse[:, :T].clone()))
    # against fp64 on the query as the kernels round it (times scale log2 e, to bf16): a row sum of n <= 511 fp32 terms is off by at
    # most n 2^-24 relative, its exponents (below 4 in log2 units) by less than 2^-22; rounded probabilities are off by 2^-9 each
    q2 = W.bf16_round(arrs[0][:T] * (np.float32(scale) * np.float32(1.4426950408889634)))
    _, want = A.fwd_packed(q2, arrs[1][:T], arrs[2][:T], S.build_slices(L, 4096)[0], np.log(2.0))
    for o, lse in got:
        assert np.max(np.abs(lse.cpu().numpy() - want)) <= 4e-5
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1])


# q rows of other units, which may hold anything, take no part in a tile's decision to move its references: one unit at a time, with
# ragged slices and scores that climb along the sample at a rate of each row's own, and everything outside the unit 1000 times larger.
@pytest.mark.parametrize("L", [[700, 130, 1, 300], [1, 1390, 301, 129]], ids=["short", "long"])
@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (3, 1, 128), (4, 1, 64), (3, 1, 64)])
def test_rows_of_other_units_change_no_bit(L, hq, hkv, d):
    r = np.random.default_rng(8)
    T, scale = sum(L), d ** -0.5
    arrs = [r.standard_normal((T, h, d), dtype=np.float32) * np.float32(f) for h, f in ((hq, 0.5), (hkv, 0.5), (hkv, 0.5), (hq, 0.1))]
    arrs[0][:, :, 0] = r.uniform(0.0, 4.0, (T, hq))
    arrs[1][:, :, 0] = (np.concatenate([np.arange(n) for n in L]) * (100.0 / (scale * 4.0 * 700)))[:, None]
    arrs = [W.bf16_round(a) for a in arrs]
    cu, sl = S.build_slices(L, 97)
    units = (np.arange(len(sl) + 1), np.arange(len(sl)))
    prob = H.make_problem(*arrs, cu, sl, units, units, bf16=True, scale=scale)
    q, got = prob.q.clone(), []
    for foreign in (1.0, 1000.0):
        prob.o.fill_(float("nan"))
        prob.lse.fill_(float("nan"))
        for u in range(len(sl)):
            a, b = int(sl[u][2]), int(sl[u][2] + sl[u][3])
            prob.q.copy_(q).mul_(foreign)
            prob.q[a:b] = q[a:b]
            prob.forward(unit_lo=u, unit_hi=u + 1)
        torch.cuda.synchronize()
        got.append((prob.o.clone(), prob.lse.clone()))
    want_o, want_lse = A.fwd_packed(*arrs[:3], cu, scale)
    assert float(np.max(np.abs(H.device_to_f32(prob.o) - want_o))) <= TOL
    assert float(np.max(np.abs(prob.lse.cpu().numpy() - want_lse) / (1.0 + np.abs(want_lse)))) <= TOL
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1])


# Keys that take no part in the softmax (scores of -inf, of a -1e9 mask, of bf16's lowest value), whole tiles of them too, on every
# forward kernel; the sample's first key is an ordinary one.
@pytest.mark.parametrize("low", [float("-inf"), -1e9, -3.3895e38])
@pytest.mark.parametrize("L,hq,hkv,d,bf16", [([1000], 4, 2, 128, True), ([500, 90], 4, 2, 128, True), ([500], 3, 1, 128, True),
                                             ([500], 4, 1, 64, True), ([300, 90], 4, 2, 64, False), ([300], 2, 2, 128, False)])
def test_keys_without_weight(L, hq, hkv, d, bf16, low):
    r = np.random.default_rng(4)
    T, scale = sum(L), d ** -0.5
    arrs = [r.standard_normal((T, h, d), dtype=np.float32) * np.float32(f) for h, f in ((hq, 0.5), (hkv, 0.5), (hkv, 0.5), (hq, 0.1))]
    arrs[0][:, :, 0] = 4.0
    arrs = [W.bf16_round(a) for a in arrs] if bf16 else arrs
    st = 0
    for n in L:
        hidden = [j for j in range(1, n) if j % 3 == 1 or 64 <= j < 200]
        arrs[1][st:st + n][hidden, :, 0] = low if np.isinf(low) else W.bf16_round(np.array([low], np.float32))[0]
        st += n
    cu, sl = S.build_slices(L, 192)
    one = S.build_units(cu, sl, "ALL")
    prob = H.make_problem(*arrs, cu, sl, one, one, bf16=bf16, scale=scale)
    prob.forward()
    torch.cuda.synchronize()
    want_o, want_lse = A.fwd_packed(*arrs[:3], cu, scale)
    tol = TOL if bf16 else 1e-5
    assert np.max(np.abs(H.device_to_f32(prob.o) - want_o)) <= tol and np.max(np.abs(prob.lse.cpu().numpy() - want_lse)) <= tol
