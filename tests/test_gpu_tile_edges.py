"""GPU parity at the sizes where a kernel's tiling can go wrong: tile edges, remainders and the ends of each variant's
range, against the CPU fp64 oracle.  Tolerances as in test_gpu_parity.py (max-abs: fp32 1e-5; bf16 2e-2 on O and lse,
5e-2 on the gradients), and relative to the result in every 32 rows (gradient_bounds.py)."""
import numpy as np
import pytest
import torch

import paper_2509_26246_amd as S
import workloads as W
from gradient_bounds import REL_BF16, REL_F32, relative_error
from oracle import attention as A
from paper_2509_26246_amd import harness as H

pytestmark = pytest.mark.gpu


def _problem(L, hq, hkv, d, bf16, slice_size, seed=7):
    r = np.random.default_rng(seed)
    T = int(sum(L))
    f = (0.5, 0.5, 0.5, 0.1) if bf16 else (1.0, 1.0, 1.0, 1.0)
    arrs = [r.standard_normal((T, h, d), dtype=np.float32) * np.float32(x) for h, x in zip((hq, hkv, hkv, hq), f)]
    q, k, v, dO = (W.bf16_round(a) if bf16 else a for a in arrs)
    cu, sl = S.build_slices(L, slice_size)
    fu = S.build_units(cu, sl, "PREFIX_FILL", m=4, w_quad=2, w_lin=0)
    bu = S.build_units(cu, sl, "PREFIX_FILL", m=5, w_quad=5, w_lin=0, backward=True)
    scale = d ** -0.5
    prob = H.make_problem(q, k, v, dO, cu, sl, fu, bu, bf16=bf16, scale=scale)
    o, lse = A.fwd_packed(q, k, v, cu, scale)
    dq, dk, dv = A.bwd_packed(q, k, v, o, lse, dO, cu, scale)
    return prob, {"o": o, "lse": lse, "dQ": dq, "dK": dk, "dV": dv}


def _poison(prob):
    for t in (prob.o, prob.lse, prob.dQ, prob.dK, prob.dV):
        t.fill_(float("nan"))
    prob.workspace.fill_(0xFF)


def _check(prob, ref, bf16, tag):
    for name, want in ref.items():
        t = getattr(prob, name)
        got = t.cpu().numpy() if name == "lse" else H.device_to_f32(t)
        assert np.isfinite(got).all(), f"{tag} {name} not finite"
        err = float(np.max(np.abs(got.astype(np.float64) - want)))
        tol = 1e-5 if not bf16 else 2e-2 if name in ("o", "lse") else 5e-2
        assert err <= tol, f"{tag} {name}: max-abs {err:.3e} > {tol}"
        if name != "lse":
            rel = relative_error(name, got, want)
            assert rel <= (REL_BF16 if bf16 else REL_F32), f"{tag} {name}: {rel:.3e} of the result in a block of rows"


def _fused_and_per_unit(L, hq, hkv, d, bf16, slice_size):
    prob, ref = _problem(L, hq, hkv, d, bf16, slice_size)
    for flags in (0, S.FLAG_PER_UNIT_LAUNCH):
        _poison(prob)
        prob.forward(flags=flags)
        prob.backward(flags=flags)
        torch.cuda.synchronize()
        _check(prob, ref, bf16, f"{hq}/{hkv}/{d} bf16={bf16} flags={flags}")
    return prob


# 32-row blocks of 64-row tiles, four waves taking key (query) tiles in turn; (900, ...) at 4/1 heads: walks divided in two
@pytest.mark.parametrize("L", [[1, 31, 32, 33, 63, 64, 65], [127, 128, 129, 161], [900, 2, 95]], ids=["sub-tile", "tile", "divided"])
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 16), (4, 1, 32), (2, 2, 64), (4, 1, 128)])
def test_fp32_tile_edges(L, hq, hkv, d):
    prob = _fused_and_per_unit(L, hq, hkv, d, False, 80)
    first = []
    for _ in range(2):                                  # fixed summation order: bitwise repeatable
        _poison(prob)
        prob.forward(); prob.backward(); torch.cuda.synchronize()
        first.append([t.clone() for t in (prob.o, prob.lse, prob.dQ, prob.dK, prob.dV)])
    assert all(torch.equal(a, b) for a, b in zip(*first))


# launches of more than 256 and fewer than 512 blocks of 32 rows, a multiple of 8 and not, dK/dV undivided: a second block for some compute units
@pytest.mark.parametrize("L,h", [([300, 333, 395], 8), ([700, 1013], 9), ([1010, 999], 8)])
@pytest.mark.parametrize("d", [16, 128])
def test_fp32_partial_second_round(L, h, d):
    _fused_and_per_unit(L, h, h, d, False, 4096)


# fp32 walks divided and not, on either side of the rule's lines: 128 blocks of up to 2 steps and 132; 136 of 4; of more, 272 blocks of up to 6 steps (a compute
# unit's share is 2.5), 320 of 8 (4.3), 400 of 8 (5.6, undivided)
@pytest.mark.parametrize("L,hq,hkv", [([256] * 8, 2, 2), ([256] * 8 + [64], 2, 2), ([512, 512, 64], 4, 4), ([768, 256, 64], 8, 8), ([640, 384, 64], 8, 8),
                                      ([1024, 256], 8, 8), ([1024, 1024, 512], 5, 5)])
def test_fp32_walks_divided_in_two(L, hq, hkv):
    _fused_and_per_unit(L, hq, hkv, 32, False, 4096)


# few key tiles for the chip and several query heads per KV head: every tile's walk divided by heads, group sizes that the
# number of parts does not divide included, beside tiles divided by rows (4096 rows on one KV head)
@pytest.mark.parametrize("L,hq,hkv,d", [([511, 37, 200, 128], 8, 1, 128), ([300, 257, 1], 6, 1, 64), ([900, 255, 256], 7, 1, 128),
                                        ([640, 31], 10, 2, 64), ([2304, 100], 16, 1, 128)])
def test_bf16_key_tiles_divided_by_heads(L, hq, hkv, d):
    _fused_and_per_unit(L, hq, hkv, d, True, 320)


# walks divided by steps too: over several runs of query rows (every third slice, ragged), parts that begin inside a run and at its end, halves of
# an item with fewer steps than parts; beside a division by heads and without one
@pytest.mark.parametrize("L,hq,hkv,d,whole,units", [([1100, 290], 3, 1, 128, (3, 3), [(3, 3), (3, 3), (3, 1)]), ([1100, 290], 8, 2, 64, (4, 1), [(4, 3), (4, 2), (4, 1)]),
                                                    ([300, 290], 2, 1, 128, (1, 4), [(1, 1)] * 3)])
def test_bf16_key_tiles_divided_by_steps(L, hq, hkv, d, whole, units):
    r = np.random.default_rng(5)
    q, k, v, dO = (W.bf16_round(r.standard_normal((sum(L), h, d), dtype=np.float32) * np.float32(x)) for h, x in ((hq, .5), (hkv, .5), (hkv, .5), (hq, .1)))
    cu, sl = S.build_slices(L, 97)
    fu = S.build_units(cu, sl, "PREFIX_FILL", m=4, w_quad=2, w_lin=0)
    bu = S.build_units(cu, sl, "ROUND_ROBIN", m=3, descending=True, backward=True)
    prob = H.make_problem(q, k, v, dO, cu, sl, fu, bu, bf16=True, scale=d ** -0.5)
    assert [S.bwd_dkdv_plan(prob.tables, hq, hkv, d, u)[:3] for u in range(-1, 3)] == [(128,) + by for by in [whole] + units]
    o, lse = A.fwd_packed(q, k, v, cu, d ** -0.5)
    dq, dk, dv = A.bwd_packed(q, k, v, o, lse, dO, cu, d ** -0.5)
    for flags in (0, S.FLAG_PER_UNIT_LAUNCH):
        _poison(prob)
        prob.forward(flags=flags)
        prob.backward(flags=flags)
        torch.cuda.synchronize()
        _check(prob, {"o": o, "lse": lse, "dQ": dq, "dK": dk, "dV": dv}, True, f"{hq}/{hkv}/{d} flags={flags}")


# key tiles divided by query rows in the division classes of 16 and of 32 and more KV heads: 1536 rows on as many heads, where the
# first tiles exceed three quarters of a slot's share (1536 against 336 and 672 rows)
@pytest.mark.parametrize("heads,d", [(16, 128), (20, 64), (32, 64), (33, 128)])
def test_bf16_key_tiles_divided_with_many_kv_heads(heads, d):
    prob, ref = _problem([1536], heads, heads, d, True, 640)
    _poison(prob)
    prob.forward()
    S.profile_enable(64)
    prob.backward()
    launches = S.profile_read()["reduce"][1]
    S.profile_enable(0)
    assert launches == 1
    _check(prob, ref, True, f"{heads} KV heads, d {d}")


# fp32 against fp64, relative 2-norm of each output: a random walk over sums of up to n = 4 x 900 terms in fp32, sqrt(n) 2^-24 = 3.6e-6 (largest
# seen 9e-7); the max-abs bound above allows ten times as much
@pytest.mark.parametrize("L,hq,hkv,d", [([511, 37, 200, 128], 2, 2, 64), ([900], 4, 1, 128), ([337], 3, 1, 32)])
def test_fp32_relative_error(L, hq, hkv, d):
    prob, ref = _problem(L, hq, hkv, d, False, 256)
    prob.forward()
    prob.backward()
    torch.cuda.synchronize()
    for name, want in ref.items():
        got = getattr(prob, name).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - want) <= 3.6e-6 * np.linalg.norm(want), name


def test_bf16_head_parts_leave_the_static_scratch_enough():
    """The partial tiles of a division by heads are limited so that the pack still fits the built-in scratch array."""
    L = [4000, 1300] + [256] * 17
    prob, ref = _problem(L, 4, 1, 128, True, 4096)
    assert S.bwd_workspace_bytes(prob.tables, 4, 1, 128) <= S.STATIC_SCRATCH_BYTES
    _poison(prob)
    prob.forward()
    S.bwd_static(prob.q, prob.k, prob.v, prob.o, prob.lse, prob.dO, prob.tables, prob.dQ, prob.dK, prob.dV, **prob._kw())
    torch.cuda.synchronize()
    _check(prob, ref, True, "static scratch")


# Head dim 64, 32 keys per wave and query steps in pairs: tiles with few waves in use, one step alone, odd and even numbers of
# steps (odd groups), steps that end inside a run, runs that start inside a wave's keys
@pytest.mark.parametrize("L", [[1, 31, 32, 33], [63, 65, 224, 225], [255, 257, 300]], ids=["wave", "waves", "tile"])
@pytest.mark.parametrize("hq,hkv,slice_size", [(1, 1, 1000), (3, 1, 97), (4, 2, 64)])
def test_bf16_dkdv_head_dim_64(L, hq, hkv, slice_size):
    _fused_and_per_unit(L, hq, hkv, 64, True, slice_size)


# Head dim 128, short walks: the halves of 256-row items as blocks of their own, tiles with few waves in use, walks of one step, an odd and an
# even number of steps, steps that end inside a run, runs that start inside a wave's keys
@pytest.mark.parametrize("L", [[1, 31, 32, 33], [95, 127, 128, 129], [160, 255, 257, 385]], ids=["wave", "half", "tile"])
@pytest.mark.parametrize("hq,hkv,slice_size", [(1, 1, 1000), (3, 1, 97), (4, 2, 64)])
def test_bf16_dkdv_short_walks(L, hq, hkv, slice_size):
    prob = _fused_and_per_unit(L, hq, hkv, 128, True, slice_size)
    assert S.bwd_dkdv_plan(prob.tables, hq, hkv, 128)[0] == 128


# ... and more than 112 steps per item on average in a launch that fills the chip (10 items of 16 KV heads, 123 steps): the one-wave kernel
def test_bf16_dkdv_long_walks():
    prob = _fused_and_per_unit([510, 440, 330, 300, 290], 256, 16, 128, True, 1000)
    assert S.bwd_dkdv_plan(prob.tables, 256, 16, 128) == (256, 1, 1, 0)


# Tails of at most 64 (32) rows, for which a block takes two (four) heads, as far as the group's size allows: on the edges, tails only, and beside a sample
# of more than 1024 keys (whole list: one head per block; the units of the short samples: shared)
@pytest.mark.parametrize("L", [[160, 33, 1, 192, 300], [32, 64, 65], [1153, 20, 190, 129]], ids=["short", "tails", "long"])
@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (4, 1, 128), (8, 1, 64), (6, 2, 128), (3, 1, 64), (12, 2, 128)])
def test_bf16_tails_shared_by_heads(L, hq, hkv, d):
    _fused_and_per_unit(L, hq, hkv, d, True, 500)


# Calls of one unit take the same blocks as the unit's own launches in a call of all units; calls of several units share no heads.  The rows are the same bits
@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (8, 2, 128), (3, 1, 128), (6, 1, 64)])
def test_bf16_tails_by_calls_of_units(hq, hkv, d):
    prob = _fused_and_per_unit([160, 33, 1, 192, 300, 64, 32], hq, hkv, d, True, 90)
    want = [x.clone() for x in (prob.o, prob.lse, prob.dQ, prob.dK, prob.dV)]
    nf, nb = prob.tables.n_fwd_units, prob.tables.n_bwd_units
    for step in (1, 3):
        for x in (prob.o, prob.lse, prob.dQ, prob.dK, prob.dV):
            x.fill_(7.0)
        for u in range(0, nf, step):
            prob.forward(unit_lo=u, unit_hi=min(u + step, nf))
        for u in range(0, nb, step):
            prob.backward(unit_lo=u, unit_hi=min(u + step, nb))
        torch.cuda.synchronize()
        for name, x, w in zip(("o", "lse", "dQ", "dK", "dV"), (prob.o, prob.lse, prob.dQ, prob.dK, prob.dV), want):
            assert torch.equal(x, w), f"{name}, {step} units a call"


# fp32 dQ: a key with a NaN or an infinity reaches the rows that see it and no row in front of it, in the middle of a tile too; a key of
# -inf (score -inf, probability 0) spoils only its own dim of those rows
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
def test_fp32_dq_of_rows_in_front_of_a_key_that_is_not_finite(d, value):
    at = 90
    prob, ref = _problem([37, 130], 2, 1, d, False, 1000)
    prob.q[:, :, 3] = prob.q[:, :, 3].abs() + 0.5
    prob.dO.mul_(0.1)
    prob.forward()
    prob.backward()
    torch.cuda.synchronize()
    want = prob.dQ.clone()
    prob.k[at, 0, 3] = value
    prob.dQ.fill_(7.0)
    prob.forward()
    prob.backward()
    torch.cuda.synchronize()
    assert torch.equal(prob.dQ[:at], want[:at])
    assert not torch.isfinite(prob.dQ[at:, :, 3]).any()
    if value < 0:
        dims = [c for c in range(d) if c != 3]
        assert torch.isfinite(prob.dQ[at:][:, :, dims]).all()
    else:
        assert torch.isnan(prob.dQ[at:]).all()
