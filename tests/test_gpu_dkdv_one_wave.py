"""The one-wave dK/dV kernel (head dim 128, long walks) on every path it has, in packs that are small because their head groups are large: key tiles divided among
blocks by query rows, by query heads, units of several runs of query rows whose sums continue from unit to unit, rows of other units that hold
NaN.  Against a plain fp64 evaluation on the GPU, relative to the result (gradient_bounds.py); which kernel a launch takes is asserted."""
import numpy as np
import pytest
import torch

import paper_2509_26246_amd as S
from gradient_bounds import REL_BF16, relative_error
from paper_2509_26246_amd import harness as H

pytestmark = pytest.mark.gpu
D = 128


def _problem(L, hq, hkv, slice_size, units):
    T = sum(L)
    gen = torch.Generator(device="cuda").manual_seed(sum(L) + hq)
    new = lambda h, f: (f * torch.randn((T, h, D), generator=gen, device="cuda")).to(torch.bfloat16)
    out = lambda h: torch.empty((T, h, D), dtype=torch.bfloat16, device="cuda")
    cu, sl = S.build_slices(L, slice_size)
    bu = S.build_units(cu, sl, units[0], **units[1]) if units else S.build_units(cu, sl, "ALL")
    fu = S.build_units(cu, sl, "ALL")
    tables = S.tables_create(cu, sl, *fu, *bu)
    ws = torch.empty(S.bwd_workspace_bytes(tables, hq, hkv, D), dtype=torch.uint8, device="cuda")
    prob = H.Problem(tables, hq, hkv, D, S.BF16, D ** -0.5, new(hq, 0.5), new(hkv, 0.5), new(hkv, 0.5), new(hq, 0.1), out(hq),
                     torch.empty((hq, T), device="cuda"), out(hq), out(hkv), out(hkv), ws)
    return prob, cu, sl, bu


def _reference(prob, cu):
    """O, dQ, dK, dV in fp64, one head of one sample after the other."""
    g = prob.n_q_heads // prob.n_kv_heads
    o, dq = (torch.zeros(prob.q.shape, dtype=torch.float64, device="cuda") for _ in range(2))
    dk, dv = (torch.zeros(prob.k.shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for a, b in zip(cu[:-1], cu[1:]):
        a, b = int(a), int(b)
        hidden = torch.ones((b - a, b - a), dtype=torch.bool, device="cuda").triu(1)
        for h in range(prob.n_q_heads):
            q, do, k, v = (x[a:b, i].double() for x, i in ((prob.q, h), (prob.dO, h), (prob.k, h // g), (prob.v, h // g)))
            p = torch.softmax((prob.scale * (q @ k.t())).masked_fill(hidden, -float("inf")), 1)
            o[a:b, h] = p @ v
            ds = p * (do @ v.t() - (do * o[a:b, h]).sum(1, keepdim=True))
            dq[a:b, h] = prob.scale * (ds @ k)
            dk[a:b, h // g] += prob.scale * (ds.t() @ q)
            dv[a:b, h // g] += p.t() @ do
    return {"o": o.cpu().numpy(), "dQ": dq.cpu().numpy(), "dK": dk.cpu().numpy(), "dV": dv.cpu().numpy()}


def _poison(prob):
    for t in (prob.dQ, prob.dK, prob.dV):
        t.fill_(float("nan"))
    prob.workspace.fill_(0xFF)


def _outputs(prob):
    torch.cuda.synchronize()
    return {n: getattr(prob, n).clone() for n in ("dQ", "dK", "dV")}


def _check(got, want, tag):
    for name, x in got.items():
        rel = relative_error(name, H.device_to_f32(x), want[name])
        assert rel <= REL_BF16, f"{tag} {name}: {rel:.3e} of the result in a block of rows"


# tiles divided by query rows (and the reduction), by query heads too, neither; ragged last tiles
@pytest.mark.parametrize("L,hq,hkv,plan", [([2500, 300], 48, 3, (256, 1, 1, True)), ([1500], 256, 2, (256, 7, 1, True)), ([510, 440, 331, 300, 290], 256, 16, (256, 1, 1, False))])
def test_whole_list(L, hq, hkv, plan):
    prob, cu, _, _ = _problem(L, hq, hkv, 4096, None)
    got_plan = S.bwd_dkdv_plan(prob.tables, hq, hkv, D)
    assert got_plan[:3] + (got_plan[3] > 0,) == plan, got_plan
    prob.forward()
    want = _reference(prob, cu)
    runs = []
    for _ in range(2):
        _poison(prob)
        prob.backward()
        runs.append(_outputs(prob))
    _check(runs[0] | {"o": prob.o}, want, f"{hq}/{hkv}")
    graph = prob.capture_step()
    for _ in range(3):                                  # eager work between the replays
        _poison(prob)
        torch.cuda.synchronize()
        graph.replay()
        runs.append(_outputs(prob))
    assert all(torch.equal(runs[0][n].view(torch.int16), r[n].view(torch.int16)) for r in runs[1:] for n in r)      # fixed order of sums


# units of every third slice: several runs of query rows each, key rows that collect from all three; one unit at a time, everything of other units
# NaN; released rows final at once and never touched again
@pytest.mark.parametrize("L,hq,hkv", [([2000, 290], 320, 10), ([900, 255, 33], 768, 12)])
def test_units_with_inputs_arriving_late(L, hq, hkv):
    prob, cu, sl, bu = _problem(L, hq, hkv, 97, ("ROUND_ROBIN", {"m": 3, "descending": True, "backward": True}))
    n_units = prob.tables.n_bwd_units
    plans = [S.bwd_dkdv_plan(prob.tables, hq, hkv, D, u) for u in range(n_units)]
    assert n_units == 3 and all(p[0] == 256 for p in plans) and {p[1] for p in plans} == {1, 2}      # with and without division by heads
    prob.forward()
    want = _reference(prob, cu)
    _poison(prob)
    prob.backward(flags=S.FLAG_PER_UNIT_LAUNCH)
    whole = _outputs(prob)
    _check(whole, want, f"{hq}/{hkv} by units")
    full = {n: getattr(prob, n).clone() for n in ("q", "dO", "o", "lse")}
    _poison(prob)
    released = np.zeros(sum(L), bool)
    for u in range(n_units):
        rows = torch.from_numpy(np.concatenate([np.arange(sl[t][2], sl[t][2] + sl[t][3]) for t in bu[1][bu[0][u]:bu[0][u + 1]]]).astype(np.int64)).cuda()
        for n, t in full.items():
            mine = getattr(prob, n)
            mine.fill_(float("nan"))
            if n == "lse":
                mine[:, rows] = t[:, rows]
            else:
                mine[rows] = t[rows]
        prob.backward(unit_lo=u, unit_hi=u + 1)
        got = _outputs(prob)
        for a, b in S.bwd_released_rows(prob.tables, u):
            released[a:b] = True
        free = torch.from_numpy(released).cuda()
        for n in ("dK", "dV"):                          # the bits of the whole list's units, as soon as they are released; no other row written
            assert torch.equal(got[n][free].view(torch.int16), whole[n][free].view(torch.int16)), f"unit {u} {n}"
            assert torch.isnan(got[n][~free]).all(), f"unit {u} {n}"
        assert torch.equal(got["dQ"][rows].view(torch.int16), whole["dQ"][rows].view(torch.int16)), f"unit {u} dQ"
    assert released.all()
