"""Forward calls over a part of the unit list whose few query tiles see a long prefix: their keys are divided among blocks and
the parts added up by a second kernel.  Against the CPU fp64 oracle on sampled rows (tolerance as in test_gpu_parity.py: 2e-2
max-abs on O and lse), at the edges of the division, with rows behind the slice set to NaN, repeatable bit for bit, and with
more streams at once than there are arrays for the partial results."""
import numpy as np
import pytest
import torch

import paper_2509_26246_amd as S
import workloads as W
from oracle import attention as A
from paper_2509_26246_amd import harness as H

pytestmark = pytest.mark.gpu
TOL = 2e-2


def _slices(L, hq, hkv, d, slice_size, seed=3):
    r = np.random.default_rng(seed)
    T = int(sum(L))
    arrs = [W.bf16_round(r.standard_normal((T, h, d), dtype=np.float32) * np.float32(f)) for h, f in ((hq, 0.5), (hkv, 0.5), (hkv, 0.5), (hq, 0.1))]
    cu, sl = S.build_slices(L, slice_size)
    units = (np.arange(len(sl) + 1), np.arange(len(sl)))
    return H.make_problem(*arrs, cu, sl, units, units, bf16=True, scale=d ** -0.5), arrs, cu, sl


def _check(prob, arrs, cu, first, end, got_o, got_lse, tag):
    r = np.random.default_rng(1)
    rows = np.unique(np.concatenate([[first, end - 1, min(end - 1, first + 63), min(end - 1, first + 128)], r.integers(first, end, 24)]))
    rows = np.repeat(rows, 2)
    heads = r.integers(0, prob.n_q_heads, len(rows))
    ro, rl = A.fwd_rows(arrs[0], arrs[1], arrs[2], cu, prob.scale, rows, heads)
    eo, el = np.max(np.abs(got_o[rows, heads] - ro)), np.max(np.abs(got_lse[heads, rows] - rl))
    assert eo <= TOL and el <= TOL, f"{tag}: O {eo:.3e} lse {el:.3e}"


# Last slice of the first sample.  Prefixes around the shortest that is divided (48 tiles of 64 keys), parts of unequal size, a
# slice that starts inside a tile, one-row slices, several query tiles; the one-wave kernel (even groups at head dim 128) and
# the one-head kernel (odd groups, head dim 64).
@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (4, 2, 128), (6, 1, 64), (5, 5, 128), (3, 1, 64)])
@pytest.mark.parametrize("length,slice_size", [(3071, 3000), (3073, 3072), (6145, 256), (7777, 1000), (9000, 999)])
def test_last_slice_of_a_long_sample(hq, hkv, d, length, slice_size):
    prob, arrs, cu, sl = _slices([length, 70], hq, hkv, d, slice_size)
    last = [t for t in range(len(sl)) if sl[t][0] == 0][-1]
    first, end = int(sl[last][2]), int(sl[last][2] + sl[last][3])
    nan = float("nan")
    for t in (prob.q, prob.k, prob.v):
        t[end:] = nan                                     # the next sample has not arrived
    runs = []
    for _ in range(2):
        prob.o.fill_(nan)
        prob.lse.fill_(nan)
        prob.forward(unit_lo=last, unit_hi=last + 1)
        torch.cuda.synchronize()
        runs.append((prob.o.clone(), prob.lse.clone()))
    o, lse = H.device_to_f32(prob.o), prob.lse.cpu().numpy()
    assert np.isfinite(o[first:end]).all() and np.isfinite(lse[:, first:end]).all()
    assert np.isnan(o[:first]).all() and np.isnan(o[end:]).all() and np.isnan(lse[:, :first]).all() and np.isnan(lse[:, end:]).all()
    _check(prob, arrs, cu, first, end, o, lse, f"{hq}/{hkv}/{d} {length}/{slice_size}")
    assert torch.equal(runs[0][0][first:end].view(torch.int16), runs[1][0][first:end].view(torch.int16))
    assert torch.equal(runs[0][1][:, first:end], runs[1][1][:, first:end])


@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (3, 1, 128), (4, 2, 64)])
def test_long_and_short_prefixes_in_one_call(hq, hkv, d):
    # the last slices of a long, a middling (fewer parts) and a short sample (not divided) in one launch
    prob, arrs, cu, sl = _slices([6000, 2100, 40], hq, hkv, d, 500)
    picks = [[t for t in range(len(sl)) if sl[t][0] == s][-1] for s in range(3)]
    order = [t for t in range(len(sl)) if t not in picks] + picks
    units = (np.concatenate([[0], np.arange(len(order) - 3, len(order) + 1)]), np.asarray(order))
    prob.tables = S.tables_create(cu, sl, *units, *units)
    prob.o.fill_(float("nan"))
    prob.lse.fill_(float("nan"))
    prob.forward(unit_lo=1, unit_hi=4)
    torch.cuda.synchronize()
    o, lse = H.device_to_f32(prob.o), prob.lse.cpu().numpy()
    for t in picks:
        _check(prob, arrs, cu, int(sl[t][2]), int(sl[t][2] + sl[t][3]), o, lse, f"{hq}/{hkv}/{d} slice {t}")


def test_scores_that_climb_from_part_to_part():
    # each part's scores lie far above the one before it (by more than fp32's exponent range over the sample): parts are
    # weighted by their references
    hq, hkv, d, n = 4, 1, 128, 5000
    prob, arrs, cu, sl = _slices([n], hq, hkv, d, 500, 9)
    q, k, v, _ = arrs
    q[:, :, 0] = 4.0
    k[:, 0, 0] = W.bf16_round(np.linspace(-300, 300, n).astype(np.float32) // 8 * 8)
    prob = H.make_problem(*arrs, cu, sl, *[(np.arange(len(sl) + 1), np.arange(len(sl)))] * 2, bf16=True, scale=d ** -0.5)
    u = len(sl) - 1
    prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    rows, heads = np.arange(4500, 5000, 7), np.arange(72) % hq
    rows = rows[:72]
    ro, rl = A.fwd_rows(q, k, v, cu, prob.scale, rows, heads)
    # (lse relative: the scaled query is rounded to bf16 once, a relative error of 2^-9 of each score)
    assert np.max(np.abs(H.device_to_f32(prob.o)[rows, heads] - ro)) <= TOL
    assert np.max(np.abs(prob.lse.cpu().numpy()[heads, rows] - rl) / (1.0 + np.abs(rl))) <= TOL


def test_more_streams_than_arrays_and_graph_replays():
    prob, arrs, cu, sl = _slices([8000], 8, 1, 128, 512)
    u = len(sl) - 1
    first, end = int(sl[u][2]), int(sl[u][2] + sl[u][3])
    prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    _check(prob, arrs, cu, first, end, H.device_to_f32(prob.o), prob.lse.cpu().numpy(), "one stream")
    want = (prob.o[first:end].clone(), prob.lse[:, first:end].clone())
    streams = [torch.cuda.Stream() for _ in range(7)]
    outs = [(torch.empty_like(prob.o), torch.empty_like(prob.lse)) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(3):
        for s, (o, lse) in zip(streams, outs):
            with torch.cuda.stream(s):
                S.fwd(prob.q, prob.k, prob.v, prob.tables, o, lse, **prob._kw(unit_lo=u, unit_hi=u + 1))
    torch.cuda.synchronize()
    for i, (o, lse) in enumerate(outs):                     # divided or, where no array was free, walked part by part
        _check(prob, arrs, cu, first, end, H.device_to_f32(o), lse.cpu().numpy(), f"stream {i}")
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        prob.forward(unit_lo=u, unit_hi=u + 1)
    for _ in range(3):
        prob.o.fill_(float("nan"))
        prob.lse.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(prob.o[first:end].view(torch.int16), want[0].view(torch.int16)) and torch.equal(prob.lse[:, first:end], want[1])
        S.fwd(prob.q, prob.k, prob.v, prob.tables, outs[0][0], outs[0][1], **prob._kw(unit_lo=u, unit_hi=u + 1))
        torch.cuda.synchronize()
        assert torch.equal(outs[0][0][first:end].view(torch.int16), want[0].view(torch.int16))


# Keys that take no part in the softmax (a component of -inf, or one of -1e9 as masks use) at the first key of every tile but the
# sample's first, hence at the first key of every part, on each kernel that divides.  Each row of the last slice has most of its
# weight on one key, in a tile of its own choice, so that a part which loses its first tile's scores shows.  The last pack has an
# even group and 331 keys per row on average: the one-head kernel at head dim 128.
@pytest.mark.parametrize("low", [float("-inf"), -1e9])
@pytest.mark.parametrize("L,hq,hkv,d,first", [([9088], 8, 1, 128, 8960), ([9088], 3, 1, 128, 8960), ([9088], 4, 2, 64, 8960),
                                              ([3500] + [64] * 260, 2, 1, 128, 3392)])
def test_keys_without_weight_at_every_tile_edge(L, hq, hkv, d, first, low):
    prob, arrs, cu, sl = _slices(L, hq, hkv, d, first)
    q, k, v, dO = arrs
    rows, tiles = np.arange(first, L[0]), 1 + np.arange(L[0] - first) % (first // 64 - 1)
    signs = np.sign(np.random.default_rng(2).standard_normal((len(tiles), 1, d))).astype(np.float32)
    signs[:, :, 0] = 0.0
    k[64 * tiles + 8] = signs[tiles - 1] * np.float32(160 / d)
    q[rows] = signs[tiles - 1]                             # score 160 d^-1/2 with its key, far less with the others
    q[:, :, 0] = 4.0
    k[64:L[0]:64, :, 0] = low if np.isinf(low) else W.bf16_round(np.array([low], np.float32))[0]
    prob = H.make_problem(q, k, v, dO, cu, sl, *[(np.arange(len(sl) + 1), np.arange(len(sl)))] * 2, bf16=True, scale=d ** -0.5)
    prob.forward(unit_lo=1, unit_hi=2)
    torch.cuda.synchronize()
    o, lse = H.device_to_f32(prob.o), prob.lse.cpu().numpy()
    assert np.isfinite(o[rows]).all() and np.isfinite(lse[:, rows]).all()
    heads = rows % hq
    ro, rl = A.fwd_rows(q, k, v, cu, prob.scale, rows, heads)
    # (lse relative: the scaled query is rounded to bf16 once, a relative error of 2^-9 of the heavy key's score)
    assert np.max(np.abs(o[rows, heads] - ro)) <= TOL
    assert np.max(np.abs(lse[heads, rows] - rl) / (1.0 + np.abs(rl))) <= TOL


def test_handles_hold_their_tables_only():
    """The arrays for partial results belong to the library: a handle with a long sample in several units takes no more device memory
    than its tables, also where it is the process's only one."""
    cu, sl = S.build_slices([40000], 2048)
    units = (np.arange(len(sl) + 1), np.arange(len(sl)))
    S.tables_create(cu, sl, *units, *units).destroy()         # the library's own set-up
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    t = S.tables_create(cu, sl, *units, *units)
    assert free - torch.cuda.mem_get_info()[0] <= 8 << 20     # 20 units' lists: far below 1 MB, in whole allocation blocks
    t.destroy()


# More launches at once than there are arrays: those that find none free walk their parts one after another, to the same bits.  Every
# kernel that divides; eager calls on many streams beside replays of a graph.  The streams start together, behind some milliseconds of other
# work: small launches would otherwise end before the host has issued the next ones.
@pytest.mark.parametrize("L,hq,hkv,d", [([32768], 8, 1, 128), ([20000], 3, 1, 128), ([20000], 4, 2, 64), ([9000] + [64] * 3000, 2, 1, 128)])
def test_concurrent_launches_have_the_bits_of_one_alone(L, hq, hkv, d):
    prob, arrs, cu, sl = _slices(L, hq, hkv, d, 1024)
    u = [t for t in range(len(sl)) if sl[t][0] == 0][-1]
    first, end = int(sl[u][2]), int(sl[u][2] + sl[u][3])
    prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    _check(prob, arrs, cu, first, end, H.device_to_f32(prob.o), prob.lse.cpu().numpy(), "alone")
    want = (prob.o[first:end].clone(), prob.lse[:, first:end].clone())
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        prob.forward(unit_lo=u, unit_hi=u + 1)
    streams = [torch.cuda.Stream() for _ in range(8)]
    outs = [(torch.empty_like(prob.o), torch.empty_like(prob.lse)) for _ in streams]
    before, in_turn = S.fwd_divided_counts(), 0
    other, start = torch.empty(1 << 30, dtype=torch.uint8, device="cuda"), torch.cuda.Event()
    for _ in range(4):
        for t in [prob.o, prob.lse] + [t for pair in outs for t in pair]:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        for n in range(32):
            other.fill_(n)
        start.record()
        for s in streams + [side]:
            s.wait_event(start)
        for _ in range(3):
            for s, (o, lse) in zip(streams, outs):
                with torch.cuda.stream(s):
                    S.fwd(prob.q, prob.k, prob.v, prob.tables, o, lse, **prob._kw(unit_lo=u, unit_hi=u + 1))
            with torch.cuda.stream(side):
                g.replay()
        torch.cuda.synchronize()
        after = S.fwd_divided_counts()
        assert after[0] + after[1] - before[0] - before[1] == 27 and after[2] == 0, (before, after)
        in_turn += after[1] - before[1]
        before = after
        for i, (o, lse) in enumerate(outs + [(prob.o, prob.lse)]):
            assert torch.equal(o[first:end].view(torch.int16), want[0].view(torch.int16)), f"stream {i}: O"
            assert torch.equal(lse[:, first:end], want[1]), f"stream {i}: lse"
            assert torch.isnan(o[:first]).all() and torch.isnan(o[end:]).all()
    assert in_turn > 0, "no launch found both arrays taken" # both ways to finish a launch have run


@pytest.mark.parametrize("L,hq,hkv,d", [([9000], 8, 1, 128), ([9000], 3, 1, 128), ([9000], 4, 2, 64), ([3500] + [64] * 260, 2, 1, 128),
                                        ([3073], 8, 1, 128), ([3071], 8, 1, 128)])
def test_divided_launches_are_counted(L, hq, hkv, d):
    """A call over part of the list with a long prefix is divided, each time; per-unit and whole-list launches are not, nor is a prefix
    below 3072 keys."""
    prob, _, _, sl = _slices(L, hq, hkv, d, 400)
    u = [t for t in range(len(sl)) if sl[t][0] == 0][-1]

    def counted(**kw):
        before = S.fwd_divided_counts()
        prob.forward(**kw)
        torch.cuda.synchronize()
        after = S.fwd_divided_counts()
        assert after[2] == 0
        return after[0] - before[0], after[1] - before[1]

    for _ in range(3):
        assert counted(unit_lo=u, unit_hi=u + 1) == ((1, 0) if L[0] > 3071 else (0, 0))
    assert counted(unit_lo=u, unit_hi=u + 1, flags=S.FLAG_PER_UNIT_LAUNCH) == (0, 0)
    assert counted() == (0, 0)


def test_a_call_that_fails_gives_its_array_back():
    """A launch reports an earlier error of the thread's HIP calls as its own: such a call fails behind its claim."""
    prob, _, _, sl = _slices([9000], 8, 1, 128, 400)
    u = len(sl) - 1
    prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    for _ in range(3):
        assert S.load_library().hipSetDevice(999) != 0        # refused, and remembered by the runtime; the device stays
        with pytest.raises(S.SlimAttnError):
            prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    before = S.fwd_divided_counts()
    assert before[2] == 0
    prob.forward(unit_lo=u, unit_hi=u + 1)
    torch.cuda.synchronize()
    assert S.fwd_divided_counts() == (before[0] + 1, before[1], 0)
