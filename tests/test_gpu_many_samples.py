"""Packs of very many one-token samples: more work items than one launch can have blocks for.  Every row sees one key, itself, so the
results are known: O = V, lse = scale q k, dV = the sum of dO over the group, dQ = dK = 0 (dP and delta are the same product, formed
twice)."""
import numpy as np
import pytest
import torch

import paper_2509_26246_amd as S
from paper_2509_26246_amd import harness as H

pytestmark = pytest.mark.gpu


# items x heads x 2 (fp32, both passes), items x heads (bf16 forward of short samples, dQ) and items x KV heads x 2 (dK/dV at head dim 64)
# just reach 2^32 threads
@pytest.mark.parametrize("T,hq,hkv,d,bf16,backward", [(131073, 64, 64, 16, False, True), (262145, 64, 8, 128, True, False),
                                                      (131073, 64, 64, 64, True, True), (262145, 64, 64, 64, True, True)])
def test_more_items_than_a_launch_has_blocks(T, hq, hkv, d, bf16, backward):
    dt = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(1)
    # (the distributions the bf16 tolerances are for: forward and backward round the scaled query and the scaled key, 2^-9 of a score
    # each, and P = exp(S - lse) is off by as much; with unit-normal values scores reach 8 and P is off by 3e-2)
    new = lambda h, f: (f * torch.randn((T, h, d), generator=gen, device="cuda")).to(dt)
    q, k, v, dO = new(hq, 0.5), new(hkv, 0.5), new(hkv, 0.5), new(hq, 0.1)
    cu, sl = S.build_slices([1] * T, 64)
    one = S.build_units(cu, sl, "ALL")
    tables = S.tables_create(cu, sl, *one, *one)
    nan = lambda *shape: torch.full(shape, float("nan"), dtype=dt, device="cuda")
    ws = torch.empty(S.bwd_workspace_bytes(tables, hq, hkv, d) if backward else 256, dtype=torch.uint8, device="cuda")
    prob = H.Problem(tables, hq, hkv, d, S.BF16 if bf16 else S.F32, d ** -0.5, q, k, v, dO, nan(T, hq, d), nan(hq, T).float(), nan(T, hq, d),
                     nan(T, hkv, d), nan(T, hkv, d), ws)
    prob.forward()
    torch.cuda.synchronize()
    g = hq // hkv
    tol = 2e-2 if bf16 else 1e-5                               # as in test_gpu_parity.py
    assert torch.equal(prob.o.view(T, hkv, g, d), v.unsqueeze(2).expand(T, hkv, g, d))
    for a in range(0, T, 65536):
        b = min(T, a + 65536)
        want = (q[a:b].float().view(b - a, hkv, g, d) * k[a:b].float().unsqueeze(2)).sum(-1).view(b - a, hq) * d ** -0.5
        assert float(((prob.lse[:, a:b].t() - want).abs() / (1 + want.abs())).max()) <= tol
    if backward:
        prob.backward()
        torch.cuda.synchronize()
        tol = 5e-2 if bf16 else 1e-5
        assert float((prob.dV.float() - dO.float().view(T, hkv, g, d).sum(2)).abs().max()) <= tol
        assert float(prob.dQ.float().abs().max()) <= tol and float(prob.dK.float().abs().max()) <= tol
