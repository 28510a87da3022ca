"""Backward of sharp attention (queries scaled by 4, so that most key tiles hold
a probability above 1/16 and their products take the bf16 residuals too) at every
number of heads per dK/dV iteration and both head dims, with ragged documents:
against the fp64 oracle, and dQ added by the key-major pass against the
deterministic one.

Tolerances (2-norm, relative): one rounding to bf16 is at most 2^-9 of a term. dQ
rounds dS once, with rows of very different size in one sum: 2^-8. dK and dV
round P and dS only where no residual is taken: 2^-9. The two dQ hold the same
bf16 dS and add them in another order in fp32: 2e-5 (a few hundred roundings of
2^-24).
"""
import pytest
import torch

import _cases
from paper_2606_08476_amd import flashcp as F
from test_gpu_parity import Run, dev, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _rel(a, ref):
    a, ref = a.cpu().double(), ref.double()
    return float((a - ref).norm() / ref.norm().clamp_min(1e-30))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (4, 2), (3, 3)])
def test_sharp_backward(hq, hkv, d, dev):  # noqa: F811
    case = _cases.make_case(f"sharp_{hq}_{hkv}_{d}", "llama8b", lens=[1, 33, 129, 700, 257, 8], cp=2,
                            rank=1, hq=hq, hkv=hkv, d=d, plan="per_doc")
    x = _cases.inputs(case)
    x["q"] = x["q"] * 4
    r = Run(case, dev, x=x)
    tq = r.v.info["t_q"]
    dq, dk, dv = r.oracle_bwd()
    e = dict(dq=_rel(r.dq, dq), dk=_rel(torch.cat([r.dk_loc, r.dk_recv]), dk),
             dv=_rel(torch.cat([r.dv_loc, r.dv_recv]), dv))
    a = r.bwd_outputs()
    ws = torch.empty(r.v.workspace_size()[1], dtype=torch.uint8, device=dev)
    F.fc_attn_bwd(r.v, r.q, r.k_loc, r.v_loc, r.k_recv, r.v_recv, r.o, r.lse, r.do, 0.0, *a, ws,
                  deterministic=False, o_f32=r.o32)
    torch.cuda.synchronize()
    e["order"] = _rel(a[0], r.dq.cpu())
    say(f"[gpu] {case.name} t_q {tq}: " + " ".join(f"{k} {v:.2e}" for k, v in e.items()))
    assert e["dq"] <= 2.0 ** -8 and max(e["dk"], e["dv"]) <= 2.0 ** -9 and e["order"] <= 2e-5, e
