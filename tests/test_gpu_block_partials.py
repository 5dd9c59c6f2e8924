"""Bound low-precision block products whose last GEMM leaves two partial
products: they are added up while the product moves back to FP64, eagerly and
behind a captured graph, in both layouts and at sector sizes below, at and above
a relayout tile.  Tolerances as for the unsplit product
(test_gpu_block_layouts.py): FP32 3e-5 of the largest entry, BF16 the rounding
model of test_gpu_parity.bf16_bound."""
import numpy as np
import pytest
import torch

from oracle import contract as C

pytestmark = pytest.mark.gpu

abi = pytest.importorskip("paper_1501_05504_amd.abi")

from tests.test_gpu_block_layouts import DEV, dev, make_plan, packed_case, rel_err, unpack_site   # noqa: E402
from tests.test_gpu_parity import bf16_bound, bf16_round                                         # noqa: E402


@pytest.mark.parametrize("layout", ["dense", "packed"])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("ml, mr, seed", [(9, 8, 31), (64, 96, 32), (130, 257, 33)])
def test_split_bound_product(layout, prec, ml, mr, seed):
    case = packed_case(ml, mr, seed)
    rnd = bf16_round if prec == "bf16" else (lambda a: np.asarray(a, dtype=np.float32).astype(np.float64))
    Lr, Rr, pr = rnd(case["L"]), rnd(case["R"]), rnd(case["psi"])
    Wf = np.asarray(case["W"], dtype=np.float32).astype(np.float64)
    ref = C.apply_heff(Lr, Wf, Rr, pr)
    packed = layout == "packed"
    c = abi.Context(0)
    c.set_block_split(0.0)
    plan = make_plan(c, case, abi.LAYOUT_PACKED if packed else abi.LAYOUT_DENSE)
    L, R, psi = (case[k + "p"] if packed else case[k] for k in ("L", "R", "psi"))
    plan.bind(dev(L), dev(case["W"]), dev(R), abi.F32 if prec == "f32" else abi.BF16)
    for use_graph in (False, True, True):
        out = torch.full((plan.npsi,), float("nan"), dtype=torch.float64, device=DEV)
        plan.apply_bound(dev(psi), out, use_graph=use_graph)
        torch.cuda.synchronize()
        o = out.cpu().numpy()
        if packed:
            o = unpack_site(o, case["psi"].shape, case["qL"], case["dL"], case["qR"], case["dR"], case["phys"])
        else:
            o = o.reshape(case["psi"].shape)
            assert np.all(o[case["mask"] == 0] == 0.0)
        if prec == "f32":
            assert rel_err(o, ref) < 3e-5
        else:
            assert np.all(np.abs(o - ref) <= bf16_bound(Lr, Wf, Rr, pr))
    plan.close()
    c.close()
