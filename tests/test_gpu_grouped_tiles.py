"""The register-tiled grouped convolutions at the sizes where their tiling can
go wrong: group counts that leave 1, 2 or 4 groups a workgroup (and, for the
weight gradient, those that take the general kernel), frame counts with a
ragged last workgroup, and enough pixels for two a thread; forward, data and
weight gradient through the benchmark entry against torch's grouped
convolution in float64 on the same operands (bfloat16 operands rounded first,
so that each product is exact in float32)."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import rollout as R
from synth.configs import SERESNEXT_NET
from tests.gpu_util import assert_close
from tests.nets import MINI_SERESNEXT
from tests.test_gpu_seresnext import _get, _put, _scratch_offsets

pytestmark = pytest.mark.gpu

# name: (net, frames per stage)
CASES = {
    "2_groups": (MINI_SERESNEXT, (1, 7, 7, 7)),
    "4_groups": (dataclasses.replace(MINI_SERESNEXT, base_width=8, cardinality=4), (7, 3, 1, 5)),
    "6_groups": (dataclasses.replace(MINI_SERESNEXT, base_width=12, cardinality=6), (3, 3, 3, 3)),
    # 16 groups; past 2 * 2048 workgroup rows of pixels a thread takes two
    "paper_two_pixels": (SERESNEXT_NET, (65, 129, 257, 513)),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_grouped_conv_tiles(P, monkeypatch, name, dtype):
    from paper_1911_00357_amd import api
    from paper_1911_00357_amd._lib import PPO_OP_LEARN
    monkeypatch.setattr(api, "POISON_WS", False)   # the operands are written into the workspace first
    net, frames = CASES[name]
    n = P.Net(net, dtype)
    flat = R.init_params(net, 5)
    params = torch.tensor(flat, device="cuda")
    lp = P.cast_bf16(params) if dtype == "bf16" else None
    grad = torch.zeros_like(params)
    off = {nm: (o, cnt) for nm, o, cnt in n.tensors()}
    g, done, tol = np.random.default_rng(7), set(), 1e-5
    rnd = R.round_bf16 if dtype == "bf16" else (lambda a: a)
    for u in range(n.probe(PPO_OP_LEARN, 1, 1, 3)[3][0]):
        unit, _, _, (ho, _, co, _) = n.probe(PPO_OP_LEARN, 1, 1, 0, u)
        if not unit.endswith(".c2"):
            continue
        s, j = int(unit.split(".")[1][1:]), int(unit.split(".")[2][1:])
        stride = 2 if (j == 0 and s > 0) else 1
        if (co, stride) in done:
            continue
        done.add((co, stride))
        F, G, hi = frames[s], net.cardinality, ho * stride
        cg = co // G
        print(f"grouped tiles {name} {unit}: {F} frames, {co} channels in {G} groups, {hi} -> {ho}, {dtype}", flush=True)
        ws = n.workspace(PPO_OP_LEARN, F, 1, params.device)
        offs = _scratch_offsets(n, F)
        x = g.standard_normal((F, hi, hi, co)).astype(np.float32)
        dy = g.standard_normal((F, ho, ho, co)).astype(np.float32)
        _put(ws, offs["ga"], x)
        _put(ws, offs["gb"], dy)
        o, cnt = off[unit + ".w"] if unit + ".w" in off else off[unit]
        w = rnd(flat[o:o + cnt].reshape(co, 3, 3, cg))
        to = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64)
        xt = to(rnd(x).transpose(0, 3, 1, 2)).requires_grad_()
        wt = to(w.transpose(0, 3, 1, 2)).requires_grad_()
        y_ref = torch.nn.functional.conv2d(xt, wt, stride=stride, padding=1, groups=G)
        dx_ref, dw_ref = torch.autograd.grad(y_ref, (xt, wt), to(dy.transpose(0, 3, 1, 2)))
        outs = (("forward", F * ho * ho * co, (F, ho, ho, co), y_ref.detach()),
                ("data gradient", F * hi * hi * co, (F, hi, hi, co), dx_ref))
        for op, (what, cells, shape, ref) in enumerate(outs):
            n.bench_unit_gemm(op, u, F, params, lp, grad, 1)
            torch.cuda.synchronize()
            got = _get(ws, offs["gu"], cells).reshape(shape).transpose(0, 3, 1, 2)
            assert_close(f"{unit} {what}", got, ref.numpy(), tol)
        n.bench_unit_gemm(2, u, F, params, lp, grad, 1)
        torch.cuda.synchronize()
        dw = grad[o:o + cnt].cpu().numpy().reshape(co, 3, 3, cg).transpose(0, 3, 1, 2)
        assert_close(f"{unit} weight gradient", dw, dw_ref.numpy(), tol)
    assert {c // net.cardinality for c, _ in done} == {4, 8, 16, 32}
