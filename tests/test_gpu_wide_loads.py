"""The kernels that read four elements at a time, at the sizes where that can
go wrong: frames at every element alignment, gradients with a remainder past
the last quad, weight gradients on every tile,
the recomputed ReLU mask at its border, pooling at odd channel-quad counts, and the packing of
minibatches whose lengths reach every form (one env, length 1, more frames
than a workgroup)."""
import dataclasses

import numpy as np
import pytest
import torch

from synth import rollout as R
from tests.gpu_util import DEV, assert_close, random_record, to_device
from tests.nets import MINI_RESNET, RESNET_64, TINY_PLUS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [4, 12])
def test_encode_is_the_same_at_any_frame_alignment(P, dtype, width):
    """Frames aligned to a pixel pair take the wide pooling kernel, others the
    elementwise one: both form 0.25 ((a + b) + (c + d)), bit for bit."""
    net = dataclasses.replace(MINI_RESNET, base_width=width, gn_groups=2)
    n = P.Net(net, dtype)
    params = torch.tensor(R.init_params(net, 1, random_affine=True), device=DEV)
    lp = P.cast_bf16(params) if dtype == "bf16" else None
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    F, k = 3, 3 * net.in_ch * net.in_hw ** 2
    x = torch.rand(k, generator=torch.Generator().manual_seed(2)).to(td).to(DEV)
    ref = None
    for off in range(4):
        print(f"encode {dtype} width {width}: frames {off} elements past an aligned address", flush=True)
        buf = torch.zeros(k + 4, dtype=td, device=DEV)
        buf[off:off + k] = x
        out = n.encode(buf[off:off + k].view(F, net.in_ch, net.in_hw, net.in_hw), params, lp)
        torch.cuda.synchronize()
        ref = out if ref is None else ref
        assert torch.isfinite(out).all() and torch.equal(out, ref), off


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 1027, 4 * 256 * 1024 + 3])
def test_adam_finds_a_non_finite_gradient_anywhere(P, n):
    print(f"adam check of {n} gradients", flush=True)
    for bad in (float("inf"), float("-inf"), float("nan")):
        for i in sorted({0, n // 2, max(n - 4, 0), max(n - 3, 0), max(n - 2, 0), n - 1}):
            master = torch.ones(n, device=DEV)
            opt = P.Adam(n, DEV, lr=1e-3, loss_scale=1.0, growth_interval=0)
            g = torch.ones(n, device=DEV)
            opt.step(master, g)
            assert opt.state()["skipped"] == 0 and opt.state()["step"] == 1
            before = master.clone()
            g[i] = bad
            opt.step(master, g)
            assert opt.state()["skipped"] == 1 and torch.equal(master, before), (bad, i)


@pytest.mark.parametrize("T,lens", [(1, [1]), (1, [1, 1, 1]), (130, [130]), (7, [7, 1, 1, 3]),
                                    (300, [1, 300, 299, 2]), (3, [1 + i % 3 for i in range(256)])],
                         ids=["one", "ones", "one_env", "short", "long", "256_envs"])
def test_frame_packing(P, T, lens):
    """dvalues of the loss head at V = 0 is -value_coef w ret of the frame's
    (step, env): returns that number the cells show the packing (time-major,
    longest env first).  A product of three float32 factors: 4 roundings."""
    print(f"frame packing T={T} envs={len(lens)}", flush=True)
    n, N = P.Net(TINY_PLUS, "f32"), len(lens)
    rec = random_record(TINY_PLUS, T, N, 3, lengths=lens)
    ro = to_device(rec)
    ro["ret"] = torch.arange(1, T * N + 1, dtype=torch.float32, device=DEV).view(T, N)
    F = sum(lens)
    cfg = P.LossCfg()
    dv = n.loss_head(ro, list(range(N)), lens, torch.zeros(F, n.A, device=DEV), torch.zeros(F, device=DEV), cfg)[1]
    order = sorted(range(N), key=lambda e: -lens[e])
    want = [-cfg.value_coef / (N * lens[e]) * (t * N + e + 1) for t in range(T) for e in order if lens[e] > t]
    np.testing.assert_allclose(dv.cpu().numpy(), np.array(want), rtol=4 * 2.0 ** -23)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [4, 12])
def test_weight_gradient_tiles(P, dtype, width):
    """The convolutions' weight gradients forced onto every tile shape, split
    over K and not, at widths and frame counts with ragged tiles (7 frames, 1x1
    to 16x16 maps: reductions of 7 to 1792 rows, 4 to 192 channels): the gradient
    is that of the tuned tiles up to the order of float32 sums."""
    print(f"weight gradient tiles {dtype} width {width}", flush=True)
    net = dataclasses.replace(MINI_RESNET, base_width=width)
    lengths, envs = [3, 2, 2], [0, 1, 2]
    rec = random_record(net, 3, 3, 46, lengths=lengths, bf16=dtype == "bf16")
    n = P.Net(net, dtype)
    params = torch.tensor(R.init_params(net, 45, random_affine=True), device=DEV)
    lp = P.cast_bf16(params) if dtype == "bf16" else None
    ro, scale = to_device(rec, bf16=dtype == "bf16"), torch.tensor([1.0], device=DEV)

    def grad():
        g, _ = n.loss_backward(ro, envs, lengths, params, lp, P.LossCfg(), loss_scale=scale)
        torch.cuda.synchronize()
        return g.cpu().numpy().astype(np.float64)

    n.autotune(1)
    grad()
    n.autotune(0)
    g0 = grad()                                   # every product on its tuned tile
    rows = [r for r in n.tile_table() if r[0] in (3, 4)]
    assert {r[0] for r in rows} >= {3}
    for tile in range(6):
        for split in (None, 1):
            print(f"  tile {tile} split {split}", flush=True)
            n.tile_table([r[:5] + [tile, split or r[6]] for r in rows])
            assert_close(f"gradient, tile {tile} split {split or 'tuned'}", grad(), g0, 1e-5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [4, 12])
def test_tile_shape_does_not_change_a_bit(P, dtype, width):
    """The launched tile is chosen apart from the K split, so every convolution
    product (forward, data and weight gradient; ragged tiles as above) forced
    onto any tile at one split leaves the whole gradient bit for bit."""
    print(f"tiles bit for bit {dtype} width {width}", flush=True)
    net = dataclasses.replace(MINI_RESNET, base_width=width)
    lengths, envs = [3, 2, 2], [0, 1, 2]
    rec = random_record(net, 3, 3, 46, lengths=lengths, bf16=dtype == "bf16")
    n = P.Net(net, dtype)
    params = torch.tensor(R.init_params(net, 45, random_affine=True), device=DEV)
    lp = P.cast_bf16(params) if dtype == "bf16" else None
    ro, scale = to_device(rec, bf16=dtype == "bf16"), torch.tensor([1.0], device=DEV)

    def grad():
        g, s = n.loss_backward(ro, envs, lengths, params, lp, P.LossCfg(), loss_scale=scale)
        torch.cuda.synchronize()
        return g.clone(), s.clone()

    n.autotune(1)
    grad()
    n.autotune(0)
    rows = [r for r in n.tile_table() if r[0] in (1, 2, 3, 4)]
    assert {1, 2, 3} <= {r[0] for r in rows}
    g0, s0 = grad()
    assert torch.isfinite(g0).all() and g0.abs().sum() > 0
    for tile in range(6):
        n.tile_table([r[:5] + [tile, r[6]] for r in rows])
        g1, s1 = grad()
        assert torch.equal(g1, g0) and torch.equal(s1, s0), tile


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("frames", [1, 3, 9])
def test_encode_is_the_same_at_any_weight_alignment(P, dtype, frames):
    """Convolutions of 32n channels copy weight rows as stored where they lie
    on 16 bytes and take the general loaders elsewhere: the paper's widths (1x1
    to 16x16 maps, one to nine frames) encode to the same bits at every element
    alignment of the weights."""
    n = P.Net(RESNET_64, dtype)
    params = torch.tensor(R.init_params(RESNET_64, 1, random_affine=True), device=DEV)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    obs = torch.rand((frames, 4, 64, 64), generator=torch.Generator().manual_seed(3)).to(td).to(DEV)
    ref = None
    for off in range(4):
        print(f"encode {dtype} {frames} frames: weights {off} elements past an aligned address", flush=True)
        buf = torch.zeros(n.P + 4, dtype=td, device=DEV)
        w = buf[off:off + n.P]
        w.copy_(params)
        out = n.encode(obs, params, w) if dtype == "bf16" else n.encode(obs, w)
        torch.cuda.synchronize()
        ref = out if ref is None else ref
        assert torch.isfinite(out).all() and torch.equal(out, ref), off


@pytest.mark.parametrize("fwd", ["apply", "fused"])
def test_recomputed_relu_mask_at_its_border(P, monkeypatch, fwd):
    """The GroupNorm backward forms the ReLU mask again from y as the forward's
    kernel did (three-launch or one-launch).  Channels of scale 0 put out their
    shift at every pixel: 0, -tiny and +tiny decide the mask alone, so a channel
    whose output is not positive has gradients of exactly 0 and one at +tiny
    has not.  Float32; the whole gradient against the one-launch backward, which
    masks by the saved output (other orders of float32 sums)."""
    print(f"recomputed mask, forward {fwd}", flush=True)
    net = dataclasses.replace(MINI_RESNET, base_width=12)
    rec, envs, lengths = random_record(net, 3, 3, 5, lengths=[3, 2, 2]), [0, 1, 2], [3, 2, 2]
    n = P.Net(net, "f32")
    off = {nm: (o, c) for nm, o, c in n.tensors()}
    flat = np.array(R.init_params(net, 6, random_affine=True))
    units = [nm[:-5] for nm in off if nm.endswith(".gn.g") and (nm.endswith("c1.gn.g") or nm.endswith("c2.gn.g"))]
    tiny = np.float32(1e-30)
    for u in units:
        g, b = off[u + ".gn.g"][0], off[u + ".gn.b"][0]
        flat[g:g + 3] = 0.0
        flat[b:b + 3] = (0.0, -tiny, tiny)
    params, ro = torch.tensor(flat, device=DEV), to_device(rec)

    def grad(bwd_max):
        monkeypatch.setenv("DDPPO_GN_FUSED_MAX", "0" if fwd == "apply" else str(1 << 30))
        monkeypatch.setenv("DDPPO_GNB_FUSED_MAX", str(bwd_max))
        g, _ = n.loss_backward(ro, envs, lengths, params, None, P.LossCfg())
        torch.cuda.synchronize()
        return g.cpu().numpy().astype(np.float64)

    got, ref = grad(0), grad(1 << 30)
    for u in units:
        b = off[u + ".gn.b"][0]
        assert got[b] == 0 and got[b + 1] == 0 and got[b + 2] != 0, (u, got[b:b + 3])
    assert_close("gradient", got, ref, 1e-5)
