"""Which kernel the library launches, and over how many workgroups, where a
size limit or an option decides: on the CPU, launches recorded instead of run."""
import pytest

from tests.launch_recorder import record


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_convolutions_past_32_bit_offsets_take_the_general_loaders(tmp_path_factory, dtype):
    """The scalar-tap loaders add a 32-bit element offset to the base of the
    input (forward) or output gradient (data gradient): they are launched up to
    2^31 elements, the general ones, which add the offset in an image in 64
    bits, above.  Both maps of this net's second convolution have 25088
    elements a frame."""
    most = (1 << 31) // 25088
    out = record(tmp_path_factory, f"""
h = net("{dtype}", trunk=L.PPO_TRUNK_TINY, in_hw=56, avgpool=0)
out = [[n for n, _ in act(h, {most})], [n for n, _ in act(h, {most + 1})],
       [n for n, _ in loss_backward(h, {most})], [n for n, _ in loss_backward(h, {most + 1})]]
""")

    def count(names, what):
        return sum(what in n for n in names)

    for names, uniform in zip(out, (1, 0, 1, 0)):
        assert count(names, "ConvFwdUProb") == uniform and count(names, "ConvFwdProb") == 2 - uniform
    for names, uniform in zip(out[2:], (1, 0)):   # stride 2: four classes of input pixels
        assert count(names, "ConvDgradUProb") == 4 * uniform and count(names, "ConvDgradProb") == 4 * (1 - uniform)


def test_groupnorm_passes_stay_within_32_bit_indices(tmp_path_factory):
    """The GroupNorm passes step a 32-bit quad index by their grid: index plus
    one step stays within 2^31 up to 2^31 - 2^21 quads, the most that 8192
    workgroups can step.  This net's convolutions put out 4 and 1024 quads a frame."""
    frames = [1 << 20, (1 << 21) - (1 << 18), (1 << 21) - (1 << 18) + 1, (1 << 21) - (1 << 11)]
    out = record(tmp_path_factory, f"""
h = net("f32", trunk=L.PPO_TRUNK_TINY, in_ch=1, in_hw=4, avgpool=0, tiny_ch=(4, 4096), gn_groups=4)
grids = lambda ls, what: [g for n, g in ls if what in n]
out = [[grids(act(h, f), "gn_apply"), grids(loss_backward(h, f), "gnb_apply")] for f in {frames}]
""")
    for f, (fwd, bwd) in zip(frames, out):
        for quads, grid in zip((4 * f, 1024 * f, 1024 * f, 4 * f), fwd + bwd, strict=True):
            assert quads + 256 * grid <= 1 << 31, (f, quads, grid)
            assert grid == 8192 or grid == min(1 << 20, -(-quads // 256))


def test_pooling_frame_prep_stays_within_32_bit_indices(tmp_path_factory):
    """The pixel-wide frame prep steps a 32-bit pixel index by 8192 workgroups;
    past 2^31 - 2^21 output pixels the elementwise form runs.  4 pixels a frame."""
    most = ((1 << 31) - (1 << 21)) // 4
    out = record(tmp_path_factory, f"""
h = net("f32", trunk=L.PPO_TRUNK_TINY, in_hw=4, avgpool=1, tiny_ch=(4, 4), gn_groups=4)
out = [act(h, f)[0][0] for f in ({most}, {most + 1})]
""")
    assert "prep4_kernel" in out[0] and "prep_kernel" in out[1]


def test_act_graphs_pin_the_net_only_while_there_are_any(tmp_path_factory):
    """A net's act graphs live on one device: a graph-mode call on another is
    refused while there is one, and not after a capture that failed or once they
    were cleared."""
    out = record(tmp_path_factory, """
def collect(h, device, fail=0):
    io = L.CollectIO(T=2, N=2, t_begin=0, t_end=3)
    for f in "obs goal mask u params params_lp actions logp value h_hist c_hist h_last c_last".split():
        setattr(io, f, FAKE)
    C.c_int.in_dll(rec, "rec_device").value = device
    C.c_int.in_dll(rec, "rec_fail_capture").value = fail
    return lib.ppo_collect(h, C.byref(io), L.PPO_COLLECT_GRAPH, FAKE, 1 << 62, None)
h = net("f32", trunk=L.PPO_TRUNK_TINY, in_hw=32, avgpool=0)
count = lambda: lib.ppo_collect_graph_count(h)
out = [collect(h, 0, fail=1), count(), collect(h, 1), count(), collect(h, 0), count(), collect(h, 1),
       lib.ppo_collect_clear(h), collect(h, 0), count(), collect(h, 1)]
""")
    EDEVICE, EINVAL, OK = -5, -1, 0
    assert out == [EDEVICE, 0, OK, 1, EINVAL, 1, OK, 1, OK, 1, EINVAL]


@pytest.mark.parametrize("fwd", ["one_launch", "three_launch"])
def test_groupnorm_backward_takes_its_mask_as_the_forward_formed_it(tmp_path_factory, fwd):
    """Three-launch backward: units with a residual are masked by the saved
    output (1), projection shortcuts not at all (0), the others by the value
    formed again as the forward's kernel formed it (one-launch 3, three-launch
    2).  Group widths that divide 256, so the one-launch form takes every unit:
    the stem and the compression among them."""
    out = record(tmp_path_factory, """
h = net("f32", in_hw=64, base_width=8, gn_groups=2, compress_ch=8)
out = [n for n, _ in loss_backward(h, 7) if "gn" in n]
""", {"DDPPO_GN_FUSED_MAX": "0" if fwd == "three_launch" else str(1 << 30), "DDPPO_GNB_FUSED_MAX": "0"})
    fused = sum("gn_fused_kernel" in n for n in out)
    assert fused == (18 if fwd == "one_launch" else 0)   # stem, 4 x (c1, c2, c3, ds), compression
    for kernel in ("gnb_partial_kernel", "gnb_apply_kernel"):
        masks = [int(n.split("ILi")[1].split("E")[0]) for n in out if kernel in n]
        want = 3 if fwd == "one_launch" else 2
        block = [1, want, want, 0]                       # c3, c2, c1, ds
        assert masks == [want] + 4 * block + [want], kernel


@pytest.mark.parametrize("dtype,in_ch,width,rt", [("f32", 4, 32, 1), ("f32", 12, 8, 1), ("f32", 8, 32, 0),
                                                  ("f32", 4, 64, 0), ("f32", 4, 4, 0), ("f32", 3, 32, 0),
                                                  ("bf16", 4, 32, 0)])
def test_float32_stem_weight_gradient_takes_row_vectors(tmp_path_factory, dtype, in_ch, width, rt):
    """8-row vectors for a float32 stem of at most 32 (8n) output channels on 4n
    but not 8n input channels; scalar loads where they are not 4n; channel quads
    elsewhere (bottleneck units among them)."""
    out = record(tmp_path_factory, f"""
h = net("{dtype}", in_ch={in_ch}, base_width={width}, gn_groups=4)
out = [n for n, _ in loss_backward(h, 4) if "ConvWgrad" in n]
""")
    stem = out[-1]                                       # the last weight gradient of a backward
    kind = "ConvWgradRTProb" if rt else "ConvWgradProb" if in_ch % 4 else "ConvWgradQProb"
    assert kind in stem and sum(kind in n for n in out) >= 1
    assert sum("ConvWgradRTProb" in n for n in out) == rt
