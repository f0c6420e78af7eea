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
