"""The two-layer recurrence kernels where the second layer's cells move to
another wavefront: minibatches that just fit half a workgroup's threads (envs
times units per workgroup = 128), one env more, and a single env, with ragged
lengths down to 1, against the per-layer kernels (whose items do not move)."""
import numpy as np
import pytest

from tests.gpu_util import rel_err
from tests.nets import TINY_BIGCORE
from tests.test_gpu_lstm_seq import TINY_2L64, _run

pytestmark = pytest.mark.gpu


# two units a workgroup at 512 hidden, four at 64
@pytest.mark.parametrize("net,nb", [(TINY_BIGCORE, 1), (TINY_BIGCORE, 64), (TINY_BIGCORE, 65), (TINY_2L64, 32),
                                    (TINY_2L64, 33)], ids=["512_1", "512_64", "512_65", "64_32", "64_33"])
def test_second_layer_items(P, net, nb):
    print(f"lstm items: hidden {net.hidden}, {nb} envs", flush=True)
    T, N = 4, nb + 1
    lengths = [4] + [1 + (7 * e) % 4 for e in range(1, N)]
    envs = list(range(nb))
    _, _, _, g2, s2 = _run(P, net, "f32", T, N, envs, lengths, 17, "seq2")
    _, _, _, g1, s1 = _run(P, net, "f32", T, N, envs, lengths, 17, "seq")
    assert np.all(np.isfinite(g2)) and not np.array_equal(g2, g1)
    assert rel_err(g2, g1) < 1e-5 and abs(s2[0] - s1[0]) <= 1e-5 * max(abs(s1[0]), 1e-6)
