"""The 16-bit copies that Adam leaves, as stored and transposed, for widths whose tiles are whole and ragged in both tile sizes, and widths that go through two
kernels: a stack made from the updated weights, whose copies another kernel makes, gives the same outputs and gradients bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from test_gpu_ops import BF16, F16

TYPE = {BF16: torch.bfloat16, F16: torch.float16}


@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("d,heads,ff,layers", [(64, 2, 64, 2), (64, 1, 192, 2), (192, 3, 320, 2), (136, 17, 264, 2), (320, 5, 1280, 2), (1216, 19, 4864, 2),
                                               (192, 3, 320, 1), (1216, 19, 4864, 1), (1728, 27, 6912, 1)])
def test_the_next_pass_uses_the_updated_weights(d, heads, ff, layers, dt):
    n_micro, s = 2, 24
    cfg = B.make_config(layers, d, heads, ff, s, 1, n_micro, dt, group=2, retain_grads=1)
    rng = np.random.default_rng(d + ff)
    params = (rng.standard_normal(layers * B.params_per_layer(cfg)) * 0.05).astype(np.float32)
    g = torch.Generator(device="cuda").manual_seed(d)
    x, dy = (torch.randn(n_micro, 1, s, d, device="cuda", generator=g).to(TYPE[dt]) for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)

    def run(st, adam=None):
        st.forward_layered(x.data_ptr(), y.data_ptr())
        st.backward_layered(dy.data_ptr(), dx.data_ptr(), adam)
        torch.cuda.synchronize()
        return [y.clone(), dx.clone()] + [torch.from_numpy(B.read_device(*st.grads(l), "float32")) for l in range(layers)]

    st = B.Stack(cfg, params)
    run(st, B.lga_adam(1e-2, 0.9, 0.999, 1e-8, 1, 0.0, 0))
    weights = np.concatenate([B.read_device(*st.params(l), "float32") for l in range(layers)])
    assert not np.array_equal(weights, params)
    again = run(st)
    fresh = run(B.Stack(cfg, weights))
    for a, b in zip(again, fresh):
        assert torch.equal(a, b) and torch.isfinite(a.float()).all()
    # an update that is left out leaves the copies alone
    dy[0, 0, 0, 0] = float("inf")
    run(st, B.lga_adam(1e-2, 0.9, 0.999, 1e-8, 2, 2.0, 1))
    dy[0, 0, 0, 0] = 0.5
    want = run(B.Stack(cfg, weights))
    for a, b in zip(run(st), want):
        assert torch.equal(a, b)
