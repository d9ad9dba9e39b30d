"""Weight gradients of slabs long enough to be split into units of rows (over
24 stages of 64 rows), against the oracle by the protocol of
tests/test_gpu_backward.py (MI355X only), and bitwise repeatable."""
import pytest

from synth import generate, get_config, layer_config, upstream_grad
from tests.test_gpu_backward import run_backward

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# b = 1 of 2 blocks, block 0 by prefix: every token is on slab (0, 0), and its
# residual expert's pair on block 1. (A few tokens near a tie are left out.)
PREFIX = dict(n_blocks=2, alpha_mode="fixed", alpha_fixed=0.5, select_mode="prefix")
CASES = {
    # just past 24 stages: two parts
    "25_stages": dict(n_tokens=24 * 64 + 20, **PREFIX),
    # 24 stages: not split
    "24_stages": dict(n_tokens=24 * 64, **PREFIX),
    # six parts, a ragged last one
    "141_stages": dict(n_tokens=9001, **PREFIX),
    # two parts in some slabs, one in others, wider tiles
    "mixed": dict(n_tokens=5000, n_blocks=3, d_model=256, block_width=128),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_slabs(name):
    over = dict(dict(d_model=128, n_experts=2, block_width=64), **CASES[name])
    g = generate(get_config("vit_s16", max_shared=over["n_blocks"], **over))
    run_backward(g, f"units {name}")
    from paper_2608_10392_amd.layer import DeviceLayer
    dev = DeviceLayer(layer_config(g["cfg"]), g["X"], g["valid"], g["W_router"], g["prototypes"], g["W_up"],
                      g["W_down"])
    dY = upstream_grad(g)
    a = {k: v.clone() for k, v in dev.backward(dY).items()}
    b = dev.backward(dY)
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k], b[k]), f"{k} is not bitwise repeatable"
