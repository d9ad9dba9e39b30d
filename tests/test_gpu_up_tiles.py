"""The up-projection's tile heights at the sizes where they change over, and
slabs of a row more or less than a tile, against the oracle (MI355X only), by
the protocols of tests/parity.py and tests/test_gpu_backward.py. With K = 4,
calls of up to 960 tokens take 128-row tiles (d >= 256), larger ones 384 (256
for blocks of 256 channels); more than 128 slabs of 64 or 256 channels take
them up to 32 tokens per expert. b = 1 of 2 blocks by prefix: slab (0, 0) holds
every token."""
import pytest

from synth import generate, get_config
from tests.test_gpu_backward import run_backward
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

PREFIX = dict(n_experts=4, n_blocks=2, max_shared=2, alpha_mode="fixed", alpha_fixed=0.5, select_mode="prefix")


@pytest.mark.parametrize("M", [64, 128, 192, 256])
@pytest.mark.parametrize("n", [127, 129, 960, 961])
def test_forward(n, M):
    run_case(generate(get_config("vit_s16", n_tokens=n, d_model=256, block_width=M, **PREFIX)), f"up tiles N={n} M={M}")


@pytest.mark.parametrize("M", [64, 128, 192, 256])
@pytest.mark.parametrize("n", [129, 961])
def test_backward(n, M):
    run_backward(generate(get_config("vit_s16", n_tokens=n, d_model=256, block_width=M, **PREFIX)),
                 f"up tiles N={n} M={M}")


# K = 16, 8 blocks: 136 slabs
MANY = dict(n_experts=16, n_blocks=8, max_shared=8)


@pytest.mark.parametrize("M", [64, 192, 256])
@pytest.mark.parametrize("n", [544, 545])
def test_many_slabs(n, M):
    g = generate(get_config("vit_s16", n_tokens=n, d_model=256, block_width=M, **MANY))
    run_case(g, f"up tiles, 136 slabs N={n} M={M}")
    run_backward(g, f"up tiles, 136 slabs N={n} M={M}")
