"""fp32 layers on the matrix cores at the edges of their tiles (64 rows, 64
channels or columns, 32 k), against the oracle by the protocols of
tests/parity.py and tests/test_gpu_backward.py (MI355X only), and the
workspace-free forward of a layer whose activations do not fit its scratch,
which runs on the per-pair kernel."""
import numpy as np
import pytest

from synth import generate, get_config, layer_config
from tests import parity
from tests.test_gpu_backward import run_backward
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (tokens, d, K, B, M): rows that start at any 4-byte address (odd d and M),
# one channel per block, one more and one less than a chunk, a last stage of
# one k, many experts with few rows each
FORWARD = {
    "one_token": (1, 8, 2, 2, 3),
    "odd_rows": (130, 33, 3, 5, 7),
    "one_channel": (67, 65, 2, 64, 1),
    "chunk_minus_one": (200, 31, 4, 3, 63),
    "chunk_plus_one": (257, 129, 4, 3, 65),
    "many_experts": (100, 40, 64, 4, 33),
}


def _generate(n, d, K, B, M):
    return generate(get_config("tiny_f32", n_tokens=n, d_model=d, n_experts=K, n_blocks=B, block_width=M, max_shared=B))


@pytest.mark.parametrize("name", list(FORWARD))
def test_forward(name):
    run_case(_generate(*FORWARD[name]), f"fp32 {name}")


BACKWARD = {
    "one_token": (1, 8, 2, 2, 3),
    "chunk_minus_one": (200, 24, 4, 3, 63),
    "chunk_plus_one": (257, 136, 4, 3, 65),
    "many_experts": (100, 40, 64, 4, 33),
}


@pytest.mark.parametrize("name", list(BACKWARD))
def test_backward(name):
    run_backward(_generate(*BACKWARD[name]), f"fp32 {name}")


def test_static_forward_past_its_activations():
    """27,000 worst-case pairs x 1,536 channels are 166 MB of activations:
    more than the static scratch, so the forward without a workspace runs on
    the per-pair kernel. Both are fp32 sums of the same terms."""
    from paper_2608_10392_amd import _lib
    from paper_2608_10392_amd.layer import DeviceLayer
    g = _generate(3000, 32, 8, 8, 192)
    cfg = layer_config(g["cfg"])
    assert _lib.layer_forward_workspace_size(cfg) > _lib.STATIC_WORKSPACE_BYTES
    dev = DeviceLayer(cfg, g["X"], g["valid"], g["W_router"], g["prototypes"], g["W_up"], g["W_down"])
    Y = dev.forward().clone()
    S = torch.empty_like(Y)
    _lib.layer_forward_static(cfg, dev.X, dev.valid, dev.W_router, dev.prototypes, dev.W_up, dev.W_down, S)
    torch.cuda.synchronize()
    rms = float(Y.double().square().mean().sqrt())
    err = float((S - Y).abs().max()) / rms
    print(f"[gpu] fp32 static forward: {err:.1e} x RMS from the workspace forward", flush=True)
    assert err <= parity.KERNEL_TOL["f32"]
    assert np.isfinite(err)
