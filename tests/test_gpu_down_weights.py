"""The down-projection's two sources of fp16 weights give the same bits
(MI355X only): up to 256 tokens per expert it converts the bf16 W_down as it
reads it (up to 128 where W_down has 64 to 96 MB, at no size where it has 16 to
64 MB), past that it reads the copy the routing launch makes. A row's result
does not depend on the other tokens, so the first 1,280 tokens (K + 1 = 5) of
a 1,281-token call must equal the 1,280-token call. The weights reach into
fp16's subnormal range, where the conversion rounds."""
import numpy as np
import pytest

from synth import generate, get_config, layer_config
from synth.generate import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# one case per tile shape of the down-projection
@pytest.mark.parametrize("d", [256, 384, 640])
def test_converted_weights_equal_the_copy(d):
    from paper_2608_10392_amd.layer import DeviceLayer
    n = 256 * 5
    out = []
    for N in (n, n + 1):
        g = generate(get_config("vit_s16", n_tokens=N, d_model=d, n_experts=4, n_blocks=4, block_width=64, max_shared=4))
        scale = np.exp2(-(np.arange(g["W_down"].shape[2]) % 24.0)).astype(np.float32)
        W = f32_to_bf16_bits(bf16_bits_to_f32(g["W_down"]) * scale)
        dev = DeviceLayer(layer_config(g["cfg"]), g["X"], g["valid"], g["W_router"], g["prototypes"], g["W_up"], W)
        dev.forward()
        torch.cuda.synchronize()
        out.append(dev.output_numpy()[:n])
    assert np.any(out[0] != 0)
    np.testing.assert_array_equal(out[0], out[1])


def test_converted_weights_equal_the_copy_large():
    """W_down of 71 MB (K + 1 = 17): converted up to 2,176 tokens."""
    from paper_2608_10392_amd.layer import DeviceLayer
    n = 128 * 17
    out = []
    g = generate(get_config("vit_s16", n_tokens=n + 1, d_model=1024, n_experts=16, n_blocks=16, block_width=128,
                            max_shared=16))
    for N in (n, n + 1):
        dev = DeviceLayer(dict(layer_config(g["cfg"]), n_tokens=N), g["X"][:N], None, g["W_router"], g["prototypes"],
                          g["W_up"], g["W_down"])
        dev.forward()
        torch.cuda.synchronize()
        out.append(dev.output_numpy()[:n])
    assert np.any(out[0] != 0)
    np.testing.assert_array_equal(out[0], out[1])
