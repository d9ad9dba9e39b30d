"""fp32 layers on the matrix cores at the edges of their tiles (64 rows, 64
channels or columns, 32 k), against the oracle by the protocols of
tests/parity.py and tests/test_gpu_backward.py (MI355X only), and the
workspace-free forward of a layer whose activations do not fit its scratch,
which runs on the per-pair kernel. A weight that is not finite reaches the
tokens that run its block and no others. Layers whose activations take more
than 1 GiB run in passes over ranges of experts, blocks or channels."""
import numpy as np
import pytest

from synth import generate, get_config, layer_config, upstream_grad
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


def _spoiled(blocks_of):
    """The layer of the test above with an Inf and a NaN in W_down (or W_up,
    for the backward) of two blocks of two experts, and which tokens run one."""
    from paper_2608_10392_amd.layer import DeviceLayer
    g = _generate(3000, 32, 8, 8, 192)
    bad = {k: g[k].copy() for k in ("W_up", "W_down")}
    bad[blocks_of] = bad[blocks_of].copy()
    for e, c, v in ((0, 2, np.inf), (3, 5, np.nan)):
        if blocks_of == "W_down":
            bad["W_down"][e, 7, c * 192 + 100] = v
        else:
            bad["W_up"][e, c * 192 + 100, 7] = v
    cfg = layer_config(g["cfg"])
    dev = [DeviceLayer(cfg, g["X"], g["valid"], g["W_router"], g["prototypes"], w["W_up"], w["W_down"])
           for w in (g, bad)]
    dev[0].forward()
    r = dev[0].routing_numpy()
    shared = (r["shared_mask"][:, None] >> np.arange(8, dtype=np.uint64)) & np.uint64(1) == 1
    chosen = np.array([3 in r["expert_ids"][t, :r["n_res"][t]] for t in range(3000)])
    uses = shared[:, 2] | (chosen & ~shared[:, 5])
    assert 100 < uses.sum() < 2900
    return g, cfg, dev, uses


def test_weights_that_are_not_finite_stay_in_their_block():
    """Tokens that do not run a block get the output they would get without
    its Inf or NaN, whichever kernel runs; those that do get one that is not
    finite."""
    from paper_2608_10392_amd import _lib
    g, cfg, (clean, bad), uses = _spoiled("W_down")
    ref = clean.Y.cpu().numpy().astype(np.float64)
    rms = np.sqrt(np.mean(ref ** 2))
    bad.forward()
    S = torch.empty_like(bad.Y)
    _lib.layer_forward_static(cfg, bad.X, bad.valid, bad.W_router, bad.prototypes, bad.W_up, bad.W_down, S)
    torch.cuda.synchronize()
    for Y in (bad.Y, S):
        y = Y.cpu().numpy().astype(np.float64)
        assert not np.any(np.isfinite(y[uses, 7]))
        assert np.all(np.isfinite(y[~uses]))
        assert np.abs(y[~uses] - ref[~uses]).max() <= parity.KERNEL_TOL["f32"] * rms


def test_gradients_past_weights_that_are_not_finite():
    g, cfg, (clean, bad), uses = _spoiled("W_up")
    dY = upstream_grad(g)
    ref, got = (d.backward(dY)["dX"].cpu().numpy().astype(np.float64) for d in (clean, bad))
    assert not np.any(np.isfinite(got[uses, 7]))
    assert np.all(np.isfinite(got[~uses]))
    assert np.abs(got[~uses] - ref[~uses]).max() <= parity.KERNEL_TOL["f32"] * np.abs(ref).max()


# More than 1 GiB of worst-case activations: passes of 33 and 32 experts; of one
# expert and 4 of 8 blocks; of one expert and 4,096 or 4,095 channels of a block.
# (tokens, d, K, B, M, every how many tokens one is valid)
PASSES = {
    "experts": (3000, 32, 64, 8, 192, 1),
    "blocks": (20000, 8, 1, 8, 2048, 4),
    "parts": (40000, 8, 1, 2, 8191, 8),
}


@pytest.mark.parametrize("name", list(PASSES))
def test_forward_in_passes(name):
    """The same bits as in one pass, which a capacity of the pairs that the
    routing needs allows, for the layer and with biases; past weights that are
    not finite the same values; and the oracle's values."""
    from paper_2608_10392_amd import _lib
    n, d, K, B, M, every = PASSES[name]
    g = generate(get_config("tiny_f32", n_tokens=n, d_model=d, n_experts=K, n_blocks=B, block_width=M, max_shared=B,
                            mass_mode="topk", fixed_k=min(2, K)))
    g["valid"] = (np.arange(n) % every == 0).astype(np.uint8)
    dev, orec, grec, Y = run_case(g, f"fp32 passes {name}", n_sample=64)
    cfg = layer_config(g["cfg"])
    pairs = int(g["valid"].sum()) * (1 + min(2, K))
    one = dict(cfg, max_pairs=pairs)
    assert 4 * n * (K + 1) * B * M > 1 << 30 > 4 * pairs * B * M
    f = dict(dtype=torch.float32, device="cuda:0")
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    blk = dict(norm="none", residual=True, ln_eps=1e-6, ln_gamma=None, ln_beta=None,
               b_up=torch.randn(K + 1, B * M, generator=gen, **f), b_down=torch.randn(K + 1, d, generator=gen, **f))
    bad = dev.W_down.clone()
    bad[0, 3, M + 1] = float("nan")
    bad[min(2, K), 5, M - 1] = float("inf")
    for W_down, block in ((dev.W_down, None), (dev.W_down, blk), (bad, None)):
        out = []
        for c in (cfg, one):
            y = torch.empty_like(dev.Y)
            layer = (dev.X, dev.valid, dev.W_router, dev.prototypes, dev.W_up, W_down, y)
            if block is None:
                ws = _lib.alloc_workspace(_lib.layer_forward_workspace_size(c))
                _lib.layer_forward(c, *layer, ws)
            else:
                ws = _lib.alloc_workspace(_lib.block_forward_workspace_size(c, block))
                _lib.block_forward(c, block, *layer, ws)
            out.append(y)
        finite = torch.isfinite(out[0])
        assert torch.equal(finite, torch.isfinite(out[1]))
        assert bool(finite.all()) == (W_down is dev.W_down)
        if W_down is dev.W_down:
            assert torch.equal(out[0], out[1])
        else:   # rows formed again are summed in another order
            err = (out[0][finite] - out[1][finite]).abs().max() / out[1][finite].square().mean().sqrt()
            assert err <= parity.KERNEL_TOL["f32"]
    assert np.array_equal(Y, dev.output_numpy())
    del dev, bad, ws
    torch.cuda.empty_cache()
