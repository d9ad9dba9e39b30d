"""The post-LN merge (one workgroup per token) at the row lengths where its
shape changes: one wave, whole waves, several chunks per thread, and rows that
leave no LDS for the waves' sums (one wave again), against the oracle by the
protocol of tests/parity.py (MI355X only). More pathways than one batch of the
merge holds, with biases and the residual. From 8,192 tokens of at most 512
chunks a token takes one wave; more than 2^32 threads take a grid of two
dimensions."""
import pytest

from synth import block_inputs, generate, get_config
from tests.test_gpu_block import run_block

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = {
    "f32_one_wave": ("tiny_f32", dict(n_tokens=70, d_model=33)),
    "f32_two_waves": ("tiny_f32", dict(n_tokens=70, d_model=65)),
    "f32_several_chunks": ("tiny_f32", dict(n_tokens=9, d_model=777)),
    "f32_longest_with_sums": ("tiny_f32", dict(n_tokens=3, d_model=40952)),
    "f32_longest": ("tiny_f32", dict(n_tokens=3, d_model=40960)),
    "bf16_one_wave": ("vit_s16", dict(n_tokens=70, d_model=128)),
    "bf16_several_chunks": ("vit_s16", dict(n_tokens=40, d_model=2176)),
}


@pytest.mark.parametrize("name", list(ROWS))
def test_post_ln_rows(name):
    base, over = ROWS[name]
    wide = over["d_model"] > 4096
    g = generate(get_config(base, n_experts=2 if wide else 11, n_blocks=2, block_width=2 if wide else 64, max_shared=2,
                            mass_mode="topk", fixed_k=2 if wide else 9, **over))
    blk, X = block_inputs(g, "post", residual=True, eps=1e-6)
    run_block(g, blk, X, name)


MANY = {
    "f32_workgroup": ("tiny_f32", dict(n_tokens=8191, d_model=129)),
    "f32_wave": ("tiny_f32", dict(n_tokens=8192, d_model=129)),
    "f32_wave_512_chunks": ("tiny_f32", dict(n_tokens=8193, d_model=512)),
    "f32_workgroup_513_chunks": ("tiny_f32", dict(n_tokens=8193, d_model=513)),
    "bf16_wave": ("vit_s16", dict(n_tokens=8192, d_model=640)),
}


@pytest.mark.parametrize("name", list(MANY))
def test_post_ln_many_tokens(name):
    base, over = MANY[name]
    g = generate(get_config(base, n_experts=3, n_blocks=2, block_width=64, max_shared=2, **over))
    blk, X = block_inputs(g, "post", residual=True, eps=1e-6)
    run_block(g, blk, X, name, n_sample=200)


def test_post_ln_more_threads_than_a_grid_row():
    """2^24 padded tokens of 520 values, a workgroup of four waves each: 2^32
    threads. A padded token's FFN part is 0, so Y = LN(x)."""
    from paper_2608_10392_amd import _lib
    N, d = 1 << 24, 520
    cfg = dict(n_tokens=N, d_model=d, n_experts=1, n_blocks=2, block_width=2, dtype="f32", mass_threshold=0.6, max_pairs=1)
    f = dict(dtype=torch.float32, device="cuda:0")
    X = torch.zeros(N, d, **f)
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rows = [0, 1, (1 << 22) - 1, 1 << 22, 12345678, N - 2, N - 1]
    X[rows] = torch.randn(len(rows), d, generator=gen, **f)
    valid = torch.zeros(N, dtype=torch.uint8, device="cuda:0")
    blk = dict(norm="post", residual=True, ln_eps=1e-6, ln_gamma=torch.rand(d, generator=gen, **f),
               ln_beta=torch.rand(d, generator=gen, **f), b_up=None, b_down=None)
    W = [torch.randn(*s, generator=gen, **f) for s in ((2, d), (2, d), (2, 4, d), (2, d, 4))]
    Y = torch.full((N, d), float("nan"), **f)
    ws = _lib.alloc_workspace(_lib.block_forward_workspace_size(cfg, blk))
    _lib.block_forward(cfg, blk, X, valid, *W, Y, ws)
    ref = torch.nn.functional.layer_norm(X[rows].double(), (d,), blk["ln_gamma"].double(), blk["ln_beta"].double(), 1e-6)
    assert (Y[rows].double() - ref).abs().max() <= 2e-6
    assert bool((Y[2:(1 << 22) - 1] == blk["ln_beta"]).all()) and bool((Y[(1 << 22) + 1:12345678] == blk["ln_beta"]).all())
    del X, Y, ws
    torch.cuda.empty_cache()
