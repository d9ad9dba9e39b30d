"""The post-LN merge (one workgroup per token) at the row lengths where its
shape changes: one wave, whole waves, several chunks per thread, and rows that
leave no LDS for the waves' sums (one wave again), against the oracle by the
protocol of tests/parity.py (MI355X only). More pathways than one batch of the
merge holds, with biases and the residual."""
import pytest

from synth import block_inputs, generate, get_config
from tests.test_gpu_block import run_block

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

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
