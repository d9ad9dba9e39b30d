"""The routing launches at the sizes where they change over, against the
oracle (MI355X only): one tile per workgroup up to 256 tiles of 64 tokens
(512 where the router has at most 16 columns), past that the register-held router (at most 32 columns, d <= 1024) or the
streamed one, and the fp32 logits at row lengths that are not a multiple of
any vector width. Decisions are compared by the protocol of tests/parity.py
(exact beyond a margin of 1e-4; alpha and affinities within 1e-5, the fp32
accumulation-order spread it derives)."""
import numpy as np
import pytest

import oracle.unif_moe_oracle as O
from synth import generate, get_config, layer_config
from tests import parity
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    # (tokens, d, K, B, dtype): lists of 8, 16, 32 and 64 entries, one and
    # all columns of the last 16-column tile used, an odd count of k steps
    "split_8": (16384, 96, 8, 8, "bf16"),
    "split_33_columns": (130, 1056, 32, 2, "bf16"),
    "split_128_columns": (64, 64, 64, 64, "bf16"),
    "held_16_columns": (16385, 96, 8, 8, "bf16"),
    "held_32_columns": (16449, 1024, 2, 30, "bf16"),
    "wide_d_over_1024": (16385, 1056, 3, 4, "bf16"),
    "split_narrow_last": (32768, 160, 7, 9, "bf16"),
    "held_narrow_first": (32769, 160, 7, 9, "bf16"),
    "wide_narrow_first": (32769, 1056, 3, 4, "bf16"),
    "wide_33_columns": (16385, 96, 16, 17, "bf16"),
    "wide_64_columns": (16700, 128, 32, 32, "bf16"),
    "wide_65_columns": (16385, 32, 64, 2, "bf16"),
    "wide_128_columns": (16641, 160, 64, 64, "bf16"),
    "f32_one_expert": (65, 5, 1, 2, "f32"),
    "f32_129_columns": (200, 33, 64, 64, "f32"),
    "f32_long_rows": (63, 1027, 7, 9, "f32"),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("padded", [False, True])
def test_route(name, padded):
    from paper_2608_10392_amd.layer import DeviceLayer
    N, d, K, B, dtype = CASES[name]
    print(f"\n[gpu] route {name}: N={N} d={d} K={K} B={B} {dtype} padded={padded}", flush=True)
    base = "vit_s16" if dtype == "bf16" else "tiny_f32"
    g = generate(get_config(base, n_tokens=N, d_model=d, n_experts=K, n_blocks=B, block_width=64, max_shared=B),
                 weights=False)
    cfg = g["cfg"]
    valid = (np.arange(N) % 7 != 3).astype(np.uint8) if padded else None
    dev = DeviceLayer(layer_config(cfg), g["X"], valid, g["W_router"], g["prototypes"])
    dev.route()
    torch.cuda.synchronize()
    orec = O.route(cfg, g["X"], valid, g["W_router"], g["prototypes"])
    s = parity.check_routing(cfg, orec, dev.routing_numpy())
    print(f"[gpu] route {name}: {s['n_checked']}/{s['n_valid']} decisions, alpha err {s['max_alpha_err']:.1e}, "
          f"p err {s['max_p_err']:.1e}", flush=True)


# The same launches in a forward, where the decisions also take the pairs'
# slots and the tile's counts: every row of the expert FFNs depends on them.
# One tile, the last and the first sizes of each launch (256 tiles; 1,280
# tiles, past which one wave does a tile), lists of 8 to 64 entries, and the
# slots gathered over a wave (prefix selection, at most 4 mask bits).
FORWARDS = {
    "one_tile": (33, 12, 8, {}),
    "split_last": (16384, 16, 16, {}),
    "held_first": (16385, 16, 16, {}),
    "split_narrow_last": (32768, 8, 8, {}),
    "held_narrow_first": (32769, 8, 8, {}),
    "held_prefix": (16400, 9, 12, dict(select_mode="prefix")),
    "held_4_blocks": (16400, 16, 4, {}),
    "held_topk": (16400, 16, 8, dict(mass_mode="topk", fixed_k=16)),
    "held_last_shared": (1280 * 64, 16, 8, {}),
    "held_one_wave": (1280 * 64 + 1, 16, 8, {}),
    "wide_33_columns": (16385, 16, 17, {}),
    "wide_65_columns": (16385, 63, 2, {}),
    "wide_128_columns": (16641, 64, 64, {}),
}


@pytest.mark.parametrize("name", list(FORWARDS))
def test_forward(name):
    N, K, B, modes = FORWARDS[name]
    g = generate(get_config("vit_s16", n_tokens=N, d_model=128, n_experts=K, n_blocks=B, block_width=64, max_shared=B,
                            **modes))
    g["valid"] = (np.arange(N) % 7 != 3).astype(np.uint8)
    run_case(g, f"routing launch {name}", n_sample=96)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("select", ["prototype", "prefix"])
def test_route_ties_and_prefix(select):
    """Equal affinities and priorities rank by index: tokens of zeros tie
    everywhere, so I_shr is the first b blocks and q = 1..K in order. With
    prefix selection I_shr is the first b blocks of every token."""
    from paper_2608_10392_amd.layer import DeviceLayer
    N, d, K, B = 129, 64, 12, 20
    g = generate(get_config("vit_s16", n_tokens=N, d_model=d, n_experts=K, n_blocks=B, block_width=64, max_shared=B,
                            select_mode=select), weights=False)
    X = g["X"].copy()
    X[::2] = 0
    dev = DeviceLayer(layer_config(g["cfg"]), X, None, g["W_router"], g["prototypes"])
    dev.route()
    torch.cuda.synchronize()
    r = dev.routing_numpy()
    for t in range(N):
        b = int(r["n_shared"][t])
        if t % 2 == 0 or select == "prefix":
            assert int(r["shared_mask"][t]) == (1 << b) - 1
        if t % 2 == 0:
            assert r["expert_ids"][t].tolist() == list(range(1, K + 1))
            assert np.all(r["weights"][t] == r["weights"][t, 0])
