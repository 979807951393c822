"""The fp32 mode's matrix product and attention at the sizes where their tiles end: segments around one 32-key block, one
round of the four waves (128 keys) and a remainder, every head width the kernel is built for, and every form of the product.

Tolerance: the fp32 bar of the parity tests allows for a dozen layers.  Two blocks round about fourteen times in a row (twice
LayerNorm, four products, attention), each time by a few units of 2^-24 = 6e-8 of the token's largest value, which add up
like random steps: 6e-8 x 3 x sqrt(14) = 7e-7.  Measured 3.7e-7 to 6.4e-7; the bar is four times the largest."""
import numpy as np
import pytest

import gen
from oracle import vit_oracle as O
from parity_util import assert_parity, say
from test_gpu_parity import gpu_encode

pytestmark = pytest.mark.gpu

REL = 2.6e-6


def _cfg(**kw):
    cfg = {"image_size": 24, "patch_size": 4, "channels": 3, "hidden": 64, "heads": 1, "mlp": 128, "layers_local": 1,
           "layers_global": 1, "has_cls": 1, "final_ln": 1, "ln_eps": 1e-6, "proj_layers": 0, "proj_dims": (), "dtype": "fp32",
           "token_merge": 1}
    cfg.update(kw)
    return cfg


@pytest.mark.parametrize("dh,heads,grid,has_cls,tiles", [
    (64, 3, 2, 1, [6, 1, 13]),    # 5 tokens a tile; global segments of 30, 5 and 65 keys
    (72, 2, 4, 0, [2, 8, 1, 9]),  # 16 tokens a tile; global segments of 32, 128, 16 and 144 keys
    (80, 1, 8, 0, [1, 2, 4]),     # 64, 128 and 256 keys
    (96, 2, 11, 1, [1, 3]),       # 122 and 366 keys
    (128, 1, 14, 1, [1, 2]),      # 197 and 394 keys
])
def test_segment_lengths_and_head_dims(dh, heads, grid, has_cls, tiles):
    cfg = _cfg(image_size=4 * grid, hidden=dh * heads, heads=heads, mlp=8 * (dh + 3), has_cls=has_cls)
    say(f"case fp32 head dim {dh} x {heads}, {grid * grid + has_cls} tokens a tile, tiles {tiles}")
    to = np.concatenate([[0], np.cumsum(tiles)]).astype(np.int32)
    w, px = gen.make_weights(cfg, seed=dh), gen.make_pixels(cfg, int(to[-1]), seed=grid)
    got, _ = gpu_encode(cfg, w, px, [len(tiles)], to)
    want, _ = O.vit_oracle_encode(cfg, w, px, [len(tiles)], to)
    assert assert_parity(got, want, "fp32", f"fp32 dh{dh}")[0] <= REL


def _forms(cfg, n):
    """The forms of the fp32 product that an encode of n tiles takes: tile side x k-blocks in flight (launch_gemm_f32's rule)."""
    rows, D, M, up64 = n * gen.tokens_per_tile(cfg), cfg["hidden"], cfg["mlp"], lambda v: -(-v // 64) * 64
    forms = set()
    for m, c, k in [(n * (gen.tokens_per_tile(cfg) - cfg["has_cls"]), D, up64(48)), (rows, 3 * D, up64(D)), (rows, D, up64(D)), (rows, up64(M), up64(D)),
                    (rows, D, up64(M))] + [(rows, d, up64(D)) for d in cfg["proj_dims"]]:
        t64, t32 = -(-m // 64) * -(-c // 64), -(-m // 32) * -(-c // 32)
        large = t64 >= 512 and -(-t64 // 256) * 400 <= -(-t32 // 256) * 118 if k >= 768 else t64 >= 2560
        forms.add(("64 x 2" if k >= 768 else "64 x 1") if large else "32 x 3")
    return forms


@pytest.mark.parametrize("hidden,heads,mlp,proj,n,takes", [
    (384, 6, 520, (200,), 86, {"32 x 3"}),                # 5590 rows: more workgroups than the units hold at once
    (384, 6, 520, (200,), 560, {"64 x 1", "32 x 3"}),     # 36 400 rows; 2276 large tiles in the projector, under the line
    (128, 2, 1024, (), 256, {"64 x 1", "32 x 3"}),        # fc1 of two k-blocks on 4160 large tiles
    (768, 12, 1536, (136,), 64, {"64 x 2", "32 x 3"}),    # shares of 10 against 9.25 in QKV, 4 against 3.25 in out-proj
    (256, 4, 1032, (), 185, {"64 x 2", "64 x 1", "32 x 3"}),  # fc2 of 17 k-blocks, an odd number
])
def test_forms_of_the_product_give_the_same_bits(hidden, heads, mlp, proj, n, takes):
    """Tiles of 32 x 32 and 64 x 64 with one to three k-blocks in flight; an image alone takes 32 x 32 ones in every product."""
    cfg = _cfg(image_size=32, hidden=hidden, heads=heads, mlp=mlp, proj_layers=len(proj), proj_dims=proj)
    assert _forms(cfg, n) == takes and _forms(cfg, 1) == {"32 x 3"}, _forms(cfg, n)
    say(f"case fp32 forms, width {hidden}, {n} images")
    w, px = gen.make_weights(cfg, seed=1), gen.make_pixels(cfg, n, seed=2)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    for i in sorted({0, n // 2, n - 1}):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], np.array([0, 1], dtype=np.int32))
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-2:], [2], np.arange(3, dtype=np.int32))
    assert assert_parity(whole[-2 * T:], want, "fp32", f"fp32 forms width {hidden}")[0] <= REL
