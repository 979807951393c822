"""The fp32 mode's matrix product and attention at the sizes where their tiles end: segments around one 32-key block, one
round of the four waves (128 keys) and a remainder, every head width the kernel is built for, and both tile sizes.

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


def test_tile_sizes_give_the_same_bits():
    """86 images (5590 rows): more workgroups than the units hold at once, an image alone far fewer."""
    cfg = _cfg(image_size=32, hidden=384, heads=6, mlp=520, proj_layers=1, proj_dims=(200,))
    say("case fp32 tile sizes")
    n = 86
    w, px = gen.make_weights(cfg, seed=1), gen.make_pixels(cfg, n, seed=2)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    for i in (0, 43, n - 1):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], np.array([0, 1], dtype=np.int32))
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-2:], [2], np.arange(3, dtype=np.int32))
    assert assert_parity(whole[-2 * T:], want, "fp32", "fp32 large tiles")[0] <= REL


def test_large_tiles_give_the_same_bits():
    """560 images (36 400 rows, 35 840 of patches) take 64 x 64 tiles in all but the projector (2276 tiles; the line is at 2560),
    an image alone 32 x 32 in every product."""
    cfg = _cfg(image_size=32, hidden=384, heads=6, mlp=520, proj_layers=1, proj_dims=(200,))
    say("case fp32 large tiles")
    n = 560
    w, px = gen.make_weights(cfg, seed=1), gen.make_pixels(cfg, n, seed=2)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    for i in (0, 281, n - 1):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], np.array([0, 1], dtype=np.int32))
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-2:], [2], np.arange(3, dtype=np.int32))
    assert assert_parity(whole[-2 * T:], want, "fp32", "fp32 large tiles")[0] <= REL
