"""Every tile of the small-problem matrix product: batch sizes at which the products of one encoder take tiles of 64 to 256 rows
by 64 or 128 columns, with ragged last row and column blocks, and the persistent kernel.  An image's tokens must not depend on
the tile (bit for bit against the image alone), and the image alone is held to the oracle at the bar of the parity tests."""
import numpy as np
import pytest

import gen
import paper_2502_00937_amd as V
from oracle import vit_oracle as O
from parity_util import assert_parity, say
from test_gpu_parity import gpu_encode

pytestmark = pytest.mark.gpu

CFG = {"image_size": 60, "patch_size": 4, "channels": 3, "hidden": 512, "heads": 8, "mlp": 2056, "layers_local": 2,
       "layers_global": 0, "has_cls": 1, "final_ln": 1, "ln_eps": 1e-6, "proj_layers": 1, "proj_dims": (1096,), "dtype": "bf16",
       "token_merge": 1}


@pytest.mark.parametrize("n", [2, 3, 5, 9, 20, 33, 80])
def test_tokens_do_not_depend_on_the_tile(n):
    say(f"case matrix-product tiles, {n} images of 226 tokens")
    w, px = gen.make_weights(CFG, seed=3), gen.make_pixels(CFG, n, seed=n)
    whole, _ = gpu_encode(CFG, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(CFG)
    one = np.array([0, 1], dtype=np.int32)
    for i in sorted({0, n // 2, n - 1}):
        alone, _ = gpu_encode(CFG, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(CFG, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"tiles n={n}")


@pytest.mark.parametrize("n", [30, 33, 37])
def test_rows_alone_cut_over_the_xcds(n):
    """Five tile columns: only the rows are dealt over the XCDs, and the last one has 4, 4 and 3 of the others' 7, 8 and 9
    row blocks of 128."""
    cfg = dict(CFG, hidden=576, heads=9, mlp=1160, layers_local=1)
    say(f"case matrix-product tiles, {n} images of 226 tokens, width 576")
    w, px = gen.make_weights(cfg, seed=4), gen.make_pixels(cfg, n, seed=n)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    one = np.array([0, 1], dtype=np.int32)
    for i in (0, n // 2, n - 1):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"row cut n={n}")


@pytest.mark.parametrize("n,hidden,mlp", [(14, 512, 2056), (28, 512, 2056), (44, 512, 2056), (50, 512, 2056), (60, 512, 2056),
                                          (40, 64, 4104), (40, 128, 4104), (40, 192, 4104)])
def test_tile_heights_and_short_products(n, hidden, mlp):
    """Tiles of 96 to 256 rows (none of which divides n * 226), with one and with two workgroups to a unit, under every epilogue;
    and products of one, two and three k-stages, fewer than the tiles' rings hold."""
    cfg = dict(CFG, hidden=hidden, heads=hidden // 64, mlp=mlp, layers_local=1)
    say(f"case matrix-product tiles, {n} images of 226 tokens, width {hidden}")
    w, px = gen.make_weights(cfg, seed=5), gen.make_pixels(cfg, n, seed=n)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    one = np.array([0, 1], dtype=np.int32)
    for i in sorted({0, n // 3, n // 2, n - 1}):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"tile heights n={n} width={hidden}")


@pytest.mark.parametrize("mlp", [4096, 4104, 4424])
def test_five_stage_ring(mlp):
    """fc2 of 64 to 70 k-stages: on 64 x 64 tiles with a ring of five stages for one and three images, on larger tiles for 40."""
    cfg = dict(CFG, mlp=mlp, layers_local=1, proj_layers=0, proj_dims=())
    say(f"case ring of five stages, mlp {mlp}")
    n = 40
    w, px = gen.make_weights(cfg, seed=8), gen.make_pixels(cfg, n, seed=mlp)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    for i, k in ((0, 1), (17, 3), (n - 1, 1)):
        some, _ = gpu_encode(cfg, w, px[i:i + k], [k], np.arange(k + 1, dtype=np.int32))
        assert np.array_equal(some, whole[i * T:(i + k) * T]), i
    one = np.array([0, 1], dtype=np.int32)
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"five stages mlp={mlp}")


@pytest.mark.parametrize("hidden,mlp,n", [(320, 2056, 273), (576, 3016, 182), (832, 3016, 127), (832, 3016, 182), (1088, 2056, 100)])
def test_tokens_do_not_depend_on_the_persistent_kernel(hidden, mlp, n):
    """Products that the persistent kernel takes, several tiles to a workgroup, at odd numbers of k-stages: QKV of 5, 13 and 17
    (four tile columns, the last of them ragged, and 8 + 2 and 12 + 1 of them), fc1 of 9 and 13; and fc2 of 832 columns at 127
    images, whose last round of rows is a launch of its own.  An image alone takes one tile per workgroup."""
    cfg = dict(CFG, hidden=hidden, heads=hidden // 64, mlp=mlp, layers_local=1, proj_layers=0, proj_dims=())
    say(f"case persistent matrix product, {n} images of 226 tokens, width {hidden}")
    w, px = gen.make_weights(cfg, seed=7), gen.make_pixels(cfg, n, seed=n)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    one = np.array([0, 1], dtype=np.int32)
    for i in sorted({0, n // 3, n // 2, n - 1}):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"persistent n={n} width={hidden}")


@pytest.mark.parametrize("dh,heads,n", [(64, 16, 100), (72, 4, 70), (80, 4, 70), (96, 4, 70), (128, 4, 70)])
def test_tokens_do_not_depend_on_the_attention_kernel(dh, heads, n):
    """Two query blocks per image and head: the whole batch has more workgroups than the pipelined form of the attention kernel
    takes, an image alone has 8 to 32.  170 keys: two full tiles, then one of more than 32 keys."""
    cfg = dict(CFG, image_size=52, hidden=dh * heads, heads=heads, mlp=64, layers_local=1, proj_layers=0, proj_dims=())
    say(f"case attention forms, head dim {dh}, {n} images of 170 tokens")
    w, px = gen.make_weights(cfg, seed=6), gen.make_pixels(cfg, n, seed=dh)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    one = np.array([0, 1], dtype=np.int32)
    for i in (0, n // 2, n - 1):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"attention forms dh={dh}")


@pytest.mark.parametrize("form", [None, *V.PRODUCT_FORMS])
def test_timing_aid_takes_every_form(form):
    import torch

    say(f"case timing of a product, {form}")
    ws = torch.empty(64 << 20, dtype=torch.bfloat16, device="cuda").uniform_(-1.0, 1.0)
    for epilogue in V.PRODUCT_EPILOGUES:
        us = V.vit_product_time(epilogue, 700, 328, 192, ws.data_ptr(), ws.numel() * 2, form)
        assert 1.0 < us < 2000.0, (epilogue, us)
    with pytest.raises(V.VitError):
        V.vit_product_time("bias", 700, 328, 192, ws.data_ptr(), 1 << 20, form)
