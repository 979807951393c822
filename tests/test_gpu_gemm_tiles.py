"""Every form of the bf16 matrix product: tiles of 64 to 256 rows by 64 or 128 columns, one or two workgroups to a unit, with
ragged last row and column blocks; the persistent kernel; and its last rows as a second launch.  An image's tokens must not
depend on the form (bit for bit against the image alone), and one image is held to the oracle at the bar of the parity tests.
Which forms a case is there for is asserted, so that a change of the choice shows."""
import numpy as np
import pytest

import gen
import paper_2502_00937_amd as V
from oracle import vit_oracle as O
from parity_util import assert_parity, planned_products, say
from test_gpu_parity import gpu_encode

pytestmark = pytest.mark.gpu

PERSISTENT = V.PRODUCT_FORMS[9]
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
def test_width_of_an_odd_number_of_64_column_blocks(n):
    """Nine blocks of 64 columns, 27 of QKV and 19 of the MLP: tiles of 128 columns end half way."""
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
    """Tiles of 96 to 256 rows (none of which divides n * 226), with one and with two workgroups to a unit; and products of one,
    two and three k-stages, fewer than the tiles' rings hold."""
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


@pytest.mark.parametrize("hidden,mlp,n,takes", [(320, 2056, 273, {"qkv", "fc1"}), (576, 3016, 182, {"fc1"}), (832, 3016, 127, {"fc1", "fc2"}),
                                                (832, 3016, 182, {"qkv", "fc1", "fc2"}), (1088, 2056, 100, {"qkv"})])
def test_tokens_do_not_depend_on_the_persistent_kernel(hidden, mlp, n, takes):
    """Products that the persistent kernel takes, several tiles to a workgroup, at odd numbers of k-stages: QKV of 5, 13 and 17
    (four tile columns, the last of them ragged, and 8 + 2 and 12 + 1 of them), fc1 of 9 and 13; and fc2 of 832 columns at 127
    images, whose last round of rows is a launch of its own.  An image alone takes one tile per workgroup."""
    cfg = dict(CFG, hidden=hidden, heads=hidden // 64, mlp=mlp, layers_local=1, proj_layers=0, proj_dims=())
    plan = planned_products(cfg, n)
    assert {name for name, p in plan.items() if p[4] == PERSISTENT} >= takes, plan
    assert plan["fc2"][5] > 0 or (hidden, n) != (832, 127), plan
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


# (patch, width, heads, MLP, projector, images, what they are there for): of every form under every epilogue that the choice
# gives it ("heads": QKV stored head by head), and of every form that takes the last rows of a product on the persistent kernel
# ("rest"), the ones that few images reach.
FORMS_TAKEN = [
    (4, 192, 3, 2056, (512, 1024), 302, "bias persistent 256x256, bias rest 96x128, gelu 192x128 two a unit, "
     "gelu persistent 256x256, heads 192x128 two a unit, patch 64x64, residual 64x64, residual persistent 256x256, "
     "residual rest 64x64"),
    (4, 320, 4, 64, (512, 1024), 61, "bias 160x128 two a unit, bias 256x128, gelu 256x128, gelu 64x64, "
     "patch 160x128 two a unit, residual 160x128 two a unit, residual 192x128 two a unit"),
    (16, 512, 8, 1024, (512, 1024), 10, "bias 96x128, gelu 64x128, gelu 96x128, heads 128x128, patch 64x128, residual 64x128"),
    (14, 384, 6, 4104, (512, 1024), 27, "bias 192x128, gelu 128x128, gelu 160x128 two a unit, heads 256x128, patch 96x128, "
     "residual 96x128"),
    (14, 640, 10, 1024, (256,), 23, "bias 64x128, gelu 192x128, heads 160x128 two a unit, patch 128x128, residual 128x128"),
    (4, 512, 8, 1024, (1096,), 334, "bias 192x128 two a unit, gelu rest 160x128 two a unit, heads persistent 256x256, "
     "patch persistent 256x256, residual rest 192x128"),
    (14, 640, 10, 1024, (1096,), 30, "patch 160x128, residual 160x128, residual 192x128"),
    (16, 512, 8, 64, (256,), 56, "bias 128x128, patch 256x128, residual 256x128"),
    (4, 192, 3, 256, (256,), 1, "bias 64x64, heads 64x64"),
    (4, 640, 10, 1024, (512, 1024), 232, "bias rest 128x128, gelu rest 128x128, patch 192x128 two a unit"),
    (4, 192, 3, 64, (1096,), 8, "heads 96x128"),
    (4, 640, 10, 64, (), 3, "heads 64x128"),
    (4, 384, 6, 64, (256,), 16, "heads 192x128"),
    (14, 1024, 16, 512, (), 7, "heads 160x128"),
    (4, 64, 1, 256, (512, 1024), 313, "bias rest 192x128"),
    (4, 128, 2, 256, (512, 1024), 252, "bias rest 256x128"),
    (4, 128, 1, 64, (512, 1024), 328, "bias rest 160x128 two a unit"),
    (4, 192, 3, 2056, (256,), 318, "residual rest 64x128"),
    (4, 1024, 16, 512, (), 238, "residual rest 160x128, residual rest 160x128 two a unit"),
    (4, 256, 4, 2056, (512, 1024), 327, "residual rest 96x128"),
    (4, 640, 10, 1024, (512, 1024), 167, "gelu rest 192x128"),
    (4, 640, 10, 1024, (256,), 195, "gelu rest 192x128 two a unit"),
    (4, 320, 4, 4104, (512, 1024), 221, "residual rest 256x128"),
    (4, 512, 8, 1024, (512, 1024), 324, "residual rest 128x128"),
    (4, 512, 8, 2056, (512, 1024), 236, "residual rest 192x128 two a unit"),
    (4, 640, 10, 1024, (1096,), 252, "gelu rest 256x128"),
    (4, 640, 10, 1024, (), 303, "gelu rest 96x128"),
]


@pytest.mark.parametrize("patch,hidden,heads,mlp,proj,n,there_for", FORMS_TAKEN)
def test_tokens_do_not_depend_on_the_form(patch, hidden, heads, mlp, proj, n, there_for):
    """Two layers: each product is walked from both ends."""
    cfg = dict(CFG, image_size=15 * patch, patch_size=patch, hidden=hidden, heads=heads, mlp=mlp, proj_layers=len(proj), proj_dims=proj)
    taken = set()
    for name, (epilogue, _, _, _, form, rest, rest_form) in planned_products(cfg, n).items():
        kind = "heads" if name == "qkv" and hidden // heads in (64, 128) else epilogue
        taken |= {f"{kind} {form}"} | ({f"{kind} rest {rest_form}"} if rest else set())
    assert taken >= set(there_for.split(", ")), taken
    say(f"case forms of matrix products: {n} images, patches of {patch}, width {hidden}: {there_for}")
    w, px = gen.make_weights(cfg, seed=11), gen.make_pixels(cfg, n, seed=n)
    whole, _ = gpu_encode(cfg, w, px, [n], np.arange(n + 1, dtype=np.int32))
    T = gen.tokens_per_tile(cfg)
    one = np.array([0, 1], dtype=np.int32)
    for i in sorted({0, n // 3, n // 2, max(n - 2, 0), n - 1}):
        alone, _ = gpu_encode(cfg, w, px[i:i + 1], [1], one)
        assert np.array_equal(alone, whole[i * T:(i + 1) * T]), i
    want, _ = O.vit_oracle_encode(cfg, w, px[-1:], [1], one)
    assert_parity(whole[-T:], want, "bf16", f"forms n={n} width={hidden}")


# (rows, columns, k-stages): one tile and many, ends of tiles in rows and columns,
# fewer stages than any ring holds, and several rounds of the persistent kernel with odd and even numbers of stages
@pytest.mark.parametrize("epilogue", ["bias", "gelu", "patch"])
@pytest.mark.parametrize("rows,columns,stages", [(1, 8, 1), (63, 64, 2), (65, 136, 3), (191, 264, 4), (257, 128, 5), (700, 328, 6), (1729, 1032, 2),
                                                 (3000, 4104, 1), (8200, 3080, 3), (20000, 1288, 7)])
def test_every_form_gives_the_same_bits(epilogue, rows, columns, stages):
    """Every form through the timing aid, whose workspace starts with the output and goes on with operand, bias, position rows and
    one copy of the weights, each 256-byte aligned.  Against a product in fp32 of the same bf16 values: rounding of the result
    (2^-8 relative to the largest value in a row, GELU's derivative is at most 1.13) and of fp32 sums."""
    import torch

    say(f"case every form, {epilogue}, {rows} x {columns}, {stages} k-stages")
    depth, up = 64 * stages, lambda v, m: -(-v // m) * m
    out_rows = rows if epilogue != "patch" else -(-rows // 576) * 577
    sizes = [out_rows * columns * (4 if epilogue == "patch" else 2), up(rows, 256) * depth * 2, up(columns, 256) * 4, 577 * columns * 4,
             up(columns, 256) * depth * 2]
    at = np.concatenate([[0], np.cumsum([up(b, 256) for b in sizes])])
    ws = torch.empty(int(at[-1]), dtype=torch.uint8, device="cuda")
    part = lambda i, dtype: ws[int(at[i]):int(at[i]) + sizes[i]].view(dtype)
    g = torch.Generator(device="cuda").manual_seed(rows)
    ws.view(torch.bfloat16).uniform_(-1.0, 1.0, generator=g)
    part(2, torch.float32).uniform_(-1.0, 1.0, generator=g)
    part(3, torch.float32).uniform_(-1.0, 1.0, generator=g)
    a, w = part(1, torch.bfloat16).view(-1, depth)[:rows].float(), part(4, torch.bfloat16).view(-1, depth)[:columns].float()
    want = (a.double() @ w.double().t() if rows * columns < 1 << 20 else a @ w.t()).double() + part(2, torch.float32)[:columns].double()
    if epilogue == "gelu":
        want = torch.nn.functional.gelu(want)
    if epilogue == "patch":
        tok = torch.arange(rows, device="cuda") % 576 + 1
        want += part(3, torch.float32).view(577, columns)[tok].double()
    fill = torch.full_like(part(0, torch.uint8), 0x5A)
    first = None
    for form in (*V.PRODUCT_FORMS, None):
        part(0, torch.uint8).copy_(fill)
        V.vit_product_time(epilogue, rows, columns, depth, ws.data_ptr(), ws.numel(), form)
        got = part(0, torch.uint8).clone()
        if first is None:
            first = got
            values = got.view(torch.float32 if epilogue == "patch" else torch.bfloat16).view(-1, columns)
            if epilogue == "patch":
                row = torch.arange(rows, device="cuda")
                values = values[row // 576 * 577 + row % 576 + 1]
            bar = (2.0 ** -8 if epilogue != "patch" else 0.0) * want.abs().amax(1, keepdim=True) + 2.0 ** -22 * depth
            assert bool(((values.double() - want).abs() <= bar).all()), (form, float((values.double() - want).abs().max()))
        assert torch.equal(got, first), (form, int((got != first).sum()))


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
