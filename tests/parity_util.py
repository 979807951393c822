"""Helpers shared by the GPU parity tests: run the HIP library and the oracle on the same seeded inputs."""
import time

import numpy as np

import gen
from oracle import vit_oracle as O

# Parity bar of this project for bf16 arithmetic: per token, max-norm error relative to the
# token's max-norm, and cosine similarity.  fp32 arithmetic is held to a tighter bar that
# reflects fp32 accumulation over at most ~5000-term dot products and a dozen layers.
BF16_REL, BF16_COS = 2e-2, 0.999
FP32_REL, FP32_COS = 2e-4, 0.999999


def say(msg):
    import conftest

    conftest.progress(msg)


def token_metrics(got: np.ndarray, want: np.ndarray):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    assert got.shape == want.shape, (got.shape, want.shape)
    assert np.isfinite(got).all(), "non-finite values in the GPU output"
    rel = np.abs(got - want).max(-1) / np.abs(want).max(-1)
    cos = (got * want).sum(-1) / (np.linalg.norm(got, axis=-1) * np.linalg.norm(want, axis=-1))
    return float(rel.max()), float(cos.min())


def assert_parity(got, want, dtype: str, label=""):
    rel, cos = token_metrics(got, want)
    say(f"    parity {label}: tokens={got.shape[0]} max rel={rel:.3e} min cos={cos:.7f}")
    if dtype == "bf16":
        assert rel <= BF16_REL and cos >= BF16_COS, (label, rel, cos)
    else:
        assert rel <= FP32_REL and cos >= FP32_COS, (label, rel, cos)
    return rel, cos


def gpu_encode(cfg, weights, px, ipr, tile_offsets, enc=None):
    import torch

    import paper_2502_00937_amd as V

    own = enc is None
    if own:
        enc = V.VitEncoder(cfg, weights, device=0)
    out, rto = enc.encode(torch.from_numpy(px).cuda(), ipr, tile_offsets)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    if own:
        enc.close()
    return got, rto


def check_case(cfg, tiles_per_image, ipr, wseed=0, pseed=1, wscale=1.0, oracle_dtype=np.float64, images=None,
               label=""):
    """Encode on the GPU (whole batch) and with the oracle (whole batch or sampled images); compare."""
    weights = gen.make_weights(cfg, seed=wseed)
    if wscale != 1.0:
        weights = weights * np.float32(wscale)
        if cfg["dtype"] == "bf16":
            weights = gen.round_to_bf16(weights)
    to = np.concatenate([[0], np.cumsum(tiles_per_image)]).astype(np.int32)
    px = gen.make_pixels(cfg, int(to[-1]), seed=pseed)
    big = weights.size > (1 << 30)  # progress lines for the one case whose steps take minutes
    if big:
        say(f"    {label}: {weights.size / 1e9:.2f} G weights generated")
    t0 = time.time()
    got, rto = gpu_encode(cfg, weights, px, ipr, to)
    t1 = time.time()
    if big:
        say(f"    {label}: gpu done in {t1 - t0:.1f}s, oracle running")
    want, rto_want = O.vit_oracle_encode(cfg, weights, px, ipr, to, dtype=oracle_dtype, images=images)
    say(f"    {label}: gpu {t1 - t0:.1f}s oracle {time.time() - t1:.1f}s")
    assert list(rto) == list(rto_want)
    T = O.out_tokens_per_tile(cfg)
    if images is None:
        assert_parity(got, want, cfg["dtype"], label)
    else:
        for i in images:
            a, b = int(to[i]) * T, int(to[i + 1]) * T
            assert_parity(got[a:b], want[a:b], cfg["dtype"], f"{label} image {i}")
    return got, want


def planned_products(cfg, n_tiles):
    """{product: (epilogue, its rows, columns and depth, form, rows of a second launch, its form)} of a bf16 encode of that many
    tiles on a device of 256 units, as the library plans them (a walk from the first row to the last; every layer has both)."""
    import paper_2502_00937_amd as V

    up64 = lambda n: -(-n // 64) * 64
    D, dh = cfg["hidden"], cfg["hidden"] // cfg["heads"]
    stored = 64 if dh <= 64 else 72 if dh == 72 else 80 if dh <= 80 else 96 if dh <= 96 else 128
    patches, rows = (cfg["image_size"] // cfg["patch_size"]) ** 2, n_tiles * gen.tokens_per_tile(cfg)
    wide, mlp = cfg["heads"] * stored, up64(cfg["mlp"])
    products = {"patch": ("patch", n_tiles * patches, D, up64(cfg["channels"] * cfg["patch_size"] ** 2)),
                "qkv": ("bias", rows, 3 * wide, up64(D)), "out": ("residual", rows, D, up64(wide)),
                "fc1": ("gelu", rows, mlp, up64(D)), "fc2": ("residual", rows, D, mlp)}
    d_in, n_out, dims = up64(D * cfg["token_merge"] ** 2), n_tiles * gen.out_tokens_per_tile(cfg), cfg["proj_dims"]
    for i, d_out in enumerate(dims):
        last = i + 1 == len(dims)
        products[f"proj{i}"] = ("bias" if last else "gelu", n_out, d_out if last else up64(d_out), d_in)
        d_in = up64(d_out)
    return {name: p + V.vit_product_plan(*p)[:3] for name, p in products.items()}
