"""GPU parity of the exact block (Eq. 1) through ff_block_exact: element-wise against the
oracle at small ragged shapes (several tiles plus tails in every GEMM dimension, head dims
64 and 72, token tails), and on sampled rows at the workloads' full shapes."""
import numpy as np
import pytest
import torch

import gemm_plan
import oracle as O
import synth
from paper_2607_27842_amd import abi, pipeline
from gpu_util import TOL, dev, host, need_gpu, say

pytestmark = pytest.mark.gpu


def ragged_cfg(kind, dtype, d=64, H=5, n_txt=0, B=2, lat=(4, 1, 20, 20), mlp_ratio=2):
    C = H * d
    kinds = [kind]
    n_img = (lat[1]) * (lat[2] // 2) * (lat[3] // 2)
    return dict(name="ragged", kinds=kinds, C=C, H=H, d=d, mlp=mlp_ratio * C, n_img=n_img, n_txt=n_txt, B=B,
                lat=lat, patch=(1, 2, 2), dtype=dtype, T=4, R=2, K=1, S=2, sites=[], site_rule="fixed",
                ln_eps=1e-6, rel_eps=1e-8)


def run_block(cfg, W, u_np, c_np, rows=None):
    dt = pipeline.torch_dtype(cfg)
    sets = [W["txt"], W["img"]] if cfg["kinds"][0] == synth.MMDIT_DOUBLE else [W]
    tens = [{k: dev(v, dt) for k, v in s.items()} for s in sets]
    lw = abi.ff_layer_weights()
    for si, s in enumerate(tens):
        for k, t in s.items():
            setattr(lw.s[si], k, t.data_ptr())
    m = pipeline.model_desc(cfg)
    ws_bytes = abi.ff_workspace_bytes(m)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    u = dev(u_np, dt)
    c = dev(c_np, torch.float32)
    h = torch.empty_like(u)
    abi.ff_block_exact(m, 0, lw, c.data_ptr(), u.data_ptr(), h.data_ptr(), ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    h2 = torch.empty_like(u)
    abi.ff_block_exact(m, 0, lw, c.data_ptr(), u.data_ptr(), h2.data_ptr(), ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    bits = torch.int16 if dt == torch.bfloat16 else torch.int32   # (NaN included)
    assert torch.equal(h.view(bits), h2.view(bits)), "exact block is not deterministic"
    return host(h)


def boosted(W, kind):
    # larger modulation weights make every gate O(1) so that each branch is visible in h - u
    def b(s):
        s = dict(s)
        s["mod_w"] = (s["mod_w"] * 8).astype(np.float32)
        return s
    return {k: b(v) for k, v in W.items()} if kind == synth.MMDIT_DOUBLE else b(W)


def grown(W, cfg):
    # matrices of N(0, 0.02^2) at small widths leave the update far below the rounding of h: scaled (by a
    # power of two, exact in bf16) so that a product keeps its input's size
    up = np.float32(2.0 ** round(np.log2(1 / (0.02 * np.sqrt(cfg["C"])))))
    for s in ([W["txt"], W["img"]] if cfg["kinds"][0] == synth.MMDIT_DOUBLE else [W]):
        for k in s:
            if k.endswith("_w") and k != "mod_w":
                s[k] = s[k] * up


def check_block(cfg, W, seed=0, rows=None, tol=None):
    kind = cfg["kinds"][0]
    bf = cfg["dtype"] == synth.BF16
    B, N, C = cfg["B"], cfg["n_img"] + cfg["n_txt"], cfg["C"]
    u = synth.normal((B, N, C), 300 + seed, bf16=bf)
    c = synth.normal((B, C), 400 + seed)
    got = run_block(cfg, W, u, c)
    u64 = u.astype(np.float64)
    cs = O.silu(c.astype(np.float64))
    ref = O.block(kind, u64, cs, W, cfg, rows=rows)
    if bf:
        ref = O.round_bf16(ref)
    g = got if rows is None else got[:, rows]
    uu = u64 if rows is None else u64[:, rows]
    err = O.max_rel_err(g - uu, ref - uu)       # error relative to the block's own update h - u
    tol = TOL[cfg["dtype"]] if tol is None else tol
    say(f"  block kind={kind} dtype={cfg['dtype']} B={B} N={N} C={C} d={cfg['d']}: err(h-u)={err:.3e} tol={tol}")
    assert err <= tol, err
    return err


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("d,H", [(8, 40), (40, 8), (64, 5), (72, 5), (96, 5)])
def test_dit_block_ragged(dtype, d, H):
    # head dims from the smallest the boundary accepts (8, zero-padded to the 64-wide
    # attention tile) through the 80- and 96-wide tiles.  The small dims take many heads:
    # at C = 40 the block's update h - u is so small against h (0.12 against 3.9) that one
    # bf16 step of the stored output is 13 % of it, which the update-relative error
    # cannot tell from a wrong result.
    need_gpu()
    cfg = ragged_cfg(synth.DIT, dtype, d=d, H=H)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say(f"dit ragged dtype={dtype} d={d}")
    check_block(cfg, W)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("B", [9, 16, 27, 32])
def test_dit_block_batch_groups(dtype, B):
    # the modulation GEMV takes samples in groups of 8 (one weight read for all groups on
    # MFMA, one launch per group in fp32): full, ragged and the largest batch
    need_gpu()
    cfg = ragged_cfg(synth.DIT, dtype, d=64, H=3, B=B, lat=(4, 1, 8, 10))
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say(f"dit batch groups dtype={dtype} B={B}")
    check_block(cfg, W)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("kind", [synth.MMDIT_DOUBLE, synth.MMDIT_SINGLE])
def test_mmdit_blocks_ragged(dtype, kind):
    need_gpu()
    cfg = ragged_cfg(kind, dtype, d=64, H=3, n_txt=13, lat=(4, 1, 18, 22))
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.2), kind)
    say(f"mmdit ragged kind={kind} dtype={dtype}")
    check_block(cfg, W, seed=kind)


def test_tiny_shape_block_fp32():
    need_gpu()
    cfg = synth.get_config("tiny", kinds=[synth.DIT])
    W = synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1)
    say("tiny block")
    check_block(cfg, W)


def test_dit_xl2_block_full_shape():
    need_gpu()
    cfg = synth.get_config("dit_xl2", kinds=[synth.DIT])
    W = synth.make_layer_weights(cfg, 0, bias_std=0.02)
    say("dit_xl2 full block B=8 N=256 C=1152 d=72")
    check_block(cfg, W)


SAMPLE_ROWS = {
    "flux": [0, 1, 511, 512, 513, 2000, 4095, 4607],
    "qwen": [0, 255, 256, 257, 3000, 4351],
    "hunyuan": [0, 255, 256, 300, 7000, 14309, 14565],
}


@pytest.mark.parametrize("name,kind", [("flux", synth.MMDIT_SINGLE), ("flux", synth.MMDIT_DOUBLE),
                                       ("qwen", synth.MMDIT_DOUBLE), ("hunyuan", synth.MMDIT_DOUBLE)])
def test_mmdit_block_full_shape_sampled_rows(name, kind):
    need_gpu()
    cfg = synth.get_config(name, kinds=[kind])
    W = synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1)
    say(f"{name} full block kind={kind} N={cfg['n_img'] + cfg['n_txt']} (sampled rows)")
    check_block(cfg, W, rows=np.array(SAMPLE_ROWS[name]))


def test_dit_block_gemm_tile_paths():
    """A DiT block with K = 2080, half a stage past the 64 grid: qkv takes 256x256 tiles, fc1
    256x192, proj 128x192, fc2 (K = 8320) 128x96; attention with head dim 104."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=104, H=20, B=2, lat=(4, 1, 64, 64), mlp_ratio=4)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say("dit block C=2080 d=104 N=1024 B=2 (sampled rows)")
    check_block(cfg, W, rows=np.array([0, 1, 255, 256, 511, 700, 1022, 1023]))


def test_dit_block_ragged_wide_tiles():
    """A DiT block with 2000 token rows (ragged against both the 256- and 128-row tiles):
    fc1 (N = 4608) takes 256x192 tiles, qkv 256x128, proj and fc2 128x96."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=72, H=16, B=4, lat=(4, 1, 50, 40), mlp_ratio=4)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say("dit block C=1152 d=72 N=500 B=4 (sampled rows)")
    check_block(cfg, W, rows=np.array([0, 1, 127, 128, 255, 256, 420, 450, 498, 499]))


def test_dit_block_c2048_tiles():
    """A DiT block with C = 2048 (16 heads of 128) and 2048 rows: qkv takes 256x192 and fc1
    256x256 tiles, proj and fc2 (N = 2048, 256 tiles) one 128x128 tile per CU; attention with
    head dim 128."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=128, H=16, B=2, lat=(4, 1, 64, 64), mlp_ratio=4)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say("dit block C=2048 d=128 N=1024 B=2 (sampled rows)")
    check_block(cfg, W, rows=np.array([0, 1, 127, 128, 511, 777, 1023]))



def test_dit_block_attention_wide_ragged():
    """Head dim 128 with 32 queries per wave (4 query blocks of 256 x 16 heads x 4 samples =
    256 workgroups): 1000 tokens per sample, so the last query block holds 232 queries and
    the last 64-key tile 40 keys."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=128, H=16, B=4, lat=(4, 1, 50, 80), mlp_ratio=4)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say("dit block C=2048 d=128 N=1000 B=4 (sampled rows)")
    check_block(cfg, W, rows=np.array([0, 1, 255, 256, 511, 767, 768, 959, 960, 998, 999]))


def test_dit_block_narrow_tiles():
    """A DiT block with 510 token rows (two samples of 255 tokens; the last 128-row tile
    holds 126): qkv takes 128x64 tiles, fc1 128x96, proj and fc2 64x64."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=72, H=16, B=2, lat=(4, 1, 30, 34), mlp_ratio=4)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    say("dit block C=1152 d=72 N=255 B=2")
    check_block(cfg, W)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("kind", [synth.MMDIT_DOUBLE, synth.MMDIT_SINGLE])
def test_mmdit_blocks_rope(dtype, kind):
    """Rotary embedding of q and k (3-axis ids: text rows 0, image rows (frame, row,
    column)) on a two-frame latent with ragged text and image rows."""
    need_gpu()
    cfg = ragged_cfg(kind, dtype, d=64, H=3, n_txt=13, lat=(4, 2, 18, 22))
    cfg["rope_axes"], cfg["rope_theta"] = (16, 24, 24), 10000.0
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.2), kind)
    say(f"mmdit rope kind={kind} dtype={dtype}")
    check_block(cfg, W, seed=kind)


@pytest.mark.parametrize("kind", [synth.MMDIT_SINGLE, synth.MMDIT_DOUBLE])
def test_flux_block_rope_full_shape_sampled_rows(kind):
    need_gpu()
    cfg = synth.get_config("flux", kinds=[kind])
    cfg["rope_axes"], cfg["rope_theta"] = (16, 56, 56), 10000.0
    W = synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1)
    say(f"flux rope full block kind={kind} (sampled rows)")
    check_block(cfg, W, rows=np.array(SAMPLE_ROWS["flux"]))


@pytest.mark.parametrize("kind,H,B,lat,n_txt", [c[:5] for c in gemm_plan.OFF_64])
def test_block_gemm_tiles_off_the_64_grid(kind, H, B, lat, n_txt):
    """K not a multiple of 64: a partial last stage in the 256-row tiles (large grids) and the smaller
    ones, row and column tails, rows through a row map."""
    need_gpu()
    cfg = ragged_cfg(kind, synth.BF16, d=8, H=H, n_txt=n_txt, B=B, lat=lat)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), kind)
    check_block(cfg, W, seed=H)


@pytest.mark.parametrize("kind,H,B,lat,n_txt,ratio", [c[:6] for c in gemm_plan.LARGE])
def test_block_gemm_large_pairs_off_the_64_grid(kind, H, B, lat, n_txt, ratio):
    """Both streams of a double block, or both parts of a single block's first projection, in one launch
    of 256- and 128-row tiles, with a partial last K stage and tiles across samples."""
    need_gpu()
    cfg = ragged_cfg(kind, synth.BF16, d=8, H=H, n_txt=n_txt, B=B, lat=lat, mlp_ratio=ratio)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), kind)
    n = cfg["n_img"] + n_txt
    check_block(cfg, W, seed=H, rows=np.array([r for r in (0, n_txt - 1, n_txt, 127, 128, 200, 255, 256, 300, n - 100, n - 2, n - 1) if r < n]))


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("kind,d,H,axes", [
    (synth.MMDIT_DOUBLE, 24, 7, None),            # 3 or 6 lanes a head
    (synth.MMDIT_DOUBLE, 40, 13, None),           # 5 or 10 lanes, a last group with 2 of its 12 heads
    (synth.MMDIT_SINGLE, 96, 3, (16, 40, 40)),    # 12 or 24 lanes, rotated
    (synth.MMDIT_DOUBLE, 128, 5, (16, 56, 56)),   # 16 or 32 lanes, rotated; 10 heads in groups of 4 or 2
    # one or two lanes a head.  (C = 264: at C = 8, one head, the update is about 0.015 at most, and
    # the rounding of h alone, 2^-24 of |h| <= 4, is 1.6e-5 of it in fp32.)
    (synth.MMDIT_SINGLE, 8, 33, (4, 2, 2)),
])
def test_block_qk_norm_head_dims(dtype, kind, d, H, axes):
    """q/k norm and rotation for head dims whose lanes do and do not divide a wavefront."""
    need_gpu()
    cfg = ragged_cfg(kind, dtype, d=d, H=H, n_txt=13, lat=(4, 2, 14, 10))
    if axes:
        cfg["rope_axes"], cfg["rope_theta"] = axes, 10000.0
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.2), kind)
    check_block(cfg, W, seed=d)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("kind,d,H,axes", [
    (synth.MMDIT_DOUBLE, 40, 37, (8, 16, 16)),    # 7 or 13 groups of heads a row
    (synth.MMDIT_SINGLE, 64, 24, (16, 24, 24)),   # 6 or 12
    (synth.MMDIT_DOUBLE, 128, 12, (16, 56, 56)),  # 6 or 12
])
def test_block_qk_norm_rotated_rows_walked(dtype, kind, d, H, axes):
    """Rotated q and k with enough rows that a wavefront walks the groups of a row (1440 image
    rows: three wavefronts a row), several groups' loads at a time and, in fp32, a second turn."""
    need_gpu()
    cfg = ragged_cfg(kind, dtype, d=d, H=H, n_txt=13, lat=(4, 2, 40, 36), mlp_ratio=1)
    cfg["rope_axes"], cfg["rope_theta"] = axes, 10000.0
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.2), kind)
    check_block(cfg, W, seed=d, rows=np.array([0, 12, 13, 14, 31, 200, 372, 373, 500, 731, 732]))


@pytest.mark.parametrize("kind,H,B,lat,n_txt", [c[:5] for c in gemm_plan.SPLIT_K])
def test_block_gemm_tiles_split_k(kind, H, B, lat, n_txt):
    """The GEMM tiles whose waves split K, small grids: row, column and K tails, the fewest
    stages of a tile, grouped problems."""
    need_gpu()
    cfg = ragged_cfg(kind, synth.BF16, d=8, H=H, n_txt=n_txt, B=B, lat=lat)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), kind)
    check_block(cfg, W, seed=H)


@pytest.mark.parametrize("d,H,B,lat", [
    (16, 12, 2, (4, 1, 2, 4)),      # 2 keys
    (48, 4, 1, (4, 1, 18, 14)),     # 63 keys: one tile, one short
    (56, 4, 1, (4, 1, 16, 16)),     # 64 keys: exactly one tile
    (64, 3, 1, (4, 1, 26, 10)),     # 65 keys: one key in the second tile
    (80, 3, 2, (4, 1, 24, 22)),     # 132 keys, query blocks of 128 and 4
    (88, 3, 1, (4, 1, 40, 26)),     # 260 keys
    (104, 3, 1, (4, 1, 36, 34)),    # 306 keys, padded 128-wide tiles
    (128, 2, 1, (4, 1, 50, 62)),    # 775 keys
    (128, 8, 24, (4, 1, 18, 30)),   # 135 keys over 192 heads: 32 queries per wave
    (72, 8, 24, (4, 1, 34, 30)),    # 255 keys over 192 heads: 32 queries per wave
    (96, 8, 24, (4, 1, 34, 30)),    # the same at the 96-wide tiles
    (88, 8, 24, (4, 1, 18, 30)),    # and padded to them, 135 keys
])
def test_block_attention_tiles(d, H, B, lat):
    """Attention at the edges of its 64-key tiles and query blocks, for every head-dim class."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, synth.BF16, d=d, H=H, B=B, lat=lat, mlp_ratio=1)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    check_block(cfg, W, seed=d)


@pytest.mark.parametrize("d,H,B", [(64, 4, 1), (128, 3, 1), (128, 8, 24)])
def test_block_attention_raised_maximum(d, H, B):
    """Gains of 3.3 on the normalised q and k spread the scores over some +-40 (log2 units 58),
    so that the running maximum is raised in later key tiles.  bf16 q and k (2^-9 relative
    per element, independent) move a score of standard deviation 11 by about 0.02, and a
    probability by 2 %; the update sums many of them."""
    need_gpu()
    cfg = ragged_cfg(synth.MMDIT_SINGLE, synth.BF16, d=d, H=H, n_txt=9, B=B, lat=(4, 1, 32, 36) if H < 9 else (4, 1, 18, 30),
                     mlp_ratio=1)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.MMDIT_SINGLE)
    W["q_g"] = W["q_g"] * np.float32(3.3)
    W["k_g"] = synth.to_bf16_values(W["k_g"] * np.float32(3.3))
    W["q_g"] = synth.to_bf16_values(W["q_g"])
    check_block(cfg, W, seed=d + 1)


@pytest.mark.parametrize("kind,H,d,B,lat,n_txt", [
    (synth.DIT, 41, 8, 2, (4, 1, 40, 50), 0),            # 64x64 GEMM tiles, K tail of 8; two query tiles per workgroup
    (synth.DIT, 5, 72, 1, (4, 1, 38, 26), 0),            # 32x32 tiles, K = 360 / 720 off the 64-wide stage
    (synth.DIT, 3, 40, 1, (4, 1, 2, 2), 0),              # one token: 16x16 tiles, K = 120
    (synth.MMDIT_DOUBLE, 2, 128, 2, (4, 1, 18, 22), 33),  # rows through a row map, 132 keys
    (synth.MMDIT_SINGLE, 3, 96, 1, (4, 1, 16, 16), 1),   # 65 keys
])
def test_block_fp32_tiles(kind, H, d, B, lat, n_txt):
    """fp32 blocks over the GEMM tile classes and attention key blocks, with tails."""
    need_gpu()
    cfg = ragged_cfg(kind, synth.F32, d=d, H=H, n_txt=n_txt, B=B, lat=lat)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), kind)
    check_block(cfg, W, seed=H)


@pytest.mark.parametrize("kind,H,B,lat,n_txt,ratio", [c[:6] for c in gemm_plan.SHORT_K])
def test_block_gemm_short_k(kind, H, B, lat, n_txt, ratio):
    """GEMMs of one to four K stages: a part of a stage, fewer stages than buffers, the register-staged
    kernel on large grids, pairs."""
    need_gpu()
    cfg = ragged_cfg(kind, synth.BF16, d=8, H=H, n_txt=n_txt, B=B, lat=lat, mlp_ratio=ratio)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), kind)
    grown(W, cfg)
    n = cfg["n_img"] + n_txt
    rows = np.array(sorted({0, 1, n_txt, n_txt + 1, 14, 63, 64, 127, 128, 255, 256, n // 2, n - 2, n - 1} & set(range(n))))
    check_block(cfg, W, seed=H, rows=rows)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("d,H,B,lat,row", [
    (64, 3, 2, (4, 1, 18, 30), 0),      # 135 keys: the first tile
    (72, 4, 2, (4, 1, 26, 24), 155),    # 156 keys: the last key, in a tile with 28
    (128, 2, 2, (4, 1, 18, 30), 70),    # a tile in the middle
    (72, 14, 8, (4, 1, 40, 30), 299),   # 32 queries per wave in bf16
])
def test_block_attention_nan_key(dtype, d, H, B, lat, row):
    """A NaN in one row of sample 0 makes its key NaN, so every row of that sample's output is NaN; the other
    samples keep their bits."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, dtype, d=d, H=H, B=B, lat=lat, mlp_ratio=1)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.DIT)
    bf = dtype == synth.BF16
    u = synth.normal((B, cfg["n_img"], cfg["C"]), 17, bf16=bf)
    c = synth.normal((B, cfg["C"]), 18)
    clean = run_block(cfg, W, u, c)
    u[0, row, 5] = np.nan
    got = run_block(cfg, W, u, c)
    assert np.isnan(got[0]).all()
    assert np.array_equal(got[1:], clean[1:])


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("d,H,lat,live", [
    (64, 3, (4, 1, 40, 20), slice(150, 200)),    # 200 keys: two tiles without a finite score before the first
    (64, 3, (4, 1, 40, 20), slice(3, 4)),        # one key, in the first tile
    (128, 2, (4, 1, 40, 20), slice(199, 200)),   # the last key alone
    (72, 4, (4, 1, 16, 16), slice(0, 64)),       # all of one tile
    (40, 3, (4, 1, 24, 22), slice(64, 128)),     # a tile between two without
])
def test_block_attention_scores_below_the_range(dtype, d, H, lat, live):
    """Scores of -1e40 (-inf in fp32) but for the keys `live`, whose scores are 0: probabilities of exactly 0
    and 1 / n, also while no key tile has had a finite score.  q is 1e20 in each head's first dim, k is
    1e20 times the normalised first channel, which is 0 in the live rows and negative in the others (their
    first two channels cancel, so that the row mean is 0 without rounding)."""
    need_gpu()
    cfg = ragged_cfg(synth.DIT, dtype, d=d, H=H, B=1, lat=lat, mlp_ratio=1)
    C, n, bf = cfg["C"], cfg["n_img"], dtype == synth.BF16
    fix = synth.to_bf16_values if bf else (lambda a: a)
    W = synth.make_layer_weights(cfg, 0, bias_std=0.02)
    W["mod_w"] = np.zeros_like(W["mod_w"])
    W["mod_b"] = np.zeros_like(W["mod_b"])
    W["mod_b"][2 * C:3 * C] = W["mod_b"][5 * C:] = 1   # gates 1, no shift, no scale
    big = float(fix(np.array([1e20], np.float32))[0])
    W["qkv_w"][:2 * C] = 0
    W["qkv_b"][:2 * C] = 0
    W["qkv_b"][:C:d] = big
    W["qkv_w"][C:2 * C:d, 0] = big
    # the rounding of h, up to 2^-7 for 2 <= |h| < 4 in bf16, is 6 % of the update without these factors
    W["qkv_w"][2 * C:] *= 8
    W["o_w"] = W["o_w"] * 8
    half = np.random.default_rng(3).integers(-24, 25, size=(1, n, C // 2)).astype(np.float32) / 8   # exact sums
    u = np.stack([half, -half], -1).reshape(1, n, C)
    u[0, :, 0], u[0, :, 1] = -2, 2
    u[0, live, 0] = u[0, live, 1] = 0
    c = synth.normal((1, C), 19)
    got = run_block(cfg, W, u, c)
    ref = O.block(synth.DIT, u.astype(np.float64), O.silu(c.astype(np.float64)), W, cfg)
    err = O.max_rel_err(got - u, (O.round_bf16(ref) if bf else ref) - u)
    say(f"  d={d} live={live}: err(h-u)={err:.3e}")
    assert np.isfinite(got).all() and err <= TOL[dtype], err


@pytest.mark.parametrize("n_txt", [1, 8])
def test_block_rows_beyond_32_bit_offsets(n_txt):
    """fc2 of the text stream, whose samples lie 5409 and more rows of 12 288 elements apart: 256 rows span
    more than 4 GB.  One text row a sample leaves no tile (the register-staged kernel), eight the 128x64 that
    the image stream takes too."""
    need_gpu()
    cfg = ragged_cfg(synth.MMDIT_DOUBLE, synth.BF16, d=8, H=8, n_txt=n_txt, B=32, lat=(4, 1, 32, 676), mlp_ratio=192)
    W = boosted(synth.make_layer_weights(cfg, 0, bias_std=0.02, gain_std=0.1), synth.MMDIT_DOUBLE)
    grown(W, cfg)
    check_block(cfg, W, seed=n_txt, rows=np.array([0, n_txt - 1, n_txt, 255, 3000, 5407 + n_txt]))
