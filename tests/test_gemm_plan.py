"""The host-side choice of the bf16 GEMM tiles (no GPU)."""
import random

import gemm_plan as g
import pytest
import synth


def test_stream_beyond_32_bit_offsets_leaves_the_other_its_tile():
    """A double block's fc2 with few text rows a sample: a 256-row tile of the text stream spans 31
    samples, more than the DMA's 32-bit offsets reach.  The image stream must keep the tile that
    it takes alone, and the text stream one whose rows span less."""
    B, n_txt, N, C, mlp = 32, 8, 5400, 3072, 12288
    txt = g.shape(B * n_txt, C, mlp, seg=n_txt, rows=N)
    img = g.shape(B * (N - n_txt), C, mlp, seg=N - n_txt, rows=N)
    assert g.tile(img).startswith("256x")
    assert g.tile(txt) not in ("reg", "256x256", "256x192", "256x128")
    assert not g.grouped(txt, img) or g.tile(txt, img) == g.tile(img)


def test_no_tile_for_one_problem_is_no_group():
    """Rows 256 MB apart: no tile's rows lie within a 32-bit offset."""
    far = g.shape(512, 256, 1024, lda=1 << 27)
    near = g.shape(4096, 3072, 1024)
    assert g.tile(far) == "reg" and g.tile(near) != "reg"
    assert g.tile(far, near) == "reg" and not g.grouped(far, near) and not g.grouped(near, far)
    assert g.grouped(far, far)   # neither has a tile of its own to lose


@pytest.mark.parametrize("n_txt,want", [(1, ["fc2 reg", "fc2 128x64"]), (8, ["fc2 128x64 x2"])])
def test_blocks_with_rows_beyond_32_bit_offsets(n_txt, want):
    """The tiles of the GPU test's fc2: the text stream's, then the image stream's, or both."""
    tiles = g.block_tiles(g.block_cfg(synth.MMDIT_DOUBLE, 8, 8, 32, (4, 1, 32, 676), n_txt, 192))
    assert [t for t in tiles if t.startswith("fc2")] == want


def listed(case):
    kind, H, B, lat, n_txt, ratio, tiles = case
    return g.block_tiles(g.block_cfg(kind, 8, H, B, lat, n_txt, ratio)), tiles.split(", ")


@pytest.mark.parametrize("case", g.SHORT_K + g.OFF_64 + g.SPLIT_K + g.LARGE)
def test_blocks_take_the_listed_tiles(case):
    """The GPU tests' blocks run the kernels that they are there for."""
    got, want = listed(case)
    assert got == want


@pytest.mark.parametrize("name", g.IN_WORDS)
def test_blocks_take_the_tiles_that_their_tests_state(name):
    kind, d, H, B, lat, ratio, tiles = g.IN_WORDS[name]
    assert g.block_tiles(g.block_cfg(kind, d, H, B, lat, 0, ratio)) == tiles.split(", ")


@pytest.mark.parametrize("name", g.REFRESH)
def test_history_is_refreshed_from_the_listed_tile(name):
    kind, d, H, B, lat, n_txt, ratio, last = g.REFRESH[name]
    assert g.block_tiles(g.block_cfg(kind, d, H, B, lat, n_txt, ratio))[-1] == last


def test_listed_blocks_reach_every_tile():
    """Each tile with the plain and the gated epilogue, and in one launch for two problems."""
    seen = {(t.split(" ", 1)[0] in ("proj", "fc2", "lin2"), t.split(" ", 1)[1])
            for case in g.SHORT_K + g.OFF_64 + g.SPLIT_K + g.LARGE for t in listed(case)[1]}
    for t in g.TILES:
        assert (False, t) in seen or (False, t + " x2") in seen, t
        assert (True, t) in seen or (True, t + " x2") in seen, t
        assert (False, t + " x2") in seen or (True, t + " x2") in seen, t


def test_short_k_on_a_small_grid_takes_a_small_tile():
    """Up to three stages of K: 256-row tiles only where they are not a handful on the whole card."""
    for K in range(8, 200, 8):
        for M in (1, 15, 64, 256, 512, 1024, 2048):
            for N in (8, 64, 192, 576):
                t = g.tile(g.shape(M, N, K))
                assert t.startswith("short") or (t == "reg" and M > 1024), (M, N, K, t)


def test_tiles_have_the_stages_they_need():
    """Whatever the sizes: the kernels' prologues take stages that are there, the short tiles no more than
    they have buffers for."""
    rng = random.Random(5)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    for _ in range(20000):
        K = 8 * log(1, 600)
        a = g.shape(log(1, 200000), 8 * log(1, 2000), K)
        pair = g.shape(log(1, 5000), 8 * log(1, 2000), K) if rng.random() < 0.3 else None
        t, nk = g.tile(a, pair), -(-K // 64)
        if t.startswith("short"):
            assert nk <= 3
        elif t == "reg":
            assert K <= 256
        else:
            assert nk >= (3 if t.startswith("256x") else 5 if t == "128x128" else 4), (K, t)
