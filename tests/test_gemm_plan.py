"""The host-side choice of the bf16 GEMM tiles (no GPU)."""
import gemm_plan as g


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
