"""The host-side choice of the bf16 GEMM tiles (csrc/gemm_plan.h, plain C++), compiled with g++ and
called from tests: which tile each GEMM of an exact block takes, and which of them share a launch."""
import ctypes
import functools
import os
import subprocess
import tempfile

import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_27842_amd", "csrc")
SRC = r"""
#include "gemm_plan.h"
static ff::GemmShape shape(const int* v) { return {v[0], v[1], v[2], v[3], v[4], v[5], v[6]}; }
extern "C" int tile(const int* a, const int* b) {
  const ff::GemmShape s[2] = {shape(a), shape(b ? b : a)};
  return ff::plan_tiles(s, b ? 2 : 1).tile;
}
static_assert(ff::kTileReg == 12, "TILES below");
extern "C" int grouped(const int* a, const int* b) { return ff::plan_grouped(shape(a), shape(b)); }
"""

# in the order of the enum; "short" tiles take up to three 64-wide K stages, "reg" is the register-staged kernel
TILES = ("256x256", "256x192", "256x128", "128x192", "128x128", "128x96", "128x64", "64x96", "64x64", "64x32",
         "short 64x64", "short 64x32", "reg")


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
        return ctypes.CDLL(so)


def shape(M, N, K, lda=None, ldw=None, seg=None, rows=None):
    """A problem: M x N over K; row r of A is row r % seg of sample r / seg, samples `rows` rows apart."""
    seg = M if seg is None else seg
    return (ctypes.c_int * 7)(M, N, K, K if lda is None else lda, K if ldw is None else ldw, seg,
                              seg if rows is None else rows)


def tile(a, b=None):
    """The tile that problem a, or a and b in one launch, take."""
    return TILES[_lib().tile(a, b)]


def grouped(a, b):
    return bool(_lib().grouped(a, b))


def block_tiles(cfg):
    """The launches of one exact block of cfg (bf16), in order: "gemm tile", or "gemm tile x2" for two
    problems in one launch."""
    kind, C, M, B, nt = cfg["kinds"][0], cfg["C"], cfg["mlp"], cfg["B"], cfg["n_txt"]
    N = cfg["n_img"] + nt
    out = []

    def put(name, probs):
        if len(probs) == 2 and grouped(*probs):
            out.append("%s %s x2" % (name, tile(*probs)))
        else:
            out.extend("%s %s" % (name, tile(p)) for p in probs)

    if kind == synth.MMDIT_SINGLE:
        put("lin1", [shape(B * N, 3 * C, C, seg=N), shape(B * N, M, C, seg=N)])
        put("lin2", [shape(B * N, C, C + M, seg=N)])
        return out
    segs = [(nt, N), (N - nt, N)] if kind == synth.MMDIT_DOUBLE and nt else [(N - nt, N)]
    for name, n, k in (("qkv", 3 * C, C), ("proj", C, C), ("fc1", M, C), ("fc2", C, M)):
        put(name, [shape(B * s, n, k, seg=s, rows=r) for s, r in segs])
    return out


def block_cfg(kind, d, H, B, lat, n_txt, ratio):
    return dict(kinds=[kind], C=H * d, mlp=ratio * H * d, B=B, n_txt=n_txt,
                n_img=lat[1] * (lat[2] // 2) * (lat[3] // 2))


# Blocks of the GPU tests with the tiles that their GEMMs take: kind, heads (of 8 dims), batch, latent, text
# rows, MLP ratio, launches
SHORT_K = [
    (synth.DIT, 2, 2, (4, 1, 26, 44), 0, 2,       # K = 16 / 32: one stage, part of it
     "qkv short 64x32, proj short 64x32, fc1 short 64x32, fc2 short 64x32"),
    (synth.DIT, 9, 8, (4, 1, 64, 64), 0, 2,       # K = 72 / 144: two and three stages
     "qkv reg, proj short 64x32, fc1 short 64x64, fc2 short 64x32"),
    (synth.DIT, 23, 8, (4, 1, 32, 60), 0, 2,      # K = 184: three stages, row tails
     "qkv short 64x64, proj short 64x32, fc1 short 64x64, fc2 64x64"),
    (synth.DIT, 31, 2, (4, 1, 64, 62), 0, 2,      # K = 248: four stages, fewer than the longest rings
     "qkv 64x96, proj 64x32, fc1 64x64, fc2 64x32"),
    (synth.DIT, 31, 16, (4, 1, 64, 62), 0, 1,     # K = 248, M = 15872
     "qkv reg, proj reg, fc1 reg, fc2 reg"),
    (synth.DIT, 21, 24, (4, 1, 44, 62), 0, 3,     # K = 168 / 504, M = 16368: three stages of 256 rows
     "qkv 256x128, proj reg, fc1 256x128, fc2 64x96"),
    (synth.MMDIT_DOUBLE, 15, 4, (4, 1, 40, 50), 13, 2,   # pairs, rows through a row map
     "qkv short 64x64 x2, proj short 64x32 x2, fc1 short 64x32 x2, fc2 64x32 x2"),
    (synth.MMDIT_DOUBLE, 23, 8, (4, 1, 64, 62), 13, 1,
     "qkv reg x2, proj short 64x64 x2, fc1 short 64x64 x2, fc2 short 64x64 x2"),
    (synth.MMDIT_SINGLE, 23, 4, (4, 1, 40, 50), 13, 2,   # bias and bias + GELU in one launch
     "lin1 short 64x64 x2, lin2 64x32"),
]
# 256-row tiles and others with a partial last K stage, row and column tails, rows through a row map
OFF_64 = [
    (synth.DIT, 33, 32, (4, 1, 28, 64), 0, 2,            # K = 264 / 528, M = 14336
     "qkv 256x256, proj 256x128, fc1 256x192, fc2 128x192"),
    (synth.DIT, 33, 20, (4, 1, 32, 64), 0, 2,            # M = 10240
     "qkv 256x192, proj 64x96, fc1 256x128, fc2 64x96"),
    (synth.DIT, 23, 3, (4, 1, 26, 44), 0, 2,             # K = 184 (three stages) / 368, M = 858
     "qkv short 64x32, proj short 64x32, fc1 short 64x32, fc2 64x32"),
    (synth.DIT, 31, 1, (4, 1, 6, 10), 0, 2,              # K = 248 / 496, M = 15: one short row tile
     "qkv 64x32, proj 64x32, fc1 64x32, fc2 64x32"),
    (synth.MMDIT_DOUBLE, 25, 3, (4, 1, 18, 22), 13, 2,   # K = 200 / 400, text rows of three samples in one tile
     "qkv 64x32 x2, proj 64x32 x2, fc1 64x32 x2, fc2 64x32 x2"),
    (synth.MMDIT_SINGLE, 35, 2, (4, 1, 20, 30), 21, 2,   # K = 280 / 840: odd and even stage counts
     "lin1 64x64 x2, lin2 64x32"),
]
# tiles whose waves split K
SPLIT_K = [
    (synth.DIT, 33, 1, (4, 1, 22, 60), 0, 2,             # M = 330, K = 264 (five stages) / 528
     "qkv 64x32, proj 64x32, fc1 64x32, fc2 64x32"),
    (synth.DIT, 49, 3, (4, 1, 40, 50), 0, 2,             # M = 1500, K = 392 / 784
     "qkv 128x64, proj 64x64, fc1 64x96, fc2 64x64"),
    (synth.DIT, 65, 3, (4, 1, 56, 50), 0, 2,             # M = 2100, K = 520 / 1040: two 64x96 per CU
     "qkv 128x128, proj 64x96, fc1 64x96, fc2 64x96"),
    (synth.DIT, 89, 2, (4, 1, 52, 100), 0, 2,            # M = 2600, K = 712 / 1424: two epilogue passes of 128x192
     "qkv 128x192, proj 128x64, fc1 128x128, fc2 128x64"),
    (synth.DIT, 144, 8, (4, 1, 32, 30), 0, 2,            # M = 1920, K = 1152 / 2304
     "qkv 256x128, proj 128x96, fc1 128x192, fc2 128x96"),
    (synth.MMDIT_DOUBLE, 49, 4, (4, 1, 18, 22), 13, 2,   # text and image rows of four samples through a row map
     "qkv 64x64 x2, proj 64x32 x2, fc1 64x32 x2, fc2 64x32 x2"),
    (synth.MMDIT_SINGLE, 41, 1, (4, 1, 20, 30), 7, 2,    # K = 328 / 984, bias and bias + GELU in one launch
     "lin1 64x32 x2, lin2 64x32"),
]
# large grids off the 64 grid: two streams in one launch, tiles across samples, gated 256-row tiles
LARGE = [
    (synth.MMDIT_DOUBLE, 185, 2, (4, 1, 74, 86), 77, 2,  # K = 1480 / 2960, 1591 + 77 rows a sample
     "qkv 256x256 x2, proj 128x192 x2, fc1 256x192 x2, fc2 128x192 x2"),
    (synth.MMDIT_DOUBLE, 185, 3, (4, 1, 38, 50), 13, 2,  # 475 + 13 rows a sample
     "qkv 256x128 x2, proj 128x96 x2, fc1 128x192 x2, fc2 128x96 x2"),
    (synth.MMDIT_DOUBLE, 65, 6, (4, 1, 50, 82), 13, 2,   # K = 520 / 1040
     "qkv 256x192 x2, proj 128x128 x2, fc1 256x128 x2, fc2 128x128 x2"),
    (synth.MMDIT_DOUBLE, 89, 2, (4, 1, 52, 100), 13, 2,  # K = 712 / 1424
     "qkv 256x128 x2, proj 64x64 x2, fc1 128x64 x2, fc2 64x64 x2"),
    (synth.MMDIT_DOUBLE, 121, 12, (4, 1, 50, 82), 13, 1,  # K = 968
     "qkv 256x256 x2, proj 256x256 x2, fc1 256x256 x2, fc2 256x256 x2"),
    (synth.MMDIT_DOUBLE, 81, 12, (4, 1, 50, 82), 13, 1,  # K = 648
     "qkv 256x256 x2, proj 256x192 x2, fc1 256x192 x2, fc2 256x192 x2"),
    (synth.MMDIT_DOUBLE, 145, 4, (4, 1, 32, 30), 13, 2,  # K = 1160 / 2320
     "qkv 128x128 x2, proj 64x96 x2, fc1 128x96 x2, fc2 64x96 x2"),
    (synth.MMDIT_SINGLE, 89, 3, (4, 1, 52, 100), 13, 2,  # K = 712 / 2136
     "lin1 256x256 x2, lin2 128x96"),
    (synth.MMDIT_SINGLE, 121, 12, (4, 1, 50, 82), 13, 1,  # K = 968 / 1936
     "lin1 256x128 x2, lin2 256x256"),
]
# blocks whose last GEMM also writes the history, all off the 64 grid but the first
REFRESH = {
    "dit_128x96": (synth.DIT, 72, 16, 8, (4, 1, 32, 30), 0, 2, "fc2 128x96"),
    "dit_128x192": (synth.DIT, 88, 3, 12, (4, 1, 50, 82), 0, 2, "fc2 128x192"),
    "dit_256x128": (synth.DIT, 88, 3, 12, (4, 1, 50, 82), 0, 1, "fc2 256x128"),
    "dit_256x192": (synth.DIT, 72, 9, 12, (4, 1, 50, 82), 0, 1, "fc2 256x192"),
    "dit_256x256": (synth.DIT, 88, 11, 12, (4, 1, 50, 82), 0, 1, "fc2 256x256"),
    "dit_register": (synth.DIT, 8, 31, 16, (4, 1, 64, 62), 0, 1, "fc2 reg"),
    "dit_short": (synth.DIT, 8, 9, 8, (4, 1, 64, 64), 0, 2, "fc2 short 64x32"),
    "double_128x192": (synth.MMDIT_DOUBLE, 88, 3, 12, (4, 1, 50, 82), 13, 2, "fc2 128x192 x2"),
    "double_256x192": (synth.MMDIT_DOUBLE, 72, 9, 12, (4, 1, 50, 82), 13, 1, "fc2 256x192 x2"),
    "double_256x256": (synth.MMDIT_DOUBLE, 88, 11, 12, (4, 1, 50, 82), 13, 1, "fc2 256x256 x2"),
    "single_128x192": (synth.MMDIT_SINGLE, 88, 3, 12, (4, 1, 50, 82), 13, 1, "lin2 128x192"),
    "single_256x192": (synth.MMDIT_SINGLE, 72, 9, 12, (4, 1, 50, 82), 13, 1, "lin2 256x192"),
    "single_256x256": (synth.MMDIT_SINGLE, 88, 11, 12, (4, 1, 50, 82), 13, 1, "lin2 256x256"),
}
# blocks whose tests say in words which tiles they take: kind, head dim, heads, batch, latent, MLP ratio, launches
IN_WORDS = {
    "test_dit_block_gemm_tile_paths": (synth.DIT, 104, 20, 2, (4, 1, 64, 64), 4,
                                       "qkv 256x256, proj 128x192, fc1 256x192, fc2 128x96"),
    "test_dit_block_ragged_wide_tiles": (synth.DIT, 72, 16, 4, (4, 1, 50, 40), 4,
                                         "qkv 256x128, proj 128x96, fc1 256x192, fc2 128x96"),
    "test_dit_block_c2048_tiles": (synth.DIT, 128, 16, 2, (4, 1, 64, 64), 4,
                                   "qkv 256x192, proj 128x128, fc1 256x256, fc2 128x128"),
    "test_dit_block_narrow_tiles": (synth.DIT, 72, 16, 2, (4, 1, 30, 34), 4,
                                    "qkv 128x64, proj 64x64, fc1 128x96, fc2 64x64"),
}
