"""Proxy projections on images whose pixel count is not a multiple of 8 (requests at element alignment, last pixels taken
twice), with the k-steps of a tile shared by the waves of a workgroup or not, and the weight gradient in tiles of 32 x 32 or 16 x
16, its rows through LDS or not: against the fp64 oracle, and bit-for-bit copies with a selection matrix."""
import numpy as np
import pytest

from gpu_util import TOL, rel_inf_err
from oracle import gspn_oracle as O
from paper_2512_07884_amd import workloads as WL
from test_gpu_proxy import run_project, run_project_bwd

pytestmark = pytest.mark.gpu

# N = 9, 15, 63, 127, 129, 255, 257, 7020; K in whole and half 16-value steps, fewer steps than waves, ragged row tiles; the
# larger ones have enough tiles for a wave per tile (forward) and for rows through LDS (weight gradient)
SHAPES = [(1, 64, 40, 3, 3), (2, 96, 8, 3, 5), (2, 96, 8, 7, 9), (1, 72, 33, 1, 127), (3, 40, 70, 3, 43), (1, 1152, 144, 5, 51),
          (1, 144, 1152, 1, 257), (1, 96, 24, 90, 78), (9, 200, 130, 11, 13), (64, 24, 96, 33, 31), (2, 8, 96, 17, 19), (2, 96, 24, 23, 23), (1, 40, 33, 16, 40)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_projection_and_gradients(shape, dtype):
    B, K, M, H, W = shape
    rng = np.random.default_rng([29, K, M, H])
    x = WL.to_storage(rng.standard_normal((B, K, H, W)), dtype)
    P = WL.to_storage(rng.standard_normal((M, K)) / np.sqrt(K), dtype)
    g = WL.to_storage(rng.standard_normal((B, M, H, W)), dtype)
    xf, Pf, gf = (WL.storage_to_f64(a, dtype) for a in (x, P, g))
    assert rel_inf_err(run_project(x, P, dtype), O.proxy_project(xf, Pf)) <= TOL[dtype]
    gin_ref, gP_ref = O.proxy_project_bwd(gf, xf, Pf)
    gin, gP = run_project_bwd(g, x, P, dtype)
    assert rel_inf_err(gin, gin_ref) <= TOL[dtype], rel_inf_err(gin, gin_ref)
    assert rel_inf_err(gP, gP_ref) <= 1e-5, rel_inf_err(gP, gP_ref)       # accumulated and returned in fp32
    gin2, gP2 = run_project_bwd(g, x, P, dtype)
    assert np.array_equal(gin, gin2) and np.array_equal(gP, gP2)


# Whole rows at the lines of the dispatch: k-steps shared by the waves up to 448 waves from 16 steps on and up to 768 from 48;
# buffer requests for P^T, for steps of 8 and from 1024 waves on (either side of each)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(14, 256, 1024, 3, 8), (15, 256, 1024, 3, 8), (3, 240, 40, 5, 8), (24, 768, 1024, 1, 8), (25, 768, 1024, 1, 8),
                                   (31, 48, 1024, 1, 8), (32, 48, 1024, 1, 8), (5, 136, 40, 9, 8), (2, 1024, 24, 16, 33)],
                         ids=lambda s: "x".join(map(str, s)))
def test_whole_rows_at_the_lines_of_the_dispatch(shape, dtype):
    test_projection_and_gradients(shape, dtype)


# The weight gradient at the lines of its dispatch: 16 x 16 tiles from 4096 pixels on (1024 where rows start anywhere), 32 x 32
# tiles, their rows through LDS, with ragged rows and columns in one turn of workgroups and in several, the same just short of 2048
# pixels, whole rows of half a 16-pixel step
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 56, 40, 64, 64), (1, 56, 40, 64, 63), (1, 56, 40, 25, 41), (1, 56, 40, 31, 33), (9, 104, 232, 8, 256),
                                   (9, 104, 232, 8, 255), (9, 104, 232, 7, 293), (18, 72, 232, 16, 129), (2, 40, 24, 3, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_weight_gradient_at_the_lines_of_the_dispatch(shape, dtype):
    test_projection_and_gradients(shape, dtype)


# ... the rows through LDS: from 2048 pixels on, from 1024 with 64 tiles, from 512 with 256, a single tile on one side from 4096 (1024
# where rows start anywhere); either side of each, one piece, one pixel and all but one beyond a stage of 128
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 72, 40, 8, 256), (1, 72, 40, 1, 2047), (1, 72, 40, 1, 2049), (1, 104, 72, 23, 93), (1, 264, 232, 8, 128), (1, 264, 200, 8, 128),
                                   (1, 232, 264, 3, 343), (2, 488, 264, 8, 64), (2, 488, 264, 8, 63), (2, 488, 264, 3, 171), (2, 264, 488, 8, 71),
                                   (1, 96, 24, 64, 64), (1, 24, 96, 9, 113), (1, 96, 24, 31, 33), (2, 96, 24, 9, 127)],
                         ids=lambda s: "x".join(map(str, s)))
def test_weight_gradient_through_lds(shape, dtype):
    test_projection_and_gradients(shape, dtype)


# pairs of row tiles, the last pair with 8 rows: whole rows and rows at any element, k-steps of 16 and 8, the matrix and (outputs and
# contraction exchanged) its transpose
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 256, 136, 8, 832), (1, 264, 136, 60, 111), (1, 136, 256, 60, 111), (1, 136, 264, 8, 832)], ids=lambda s: "x".join(map(str, s)))
def test_pairs_of_row_tiles(shape, dtype):
    test_projection_and_gradients(shape, dtype)


@pytest.mark.parametrize("K,H,W", [(64, 16, 24), (1152, 16, 24), (64, 13, 7), (72, 11, 13), (1152, 5, 29)])
def test_selection_matrix_copies(K, H, W):
    rng = np.random.default_rng(31)
    B, M = 2, 40
    x = WL.to_storage(rng.standard_normal((B, K, H, W)), "bf16")
    pick = rng.permutation(K)[:M]
    P = np.zeros((M, K))
    P[np.arange(M), pick] = 1.0
    got = run_project(x, WL.to_storage(P, "bf16"), "bf16")
    assert np.array_equal(got, WL.storage_to_f64(x, "bf16")[:, pick])
