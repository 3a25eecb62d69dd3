"""The tile a product is computed in, as the library's host code states it (no GPU)."""
import os
import subprocess
import sys

import pytest

from paper_2505_05856_amd import binding as B
from test_ops_gpu import GEMM_TILES, GEMM_TILES_192, LINEAR_BWD


@pytest.mark.parametrize("tile,mode,M,N,ks", GEMM_TILES)
def test_the_gpu_tests_reach_every_tile_ragged(tile, mode, M, N, ks):
    assert M % tile[0] and N % tile[1] and all(k % 64 for k in ks)
    for k in ks:
        assert B.op_gemm_tile(mode, M, N, k) == tile


@pytest.mark.parametrize("tile,mode,M,N,ks", GEMM_TILES_192)
def test_the_gpu_tests_reach_every_192_tile_ragged(tile, mode, M, N, ks):
    test_the_gpu_tests_reach_every_tile_ragged(tile, mode, M, N, ks)


# 192 rows or columns for at most four rounds of 256 tiles
@pytest.mark.parametrize("tile,mode,M,N,K", [((256, 192), 0, 4096, 4800, 1600), ((256, 192), 1, 6144, 6144, 2048), ((256, 192), 1, 11648, 4200, 1208),
                                             ((256, 256), 0, 5828, 12576, 840), ((256, 256), 0, 12143, 5960, 1256),
                                             ((256, 256), 1, 6016, 14232, 1608), ((256, 256), 0, 8989, 8112, 2280)])
def test_where_tiles_of_192_end(tile, mode, M, N, K):
    assert B.op_gemm_tile(mode, M, N, K) == tile


def test_the_gpu_tests_reach_every_tile_of_a_linear_backward_ragged():
    for T, n_in, n_out, nt, tn in LINEAR_BWD:
        assert B.op_linear_bwd_tiles(T, n_in, n_out) == (nt, tn)
        assert T % nt[0] and n_in % nt[1] and n_in % tn[0] and n_out % tn[1] and T % 64 and n_out % 64
    tiles = {(256, 256), (256, 192), (192, 256), (256, 128), (128, 256), (128, 128), (128, 64), (64, 128), (64, 64)}
    assert {c[3] for c in LINEAR_BWD} == tiles == {c[4] for c in LINEAR_BWD}
    for T, n_in, n_out in ((127, 128, 128), (128, 120, 128), (0, 128, 128), (200, 200, 132)):   # two launches
        assert B.op_linear_bwd_tiles(T, n_in, n_out) == ((0, 0), (0, 0))


# Workgroups are dealt in turn to 32 groups of 8 CUs; a tile choice that takes the 256 CUs for one group was longer than two launches
# here (us, two launches / that choice / these tiles): 135 / 158 / 126, 33 / 34 / 24, 192 / 209 / 177, 376 / 396 / 374
@pytest.mark.parametrize("T,n_in,n_out,nt,tn", [(2874, 2688, 5376, (256, 128), (256, 256)), (323, 1408, 4224, (64, 64), (256, 256)),
                                                (2471, 2432, 9728, (256, 128), (256, 256)), (10112, 2688, 5376, (256, 256), (256, 256))])
def test_tiles_of_a_linear_backward_fit_the_groups_of_cus(T, n_in, n_out, nt, tn):
    assert B.op_linear_bwd_tiles(T, n_in, n_out) == (nt, tn)


# two launches / the best pair, us: 291 / 305, 177 / 181
@pytest.mark.parametrize("T,n_in,n_out", [(6296, 2496, 7488), (6016, 1472, 5888)])
def test_two_launches_where_they_end_sooner(T, n_in, n_out):
    assert B.op_linear_bwd_tiles(T, n_in, n_out) == ((0, 0), (0, 0))


# the tuning aid names the tile of every product that can run in it: the three whose rings are filled first need three k-steps
@pytest.mark.parametrize("asked,tiles", [("128x128", [(128, 128)] * 3), ("192x192", [(192, 192)] * 3),
                                         ("256x192", [None, None, (256, 192)]), ("256x256", [None, None, (256, 256)])])
def test_the_tile_asked_for_is_taken_where_it_runs(asked, tiles):
    code = "from paper_2505_05856_amd import binding as B; print([B.op_gemm_tile(0, 4096, 1024, k) for k in (64, 128, 192)])"
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, DPSTAGE_GEMM_TILE=asked), cwd=root, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    own = [B.op_gemm_tile(0, 4096, 1024, k) for k in (64, 128, 192)]
    assert eval(out.stdout) == [t or o for t, o in zip(tiles, own)]


def test_other_kernels_products_have_no_tile():
    for mode, m, n, k in ((0, 128, 128, 63), (0, 127, 128, 64), (0, 128, 130, 64), (0, 128, 128, 68), (1, 132, 128, 64),
                          (0, 0, 128, 64)):
        assert B.op_gemm_tile(mode, m, n, k) == (0, 0)
    with pytest.raises(B.DpError):
        B.op_gemm_tile(2, 128, 128, 64)
