"""The residual products of a few hundred rows (gemm_few_kernel): a sequence has the bits that the tiled kernel gives it in a
larger batch, alone and at the edges of every height of the tiles, with and without a workgroup that reads the weights ahead,
with and without low terms.  That the shapes reach all of it is asked of the library on the CPU."""
import pytest

from paper_2603_18464_amd.binding import vla_gemm_tile_rows, vla_gemm_variant
from tests import test_gemm_variants as V

# (d_model, d_ffn, head_dim, rows): 33 rows alone and in batches; 385 and more take the tiled kernel
CASES = [(512, 2816, 64, [34, 48, 64, 65, 384, 385]), (768, 2048, 64, [47, 290, 1300]),
         (3072, 64, 128, [49, 97, 128, 165, 192, 230, 290, 384, 400]), (4096, 64, 128, [289, 290, 320, 384, 700])]
HEIGHTS = {f"{rows}x64" for rows in range(32, 129, 16)}


def test_the_cases_reach_every_height():
    for two in (False, True):
        reached = {vla_gemm_variant(m, n, k, two, 32) for d, f, hd, rows in CASES for m in [33] + rows for n, k in ((d, d), (d, f))}
        assert HEIGHTS <= reached


def test_which_products_take_the_small_tiles():
    few = {(m, n, k, two, span): vla_gemm_variant(m, n, k, two, span) in HEIGHTS
           for m in (1, 33, 384, 385, 2000) for n in (384, 512, 768, 4096, 8192, 16384, 32768) for k in (64, 128, 192, 768, 896, 4096, 32768)
           for two in (False, True) for span in (32, 64, 128)}
    for (m, n, k, two, span), is_few in few.items():
        if is_few:                                        # residual adds of whole slabs, no wider than their contraction
            assert span == 32 and m <= 384 and 512 <= n <= k and k % (256 if two else 128) == 0
            assert vla_gemm_variant(m, n, k, two, span) == f"{vla_gemm_tile_rows(m, n, k, two, span)}x64"
        elif span == 32 and m <= 384 and 512 <= n <= min(k, 4096) and k % 256 == 0:
            raise AssertionError((m, n, k, two))
    assert few[384, 8192, 32768, False, 32] is False      # more tiles than the chip has compute units


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
