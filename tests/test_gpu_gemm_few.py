"""The residual products of a few hundred rows (gemm_few_kernel): a sequence has the bits that the tiled kernel gives it in a
larger batch, alone and at the edges of every height of the tiles, with and without workgroups that read the weights ahead, with
and without low terms, with every remainder of the slab loops.  That the shapes reach all of it is asked of the library on the CPU."""
import pytest

from paper_2603_18464_amd.binding import vla_gemm_tile_rows, vla_gemm_variant
from tests import test_gemm_variants as V

# (d_model, d_ffn, head_dim, rows): 33 rows alone and in batches, the last of which takes the tiled kernel
CASES = [(512, 2816, 64, [34, 48, 64, 65, 385, 900, 1224, 1225]), (768, 2048, 64, [47, 290, 700, 1065, 1066]),
         (3072, 64, 128, [49, 97, 128, 165, 192, 230, 290, 384, 490, 491]), (4096, 64, 128, [289, 290, 320, 384, 700]),
         (640, 1280, 64, [384, 1200]), (896, 1024, 64, [386, 1100])]
# heights without a workgroup that reads ahead, where the last tile has sixteen rows at most
BRIEF = [(2048, 64, 128, [337, 700]), (2560, 64, 64, [321, 600]), (2816, 64, 128, [321, 560]), (3328, 64, 128, [337, 500]),
         (4352, 64, 128, [257, 400])]
HEIGHTS = {f"{rows}x64" for rows in range(32, 129, 16)}
FORMS = HEIGHTS | {name + " ahead" for name in HEIGHTS}


def test_the_cases_reach_every_form():
    reached, left = set(), set()
    for d, f, hd, rows in CASES + BRIEF:
        for m in [33] + rows:
            for n, k in ((d, d), (d, f)):
                for two in (False, True):
                    variant = vla_gemm_variant(m, n, k, two, 32)
                    reached.add((two, variant))
                    if variant in FORMS:
                        left.add((two, k // (256 if two else 128) % 4))      # slabs behind the loops of four
    assert {(two, form) for two in (False, True) for form in FORMS} <= reached
    assert left == {(two, r) for two in (False, True) for r in range(4)}


def takes(m, n, k, two):
    return 512 <= n <= k and k % (256 if two else 128) == 0 and m * (n + 1200) <= 2 ** 21


def test_which_products_take_the_small_tiles():
    few = {(m, n, k, two, span): vla_gemm_variant(m, n, k, two, span)
           for m in (1, 33, 384, 385, 480, 640, 900, 1065, 1066, 2000) for n in (384, 512, 768, 1024, 2048, 4096, 8192, 16384, 32768)
           for k in (64, 128, 192, 768, 896, 4096, 32768) for two in (False, True) for span in (32, 64, 128)}
    for (m, n, k, two, span), name in few.items():
        if name in FORMS:                                 # residual adds of whole slabs, no wider than their contraction
            assert span == 32 and takes(m, n, k, two)
            assert name.startswith(f"{vla_gemm_tile_rows(m, n, k, two, span)}x64")
        elif span == 32 and takes(m, n, k, two) and n <= 4096:
            raise AssertionError((m, n, k, two))
    assert few[1065, 768, 768, False, 32] in FORMS and few[1066, 768, 768, False, 32] not in FORMS
    assert few[384, 8192, 32768, False, 32] not in FORMS  # more tiles than the chip has compute units


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES + BRIEF)
def test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
