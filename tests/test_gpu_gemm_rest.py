"""Products of two launches, whole rounds of tiles and the rest of them (gemm_f16_first_rows): a sequence has the same bits at the
front, in the middle and at the end of such a batch, which lies in the second launch, as alone.  That every epilogue is split, with
and without low terms, is asked of the library on the CPU."""
import pytest

from paper_2603_18464_amd.binding import vla_gemm_first_rows
from tests import test_gemm_variants as V

# (d_model, d_ffn, head_dim, rows): gate/up 4480 + 941 rows; QKV of both head sizes 4352 + 1278 and 4800 + 1763; the output
# projection 4416 + 2184
CASES = [(768, 8192, 64, [5421]), (2560, 64, 128, [5630, 6563]), (2560, 64, 64, [5630]), (5632, 704, 64, [6600])]


def test_every_epilogue_is_split():
    split = set()
    for d, f, hd, rows_list in CASES:
        for rows in rows_list:
            for two in (False, True):
                for epi, n, k in ((f"qkv{hd}", 3 * d, d), ("resid", d, d), ("gate/up", 2 * f, d), ("resid", d, f)):
                    first = vla_gemm_first_rows(rows, n, k, two, V.SPAN[epi])
                    assert first % 32 == 0 and 0 <= first < rows
                    if first:
                        split.add((two, epi))
    assert split == {(two, epi) for two in (False, True) for epi in V.SPAN}


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_both_launches(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
