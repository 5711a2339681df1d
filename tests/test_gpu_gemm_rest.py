"""Products whose last round goes into a launch of its own, with lower tiles (first_rows): a sequence has the same bits at the
front, in the middle and at the end of such a batch, which lies in the second launch, as alone."""
import pytest

from tests import test_gemm_variants as V

pytestmark = pytest.mark.gpu

# (d_model, d_ffn, head_dim, rows): gate/up 3072 + 545 rows; QKV of both head sizes 4352 + 1278 and 3808 + 1855
CASES = [(768, 8192, 64, [3617]), (2560, 64, 128, [5630, 5663]), (2560, 64, 64, [5630])]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_both_launches(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
