"""The norm of a prefill has a form for the row count and the width (rows a workgroup, waves a row, pieces in registers): a sequence
has the same bits alone (33 rows) and in batches on both sides of every border."""
import pytest

from tests import test_gemm_variants as V

pytestmark = pytest.mark.gpu

# (d_model, d_ffn, head_dim, rows); the last has more float32 rows than the last-level cache holds (and a d_ffn whose buffer takes the
# compact rows of the last layer)
CASES = [(768, 64, 64, [1000, 1001, 3500, 3501]), (1152, 64, 64, [500, 501, 1400, 1401]),
         (4224, 64, 128, [700, 701, 1401, 3000, 3001]), (6272, 64, 128, [700, 701]), (7680, 192, 128, [8000])]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_every_form(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
