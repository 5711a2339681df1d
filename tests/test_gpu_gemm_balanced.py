"""Prefill GEMMs whose tiles have 160, 192, 224 or 256 rows, whichever fills the last round best: together with the shapes of
test_gemm_variants.py these reach each height with every epilogue, with and without low terms, at ragged row counts, and a
sequence has the same bits as alone (which are the oracle's)."""
import pytest

from paper_2603_18464_amd.binding import vla_gemm_tile_rows, vla_gemm_variant
from tests import test_gemm_variants as V

CASES = V.BALANCED
HEIGHTS = (160, 192, 224, 256)


def test_the_cases_reach_every_height():
    reached = set()
    for d, f, hd, rows_list in V.CASES + CASES:
        for rows in rows_list:
            for two in (False, True):
                for epi, n, k in ((f"qkv{hd}", 3 * d, d), ("resid", d, d), ("gate/up", 2 * f, d), ("resid", d, f)):
                    height = vla_gemm_tile_rows(rows, n, k, two)
                    reached.add((two, epi, height))
                    if height == 256:
                        reached.add((two, epi, vla_gemm_variant(rows, n, k, two, V.SPAN[epi])))
    assert {(two, epi, h) for two in (False, True) for epi in V.SPAN for h in HEIGHTS} <= reached
    assert {(False, epi, "256x256 spread") for epi in V.SPAN} <= reached
    assert vla_gemm_tile_rows(64, 100, 128, False) == vla_gemm_tile_rows(0, 128, 128, False) == 0


def test_the_height_needs_the_least_rounds_times_rows():
    def cost(m, n, rows):
        return -(-(-(-m // rows) * (n // 256)) // 256) * (rows + 90)

    for n, k in ((12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (2304, 768), (768, 2048)):
        for m in range(33, 40000, 271):
            for two in (False, True):
                rows, costs = vla_gemm_tile_rows(m, n, k, two), {h: cost(m, n, h) for h in HEIGHTS}
                if not vla_gemm_variant(m, n, k, two, 64).startswith(tuple(f"{h}x256" for h in HEIGHTS)):
                    assert rows < 160                     # the model's choice, 64 or 128 rows
                    continue
                assert 40 * min(costs.values()) >= 39 * costs[rows]
                if rows in (160, 224):                    # instead of 192 or 256
                    assert costs[rows] == min(costs.values()) and 40 * costs[rows] < 39 * max(costs[192], costs[256])


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list):
    V.test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list)
