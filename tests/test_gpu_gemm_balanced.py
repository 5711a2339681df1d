"""Prefill GEMMs whose tiles have 160, 192, 224 or 256 rows, whichever fills the last round best: together with the shapes of
test_gemm_variants.py these reach each height with every epilogue, with and without low terms, at ragged row counts, and a
sequence has the same bits as alone (which are the oracle's)."""
import numpy as np
import pytest

import workloads as W
from oracle import vla_oracle as O
from paper_2603_18464_amd.binding import vla_gemm_tile_rows, vla_gemm_variant
from tests import parity as P
from tests import test_gemm_variants as V
from tests.test_gpu_parity import ragged_obs

CASES = V.BALANCED
HEIGHTS = (160, 192, 224, 256)
# (d_model, d_ffn, head_dim, sequences of 33 rows): tiles of 160 and of 224 rows with every epilogue, with and without 8-bit low terms
COPIES = [(512, 1024, 64, 188), (768, 1024, 128, 128), (1280, 64, 64, 200), (512, 64, 128, 248), (1536, 64, 64, 248)]


def test_the_cases_reach_every_height():
    reached = set()
    for d, f, hd, rows_list in V.CASES + CASES:
        for rows in rows_list:
            for two in (False, True):
                for epi, n, k in ((f"qkv{hd}", 3 * d, d), ("resid", d, d), ("gate/up", 2 * f, d), ("resid", d, f)):
                    for m in V.parts(rows, n, k, two, V.SPAN[epi]):
                        height = vla_gemm_tile_rows(m, n, k, two, V.SPAN[epi])
                        reached.add((two, epi, height))
                        if height == 256:
                            reached.add((two, epi, vla_gemm_variant(m, n, k, two, V.SPAN[epi])))
    assert {(two, epi, h) for two in (False, True) for epi in V.SPAN for h in HEIGHTS} <= reached
    assert {(False, epi, "256x256 spread") for epi in V.SPAN} <= reached
    assert vla_gemm_tile_rows(64, 100, 128, False, 32) == vla_gemm_tile_rows(0, 128, 128, False, 32) == vla_gemm_tile_rows(64, 128, 128, False, 1) == 0


def test_the_height_needs_the_least_rounds_times_rows():
    def cost(m, n, rows):
        return -(-(-(-m // rows) * (n // 256)) // 256) * (rows + 90)

    for n, k in ((12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (2304, 768), (768, 2048)):
        for m in range(33, 40000, 271):
            for two in (False, True):
                rows, costs = vla_gemm_tile_rows(m, n, k, two, 64), {h: cost(m, n, h) for h in HEIGHTS}
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


def test_the_copies_reach_both_new_heights():
    reached = set()
    for d, f, hd, n in COPIES:
        for two in (False, True):
            for epi, cols, k in ((f"qkv{hd}", 3 * d, d), ("resid", d, d), ("gate/up", 2 * f, d), ("resid", d, f)):
                for m in V.parts(33 * n, cols, k, two, V.SPAN[epi]):
                    reached.add((two and k % 128 == 0, epi, vla_gemm_tile_rows(m, cols, k, two, V.SPAN[epi])))
    assert {(low8, epi, h) for low8 in (False, True) for epi in V.SPAN for h in (160, 224)} <= reached


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,n", COPIES)
def test_every_row_of_a_tile_has_the_bits_of_the_sequence_alone(d, f, hd, n):
    """A batch of copies of one sequence: each row of each tile belongs to one of them, and a wrong row of any product changes the
    keys and values that its sequence's last row, which is compared, attends to (or is that row)."""
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(3, d, d // hd, hd, f, 700, dtype="bf16")
    weights = W.make_weights(shape, 5)
    wl = W.Workload("Gc", 99, shape, batch=1, n_patches=33, instr_len=(0, 0), n_tokens=1)
    obs = ragged_obs(wl, [33], [0], seed=16)
    pol = VlaPolicy(shape, n, 35, 16384, two_term_layers=1)     # (capacity: the last layer always in compact rows)
    pol.load_weights(weights)
    got = {}
    for b in (1, n):
        dev = P.device_inputs(pol, {**obs, "patch_emb": np.concatenate([obs["patch_emb"]] * b)})
        got[b] = pol.prefill(dev["patch_emb"], 33 * np.arange(b + 1), dev["instr_ids"], np.zeros(b + 1, np.int32)).cpu().numpy()
    pol.close()
    pes, ids = P.split_obs(obs, [0])
    ora = O.OraclePolicy(shape, weights).policy_step(pes, ids, 1, mode="cached")
    assert np.abs(got[1][0] - ora["logits"][0, 0]).max() <= P.tolerances(wl, False)["logit"]
    wrong = [b for b in range(n) if not np.array_equal(got[n][b], got[1][0])]
    assert not wrong, (len(wrong), wrong[:5])
