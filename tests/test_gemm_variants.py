"""Every variant of the prefill GEMM (tile, ring depth, epilogue, with and without low terms) that the choice of tile
reaches: a sequence has the same bits at the front, in the middle and at the end of every batch as alone, and alone it is
the oracle's.  That the shapes do reach all of them is asked of the library on the CPU, so that a change of the cost
model cannot quietly take a variant out of the test."""
import numpy as np
import pytest

import workloads as W
from oracle import vla_oracle as O
from paper_2603_18464_amd.binding import vla_gemm_first_rows, vla_gemm_tile_rows, vla_gemm_variant
from tests import parity as P
from tests.test_gpu_parity import ragged_obs

ALL = {"64x128 8 waves", "64x128 6 stages", "64x128 3 stages", "128x128", "64x256", "128x256", "160x256", "192x256", "224x256",
       "256x256", "256x256 spread"}
SPAN = {"resid": 32, "gate/up": 64, "qkv64": 64, "qkv128": 128}
# Not reached: of the forms of a launch of few 64x128 tiles each epilogue has one; three stages need more than 256 of these
# tiles to be the fastest choice, which takes a wide matrix of a short contraction (gate/up only); 8-bit low terms have one
# form of 256x256 and the residual add another (with low terms it has both: those of a d_ffn that is an odd multiple of 64 are
# halves).
REACHED = {(two, epi): ALL - {"64x128 8 waves" if epi == "qkv128" else "64x128 6 stages"}
           - ({"64x128 3 stages"} if epi != "gate/up" else set())
           - ({"256x256"} if epi == "resid" and not two else set())
           - ({"256x256 spread"} if two and epi != "resid" else set())
           for two in (False, True) for epi in SPAN}
# A single-term product that requests its weights together has a matrix of 100 MB or so.  Here for heads of 64; the 7B workloads
# run the other two (gate/up of any 256-row tiles, heads of 128 from 17 000 rows on).
BY_7B = [("gate/up", 64 * 290, 22016), ("qkv128", 256 * 290, 12288)]
for epi, _, _ in BY_7B:
    REACHED[False, epi] -= {"256x256"}

# (d_model, d_ffn, head_dim, rows): three layers, the first two-term, the last one partly on the rows of the head only
CASES = [(128, 192, 64, [64, 6000]), (768, 64, 128, [2881, 4100, 6000]), (768, 64, 64, [2881, 4100, 6000]),
         (128, 2048, 128, [1100, 2300]), (512, 2048, 64, [3500]), (1536, 64, 128, [8000]), (128, 16448, 64, [64]),
         (1024, 64, 64, [1300]), (2048, 704, 128, [8000]), (512, 4096, 128, [6000]), (1280, 2816, 128, [700]),
         (3072, 64, 128, [400, 1300]), (1280, 64, 64, [1088]), (2048, 64, 64, [8000]), (5632, 64, 64, [4500])]
# (in test_gpu_gemm_balanced.py)
BALANCED = [(768, 1024, 64, [5200]), (1280, 1024, 64, [8000]), (768, 64, 128, [7000])]


def parts(rows, n, k, two, span):
    """Rows of each launch of a product."""
    first = vla_gemm_first_rows(rows, n, k, two, span)
    return [first, rows - first] if first else [rows]


def launches(d, f, hd, rows):
    for two in (False, True):
        for epi, n, k in ((f"qkv{hd}", 3 * d, d), ("resid", d, d), ("gate/up", 2 * f, d), ("resid", d, f)):
            for m in parts(rows, n, k, two, SPAN[epi]):
                yield (two, epi), vla_gemm_variant(m, n, k, two, SPAN[epi])


def test_the_cases_reach_every_variant():
    reached = {key: set() for key in REACHED}
    for d, f, hd, rows_list in CASES + BALANCED:
        for rows in rows_list:
            for key, variant in launches(d, f, hd, rows):
                if not variant.split()[0].endswith("x64"):    # (test_gpu_gemm_few.py has the few-row tiles)
                    reached[key].add(variant)
    assert reached == REACHED
    for epi, rows, n in BY_7B:
        assert vla_gemm_variant(rows, n, 4096, False, SPAN[epi]) == "256x256"
    assert vla_gemm_variant(64, 100, 128, False, 32) == vla_gemm_variant(64, 128, 128, False, 1) == ""


def test_the_variant_is_what_the_launch_runs():
    """Where the rounds are balanced the launch runs other tiles than the cost model picks: the name is that of the launch.  Where
    a product takes two launches each has one."""
    for rows, n, k, span, want in ((2320, 22016, 4096, 64, "224x256"), (2208, 22016, 4096, 64, "160x256"), (290, 22016, 4096, 64, "160x256"),
                                   (4100, 12288, 4096, 128, "160x256"), (10533, 22016, 4096, 64, "256x256"),
                                   (2320, 4096, 4096, 32, "160x256")):
        assert vla_gemm_variant(rows, n, k, False, span) == want, (rows, n, k)
    for rows, n, k, span, want in ((18560, 4096, 11008, 32, [(16384, "256x256 spread"), (2176, "160x256")]),
                                   (9280, 4096, 4096, 32, [(6144, "192x256"), (3136, "224x256")])):
        assert [(m, vla_gemm_variant(m, n, k, False, span)) for m in parts(rows, n, k, False, span)] == want, (rows, n, k)
    for n, k, span in ((12288, 4096, 128), (22016, 4096, 64), (4096, 11008, 32), (2304, 768, 64), (768, 2048, 32)):
        for rows in range(1, 30000, 173):
            for two in (False, True):
                for m in parts(rows, n, k, two, span):
                    assert 0 < m <= rows and vla_gemm_variant(m, n, k, two, span).startswith(f"{vla_gemm_tile_rows(m, n, k, two, span)}x")
    assert vla_gemm_tile_rows(300, 512, 768, False, 32) == 32           # of an epilogue that the few-row kernel has, and of one
    assert vla_gemm_tile_rows(300, 512, 768, False, 64) == 64           # that it does not have
    assert vla_gemm_first_rows(18560, 4000, 4096, False, 32) == vla_gemm_first_rows(0, 4096, 4096, False, 32) == 0
    assert vla_gemm_first_rows(18560, 4096, 4096, False, 1) == 0


def test_when_weights_are_requested_goes_by_the_bytes_that_are_read_again():
    """The same tile, spread where weights and half of the activations stay below 170 MB: whatever the epilogue."""
    for span in (64, 128):
        for rows, n, k, together in ((9280, 12288, 4096, False), (18560, 12288, 4096, True), (18560, 22016, 4096, True),
                                     (2560, 22016, 4096, True), (18560, 11008, 2048, False), (18560, 16384, 3072, False),
                                     (18560, 49152, 2048, True), (9280, 18432, 6144, True)):
            want = "256x256" if together else "256x256 spread"
            assert vla_gemm_variant(rows, n, k, False, span) == want, (rows, n, k)


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,rows_list", CASES)
def test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, rows_list):
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(3, d, d // hd, hd, f, 700, dtype="bf16")
    weights = W.make_weights(shape, 5)
    own = 33                                                  # rows of the sequence that is compared: no multiple of a tile
    alone = None
    for rows in [own] + rows_list:
        rest = rows - own if rows < 3 * own else rows - 3 * own
        nps = [own] + [120] * (rest // 120) + ([rest % 120] if rest % 120 else [])
        where = [0]
        if rows >= 3 * own:
            nps = nps[:len(nps) // 2 + 1] + [own] + nps[len(nps) // 2 + 1:] + [own]
            where += [i for i in range(1, len(nps)) if i == len(nps) - 1 or (nps[i] == own and i not in where)]
        assert sum(nps) == rows
        wl = W.Workload("Gv", 92, shape, batch=len(nps), n_patches=120, instr_len=(0, 0), n_tokens=1)
        obs = ragged_obs(wl, nps, [0] * len(nps), seed=15)
        cu = obs["cu_patch"]
        for i in where:
            obs["patch_emb"][cu[i]:cu[i + 1]] = obs["patch_emb"][:own]
        pol = VlaPolicy(shape, len(nps), 122, 8192, two_term_layers=1)   # (capacity: the last layer always in compact rows)
        pol.load_weights(weights)
        dev = P.device_inputs(pol, obs)
        got = pol.prefill(dev["patch_emb"], cu, dev["instr_ids"], obs["cu_instr"]).cpu().numpy()
        pol.close()
        assert np.isfinite(got).all(), rows
        if alone is None:
            alone, first = got[0], obs["patch_emb"][:own].copy()
            pes, ids = P.split_obs(obs, [0])
            ora = O.OraclePolicy(shape, weights).policy_step(pes, ids, 1, mode="cached")
            assert np.abs(alone - ora["logits"][0, 0]).max() <= P.tolerances(wl, False)["logit"]
        assert np.array_equal(obs["patch_emb"][:own], first)   # (the generator draws the sequences in order)
        for i in where:
            assert np.array_equal(got[i], alone), f"{rows} rows, sequence {i}"
