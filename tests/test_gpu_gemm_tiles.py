"""The prefill GEMMs choose their tile by the number of rows: at row counts on both sides of the tiles' edges a sequence
gets the same bits whatever its batch (one chain of matrix instructions over ascending k per element), and those bits are
the oracle's within the tolerance of the 16-bit path.  (test_gemm_variants.py reaches every variant of the kernel.)"""
import numpy as np
import pytest

import workloads as W
from oracle import vla_oracle as O
from tests import parity as P
from tests.test_gpu_parity import ragged_obs

pytestmark = pytest.mark.gpu

# one prefix of 63 rows is filled up to: the edges of the 64-, 128- and 256-row tiles, and enough rows that the cost
# model moves on to each larger tile (the wide matrices of this shape: 3072 and 5632 columns)
ROWS = [63, 64, 65, 127, 128, 129, 255, 257, 700, 1500, 4100]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("hd,ffn,fast", [(128, 2816, False), (128, 2816, True), (64, 1472, False), (64, 704, True)])
def test_rows_do_not_depend_on_the_tile(hd, ffn, fast):
    from paper_2603_18464_amd import VlaPolicy
    # 1472 and 704: gate/up widths that are multiples of 128 only, contractions that are odd multiples of 64
    shape = W.PolicyShape(2, 1024, 1024 // hd, hd, ffn, 700, dtype="bf16")
    weights = W.make_weights(shape, 5)
    first, ref = 63, None
    for rows in ROWS:
        rest = rows - first
        nps = [first - 5] + [120] * (rest // 120) + ([rest % 120] if rest % 120 else [])
        lens = [5] + [0] * (len(nps) - 1)
        wl = W.Workload("Gt", 77, shape, batch=len(nps), n_patches=120, instr_len=(0, 5), n_tokens=1)
        obs = ragged_obs(wl, nps, lens, seed=11)
        obs["instr_ids"][:] = [3, 99, 5, 400, 17]             # (the generator draws them behind the patches)
        pol = VlaPolicy(shape, len(nps), 130, rows, precision=1 if fast else 0, two_term_layers=1)
        pol.load_weights(weights)
        dev = P.device_inputs(pol, obs)
        got = pol.prefill(dev["patch_emb"], obs["cu_patch"], dev["instr_ids"], obs["cu_instr"]).cpu().numpy()
        pol.close()
        assert np.isfinite(got).all(), rows
        if ref is None:
            ref = got[0]
            pes, ids = P.split_obs(obs, [0])
            ora = O.OraclePolicy(shape, weights).policy_step(pes, ids, 1, mode="cached")
            assert np.abs(ref - ora["logits"][0, 0]).max() <= P.tolerances(wl, fast)["logit"]
        assert np.array_equal(got[0], ref), f"{rows} rows"


@pytest.mark.timeout(300)
@pytest.mark.parametrize("rows", [2881, 2945, 3072])     # 16 row tiles of 192: one row, a ragged half and all of the last
def test_192_row_tile(rows):
    """4096 gate/up columns of a short contraction fill the chip once with tiles of 192 rows."""
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(2, 256, 2, 128, 2048, 700, dtype="bf16")
    weights = W.make_weights(shape, 5)
    nps = [120] * (rows // 120) + ([rows % 120] if rows % 120 else [])
    wl = W.Workload("Gt2", 78, shape, batch=len(nps), n_patches=120, instr_len=(0, 0), n_tokens=1)
    obs = ragged_obs(wl, nps, [0] * len(nps), seed=12)
    pol = VlaPolicy(shape, len(nps), 130, rows, two_term_layers=1)
    pol.load_weights(weights)
    dev = P.device_inputs(pol, obs)
    got = pol.prefill(dev["patch_emb"], obs["cu_patch"], dev["instr_ids"], obs["cu_instr"]).cpu().numpy()
    pol.close()
    check = [0, len(nps) // 2, len(nps) - 2, len(nps) - 1]
    pes, ids = P.split_obs(obs, check)
    ora = O.OraclePolicy(shape, weights).policy_step(pes, ids, 1, mode="cached")
    assert np.abs(got[check] - ora["logits"][:, 0]).max() <= P.tolerances(wl, False)["logit"]


@pytest.mark.timeout(300)
def test_operand_beyond_4_gib():
    """The activations of the down projection span more than 2^32 bytes (88 200 rows of 49 152): row offsets inside a tile
    are 32-bit, everything above a tile is not.  The first and the last sequences have the bits of a small batch."""
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(2, 128, 2, 64, 16384, 700, dtype="bf16")
    weights = W.make_weights(shape, 5)
    n, L = 700, 126
    wl = W.Workload("Gt3", 79, shape, batch=n, n_patches=L, instr_len=(0, 0), n_tokens=1)
    obs = ragged_obs(wl, [L] * n, [0] * n, seed=13)

    def prefill(seqs):
        rows = np.concatenate([np.arange(b * L, (b + 1) * L) for b in seqs])
        pol = VlaPolicy(shape, len(seqs), L + 2, len(rows), two_term_layers=1)
        pol.load_weights(weights)
        pe = pol.to_device(np.ascontiguousarray(obs["patch_emb"][rows]))
        cu = (np.arange(len(seqs) + 1) * L).astype(np.int32)
        ids = P.device_inputs(pol, obs)["instr_ids"]
        got = pol.prefill(pe, cu, ids, np.zeros(len(seqs) + 1, np.int32)).cpu().numpy()
        pol.close()
        return got

    assert n * L * shape.d_ffn * 3 > 2 ** 32
    few = [0, 1, n - 2, n - 1]
    small = prefill(few)
    assert np.isfinite(small).all()
    assert np.array_equal(prefill(list(range(n)))[few], small)
