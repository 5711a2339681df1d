"""The heads.  The action head on both sides of the width from which a wave keeps eight loads in flight, with widths that end inside a
step of 256 columns, and with every split of the action rows over workgroups: the logits are the oracle's, and a row has
the same bits whatever batch it is in.  The value head on both sides of its rule for the rows of a wave."""
import numpy as np
import pytest

import workloads as W
from tests import parity as P
from tests.test_gpu_parity import _value_case, ragged_obs, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("heads,bins", [(1, 17), (15, 256), (16, 40), (17, 256), (17, 1000)])
def test_head_widths_and_splits(heads, bins):
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(1, 128 * heads, heads, 128, 128, 1100, n_action_bins=bins, dtype="bf16")
    weights = W.make_weights(shape, 5)
    batch = 300
    wl = W.Workload("Hd", 91, shape, batch=batch, n_patches=2, instr_len=(0, 0), n_tokens=1)
    obs = ragged_obs(wl, [2] * batch, [0] * batch, seed=4)
    run_both(wl, obs=obs, rows=[0, 1, 150, 299])
    got = {}
    for n in (1, 4, 33, 70, 300):
        pol = VlaPolicy(shape, n, 4, 2 * n)
        pol.load_weights(weights)
        dev = P.device_inputs(pol, obs)
        got[n] = pol.prefill(dev["patch_emb"][:2 * n].contiguous(), obs["cu_patch"][:n + 1], dev["instr_ids"],
                             obs["cu_instr"][:n + 1]).cpu().numpy()
        pol.close()
    for n in got:
        assert np.array_equal(got[n], got[300][:n]), n


@pytest.mark.timeout(300)
@pytest.mark.parametrize("batch", [3, 56, 57])               # 7 groups of 8 rows x 32: four rows of W1 a wave; 8: sixteen
def test_value_head_rows_per_wave(batch):
    shape = W.PolicyShape(1, 2048, 16, 128, 128, 700, dtype="bf16")
    wl = W.Workload("Vh", 93, shape, batch=batch, n_patches=2, instr_len=(0, 0), n_tokens=2)
    _value_case(wl, ragged_obs(wl, [2] * batch, [0] * batch, seed=8), None, n_steps=5, tol=2e-3)
