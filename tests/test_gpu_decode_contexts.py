"""Decode attention against the fp64 oracle with contexts on both sides of the rows a workgroup requests at once (256 and, with
low terms, 192 of them for heads of 64; 128 and 96 for heads of 128), of twice and three times as many, and of one instruction's
rows: the new row, which comes from on-chip memory, is then the first, the last or the only one of a group."""
import pytest

import workloads as W
from tests.test_gpu_parity import ragged_obs, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fast", [False, True])
@pytest.mark.parametrize("hd,one", [(64, 64), (128, 32)])
def test_decode_contexts(hd, one, fast):
    nps = sorted({1, 2} | {g * one + e for g in (1, 3, 4, 6, 8, 9) for e in (-3, -2, -1, 0, 1)})
    shape = W.PolicyShape(2, 256, 256 // hd, hd, 192, 700, n_action_bins=40, dtype="bf16")
    wl = W.Workload("Dc", 96, shape, batch=len(nps), n_patches=max(nps), instr_len=(0, 0), n_tokens=4)
    run_both(wl, obs=ragged_obs(wl, nps, [0] * len(nps), seed=hd), fast=fast)
