"""Decode steps at the edges of their kernels: batches on both sides of the 32-row blocks, the 128-row launches and the
256-row split-K chunks, and prefixes on both sides of the groups of cache rows the attention requests together."""
import pytest

import workloads as W
from tests.test_gpu_parity import ragged_obs, run_both

pytestmark = pytest.mark.gpu

PREFIX = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("batch,heads,hd,f,mode", [
    (16, 2, 128, 704, "first"), (16, 4, 64, 192, False), (32, 2, 64, 64, "first"), (33, 2, 64, 704, False),
    (64, 2, 128, 192, "first"), (65, 2, 64, 1024, True), (96, 2, 64, 192, "first"), (97, 2, 64, 192, False),
    (128, 2, 128, 704, "first"), (129, 2, 128, 704, "first"), (256, 4, 64, 1024, "first"), (257, 2, 128, 512, False)])
def test_decode_batches_and_prefixes(batch, heads, hd, f, mode):
    shape = W.PolicyShape(2, heads * hd, heads, hd, f, 400, n_action_bins=64, dtype="bf16")
    wl = W.Workload("De", 90, shape, batch=batch, n_patches=max(PREFIX), instr_len=(0, 0), n_tokens=3)
    nps = [PREFIX[(b * 5) % len(PREFIX)] for b in range(batch)]
    rows = sorted({0, 1, 2, 3, 31 % batch, 32 % batch, 63 % batch, 64 % batch, 96 % batch, 127 % batch, 128 % batch,
                   batch // 2, batch - 2, batch - 1})
    run_both(wl, obs=ragged_obs(wl, nps, [0] * batch, seed=batch), rows=rows, fast=mode)
