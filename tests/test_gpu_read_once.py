"""Decode steps whose keys and values outgrow the last-level cache read them as data that does not come again: the sequences
that a batch on either side of that rule shares have the same bits."""
import numpy as np
import pytest

import workloads as W
from tests import parity as P
from tests.test_gpu_parity import ragged_obs

pytestmark = pytest.mark.gpu
KEEP = 245_000_000                                         # bytes of weights, keys and values


@pytest.mark.timeout(300)
@pytest.mark.parametrize("hd,fast,batches", [(128, False, (36, 42)), (64, False, (36, 42)), (128, True, (56, 62)), (64, True, (56, 62))])
def test_the_same_bits_on_both_sides(hd, fast, batches):
    from paper_2603_18464_amd import VlaPolicy
    d, layers, long = 256, 2, 2000
    shape = W.PolicyShape(layers, d, d // hd, hd, 192, 700, n_action_bins=40, dtype="bf16")
    weights = W.make_weights(shape, 5)
    got = []
    for B in batches:                                      # ragged ends first: one row of a group, all of it, one more
        nps = [long - 31 + b for b in range(20)] + [long] * (B - 20)
        wl = W.Workload("Ro", 97, shape, batch=B, n_patches=long, instr_len=(0, 0), n_tokens=3)
        obs = ragged_obs(wl, nps, [0] * B, seed=21)        # (the generator draws the sequences in order)
        pol = VlaPolicy(shape, B, long + 4, sum(nps), precision=1 if fast else 0)
        pol.load_weights(weights)
        dev = P.device_inputs(pol, obs)
        out = pol.policy_step(dev["patch_emb"], obs["cu_patch"], dev["instr_ids"], obs["cu_instr"], 3, want_logits=True)
        got.append(out["logits"].cpu().numpy())
        pol.close()
        kv = sum(nps) * d * layers * (4 if fast else 6)
        assert (2 * layers * d * (4 * d + 3 * 192) + kv > KEEP) == (B == batches[1])
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0], got[1][:batches[0]])
