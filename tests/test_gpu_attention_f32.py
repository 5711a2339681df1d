"""float32 attention against the fp64 oracle with contexts on both sides of the keys a wave requests together (64, 48, 24 and 12
of them for heads of 32, 64, 128 and 256, in two groups), and of two and three times as many."""
import pytest

import workloads as W
from tests.test_gpu_parity import ragged_obs, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,together", [(32, 64), (64, 48), (128, 24), (256, 12)])
def test_float32_attention_contexts(hd, together):
    nps = [1, 2, together // 2 - 1, together // 2, together // 2 + 1, together - 2, together - 1, together, together + 1, 2 * together - 1, 2 * together, 3 * together + 1]
    shape = W.PolicyShape(2, 256, 256 // hd, hd, 96, 300, n_action_bins=40, dtype="f32")
    wl = W.Workload("Fa", 95, shape, batch=len(nps), n_patches=max(nps), instr_len=(0, 0), n_tokens=4)
    run_both(wl, obs=ragged_obs(wl, nps, [0] * len(nps), seed=hd))


def test_float32_attention_of_the_longest_context():
    """A cache of 4095 positions takes all of the 64 KiB of scores."""
    shape = W.PolicyShape(1, 128, 1, 128, 96, 300, n_action_bins=40, dtype="f32")
    wl = W.Workload("Fl", 97, shape, batch=1, n_patches=4091, instr_len=(0, 0), n_tokens=4)
    assert wl.max_seq == 4095
    run_both(wl)
