"""Decode steps of a few rows, whose products take the norm and the residual add with them: a sequence has the same bits in
batches on both sides of every rule of theirs (16 rows; 32 of a narrow model, 33) and those bits are the oracle's.  The widths
give slices of an odd number of k-blocks, of fewer than are kept in flight, and rows of more spans than a lane requests at once,
and with d_ffn above 2048 slices of the down product that take more than one round of every depth at 17 rows and more.  4160
is so long that from 17 rows on the two-term layer's down product is apart while the single-term ones stay inside (3 layers: the
route changes from one to the other and back with a norm behind it)."""
import numpy as np
import pytest

import workloads as W
from oracle import vla_oracle as O
from tests import parity as P
from tests.test_gpu_parity import ragged_obs

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("d,f,hd,two_layers", [(256, 192, 64, 1), (768, 2048, 64, 0), (896, 704, 128, 2), (1152, 1600, 64, 1),
                                               (4224, 512, 64, 1), (256, 2112, 64, 1), (768, 4160, 64, 1)])
def test_a_sequence_has_the_same_bits_in_every_batch(d, f, hd, two_layers):
    from paper_2603_18464_amd import VlaPolicy
    shape = W.PolicyShape(3 if f > 2048 else 2, d, d // hd, hd, f, 700, n_action_bins=64, dtype="bf16")
    weights = W.make_weights(shape, 5)
    K, lengths = 3, [37, 5, 64, 20]                       # the prefixes repeat, so row b is sequence b % 4 of every batch
    base = ragged_obs(W.Workload("Df", 94, shape, batch=4, n_patches=64, instr_len=(0, 0), n_tokens=K), lengths, [0] * 4, seed=17)
    pes, ids = P.split_obs(base, range(4))
    ref = None
    for B in (4, 1, 15, 16, 17, 31, 32, 33):
        patch = np.concatenate([pes[b % 4] for b in range(B)])
        cu = np.concatenate([[0], np.cumsum([lengths[b % 4] for b in range(B)])]).astype(np.int32)
        pol = VlaPolicy(shape, B, 64 + K, 2200, two_term_layers=two_layers)   # (capacity: the last layer always in compact rows)
        pol.load_weights(weights)
        dev = P.device_inputs(pol, {**base, "patch_emb": patch, "cu_patch": cu})
        out = pol.policy_step(dev["patch_emb"], cu, dev["instr_ids"], np.zeros(B + 1, np.int32), K, want_logits=True)
        got, tokens = out["logits"].cpu().numpy(), out["tokens"].cpu().numpy()
        pol.close()
        assert np.isfinite(got).all(), B
        if ref is None:
            ref = got
            ora = O.OraclePolicy(shape, weights).policy_step(pes, ids, K, mode="cached", forced_tokens=tokens)
            wl = W.Workload("Df", 94, shape, batch=4, n_patches=64, instr_len=(0, 0), n_tokens=K)
            assert np.abs(ref - ora["logits"]).max() <= P.tolerances(wl, False)["logit"]
        for b in range(B):
            assert np.array_equal(got[b], ref[b % 4]), f"batch {B}, row {b}"
