"""Decode steps whose keys and values outgrow the last-level cache read them as data that does not come again: the sequences
that a batch on either side of that rule shares have the same bits."""
import numpy as np
import pytest

import workloads as W
from paper_2603_18464_amd.binding import vla_decode_reads_once
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


def rows_have_the_same_bits(shape, two_layers, batches, once):
    """A decode step's rows in every batch, which are the oracle's."""
    from oracle import vla_oracle as O
    from paper_2603_18464_amd import VlaPolicy
    weights = W.make_weights(shape, 5)
    wl = W.Workload("Rw", 98, shape, batch=3, n_patches=9, instr_len=(0, 0), n_tokens=2)
    few = ragged_obs(wl, [9, 4, 7], [0] * 3, seed=22)
    pol = VlaPolicy(shape, max(batches), 16, max(batches) * 9, two_term_layers=two_layers)
    pol.load_weights(weights)
    ref = None
    for B in batches:
        reps = [b % 3 for b in range(B)]
        cu = few["cu_patch"]
        obs = {"patch_emb": np.concatenate([few["patch_emb"][cu[r]:cu[r + 1]] for r in reps]),
               "cu_patch": np.concatenate([[0], np.cumsum([cu[r + 1] - cu[r] for r in reps])]).astype(np.int32),
               "instr_ids": few["instr_ids"], "cu_instr": np.zeros(B + 1, dtype=np.int32)}
        assert vla_decode_reads_once(pol.ctx, B, int(obs["cu_patch"][-1])) == once
        dev = P.device_inputs(pol, obs)
        out = pol.policy_step(dev["patch_emb"], obs["cu_patch"], dev["instr_ids"], obs["cu_instr"], 2, want_logits=True)
        got = out["logits"].cpu().numpy()
        if ref is None:
            ref = got
            ora = O.OraclePolicy(shape, weights).policy_step(P.split_obs(few, range(3))[0], P.split_obs(few, range(3))[1], 2, mode="cached")
            assert np.abs(ref[:, 0] - ora["logits"][:, 0]).max() <= P.tolerances(wl)["logit"]
            same = out["tokens"].cpu().numpy()[:, 0] == ora["tokens"][:, 0]
            assert same.any()                              # the step behind an equal token is comparable
            assert np.abs(ref[same, 1] - ora["logits"][same, 1]).max() <= P.tolerances(wl)["logit"]
        for b in range(B):
            assert np.array_equal(got[b], ref[b % 3]), (B, b)
    pol.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("hd,d,f,two_layers", [(128, 4096, 9728, 1), (64, 4096, 9728, 4), (128, 128, 192, 1)])
def test_weights_read_once(hd, d, f, two_layers):
    """Weights that outgrow the last-level cache: a decode step's rows have the same bits in batches of every form of its
    products (normalising ones, those with planes above and below the size that takes part, one to four blocks of rows), which
    are the oracle's.  The small model reads its weights as ever."""
    shape = W.PolicyShape(2, d, d // hd, hd, f, 600, n_action_bins=40, dtype="bf16")
    assert (2 * 2 * d * (4 * d + 3 * f) > KEEP) == (d == 4096)
    rows_have_the_same_bits(shape, two_layers, (3, 17, 33, 70, 128), once=int(d == 4096))


@pytest.mark.timeout(300)
@pytest.mark.parametrize("layers,f,hd", [(14, 2048, 64), (9, 4096, 128)])
def test_weights_of_a_narrow_deep_model_read_once(layers, f, hd):
    """Up to 32 rows of a narrow model all products normalise their rows or add to the residual ones: with short slices (f 2048)
    and long ones, with and without low terms, up to 16 rows and above."""
    shape = W.PolicyShape(layers, 1024, 1024 // hd, hd, f, 600, n_action_bins=40, dtype="bf16")
    rows_have_the_same_bits(shape, 2, (3, 1, 16, 17, 24, 32, 33, 128), once=1)
