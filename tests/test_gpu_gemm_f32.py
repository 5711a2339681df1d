"""The float32 path's GEMM against the fp64 oracle where its tiles can go wrong: widths that leave a ragged last column tile
or rows that are not 16-byte aligned (odd d_ffn), K shorter than the four waves' shares, every rotary pair layout, row
counts on both sides of the 16- and 32-row tiles."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import ragged_obs, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,hd,f,batch,n_patches", [
    (1, 32, 1, 1, 1),          # one k-step for four waves, one column of a tile, one row
    (2, 32, 37, 3, 5),         # odd K: element-wise loads
    (1, 64, 70, 2, 16),        # K a multiple of 2 only
    (4, 64, 704, 17, 3),       # decode rows one past a 16-row tile
    (1, 256, 52, 5, 9),        # the widest head
    (3, 128, 1408, 9, 120),    # enough tiles for the 32-row form, ragged rows
    (3, 128, 1411, 9, 120),    # the same with odd K
])
def test_float32_tiles(heads, hd, f, batch, n_patches):
    shape = W.PolicyShape(2, heads * hd, heads, hd, f, 300, n_action_bins=40, dtype="f32")
    wl = W.Workload("F32", 77, shape, batch=batch, n_patches=n_patches, instr_len=(0, 7), n_tokens=3)
    rng = np.random.default_rng(batch)
    nps, lens = rng.integers(1, n_patches + 1, size=batch), rng.integers(0, 8, size=batch)
    if n_patches >= 100:
        nps[:] = n_patches     # more than 1024 tiles of 16 rows: 9 x 120 rows x (3 * 384 / 32) columns
    run_both(wl, obs=ragged_obs(wl, list(nps), list(lens), seed=3))
