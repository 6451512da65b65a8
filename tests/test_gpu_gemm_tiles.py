"""The residual product's tiles (256 x 256, 256 x 192, 128 x 128) at the sizes where
the choice changes and at their row remainders, against the oracle (the bound of
test_gpu_fgram_model.py) and, bit for bit, against a call small enough for
128 x 128 tiles: the order of an element's sum does not depend on the tile."""
import numpy as np
import pytest
import torch

from oracle import fgram_model as orc
from workloads.fgram_model import ModelConfig, make_params, make_token_rows, bf16_bits_to_f64
from test_gpu_fgram_model import as_f64, assert_close, bf16_dev, random_fgrams, run

pytestmark = pytest.mark.gpu


# (d, heads, d_ff, n): N = 1536 below and above the first line, at the end of one
# round of 192-wide tiles and past it; N = 512 and 1024 (no 192); the shortest sums
# (d_ff = 128, two slabs) and an odd number of slabs.
@pytest.mark.parametrize("d,heads,ff,n", [
    (1536, 12, 128, 5376), (1536, 12, 128, 5377), (1536, 12, 1152, 6913),
    (1536, 12, 384, 8192), (1536, 12, 256, 8193), (512, 8, 128, 32_700),
    (1024, 8, 640, 16_300)])
def test_tile_choice(d, heads, ff, n):
    cfg = ModelConfig(d, heads, ff, 1, 3)
    rng = np.random.default_rng(n)
    V = 700
    P = make_params(cfg, seed=5)
    T = make_token_rows(V, d, seed=6)
    fg, lengths = random_fgrams(rng, V, n, 3)
    ids = np.arange(n, dtype=np.int32)
    got = run(cfg, fg, lengths, ids, T, P, n)
    # rows of the products follow the sorted order: its ends, and tile edges
    order = np.lexsort(fg.T[::-1])
    at = [k for e in (0, 128, 256, 4096, n // 256 * 256, n) for k in range(e - 9, e + 9)]
    pick = np.unique(np.concatenate([order[[k for k in at if 0 <= k < n]],
                                     rng.integers(0, n, 60)]))
    mine = got[torch.from_numpy(pick).cuda()]
    ref = orc.forward(fg[pick], lengths[pick], bf16_bits_to_f64(T),
                      {k: bf16_bits_to_f64(v) for k, v in P.items()}, 1, heads)
    assert_close(as_f64(mine), ref, 1)
    step = 1000                       # every row, from calls of their own
    for k in range(0, n, step):
        part = slice(k, min(n, k + step))
        alone = run(cfg, fg[part], lengths[part], np.arange(part.stop - k, dtype=np.int32), T, P,
                    part.stop - k)
        assert torch.equal(alone.view(torch.int16), got[part].view(torch.int16)), k


# 256 x 256 tiles: k_gemm's for few rounds of sums up to 4,096, k_gemm_resid's
# for longer ones (8,192, and 4,224: 66 slabs) and for four rounds (24,700 rows, N = 2,048).
@pytest.mark.parametrize("d,heads,ff,n", [
    (512, 8, 4096, 32_700), (512, 8, 4224, 32_700), (1024, 16, 8192, 16_300),
    (1024, 16, 640, 16_129), (512, 4, 384, 65_000), (2048, 32, 128, 24_700)])
def test_whole_tiles_by_length_and_rounds(d, heads, ff, n):
    test_tile_choice(d, heads, ff, n)
