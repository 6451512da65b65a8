"""The precompute's prefix tree (csrc/fgram_tree.h): f-grams that share prefixes,
in one chunk and in several, sorted by ranks or by radix passes.

The oracle computes every f-gram on its own; the bound is that of
test_gpu_fgram_model.py.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_2502_01637_amd as S
from oracle import fgram_model as orc
from workloads.fgram_model import ModelConfig, make_params, make_token_rows, bf16_bits_to_f64
from gpu_util import dev
from test_gpu_fgram_model import as_f64, assert_close, bf16_dev, random_fgrams, run

# (n, vocabulary, K): one f-gram; prefixes that nearly all share, duplicates
# among them; rank sorts with key values of one, two and three bytes; radix sorts:
# one prefix group over several chunks; many chunks
CASES = [(1, 5, 7), (3000, 2, 7), (8192, 300, 5), (8193, 300, 5), (9000, 255, 3),
         (9000, 256, 6), (9000, 65535, 3), (9000, 65536, 3), (9000, 70000, 4),
         (150_000, 1, 2), (70_001, 30, 4), (120_000, 3000, 3)]


def pytest_id(c):
    return "n%d_V%d_K%d" % c


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=pytest_id)
def test_shared_prefixes(case):
    n, V, K = case
    cfg = ModelConfig(512, 8, 128, 1, K)
    rng = np.random.default_rng(n + V + K)
    P = make_params(cfg, seed=1)
    T = make_token_rows(V, cfg.d, seed=2)
    fg, lengths = random_fgrams(rng, V, n, K)
    fg[lengths == K, 0] = V - 1                      # a large group with one first token
    ids = rng.permutation(n).astype(np.int32)
    got = run(cfg, fg, lengths, ids, T, P, n)
    # the ends of the sorted order and of the input, and a random sample
    order = np.lexsort(fg.T[::-1])
    pick = np.unique(np.concatenate([order[:20], order[-20:], order[n // 2:n // 2 + 20],
                                     [0, n - 1], rng.integers(0, n, 100)]))
    ref = orc.forward(fg[pick], lengths[pick], bf16_bits_to_f64(T),
                      {k: bf16_bits_to_f64(v) for k, v in P.items()}, 1, 8)
    assert_close(as_f64(got[torch.from_numpy(ids[pick].astype(np.int64)).cuda()]), ref, 1)
    # the same bits as in a call of their own (another sort, other neighbours)
    alone = run(cfg, fg[pick], lengths[pick], np.arange(len(pick), dtype=np.int32), T, P,
                len(pick))
    assert torch.equal(alone.view(torch.int16),
                       got[torch.from_numpy(ids[pick].astype(np.int64)).cuda()].view(torch.int16))



# n * n = 1e8 per radix pass is the most that ranks are counted for: one, four
# (two bytes of a key of two tokens) and eighteen passes; then radix passes over
# the largest and smallest key values of one, two and three bytes.
@pytest.mark.gpu
@pytest.mark.parametrize("case", [(10_000, 200, 2), (10_001, 200, 2), (20_000, 300, 3),
                                  (20_001, 300, 3), (42_426, 65_536, 7), (42_427, 65_536, 7),
                                  (14_143, 255, 3), (20_001, 256, 3), (20_001, 65_535, 3),
                                  (24_495, 65_536, 3)], ids=pytest_id)
def test_both_sorts_at_their_line(case):
    test_shared_prefixes(case)


# Fewer than 256 f-grams are sorted and linked by one workgroup.
@pytest.mark.gpu
@pytest.mark.parametrize("case", [(1, 5, 2), (2, 1, 2), (3, 2, 3), (64, 3, 4), (65, 300, 5),
                                  (254, 70_000, 6), (255, 2, 7), (256, 2, 7)], ids=pytest_id)
def test_short_lists(case):
    test_shared_prefixes(case)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 255, 256])
def test_errors_of_short_lists(n):
    cfg = ModelConfig(512, 8, 128, 1, 3)
    rng = np.random.default_rng(n)
    P, T = make_params(cfg, seed=1), make_token_rows(50, cfg.d, seed=2)
    model = S.FgramModel(P, cfg.d, cfg.n_heads, cfg.d_ff, 1, 3)
    for what, code in [("length", S.scone.ELEN), ("token", S.scone.ETOKEN), ("row", S.scone.EROW)]:
        fg, lengths = random_fgrams(rng, 50, n, 3)
        ids = np.arange(n, dtype=np.int32)
        if what == "length":
            lengths[-1], fg[0, 0] = 1, 50          # the length comes first
        elif what == "token":
            fg[-1, 1] = -1
        else:
            ids[0] = n
        rows = torch.zeros((n, cfg.d), dtype=torch.bfloat16, device="cuda")
        with pytest.raises(S.SconeError) as e:
            S.precompute_fgram_rows(model, dev(fg), dev(lengths), dev(ids), bf16_dev(T), rows)
        assert e.value.code == code
        assert what != "length" or not rows.any()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 9000, 70_001])
def test_no_layers(n):
    """Rows of a model with no layers: LNf(T + P) of the last token alone, in one
    chunk and in several; a bad length writes nothing."""
    K, V = 5, 65_535
    cfg = ModelConfig(512, 8, 128, 0, K)
    rng = np.random.default_rng(n)
    P, T = make_params(cfg, seed=1), make_token_rows(V, cfg.d, seed=2)
    fg, lengths = random_fgrams(rng, V, n, K)
    fg[:, 0] = 7
    ids = rng.permutation(n).astype(np.int32)
    got = run(cfg, fg, lengths, ids, T, P, n)
    pick = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 300)]))
    ref = orc.forward(fg[pick], lengths[pick], bf16_bits_to_f64(T),
                      {k: bf16_bits_to_f64(v) for k, v in P.items()}, 0, 8)
    assert_close(as_f64(got[torch.from_numpy(ids[pick].astype(np.int64)).cuda()]), ref, 0)
    assert (got.float().abs().sum(1) > 0).all()
    lengths[n // 2] = K + 1
    model = S.FgramModel(P, cfg.d, cfg.n_heads, cfg.d_ff, 0, K)
    rows = torch.zeros((n, cfg.d), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(S.SconeError) as e:
        S.precompute_fgram_rows(model, dev(fg), dev(lengths), dev(ids), bf16_dev(T), rows)
    assert e.value.code == S.scone.ELEN and not rows.any()


@pytest.mark.gpu
def test_workspace_argument():
    """The C call in the caller's scratch: the same rows; a short, misaligned or
    overlapping workspace is refused."""
    cfg = ModelConfig(512, 8, 256, 2, 3)
    rng = np.random.default_rng(3)
    V, n = 100, 500
    P, T = make_params(cfg, seed=5), make_token_rows(V, cfg.d, seed=6)
    fg, lengths = random_fgrams(rng, V, n, 3)
    ids = np.arange(n, dtype=np.int32)
    want = run(cfg, fg, lengths, ids, T, P, n)
    model = S.FgramModel(P, cfg.d, cfg.n_heads, cfg.d_ff, cfg.n_layers, 3)
    L = S.scone.lib()
    need = L.scone_fgram_model_workspace(n, 3, cfg.d, cfg.n_heads, cfg.d_ff)
    t = [dev(fg), dev(lengths), dev(ids), bf16_dev(T), torch.zeros_like(want),
         torch.empty(need + 512, dtype=torch.uint8, device="cuda")]
    st = torch.cuda.current_stream().cuda_stream

    def call(ws, nbytes, rows=t[4]):
        return L.scone_fgram_model_forward_in(
            t[0].data_ptr(), t[1].data_ptr(), t[2].data_ptr(), n, 3, t[3].data_ptr(), V,
            model.blob.data_ptr(), cfg.d, cfg.n_heads, cfg.d_ff, cfg.n_layers, rows.data_ptr(), n,
            ctypes.c_void_p(ws), nbytes, st)

    for ws, nbytes in [(t[5].data_ptr(), need), (None, 0)]:
        t[4].zero_()
        assert call(ws, nbytes) == S.scone.OK
        assert torch.equal(t[4].view(torch.int16), want.view(torch.int16))
    assert call(t[5].data_ptr(), need - 1) == S.scone.EINVAL
    assert call(t[5].data_ptr() + 16, need) == S.scone.EINVAL
    assert call(t[4].data_ptr(), need) == S.scone.EINVAL


def test_workspace_sizes():
    L = S.scone.lib()
    w = L.scone_fgram_model_workspace
    assert w(1000, 3, 500, 8, 512) == -1 and w(-1, 3, 512, 8, 512) == -1
    assert w(1000, 8, 512, 8, 512) == -1 and w(1 << 31, 3, 512, 8, 512) == -1
    # activations of 3,000 rows, and of a whole chunk however many f-grams follow
    assert 3000 * (12 * 512 + 2 * 512) <= w(1000, 3, 512, 8, 512) <= 3300 * (12 * 512 + 1024)
    big = w(1_000_000, 3, 1024, 16, 4096)
    assert 0 < big - 65536 * (12 * 1024 + 2 * 4096) <= 25 * 1_000_000
