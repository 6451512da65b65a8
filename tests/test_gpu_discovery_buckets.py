"""Discovery's bucketed counting where its shapes change, against the oracle
(small corpora) and against torch.unique (corpora too large for it): one
bucket and many, chunks of every length, remainders, buckets with more codes
than one LDS table holds, one n-gram at every position."""
import ctypes
import time

import numpy as np
import pytest
import torch

from oracle import discovery
import paper_2502_01637_amd as S
from gpu_util import dev
from test_gpu_discovery import check_top_s

pytestmark = pytest.mark.gpu


def scans(X, K, min_count):
    """{(tokens): count} of every candidate, by whole-corpus torch.unique."""
    X = X.long()
    out, prev, toks = [], None, None
    for n in range(2, K + 1):
        if n == 2:
            code, ok = X[:, :-1] << 16 | X[:, 1:], torch.ones_like(X[:, 1:], dtype=torch.bool)
        else:
            p, s = prev[:, :-1], prev[:, 1:]
            code, ok = p << 16 | X[:, n - 1:], (p >= 0) & (s >= 0)
        keys, inv, count = torch.unique(code[ok], return_inverse=True, return_counts=True)
        head = (keys >> 16)[:, None] if n == 2 else toks[keys >> 16]
        rows = torch.cat([head, (keys & 0xFFFF)[:, None]], 1)
        alive = count >= min_count
        keep = torch.ones_like(alive) if n == 2 else alive
        pad = torch.full((int(keep.sum()), K - n), -1, dtype=torch.int64, device=X.device)
        out.append(torch.cat([rows[keep], pad, count[keep, None]], 1))
        dense = torch.where(alive, torch.cumsum(alive, 0) - 1, -1)
        prev = torch.full_like(code, -1)
        prev[ok] = dense[inv]
        toks = rows[alive]
    return torch.cat(out)


def ordered(rows):
    for j in reversed(range(rows.shape[1])):
        rows = rows[torch.sort(rows[:, j], stable=True)[1]]
    return rows


def check_all(X, K, min_count):
    """Every candidate, tokens and count, when S takes them all."""
    want = scans(X, K, min_count)
    assert int(want[:, :K].max()) < 65_536  # torch's own rows: wrong past 2 GiB of them
    fg, ln, ct = S.discover_fgrams(X, K, want.shape[0] + 5, min_count)
    got = torch.cat([fg, ct[:, None]], 1).long()
    assert got.shape == want.shape
    assert torch.equal(ordered(got), ordered(want))
    assert torch.equal(ln.long(), (fg >= 0).sum(1))


@pytest.mark.parametrize("BT", [1, 2, 15, 16, 255, 1023, 1024, 1025, 4096, 4097, 8193, 12289])
@pytest.mark.parametrize("T", [1, 7, 1024, None])
def test_small_corpora_match_the_oracle(BT, T):
    T = min(T or BT, BT)
    B = BT // T
    rng = np.random.default_rng(BT * 7 + T)
    X = rng.integers(0, 12, size=(B, T)).astype(np.int32)
    for K, mc in [(2, 1), (4, 2), (7, 1)]:
        cands = discovery.candidates(X, K, mc)
        for Sn in (3, 10 ** 6):
            fg, ln, ct = S.discover_fgrams(dev(X), K, Sn, mc)
            check_top_s(fg, ln, ct, cands, Sn)


# Chunk lengths of 1,024 to 8,192 and both sides of the largest bucket count.
@pytest.mark.parametrize("B,T", [(1, 524_287), (3, 349_525), (257, 4096), (1000, 4201),
                                 (33, 131_071)])
@pytest.mark.parametrize("V", [50, 65_536])
def test_chunk_lengths(B, T, V):
    g = torch.Generator(device="cuda").manual_seed(B)
    X = torch.randint(0, V, (B, T), device="cuda", generator=g, dtype=torch.int32)
    check_all(X, 3, 2 if V == 50 else 1)


def test_buckets_with_more_codes_than_a_table():
    """16.8M positions whose 2-grams are nearly all distinct: 16,384 codes per
    bucket, twice the slots, counted in four parts; all survive and so on."""
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randint(0, 65_536, (4099, 4095), device="cuda", generator=g, dtype=torch.int32)
    check_all(X, 3, 1)


@pytest.mark.parametrize("B,T", [(1, 2), (5, 1000), (700, 5000)])
def test_one_ngram_everywhere(B, T):
    X = torch.full((B, T), 65_535, device="cuda", dtype=torch.int32)
    check_all(X, 6 if T > 6 else 2, 1)


@pytest.mark.parametrize("where", [0, 1, 4999, 123_456])
def test_rejected_corpus_leaves_the_outputs(where):
    """A token out of range: an error, and the outputs as they were."""
    B, T, K, Sn = 50, 5000, 4, 1000
    g = torch.Generator(device="cuda").manual_seed(2)
    X = torch.randint(0, 900, (B, T), device="cuda", generator=g, dtype=torch.int32)
    X.view(-1)[where] = 65_536 if where % 2 else -1
    fg = torch.full((Sn, K), -77, dtype=torch.int32, device="cuda")
    ln, ct = fg[:, 0].clone(), fg[:, 0].clone()
    n = ctypes.c_int64(5)
    rc = S.scone.lib().scone_discover_fgrams(
        X.data_ptr(), B, T, K, 1, Sn, fg.data_ptr(), ln.data_ptr(), ct.data_ptr(),
        ctypes.byref(n), None, 0, torch.cuda.current_stream().cuda_stream)
    assert rc == S.scone.ETOKEN and n.value == 0
    for t in (fg, ln, ct):
        assert (t == -77).all()


# Both sides of the line where buckets are split once more, and the next number
# of sub-buckets; many and few codes per bucket, codes that fill one bucket.
@pytest.mark.parametrize("B,T", [(8192, 4096), (8193, 4096), (16_385, 4099)])
@pytest.mark.parametrize("V", [1, 50, 65_536])
def test_second_level(B, T, V):
    g = torch.Generator(device="cuda").manual_seed(B)
    X = torch.randint(0, V, (B, T), device="cuda", generator=g, dtype=torch.int32)
    K = 2 if V == 65_536 and B * T > 1 << 26 else 3   # rows of the reference below 2 GiB
    check_all(X, K, 1 if V == 65_536 else 2)


def test_cost_is_linear_in_the_corpus():
    """Nearly distinct 2-grams: 32 times the positions take about 32 times as
    long (reading buckets once per part took 170 times as long)."""
    def per_position(B):
        X = torch.randint(0, 65_536, (B, 4096), device="cuda", dtype=torch.int32,
                          generator=torch.Generator(device="cuda").manual_seed(1))
        best = float("inf")
        for _ in range(3):
            torch.cuda.synchronize()
            start = time.perf_counter()
            S.discover_fgrams(X, 2, 1000, 1)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - start)
        del X
        torch.cuda.empty_cache()
        return best / (B * 4096)

    assert per_position(131_072) < 2.5 * per_position(4096)
