"""Rows of any width and alignment through the copies that move them in 16-byte
units (gather, embed, the pipelined step, decode): edges of the units, of a workgroup's
1,024 units and of the row, unaligned tables and outputs, ids out of range."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_01637_amd as S
from gpu_util import build_gpu, dev

pytestmark = pytest.mark.gpu

V, N = 40, 60
WIDTHS = [1, 15, 16, 17, 31, 32, 33, 48, 63, 240, 1000, 1023, 1025, 1536, 2002, 3072, 3074, 4100,
          12289, 16384 + 48, 70001]


@pytest.mark.parametrize("row_bytes", WIDTHS)
@pytest.mark.parametrize("at", [(0, 0), (1, 0), (0, 2), (7, 13)])
def test_widths_and_alignments(row_bytes, at):
    rng = np.random.default_rng(row_bytes)
    pairs = rng.permutation(V * V)[:N]
    fg = np.stack([pairs // V, pairs % V], 1).astype(np.int32)
    ln = np.full(N, 2, dtype=np.int32)
    n_rows = V + N - 3                         # the last three f-grams have no row
    ids = (V + np.arange(N)).astype(np.int32)
    X = rng.integers(0, V, (3, 37)).astype(np.int32)
    o = oracle.OracleTable(fg, ln, ids)
    want_ids, _ = o.lookup(X, 2)
    E = rng.integers(0, 256, (n_rows, row_bytes), dtype=np.uint8)
    bad = want_ids >= n_rows
    want = E[np.where(bad, 0, want_ids)]
    want[bad] = 0
    store = torch.zeros(n_rows * row_bytes + 32, dtype=torch.uint8, device="cuda")
    rows = store[at[0]:at[0] + n_rows * row_bytes].view(n_rows, row_bytes)
    rows.copy_(dev(E))
    table = build_gpu(fg, ln, ids)
    cur, _ = S.lookup(table, dev(X), 2)
    for call in ("gather", "embed", "pipelined"):
        size = X.size * row_bytes
        hold = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        out = hold[at[1]:at[1] + size].view(3, 37, row_bytes)
        if call == "gather":
            S.gather(cur, rows, out=out)
        elif call == "embed":
            S.embed(table, dev(X), 2, rows, out=out)
        else:
            nxt = torch.empty_like(cur)
            S.embed_pipelined(table, dev(X), 2, nxt, cur, rows, out=out)
            assert np.array_equal(nxt.cpu().numpy(), want_ids)
        assert S.check() == (S.scone.EROW if bad.any() else S.scone.OK)
        assert np.array_equal(out.cpu().numpy(), want), call
        edge = torch.cat([hold[:at[1]], hold[at[1] + size:]]).cpu().numpy()
        assert (edge == 0xA5).all(), call
    # a decoding step with the row's second-to-last token as context
    size = 3 * row_bytes
    hold = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    out = hold[at[1]:at[1] + size].view(3, row_bytes)
    ctx, one = dev(X[:, -2:-1].copy()), torch.ones(3, dtype=torch.int32, device="cuda")
    S.decode_step(table, ctx, one, dev(X[:, -1].copy()), 2, rows, out)
    assert S.check() == (S.scone.EROW if bad[:, -1].any() else S.scone.OK)
    assert np.array_equal(out.cpu().numpy(), want[:, -1])
    edge = torch.cat([hold[:at[1]], hold[at[1] + size:]]).cpu().numpy()
    assert (edge == 0xA5).all()


def test_rows_past_2_gib():
    """The widest unit path of the fused kernel takes 64-bit indexes."""
    row_bytes = (1 << 31) + 5
    row = torch.empty((1, row_bytes), dtype=torch.uint8, device="cuda")
    row.random_(0, 256, generator=torch.Generator(device="cuda").manual_seed(1))
    table = build_gpu(np.zeros((0, 2), np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32))
    X = torch.zeros((1, 2), dtype=torch.int32, device="cuda")
    out = S.embed(table, X, 2, row)
    S.check_ok()
    assert torch.equal(out[0, 0], row[0]) and torch.equal(out[0, 1], row[0])


# Gathered in 8-byte units (8 divides the row but 16 does not, below 4 KiB) and, over
# PCIe, in 4-byte ones (below 2 KiB) or with one unit per thread (the fused kernel from
# 1 KiB on): the edges of these ranges and of a workgroup's units, aligned and not.
@pytest.mark.parametrize("row_bytes", [20, 24, 28, 40, 1000, 1016, 1020, 1028, 2040, 2044, 2052,
                                       4088, 4104])
@pytest.mark.parametrize("host,at", [(False, (0, 0)), (False, (8, 8)), (False, (4, 0)),
                                     (False, (0, 4)), (False, (1, 0)), (True, (0, 0)),
                                     (True, (0, 4))])
def test_narrow_units(row_bytes, host, at):
    rng = np.random.default_rng(row_bytes)
    pairs = rng.permutation(V * V)[:N]
    fg = np.stack([pairs // V, pairs % V], 1).astype(np.int32)
    ln = np.full(N, 2, dtype=np.int32)
    n_rows = V + N - 3                         # the last three f-grams have no row
    ids = (V + np.arange(N)).astype(np.int32)
    X = rng.integers(0, V, (3, 701)).astype(np.int32)
    want_ids, _ = oracle.OracleTable(fg, ln, ids).lookup(X, 2)
    E = rng.integers(0, 256, (n_rows, row_bytes), dtype=np.uint8)
    bad = want_ids >= n_rows
    want = E[np.where(bad, 0, want_ids)]
    want[bad] = 0
    if host:
        rows = S.HostRows(n_rows, (row_bytes,), torch.uint8)
        rows.tensor().copy_(torch.from_numpy(E))
    else:
        store = torch.zeros(n_rows * row_bytes + 32, dtype=torch.uint8, device="cuda")
        rows = store[at[0]:at[0] + n_rows * row_bytes].view(n_rows, row_bytes)
        rows.copy_(dev(E))
    table = build_gpu(fg, ln, ids)
    cur, _ = S.lookup(table, dev(X), 2)
    size = X.size * row_bytes
    for call in ("gather", "embed", "pipelined"):
        hold = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        out = hold[at[1]:at[1] + size].view(3, 701, row_bytes)
        if call == "gather":
            S.gather(cur, rows, out=out)
        elif call == "embed":
            S.embed(table, dev(X), 2, rows, out=out)
        else:
            S.embed_pipelined(table, dev(X), 2, torch.empty_like(cur), cur, rows, out=out)
        assert S.check() == (S.scone.EROW if bad.any() else S.scone.OK)
        assert np.array_equal(out.cpu().numpy(), want), call
        edge = torch.cat([hold[:at[1]], hold[at[1] + size:]]).cpu().numpy()
        assert (edge == 0xA5).all(), call
