"""The work that the speed of this framework is measured on.

Each case is one call sequence of a program that uses the framework, through
the functions of ``paper_2502_01637_amd``: a decoding step, a prefill, a step of
a stream of batches, host-resident rows, and the offline calls that make the
tables (discovery, the dictionary's build, tagging, the precompute of F).

Inputs are drawn on the GPU from the seed alone: Zipf(1.1) token streams with
planted f-grams, f-gram sets of distinct Zipf n-grams with lengths uniform in
[2, K], normal rows and weights.  The shapes are those of ``workloads`` and
``bench.py`` (tiny, c2_1m, c3_10m_k5, c4_host, c5_decode, the tagger, discovery
and the WebText 128M f-gram model) and of the tests' other model shapes.
"""
import math

import torch

import paper_2502_01637_amd as S

COVERAGE = 0.5      # share of the positions that lie inside planted f-grams
MIN_COUNT = 5       # discovery's minimum count (Section 3.1)


# ------------------------------------------------------------------ cases ----

def listed():
    return [
        # One token for each of eight conversations: what an interactive
        # server does between two steps of its model.  Launch-bound.
        {"name": "decode_8", "kind": "decode", "V": 32768, "n": 1_000_000, "K": 5, "S": 8,
         "d": 2048, "dtype": "bf16"},
        # The same for a full batch (c5_decode: 256 sequences, 4 KiB rows).
        {"name": "decode_256", "kind": "decode", "V": 32768, "n": 1_000_000, "K": 3, "S": 256,
         "d": 2048, "dtype": "bf16"},
        # A small model's prefill (tiny: 16 x 512 tokens, 64 fp32 per row).
        {"name": "prefill_tiny", "kind": "embed", "V": 1000, "n": 10_000, "K": 3, "B": 16,
         "T": 512, "d": 64, "dtype": "f32"},
        # Prefill of a GPT-2 scale batch (c2_1m: 64 x 2048, 2 KiB rows).
        {"name": "prefill_c2", "kind": "embed", "V": 32768, "n": 1_000_000, "K": 3, "B": 64,
         "T": 2048, "d": 1024, "dtype": "bf16"},
        # A ragged prefill at a width that is no power of two (d = 1536).
        {"name": "prefill_1536", "kind": "embed", "V": 32768, "n": 700_001, "K": 5, "B": 13,
         "T": 1999, "d": 1536, "dtype": "bf16"},
        # One step of a stream of batches at the paper's inference size
        # (c3_10m_k5: 10M f-grams, K = 5, 4 KiB rows, a 41 GB table).
        {"name": "stream_c3", "kind": "stream", "V": 32768, "n": 10_000_000, "K": 5, "B": 32,
         "T": 4096, "d": 2048, "dtype": "bf16"},
        # F in pinned host memory, T on the GPU (c4_host's batch; a smaller
        # table, as only the rows of the batch cross PCIe).
        {"name": "host_rows_c4", "kind": "host", "V": 32768, "n": 300_000, "K": 3, "B": 64,
         "T": 2048, "d": 2048, "dtype": "bf16"},
        # Tagging a training stream with match lengths (64 batches of c3).
        {"name": "tag_c3", "kind": "tag", "V": 32768, "n": 10_000_000, "K": 5, "B": 2048,
         "T": 4096},
        # Building the dictionary of 10M f-grams and answering a first batch.
        {"name": "build_10m", "kind": "build", "V": 32768, "n": 10_000_000, "K": 5, "B": 32,
         "T": 4096},
        # The S most frequent n-grams of a 16.8M-token corpus.
        {"name": "discover_16m", "kind": "discover", "V": 32768, "n": 1_000_000, "K": 5,
         "B": 4096, "T": 4096, "keep": 1_000_000},
        # Rows of a few new f-grams, with the wide-headed model of the tests.
        {"name": "precompute_3k", "kind": "precompute", "V": 32768, "n": 3001, "K": 5, "d": 1536,
         "heads": 12, "ff": 6144, "layers": 2},
        # The whole F of c2_1m by the WebText 128M model (d 1024, 6 layers).
        {"name": "precompute_1m", "kind": "precompute", "V": 32768, "n": 1_000_000, "K": 3,
         "d": 1024, "heads": 16, "ff": 4096, "layers": 6},
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], uniform in its logarithm, odd or even alike."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "embed", "embed", "stream", "host", "tag", "build", "discover",
                       "precompute", "precompute"])
    V = rng.choice([32768, 32768, 50257, 16001])
    K = rng.choice([2, 3, 3, 4, 5, 5, 6, 7])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    # any width: the models' multiples of 128, and a few that are not
    d = rng.choice([128 * rng.randint(1, 16), 64 * rng.randint(1, 32), rng.randint(33, 2048)])
    n = _log(rng, 3000, 2_000_000)
    case = {"kind": kind, "V": V, "n": n, "K": K}
    if kind == "decode":
        case.update(S=_log(rng, 1, 1024), d=d, dtype=dtype)
    elif kind in ("embed", "stream"):
        tok = _log(rng, 200, 131_072)
        B = _log(rng, 1, min(128, tok // 50))
        case.update(B=B, T=max(1, tok // B), d=d, dtype=dtype)
    elif kind == "host":
        tok = _log(rng, 2000, 131_072)
        B = _log(rng, 1, min(128, tok // 50))
        case.update(n=_log(rng, 3000, 200_000), B=B, T=tok // B, d=8 * rng.randint(32, 256),
                    dtype="bf16")
    elif kind in ("tag", "build"):
        tok = _log(rng, 2000, 8_000_000 if kind == "tag" else 131_072)
        B = _log(rng, 1, min(2048, tok // 50))
        case.update(n=_log(rng, 3000, 9_000_000), B=B, T=tok // B)
    elif kind == "discover":
        tok = _log(rng, 20_000, 16_000_000)
        B = _log(rng, 1, min(4096, tok // 50))
        case.update(K=max(3, K), B=B, T=tok // B, keep=_log(rng, 1000, 1_000_000))
    else:
        dm, heads = rng.choice([(512, 8), (1024, 16), (1024, 8), (1536, 12), (2048, 32)])
        layers = rng.randint(1, 4)
        most = 60_000_000_000_000 // (24 * dm * dm * layers * K)
        case.update(n=_log(rng, 300, min(200_000, most)), d=dm, heads=heads,
                    ff=128 * rng.randint(dm // 128, 4 * dm // 128), layers=layers)
    return case


# ----------------------------------------------------------------- inputs ----

DEV = "cuda"


def _rng(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + part) & ((1 << 62) - 1))
    return g


def _zipf(g, V, shape):
    w = torch.arange(1, V + 1, dtype=torch.float64, device=DEV) ** -1.1
    cdf = torch.cumsum(w, 0)
    u = torch.rand(shape, dtype=torch.float64, device=DEV, generator=g) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1).to(torch.int32)


def _print(fgrams):
    """A 64-bit fingerprint of each row (padding included)."""
    h = torch.zeros(fgrams.shape[0], dtype=torch.int64, device=fgrams.device)
    for j in range(fgrams.shape[1]):
        h = (h ^ (fgrams[:, j].long() + 2)) * -7046029254386353131
        h = h ^ ((h >> 29) & 0x7FFFFFFFF)
    return h


def _fgrams(g, V, n, K):
    """n distinct f-grams [n, K] (padded with -1) and their lengths."""
    have = torch.empty((0, K), dtype=torch.int32, device=DEV)
    more = n + n // 4 + 1000
    while have.shape[0] < n:
        length = torch.randint(2, K + 1, (more, 1), device=DEV, generator=g)
        new = _zipf(g, V, (more, K))
        new = new.masked_fill_(torch.arange(K, device=DEV)[None, :] >= length, -1)
        have = torch.cat([have, new])
        fp, order = torch.sort(_print(have), stable=True)
        first = torch.ones_like(fp, dtype=torch.bool)
        first[1:] = fp[1:] != fp[:-1]
        have = have[torch.sort(order[first])[0]]
        more = 2 * more
    have = have[:n].contiguous()
    return have, (have >= 0).sum(1).to(torch.int32)


def _queries(g, V, fgrams, lengths, B, T):
    """[B, T] tokens: f-grams of the set and single Zipf tokens, one after another."""
    n = lengths.numel()
    mean = float(lengths.double().mean())
    p = COVERAGE / (mean * (1 - COVERAGE) + COVERAGE)
    out = torch.empty((B, T), dtype=torch.int32, device=DEV)
    step = max(1, (1 << 22) // T)
    for b in range(0, B, step):
        e = min(B, b + step) - b
        kind = torch.rand((e, T), device=DEV, generator=g) < p
        choice = torch.randint(0, n, (e, T), device=DEV, generator=g)
        seg = torch.where(kind, lengths[choice].long(), 1)
        ends = torch.cumsum(seg, 1)
        t = torch.arange(T, device=DEV).expand(e, T).contiguous()
        at = torch.searchsorted(ends, t, right=True)
        off = t - (ends.gather(1, at) - seg.gather(1, at))
        planted = fgrams.reshape(-1)[choice.gather(1, at) * fgrams.shape[1] + off]
        out[b:b + e] = torch.where(kind.gather(1, at), planted, _zipf(g, V, (e, T)))
    return out


def _rows(g, n, d, dtype):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return torch.empty((n, d), dtype=dt, device=DEV).normal_(0.0, 0.02, generator=g)


def _params(case, seed):
    """The f-gram model's parameters in bf16, scaled so that every term counts."""
    g = _rng(seed, 7)
    d, ff = case["d"], case["ff"]

    def normal(*shape, std, mean=0.0):
        x = torch.empty(shape, device=DEV).normal_(mean, std, generator=g)
        return x.to(torch.bfloat16)

    p = {"pos": normal(case["K"], d, std=1.0)}
    for i in range(case["layers"]):
        q = f"l{i}."
        p.update({q + "ln1_g": normal(d, std=0.1, mean=1.0), q + "ln1_b": normal(d, std=0.1),
                  q + "w_qkv": normal(3 * d, d, std=d ** -0.5), q + "b_qkv": normal(3 * d, std=0.1),
                  q + "w_o": normal(d, d, std=d ** -0.5), q + "b_o": normal(d, std=0.1),
                  q + "ln2_g": normal(d, std=0.1, mean=1.0), q + "ln2_b": normal(d, std=0.1),
                  q + "w_fc1": normal(ff, d, std=d ** -0.5), q + "b_fc1": normal(ff, std=0.1),
                  q + "w_fc2": normal(d, ff, std=ff ** -0.5), q + "b_fc2": normal(d, std=0.1)})
    p.update({"lnf_g": normal(d, std=0.1, mean=1.0), "lnf_b": normal(d, std=0.1)})
    return p


def _model_inputs(case, seed):
    """(fgrams, lengths, token rows) of a precompute case."""
    fg, ln = _fgrams(_rng(seed, 1), case["V"], case["n"], case["K"])
    tok = torch.empty((case["V"], case["d"]), device=DEV).normal_(generator=_rng(seed, 3))
    return fg, ln, tok.to(torch.bfloat16)


def prepare(case, seed):
    kind, V, n, K = case["kind"], case["V"], case["n"], case["K"]
    s = {"case": case, "K": K}
    if kind == "precompute":
        fg, ln, tok = _model_inputs(case, seed)
        rows = torch.zeros((V + n, case["d"]), dtype=torch.bfloat16, device=DEV)
        rows[:V] = tok
        s["model"] = S.FgramModel(_params(case, seed), case["d"], case["heads"], case["ff"],
                                  case["layers"], K)
        s.update(fgrams=fg, lengths=ln, rows=rows,
                 ids=torch.arange(V, V + n, dtype=torch.int32, device=DEV))
        return s
    fg, ln = _fgrams(_rng(seed, 1), V, n, K)
    ids = torch.arange(V, V + n, dtype=torch.int32, device=DEV)
    if kind == "discover":
        s["tokens"] = _queries(_rng(seed, 2), V, fg, ln, case["B"], case["T"])
        return s
    if kind == "build":
        s.update(fgrams=fg, lengths=ln, ids=ids,
                 tokens=_queries(_rng(seed, 2), V, fg, ln, case["B"], case["T"]))
        return s
    s["table"] = S.build_fgram_table(fg, ln, ids)
    if kind == "decode":
        # conversations in their middle: the last K - 1 tokens of each are kept
        X = _queries(_rng(seed, 2), V, fg, ln, case["S"], 16)
        keep = max(K - 1, 1)
        s["ctx"] = X[:, 15 - keep:15].contiguous()
        s["ctx_len"] = torch.full((case["S"],), keep, dtype=torch.int32, device=DEV)
        s["new"] = X[:, 15].contiguous()
        s["rows"] = _rows(_rng(seed, 3), V + n, case["d"], case["dtype"])
        s["out"] = torch.empty((case["S"], case["d"]), dtype=s["rows"].dtype, device=DEV)
        return s
    s["tokens"] = _queries(_rng(seed, 2), V, fg, ln, case["B"], case["T"])
    if kind == "tag":
        s["len"] = torch.empty((case["B"], case["T"]), dtype=torch.int8, device=DEV)
        s["hist"] = torch.zeros(S.scone.MAX_FGRAM_LEN + 1, dtype=torch.int64, device=DEV)
    elif kind == "host":
        s["near"] = _rows(_rng(seed, 3), V, case["d"], case["dtype"])
        s["far"] = S.HostRows(n, (case["d"],), torch.bfloat16)
        s["far"].tensor().copy_(_rows(_rng(seed, 4), n, case["d"], case["dtype"]))
        need = S.scone.split_workspace_bytes(case["B"] * case["T"], 2 * case["d"])
        s["work"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    else:
        s["rows"] = _rows(_rng(seed, 3), V + n, case["d"], case["dtype"])
        if kind == "stream":
            s["cur"], _ = S.lookup(s["table"], s["tokens"], K)
            s["tokens"] = _queries(_rng(seed, 5), V, fg, ln, case["B"], case["T"])
            s["next"] = torch.empty_like(s["tokens"])
    return s


# -------------------------------------------------------------------- run ----

def run(s):
    kind, K = s["case"]["kind"], s["K"]
    if kind == "decode":
        out = S.decode_step(s["table"], s["ctx"], s["ctx_len"], s["new"], K, s["rows"], s["out"])
        return {"out": out, "ctx": s["ctx"]}
    if kind == "embed":
        return S.embed(s["table"], s["tokens"], K, s["rows"])
    if kind == "stream":
        out = S.embed_pipelined(s["table"], s["tokens"], K, s["next"], s["cur"], s["rows"])
        return {"out": out, "next": s["next"]}
    if kind == "host":
        ids, _ = S.lookup(s["table"], s["tokens"], K)
        return {"out": S.gather_split(ids, s["near"], s["far"], s["work"]), "ids": ids}
    if kind == "tag":
        return S.tag(s["table"], s["tokens"], K, match_len=s["len"], hist=s["hist"])
    if kind == "build":
        table = S.build_fgram_table(s["fgrams"], s["lengths"], s["ids"])
        ids, length = S.lookup(table, s["tokens"], K, want_len=True)
        S.check_ok()
        table.close()
        return ids, length
    if kind == "discover":
        fg, ln, ct = S.discover_fgrams(s["tokens"], K, s["case"]["keep"], MIN_COUNT)
        # The order of the f-grams and the choice among those at the cut are
        # unspecified; a program that hands out the same ids for the same
        # corpus keeps those above the cut, in the order of a fingerprint,
        # in a list of the asked size.
        above = ct > ct.min()
        fg, ln, ct = fg.masked_fill(~above[:, None], -1), ln * above, ct * above
        order = torch.argsort(_print(fg))
        fg, ln, ct = fg[order], ln[order], ct[order]
        more = s["case"]["keep"] - ct.numel()
        if more:
            fg = torch.nn.functional.pad(fg, (0, 0, 0, more), value=-1)
            ln, ct = (torch.nn.functional.pad(x, (0, more)) for x in (ln, ct))
        return fg, ln, ct
    V = s["case"]["V"]
    S.precompute_fgram_rows(s["model"], s["fgrams"], s["lengths"], s["ids"], s["rows"][:V],
                            s["rows"])
    return s["rows"][V:]


# ------------------------------------------------------- work and results ----

def work(case):
    """Bytes and operations of one pass, each input read and output written once.

    A gathered row counts once per token, as in ``bench.py``; the dictionary's
    probes are a way to find a match and are not counted.  An f-gram's prefixes
    may be shared, so the precompute counts the last position of every f-gram
    in every layer and nothing else.
    """
    kind, n, K = case["kind"], case["n"], case["K"]
    elem = 4 if case.get("dtype") == "f32" else 2
    tok = case.get("B", 0) * case.get("T", 0)
    if kind == "decode":
        return {"bytes": case["S"] * (2 * elem * case["d"] + 8 * K), "flops": 0}
    if kind in ("embed", "stream", "host"):
        return {"bytes": tok * (2 * elem * case["d"] + (12 if kind == "stream" else 4)),
                "flops": 0}
    if kind == "tag":
        return {"bytes": 5 * tok, "flops": 0}
    if kind == "build":
        return {"bytes": n * (4 * K + 8 + 16) + 9 * tok, "flops": 0}
    if kind == "discover":
        return {"bytes": 4 * tok + case["keep"] * (4 * K + 8), "flops": 0}
    d, ff, layers = case["d"], case["ff"], case["layers"]
    weights = layers * (4 * d * d + 2 * d * ff)
    return {"bytes": 2 * weights + n * (2 * d + 4 * K + 8) + 2 * case["V"] * d,
            "flops": 2 * weights * n}


def tolerance(case):
    # Ids, lengths, counts and copied rows are the same bits.  The rows of F
    # are bf16 with bf16 products between the layers: 0.0024 to 0.0037 off the
    # 64-bit result with one to six layers.
    return {"rel": 0.015, "max": 0.1} if case["kind"] == "precompute" else "exact"


def _norm(x, g, b):
    c = x - x.mean(-1, keepdim=True)
    return c * torch.rsqrt((c * c).mean(-1, keepdim=True) + 1e-5) * g + b


def exact(case, seed):
    """The rows of F in 64 bits (padding on the right, causal attention)."""
    if case["kind"] != "precompute":
        return None
    # about 40 TFLOP/s in 64 bits
    if case["n"] * case["K"] * 2 * case["layers"] * (4 * case["d"] ** 2
                                                     + 2 * case["d"] * case["ff"]) > 6e14:
        return None
    fg, ln, tok = _model_inputs(case, seed)
    p = {k: v.double() for k, v in _params(case, seed).items()}
    d, H = case["d"], case["heads"]
    out = torch.empty((case["n"], d), dtype=torch.float64, device=DEV)
    for L in range(2, case["K"] + 1):
        for at in torch.nonzero(ln == L).reshape(-1).split(16384 // L):
            x = tok[fg[at, :L].long()].double() + p["pos"][:L]
            for i in range(case["layers"]):
                w = {k[len(f"l{i}."):]: v for k, v in p.items() if k.startswith(f"l{i}.")}
                a = _norm(x, w["ln1_g"], w["ln1_b"])
                qkv = (a.reshape(-1, d) @ w["w_qkv"].t() + w["b_qkv"]).view(-1, L, 3, H, d // H)
                q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
                o = torch.empty_like(q)
                for j in range(L):
                    sc = (q[:, j:j + 1] * k[:, :j + 1]).sum(-1) / math.sqrt(d // H)
                    o[:, j] = (torch.softmax(sc, 1)[..., None] * v[:, :j + 1]).sum(1)
                x = x + (o.reshape(-1, d) @ w["w_o"].t() + w["b_o"]).view(-1, L, d)
                a = _norm(x, w["ln2_g"], w["ln2_b"]).reshape(-1, d)
                f = torch.nn.functional.gelu(a @ w["w_fc1"].t() + w["b_fc1"])
                x = x + (f @ w["w_fc2"].t() + w["b_fc2"]).view(-1, L, d)
            out[at] = _norm(x[:, -1], p["lnf_g"], p["lnf_b"])
    return out
