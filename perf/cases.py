"""The work that a user of the library has it do, as cases that can be timed and compared.

Five kinds of pass, each through the public calls of ``paper_2609_27233_amd.lib``:

  decode    attention layer of a few decode steps, the last of which merges a span
  merge     surrogates of a list of spans (directly, or from the token table)
  prefill   attention layer of a prompt (or of a chunk of one) over the paged cache
  compress  a prompt batch from token ids to packed rows (match, dedupe, merge, pack)
  step      what precedes the layers in a decode step (rule check, input row, first K/V state)

Every pass leaves the cache as long as it found it, so it can be called again.
"""
import math

import numpy as np
import torch

from paper_2609_27233_amd import lib as sm

VOCAB = 128256
EPS = 1e-5
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# --------------------------------------------------------------------------
# the cases

def listed():
    return [
        # one chat session on the 8B-shaped layer: launches and latency count
        dict(name="decode-one", kind="decode", dtype="bf16", n=1, Hq=32, Hkv=8, D=128, bs=16, lo=1475, hi=1475,
             plain=2, shuffled=True),
        # the benchmark's decode batch: 16 prompts of 4096 tokens, compacted, some way into generation
        dict(name="decode-8b-batch", kind="decode", dtype="bf16", n=16, Hq=32, Hkv=8, D=128, bs=16, lo=2458, hi=2842,
             plain=2, shuffled=False),
        # the 7B-shaped serving batch: 128 sessions of all ages
        dict(name="decode-7b-ragged", kind="decode", dtype="bf16", n=128, Hq=28, Hkv=4, D=128, bs=16, lo=512, hi=4096,
             plain=2, shuffled=True),
        # few long documents: 4 x 32768 tokens, compacted, on pages handed out in any order
        dict(name="decode-8b-long", kind="decode", dtype="bf16", n=4, Hq=32, Hkv=8, D=128, bs=16, lo=19661, hi=19700,
             plain=2, shuffled=True),
        # one prompt of 4096 tokens merged on arrival, the first stage looked up by token
        dict(name="merge-prompt", kind="merge", dtype="bf16", d=4096, h=4, spans=609, nlo=2, nhi=8, tabled=True),
        # a decode step at which every one of 128 sessions completes a span of 3 to 5 tokens
        dict(name="merge-steps", kind="merge", dtype="bf16", d=3584, h=4, spans=128, nlo=3, nhi=5, tabled=False),
        # the 70B-shaped prompt batch, 32 x 8192 tokens: the largest call there is
        dict(name="merge-70b-batch", kind="merge", dtype="bf16", d=8192, h=4, spans=38847, nlo=2, nhi=8, tabled=False),
        # the small fp32 model: one prompt of 512 tokens, 30% of it in spans
        dict(name="merge-small-f32", kind="merge", dtype="f32", d=256, h=4, spans=51, nlo=2, nhi=4, tabled=False),
        # prefill of the benchmark's compacted prompt batch
        dict(name="prefill-batch", kind="prefill", n=16, Hq=32, Hkv=8, D=128, bs=16, rows=2458, past=0),
        # a long document prefilled in chunks: the next 512 rows of one sequence over what is cached
        dict(name="prefill-chunk", kind="prefill", n=1, Hq=32, Hkv=8, D=128, bs=16, rows=512, past=16384),
        # a long document compressed on arrival
        dict(name="compress-document", kind="compress", B=1, T=32768, d=4096, h=4, rules=2167573, removal=0.4, zipf=1.2),
        # the input side of four decode steps of the benchmark batch
        dict(name="step-inputs", kind="step", n=16, d=4096, Hkv=8, D=128, bs=16, length=2650, rules=500000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads, kv heads, head dim) of the layers the library is configured and tested with
_LAYERS = ((32, 8, 128), (28, 4, 128), (64, 8, 128), (16, 4, 64), (4, 4, 64), (8, 8, 128))
_WIDTHS = (256, 512, 1024, 2048, 3584, 4096, 5120, 8192)


def draw(rng):
    kind = rng.choice(("decode", "decode", "merge", "merge", "prefill", "compress", "step"))
    if kind == "decode":
        Hq, Hkv, D = rng.choice(_LAYERS)
        dtype = "f32" if D == 64 and rng.random() < 0.4 else "bf16"
        n = _log_int(rng, 1, 192)
        hi = _log_int(rng, 48, max(64, min(32768, int((24576 if dtype == "f32" else 524288) * 8 / (n * Hkv)))))
        return dict(kind=kind, dtype=dtype, n=n, Hq=Hq, Hkv=Hkv, D=D, bs=rng.choice((16, 16, 32, 64)),
                    lo=max(8, int(hi * rng.uniform(0.1, 1.0))), hi=hi, plain=rng.choice((0, 1, 2)),
                    shuffled=rng.random() < 0.5)
    if kind == "merge":
        f32 = rng.random() < 0.2
        d = rng.choice((256, 512, 1024) if f32 else _WIDTHS)
        nlo = rng.choice((2, 2, 3))
        spans = _log_int(rng, 1, min(40000, int((2 << 30 if f32 else 1600 << 30) / (d * d))))
        return dict(kind=kind, dtype="f32" if f32 else "bf16", d=d, h=rng.choice((4, 4, 2)), spans=spans, nlo=nlo,
                    nhi=nlo + rng.choice((1, 2, 6)), tabled=rng.random() < 0.5)
    if kind == "prefill":
        Hq, Hkv, D = rng.choice(_LAYERS)
        n = rng.choice((1, 1, 2, 3, 5, 8, 16))
        rows = _log_int(rng, 16, min(8192, int(49152 / n)))
        past = 0 if rng.random() < 0.5 else _log_int(rng, 64, 24576)
        while n * rows * (past + rows / 2) * Hq * D > 16 * 4096 * 2048 * 32 * 128:
            past //= 2
        return dict(kind=kind, n=n, Hq=Hq, Hkv=Hkv, D=D, bs=rng.choice((16, 16, 32, 64)), rows=rows, past=past)
    if kind == "compress":
        B = rng.choice((1, 1, 2, 4, 7, 16))
        return dict(kind=kind, B=B, T=_log_int(rng, 64, 65536 // B), d=rng.choice((2048, 3584, 4096)), h=4,
                    rules=_log_int(rng, 20000, 2167573), removal=round(rng.uniform(0.05, 0.4), 3),
                    zipf=rng.choice((0.0, 1.2)))
    Hq, Hkv, D = rng.choice(((32, 8, 128), (28, 4, 128), (64, 8, 128), (16, 4, 64)))
    return dict(kind="step", n=_log_int(rng, 1, 256), d=rng.choice((1024, 2048, 3584, 4096, 8192)), Hkv=Hkv, D=D,
                bs=rng.choice((16, 32)), length=_log_int(rng, 20, 8192), rules=_log_int(rng, 20000, 500000))


# --------------------------------------------------------------------------
# inputs (plain torch and numpy)

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, shape, dtype, std=1.0, mean=0.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _i32(a):
    return torch.as_tensor(np.array(a, dtype=np.int32, order="C")).cuda()


def _cache_inputs(g, rs, dtype, lengths, most, Hkv, D, bs, shuffled):
    """Pools, block table and free list of a cache whose sequences hold `lengths` entries and may come to hold `most`."""
    n = len(lengths)
    cap = -(-most // bs)                                             # blocks of a sequence
    used = -(-lengths // bs)
    total = n * cap
    order = rs.permutation(total) if shuffled else np.arange(total)
    table = np.full((n, cap), -1, np.int32)
    at = 0
    for s in range(n):
        table[s, :used[s]] = order[at:at + used[s]]
        at += used[s]
    return dict(k_pool=_randn(g, (total, Hkv, bs, D), dtype), v_pool=_randn(g, (total, Hkv, D, bs), dtype),
                table=table, lengths=lengths.astype(np.int32), free=order[at:].astype(np.int32),
                cap=cap, blocks=total)


def _merge_params(g, d, h, dtype):
    w = lambda *shape: _randn(g, shape, dtype, 0.02)                 # noqa: E731
    return dict(Q=_randn(g, (h, d // h), dtype), W_kv=w(d, d), b_kv=w(d), W_o=w(d, d), b_o=w(d),
                g_kv=_randn(g, (d,), dtype, 0.1, 1.0), beta_kv=_randn(g, (d,), dtype, 0.1),
                g_o=_randn(g, (d,), dtype, 0.1, 1.0), beta_o=_randn(g, (d,), dtype, 0.1))


def _token_table(g, d, dtype):
    """First-stage rows GELU(Linear(e)) of every token, as a program has them from its weights."""
    out = torch.empty((VOCAB, d), dtype=dtype, device="cuda")
    for a in range(0, VOCAB, 16384):
        part = out[a:a + 16384]
        part.copy_(torch.nn.functional.gelu(torch.empty(part.shape, device="cuda").normal_(0, 0.4, generator=g)))
    return out


def _rules(g, count):
    """Random 2-, 3- and 4-grams, in the proportions of the rule set mined for the Llama-3 tokenizer."""
    r = torch.randint(0, VOCAB, (count, 4), dtype=torch.int32, device="cuda", generator=g)
    kind = torch.rand(count, device="cuda", generator=g)
    r[kind < 0.416, 3] = -1
    r[kind < 0.100, 2] = -1
    return r


def _plant(rs, rules, B, T, removal, zipf):
    """B sequences of T random tokens with rules planted at random places until removal x T positions go."""
    n_rules = rules.shape[0]
    most = max(1, int(removal * T))
    ids = rs.randint(0, VOCAB, (B, T)).astype(np.int32)
    pick = (rs.zipf(zipf, (B, most)) - 1) % n_rules if zipf else rs.randint(0, n_rules, (B, most))
    grams = rules[torch.from_numpy(pick.reshape(-1)).cuda()].cpu().numpy().reshape(B, most, 4)
    lens = (grams >= 0).sum(2)
    for b in range(B):
        k = max(1, int((np.cumsum(lens[b] - 1) <= removal * T).sum()))
        ln = lens[b, :k]
        cuts = np.sort(rs.choice(T - int(ln.sum()) + k, size=k, replace=False))
        starts = cuts - np.arange(k) + np.cumsum(ln) - ln
        for j in range(4):
            m = ln > j
            ids[b, starts[m] + j] = grams[b, :k][m, j]
    return ids.reshape(-1)


def _inputs(case, seed):
    g, rs = _gen(seed), np.random.RandomState(seed % (1 << 31))
    k = case["kind"]
    dtype = DTYPES[case.get("dtype", "bf16")]
    x = {}
    if k == "decode":
        n, H, D, p = case["n"], case["Hkv"], case["D"], case["plain"]
        lengths = rs.randint(case["lo"], case["hi"] + 1, n)
        x["cache"] = _cache_inputs(g, rs, dtype, lengths, case["hi"] + p + 2, H, D, case["bs"], case["shuffled"])
        x["K"], x["V"] = _randn(g, (p + 1, n, H, D), dtype), _randn(g, (p + 1, n, H, D), dtype)
        x["q"] = _randn(g, (p + 1, n, case["Hq"], D), dtype)
        x["ids"] = rs.permutation(n)
    elif k == "merge":
        d = case["d"]
        n = rs.randint(case["nlo"], case["nhi"] + 1, case["spans"])
        x["offsets"] = np.concatenate([[0], np.cumsum(n)])
        x["rows"] = rs.randint(0, VOCAB, int(n.sum()))
        x["params"] = _merge_params(g, d, case["h"], dtype)
        x["table" if case["tabled"] else "emb"] = (_token_table(g, d, dtype) if case["tabled"]
                                                   else _randn(g, (VOCAB, d), dtype, 0.02))
    elif k == "prefill":
        n, H, D, m = case["n"], case["Hkv"], case["D"], case["rows"]
        lens = rs.permutation(m - np.arange(n) * (m // 16) // n)     # prompts compact to similar lengths
        past = np.full(n, case["past"])
        x["cache"] = _cache_inputs(g, rs, dtype, past, case["past"] + m, H, D, case["bs"], True)
        x["offsets"] = np.concatenate([[0], np.cumsum(lens)])
        R = int(lens.sum())
        x["K"], x["V"] = _randn(g, (R, H, D), dtype), _randn(g, (R, H, D), dtype)
        x["q"] = _randn(g, (R, case["Hq"], D), dtype)
    elif k == "compress":
        d = case["d"]
        x["rules"] = _rules(g, case["rules"])
        x["tokens"] = _plant(rs, x["rules"], case["B"], case["T"], case["removal"], case["zipf"])
        x["params"] = _merge_params(g, d, case["h"], dtype)
        x["table"], x["emb"] = _token_table(g, d, dtype), _randn(g, (VOCAB, d), dtype, 0.02)
    else:
        n, H, D, d = case["n"], case["Hkv"], case["D"], case["d"]
        lengths = np.maximum(8, rs.randint(case["length"] // 2, case["length"] + 1, n))
        x["cache"] = _cache_inputs(g, rs, dtype, lengths, max(8, case["length"]) + 4, H, D, case["bs"], True)
        x["rules"] = _rules(g, case["rules"])
        x["lut"] = _randn(g, (case["rules"], d), dtype)
        x["emb"] = _randn(g, (VOCAB, d), dtype, 0.02)
        x["W_k"], x["W_v"] = _randn(g, (H * D, d), dtype, 0.02), _randn(g, (H * D, d), dtype, 0.02)
        x["ids"] = rs.permutation(n)
        # a quarter of the sequences generate a 4-gram rule token by token, the others anything
        four = torch.nonzero(x["rules"][:, 3] >= 0).reshape(-1).cpu().numpy()
        x["tokens"] = rs.randint(0, VOCAB, (4, n))
        x["picked"] = np.full(n, -1)
        for i in range(0, n, 4):
            x["picked"][i] = four[rs.randint(len(four))]
            x["tokens"][:, i] = x["rules"][x["picked"][i]].cpu().numpy()
    return x


# --------------------------------------------------------------------------
# what a program has in hand

def _paged(c, dtype, Hkv, D, bs):
    n = len(c["lengths"])
    p = sm.PagedCache(dtype=dtype, num_kv_heads=Hkv, head_dim=D, block_size=bs, num_blocks=c["blocks"], max_seqs=n,
                      max_blocks_per_seq=c["cap"])
    p.k_pool.copy_(c["k_pool"])
    p.v_pool.copy_(c["v_pool"])
    p.block_table.copy_(_i32(c["table"]))
    p.lengths.copy_(_i32(c["lengths"]))
    p.free_stack.zero_()
    p.free_stack[:len(c["free"])] = _i32(c["free"][::-1])            # the last one is handed out first
    p.free_top.fill_(len(c["free"]))
    return p


def _err():
    return torch.zeros(1, dtype=torch.int32, device="cuda")


def _bytes(n):
    return torch.zeros(max(1, n), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    x = _inputs(case, seed)
    k = case["kind"]
    dtype = DTYPES[case.get("dtype", "bf16")]
    s = dict(case=case, x=x)
    if "cache" in x:
        s["cache"] = _paged(x["cache"], dtype, case["Hkv"], case["D"], case["bs"])
        for name in ("k_pool", "v_pool"):
            del x["cache"][name]
    if k == "decode":
        n, p = case["n"], case["plain"]
        s["ids"] = _i32(x["ids"])
        s["crop"] = torch.full((n,), p + 1, dtype=torch.int32, device="cuda")
        s["max_len"] = int(x["cache"]["lengths"].max()) + p + 1
        s["out"] = torch.zeros_like(x["q"])
        s["ws"] = _bytes(sm.decode_workspace_bytes(n, case["Hq"], case["D"], s["max_len"]))
    elif k == "merge":
        R, S, d = len(x["rows"]), case["spans"], case["d"]
        s["rows"], s["offsets"] = _i32(x["rows"]), _i32(x["offsets"])
        s["out"] = torch.zeros((S, d), dtype=dtype, device="cuda")
        s["ws"] = _bytes(sm.merge_workspace_bytes(0 if case["tabled"] else R, S, d, dtype))
        s["err"] = _err()
    elif k == "prefill":
        lens = np.diff(x["offsets"])
        s["ids"], s["offsets"], s["lens"] = _i32(np.arange(case["n"])), _i32(x["offsets"]), _i32(lens)
        s["max_rows"] = int(lens.max())
        s["out"] = torch.zeros_like(x["q"])
    elif k == "compress":
        B, T, d = case["B"], case["T"], case["d"]
        N = B * T
        i32 = lambda m: torch.zeros(m, dtype=torch.int32, device="cuda")  # noqa: E731
        s["rules"] = sm.RuleTable(sm.RuleTable.capacity_for(case["rules"]))
        sm.rules_build(s["rules"], x["rules"])
        s["tokens"], s["offsets"] = _i32(x["tokens"]), _i32(np.arange(B + 1) * T)
        s.update(span_start=i32(N // 2), span_len=i32(N // 2), span_rule=i32(N // 2), span_offsets=i32(B + 1),
                 uniq=i32(N // 2), slot=i32(N // 2), uniq_rows=i32(N), uniq_offsets=i32(N // 2 + 1), num_uniq=i32(1),
                 pi=i32(N), packed_offsets=i32(B + 1), packed_src=i32(N))
        s["z"], s["surrogates"] = (torch.zeros((N // 2, d), dtype=dtype, device="cuda") for _ in range(2))
        s["packed"] = torch.zeros((N, d), dtype=dtype, device="cuda")
        s["match_ws"] = _bytes(sm.match_prompt_workspace_bytes(B, N))
        s["dedupe_ws"] = _bytes(sm.load().sm_span_dedupe_workspace_bytes(N // 2, case["rules"]))
        s["merge_ws"] = _bytes(sm.merge_workspace_bytes(0, N // 2, d, dtype))
        s["err"] = _err()
    else:
        n, d = case["n"], case["d"]
        s["rules"] = sm.RuleTable(sm.RuleTable.capacity_for(case["rules"]))
        sm.rules_build(s["rules"], x["rules"])
        s["ids"], s["tokens"] = _i32(x["ids"]), _i32(x["tokens"])
        s["state"] = torch.zeros((n, 4), dtype=torch.int32, device="cuda")
        s["undo"] = _i32(np.where(x["picked"] >= 0, 1, 4))
        s["crop"], s["rule"] = (torch.zeros((4, n), dtype=torch.int32, device="cuda") for _ in range(2))
        s["rows"] = torch.zeros((4, n, d), dtype=dtype, device="cuda")
        s["ws"] = _bytes(sm.kv_project_workspace_bytes(n, d, case["Hkv"], case["D"]))
        s["err"] = _err()
    return s


# --------------------------------------------------------------------------
# one pass

def run(s):
    k, x = s["case"]["kind"], s["x"]
    if k == "decode":
        c, p, ids, ws, top = s["cache"], s["case"]["plain"], s["ids"], s["ws"], s["max_len"]
        for j in range(p):
            sm.decode_step(c, ids, x["K"][j], x["V"][j], x["q"][j], s["out"][j], ws, top)
        # a span of p + 2 tokens is complete: its p + 1 cached entries go and its surrogate's state comes
        if c.dtype == torch.bfloat16:
            sm.decode_merge_step(c, ids, s["crop"], x["K"][p], x["V"][p], x["q"][p], s["out"][p], ws, top)
        else:
            sm.kv_rollback(c, ids, s["crop"])
            sm.decode_step(c, ids, x["K"][p], x["V"][p], x["q"][p], s["out"][p], ws, top)
        return dict(out=s["out"], **_cache_outputs(c))
    if k == "merge":
        if s["case"]["tabled"]:
            sm.merge_spans_tabled(x["table"], s["rows"], s["offsets"], x["params"], s["case"]["h"], s["out"], s["ws"],
                                  s["err"], ln_eps=EPS)
        else:
            sm.merge_spans(x["emb"], s["rows"], s["offsets"], x["params"], s["case"]["h"], s["out"], s["ws"],
                           s["err"], ln_eps=EPS)
        return dict(out=s["out"], err=s["err"])
    if k == "prefill":
        c = s["cache"]
        sm.kv_append(c, s["ids"], s["offsets"], x["K"], x["V"])
        sm.prefill_attention(c, s["ids"], s["offsets"], x["q"], s["out"], s["max_rows"])
        sm.kv_rollback(c, s["ids"], s["lens"])                       # the request ends
        return dict(out=s["out"], **_cache_outputs(c))
    if k == "compress":
        sm.match_prompt(s["rules"], s["tokens"], s["offsets"], s["span_start"], s["span_len"], s["span_rule"],
                        s["span_offsets"], s["match_ws"])
        S = int(s["span_offsets"][-1])
        start, ln, rule, slot = (s[name][:S] for name in ("span_start", "span_len", "span_rule", "slot"))
        sm.span_dedupe(rule, start, ln, s["case"]["rules"], s["tokens"], s["uniq"][:S], slot, s["uniq_rows"],
                       s["uniq_offsets"], s["num_uniq"], s["err"], ws=s["dedupe_ws"])
        U = int(s["num_uniq"])
        R = int(s["uniq_offsets"][U])
        z, surrogates = s["z"][:U], s["surrogates"][:S]
        sm.merge_spans_tabled(x["table"], s["uniq_rows"][:R], s["uniq_offsets"][:U + 1], x["params"], s["case"]["h"],
                              z, s["merge_ws"], s["err"], ln_eps=EPS)
        sm.gather_surrogates(z, slot, surrogates, s["err"])
        sm.pack_spans(s["offsets"], start, ln, s["span_offsets"], s["pi"], s["packed_offsets"], s["packed_src"],
                      s["err"], s["tokens"].numel(), token_ids=s["tokens"], emb=x["emb"], surrogates=surrogates,
                      packed=s["packed"])
        return {name: s[name] for name in _COMPRESSED}
    c = s["cache"]
    for j in range(4):
        sm.match_decode(s["rules"], s["state"], s["ids"], s["tokens"][j], s["crop"][j], s["rule"][j], cache=c)
        sm.gather_surrogates(x["lut"], s["rule"][j], s["rows"][j], s["err"], emb=x["emb"], token_ids=s["tokens"][j])
        sm.kv_append_projected(c, s["ids"], s["rows"][j], x["W_k"], x["W_v"], ws=s["ws"])
    sm.kv_rollback(c, s["ids"], s["undo"])                           # the candidate continuation is dropped
    return dict(crop=s["crop"], rule=s["rule"], rows=s["rows"], state=s["state"], err=s["err"], **_cache_outputs(c))


_COMPRESSED = ("span_start", "span_len", "span_rule", "slot", "span_offsets", "uniq", "uniq_rows", "uniq_offsets", "pi",
               "packed_offsets", "packed_src", "packed", "err")


def _cache_outputs(c):
    return dict(k_pool=c.k_pool, v_pool=c.v_pool, block_table=c.block_table, lengths=c.lengths, free_top=c.free_top,
                cache_err=c.err)


# --------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    k = case["kind"]
    es = 4 if case.get("dtype") == "f32" else 2
    if k == "decode":
        n, Hq, Hkv, D, steps = case["n"], case["Hq"], case["Hkv"], case["D"], case["plain"] + 1
        L = n * (case["lo"] + case["hi"]) / 2
        return dict(bytes=steps * es * D * (2 * Hkv * (L + 2 * n) + 2 * n * Hq), flops=steps * 4 * L * Hq * D)
    if k == "merge":
        d, S, R = case["d"], case["spans"], case["spans"] * (case["nlo"] + case["nhi"]) / 2
        first = 0 if case["tabled"] else 1
        return dict(bytes=es * d * (R + S + (1 + first) * d), flops=2 * d * d * (S + first * R))
    if k == "prefill":
        n, Hq, Hkv, D, past = case["n"], case["Hq"], case["Hkv"], case["D"], case["past"]
        m = case["rows"] - (n - 1) / 2 * (case["rows"] // 16) / n
        return dict(bytes=2 * n * D * (2 * m * Hq + 2 * Hkv * (past + m) + 4 * Hkv * m),
                    flops=4 * n * Hq * D * m * (past + m / 2))
    if k == "compress":
        N, d = case["B"] * case["T"], case["d"]
        spans = case["removal"] * N / 2.484                          # 2.484 positions go with the mean rule
        uniq = spans * (0.3 if case["zipf"] else 1.0)
        kept = N * (1 - case["removal"])
        return dict(bytes=N * (4 + 3 * 16 + 4 + 4) + 2 * d * (2 * kept - spans + 3.484 * uniq + d), flops=2 * d * d * uniq)
    n, d, HD = case["n"], case["d"], case["Hkv"] * case["D"]
    return dict(bytes=4 * (2 * (2 * HD * d + 2 * n * d + 2 * n * HD) + n * 3 * 16), flops=4 * 4 * HD * d * n)


def tolerance(case):
    if case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 results of sums in fp32: two correct results differ by roundings of 2^-9 of a value, and where
    # intermediate rows are rounded too (merge, compress) by those of the rows as well
    return {"rel": 1e-2, "max": 0.1}


# --------------------------------------------------------------------------
# the same in 64 bits

def _attend(q, K, V, first):
    """q [m, Hq, D], K and V [L, H, D], all 64-bit: row r sees entries 0 .. first + r."""
    m, Hq, D = q.shape
    L, H, _ = K.shape
    G = Hq // H
    out = torch.empty_like(q)
    qh = q.view(m, H, G, D)
    seen = torch.arange(L, device=q.device)
    for r0 in range(0, m, 1024):
        r1 = min(m, r0 + 1024)
        hide = seen[None, :] > first + torch.arange(r0, r1, device=q.device)[:, None]
        for h in range(H):
            a = qh[r0:r1, h].permute(1, 0, 2).reshape(G * (r1 - r0), D) @ K[:, h].t().contiguous() * D ** -0.5
            a = torch.softmax(a.view(G, r1 - r0, L).masked_fill(hide, -math.inf), -1).view(G * (r1 - r0), L)
            out.view(m, H, G, D)[r0:r1, h] = (a @ V[:, h].contiguous()).view(G, r1 - r0, D).permute(1, 0, 2)
    return out


def _entries(c, s):
    """Cached K and V of sequence s, [L, H, D] in 64 bits."""
    L = int(c["lengths"][s])
    bs = c["k_pool"].shape[2]
    blk = torch.as_tensor(c["table"][s, :-(-L // bs)].astype(np.int64)).cuda()
    H, D = c["k_pool"].shape[1], c["k_pool"].shape[3]
    K = c["k_pool"][blk].double().permute(0, 2, 1, 3).reshape(-1, H, D)[:L]
    V = c["v_pool"][blk].double().permute(0, 3, 1, 2).reshape(-1, H, D)[:L]
    return K, V


def _layer_norm(x, g, b):
    return torch.nn.functional.layer_norm(x, x.shape[-1:], g.double(), b.double(), EPS)


def _merge(first_rows, offsets, p, h):
    """Surrogates of spans whose first-stage rows GELU(Linear_kv(e)) come from first_rows(a, b), in 64 bits."""
    S, d = len(offsets) - 1, p["W_o"].shape[0]
    off = torch.as_tensor(np.asarray(offsets, np.int64)).cuda()
    W, q = p["W_o"].double().t().contiguous(), p["Q"].double()
    out = torch.empty((S, d), dtype=torch.float64, device="cuda")
    for s0 in range(0, S, 4096):
        s1 = min(S, s0 + 4096)
        a, b = int(off[s0]), int(off[s1])
        P = _layer_norm(first_rows(a, b), p["g_kv"], p["beta_kv"]).view(b - a, h, d // h)
        score = (P * q).sum(-1) / math.sqrt(d // h)
        span = torch.repeat_interleave(torch.arange(s1 - s0, device="cuda"), off[s0 + 1:s1 + 1] - off[s0:s1])
        top = torch.full((s1 - s0, h), -math.inf, dtype=torch.float64, device="cuda")
        top.scatter_reduce_(0, span[:, None].expand(-1, h), score, "amax")
        e = torch.exp(score - top[span])
        z = torch.zeros((s1 - s0, h), dtype=torch.float64, device="cuda").index_add_(0, span, e)
        w = (e / z[span])[:, :, None]
        c = torch.zeros((s1 - s0, h, d // h), dtype=torch.float64, device="cuda").index_add_(0, span, w * P)
        y = torch.nn.functional.gelu(c.view(-1, d) @ W + p["b_o"].double())
        out[s0:s1] = _layer_norm(y, p["g_o"], p["beta_o"])
    return out


def _gram_keys(g4, n):
    """64-bit keys of the first n tokens of [m, 4] grams (distinct but for a chance in about 1e8)."""
    k = g4[:, 0].long()
    for j in range(1, n):
        k = k * 6364136223846793005 + (g4[:, j].long() + 1442695040888963407)
        k = k ^ (k >> 29)
    return k


def _spans(x, B, T):
    """Left to right, longest first: (start, length) of every span of the batch."""
    tok = torch.as_tensor(x["tokens"]).cuda().view(B, T)
    pad = torch.nn.functional.pad(tok, (0, 3), value=-1)
    win = torch.stack([pad[:, j:j + T] for j in range(4)], -1).reshape(-1, 4)
    best = torch.zeros(B * T, dtype=torch.int64, device="cuda")
    size = (x["rules"] >= 0).sum(1)
    for n in (2, 3, 4):
        keys = _gram_keys(x["rules"][size == n], n).sort().values
        if len(keys):
            k = _gram_keys(win, n)
            hit = keys[torch.searchsorted(keys, k).clamp(max=len(keys) - 1)] == k
            best[hit & (win[:, :n] >= 0).all(1)] = n
    best = best.cpu().numpy().reshape(B, T)
    spans = []
    for b in range(B):
        t, row = 0, best[b].tolist()
        while t < T:
            if row[t]:
                spans.append((b * T + t, row[t]))
            t += max(1, row[t])
    return spans


def exact(case, seed):
    k = case["kind"]
    x = _inputs(case, seed)
    nothing = dict(k_pool=None, v_pool=None, block_table=None, lengths=None, free_top=None, cache_err=None)
    if k == "decode":
        p = case["plain"]
        out = torch.empty(x["q"].shape, dtype=torch.float64, device="cuda")
        for i, s in enumerate(x["ids"]):
            K, V = _entries(x["cache"], s)
            for j in range(p + 1):
                if j == p:                                           # p appended rows and one more are dropped
                    K, V = (t[:t.shape[0] - p - 1] for t in (K, V))
                K = torch.cat([K, x["K"][j, i][None].double()])
                V = torch.cat([V, x["V"][j, i][None].double()])
                out[j, i] = _attend(x["q"][j, i][None].double(), K, V, K.shape[0] - 1)[0]
        return dict(out=out, **nothing)
    if k == "prefill":
        out = torch.empty(x["q"].shape, dtype=torch.float64, device="cuda")
        for i in range(case["n"]):
            a, b = int(x["offsets"][i]), int(x["offsets"][i + 1])
            K, V = _entries(x["cache"], i)
            K, V = torch.cat([K, x["K"][a:b].double()]), torch.cat([V, x["V"][a:b].double()])
            out[a:b] = _attend(x["q"][a:b].double(), K, V, case["past"])
        return dict(out=out, **nothing)
    if k == "merge":
        rows, p = torch.as_tensor(x["rows"]).cuda(), x["params"]
        if case["tabled"]:
            first = lambda a, b: x["table"][rows[a:b]].double()      # noqa: E731
        else:
            W, bias = p["W_kv"].double().t().contiguous(), p["b_kv"].double()
            first = lambda a, b: torch.nn.functional.gelu(x["emb"][rows[a:b]].double() @ W + bias)  # noqa: E731
        return dict(out=_merge(first, x["offsets"], p, case["h"]), err=None)
    if k == "compress":
        B, T, N = case["B"], case["T"], case["B"] * case["T"]
        spans = _spans(x, B, T)
        tokens = torch.as_tensor(x["tokens"].astype(np.int64)).cuda()
        start, ln = (np.array(v, np.int64) for v in zip(*spans))
        offsets = np.concatenate([[0], np.cumsum(ln)])
        inside = torch.as_tensor(np.concatenate([np.arange(a, a + n) for a, n in spans])).cuda()
        z = _merge(lambda a, b: x["table"][tokens[inside[a:b]]].double(), offsets, x["params"], case["h"])
        keep = torch.ones(N, dtype=torch.bool, device="cuda")
        keep[inside] = False
        last = torch.as_tensor(start + ln - 1).cuda()
        keep[last] = True
        where = torch.cumsum(keep, 0) - 1
        packed = torch.zeros((N, case["d"]), dtype=torch.float64, device="cuda")
        packed[:int(keep.sum())] = x["emb"][tokens[keep]].double()
        packed[where[last]] = z
        return dict(dict.fromkeys(_COMPRESSED), packed=packed)
    # step: the pools with the rows that the four steps write
    n, H, D, bs, c = case["n"], case["Hkv"], case["D"], case["bs"], x["cache"]
    k_pool, v_pool = c["k_pool"].double(), c["v_pool"].double()
    free = list(c["free"])
    table = c["table"].copy()
    length = c["lengths"].astype(np.int64).copy()
    freq = 500000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device="cuda") / D)
    Wk, Wv = x["W_k"].double().t().contiguous(), x["W_v"].double().t().contiguous()
    tokens = torch.as_tensor(x["tokens"]).cuda()
    for j in range(4):
        row = x["emb"][tokens[j]].double()
        if j == 3:
            hit = torch.as_tensor(np.nonzero(x["picked"] >= 0)[0]).cuda()
            row[hit] = x["lut"][torch.as_tensor(x["picked"][x["picked"] >= 0]).cuda()].double()
            for i in reversed(range(n)):                             # the crops, last request first
                if x["picked"][i] >= 0:
                    s = x["ids"][i]
                    for lb in range((length[s] + bs - 1) // bs - 1, (length[s] - 3 + bs - 1) // bs - 1, -1):
                        free.insert(0, table[s, lb])
                    length[s] -= 3
        row = row / torch.sqrt((row * row).mean(-1, keepdim=True) + 1e-5)
        K, V = (row @ Wk).view(n, H, D), (row @ Wv).view(n, H, D)
        at = torch.as_tensor(length[x["ids"]]).cuda().double()[:, None, None] * freq
        lo, hi = K[..., :D // 2], K[..., D // 2:]
        K = torch.cat([lo * at.cos() - hi * at.sin(), hi * at.cos() + lo * at.sin()], -1)
        for i in range(n):
            s = x["ids"][i]
            if length[s] % bs == 0:
                table[s, length[s] // bs] = free.pop(0)
            b, slot = int(table[s, length[s] // bs]), int(length[s] % bs)
            k_pool[b, :, slot], v_pool[b, :, :, slot] = K[i], V[i]
            length[s] += 1
    return dict(crop=None, rule=None, rows=None, state=None, err=None, block_table=None, lengths=None, free_top=None,
                cache_err=None, k_pool=k_pool, v_pool=v_pool)
