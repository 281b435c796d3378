"""Prompt matching and pack indices at the edges of their pieces (256 and 1024
or 4096 positions of the whole batch, whatever the sequences' lengths), against
the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import dev, i32, say
from paper_2609_27233_amd import lib as sm

pytestmark = pytest.mark.gpu


def _rules(rng, count, V):
    out = np.full((count, 4), -1, np.int32)
    for r in range(count):
        n = rng.randint(2, 5)
        out[r, :n] = rng.randint(0, V, n)
    return out


MATCH = [
    # vocabulary, rules, lengths
    (5, 30, [255, 1, 256, 257, 0, 511, 2, 0, 0, 1]),      # sequences that end and start on block edges
    (3, 9, [256] * 5),
    (4, 12, [1] * 700),                                     # no window fits
    (6, 40, [3] * 2500),                                    # offsets beyond the LDS copy
    (4, 20, [70000, 5]),                                    # more blocks than threads that fold them
    (2, 3, [1023]),
    (5, 25, [524288]),                                      # as many positions as emit workgroups fold by themselves,
    (5, 25, [524288, 1]),                                   # one more,
    (3, 9, [300001, 0, 1, 700003, 1026, 99999]),            # more of them than threads of the scan,
    (4, 20, [251] * 2400),                                  # and the scan with offsets beyond the LDS copy
]


@pytest.mark.parametrize("case", range(len(MATCH)))
def test_match_prompt_block_edges(orc, case):
    V, nr, lens = MATCH[case]
    rng = np.random.RandomState(900 + case)
    rules = _rules(rng, nr, V)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(offs[-1]), len(lens)
    toks = rng.randint(0, V, T).astype(np.int32)
    st, s0, ln, ru, sso = orc.OracleRules(rules).match_prompt(toks, offs)
    assert st == orc.OK
    t = sm.RuleTable(sm.RuleTable.capacity_for(nr))
    sm.rules_build(t, i32(rules))
    out = [torch.full((T // 2 + 1,), -7, dtype=torch.int32, device=dev()) for _ in range(3)]
    gs = torch.full((B + 1,), -7, dtype=torch.int32, device=dev())
    ws = torch.empty(sm.match_prompt_workspace_bytes(B, T), dtype=torch.uint8, device=dev())
    say("match blocks", V, nr, lens[:10], "spans", len(s0))
    sm.match_prompt(t, i32(toks), i32(offs), *out, gs, ws)
    torch.cuda.synchronize()
    assert t.error_bits() == 0
    np.testing.assert_array_equal(gs.cpu().numpy(), sso)
    for got, ref in zip(out, (s0, ln, ru)):
        np.testing.assert_array_equal(got.cpu().numpy()[:len(s0)], ref)
        assert (got.cpu().numpy()[len(s0):] == -7).all()


def test_match_prompt_bad_offsets_keep_the_good_sequences(orc):
    """A sequence past the end of the tokens gets no spans and EINVAL; those
    before it get theirs."""
    rng = np.random.RandomState(5)
    rules = _rules(rng, 30, 5)
    toks = rng.randint(0, 5, 6000).astype(np.int32)
    good = np.array([0, 300, 5200], np.int32)
    st, s0, ln, ru, sso = orc.OracleRules(rules).match_prompt(toks[:5200], good)
    t = sm.RuleTable(sm.RuleTable.capacity_for(30))
    sm.rules_build(t, i32(rules))
    out = [torch.full((3000,), -7, dtype=torch.int32, device=dev()) for _ in range(3)]
    gs = torch.full((4,), -7, dtype=torch.int32, device=dev())
    ws = torch.empty(sm.match_prompt_workspace_bytes(3, 6000), dtype=torch.uint8, device=dev())
    say("match with a sequence out of range")
    sm.match_prompt(t, i32(toks), i32([0, 300, 5200, 6001]), *out, gs, ws)
    torch.cuda.synchronize()
    assert t.error_bits() == sm.ERR_EINVAL
    assert gs.cpu().tolist() == sso.tolist() + [len(s0)]
    for got, ref in zip(out, (s0, ln, ru)):
        np.testing.assert_array_equal(got.cpu().numpy()[:len(s0)], ref)


@pytest.mark.parametrize("B,T,tail", [(1, 700, [9]), (40, 3000, [1]), (700, 300, [1, 5]), (2100, 40, [3]),
                                      (3, 300000, [1])])
def test_match_prompt_bad_offsets_many_sequences(orc, B, T, tail):
    """Sequences past the end of the tokens after B good ones of up to T
    positions: more sequences than workgroups and fewer, than threads, than
    offsets in the LDS copy, and a batch whose entries are scanned."""
    rng = np.random.RandomState(B)
    rules = _rules(rng, 30, 5)
    lens = rng.randint(0, T + 1, B)
    good = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N = int(good[-1])
    toks = rng.randint(0, 5, N).astype(np.int32)
    st, s0, ln, ru, sso = orc.OracleRules(rules).match_prompt(toks, good)
    t = sm.RuleTable(sm.RuleTable.capacity_for(30))
    sm.rules_build(t, i32(rules))
    offs = np.concatenate([good, N + np.cumsum(tail)])
    out = [torch.full((N // 2 + 1,), -7, dtype=torch.int32, device=dev()) for _ in range(3)]
    gs = torch.full((len(offs),), -7, dtype=torch.int32, device=dev())
    ws = torch.empty(sm.match_prompt_workspace_bytes(len(offs) - 1, N), dtype=torch.uint8, device=dev())
    say("match with sequences out of range", B, T, "spans", len(s0))
    sm.match_prompt(t, i32(toks), i32(offs), *out, gs, ws)
    torch.cuda.synchronize()
    assert t.error_bits() == sm.ERR_EINVAL
    assert gs.cpu().tolist() == sso.tolist() + [len(s0)] * len(tail)
    for got, ref in zip(out, (s0, ln, ru)):
        np.testing.assert_array_equal(got.cpu().numpy()[:len(s0)], ref)
        assert (got.cpu().numpy()[len(s0):] == -7).all()


def test_match_prompt_overlapping_sequences_stay_in_the_outputs():
    """Offsets that go back: two good sequences over the same positions hold
    more spans than the outputs take; those past the end are dropped."""
    t = sm.RuleTable(16)
    sm.rules_build(t, i32([[0, 0, -1, -1]]))
    out = [torch.full((3001,), -7, dtype=torch.int32, device=dev()) for _ in range(3)]
    gs = torch.full((4,), -7, dtype=torch.int32, device=dev())
    ws = torch.empty(sm.match_prompt_workspace_bytes(3, 6000), dtype=torch.uint8, device=dev())
    say("match with overlapping sequences")
    sm.match_prompt(t, i32(np.zeros(6000)), i32([0, 4000, 1000, 6000]), *out, gs, ws)
    torch.cuda.synchronize()
    assert t.error_bits() == sm.ERR_EINVAL
    assert gs.cpu().tolist() == [0, 2000, 2000, 3000]
    start = out[0].cpu().numpy()
    np.testing.assert_array_equal(start[:3000], np.concatenate([np.arange(0, 4000, 2), np.arange(1000, 3000, 2)]))
    assert all(int(v[3000]) == -7 for v in out) and (out[1][:3000] == 2).all() and (out[2][:3000] == 0).all()


@pytest.mark.parametrize("offs", [
    [6005, 300, 5200, 6000],      # the first offset past the tokens: its sequence alone gets no spans
    [200, 100, 5200, 6000],       # or past the second one
    [2**31 - 1, 300, 5200, 6000],
    [-1, 300, 5200, 6000],
    [6005, 6005, 100, 6000],
    [300, 400, 0, 6000],          # a good sequence before the first one
    [2500, 2700, 0, 2500],
    [2500, 2700, 6000],           # no error: tokens before the first sequence
])
def test_match_prompt_bad_first_offset(offs):
    t = sm.RuleTable(16)
    sm.rules_build(t, i32([[0, 0, -1, -1]]))
    B = len(offs) - 1
    out = [torch.full((3001,), -7, dtype=torch.int32, device=dev()) for _ in range(3)]
    gs = torch.full((B + 1,), -7, dtype=torch.int32, device=dev())
    ws = torch.empty(sm.match_prompt_workspace_bytes(B, 6000), dtype=torch.uint8, device=dev())
    say("match with a bad first offset", offs)
    sm.match_prompt(t, i32(np.zeros(6000)), i32(offs), *out, gs, ws)
    torch.cuda.synchronize()
    good = [0 <= lo <= hi <= 6000 for lo, hi in zip(offs, offs[1:])]
    starts = [np.arange(lo, hi - 1, 2) if ok else np.arange(0) for ok, lo, hi in zip(good, offs, offs[1:])]
    want = np.concatenate(starts)[:3000]
    assert t.error_bits() == (0 if all(good) else sm.ERR_EINVAL)
    assert gs.cpu().tolist() == [0] + [min(n, 3000) for n in np.cumsum([len(s) for s in starts])]
    np.testing.assert_array_equal(out[0].cpu().numpy(), np.concatenate([want, np.full(3001 - len(want), -7)]))
    assert (out[1][:len(want)] == 2).all() and (out[2][:len(want)] == 0).all()


PACK = [
    # lengths, longest span
    ([1023, 1, 1024, 1025, 0, 2047, 2, 0], 8),
    ([1] * 3000, 1),                                        # one-token spans remove nothing
    ([7] * 4500, 5),                                        # offsets beyond the LDS copies
    ([5000, 3000], 2600),                                   # spans longer than a piece
    ([260000, 5000], 6),                                    # more than 256 pieces of 1024
    ([0, 0], 4),
    ([600000, 3, 0, 447000, 1573], 30),                     # as many pieces of 4096 as workgroups,
    ([600000, 3, 0, 447000, 1574], 30),                     # one more: two pieces each,
    ([3000, 900001, 1, 0, 1500000, 4095, 4097, 1] + [777] * 500, 60),   # three, sequences that begin in any of them,
    ([1200000, 1000000], 30000),                            # spans over several pieces,
    ([20] * 60000, 4),                                     # and offsets beyond the LDS copies
]


@pytest.mark.parametrize("case", range(len(PACK)))
def test_pack_piece_edges(orc, case):
    lens, nmax = PACK[case]
    rng = np.random.RandomState(950 + case)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    start, ln, sso = [], [], [0]
    for b, T in enumerate(lens):
        t = 0
        while t < T:
            n = int(min(T - t, rng.randint(1, nmax + 1)))
            if rng.rand() < 0.6:
                start.append(offs[b] + t)
                ln.append(n)
            t += n
        sso.append(len(start))
    start, ln, sso = (np.asarray(v, np.int32) for v in (start, ln, sso))
    T, B = int(offs[-1]), len(lens)
    st, res = orc.pack_spans(offs, start, ln, sso)
    assert st == orc.OK
    pi, src = (torch.full((max(T, 1),), -7, dtype=torch.int32, device=dev()) for _ in range(2))
    po = torch.full((B + 1,), -7, dtype=torch.int32, device=dev())
    err = torch.zeros(1, dtype=torch.int32, device=dev())
    say("pack pieces", lens[:8], "spans", len(start))
    if len(start):
        sm.pack_spans(i32(offs), i32(start), i32(ln), i32(sso), pi, po, src, err, T)
    else:                                                   # (no spans: any pointer will do)
        sm.pack_spans(i32(offs), i32([0])[:0], i32([0])[:0], i32(sso), pi, po, src, err, T)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    np.testing.assert_array_equal(po.cpu().numpy(), res["packed_offsets"])
    np.testing.assert_array_equal(pi.cpu().numpy()[:T], res["pi"])
    np.testing.assert_array_equal(src.cpu().numpy()[:po[-1].item()], res["packed_src"])


@pytest.mark.parametrize("S,rules", [(1, 3), (256, 4), (257, 1), (5000, 900), (131072, 60000), (131073, 60000),
                                     (1100000, 700000)])
def test_dedupe_block_edges(orc, S, rules):
    """Blocks of 256 spans; the last two cases have more blocks than the LDS prefix."""
    rng = np.random.RandomState(S)
    rule = rng.randint(0, rules, S).astype(np.int32)
    n_of = rng.randint(2, 5, rules)
    ln = n_of[rule].astype(np.int32)
    start = np.concatenate([[0], np.cumsum(ln)])[:-1].astype(np.int32)
    T = int(ln.sum())
    toks = rng.randint(0, 1000, T).astype(np.int32)
    # first span of each rule, in order of appearance
    uniq, first = np.unique(rule, return_index=True)
    order = np.sort(first)
    slot = np.empty(rules, np.int64)
    slot[rule[order]] = np.arange(len(order))
    rows = np.concatenate([toks[start[s]:start[s] + ln[s]] for s in order])
    out = {k: torch.full((m,), -7, dtype=torch.int32, device=dev())
           for k, m in (("uniq", S), ("slot", S), ("rows", T), ("offs", S + 1), ("n", 1))}
    err = torch.zeros(1, dtype=torch.int32, device=dev())
    say("dedupe", S, rules, "distinct", len(order))
    sm.span_dedupe(i32(rule), i32(start), i32(ln), rules, i32(toks), out["uniq"], out["slot"], out["rows"],
                   out["offs"], out["n"], err)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    assert int(err.item()) == 0 and got["n"][0] == len(order)
    np.testing.assert_array_equal(got["uniq"][:len(order)], order)
    np.testing.assert_array_equal(got["slot"], slot[rule])
    np.testing.assert_array_equal(got["offs"][:len(order) + 1], np.concatenate([[0], np.cumsum(ln[order])]))
    np.testing.assert_array_equal(got["rows"][:len(rows)], rows)
