"""GPU K/V state of input rows at their compressed positions vs the oracle's,
and the projected append against the oracle's cache bookkeeping."""
import numpy as np
import pytest
import torch

from gpu_util import assert_same_state, TOL, dev, gpu_cache_like, i32, rel_l2_max, say
from paper_2609_27233_amd import lib as sm
from paper_2609_27233_amd import workload as wl

pytestmark = pytest.mark.gpu


def _setup(orc, H, D, lens, bs=16, extra=4, seed=0):
    mb = max(-(-L // bs) for L in lens) + 2
    oc = orc.OracleCache(bf16=True, num_kv_heads=H, head_dim=D, block_size=bs,
                         num_blocks=sum(-(-L // bs) for L in lens) + len(lens) + extra,
                         max_seqs=len(lens) + 1, max_blocks_per_seq=mb)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    g = wl.generator(seed)
    K = wl.randn((int(offs[-1]), H, D), torch.bfloat16, g)
    V = wl.randn((int(offs[-1]), H, D), torch.bfloat16, g)
    assert oc.append(np.arange(len(lens)), offs, wl.to_raw(K), wl.to_raw(V)) == orc.OK
    return oc, gpu_cache_like(oc, torch.bfloat16)


def _inputs(n, d, HD, seed):
    g = wl.generator(seed)
    x = wl.randn((n, d), torch.bfloat16, g)
    Wk = wl.randn((HD, d), torch.bfloat16, g, std=d ** -0.5)
    Wv = wl.randn((HD, d), torch.bfloat16, g, std=d ** -0.5)
    return x, Wk, Wv


CASES = [
    # H, D, d, lengths of the listed sequences
    (8, 128, 4096, [0, 1, 17, 2458, 2459, 4096, 31, 700, 9, 10, 11, 12, 13, 14, 15, 16]),
    (4, 128, 3584, [5] * 3 + [1000] * 62),          # two row groups (65 rows)
    (4, 64, 256, [300]),
    (8, 128, 4096, [131000]),                        # a far position: the angles need double precision
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_project_matches_oracle(orc, case):
    H, D, d, lens = CASES[case]
    bs = 16 if max(lens) < 10000 else 512
    oc, c = _setup(orc, H, D, lens, bs=bs, seed=case)
    n = len(lens)
    ids = np.random.RandomState(case).permutation(n).astype(np.int32)
    x, Wk, Wv = _inputs(n, d, H * D, 10 + case)
    K = torch.full((n, H, D), float("nan"), dtype=torch.bfloat16, device=dev())
    V = torch.full((n, H, D), float("nan"), dtype=torch.bfloat16, device=dev())
    say("kv_project", H, D, d, "n", n)
    sm.kv_project(c, i32(ids), x.to(dev()), Wk.to(dev()), Wv.to(dev()), K, V)
    torch.cuda.synchronize()
    st, Kr, Vr = oc.kv_project(ids, wl.to_f64(x), wl.to_f64(Wk), wl.to_f64(Wv))
    assert st == orc.OK
    ek = rel_l2_max(K.float().cpu().numpy(), Kr)
    ev = rel_l2_max(V.float().cpu().numpy(), Vr)
    say("rel_l2_max K", ek, "V", ev)
    assert ek <= TOL[torch.bfloat16] and ev <= TOL[torch.bfloat16]


def test_append_projected(orc):
    H, D, d = 8, 128, 4096
    lens = [37, 0, 16, 255]
    oc, c = _setup(orc, H, D, lens, seed=3)
    ids = np.array([3, 0, 2, 1], np.int32)
    x, Wk, Wv = _inputs(len(ids), d, H * D, 4)
    xd, Wkd, Wvd = x.to(dev()), Wk.to(dev()), Wv.to(dev())
    K = torch.empty((len(ids), H, D), dtype=torch.bfloat16, device=dev())
    V = torch.empty_like(K)
    sm.kv_project(c, i32(ids), xd, Wkd, Wvd, K, V)          # the rows at the positions before the append
    sm.kv_append_projected(c, i32(ids), xd, Wkd, Wvd)
    torch.cuda.synchronize()
    assert c.error_bits() == 0
    # the oracle appends the GPU's rows: the bookkeeping must agree exactly
    assert oc.append(ids, np.arange(len(ids) + 1, dtype=np.int32), wl.to_raw(K.cpu()), wl.to_raw(V.cpu())) == orc.OK
    assert np.array_equal(c.lengths.cpu().numpy()[:len(lens)], oc.lengths[:len(lens)])
    assert np.array_equal(c.block_table.cpu().numpy(), oc.block_table)
    k_pool, v_pool = c.k_pool.cpu(), c.v_pool.cpu()
    for s in ids:
        L = int(oc.lengths[s])
        blk = int(oc.block_table[s, (L - 1) // 16])
        j = (L - 1) % 16
        assert np.array_equal(wl.to_raw(k_pool[blk, :, j, :]), oc.k_pool[blk, :, j, :])
        assert np.array_equal(wl.to_raw(v_pool[blk, :, :, j]), oc.v_pool[blk, :, :, j])
    # and the appended rows match the oracle's projection at the old lengths
    oc2, _ = _setup(orc, H, D, lens, seed=3)
    st, Kr, Vr = oc2.kv_project(ids, wl.to_f64(x), wl.to_f64(Wk), wl.to_f64(Wv))
    assert st == orc.OK
    assert rel_l2_max(K.float().cpu().numpy(), Kr) <= TOL[torch.bfloat16]


def test_append_projected_bad_id_changes_nothing(orc):
    H, D, d = 4, 64, 256
    oc, c = _setup(orc, H, D, [10, 20], seed=5)
    x, Wk, Wv = _inputs(2, d, H * D, 6)
    before = (c.lengths.clone(), c.block_table.clone())
    sm.kv_append_projected(c, i32([0, 7]), x.to(dev()), Wk.to(dev()), Wv.to(dev()))
    torch.cuda.synchronize()
    assert c.error_bits() == sm.ERR_EINVAL
    assert torch.equal(c.lengths, before[0]) and torch.equal(c.block_table, before[1])


@pytest.mark.parametrize("n,H,D,d,bs", [(1, 8, 128, 1024, 16), (5, 2, 64, 256, 64), (65, 4, 128, 512, 16),
                                        (300, 4, 64, 256, 32)])
def test_append_projected_many_rows(orc, n, H, D, d, bs):
    """Rows straight into the pages: one to more requests than the metadata
    workgroup has threads, lengths on and off page edges, against the oracle's
    append of the rows that sm_kv_project gives."""
    rng = np.random.RandomState(n)
    lens = [int(v) for v in rng.choice([0, 1, bs - 1, bs, bs + 1, 3 * bs, 70], n)]
    oc, c = _setup(orc, H, D, lens, bs=bs, seed=n)
    ids = rng.permutation(n).astype(np.int32)
    x, Wk, Wv = _inputs(n, d, H * D, n)
    xd, Wkd, Wvd = x.to(dev()), Wk.to(dev()), Wv.to(dev())
    K = torch.empty((n, H, D), dtype=torch.bfloat16, device=dev())
    V = torch.empty_like(K)
    say("append projected", n, H, D, d, bs)
    sm.kv_project(c, i32(ids), xd, Wkd, Wvd, K, V)
    sm.kv_append_projected(c, i32(ids), xd, Wkd, Wvd)
    assert oc.append(ids, np.arange(n + 1, dtype=np.int32), wl.to_raw(K.cpu()), wl.to_raw(V.cpu())) == orc.OK
    assert_same_state(c, oc)


@pytest.mark.parametrize("what", ["repeat", "full stack", "no room", "largest int", "bad stack", "frozen"])
def test_append_projected_all_or_nothing(orc, what):
    """Each failing check of the append leaves the cache as it was."""
    H, D, d, bs = 4, 64, 256, 16
    oc, c = _setup(orc, H, D, [16, 20, 32], seed=8)
    ids, bit = [0, 1, 2], sm.ERR_EINVAL
    if what == "repeat":
        ids = [0, 1, 0]
    elif what == "full stack":
        c.free_top.fill_(1)                               # two rows begin a page
        bit = sm.ERR_ENOMEM
    elif what == "no room":
        c.lengths[1] = c.max_blocks * bs
        bit = sm.ERR_ERANGE
    elif what == "largest int":                           # length + 1 does not fit 32 bits
        c.lengths[1] = 2 ** 31 - 1
        bit = sm.ERR_ERANGE
    elif what == "bad stack":
        c.free_stack[int(c.free_top.item()) - 2] = c.num_blocks
    else:
        c.err.fill_(sm.ERR_ENOMEM)
        bit = sm.ERR_ENOMEM
    x, Wk, Wv = _inputs(3, d, H * D, 9)
    before = [t.clone() for t in (c.lengths, c.block_table, c.free_stack, c.free_top, c.k_pool, c.v_pool)]
    say("append projected fails:", what)
    sm.kv_append_projected(c, i32(ids), x.to(dev()), Wk.to(dev()), Wv.to(dev()))
    torch.cuda.synchronize()
    assert c.error_bits() == bit
    for t, b in zip((c.lengths, c.block_table, c.free_stack, c.free_top, c.k_pool, c.v_pool), before):
        assert torch.equal(t, b)
