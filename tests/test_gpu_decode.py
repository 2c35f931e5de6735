"""Parity of the HIP decode path (search, attention, merge) with the CPU oracle, through
the C ABI, on graphs built by the oracle (stage isolation). GPU only."""
import numpy as np
import pytest
import torch

import paper_2409_10516_amd as ra
from oracle import attention as OA, decode as OD, mips as OM, search as OS
from paper_2409_10516_amd import synth
from tests.util import (Tally, decode_matches, integer_valued, lse_close, oracle_graphs, out_close, to_np,
                        tol_for, topk_equivalent, walk_equivalent)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cases():
    return {
        "config0_small": lambda: synth.make_config0(N=1024, M=256, T=6, window=32),
        "llama_bf16": lambda: synth.make_llama_layer(11, N=1536, M=768, T=3, n_q=8, n_kv=2,
                                                     ef=64, topk=20, window=100),
        "llama_f32_2seq": lambda: synth.make_llama_layer(12, N=700, M=300, T=2, n_seq=2, n_q=4,
                                                         n_kv=4, dtype=torch.float32, ef=48,
                                                         topk=16, window=37, deg=12, knn=9),
        "integer_ties": lambda: synth.make_integer_case(5, N=200, M=64, T=5, d=128, n_q=2,
                                                        n_kv=1, deg=8, knn=6, topk=9, ef=20,
                                                        sink=3, window=10),
    }


_cache = {}


def _prepared(name):
    if name not in _cache:
        w = _cases()[name]()
        adj, ent, L = oracle_graphs(w)
        n_seq, n_kv = w.K.shape[:2]
        n_q = w.Q_prefill.shape[1]
        idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), n_seq, n_q, n_kv)
        _cache[name] = (w, adj, ent, idx, w.K.to(DEV), w.V.to(DEV))
    return _cache[name]


@pytest.mark.parametrize("name", list(_cases()))
@pytest.mark.parametrize("expand", [1, 4, 32, 64])
def test_search_against_the_float64_oracle(name, expand):
    """The walk against the oracle's walk with plain float64 inner products: ids and counters
    identical, except where the oracle took a decision between two scores closer than 1e-5
    relative (tests/util.py::walk_equivalent); integer-valued inputs allow no difference."""
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    W = OA.static_ids(N, w.sink, w.window)
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    tally = Tally()
    for t in range(w.q_decode.shape[0]):
        ids, st = ra.ra_search(w.q_decode[t].to(DEV), idx, Kd, w.sink, w.window, w.topk, w.ef,
                               expand)
        ids, st = ids.cpu().numpy(), st.cpu().numpy()
        for s in range(n_seq):
            for h in range(n_q):
                g = s * n_q + h
                K = to_np(w.K[s, h // (n_q // n_kv)])
                qq = to_np(w.q_decode[t, s, h])
                ref, rst = OS.greedy_search(qq, K, adj[g], ent[g], w.ef, w.topk, expand, exclude=W)
                tally.add(walk_equivalent(ids[s, h], st[s, h].tolist(), ref, rst, qq, K, W, exact=exact))
    tally.check()


@pytest.mark.parametrize("name", list(_cases()))
@pytest.mark.parametrize("expand", [1, 32])
def test_search_bit_exact_against_the_fixed_order_float32_scores(name, expand):
    """For float32 inputs the kernel adds its 128 products in a documented order; the oracle's opt-in
    float32 score adds in that order, and then every id and counter must agree with no allowance at
    all. (bf16 inputs go through the two-element dot instruction, whose internal rounding has no
    float32 formula: they are covered by the float64 rule alone, unless integer-valued.)"""
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    if w.K.dtype != torch.float32 and not integer_valued(to_np(w.K), to_np(w.q_decode)):
        pytest.skip("bf16 scores use the hardware's dot instruction; see the float64 test")
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    W = OA.static_ids(N, w.sink, w.window)
    for t in range(w.q_decode.shape[0]):
        ids, st = ra.ra_search(w.q_decode[t].to(DEV), idx, Kd, w.sink, w.window, w.topk, w.ef,
                               expand)
        ids, st = ids.cpu().numpy(), st.cpu().numpy()
        for s in range(n_seq):
            for h in range(n_q):
                g = s * n_q + h
                K = to_np(w.K[s, h // (n_q // n_kv)])
                ref, rst = OS.greedy_search(to_np(w.q_decode[t, s, h]), K, adj[g], ent[g], w.ef,
                                            w.topk, expand, exclude=W, score_fn=OS.score32)
                assert ids[s, h].tolist() == ref.tolist(), (name, expand, t, s, h)
                assert st[s, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"],
                                             rst["n_returned"]], (name, expand, t, s, h)


@pytest.mark.parametrize("name", list(_cases()))
def test_attend_matches_eq2_and_eq4(name):
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    W = OA.static_ids(N, w.sink, w.window)
    rng = np.random.default_rng(3)
    rest = np.setdiff1d(np.arange(N), W)
    topk = w.topk
    ids = -np.ones((n_seq, n_q, topk), np.int32)
    for s in range(n_seq):
        for h in range(n_q):
            n_valid = topk if (s + h) % 3 else topk - 3           # some rows are padded
            ids[s, h, :n_valid] = rng.choice(rest, size=n_valid, replace=False)
    q = w.q_decode[0]
    out, lse, oo, lo, ow, lw = [x.cpu().numpy() for x in ra.ra_attend(
        q.to(DEV), idx, Kd, Vd, w.sink, w.window, torch.from_numpy(ids).to(DEV), partials=True)]
    for s in range(n_seq):
        for h in range(n_q):
            K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
            qq = to_np(q[s, h])
            om = ids[s, h][ids[s, h] >= 0]
            r_oo, r_lo = OA.partial_attention(qq, K, V, om)
            r_ow, r_lw = OA.partial_attention(qq, K, V, W)
            r_o, r_l = OA.merge(r_ow, r_lw, r_oo, r_lo)
            assert out_close(oo[s, h], r_oo, tol) and lse_close(lo[s, h], r_lo, tol)
            assert out_close(ow[s, h], r_ow, tol) and lse_close(lw[s, h], r_lw, tol)
            assert out_close(out[s, h], r_o, tol) and lse_close(lse[s, h], r_l, tol)


@pytest.mark.parametrize("name", list(_cases()))
@pytest.mark.parametrize("expand", [1, 8])
def test_decode_step_end_to_end(name, expand):
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    tally = Tally()
    for t in range(w.q_decode.shape[0]):
        out, lse, ids, st = ra.ra_decode_step(w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, w.window,
                                              w.topk, w.ef, expand)
        out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
        for s in range(n_seq):
            for h in range(n_q):
                g = s * n_q + h
                K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
                tally.add(decode_matches(out[s, h], lse[s, h], ids[s, h], st[s, h].tolist(),
                                         to_np(w.q_decode[t, s, h]), K, V, adj[g], ent[g], w.sink,
                                         w.window, w.topk, w.ef, expand, tol, exact=exact))
    tally.check()


@pytest.mark.parametrize("name", list(_cases()))
def test_decode_step_with_a_budget_per_head(name):
    """ra_decode_step_budgets: every head keeps its own number of ids (values outside [1, topk] are
    clamped); each head must equal the oracle's decode step run with that head's budget, the rest
    of its ids row is -1 and n_returned counts what was kept."""
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    rng = np.random.default_rng(3)
    budgets = rng.integers(1, w.topk + 1, size=(n_seq, n_q)).astype(np.int32)
    budgets.flat[0] = 0                   # clamped to 1
    budgets.flat[-1] = w.topk + 7         # clamped to topk
    want = np.clip(budgets, 1, w.topk)
    out, lse, ids, st = ra.ra_decode_step(w.q_decode[0].to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk,
                                          w.ef, 8, topk_per_head=torch.from_numpy(budgets).to(DEV))
    out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    for s in range(n_seq):
        for h in range(n_q):
            g = s * n_q + h
            K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
            b = int(want[s, h])
            assert (ids[s, h, b:] == -1).all()
            assert st[s, h, 3] == int((ids[s, h] >= 0).sum())
            decode_matches(out[s, h], lse[s, h], ids[s, h, :b], st[s, h].tolist(),
                           to_np(w.q_decode[0, s, h]), K, V, adj[g], ent[g], w.sink, w.window, b, w.ef, 8,
                           tol, exact=exact)


@pytest.mark.parametrize("name", list(_cases()))
def test_decode_step_helper_modes_agree_with_oracle(name):
    """ra_index_configure: the attention over W by helper workgroups (default), by the heads
    themselves (RA_HELPERS_OFF), and after a bounded wait that runs out (RA_TEST_HELPERS_SILENT with a
    tiny spin limit: no helper ever reports, every head falls back and the handle stops using
    helpers) all give the oracle's result; ids and counters stay bit-exact."""
    from paper_2409_10516_amd import binding as B
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    turn = [0]

    def check():
        # a different query on every call: a record left over from the launch before
        # would carry the other query's attention over W and fail the comparison
        t = turn[0] % w.q_decode.shape[0]
        turn[0] += 1
        out, lse, ids, st = ra.ra_decode_step(w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk,
                                              w.ef, 8)
        out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
        for s in range(n_seq):
            for h in range(n_q):
                g = s * n_q + h
                K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
                decode_matches(out[s, h], lse[s, h], ids[s, h], st[s, h].tolist(), to_np(w.q_decode[t, s, h]),
                               K, V, adj[g], ent[g], w.sink, w.window, w.topk, w.ef, 8, tol, exact=exact)

    try:
        assert idx.helpers_active
        check(); check(); check()             # back to back: the records are cleared by their readers
        assert idx.helpers_active
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_OFF)
        assert not idx.helpers_active
        check()
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, 1)
        idx.configure(B.RA_CFG_HELPER_SPIN, 3)
        check()                               # every head's wait runs out
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)   # also forgets the wait that ran out
        idx.configure(B.RA_CFG_HELPER_SPIN, 20000)
        assert idx.helpers_active
        check()
    finally:
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)
        idx.configure(B.RA_CFG_HELPER_SPIN, 20000)


def test_helpers_switch_off_after_a_wait_that_ran_out():
    from paper_2409_10516_amd import binding as B
    w, adj, ent, idx, Kd, Vd = _prepared(next(iter(_cases())))
    q = w.q_decode[0].to(DEV)
    try:
        # mode ON with silent helpers cannot be had from outside; SILENT reports "not active", so
        # look at the outputs instead: after the timed-out call the results must still be right
        # with helpers nominally on, which they can only be if the heads no longer wait on them
        a = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 8)
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, 1)
        idx.configure(B.RA_CFG_HELPER_SPIN, 2)
        b = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 8)
        c = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 8)   # off word set: no waiting
        tol = tol_for(w.K.dtype)
        for x in (b, c):
            assert torch.equal(x[2], a[2])
            assert torch.allclose(x[0], a[0], rtol=0, atol=tol * float(a[0].abs().max()))
            assert torch.allclose(x[1], a[1], rtol=tol, atol=tol)
    finally:
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)
        idx.configure(B.RA_CFG_HELPER_SPIN, 20000)


@pytest.mark.parametrize("ef,topk", [(48, 16), (300, 40)])
def test_many_searches_use_smaller_workgroups(ef, topk):
    """More searches than compute units: the launch switches to 256-thread (ef <= 256) or
    512-thread workgroups. Ids and counters must not depend on that; attention within tolerance."""
    w = synth.make_llama_layer(21, N=640, M=192, T=1, n_seq=40, n_q=8, n_kv=2, ef=ef, topk=topk,
                               window=50, deg=16, knn=12)
    adj, ent, _ = oracle_graphs(w)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    assert n_seq * n_q > 256
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), n_seq, n_q, n_kv)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    q = w.q_decode[0].to(DEV)
    tol = tol_for(w.K.dtype)
    W = OA.static_ids(N, w.sink, w.window)
    ids_s, st_s = ra.ra_search(q, idx, Kd, w.sink, w.window, topk, ef, 8)
    out, lse, ids, st = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, topk, ef, 8)
    ids_s, st_s, ids, st = ids_s.cpu().numpy(), st_s.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    tally = Tally()
    for s in range(n_seq):
        for h in range(n_q):
            g = s * n_q + h
            K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
            # the stand-alone search and the fused step take the same walk
            assert ids_s[s, h].tolist() == ids[s, h].tolist() and st_s[s, h].tolist() == st[s, h].tolist()
            tally.add(decode_matches(out[s, h], lse[s, h], ids[s, h], st[s, h].tolist(),
                                     to_np(w.q_decode[0, s, h]), K, V, adj[g], ent[g], w.sink, w.window, topk,
                                     ef, 8, tol))
    tally.check()
    idx.free()


@pytest.mark.parametrize("expand", [16, 64])
def test_beam_wider_than_the_workgroup(expand):
    """ef = 1500 > 1024 threads (the top-2000 retrieval setting of Sec. 4 needs such beams): several
    beam entries per thread in the pick and the merge. Ids and counters bit-exact, attention within
    tolerance."""
    w = synth.make_config0(N=4096, M=512, T=2, window=64)
    adj, ent, _ = oracle_graphs(w)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    K, V = to_np(w.K[0, 0]), to_np(w.V[0, 0])
    tol = tol_for(w.K.dtype)
    ef, topk = 1500, 1200
    for t in range(2):
        q = w.q_decode[t].to(DEV)
        ids_s, st_s = ra.ra_search(q, idx, Kd, w.sink, w.window, topk, ef, expand)
        out, lse, ids, st = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, topk, ef, expand)
        assert torch.equal(ids_s, ids) and torch.equal(st_s, st)
        decode_matches(out[0, 0].cpu().numpy(), lse[0, 0].cpu().numpy(), ids[0, 0].cpu().numpy(),
                       st[0, 0].tolist(), to_np(w.q_decode[t, 0, 0]), K, V, adj[0], ent[0], w.sink, w.window,
                       topk, ef, expand, tol)
    idx.free()


@pytest.mark.parametrize("ef", [1, 15, 16, 17, 64, 65, 256, 257, 300, 769, 1024])
def test_merges_at_the_limits_of_beam_and_candidates(ef):
    """The two ways of merging a step's candidates and the 16-way search of the narrow one, at beams that
    end on, before and after a block of 16, 64 and 256 entries, with one to many picks per step (one to
    hundreds of candidates): ids and counters bit-exact, stand-alone and fused."""
    w, adj, ent, idx, Kd, Vd = _prepared("config0_small")
    K, W, topk = to_np(w.K[0, 0]), OA.static_ids(w.K.shape[2], w.sink, w.window), min(ef, 10)
    for t, expand in enumerate((1, 3, 7, 64)):
        q = w.q_decode[t].to(DEV)
        ids, st = ra.ra_search(q, idx, Kd, w.sink, w.window, topk, ef, expand)
        out, lse, ids_d, st_d = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, topk, ef, expand)
        assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
        ref, rst = OS.greedy_search(to_np(w.q_decode[t, 0, 0]), K, adj[0], ent[0], ef, topk, expand, exclude=W,
                                    score_fn=OS.score32)
        assert ids[0, 0].tolist() == ref.tolist(), (ef, expand)
        assert st[0, 0].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]


@pytest.mark.parametrize("distinct", [1, 3, 40, 3000])
@pytest.mark.parametrize("ef,expand,deg", [(20, 1, 9), (64, 16, 4), (100, 64, 40), (255, 33, 31), (257, 40, 40), (300, 64, 40),
                                           (700, 4, 40), (1300, 64, 40), (2048, 256, 12)])
def test_merges_of_any_size(ef, expand, deg, distinct):
    """Merges of one to some thousand candidates, by every way there is and into beams of every length on the way, of keys that
    all differ, that share a few scores, or that all have the same (a slot then holds every candidate, and more of them
    than the threads keep): ids and counters as the oracle has them, exactly, for integer inputs over a random graph."""
    rng, N = np.random.default_rng(ef + distinct), 3000
    K = rng.integers(-4, 5, size=(distinct, 128))[rng.integers(0, distinct, size=N) if distinct < N else np.arange(N)]
    adj = rng.integers(-1, N, size=(2, N, deg)).astype(np.int32)
    ent, q, topk = np.array([5, N - 1], np.int32), rng.integers(-4, 5, size=(2, 128)), min(ef, 50)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 2, 1)
    Kd = torch.from_numpy(K).to(torch.bfloat16).reshape(1, 1, N, 128).to(DEV)
    qd = torch.from_numpy(q).to(torch.bfloat16).reshape(1, 2, 128).to(DEV)
    W = OA.static_ids(N, 4, 100)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 100, topk, ef, expand)
    _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 100, topk, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    for h in range(2):
        ref, rst = OS.greedy_search(q[h].astype(np.float32), K.astype(np.float32), adj[h], int(ent[h]), ef, topk, expand, exclude=W)
        assert ids[0, h].tolist() == ref.tolist()
        assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]
    idx.free()


@pytest.mark.parametrize("n_q,n_kv,dtype", [(8, 1, torch.bfloat16), (4, 2, torch.bfloat16), (8, 1, torch.float32),
                                            (4, 1, torch.float32)])
def test_decode_step_other_group_sizes(n_q, n_kv, dtype):
    """GQA groups of 8 (the helper makes two passes over W; four with fp32), of 2, and of 4 with fp32
    inputs, against the oracle."""
    w = synth.make_llama_layer(31, N=900, M=256, T=2, n_q=n_q, n_kv=n_kv, dtype=dtype, ef=64, topk=24,
                               window=70, deg=16, knn=12)
    adj, ent, _ = oracle_graphs(w)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, n_q, n_kv)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    tol = tol_for(w.K.dtype)
    G = n_q // n_kv
    assert idx.helpers_active
    for t in range(2):
        out, lse, ids, st = ra.ra_decode_step(w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk,
                                              w.ef, 8)
        out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
        for h in range(n_q):
            K = to_np(w.K[0, h // G]); V = to_np(w.V[0, h // G])
            decode_matches(out[0, h], lse[0, h], ids[0, h], st[0, h].tolist(), to_np(w.q_decode[t, 0, h]), K, V,
                           adj[h], ent[h], w.sink, w.window, w.topk, w.ef, 8, tol)
    assert idx.helpers_active          # no wait ran out
    idx.free()


def test_exhaustive_beam_equals_bruteforce_and_full_attention():
    """ef >= N: the search returns the exact top-k; with topk covering every non-static key
    the decode output is Eq. 1 over the whole context."""
    w = synth.make_integer_case(9, N=300, M=80, T=3, d=128, deg=8, knn=6, topk=5, ef=300,
                                sink=4, window=20)
    adj, ent, _ = oracle_graphs(w)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    K, V = to_np(w.K[0, 0]), to_np(w.V[0, 0])
    W = OA.static_ids(300, 4, 20)
    for t in range(3):
        q = w.q_decode[t].to(DEV)
        ids, st = ra.ra_search(q, idx, Kd, 4, 20, 7, 300, 5)
        assert ids[0, 0].tolist() == OM.topk_bruteforce(to_np(q[0, 0]), K, 7, exclude=W).tolist()
        assert int(st[0, 0, 0]) == 300
        out, lse, ids, _ = ra.ra_decode_step(q, idx, Kd, Vd, 4, 20, 276, 300, 3)
        ref_o, ref_l = OA.full_attention(to_np(q[0, 0]), K, V)
        assert sorted(ids[0, 0].tolist()) == list(range(4, 280))
        assert out_close(out[0, 0].cpu().numpy(), ref_o, 1e-5)
        assert lse_close(float(lse[0, 0]), ref_l, 1e-5)


@pytest.mark.parametrize("sink,window,topk", [(0, 0, 8), (500, 0, 8), (0, 500, 8), (7, 1, 60),
                                              (2, 3, 40)])
def test_edge_static_sets_and_padding(sink, window, topk):
    w = synth.make_integer_case(2, N=70, M=30, T=2, d=128, deg=6, knn=5)
    adj, ent, _ = oracle_graphs(w)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    K, V = to_np(w.K[0, 0]), to_np(w.V[0, 0])
    for t in range(2):
        q = w.q_decode[t].to(DEV)
        out, lse, ids, st = ra.ra_decode_step(q, idx, Kd, Vd, sink, window, topk, 64, 2)
        r_out, r_lse, r_ids, rst = OD.decode_step(to_np(q[0, 0]), K, V, adj[0], ent[0], sink, window,
                                                  topk, 64, 2)
        assert ids[0, 0].tolist() == r_ids.tolist()
        assert int(st[0, 0, 3]) == rst["n_returned"]
        assert out_close(out[0, 0].cpu().numpy(), r_out, 1e-5)
        assert lse_close(float(lse[0, 0]), r_lse, 1e-5)


def test_argument_errors_reach_python():
    w, adj, ent, idx, Kd, Vd = _prepared("integer_ties")
    q = w.q_decode[0].to(DEV)
    with pytest.raises(ra.RaError) as e:
        ra.ra_search(q, idx, Kd, 0, 0, 10, 5, 1)          # ef < topk
    assert e.value.status == 1
    with pytest.raises(ra.RaError) as e:
        ra.ra_search(q, idx, Kd[:, :, :100].contiguous(), 0, 0, 5, 10, 1)    # N mismatch
    assert e.value.status == 2


@pytest.mark.parametrize("grown,capacity_pad,window", [(1, 0, 64), (37, 19, 64), (200, 5, 16), (90, 0, 0)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_decode_after_generation_appended_tokens(grown, capacity_pad, window, dtype):
    """The index covers the first N_index tokens; the cache has grown by `grown` tokens and has
    spare capacity. Appended tokens are attended densely; ids come from the graph."""
    n_index, n_q, n_kv = 900, 4, 2
    N = n_index + grown
    w = synth.make_llama_layer(51, N=N, M=400, T=2, n_q=n_q, n_kv=n_kv, dtype=dtype, ef=48, topk=16,
                               window=window, deg=12, knn=9)
    from types import SimpleNamespace
    wi = SimpleNamespace(K=w.K[:, :, :n_index].contiguous(), Q_prefill=w.Q_prefill, knn=w.knn, deg=w.deg)
    adj, ent, _ = oracle_graphs(wi)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, n_q, n_kv)
    cap = N + capacity_pad
    Kc = torch.zeros((1, n_kv, cap, 128), dtype=dtype); Kc[:, :, :N] = w.K
    Vc = torch.full((1, n_kv, cap, 128), 7.0, dtype=dtype); Vc[:, :, :N] = w.V
    Kd, Vd = Kc.to(DEV), Vc.to(DEV)
    tol = tol_for(dtype)
    for t in range(2):
        out, lse, ids, st = ra.ra_decode_step(w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, window, w.topk,
                                              w.ef, 4, n_tokens=N)
        out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
        for h in range(n_q):
            K = to_np(w.K[0, h // 2]); V = to_np(w.V[0, h // 2])
            assert (ids[0, h] < n_index).all()
            decode_matches(out[0, h], lse[0, h], ids[0, h], st[0, h].tolist(), to_np(w.q_decode[t, 0, h]), K, V,
                           adj[h], ent[h], w.sink, window, w.topk, w.ef, 4, tol, n_index=n_index)
    with pytest.raises(ra.RaError) as e:
        ra.ra_decode_step(w.q_decode[0].to(DEV), idx, Kd, Vd, w.sink, window, w.topk, w.ef, 4,
                          n_tokens=n_index - 1)
    assert e.value.status == 2


def test_grown_cache_with_everything_retrieved_is_full_attention():
    n_index, grown = 300, 25
    w = synth.make_integer_case(19, N=n_index + grown, M=80, T=2, d=128, deg=8, knn=6)
    from types import SimpleNamespace
    wi = SimpleNamespace(K=w.K[:, :, :n_index].contiguous(), Q_prefill=w.Q_prefill, knn=6, deg=8)
    adj, ent, _ = oracle_graphs(wi)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    for t in range(2):
        q = w.q_decode[t].to(DEV)
        out, lse, ids, _ = ra.ra_decode_step(q, idx, Kd, Vd, 4, 20, 296, 300, 3, n_tokens=n_index + grown)
        ref_o, ref_l = OA.full_attention(to_np(q[0, 0]), to_np(w.K[0, 0]), to_np(w.V[0, 0]))
        assert sorted(ids[0, 0].tolist()) == list(range(4, 300))
        assert out_close(out[0, 0].cpu().numpy(), ref_o, 1e-5) and lse_close(float(lse[0, 0]), ref_l, 1e-5)


@pytest.mark.parametrize("name", list(_cases()))
@pytest.mark.parametrize("n_seeds,expand", [(1, 4), (7, 8), (100, 32), (300, 64), (2048, 256)])
def test_walks_from_a_seed_set(name, n_seeds, expand):
    """RA_CFG_SEEDS: the device lists the seed sets from the graph alone (the oracle's
    backbone_seeds), starts every walk from them, and counts no step for them. ra_search and
    ra_decode_step against the oracle's seeded walk; a seed set that does not fit one step's
    candidate arrays is refused; 0 restores the single-entry walk."""
    from paper_2409_10516_amd import binding as B
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    W = OA.static_ids(N, w.sink, w.window)
    ef = max(w.ef, 24)
    try:
        idx.configure(B.RA_CFG_SEEDS, n_seeds)
        assert idx.n_seeds == min(n_seeds, N)
        if idx.n_seeds > expand * idx.deg:
            with pytest.raises(ra.RaError) as e:
                ra.ra_search(w.q_decode[0].to(DEV), idx, Kd, w.sink, w.window, w.topk, ef, expand)
            assert e.value.status == 1 and "n_seeds" in str(e.value)
            return
        tally = Tally()
        for t in range(min(3, w.q_decode.shape[0])):
            q = w.q_decode[t].to(DEV)
            ids_s, st_s = ra.ra_search(q, idx, Kd, w.sink, w.window, w.topk, ef, expand)
            out, lse, ids, st = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, w.topk, ef, expand)
            assert torch.equal(ids_s, ids) and torch.equal(st_s, st)
            out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
            for s in range(n_seq):
                for h in range(n_q):
                    g = s * n_q + h
                    K = to_np(w.K[s, h // (n_q // n_kv)]); V = to_np(w.V[s, h // (n_q // n_kv)])
                    tally.add(decode_matches(out[s, h], lse[s, h], ids[s, h], st[s, h].tolist(),
                                             to_np(w.q_decode[t, s, h]), K, V, adj[g], ent[g], w.sink, w.window,
                                             w.topk, ef, expand, tol, exact=exact, n_seeds=n_seeds))
        tally.check()
        if n_seeds == 100:
            with pytest.raises(ra.RaError) as e:      # 100 seeds do not fit one expansion's candidates
                ra.ra_search(w.q_decode[0].to(DEV), idx, Kd, w.sink, w.window, w.topk, ef, 1)
            assert e.value.status == 1 and "n_seeds" in str(e.value)
    finally:
        idx.configure(B.RA_CFG_SEEDS, 0)
    assert idx.n_seeds == 0


@pytest.mark.parametrize("name", ["llama_bf16", "llama_f32_2seq", "integer_ties"])
def test_seed_shares_give_the_heads_the_same_keys(name):
    """RA_CFG_SEED_SHARES: the start sets of ra_decode_step scored by workgroups of their own (2 to 8
    shares per head, sets that do not divide evenly, sets with fewer ids than configured) or by the
    heads themselves (0) must give the same ids, counters and outputs, bit for bit - the keys are
    the same bits either way - on different queries back to back (a key left over from the launch
    before would belong to another query), and equal the oracle's seeded walk. A wait that runs out
    (silent seed workgroups, tiny spin limit) falls back to scoring in the head and switches the
    shares off until the helpers are configured again."""
    from paper_2409_10516_amd import binding as B
    w, adj, ent, idx, Kd, Vd = _prepared(name)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    tol = tol_for(w.K.dtype)
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    ef = max(w.ef, 24)
    T = w.q_decode.shape[0]
    turn = [0]

    def step(expand):
        t = turn[0] % T
        turn[0] += 1
        return t, ra.ra_decode_step(w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk, ef, expand)

    def same(a, b):
        return all(torch.equal(x, y) for x, y in zip(a, b))

    try:
        for n_seeds, expand in ((7, 8), (150, 32), (1000, 64)):
            idx.configure(B.RA_CFG_SEEDS, n_seeds)
            idx.configure(B.RA_CFG_SEED_SHARES, 0)
            assert not idx.seed_shares_active
            ref = {}
            for _ in range(T):
                t, r = step(expand)
                ref[t] = r
            # the oracle's walk, once per size
            out, lse, ids, st = (x.cpu().numpy() for x in ref[0])
            for s_ in range(n_seq):
                for h in range(n_q):
                    g = s_ * n_q + h
                    K = to_np(w.K[s_, h // (n_q // n_kv)]); V = to_np(w.V[s_, h // (n_q // n_kv)])
                    decode_matches(out[s_, h], lse[s_, h], ids[s_, h], st[s_, h].tolist(), to_np(w.q_decode[0, s_, h]),
                                   K, V, adj[g], ent[g], w.sink, w.window, w.topk, ef, expand, tol, exact=exact,
                                   n_seeds=n_seeds)
            for shares in (2, 3, 4, 8):
                idx.configure(B.RA_CFG_SEED_SHARES, shares)
                assert idx.seed_shares_active
                for _ in range(T + 1):
                    t, r = step(expand)
                    assert same(r, ref[t]), (n_seeds, shares, t)
                assert idx.seed_shares_active              # no wait ran out
        # a wait that runs out: nothing arrives, the heads score their sets themselves
        idx.configure(B.RA_CFG_SEED_SHARES, 4)
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, 1)
        idx.configure(B.RA_CFG_HELPER_SPIN, 2)
        t, r = step(64)
        assert same(r[2:], ref[t][2:])                      # ids and counters; W is attended by the heads now
        assert torch.allclose(r[0], ref[t][0], rtol=0, atol=tol * float(ref[t][0].abs().max()))
        t, r = step(64)                                     # the off word is set: no head waits any more
        assert same(r[2:], ref[t][2:])
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, 0)     # also forgets the wait that ran out
        idx.configure(B.RA_CFG_HELPER_SPIN, 20000)
        assert idx.seed_shares_active
        for _ in range(2):
            t, r = step(64)
            assert same(r, ref[t])
        assert idx.seed_shares_active
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_OFF)   # no extra workgroups of either kind
        assert not idx.seed_shares_active
        t, r = step(64)
        assert same(r[2:], ref[t][2:])
    finally:
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, 0)
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)
        idx.configure(B.RA_CFG_HELPER_SPIN, 20000)
        idx.configure(B.RA_CFG_SEED_SHARES, 6)
        idx.configure(B.RA_CFG_SEEDS, 0)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_seed_shares_in_the_variants_of_the_decode_step(dtype):
    """The decode step over 8-bit keys, with a budget per head, and on a cache that has grown past the
    index (spare capacity: the key rows of a KV head start every `capacity` rows), each with the
    start sets scored by seed workgroups and by the heads: same ids, counters and outputs, bit for
    bit, on two queries in turn; the 8-bit walk also equals ra_search over the same keys."""
    from paper_2409_10516_amd import binding as B
    n_index, grown, pad, n_q, n_kv = 1100, 40, 13, 4, 2
    N = n_index + grown
    w = synth.make_llama_layer(71, N=N, M=500, T=2, n_q=n_q, n_kv=n_kv, dtype=dtype, ef=64, topk=20,
                               window=50, deg=16, knn=12)
    from types import SimpleNamespace
    wi = SimpleNamespace(K=w.K[:, :, :n_index].contiguous(), Q_prefill=w.Q_prefill, knn=w.knn, deg=w.deg)
    adj, ent, _ = oracle_graphs(wi)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, n_q, n_kv)
    Ki, Vi = wi.K.to(DEV), w.V[:, :, :n_index].contiguous().to(DEV)
    k8 = ra.ra_quantize_keys(Ki)
    Kc = torch.zeros((1, n_kv, N + pad, 128), dtype=dtype); Kc[:, :, :N] = w.K
    Vc = torch.zeros((1, n_kv, N + pad, 128), dtype=dtype); Vc[:, :, :N] = w.V
    Kc, Vc = Kc.to(DEV), Vc.to(DEV)
    budgets = torch.tensor([[3, 20, 1, 11]], dtype=torch.int32, device=DEV)
    idx.configure(B.RA_CFG_SEEDS, 333)
    variants = {
        "q8": lambda q: ra.ra_decode_step(q, idx, Ki, Vi, w.sink, w.window, w.topk, w.ef, 32, k8=k8),
        "budgets": lambda q: ra.ra_decode_step(q, idx, Ki, Vi, w.sink, w.window, w.topk, w.ef, 32,
                                               topk_per_head=budgets),
        "grown": lambda q: ra.ra_decode_step(q, idx, Kc, Vc, w.sink, w.window, w.topk, w.ef, 32, n_tokens=N),
    }
    for name, fn in variants.items():
        ref = []
        idx.configure(B.RA_CFG_SEED_SHARES, 0)
        for t in range(2):
            ref.append(fn(w.q_decode[t].to(DEV)))
        idx.configure(B.RA_CFG_SEED_SHARES, 4)
        assert idx.seed_shares_active
        for t in (0, 1, 0):
            got = fn(w.q_decode[t].to(DEV))
            assert all(torch.equal(x, y) for x, y in zip(got, ref[t])), (name, t)
        assert idx.seed_shares_active, name
    ids8, st8 = ra.ra_search(w.q_decode[1].to(DEV), idx, Ki, w.sink, w.window, w.topk, w.ef, 32, k8=k8)
    got = variants["q8"](w.q_decode[1].to(DEV))
    assert torch.equal(got[2], ids8) and torch.equal(got[3], st8)
    idx.free()


def test_seed_shares_replayed_from_a_graph():
    """The launch with seed workgroups captured in a HIP graph and replayed with eager launches in
    between: every replay must leave the key slots as it found them (zero), so each gives the
    eager result."""
    from paper_2409_10516_amd import binding as B
    w, adj, ent, idx, Kd, Vd = _prepared("llama_bf16")
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    try:
        idx.configure(B.RA_CFG_SEEDS, 600)
        idx.configure(B.RA_CFG_SEED_SHARES, 4)
        q0, q1 = w.q_decode[0].to(DEV), w.q_decode[1].to(DEV)
        e0 = ra.ra_decode_step(q0, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64)
        e1 = ra.ra_decode_step(q1, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64)
        f32 = dict(dtype=torch.float32, device=DEV)
        out = torch.empty((n_seq, n_q, d), **f32); lse = torch.empty((n_seq, n_q), **f32)
        ids = torch.empty((n_seq, n_q, w.topk), dtype=torch.int32, device=DEV)
        st = torch.zeros((n_seq, n_q, 4), dtype=torch.int32, device=DEV)
        qbuf = q0.clone()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        cs = torch.cuda.Stream()
        with torch.cuda.stream(cs):
            ra.ra_decode_step(qbuf, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64, out=out, lse=lse, ids=ids, stats=st)
            cs.synchronize()
            with torch.cuda.graph(g, stream=cs):
                ra.ra_decode_step(qbuf, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64, out=out, lse=lse, ids=ids,
                                  stats=st)
        torch.cuda.synchronize()
        for rep in range(4):
            src, want = (q0, e0) if rep % 2 == 0 else (q1, e1)
            qbuf.copy_(src)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(ids, want[2]) and torch.equal(st, want[3]), rep
            assert torch.equal(out, want[0]) and torch.equal(lse, want[1]), rep
            mid = ra.ra_decode_step(q1 if rep % 2 == 0 else q0, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64)
            assert torch.equal(mid[2], (e1 if rep % 2 == 0 else e0)[2])
        assert idx.seed_shares_active
    finally:
        idx.configure(B.RA_CFG_SEEDS, 0)


def test_seed_sets_of_a_graph_with_missing_and_repeated_nodes():
    """An imported graph need not be a projection: slots 0 and 1 may hold -1 or lead back to a node
    already listed. The device's seed list must be the oracle's (checked through the walk: with ef
    and expand covering everything, n_visited after zero steps is the number of distinct seeds)."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(5)
    N, deg = 200, 4
    adj = rng.integers(-1, N, size=(1, N, deg)).astype(np.int32)
    adj[0, np.arange(N), 0] = np.where(adj[0, :, 0] == np.arange(N), -1, adj[0, :, 0])
    for j in range(deg):
        adj[0, adj[0, :, j] == np.arange(N), j] = -1
    adj[0, 7, 0] = -1
    adj[0, 7, 1] = 7 + 1
    ent = np.array([7], np.int32)
    K = torch.from_numpy(rng.integers(-3, 4, size=(1, 1, N, 128)).astype(np.float32))
    q = torch.from_numpy(rng.integers(-3, 4, size=(1, 1, 128)).astype(np.float32))
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    for R in (1, 2, 5, 33, 64):
        idx.configure(B.RA_CFG_SEEDS, R)
        seeds = OS.backbone_seeds(adj[0], 7, R)
        ids, st = ra.ra_search(q.to(DEV), idx, K.to(DEV), 0, 0, 10, 200, 64)
        ref, rst = OS.greedy_search(to_np(q[0, 0]), to_np(K[0, 0]), adj[0], 7, 200, 10, 64, seeds=seeds)
        assert ids[0, 0].tolist() == ref.tolist(), R
        assert st[0, 0].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]], R
    idx.free()


@pytest.mark.parametrize("n_q,n_kv,dtype", [(6, 2, torch.bfloat16), (5, 1, torch.float32), (12, 4, torch.bfloat16)])
def test_group_sizes_the_kernels_are_not_specialised_for(n_q, n_kv, dtype):
    """GQA groups of 3 and 5 query heads per KV head: ra_decode_step runs without helper workgroups,
    ra_attend and ra_flat_topk read the rows once per query head. All against the oracle."""
    w = synth.make_llama_layer(33, N=800, M=200, T=2, n_q=n_q, n_kv=n_kv, dtype=dtype, ef=48, topk=20,
                               window=60, deg=12, knn=10)
    adj, ent, _ = oracle_graphs(w)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, n_q, n_kv)
    Kd, Vd = w.K.to(DEV), w.V.to(DEV)
    tol = tol_for(dtype)
    G = n_q // n_kv
    N = 800
    W = OA.static_ids(N, w.sink, w.window)
    for t in range(2):
        q = w.q_decode[t].to(DEV)
        out, lse, ids, st = ra.ra_decode_step(q, idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 8)
        ids_s, _ = ra.ra_search(q, idx, Kd, w.sink, w.window, w.topk, w.ef, 8)
        o2, l2 = ra.ra_attend(q, idx, Kd, Vd, w.sink, w.window, ids_s)
        flat = ra.ra_flat_topk(q, Kd, w.sink, w.window, w.topk).cpu().numpy()
        assert torch.equal(ids, ids_s)
        out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
        o2, l2 = o2.cpu().numpy(), l2.cpu().numpy()
        for h in range(n_q):
            K = to_np(w.K[0, h // G]); V = to_np(w.V[0, h // G])
            qq = to_np(w.q_decode[t, 0, h])
            decode_matches(out[0, h], lse[0, h], ids[0, h], st[0, h].tolist(), qq, K, V, adj[h], ent[h], w.sink,
                           w.window, w.topk, w.ef, 8, tol)
            decode_matches(o2[0, h], l2[0, h], ids[0, h], None, qq, K, V, adj[h], ent[h], w.sink,
                           w.window, w.topk, w.ef, 8, tol)
            ref = OM.topk_bruteforce(qq, K, w.topk, exclude=W)
            topk_equivalent(flat[0, h], ref, qq, K)
    assert not idx.helpers_active
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_root_set_much_larger_than_the_beam(dtype):
    """A wide graph (deg 64) walked with a narrow beam: the root set (the entry point, its neighbours
    and theirs, the first 65 entering as expanded) is far larger than ef, so
    the step that scores it goes through the pre-filter that drops hopeless candidates ahead of the
    merge. Ids and counters against the oracle's two ordinary steps; real-valued and tie-laden inputs."""
    for w in (synth.make_llama_layer(61, N=6000, M=1500, T=3, n_q=2, n_kv=1, dtype=dtype, ef=66, topk=30,
                                     window=50, deg=64, knn=40),
              synth.make_integer_case(62, N=3000, M=800, T=3, d=128, n_q=1, n_kv=1, dtype=dtype, lo=-2, hi=2,
                                      deg=64, knn=40, topk=30, ef=66, sink=3, window=10)):
        adj, ent, _ = oracle_graphs(w)
        n_q = w.Q_prefill.shape[1]
        idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, n_q, 1)
        Kd, Vd = w.K.to(DEV), w.V.to(DEV)
        tol = tol_for(dtype)
        exact = integer_valued(to_np(w.K), to_np(w.q_decode))
        for t in range(3):
            out, lse, ids, st = [x.cpu().numpy() for x in ra.ra_decode_step(
                w.q_decode[t].to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 64)]
            for h in range(n_q):
                first = [int(x) for x in adj[h][ent[h]] if x >= 0]
                root = {int(ent[h]), *first, *(int(x) for a in first for x in adj[h][a] if x >= 0)}
                assert len(first) + 1 <= w.ef and len(root) > w.ef + 64      # the pre-filter's condition
                decode_matches(out[0, h], lse[0, h], ids[0, h], st[0, h].tolist(), to_np(w.q_decode[t, 0, h]),
                               to_np(w.K[0, 0]), to_np(w.V[0, 0]), adj[h], ent[h], w.sink, w.window, w.topk,
                               w.ef, 64, tol, exact=exact)
        idx.free()


@pytest.mark.parametrize("deg,expand,ef", [(32, 32, 64), (32, 32, 500), (31, 33, 64), (24, 256, 25), (64, 64, 900)])
@pytest.mark.parametrize("spread", [1, 1000])
def test_root_sets_ordered_by_bins(deg, expand, ef, spread):
    """Root sets beyond the pre-filter's limit (float32) are ordered through bins of their scores where a step has 1024 cells or more
    (31 * 33 are 1023), with ties by the dozen (spread 1) and with all but one key in the lowest bins (spread 1000).
    Integer inputs, so ids and counters are the oracle's."""
    rng = np.random.default_rng(deg * expand + ef)
    N = 3000
    adj = np.stack([rng.permutation(N)[:deg] for _ in range(N)]).astype(np.int32)[None]
    adj[0, ::5, 3] = -1
    ent = np.array([17], np.int32)
    first = [int(x) for x in adj[0][17] if x >= 0]
    root = {17, *first, *(int(x) for a in first for x in adj[0][a] if x >= 0)}
    assert len(root) > ef + 64 and expand >= len(first)
    K = rng.integers(-1, 2, size=(1, 1, N, 128)).astype(np.float32)
    K[0, 0, first[0]] *= spread
    K = torch.from_numpy(K)
    V = torch.from_numpy(rng.standard_normal((1, 1, N, 128)).astype(np.float32))
    q = torch.from_numpy(rng.integers(-1, 2, size=(1, 1, 128)).astype(np.float32))
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    out, lse, ids, st = ra.ra_decode_step(q.to(DEV), idx, K.to(DEV), V.to(DEV), 2, 5, 20, ef, expand)
    ids_s, st_s = ra.ra_search(q.to(DEV), idx, K.to(DEV), 2, 5, 20, ef, expand)
    assert torch.equal(ids_s, ids) and torch.equal(st_s, st)
    decode_matches(out[0, 0].cpu().numpy(), float(lse[0, 0]), ids[0, 0].tolist(), st[0, 0].tolist(), to_np(q[0, 0]),
                   to_np(K[0, 0]), to_np(V[0, 0]), adj[0], 17, 2, 5, 20, ef, expand, 1e-5, exact=True)
    idx.free()


@pytest.mark.parametrize("expand", [2, 8, 256])
def test_graphs_of_degree_one(expand):
    """The smallest degree an imported graph can have: one adjacency cell per pick. A walk has several picks
    at once there only when it starts from a seed set (a chain of keys): each pick's own cell has to
    be read. Integer inputs, so ids and counters are the oracle's."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(9)
    N = 400
    ring = rng.permutation(N)
    adj = np.empty((1, N, 1), np.int32)
    adj[0, ring, 0] = np.roll(ring, -1)
    adj[0, ring[300], 0] = -1
    ent = np.array([ring[0]], np.int32)
    K = torch.from_numpy(rng.integers(-3, 4, size=(1, 1, N, 128)).astype(np.float32))
    V = torch.from_numpy(rng.standard_normal((1, 1, N, 128)).astype(np.float32))
    q = torch.from_numpy(rng.integers(-3, 4, size=(1, 1, 128)).astype(np.float32))
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, 1, 1)
    for n_seeds in (0, 2, expand):
        idx.configure(B.RA_CFG_SEEDS, n_seeds)
        for ef in (16, 350):
            out, lse, ids, st = ra.ra_decode_step(q.to(DEV), idx, K.to(DEV), V.to(DEV), 2, 5, 10, ef, expand)
            ids_s, st_s = ra.ra_search(q.to(DEV), idx, K.to(DEV), 2, 5, 10, ef, expand)
            assert torch.equal(ids_s, ids) and torch.equal(st_s, st)
            decode_matches(out[0, 0].cpu().numpy(), float(lse[0, 0]), ids[0, 0].tolist(), st[0, 0].tolist(),
                           to_np(q[0, 0]), to_np(K[0, 0]), to_np(V[0, 0]), adj[0], int(ent[0]), 2, 5, 10, ef, expand,
                           1e-5, exact=True, n_seeds=n_seeds)
    idx.free()


@pytest.mark.parametrize("dtype,n_q,deg,expand,ef,seeds,q8", [
    (torch.bfloat16, 1, 64, 64, 1024, 0, False),       # 4096 cells, the most a worker answers for; 16 workers
    (torch.bfloat16, 20, 24, 128, 512, 1500, False),   # 8 workers, three rows of workgroups per compute die, seed sets
    (torch.float32, 3, 63, 64, 1024, 0, False),        # rows of no multiple of four cells
    (torch.float32, 2, 64, 48, 600, 0, False),         # fewer picks than the entry point has neighbours: no start set
    (torch.bfloat16, 2, 48, 64, 512, 2048, True)])     # 8-bit keys
def test_walks_that_share_their_steps(dtype, n_q, deg, expand, ef, seeds, q8):
    """Walks whose visited set is in device memory claim and score through workers of their own in ra_decode_step:
    ids and counters are those of ra_search, which walks alone, in repeated calls and when no worker answers. The
    first search's messages say that its steps were shared: one each, and one when the walk ended (a start set's
    step, and the first two of a walk from a root set, need none)."""
    from paper_2409_10516_amd import binding as B
    N, topk = 1_100_003, 100
    g = torch.Generator(device=DEV).manual_seed(deg * 1000 + n_q)
    adj = torch.randint(-1, N, (n_q, N, deg), generator=g, device=DEV, dtype=torch.int32)
    adj[:, ::7, 5:] = -1
    entry = torch.randint(0, N, (n_q,), generator=g, device=DEV, dtype=torch.int32)
    idx = ra.ra_index_import(adj.cpu(), entry.cpu(), 1, n_q, 1)
    del adj
    K = torch.randn((1, 1, N, 128), generator=g, device=DEV).to(dtype)
    V = torch.randn((1, 1, N, 128), generator=g, device=DEV).to(dtype)
    q = torch.randn((3, 1, n_q, 128), generator=g, device=DEV).to(dtype)
    idx.configure(B.RA_CFG_SEEDS, seeds)
    k8 = ra.ra_quantize_keys(K) if q8 else None
    more = {"k8": k8} if q8 else {}
    alone = [ra.ra_search(q[t], idx, None if q8 else K, 4, 500, topk, ef, expand, **more) for t in range(3)]
    assert all(st[..., 0].min() > 3000 for _, st in alone)
    outs = []
    for silent, spin in ((0, 20000), (1, 2), (0, 20000)):
        idx.test_configure(B.RA_TEST_HELPERS_SILENT, silent)
        idx.configure(B.RA_CFG_HELPER_SPIN, spin)
        assert idx.shared_steps_active == (not silent)
        for t in (0, 1, 2, 0):
            sent = idx.shared_messages
            out, lse, ids, st = ra.ra_decode_step(q[t], idx, K, V, 4, 500, topk, ef, expand, **more)
            assert torch.equal(ids, alone[t][0]) and torch.equal(st, alone[t][1]), (silent, t)
            outs.append(out)
            iters = int(st[0, 0, 2])
            if not silent:
                assert idx.shared_steps_active and iters - 1 <= idx.shared_messages - sent <= iters + 1, (t, iters)
            elif t:                                        # (the first of these calls has missed its answers)
                assert idx.shared_messages == sent
    # the same sets attended to: float32 sums over some 600 rows in another order, values of norm about 1
    assert all(torch.allclose(a, b, rtol=0, atol=1e-5) for a, b in zip(outs[:4], outs[4:8]))


@pytest.mark.parametrize("n_q,shared", [(8, True), (9, True), (12, True), (14, True), (24, True), (25, False)])
def test_workers_of_shared_steps_all_run_at_once(n_q, shared):
    """A search and its workers are on one compute die (an eighth of the compute units), with the helpers: no launch
    may have more of them there than units, or a search would wait for a worker that waits for it to end. Numbers of
    searches on either side of 8, 16 and 24, which make 2, 3 and 4 searches on one die."""
    N, deg, expand, ef, topk = 800_001, 24, 128, 1024, 64
    g = torch.Generator(device=DEV).manual_seed(n_q)
    adj = torch.randint(0, N, (n_q, N, deg), generator=g, device=DEV, dtype=torch.int32)
    idx = ra.ra_index_import(adj.cpu(), torch.zeros(n_q, dtype=torch.int32), 1, n_q, n_q)
    del adj
    K = torch.randn((1, n_q, N, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    q = torch.randn((1, n_q, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    want, st_want = ra.ra_search(q, idx, K, 4, 500, topk, ef, expand)
    assert idx.shared_steps_active == shared
    for _ in range(5):
        sent = idx.shared_messages
        out, lse, ids, st = ra.ra_decode_step(q, idx, K, K, 4, 500, topk, ef, expand)
        assert torch.equal(ids, want) and torch.equal(st, st_want)
        assert idx.shared_steps_active == shared               # no wait ran out
        assert (idx.shared_messages > sent) == shared
    idx.free()


@pytest.mark.parametrize("n_q,n_kv,N,seeds,ef", [
    (64, 16, 20_003, 1024, 256),           # helpers, seed shares
    (512, 128, 3_001, 256, 128),           # more searches than compute units: some start when others have given up
    (20, 20, 800_001, 2048, 1024)])        # shared steps
def test_hand_overs_switched_off_in_the_middle_of_a_launch(n_q, n_kv, N, seeds, ef):
    """With a wait of one poll, some heads of a launch give up and set the words that switch hand-overs off while other
    workgroups read them: whatever a workgroup has read, ids, counters and outputs are the same. (A word is
    one workgroup's decision: its wavefronts must not differ in it.)"""
    from paper_2409_10516_amd import binding as B
    deg, expand, topk = 24, 128, 64
    g = torch.Generator(device=DEV).manual_seed(n_q)
    adj = torch.randint(0, N, (n_q, N, deg), generator=g, device=DEV, dtype=torch.int32)
    idx = ra.ra_index_import(adj.cpu(), torch.zeros(n_q, dtype=torch.int32), 1, n_q, n_kv)
    del adj
    K = torch.randn((1, n_kv, N, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    q = torch.randn((1, n_q, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    idx.configure(B.RA_CFG_SEEDS, seeds)
    call = lambda: ra.ra_decode_step(q, idx, K, K, 4, 500, topk, ef, expand)
    idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_OFF)
    out, lse, ids, st = call()
    idx.configure(B.RA_CFG_HELPER_SPIN, 1)
    for _ in range(30):
        idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)       # forgets the waits that ran out
        for _ in range(2):
            o, l, i, s = call()
            assert torch.equal(i, ids) and torch.equal(s, st)
            # the same sets attended to: float32 sums over some 570 rows in another order, values of norm about 1
            assert torch.allclose(o, out, rtol=0, atol=1e-5) and torch.allclose(l, lse, rtol=1e-5, atol=1e-5)
    idx.free()


def test_shared_steps_recorded_and_after_a_wait_that_ran_out():
    """Steps are shared in a recorded launch as in others. Once a head has waited in vain, the launches that follow are
    those of walks that do not share, recorded ones walk alone, and setting RA_CFG_HELPERS starts over: the same ids,
    counters and outputs throughout."""
    from paper_2409_10516_amd import binding as B
    N, deg, expand, ef, topk, n_q = 800_001, 24, 128, 1024, 64, 4
    g = torch.Generator(device=DEV).manual_seed(5)
    adj = torch.randint(0, N, (n_q, N, deg), generator=g, device=DEV, dtype=torch.int32)
    idx = ra.ra_index_import(adj.cpu(), torch.zeros(n_q, dtype=torch.int32), 1, n_q, 1)
    del adj
    K = torch.randn((1, 1, N, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    q = torch.randn((1, n_q, 128), generator=g, device=DEV, dtype=torch.bfloat16)
    idx.configure(B.RA_CFG_SEEDS, 2048)
    ids, st = ra.ra_search(q, idx, K, 4, 500, topk, ef, expand)
    call = lambda: ra.ra_decode_step(q, idx, K, K, 4, 500, topk, ef, expand)
    base = call()

    def same(r):
        assert torch.equal(r[2], ids) and torch.equal(r[3], st)
        # the same sets attended to: float32 sums over some 570 rows in another order, values of norm about 1
        assert torch.allclose(r[0], base[0], rtol=0, atol=1e-5) and torch.allclose(r[1], base[1], rtol=1e-5, atol=1e-5)

    same(base)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        recorded = call()

    def replayed():
        for r in recorded:
            r.zero_()
        graph.replay()
        torch.cuda.synchronize()
        same(recorded)

    assert idx.shared_launches == 2
    for _ in range(3):
        sent = idx.shared_messages
        replayed()
        assert idx.shared_steps_active and idx.shared_messages > sent
        same(call())
    idx.configure(B.RA_CFG_HELPER_SPIN, 1)
    same(call())
    assert not idx.shared_steps_active
    idx.configure(B.RA_CFG_HELPER_SPIN, 20000)
    launches, sent = idx.shared_launches, idx.shared_messages
    for _ in range(3):
        same(call())
        replayed()
    assert idx.shared_launches == launches and idx.shared_messages == sent and not idx.shared_steps_active
    idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON)
    assert idx.shared_steps_active
    same(call())
    replayed()
    assert idx.shared_launches == launches + 1 and idx.shared_steps_active and idx.shared_messages > 0
    idx.free()


@pytest.mark.parametrize("deg,R,ef,expand,k,heads", [
    (24, 512, 256, 64, 0, 1), (32, 512, 256, 64, 8, 1), (32, 512, 256, 64, 9, 1), (33, 512, 256, 64, 3, 1),
    (64, 512, 256, 32, 16, 1), (64, 511, 256, 32, 17, 1), (32, 700, 512, 64, 16, 1), (32, 700, 512, 64, 17, 2),
    (32, 321, 256, 64, 4, 400), (32, 320, 256, 64, 4, 400), (24, 600, 100, 64, 30, 1)])
def test_first_step_behind_a_seed_set(deg, R, ef, expand, k, heads):
    """The step behind a seed set reads and claims only the cells that lead out of the set where these are few (at
    most one per thread, at most 16 of a pick), else all: k cells of every seed lead out (the most there can be where k
    exceeds the degree), to keys that several cells name. Integer keys, so ids and counters are the oracle's. Workgroups
    of 512, 1024 (ef 512) and 256 threads (400 heads), masks of 32 and 64 bits, sets at and below the size that is filtered."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(deg * 1000 + k)
    N, k = 1500, min(k, deg - 2)
    adj = np.full((heads, N, deg), -1, np.int32)
    t = np.arange(N)
    for j in (0, 1):                                         # the heap, as far as it stays in the set
        adj[:, :, j] = np.where(2 * t + 1 + j < R, 2 * t + 1 + j, -1)
    inside = rng.integers(0, R, size=(heads, N, deg - 2 - k))
    adj[:, :, 2:deg - k] = np.where(inside == t[None, :, None], -1, inside)
    out = rng.integers(R, N + 50, size=(heads, N, k))       # (some are no keys)
    out = np.where(out == t[None, :, None], R, out)
    adj[:, :, deg - k:] = np.where(out >= N, -1, out)
    adj[:, R, :] = np.where(adj[:, R, :] == R, -1, adj[:, R, :])
    cols = 2 + rng.permutation(deg - 2)                      # cells that lead out anywhere in the row
    adj[:, :, 2:] = adj[:, :, cols]
    ent = np.zeros(heads, np.int32)
    K = torch.from_numpy(rng.integers(-4, 5, size=(1, 1, N, 128)).astype(np.float32)).bfloat16()
    V = torch.from_numpy(rng.standard_normal((1, 1, N, 128)).astype(np.float32)).bfloat16()
    q = torch.from_numpy(rng.integers(-4, 5, size=(1, heads, 128)).astype(np.float32)).bfloat16()
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.from_numpy(ent), 1, heads, 1)
    for n in (R, R - 1, R):                                  # (a set in the place of a longer one)
        idx.configure(B.RA_CFG_SEEDS, n)
        ids, st = ra.ra_search(q.to(DEV), idx, K.to(DEV), 4, 20, 50, ef, expand)
        _, _, ids_d, st_d = ra.ra_decode_step(q.to(DEV), idx, K.to(DEV), V.to(DEV), 4, 20, 50, ef, expand)
        assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
        for h in sorted({0, heads // 2, heads - 1}):
            seeds = OS.backbone_seeds(adj[h], 0, n)
            ref, rst = OS.greedy_search(to_np(q[0, h]), to_np(K[0, 0]), adj[h], 0, ef, 50, expand, seeds=seeds,
                                        exclude=OA.static_ids(N, 4, 20))
            assert ids[0, h].tolist() == ref.tolist(), (n, h)
            assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]], (n, h)
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("deg,expand,ef,n_seeds", [
    (8, 8, 100, 64), (8, 63, 100, 65), (8, 64, 100, 65), (8, 64, 16, 500), (32, 64, 700, 600), (32, 64, 600, 601),
    (32, 64, 64, 2048), (32, 128, 1100, 2048), (8, 64, 300, 0), (24, 32, 48, 0), (64, 64, 256, 0), (64, 66, 128, 0)])
def test_first_beam_of_a_start_set(dtype, deg, expand, ef, n_seeds):
    """The first beam of a walk: a seed set or (n_seeds 0) a root set, some of whose keys enter as expanded, ordered by counting
    (64 keys or less, less than 512 words for the bins) or through bins, of fewer, as many and more keys than the beam holds,
    with scores that tie in crowds (keys are copies of 40 rows). Integer keys: ids and counters are the oracle's."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(deg + 7 * n_seeds)
    N, heads = 5000, 2
    adj = rng.integers(0, N, size=(heads, N, deg)).astype(np.int32)
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < N, 2 * t + 1 + j, -1)
    adj[adj == t[None, :, None]] = -1
    K = rng.integers(-3, 4, size=(40, 128))[rng.integers(0, 40, size=N)].astype(np.float32)
    q = rng.integers(-3, 4, size=(1, heads, 128)).astype(np.float32)
    Kd = torch.from_numpy(K[None, None]).to(dtype).to(DEV)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.zeros(heads, dtype=torch.int32), 1, heads, 1)
    idx.configure(B.RA_CFG_SEEDS, n_seeds)
    topk = min(ef, 40)
    qd = torch.from_numpy(q).to(dtype).to(DEV)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 20, topk, ef, expand)
    _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 20, topk, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    for h in range(heads):
        seeds = OS.backbone_seeds(adj[h], 0, n_seeds) if n_seeds else None
        ref, rst = OS.greedy_search(q[0, h], K, adj[h], 0, ef, topk, expand, seeds=seeds, exclude=OA.static_ids(N, 4, 20))
        assert ids[0, h].tolist() == ref.tolist()
        assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("seeds,ef,heads", [(1024, 256, 8), (2048, 300, 8), (700, 128, 4), (0, 128, 8)])
def test_decode_step_of_views_at_odd_offsets(dtype, seeds, ef, heads):
    """Queries, keys and values that start at any element of their storage (in bfloat16 also between two words): what aligned
    copies give, bit for bit, with the start sets scored by workgroups of their own, and by the head."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(seeds + ef)
    N, deg = 3000, 32
    adj = rng.integers(0, N, size=(heads, N, deg)).astype(np.int32)
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < N, 2 * t + 1 + j, -1)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.zeros(heads, dtype=torch.int32), 1, heads, 2)
    idx.configure(B.RA_CFG_SEEDS, seeds)
    q, K, V = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(dtype).to(DEV)
               for s in ((1, heads, 128), (1, 2, N, 128), (1, 2, N, 128)))
    want = ra.ra_decode_step(q, idx, K, V, 4, 50, 60, ef, 64)
    for offset in (1, 3, 6):
        views = []
        for x in (q, K, V):
            flat = torch.zeros(x.numel() + 8, dtype=dtype, device=DEV)
            views.append(flat[offset:offset + x.numel()].view(x.shape))
            views[-1].copy_(x)
        for shares in (6, 0):
            idx.configure(B.RA_CFG_SEED_SHARES, shares)
            got = ra.ra_decode_step(views[0], idx, views[1], views[2], 4, 50, 60, ef, 64)
            assert all(torch.equal(a, b) for a, b in zip(got, want)), (offset, shares)
            assert idx.seed_shares_active == (seeds > 0 and shares > 0)
    idx.free()


def _kept_per_step(q, K, adj, entry, ef, expand):
    """How many candidates each step of the walk keeps: all new ones while the beam is not full, then those better than its worst
    entry. (Score descending, id ascending; for integer inputs.)"""
    score = K @ q
    order = lambda i: (-score[i], i)
    beam, seen, done, kept = [entry], {entry}, set(), []
    while True:
        picks = [i for i in beam if i not in done][:expand]
        if not picks:
            return kept
        done.update(picks)
        new = sorted({int(j) for i in picks for j in adj[i] if 0 <= j < len(K)} - seen, key=order)
        seen.update(new)
        new = [j for j in new if len(beam) < ef or order(j) < order(beam[-1])]
        kept.append(len(new))
        beam = sorted(beam + new, key=order)[:ef]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("ef,expand,deg", [(300, 8, 33), (513, 9, 31), (1100, 5, 52), (2048, 3, 24)])
def test_merges_of_few_candidates_into_wide_beams(ef, expand, deg, dtype):
    """Workgroups of 1024 threads: merges of up to 16, of 17 to 32, of up to 64 and of more candidates, into beams of every length
    up to the widest; many scores tie. Integer keys: the oracle's ids and counters."""
    rng, N = np.random.default_rng(ef), 6000
    K = rng.integers(-3, 4, size=(N, 128)).astype(np.float32)
    adj = rng.integers(0, N, size=(1, N, deg)).astype(np.int32)
    q = rng.integers(-3, 4, size=128).astype(np.float32)
    kept = _kept_per_step(q, K, adj[0], 11, ef, expand)
    assert all(any(lo <= n <= hi for n in kept) for lo, hi in ((1, 8), (9, 16), (17, 32), (33, 64), (65, 999)))
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.tensor([11], dtype=torch.int32), 1, 1, 1)
    Kd, qd = torch.from_numpy(K)[None, None].to(dtype).to(DEV), torch.from_numpy(q)[None, None].to(dtype).to(DEV)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 20, 200, ef, expand)
    _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 20, 200, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    ref, rst = OS.greedy_search(q, K, adj[0], 11, ef, 200, expand, exclude=OA.static_ids(N, 4, 20))
    assert ids[0, 0].tolist() == ref.tolist()
    assert st[0, 0].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]
    idx.free()


@pytest.mark.parametrize("ef,expand,deg,heads", [(16, 5, 64, 1), (64, 9, 60, 1), (300, 16, 64, 1), (16, 8, 33, 400)])
def test_steps_that_keep_far_more_than_the_beam_holds(ef, expand, deg, heads):
    """A step, not a start set, whose kept candidates outnumber the beam by more than 64: all but the best are dropped ahead of
    the merge. Keys that lie farther from the entry point score higher, so that nearly all of a step's are kept, with crowds of equal
    scores. Workgroups of 512, 1024 and 256 threads."""
    rng, N = np.random.default_rng(ef + deg), 1200
    level = np.minimum(np.arange(N) // 40, 9)
    adj = np.stack([rng.permutation(np.flatnonzero(level >= min(level[i] + 1, 9)))[:deg] for i in range(N)]).astype(np.int32)
    K = rng.integers(-1, 2, size=(N, 128)).astype(np.float32)
    K[:, 0] = 3 * level + 3
    q = rng.integers(-1, 2, size=128).astype(np.float32)
    q[0] = 60.0
    assert expand < deg and expand * deg >= 256                  # (no root set is listed for so few nodes per step)
    assert max(_kept_per_step(q, K, adj, 7, ef, expand)) > ef + 64
    idx = ra.ra_index_import(torch.from_numpy(np.repeat(adj[None], heads, 0)), torch.full((heads,), 7, dtype=torch.int32), 1, heads, 1)
    Kd = torch.from_numpy(K)[None, None].bfloat16().to(DEV)
    qd = torch.from_numpy(q).bfloat16().repeat(1, heads, 1).to(DEV)
    topk = min(ef, 40)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 20, topk, ef, expand)
    _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 20, topk, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    ref, rst = OS.greedy_search(q, K, adj, 7, ef, topk, expand, exclude=OA.static_ids(N, 4, 20))
    for h in (0, heads - 1):
        assert ids[0, h].tolist() == ref.tolist()
        assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_seeds,deg,expand,ef", [
    (64, 8, 64, 100), (65, 8, 63, 100), (65, 8, 64, 100), (65, 7, 73, 100), (300, 32, 20, 200), (512, 32, 16, 200),
    (512, 32, 32, 200), (513, 32, 33, 200), (1000, 40, 64, 200), (2048, 32, 64, 300), (0, 24, 25, 48), (0, 24, 24, 48)])
def test_start_sets_at_the_limits_of_their_order(dtype, n_seeds, deg, expand, ef):
    """Start sets of 64 and 65 keys (counted, and ordered through bins), steps of 504 to 512 cells (bins from 512 on), sets with room
    for their masks and the list of new cells and without, a root set that fits its step and one that does not. Scores that tie in
    crowds, and one key far above the others, which leaves these in few bins. Integer keys: the oracle's ids and counters."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(n_seeds + deg + expand)
    N = 4000
    adj = rng.integers(0, N, size=(1, N, deg)).astype(np.int32)
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < N, 2 * t + 1 + j, -1)
    adj[adj == t[None, :, None]] = -1
    q = rng.integers(-3, 4, size=(1, 1, 128)).astype(np.float32)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.zeros(1, dtype=torch.int32), 1, 1, 1)
    idx.configure(B.RA_CFG_SEEDS, n_seeds)
    for far in (1, 500):
        K = rng.integers(-3, 4, size=(60, 128))[rng.integers(0, 60, size=N)].astype(np.float32)
        K[1] = far * np.sign(q[0, 0])
        Kd, qd = torch.from_numpy(K)[None, None].to(dtype).to(DEV), torch.from_numpy(q).to(dtype).to(DEV)
        K = to_np(Kd[0, 0])
        ids, st = ra.ra_search(qd, idx, Kd, 4, 20, 40, ef, expand)
        _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 20, 40, ef, expand)
        assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
        seeds = OS.backbone_seeds(adj[0], 0, n_seeds) if n_seeds else None
        ref, rst = OS.greedy_search(q[0, 0], K, adj[0], 0, ef, 40, expand, seeds=seeds, exclude=OA.static_ids(N, 4, 20))
        assert ids[0, 0].tolist() == ref.tolist(), far
        assert st[0, 0].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]], far
    idx.free()


@pytest.mark.parametrize("heads,R,deg", [(1, 65, 32), (2, 129, 40), (64, 300, 32), (90, 257, 33), (300, 200, 32), (520, 100, 24)])
def test_masks_of_seed_sets_in_many_and_few_heads(heads, R, deg):
    """The masks of a head's set are listed by eight workgroups, by fewer or by one, as there are heads; sets of fewer ids than these have wavefronts,
    and ragged ones. A mask with a cell too many or too few would change the keys that the first step visits: some
    cells of its picks lead out of the set. Integer keys: the oracle's ids and counters, in every head of its own graph."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(heads + R)
    N, ef, expand = 900, 64, 64
    adj = rng.integers(0, R, size=(heads, N, deg)).astype(np.int32)
    lead = rng.random((heads, N, deg)) < 8.0 / (64 * deg)    # (few enough to be listed, over the picks of a step)
    adj[lead] = rng.integers(R, N, size=int(lead.sum()))
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < R, 2 * t + 1 + j, -1)
    adj[adj == t[None, :, None]] = -1
    K = rng.integers(-4, 5, size=(N, 128)).astype(np.float32)
    q = rng.integers(-4, 5, size=(1, heads, 128)).astype(np.float32)
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.zeros(heads, dtype=torch.int32), 1, heads, 1)
    idx.configure(B.RA_CFG_SEEDS, R)
    ids, st = ra.ra_search(torch.from_numpy(q).bfloat16().to(DEV), idx, torch.from_numpy(K)[None, None].bfloat16().to(DEV), 4, 20, 30, ef, expand)
    for h in sorted({0, heads // 3, heads // 2, heads - 1}):
        ref, rst = OS.greedy_search(q[0, h], K, adj[h], 0, ef, 30, expand, seeds=OS.backbone_seeds(adj[h], 0, R), exclude=OA.static_ids(N, 4, 20))
        assert ids[0, h].tolist() == ref.tolist(), h
        assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]], h
        assert rst["n_visited"] > R
    idx.free()
