"""Parity of the HIP index build (exact KNN on the matrix cores, projection) with the CPU
oracle, through the C ABI. GPU only."""
import json
import os

import numpy as np
import pytest
import torch

import paper_2409_10516_amd as ra
from oracle import attention as OA, decode as OD, mips as OM, projection as OP
from paper_2409_10516_amd import synth
from tests.util import decode_matches, integer_valued, knn_equivalent, lse_close, out_close, to_np, tol_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GOLD = os.path.join(os.path.dirname(__file__), "golden")


@pytest.fixture(params=["filter", "lds"])
def knn_selection(request):
    """The later part of a long key stream goes through 8-bit products that rule keys out; the library
    decides by the sizes, the tests force them on (from the 129th key) or off through the test-only
    setting."""
    from paper_2409_10516_amd import binding as B
    ra.ra_test_configure(B.RA_TEST_KNN_SELECTION,
                         B.RA_TEST_KNN_FILTER if request.param == "filter" else B.RA_TEST_KNN_LDS)
    yield request.param
    ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_AUTO)


def _cases():
    return {
        "config0_small": lambda: synth.make_config0(N=1024, M=256, T=2, window=32),
        "llama_bf16": lambda: synth.make_llama_layer(11, N=1536, M=768, T=2, n_q=8, n_kv=2,
                                                     ef=64, topk=20, window=100),
        "llama_f32_ragged": lambda: synth.make_llama_layer(12, N=701, M=299, T=2, n_seq=2, n_q=4,
                                                           n_kv=4, dtype=torch.float32, ef=48,
                                                           topk=16, window=37, deg=12, knn=9),
        "integer_ties": lambda: synth.make_integer_case(5, N=200, M=64, T=2, d=128, n_q=2,
                                                        n_kv=1, deg=8, knn=6, topk=9, ef=20,
                                                        sink=3, window=10),
        "integer_bf16_knn64": lambda: synth.make_integer_case(6, N=333, M=150, T=2, d=128, n_q=1,
                                                              n_kv=1, dtype=torch.bfloat16, deg=64,
                                                              knn=64, topk=9, ef=20),
        "integer_bf16_knn48": lambda: synth.make_integer_case(7, N=777, M=130, T=2, d=128, n_q=2,
                                                              n_kv=1, dtype=torch.bfloat16, deg=48,
                                                              knn=48, topk=9, ef=20),
        "integer_bf16_knn20": lambda: synth.make_integer_case(9, N=900, M=600, T=2, d=128, n_q=2,
                                                              n_kv=1, dtype=torch.bfloat16, deg=16,
                                                              knn=20, topk=9, ef=20),
        "integer_f32_knn40": lambda: synth.make_integer_case(8, N=450, M=70, T=2, d=128, n_q=1,
                                                             n_kv=1, dtype=torch.float32, deg=16,
                                                             knn=40, topk=9, ef=20),
    }


def _heads(w):
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    for s in range(n_seq):
        for h in range(n_q):
            yield s, h, s * n_q + h, to_np(w.K[s, h // (n_q // n_kv)]), to_np(w.Q_prefill[s, h])


@pytest.mark.parametrize("name", list(_cases()))
def test_knn_lists(name, knn_selection):
    w = _cases()[name]()
    L = ra.ra_knn(w.K.to(DEV), w.Q_prefill.to(DEV), w.knn).cpu().numpy()
    for s, h, g, K, Q in _heads(w):
        ref, _ = OM.knn_lists(Q, K, w.knn)
        diff = knn_equivalent(L[s, h], ref, Q, K)
        if name.startswith("integer"):
            assert diff == 0          # integer-valued inputs: every score is exact


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("knn", [5, 32, 48, 64])
@pytest.mark.parametrize("rising", [True, False])
def test_knn_monotone_stream(dtype, knn, rising, knn_selection):
    """Scores that rise with the key id make every key of the stream qualify (the selection folds or
    inserts all the time); falling scores make none qualify after the first knn. Key i scores exactly
    +-i for every query (i = 256 * K[i,1] + K[i,0], both exact in bf16), so the lists are known."""
    N, M = 3001, 77
    K = torch.zeros((1, 1, N, 128), dtype=torch.float32)
    i = torch.arange(N)
    K[0, 0, :, 0] = (i % 256).float()
    K[0, 0, :, 1] = (i // 256).float()
    Q = torch.zeros((1, 1, M, 128), dtype=torch.float32)
    Q[0, 0, :, 0] = 1.0 if rising else -1.0
    Q[0, 0, :, 1] = 256.0 if rising else -256.0
    L = ra.ra_knn(K.to(dtype).to(DEV), Q.to(dtype).to(DEV), knn).cpu().numpy()[0, 0]
    want = np.arange(N - 1, N - 1 - knn, -1) if rising else np.arange(knn)
    assert np.array_equal(L, np.broadcast_to(want, (M, knn)))


@pytest.mark.parametrize("N", [1, 2, 1025, 8191, 8192, 8193, 20001])
@pytest.mark.parametrize("scores", ["equal", "few", "outlier", "spread", "overflow"])
def test_knn_stream_order_of_any_scores(N, scores):
    """The stream order deals a chunk of up to 8192 keys to bins of their score: one bin holds all, crowded bins, all but
    one key in one bin, no crowd, and a width that is not finite. Every key has to come out of it once: scores are
    whole numbers (float32, exact), so the lists are the best by score, then by id."""
    rng = np.random.default_rng(N)
    M, knn = 33, min(16, N)
    K = np.zeros((N, 128))
    place = {"equal": np.zeros(N), "few": rng.integers(-2, 3, N), "outlier": (np.arange(N) == N // 2) * 4e6,
             "spread": rng.integers(-4000, 4001, N), "overflow": rng.integers(-2, 3, N) * 2.0 ** 126}[scores]
    K[:, 0] = place
    K[:, 1] = rng.integers(-500, 501, N)
    Q = np.zeros((M, 128))
    Q[:, 0] = 2.0 if scores == "overflow" else 1.0            # (the mean query's products overflow; the last rows' do not)
    Q[-3:, 0] = 0
    Q[:, 1] = np.arange(M) % 3 - 1
    L = ra.ra_knn(torch.from_numpy(K).float()[None, None].to(DEV), torch.from_numpy(Q).float()[None, None].to(DEV), knn)
    L = L.cpu().numpy()[0, 0]
    for j in range(M - 3 if scores == "overflow" else 0, M):
        want = np.argsort(-(K @ Q[j]), kind="stable")[:knn]
        assert np.array_equal(L[j][:len(want)], want) and np.all(L[j][len(want):] == -1), (scores, j)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("knn", [32, 48, 64])
def test_knn_scores_that_are_no_numbers(dtype, knn):
    """Keys with a NaN or with scores of minus infinity are in no list; a list they leave short ends in -1."""
    N, M = 200, 40
    i = np.arange(N)
    K = np.zeros((N, 128))
    K[:, 0] = i % 7 + 1
    K[i % 10 != 3, 5] = np.nan
    K[i % 10 == 4, 5] = -np.inf
    Q = np.zeros((M, 128))
    Q[:, 0] = np.arange(M) % 5 + 1
    Q[:, 5] = 1.0
    got = ra.ra_knn(torch.from_numpy(K).to(dtype).to(DEV)[None, None],
                    torch.from_numpy(Q).to(dtype).to(DEV)[None, None], knn).cpu().numpy()[0, 0]
    numbers = i[i % 10 == 3]
    want = numbers[np.lexsort((numbers, -K[numbers, 0]))]
    assert np.array_equal(got[:, :20], np.broadcast_to(want, (M, 20)))
    assert (got[:, 20:] == -1).all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("knn", [1, 31, 32, 33, 48, 63, 64])
@pytest.mark.parametrize("half", [0, 1])
def test_knn_runs_of_one_lane(dtype, knn, half):
    """The keys that reach a threshold are all in the rows that one of a query's two lanes scores (four rows in eight; the
    mean query is zero, so the stream is in storage order): that lane's pending run is full again and again, the
    other's holds nothing or ties. Integer scores: the oracle's lists."""
    N, M = 515, 70
    i = np.arange(N)
    rising = np.where(i // 4 % 2 == half, i, i % 3)
    K = np.zeros((N, 128))
    K[:, 0], K[:, 1] = rising % 128, rising // 128
    Q = np.zeros((M, 128))
    Q[:, 0] = np.where(np.arange(M) % 2 == 0, 1, -1)
    Q[:, 1] = 128 * Q[:, 0]
    got = ra.ra_knn(torch.from_numpy(K).to(dtype).to(DEV)[None, None],
                    torch.from_numpy(Q).to(dtype).to(DEV)[None, None], knn).cpu().numpy()[0, 0]
    assert np.array_equal(got, OM.knn_lists(Q[:2], K, knn)[0][np.arange(M) % 2])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("knn", [7, 32, 64])
def test_knn_stream_order_against_a_minority_of_queries(dtype, knn, knn_selection):
    """The keys are streamed by descending inner product with the head's mean query. Here 60 % of
    the queries are -u and 40 % are +u, so the stream is in the best order for the majority and in
    the worst (every key beats the threshold) for the minority; the lists must not depend on it."""
    N, M = 2500, 90
    K = torch.zeros((1, 1, N, 128), dtype=torch.float32)
    i = torch.arange(N)
    K[0, 0, :, 0] = (i % 256).float()
    K[0, 0, :, 1] = (i // 256).float()
    sign = torch.where(torch.arange(M) % 5 < 3, -1.0, 1.0)
    Q = torch.zeros((1, 1, M, 128), dtype=torch.float32)
    Q[0, 0, :, 0] = sign
    Q[0, 0, :, 1] = 256.0 * sign
    L = ra.ra_knn(K.to(dtype).to(DEV), Q.to(dtype).to(DEV), knn).cpu().numpy()[0, 0]
    for j in range(M):
        want = np.arange(N - 1, N - 1 - knn, -1) if sign[j] > 0 else np.arange(knn)
        assert np.array_equal(L[j], want), j


@pytest.mark.parametrize("N,knn", [(1, 1), (3, 3), (5, 2), (33, 33), (64, 48), (65, 64)])
def test_knn_tiny_key_sets(N, knn, knn_selection):
    """Fewer keys than a stage, than a block, than the sort's smallest chunk: all equal scores, so
    the lists are the lowest ids in order."""
    M = 9
    K = torch.ones((1, 1, N, 128), dtype=torch.bfloat16)
    Q = torch.ones((1, 1, M, 128), dtype=torch.bfloat16)
    L = ra.ra_knn(K.to(DEV), Q.to(DEV), knn).cpu().numpy()[0, 0]
    assert np.array_equal(L, np.broadcast_to(np.arange(knn), (M, knn)))


def _sweep_cases():
    rng = np.random.default_rng(1234)
    cases = []
    for it in range(14):
        dtype = torch.bfloat16 if it % 3 else torch.float32
        n_kv = int(rng.choice([1, 2])); G = int(rng.choice([1, 2, 4]))
        N = int(rng.choice([31, 33, 63, 65, 100, 511, 513, 1000, 2047, 4097]))
        M = int(rng.choice([1, 5, 33, 255, 257, 511, 513, 1025]))
        knn = min(int(rng.choice([1, 2, 5, 16, 31, 32, 33, 40, 48, 49, 64])), N)
        cases.append((it, dtype, n_kv, G, N, M, knn))
    return cases


@pytest.mark.parametrize("it,dtype,n_kv,G,N,M,knn", _sweep_cases())
def test_knn_shape_sweep(it, dtype, n_kv, G, N, M, knn, knn_selection):
    """Key and query counts around the kernel's block, stage and workgroup sizes, list lengths on both
    sides of every selection's limit. Small integer inputs with a shared component: every score is
    exact, ties abound, the stream order is not the storage order."""
    g = torch.Generator(); g.manual_seed(1000 + it)
    K = torch.randint(-3, 4, (1, n_kv, N, 128), generator=g).float()
    Q = torch.randint(-3, 4, (1, n_kv * G, M, 128), generator=g).float()
    K[..., 0] += torch.randint(0, 6, (1, n_kv, N), generator=g).float()
    Q[..., 0] += 2
    L = ra.ra_knn(K.to(dtype).to(DEV), Q.to(dtype).to(DEV), knn).cpu().numpy()
    for h in range(n_kv * G):
        ref, _ = OM.knn_lists(Q[0, h].numpy().astype(np.float64), K[0, h // G].numpy().astype(np.float64), knn)
        assert np.array_equal(L[0, h], ref), h


def test_projection_hand_worked_example():
    g = json.load(open(os.path.join(GOLD, "projection_hand.json")))
    L = torch.tensor([g["L"]], dtype=torch.int32, device=DEV)
    adj, entry = ra.ra_project(L, g["N"], g["deg"])
    assert entry.cpu().tolist() == [g["entry"]]
    assert adj[0].cpu().tolist() == g["adj"]


def test_projection_regimes_of_a_large_graph():
    """More populated keys than the row kernel has LDS counters, with the three kinds of key such a
    graph holds: hubs (in half of all lists: counters in device memory, pipelined list walk), keys of
    about 60 lists (LDS hash table, one workgroup per key) and keys of a handful of lists (one
    wavefront per key). Every hub and middle key and a sample of the small ones against the oracle."""
    rng = np.random.default_rng(17)
    N, M, knn, deg = 20000, 3000, 48, 16
    hubs, mids, rest = np.arange(10), np.arange(10, 310), np.arange(310, N)
    L = np.empty((M, knn), np.int32)
    for j in range(M):
        row = np.concatenate([rng.choice(hubs, 5, replace=False), rng.choice(mids, 6, replace=False),
                              rng.choice(rest, knn - 11, replace=False)])
        L[j] = rng.permutation(row)
    adj, entry = ra.ra_project(torch.from_numpy(L[None]).to(DEV), N, deg)
    adj = adj[0].cpu().numpy()
    rows = np.concatenate([hubs, mids, rng.choice(rest, 400, replace=False)])
    radj, rent = OP.project(L, N, deg, rows=rows)
    assert int(entry[0]) == rent
    pop = np.bincount(L.ravel(), minlength=N)
    assert (pop > 0).sum() > 8192 and pop[hubs].min() > 1000 and 21 < pop[mids].min() and pop[mids].max() <= 85
    for a in rows:
        assert np.array_equal(adj[a], radj[a]), (a, adj[a], radj[a])


@pytest.mark.parametrize("name", list(_cases()))
@pytest.mark.parametrize("deg", [None, 2, 5])
def test_projection_bit_exact_on_oracle_lists(name, deg):
    w = _cases()[name]()
    deg = deg or w.deg
    N = w.K.shape[2]
    Ls, refs = [], []
    for s, h, g, K, Q in _heads(w):
        L, _ = OM.knn_lists(Q, K, w.knn)
        Ls.append(L)
        refs.append(OP.project(L, N, deg))
    adj, entry = ra.ra_project(torch.from_numpy(np.stack(Ls)).to(DEV), N, deg)
    adj, entry = adj.cpu().numpy(), entry.cpu().numpy()
    for g, (radj, rent) in enumerate(refs):
        assert entry[g] == rent
        assert np.array_equal(adj[g], radj), np.argwhere(adj[g] != radj)[:5]


def test_projection_skewed_lists():
    """Every list holds the same two hub keys plus a few others (the shape the Llama-like
    generator produces at scale), and some keys are in no list at all."""
    rng = np.random.default_rng(0)
    N, M, knn, deg = 500, 400, 8, 10
    L = np.empty((M, knn), np.int32)
    for j in range(M):
        rest = rng.choice(np.arange(2, 120), size=knn - 2, replace=False)
        L[j] = np.concatenate([[0, 1], rest])[rng.permutation(knn)]
    radj, rent = OP.project(L, N, deg)
    adj, entry = ra.ra_project(torch.from_numpy(L[None]).to(DEV), N, deg)
    assert int(entry[0]) == rent
    assert np.array_equal(adj[0].cpu().numpy(), radj)


@pytest.mark.parametrize("name", list(_cases()))
def test_build_index_then_decode(name):
    """ra_build_index = KNN + projection; its graph must be the oracle's projection of the
    device's own KNN lists (which may differ from the float64 lists only in near-ties), and a
    decode step on it must match the oracle run on the exported graph."""
    w = _cases()[name]()
    Kd, Vd, Qd = w.K.to(DEV), w.V.to(DEV), w.Q_prefill.to(DEV)
    n_seq, n_kv, N, d = w.K.shape
    n_q = w.Q_prefill.shape[1]
    L = ra.ra_knn(Kd, Qd, w.knn).cpu().numpy()
    idx = ra.ra_build_index(Kd, Qd, w.deg, w.knn)
    assert (idx.n_seq, idx.n_q_heads, idx.n_kv_heads, idx.N, idx.deg) == (n_seq, n_q, n_kv, N, w.deg)
    tol = tol_for(w.K.dtype)
    q = w.q_decode[0]
    out, lse, ids, st = ra.ra_decode_step(q.to(DEV), idx, Kd, Vd, w.sink, w.window, w.topk, w.ef, 4)
    out, lse, ids, st = out.cpu().numpy(), lse.cpu().numpy(), ids.cpu().numpy(), st.cpu().numpy()
    exact = integer_valued(to_np(w.K), to_np(w.q_decode))
    for s, h, g, K, Q in _heads(w):
        radj, rent = OP.project(L[s, h], N, w.deg)
        adj, ent = ra.ra_index_export(idx, s, h)
        assert ent == rent and np.array_equal(adj.numpy(), radj)
        V = to_np(w.V[s, h // (n_q // n_kv)])
        decode_matches(out[s, h], lse[s, h], ids[s, h], st[s, h].tolist(), to_np(q[s, h]), K, V, radj, rent,
                       w.sink, w.window, w.topk, w.ef, 4, tol, exact=exact)
    idx.free()


@pytest.mark.parametrize("room", ["own", "full", "tight", "short"])
def test_build_in_the_callers_workspace(room):
    """A build in memory of the caller's gives the graphs of one in the library's own, with the 8-bit copies and
    without room for them, and refuses less than that; the memory behind the workspace stays as it was."""
    import ctypes as C
    from paper_2409_10516_amd import binding as B
    lib = ra.lib()
    w = synth.make_llama_layer(9, 8192, 700, n_seq=1, n_q=4, n_kv=2, device=DEV, dtype=torch.float32)
    knn, deg = 16, 16
    sizes = (1, 4, 2, 8192, 700, 128, deg, knn)
    need = lib.ra_build_workspace_bytes(B.RA_F32, *sizes)
    assert need > 0 and lib.ra_build_workspace_bytes(B.RA_F32, *sizes[:-1], 0) == 0
    copies = 4 * 8192 * 128                              # 8-bit copies of the keys: a row of 128 bytes each and head
    have = {"own": 0, "full": need, "tight": need - copies // 2, "short": 1 << 16}[room]
    piece = torch.full((have + 4096,), 77, dtype=torch.uint8, device=DEV)
    ix = C.c_void_p()
    rc = lib.ra_build_index_ws(w.K.data_ptr(), w.Q_prefill.data_ptr(), B.RA_F32, *sizes, piece.data_ptr() if have else None,
                               have, torch.cuda.current_stream().cuda_stream, C.byref(ix))
    if room == "short":
        assert rc == 2 and not ix.value
        return
    assert rc == 0
    assert bool((piece[have:] == 77).all())
    got, want = B.Index(ix.value), ra.ra_build_index(w.K, w.Q_prefill, deg, knn)
    for h in range(4):
        (a, ea), (b, eb) = ra.ra_index_export(got, 0, h), ra.ra_index_export(want, 0, h)
        assert ea == eb and torch.equal(a, b)
    got.free()
    want.free()


@pytest.mark.parametrize("n,M,knn,hubs,per_list,others", [
    (7, 1500, 24, 100, 14, 400),        # hubs' arrays of their own
    (5, 700, 64, 90, 24, 9000),         # more keys than 16-bit lists are for: 32-bit lists, counters in device memory
    (5, 4000, 64, 90, 24, 7000),        # as many cells, fewer populated keys: the hubs' arrays behind the 16-bit lists
])
def test_projection_in_any_amount_of_memory(n, M, knn, hubs, per_list, others):
    """Several graphs, all at a time, a few, one by one, and without memory for the hubs' arrays: the rows of each projected
    alone; less is refused; the memory behind the workspace stays as it was."""
    import re
    lib, deg, N = ra.lib(), 32, 9500
    L = np.stack([_hub_lists(np.random.default_rng(M + g), M, knn, hubs, per_list, others) for g in range(n)])
    Ld = torch.from_numpy(np.ascontiguousarray(L)).to(DEV)
    alone = [ra.ra_project(Ld[g:g + 1].contiguous(), N, deg) for g in range(n)]
    want, entry = torch.cat([a for a, _ in alone]), torch.cat([e for _, e in alone])
    st = torch.cuda.current_stream().cuda_stream
    adj, ent = torch.empty_like(want), torch.empty_like(entry)
    piece = torch.full((4096,), 77, dtype=torch.uint8, device=DEV)
    assert lib.ra_project_ws(Ld.data_ptr(), n, N, M, knn, deg, piece.data_ptr(), 256, st, adj.data_ptr(), ent.data_ptr()) == 2
    least = int(re.search(r"needs (\d+)", lib.ra_last_error().decode()).group(1))
    one, full = (lib.ra_project_scratch_bytes(k, N, M, deg, knn) for k in (1, n))
    assert 256 < least <= one < full
    for have in sorted({least, max(least, one - 1), one, 2 * least, 3 * one, (full + one) // 2, full - 1, full, full + 4096}):
        piece = torch.full((have + 4096,), 77, dtype=torch.uint8, device=DEV)
        adj.fill_(-7)
        ent.fill_(-7)
        rc = lib.ra_project_ws(Ld.data_ptr(), n, N, M, knn, deg, piece.data_ptr(), have, st, adj.data_ptr(), ent.data_ptr())
        assert rc == 0 and torch.equal(adj, want) and torch.equal(ent, entry), have
        assert bool((piece[have:] == 77).all())
    assert lib.ra_project_ws(Ld.data_ptr(), n, N, M, knn, deg, piece.data_ptr(), least - 1, st, adj.data_ptr(), ent.data_ptr()) == 2


def test_builds_in_a_row_take_the_same_scratch_memory():
    """Builds with hundreds of megabytes of scratch memory, and the stages as their own calls: nothing is allocated or freed
    for it by the second of two calls (drivers that have to take and give as much per call hold them up), and what the first
    took goes back with torch.cuda.empty_cache()."""
    N, M, n_q, knn = 100000, 300, 32, 16
    w = synth.make_llama_layer(5, N, M, n_seq=1, n_q=n_q, n_kv=8, device=DEV)
    lib = ra.lib()
    need = lib.ra_build_workspace_bytes(1, 1, n_q, 8, N, M, 128, 32, knn)
    assert 300 << 20 < need < 1 << 30 and lib.ra_knn_scratch_bytes(1, 1, n_q, 8, N, M, 128, knn) > 300 << 20
    L = ra.ra_knn(w.K, w.Q_prefill, knn)
    calls = [lambda: ra.ra_build_index(w.K, w.Q_prefill, 32, knn).free(), lambda: ra.ra_knn(w.K, w.Q_prefill, knn),
             lambda: ra.ra_project(L.view(n_q, M, knn), N, 32)]
    torch.cuda.empty_cache()
    held = torch.cuda.memory_reserved()
    for call in calls:
        call()
        before, free = torch.cuda.memory_stats()["num_device_alloc"], torch.cuda.mem_get_info()[0]
        call()
        assert torch.cuda.memory_stats()["num_device_alloc"] == before and torch.cuda.mem_get_info()[0] == free
    assert torch.cuda.memory_reserved() - held >= need
    torch.cuda.empty_cache()
    assert torch.cuda.memory_reserved() == held


@pytest.mark.parametrize("n,N,M", [(4, 600, 600), (2, 300, 300), (7, 900, 40)])
def test_projection_of_a_small_batch_is_one_group(n, N, M):
    """A workspace of as much as is asked for takes all graphs at once: the last one's part of it is written too."""
    lib, deg, knn = ra.lib(), 32, 24
    L = torch.randint(0, N, (n, M, knn), dtype=torch.int32, device=DEV)
    one, full = (lib.ra_project_scratch_bytes(k, N, M, deg, knn) for k in (1, n))
    assert full == n * one
    piece = torch.full((full,), 77, dtype=torch.uint8, device=DEV)
    adj, ent = torch.empty((n, N, deg), dtype=torch.int32, device=DEV), torch.empty(n, dtype=torch.int32, device=DEV)
    assert lib.ra_project_ws(L.data_ptr(), n, N, M, knn, deg, piece.data_ptr(), full, torch.cuda.current_stream().cuda_stream,
                             adj.data_ptr(), ent.data_ptr()) == 0
    parts = piece.view(n, one)
    assert all(bool((parts[g] != 77).any()) for g in range(n))
    assert torch.equal(adj[n - 1:], ra.ra_project(L[n - 1:].contiguous(), N, deg)[0])


def test_build_argument_errors():
    w = synth.make_integer_case(1, N=64, M=16, d=128)
    Kd, Qd = w.K.to(DEV), w.Q_prefill.to(DEV)
    with pytest.raises(ra.RaError) as e:
        ra.ra_knn(Kd, Qd, 65)                        # knn > N
    assert e.value.status == 1
    with pytest.raises(ra.RaError) as e:
        ra.ra_build_index(Kd, Qd, 1, 4)              # deg < 2
    assert e.value.status == 1
    with pytest.raises(ra.RaError) as e:
        ra.ra_build_index(Kd[..., :64].contiguous(), Qd[..., :64].contiguous(), 8, 4)   # d != 128
    assert e.value.status == 6


def _project_case(kind):
    rng = np.random.default_rng(23)
    if kind == "wide":                # more queries than a packed candidate key takes (2^19)
        N, M, knn, deg = 300, (1 << 19) + 5, 3, 12
        p = 1.0 / np.arange(1, N + 1)
        first = rng.choice(N, M, p=p / p.sum())
        L = (first[:, None] + np.cumsum(rng.integers(1, 40, (M, knn)), 1)) % N
        L[:, 0] = first
        bad = (np.diff(np.sort(L, 1), axis=1) == 0).any(1)
        L[bad] = (L[bad][:, :1] + np.arange(knn)) % N
        return N, L, deg, np.arange(0, N, 9)
    if kind == "passes":              # keys whose lists take two, three and four passes of the hash table, and hubs
        N, M, knn, deg = 60000, 9000, 48, 33
        mids = np.arange(40)
        share = np.repeat([250, 430, 650, 850], 10)          # lists of each
        L = np.stack([40 + rng.choice(N - 40, knn, replace=False) for _ in range(M)])
        for a, n in zip(mids, share):
            j = rng.choice(M, n, replace=False)
            L[j, a] = a                                      # (its own column: rows stay distinct)
        L[:3000, 47] = 59999
        keep = ~((L[:, :47] == 59999).any(1) & (L[:, 47] == 59999))
        return N, L[keep], deg, np.concatenate([mids, [59999], rng.choice(N, 150, replace=False)])
    # "overflow": one key's co-listed keys all in one residue class of its two passes, more of them than slots
    knn, deg, hub_lists = 48, 32, 425
    N = 42000
    ids = np.arange(1, N)                                    # every other key is in one list: position = id
    res = (((ids.astype(np.uint64) * 2246822519) & 0xffffffff) >> 16) % 2
    crowd = ids[res == 0][:hub_lists * (knn - 1)]
    assert crowd.size == hub_lists * (knn - 1) > 16384
    rest = np.setdiff1d(ids, crowd)
    rest = rest[:rest.size // knn * knn]
    L = np.concatenate([np.concatenate([np.zeros((hub_lists, 1), np.int64), crowd.reshape(hub_lists, knn - 1)], 1),
                        rest.reshape(-1, knn)])
    return N, L, deg, np.concatenate([[0], rng.choice(N, 60, replace=False)])


@pytest.mark.parametrize("kind", ["wide", "passes", "overflow"])
def test_projection_row_kernels_at_their_limits(kind):
    """The ends of what each row kernel takes: more queries than a packed candidate key orders, lists that
    go through the hash table in several passes, a crowd of keys that overflows it and falls to the
    counters in device memory. Sampled rows against the oracle, bit for bit."""
    N, L, deg, rows = _project_case(kind)
    L = np.ascontiguousarray(L.astype(np.int32))
    assert (np.diff(np.sort(L[:5000], 1), axis=1) > 0).all()
    adj, entry = ra.ra_project(torch.from_numpy(L[None]).to(DEV), N, deg)
    adj = adj[0].cpu().numpy()
    pop = np.bincount(L.ravel(), minlength=N)
    pi = np.lexsort((np.arange(N), -pop))
    pos = np.empty(N, np.int64)
    pos[pi] = np.arange(N)
    assert int(entry[0]) == pi[0]
    order = np.argsort(L.ravel(), kind="stable")
    begin = np.searchsorted(L.ravel()[order], np.arange(N + 1))
    for a in rows:
        members = order[begin[a]:begin[a + 1]] // L.shape[1]
        assert adj[a].tolist() == OP.adjacency_row(L, int(a), pop, pos, pi, deg, members), a


def _hub_lists(rng, M, knn, hubs, per_list, others):
    """M lists of knn keys: per_list of the first `hubs` keys, the rest of `others` keys in turn (each of them is in some)."""
    n = knn - per_list
    L = np.empty((M, knn), np.int32)
    L[:, :per_list] = np.argsort(rng.random((M, hubs)), 1)[:, :per_list]
    turn = np.concatenate([rng.permutation(others) for _ in range(-(-M * n // others))])[:M * n].reshape(M, n)
    same = (np.diff(np.sort(turn, 1), axis=1) == 0).any(1)             # (where two turns meet)
    turn[same] = (turn[same][:, :1] + np.arange(n)) % others
    L[:, per_list:] = hubs + turn
    return L[:, rng.permutation(knn)]


@pytest.mark.parametrize("M,knn,hubs,per_list,others,form", [
    (5000, 24, 47, 14, 400, ""), (5000, 24, 48, 14, 400, ""),          # one too few, just enough for bitmaps
    (5000, 24, 64, 14, 400, ""), (5000, 24, 65, 14, 400, ""),
    (5003, 21, 128, 14, 301, "none"), (5001, 24, 129, 14, 400, ""),    # as many as there are bitmaps, one more; places without a key
    (9000, 32, 100, 14, 924, "pad"), (9000, 33, 100, 20, 925, ""),     # 1024 and 1025 populated keys
    (5000, 24, 128, 14, 1200, ""),                                     # more other keys than their counts have room
    (17000, 24, 100, 18, 1500, ""), (17000, 24, 100, 23, 1590, ""),    # other keys of every small class
    (26000, 40, 200, 21, 3896, ""), (26000, 40, 200, 21, 3897, ""),    # 4096, 4097; keys beyond the bitmaps in thousands of lists
    (34011, 64, 90, 24, 8102, ""), (26000, 40, 90, 20, 8103, ""),      # 8192, 8193
    (5000, 24, 128, 14, 300, "twice"), (5000, 40, 100, 14, 500, "twice"),
])
def test_projection_of_lists_with_hubs(M, knn, hubs, per_list, others, form):
    """Graphs whose most popular keys' lists are kept as bitmaps, at the ends of what each row kernel takes, and lists that
    hold a key twice. Every hub and a sample of the other rows, bit for bit, against counts from the lists' sparse
    matrix, ranked in whole numbers."""
    from scipy.sparse import csr_matrix
    rng = np.random.default_rng(M + knn + hubs + others)
    L = _hub_lists(rng, M, knn, hubs, per_list, others)
    N, deg = hubs + others, 32
    if form == "pad":                                    # ids spread over a larger context
        N = 20001
        L = np.sort(rng.choice(N - 1, hubs + others - 1, replace=False).astype(np.int32))[np.minimum(L, hubs + others - 2)]
        L[0, 0] = N - 1
    if form == "none":
        L[rng.random(L.shape) < 0.02] = -1
    if form == "twice":
        j = rng.choice(M, M // 10, replace=False)
        L[j, 1] = L[j, 0]
    L = np.ascontiguousarray(L)
    adj, entry = ra.ra_project(torch.from_numpy(L[None]).to(DEV), N, deg)
    adj = adj[0].cpu().numpy()
    has = L >= 0
    B = csr_matrix((np.ones(has.sum(), np.int64), (np.nonzero(has)[0], L[has])), shape=(M, N))
    pop = np.bincount(L[has], minlength=N)
    if form != "twice" and form != "none":
        assert (pop > 0).sum() == hubs + others - (1 if form == "pad" and pop[N - 1] == 0 else 0)
    pi = np.lexsort((np.arange(N), -pop))
    pos = np.empty(N, np.int64)
    pos[pi] = np.arange(N)
    assert int(entry[0]) == pi[0]
    rows = np.concatenate([pi[:min(hubs, 140)], rng.choice(pi[hubs:hubs + others], 60, replace=False)])
    C = np.asarray((B[:, rows].T @ B).todense())
    for a, c in zip(rows, C):
        t = int(pos[a])
        want = [int(pi[x]) for x in (2 * t + 1, 2 * t + 2) if x < N]
        b = np.nonzero(c)[0]
        b = b[(b != a) & ~np.isin(b, want)]
        # (fractions of whole numbers below 2^20 that differ, differ by more than 2^-40)
        rank = sorted((-(int(c[x]) << 60) // int(pop[a] + pop[x] - c[x]), -int(c[x]), int(x)) for x in b)
        want += [x for _, _, x in rank[:deg - len(want)]]
        assert adj[a].tolist() == want + [-1] * (deg - len(want)), (a, t)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N", [1, 2, 31, 33, 64, 65, 96, 129, 191, 193, 257, 449])
def test_knn_streams_of_few_stages(dtype, N):
    """Streams of one stage, of fewer than are copied ahead, and that end within one: every key in its place."""
    knn = min(N, 33 if N % 2 else 32)
    w = synth.make_integer_case(N, N=N, M=70, d=128, n_q=2, n_kv=1, dtype=dtype, knn=knn)
    L = ra.ra_knn(w.K.to(DEV), w.Q_prefill.to(DEV), knn).cpu().numpy()
    for h in range(2):
        K, Q = to_np(w.K[0, 0]), to_np(w.Q_prefill[0, h])
        assert np.array_equal(L[0, h], OM.knn_lists(Q, K, knn)[0])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,M,knn", [(65, 40, 32), (515, 70, 33), (2600, 130, 64), (17000, 8200, 32)])
def test_knn_of_views_at_odd_offsets(dtype, N, M, knn, knn_selection):
    """Keys and queries that start at any element of their storage: the lists of aligned copies, bit for bit."""
    if dtype == torch.float32 and M > 1000:
        M = 600
    K = torch.randn(2, 2, N, 128, device=DEV).to(dtype)
    Q = torch.randn(2, 4, M, 128, device=DEV).to(dtype)
    want = ra.ra_knn(K, Q, knn)
    for at in (1, 2, 3, 4, 7):
        def moved(t):
            v = torch.empty(t.numel() + at, dtype=dtype, device=DEV)[at:].view(t.shape)
            return v.copy_(t)
        Ka, Qa = moved(K), moved(Q)
        assert Ka.data_ptr() % 16 == at * K.element_size() % 16
        assert torch.equal(ra.ra_knn(Ka, Qa, knn), want)
        assert torch.equal(ra.ra_knn(Ka, Q, knn), want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,M,knn", [(129, 1, 1), (160, 255, 32), (255, 257, 64), (4097, 300, 48), (1024, 1025, 33),
                                     (70000, 96, 32)])
def test_knn_through_8bit_products(dtype, N, M, knn):
    """The later part of the key stream ruled out by 8-bit products (from the 129th key on): one key or a
    ragged stage past the first part, fewer queries than a set, sets and workgroups that end
    ragged, lists of every selection. The lists are those of the whole stream, bit for bit, and the
    oracle's. (Streams that the products give up on: test_knn_filter_gives_up.)"""
    from paper_2409_10516_amd import binding as B
    w = synth.make_llama_layer(N + knn, N, M, n_seq=2, n_q=2, n_kv=1, dtype=dtype)
    K, Q = w.K.to(DEV), w.Q_prefill.to(DEV)
    L = {}
    try:
        for how in (B.RA_TEST_KNN_LDS, B.RA_TEST_KNN_FILTER):
            ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, how)
            L[how] = ra.ra_knn(K, Q, knn).cpu().numpy()
    finally:
        ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_AUTO)
    assert np.array_equal(L[B.RA_TEST_KNN_LDS], L[B.RA_TEST_KNN_FILTER])
    assert np.array_equal(L[B.RA_TEST_KNN_LDS], ra.ra_knn(K, Q, knn).cpu().numpy())
    Kn, Qn = to_np(w.K[1, 0]), to_np(w.Q_prefill[1, 1][:40])
    knn_equivalent(L[B.RA_TEST_KNN_FILTER][1, 1][:40], OM.knn_lists(Qn, Kn, knn)[0], Qn, Kn)


END = 0x7fffffff                                     # of a stream the 8-bit products came through


def _half_streams(N, M, first_half, t):
    """K [N][128] and Q [M][128] of whole numbers that are exact in 8 bits, and t by key. Most queries look at the second
    half of the dimensions, which makes the stream order (place); those of `first_half` look at the first half, where
    the key of place p scores t(p) sum |u|: equal ones tie, and two apart the bound tells them apart."""
    rng = np.random.default_rng(32)
    u = rng.integers(1, 128, 128) * rng.choice([-1, 1], 128)
    u[[0, 64]] = 127
    place = rng.permutation(N)                       # in the stream, up to the order of those that tie
    level = np.where(place < 128, place // 16, 8 + (place - 128) * 190 // max(1, N - 128))
    K = np.concatenate([np.repeat(t(place)[:, None], 64, 1), np.repeat(100 - level[:, None], 64, 1)], 1) * np.sign(u)
    K[place == 5] = 127 * np.sign(u)
    Q = np.where(first_half[:, None] == (np.arange(128) < 64)[None, :], u[None, :], 0)
    return K, Q, place


def _knn_with_resume(K, Q, dtype, heads, knn):
    """Lists [heads][M][knn] with the 8-bit products from the 129th key on, and where each of their launches gave up:
    [launches][heads][wavefronts]."""
    from paper_2409_10516_amd import binding as B
    Kd = torch.from_numpy(K).to(dtype).to(DEV)[None, None]
    Qd = torch.from_numpy(Q).to(dtype).to(DEV).expand(1, heads, *Q.shape).contiguous()
    stops = torch.full((B.RA_TEST_KNN_RESUME_INTS,), -1, dtype=torch.int32, device=DEV)
    try:
        ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_FILTER)
        ra.ra_test_configure(B.RA_TEST_KNN_RESUME, stops.data_ptr())
        got = ra.ra_knn(Kd, Qd, knn).cpu().numpy()[0]
    finally:
        ra.ra_test_configure(B.RA_TEST_KNN_RESUME, 0)
        ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_AUTO)
    stops = stops.cpu().numpy()
    stops = stops[stops != -1]
    # sets of 32 queries per wavefront: as many as leave 2048 wavefronts in the launch
    M = Q.shape[0]
    sets = next(n for n in (4, 2, 1) if n == 1 or -(-M // (256 * n)) * 8 * heads >= 2048)
    waves = -(-M // (256 * sets)) * 8
    return got, stops.reshape(-1, heads, waves), np.arange(waves) * 32 * sets < M


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,knn,M,heads,form", [
    (2600, 32, 300, 1, "ties"), (2639, 64, 257, 2, "ties"),            # the second part is from 640 on, one segment behind
    (18000, 32, 300, 1, "ties"), (17999, 64, 300, 1, "ties"),          # ... from 2688, five segments: gives up before
    (18000, 32, 300, 1, "early"), (18001, 64, 90, 1, "early"),         # ... and comes to the end then
    (18000, 64, 300, 1, "late"),                                       # keeps nothing for four segments, gives up in the second part
    (5000, 32, 600, 128, "ties"), (5000, 33, 300, 256, "ties"),        # two and four sets of queries per wavefront
])
def test_knn_filter_gives_up(dtype, knn, N, M, heads, form):
    """Streams that the bound cannot rule out much of: the workgroups give up, the exact products go on to an eighth of the
    stream, where all are tried again, and from where they give up again to the end. That they give up is
    certain: for the queries that look at the first half of the dimensions (one in every set of 32) each key ties with
    the first part of the stream, and a key that reaches a threshold may not be ruled out; nor can it be before
    wavefronts with half of a workgroup's sets have come through a segment of 512 keys, or one alone through as many as
    make up for the others. Ties to the end, up to the 2500th key ("early") or from the 2176th on ("late"); the last keys of
    the stream are the best of all. Whole numbers: the oracle's lists."""
    first_half = (np.arange(M) % 32 == 31) | (np.arange(M) == M - 1)
    low = {"ties": (0, 0), "early": (2500, N), "late": (128, 2176)}[form]
    K, Q, place = _half_streams(N, M, first_half, lambda p: np.where(
        p >= N - 40, 51 + p % 4, np.where((p >= low[0]) & (p < low[1]), 40, 50)))
    got, stops, live = _knn_with_resume(K, Q, dtype, heads, knn)
    ref = OM.knn_lists(Q[[0, M - 1]], K, knn)[0]
    assert np.array_equal(got, np.broadcast_to(ref[first_half.astype(int)], (heads, M, knn)))
    assert stops.shape[0] == 2 and (stops[:, :, ~live] == END).all()
    a, b = stops[0][:, live], stops[1][:, live]
    again = 128 + -(-(N // 8 - 128) // 512) * 512
    assert (a % 512 == 128).all() and a.min() >= (2176 if form == "late" else 640)
    assert a.max() <= (again if form == "late" else min(again, 2176))
    assert N < 8192 or again == 2688
    if form == "early":
        assert (b == END).all()
    else:
        assert (b >= again + 512).all() and (N < again + 2560 or b.max() <= again + 2560)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,heads", [(300, 1), (257, 3), (33, 2), (600, 128), (300, 256)])
def test_knn_filter_places_without_a_query(dtype, M, heads):
    """What a workgroup has beyond its last query (whole wavefronts, sets, columns of a set) keeps no keys and makes nobody
    give up: the last query, which would stand for all of them, finds its 16 keys in the first segment and rules out the rest,
    all of which are above its threshold at the start."""
    N, knn = 18000, 16
    first_half = np.arange(M) == M - 1
    K, Q, place = _half_streams(N, M, first_half, lambda p: np.where(p < 128, 30, np.where(p < 160, 40, 34)))
    got, stops, live = _knn_with_resume(K, Q, dtype, heads, knn)
    ref = OM.knn_lists(Q[[0, M - 1]], K, knn)[0]
    assert np.array_equal(got, np.broadcast_to(ref[first_half.astype(int)], (heads, M, knn)))
    assert (stops[0][:, live] == 2688).all() and (stops[0][:, ~live] == END).all()         # (the end of the first part)
    assert (stops[1] == END).all()


# powers of two that queries and keys are multiplied by, down to where scores leave the normal range and up
# to where squares do
_SCALES = [(0, 0), (-84, 0), (0, -84), (-45, -45), (-59, -59), (-118, 0), (0, -110), (60, 40), (62, 62), (-126, 0),
           (0, -126), (-70, -70)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("knn", [20, 60])
@pytest.mark.parametrize("q_exp,k_exp", _SCALES)
def test_knn_8bit_bound_holds_at_any_scale(dtype, knn, q_exp, k_exp):
    """The bound's worst pair: queries that are exact in 8 bits and keys that are nothing but rounding error,
    aligned with them. One key of 127s sets every column's scale; the others are t / 256 times the signs of
    the query, so their 8-bit copies are zero and their scores are all in the term |q'| |e|. Most queries
    look at the second half of the dimensions, which makes the stream order; the rest look at the first
    half, where the first 128 keys of the stream are middling, most later ones worse and a few, late, the best:
    with that term lost they are ruled out. The lists of the stream without the filter, bit for bit, and
    the oracle's while every product is a normal number (all sums are exact then: the scales are powers
    of two)."""
    from paper_2409_10516_amd import binding as B
    rng = np.random.default_rng(31)
    N, M = 1500, 96
    u = rng.integers(1, 128, 128) * rng.choice([-1, 1], 128)
    u[[0, 64]] = 127
    place = rng.permutation(N)                       # in the stream
    t = np.where(place < 128, rng.integers(40, 61, N), rng.integers(-115, 40, N))
    late = rng.choice(np.nonzero((place > 300) & (place < N - 1))[0], 70, replace=False)
    t[late] = rng.integers(90, 116, 70)
    K = np.concatenate([np.repeat(t[:, None], 64, 1), np.repeat(100 - place[:, None] // 8, 64, 1)], 1) / 256.0 * np.sign(u)
    K[place == N - 1] = -127.0 * np.sign(u)
    Q = np.zeros((M, 128))
    Q[:60, 64:] = u[64:]
    Q[60:, :64] = u[:64]
    Q[np.arange(60), 65 + np.arange(60)] = 0.0
    Q[np.arange(60, M), 1 + np.arange(M - 60)] = 0.0
    Kd = (torch.from_numpy(K) * 2.0 ** k_exp).to(dtype).to(DEV)[None, None]
    Qd = (torch.from_numpy(Q) * 2.0 ** q_exp).to(dtype).to(DEV)[None, None]
    L = {}
    try:
        for how in (B.RA_TEST_KNN_LDS, B.RA_TEST_KNN_FILTER):
            ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, how)
            L[how] = ra.ra_knn(Kd, Qd, knn).cpu().numpy()[0, 0]
    finally:
        ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_AUTO)
    assert np.array_equal(L[B.RA_TEST_KNN_FILTER], L[B.RA_TEST_KNN_LDS])
    if -118 <= q_exp + k_exp <= 100:                 # (the smallest product is 2^-8, the largest score 2^21)
        assert np.array_equal(L[B.RA_TEST_KNN_LDS], OM.knn_lists(Q, K, knn)[0])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,M,knn,heads", [(640, 130, 32, 24), (1153, 600, 5, 128), (9001, 40, 33, 256), (30000, 65, 64, 2)])
def test_knn_filter_looks_early(dtype, N, M, knn, heads):
    """Queries with a large common component and keys and queries whose dimensions carry very different amounts: most
    blocks are ruled out after the first dimensions, the end of the stream without a product, and how early a
    wavefront looks changes along it. Among the queries: some opposite to the mean (their best keys come last),
    some twenty times longer, the mean itself (nothing is left of it for the products) and zero. Lists of
    the stream without the filter, bit for bit, for one, two and four query sets per wavefront (as many as leave
    2048 wavefronts in the launch)."""
    from paper_2409_10516_amd import binding as B
    g = torch.Generator().manual_seed(N)
    carry = torch.exp(torch.randn(128, generator=g))
    mean = torch.randn(128, generator=g) * 4
    K = torch.randn(1, 2, N, 128, generator=g) * carry
    Q = mean + torch.randn(1, heads, M, 128, generator=g) * carry.flip(0).sqrt()
    Q[:, :, 3::16] = -Q[:, :, 3::16]
    Q[:, :, 5::16] *= 20.0
    Q[:, :, 7::32] = mean
    Q[:, :, 9::32] = 0.0
    Kd, Qd = K.to(dtype).to(DEV), Q.to(dtype).to(DEV)
    L = {}
    try:
        for how in (B.RA_TEST_KNN_LDS, B.RA_TEST_KNN_FILTER):
            ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, how)
            L[how] = ra.ra_knn(Kd, Qd, knn).cpu().numpy()
    finally:
        ra.ra_test_configure(B.RA_TEST_KNN_SELECTION, B.RA_TEST_KNN_AUTO)
    assert np.array_equal(L[B.RA_TEST_KNN_LDS], L[B.RA_TEST_KNN_FILTER])


@pytest.mark.parametrize("call", ["ra_knn", "ra_project", "ra_build_index"])
def test_a_call_without_enough_memory_spoils_no_later_one(call):
    """Sizes no device has the scratch memory for: RA_ENOMEM before anything is read, and the calls that
    follow, of this library and of torch, are as if it had not been made."""
    import ctypes as C
    lib = ra.lib()
    w = synth.make_integer_case(3, N=64, M=16, d=128, n_q=2, n_kv=1, knn=4)
    Kd, Qd = w.K.to(DEV), w.Q_prefill.to(DEV)
    want = ra.ra_knn(Kd, Qd, 4).cpu()
    big, p, h = 0x3fffffff, Kd.data_ptr(), C.c_void_p()
    torch.cuda.synchronize()
    if call == "ra_knn":
        rc = lib.ra_knn(p, p, 0, 64, 1, 1, big, 1, 128, 8, None, p)
    elif call == "ra_project":
        rc = lib.ra_project(p, 64, big, 1, 8, 8, None, p, p)
    else:
        rc = lib.ra_build_index(p, p, 0, 64, 1, 1, big, 1, 128, 8, 8, None, C.byref(h))
    assert rc == 4 and "memory" in lib.ra_last_error().decode()
    assert not h.value
    assert torch.equal(ra.ra_knn(Kd, Qd, 4).cpu(), want)
    assert float((torch.ones(1000, device=DEV) * 2).sum()) == 2000.0


def test_knn_without_room_for_the_8bit_copies():
    """A device too full for the copies the 8-bit products need, with room for the rest: the same lists."""
    N, n_q, knn = 131072, 8, 32
    w = synth.make_llama_layer(4, N, 1500, n_seq=1, n_q=n_q, n_kv=2, device=DEV)
    want = ra.ra_knn(w.K, w.Q_prefill, knn)          # (the copies are used at this size)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    full, leave, step = [], 80 << 20, 64 << 30
    try:
        while step >= 4 << 20:
            free = torch.cuda.mem_get_info()[0]
            if free <= leave + (4 << 20):
                break
            step = min(step, free - leave)
            try:
                full.append(torch.empty(step, dtype=torch.uint8, device=DEV))
            except torch.cuda.OutOfMemoryError:
                step //= 2
        free = torch.cuda.mem_get_info()[0]
        assert 40 << 20 < free < n_q * N * 128       # (what the copies of the keys alone take)
        got = torch.empty_like(want)
        rc = ra.lib().ra_knn(w.K.data_ptr(), w.Q_prefill.data_ptr(), 1, 1, n_q, 2, N, 1500, 128, knn, None, got.data_ptr())
        assert rc == 0, ra.lib().ra_last_error()
        assert torch.equal(got, want)
    finally:
        full.clear()
        torch.cuda.empty_cache()


@pytest.mark.parametrize("M", [131071, 131072])
@pytest.mark.parametrize("H", [900, 135000])
def test_projection_candidates_in_one_word(M, H):
    """A ranked candidate's overlap, count and position share 64 bits where the largest popularity and the number of populated
    keys allow it (one key in all of 131071 lists), and do not beyond (131072): the same rows, of keys with a hundred lists in
    a small graph and with a few in one of 135000 populated keys. Many equal overlaps; -1 in some rows."""
    rng = np.random.default_rng(H)
    N, deg = H + 10, 24
    L = np.zeros((M, 3), np.int32)
    L[:, 1] = 1 + rng.integers(0, 8, size=M) if H < 1000 else 1 + rng.permutation(M) % (H - 1)
    L[:, 2] = 9 + rng.integers(0, H - 9, size=M) if H < 1000 else 1 + (rng.permutation(M) + M) % (H - 1)
    same = L[:, 1] == L[:, 2]
    L[same, 2] = L[same, 2] % (H - 1) + 1
    pop = np.bincount(L.ravel(), minlength=N)
    assert pop[0] == M and ((pop > 0).sum() >= 131072 if H > 1000 else 800 < (pop > 0).sum() < 1024)
    rows = np.arange(N) if H < 1000 else rng.choice(N, 500, replace=False)
    adj, entry = ra.ra_project(torch.from_numpy(L[None]).to(DEV), N, deg)
    radj, rent = OP.project(L, N, deg, rows=rows)
    assert int(entry[0]) == rent
    adj = adj[0].cpu().numpy()
    for a in rows:
        assert np.array_equal(adj[a], radj[a]), (a, adj[a], radj[a])
