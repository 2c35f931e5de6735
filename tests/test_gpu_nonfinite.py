"""Inputs that hold infinities and NaN, against the oracle's arithmetic: what a row that is attended to holds belongs in the
result, what a row that is not holds does not. GPU only."""
import numpy as np
import pytest
import torch

import paper_2409_10516_amd as ra
from oracle import attention as OA, search as OS
from paper_2409_10516_amd import binding as B
from tests.util import out_close, lse_close, to_np, tol_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _same(got, ref, tol):
    """The same infinities in the same places, the rest within the tolerance (relative to the largest of the rest)."""
    got = np.asarray(got, np.float64)
    fin = np.isfinite(ref)
    assert not np.isnan(ref).any() and np.array_equal(got[~fin], ref[~fin]), (got[~fin], ref[~fin])
    assert np.isfinite(got[fin]).all() and out_close(got[fin], ref[fin], tol)


def _small(rng, *shape):
    """Values whose logits are of the order of one: no weight of a softmax over them underflows."""
    return torch.from_numpy((0.5 * rng.standard_normal(shape)).astype(np.float32))


def _random_graph(rng, heads, N, deg):
    adj = rng.integers(0, N, size=(heads, N, deg)).astype(np.int32)
    return torch.from_numpy(adj), torch.from_numpy(rng.integers(0, N, size=heads).astype(np.int32))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_q,n_kv,deg,expand,ef,topk,helpers", [
    (1, 1, 8, 4, 128, 100, True), (2, 1, 16, 32, 128, 100, True), (2, 1, 16, 32, 128, 1, True), (4, 1, 16, 32, 200, 193, True),
    (1, 1, 16, 32, 300, 100, True), (400, 400, 16, 8, 100, 97, True), (2, 1, 16, 32, 128, 100, False),
    (1, 1, 16, 32, 300, 70, False), (3, 1, 16, 32, 128, 45, True), (6, 2, 8, 4, 64, 33, True)])
def test_infinite_values_in_the_last_rows(dtype, n_q, n_kv, deg, expand, ef, topk, helpers):
    """An infinity in the value row of the last id found and in the newest token's: lane groups left without a row of their own
    in the last pass over the rows (workgroups of 256, 512 and 1024 threads, few rows and several passes) must not add them in
    with a weight of zero. The static set by helpers and by the heads themselves (off, or groups they do not serve)."""
    rng = np.random.default_rng(n_q + ef + topk)
    N, sink, window = 500, 3, 50
    adj, ent = _random_graph(rng, n_q, N, deg)
    K, V, q = (_small(rng, *s).to(dtype) for s in ((1, n_kv, N, 128), (1, n_kv, N, 128), (1, n_q, 128)))
    idx = ra.ra_index_import(adj, ent, 1, n_q, n_kv)
    idx.configure(B.RA_CFG_HELPERS, B.RA_HELPERS_ON if helpers else B.RA_HELPERS_OFF)
    ids = ra.ra_decode_step(q.to(DEV), idx, K.to(DEV), V.to(DEV), sink, window, topk, ef, expand)[2].cpu().numpy()
    for kv in range(n_kv):
        last = ids[0, kv * (n_q // n_kv)]
        V[0, kv, last[last >= 0][-1], 3] = np.inf
        V[0, kv, last[last >= 0][-1], 77] = -np.inf
        V[0, kv, N - 1, 120] = np.inf
    out, lse, ids2, _ = ra.ra_decode_step(q.to(DEV), idx, K.to(DEV), V.to(DEV), sink, window, topk, ef, expand)
    assert np.array_equal(ids2.cpu().numpy(), ids)
    for h in range(n_q) if n_q < 10 else (0, 133, n_q - 1):
        rows = np.concatenate([OA.static_ids(N, sink, window), ids[0, h][ids[0, h] >= 0]])
        ref, rl = OA.partial_attention(to_np(q[0, h]), to_np(K[0, h * n_kv // n_q]), to_np(V[0, h * n_kv // n_q]), rows)
        _same(out[0, h].cpu().numpy(), ref, tol_for(dtype))
        assert lse_close(float(lse[0, h]), rl, tol_for(dtype))
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_seq,n_q,n_kv,window,topk", [(1, 2, 2, 70, 9), (2, 32, 8, 500, 64), (1, 8, 1, 100, 130), (20, 32, 4, 640, 100),
                                                        (1, 4, 1, 4100, 40), (1, 8, 1, 4100, 40)])
def test_values_of_a_row_that_is_not_attended_to(n_seq, n_q, n_kv, window, topk, dtype):
    """Places without a row, in the last chunk of a set, in a list padded with -1, and in a long range's last tile, read row 0: with
    no sink it is in neither set, and the infinity and the NaN in its value row are in no result. One in a row that is attended to
    is. Chunks of one head and of several, a long range's on the matrix cores and on the vector units."""
    rng = np.random.default_rng(n_seq * n_q + topk)
    N, lists = 5000, torch.full((n_seq, n_q, topk), -1, dtype=torch.int32)
    K, V, q = (_small(rng, *s).to(dtype) for s in ((n_seq, n_kv, N, 128), (n_seq, n_kv, N, 128), (n_seq, n_q, 128)))
    for s in range(n_seq):
        for h in range(n_q):
            n = topk - (h % 3)
            lists[s, h, :n] = 1 + torch.from_numpy(rng.permutation(N - window - 1)[:n])
    V[:, :, 0, 5] = np.inf
    V[:, :, 0, 6] = np.nan
    V[:, :, N - 1, 100] = -np.inf
    idx = ra.ra_index_import(torch.full((n_seq * n_q, N, 1), -1, dtype=torch.int32), torch.zeros(n_seq * n_q, dtype=torch.int32),
                             n_seq, n_q, n_kv)
    for noalloc in (False, True) if n_seq * n_q * (window + topk) < 20000 else (False,):
        out, lse = ra.ra_attend(q.to(DEV), idx, K.to(DEV), V.to(DEV), 0, window, lists.to(DEV), noalloc=noalloc)
        for s, h in [(0, 0), (0, n_q - 1), (n_seq - 1, 1)]:
            rows = np.concatenate([OA.static_ids(N, 0, window), lists[s, h][lists[s, h] >= 0].numpy()])
            ref, rl = OA.partial_attention(to_np(q[s, h]), to_np(K[s, h * n_kv // n_q]), to_np(V[s, h * n_kv // n_q]), rows)
            _same(out[s, h].cpu().numpy(), ref, tol_for(dtype))
            assert lse_close(float(lse[s, h]), rl, tol_for(dtype))
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_q,n_kv", [(1, 1), (2, 1), (4, 1), (8, 1), (3, 1)])
def test_full_attention_with_infinite_values(n_q, n_kv, dtype):
    """Infinities in the first and the last of 4321 value rows (a last chunk with places that read row 0)."""
    rng, N = np.random.default_rng(n_q), 4321
    K, V, q = (_small(rng, *s).to(dtype) for s in ((1, n_kv, N, 128), (1, n_kv, N, 128), (1, n_q, 128)))
    V[0, 0, 0, 9] = np.inf
    V[0, 0, N - 1, 64] = -np.inf
    out, lse = ra.ra_full_attention(q.to(DEV), K.to(DEV), V.to(DEV))
    for h in range(n_q):
        ref, rl = OA.full_attention(to_np(q[0, h]), to_np(K[0, 0]), to_np(V[0, 0]))
        _same(out[0, h].cpu().numpy(), ref, tol_for(dtype))
        assert lse_close(float(lse[0, h]), rl, tol_for(dtype))


def _ranked(q, rows):
    """Inner products whose infinities the oracle's walk can subtract: beyond every finite one, equal among themselves."""
    with np.errstate(invalid="ignore"):
        s = np.asarray(rows, np.float64) @ np.asarray(q, np.float64)
    assert not np.isnan(s).any()
    return np.clip(s, -1e6, 1e6)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("plus,minus", [(0.01, 0.0), (0.0, 0.3), (0.3, 0.3), (1.0, 0.0), (0.0, 1.0)])
@pytest.mark.parametrize("deg,expand,ef,n_seeds,heads", [
    (8, 1, 40, 0, 1), (32, 40, 64, 0, 1), (32, 40, 1100, 0, 1), (33, 7, 16, 0, 1), (32, 64, 256, 2048, 1), (8, 64, 16, 500, 1),
    (8, 20, 100, 64, 1), (16, 32, 100, 400, 400), (64, 9, 300, 0, 1)])
def test_walks_over_infinite_scores(deg, expand, ef, n_seeds, heads, plus, minus, dtype):
    """Keys whose score is an infinity, some, many and all of them: in start sets (their bins have no width then), in steps that
    keep few, many and more candidates than the beam holds. They rank above and below all others, ties by id: the oracle's
    walk. The attention over what is found: minus infinity has no weight."""
    rng = np.random.default_rng(deg + ef + int(10 * plus) + int(100 * minus))
    N = 3000
    adj = rng.integers(0, N, size=(1, N, deg)).astype(np.int32)
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < N, 2 * t + 1 + j, -1)
    K = rng.integers(-3, 4, size=(N, 128)).astype(np.float32)
    q = rng.integers(1, 4, size=128).astype(np.float32)
    kind = rng.random(N)
    K[kind < plus, 17] = np.inf
    K[kind > 1 - minus, 99] = -np.inf
    K[(kind < plus) & (kind > 1 - minus), 99] = 0
    V = rng.standard_normal((N, 128)).astype(np.float32)
    idx = ra.ra_index_import(torch.from_numpy(np.repeat(adj, heads, 0)), torch.zeros(heads, dtype=torch.int32), 1, heads, 1)
    idx.configure(B.RA_CFG_SEEDS, n_seeds)
    Kd, Vd = (torch.from_numpy(x)[None, None].to(dtype).to(DEV) for x in (K, V))
    qd = torch.from_numpy(q).to(dtype).repeat(1, heads, 1).to(DEV)
    topk = min(ef, 50)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 20, topk, ef, expand)
    out, lse, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Vd, 4, 20, topk, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    seeds = OS.backbone_seeds(adj[0], 0, n_seeds) if n_seeds else None
    W = OA.static_ids(N, 4, 20)
    ref, rst = OS.greedy_search(q, K, adj[0], 0, ef, topk, expand, exclude=W, seeds=seeds, score_fn=_ranked)
    for h in (0, heads - 1):
        assert ids[0, h].tolist() == ref.tolist()
        assert st[0, h].tolist() == [rst["n_visited"], rst["n_expanded"], rst["n_iters"], rst["n_returned"]]
    rows = np.concatenate([W, ref[ref >= 0]])
    scores = _ranked(q, K[rows])
    if scores.max() < 1e6 and scores.max() > -1e6:
        Vn = to_np(Vd[0, 0])
        ro, rl = OA.partial_attention(q, np.where(np.isinf(K), -1e30, K), Vn, rows)
        assert out_close(out[0, 0].cpu().numpy(), ro, tol_for(dtype)) and lse_close(float(lse[0, 0]), rl, tol_for(dtype))
    idx.free()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("deg,expand,ef,n_seeds", [(8, 1, 40, 0), (32, 40, 64, 0), (32, 64, 256, 2048), (64, 9, 300, 0), (8, 20, 100, 64)])
@pytest.mark.parametrize("where", ["some keys", "all keys", "query"])
def test_walks_over_scores_that_are_no_numbers(where, deg, expand, ef, n_seeds, dtype):
    """NaN in keys or in the query: the walk ends, counts what it has seen, and returns ids that are distinct, in range and
    outside the static set."""
    rng = np.random.default_rng(deg + ef)
    N = 2500
    adj = rng.integers(0, N, size=(1, N, deg)).astype(np.int32)
    t = np.arange(N)
    for j in (0, 1):
        adj[:, :, j] = np.where(2 * t + 1 + j < N, 2 * t + 1 + j, -1)
    K = rng.integers(-3, 4, size=(N, 128)).astype(np.float32)
    q = rng.integers(-3, 4, size=128).astype(np.float32)
    if where == "query":
        q[5] = np.nan
    else:
        K[:: 1 if where == "all keys" else 7, 60] = np.nan
    idx = ra.ra_index_import(torch.from_numpy(adj), torch.zeros(1, dtype=torch.int32), 1, 1, 1)
    idx.configure(B.RA_CFG_SEEDS, n_seeds)
    Kd, qd = torch.from_numpy(K)[None, None].to(dtype).to(DEV), torch.from_numpy(q)[None, None].to(dtype).to(DEV)
    topk = min(ef, 50)
    ids, st = ra.ra_search(qd, idx, Kd, 4, 20, topk, ef, expand)
    _, _, ids_d, st_d = ra.ra_decode_step(qd, idx, Kd, Kd, 4, 20, topk, ef, expand)
    assert torch.equal(ids, ids_d) and torch.equal(st, st_d)
    got, (visited, expanded, iters, returned) = ids[0, 0].cpu().numpy(), st[0, 0].tolist()
    real = got[got >= 0]
    assert len(real) == returned and len(set(real.tolist())) == returned and (got[returned:] == -1).all()
    assert not set(real.tolist()) & set(OA.static_ids(N, 4, 20).tolist()) and real.max(initial=0) < N
    assert ef <= visited <= N and ef <= expanded <= visited and iters >= 1
    idx.free()
