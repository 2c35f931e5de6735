"""Inputs that hold infinities and NaN, against the oracle's arithmetic: what a row that is attended to holds belongs in the
result, what a row that is not holds does not. GPU only."""
import numpy as np
import pytest
import torch

import paper_2409_10516_amd as ra
from oracle import attention as OA
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
