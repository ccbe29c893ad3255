"""Kernels and dispatch branches for calls that do not fill the device: sizes around their tiles,
slices and splits, against the oracle."""
import re

import numpy as np
import pytest
import torch

from oracle import basa_oracle as o
from paper_2605_19726_amd import binding as bd
from parity_util import check_output, np64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _qkv(hq, hk, Lq, Lk, d, dtype, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    r = lambda h, L: torch.randn((1, h, L, d), generator=g, device=DEV).to(dtype)
    return r(hq, Lq), r(hk, Lk), r(hk, Lk)


def _lists(hq, n_q, n_k, seed, stride):
    """Ascending lists of different lengths (1 .. n_k), the rest of a row filled with an invalid entry."""
    rng = np.random.default_rng(seed)
    count = rng.integers(1, n_k + 1, (1, hq, n_q))
    cols = np.full((1, hq, n_q, stride), n_k + 7)
    for idx in np.ndindex(count.shape):
        cols[idx][:count[idx]] = np.sort(rng.choice(n_k, count[idx], replace=False))
    t = lambda a: torch.from_numpy(a.astype(np.int32)).to(DEV)
    return t(count), t(cols), count, cols


def _perm(h, L, seed):
    return torch.stack([torch.randperm(L, generator=torch.Generator().manual_seed(seed + i)) for i in range(h)]).to(DEV, torch.int32)[None]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,shape", [(torch.float32, 0), (torch.bfloat16, 0), (torch.bfloat16, 3)])
@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("Lq,Lk", [(1, 1), (31, 33), (65, 129), (200, 1000), (130, 5000), (2048 + 77, 2048 + 77)])
def test_attention_of_short_calls_against_the_oracle(dtype, shape, d, block, Lq, Lk, causal):
    hq, hk = 2, 1
    Q, K, V = _qkv(hq, hk, Lq, Lk, d, dtype, seed=Lq + Lk + d)
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    cnt, cols, cnt_h, cols_h = _lists(hq, n_q, n_k, Lq + 3 * Lk, n_k)
    pq, pk = _perm(hq, Lq, 1), _perm(hk, Lk, 50)
    out, lse = bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, want_lse=True, attn_shape=shape, causal=causal)
    torch.cuda.synchronize()
    for h in range(hq):
        lists = [cols_h[0, h, g, :cnt_h[0, h, g]] for g in range(n_q)]
        args = (np64(Q[0, h]), np64(K[0, 0]), np64(V[0, 0]), pq[0, h].cpu().numpy(), pk[0, 0].cpu().numpy(), lists, block)
        fn = o.sparse_attention_causal if causal else o.sparse_attention
        ref, ref_lse = fn(*args, return_lse=True)
        check_output(np64(out[0, h]), ref, dtype == torch.bfloat16, f"head {h}")
        got = lse[0, h].cpu().numpy()
        assert np.array_equal(np.isinf(got), np.isinf(ref_lse))
        fin = np.isfinite(ref_lse)
        np.testing.assert_allclose(got[fin], ref_lse[fin], rtol=0, atol=2e-2 if dtype == torch.bfloat16 else 1e-4)


@pytest.mark.parametrize("d,block", [(64, 64), (128, 128)])
@pytest.mark.parametrize("Lk", [33, 64 + 1, 300])
def test_f32_infinite_scores_and_an_infinite_last_value_row(d, block, Lk):
    """Keys whose scores are -inf carry no weight, also when a whole tile is made of them, and an infinity in
    the last V row (what the positions past the end are clamped to) comes out as that infinity."""
    Q, K, V = _qkv(1, 1, 40, Lk, d, torch.float32, seed=Lk)
    Q[..., 0] = 1e20
    K[..., 0] = 0.0
    K[..., :32, 0] = -1e20                       # score -1e40: below the smallest float
    V[0, 0, -1, 5] = float("inf")
    out = bd.basa_dense_attn(Q, K, V, block)
    torch.cuda.synchronize()
    q, k, v = Q[0, 0].cpu().double(), K[0, 0].cpu().double(), V[0, 0].cpu().double()
    ref = torch.softmax(q[:, 1:] @ k[32:, 1:].T / d ** 0.5, -1) @ v[32:]
    np.testing.assert_allclose(out[0, 0].cpu().double().numpy(), ref.numpy(), rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("hq,d,block,Lk,hidden", [(2, 64, 64, 300, 64), (3, 128, 128, 1000, 128), (2, 128, 128, 4096, 64),
                                                  (2, 64, 128, 4096 + 33, 1500), (1, 128, 64, 8200, 8000)])
def test_bf16_keys_whose_scores_are_minus_infinity(hq, d, block, Lk, hidden, shape):
    """As above in bf16, on whole lists and (shape 0, above 32 tiles) on split ones: the hidden keys fill the first tile of a
    list, of a part of it, or whole parts.  Every other query sees all keys, so that within a wave some have a maximum
    and some do not; queries 4 to 7 have scores shifted by +-300 (log2 units), which the pass without running maxima
    hands on to the one with them; query 8 sees no key at all and comes out as zeros."""
    Lq = 200
    Q, K, V = _qkv(hq, 1, Lq, Lk, d, torch.bfloat16, seed=Lk + d)
    Q[:, :, 0::2, 0], Q[:, :, 1::2, 0] = 1e20, 0.0
    K[..., 0] = 0.0
    K[..., :hidden, 0] = -1e20                   # times 1e20: below the smallest float
    K[..., 1], Q[..., 1], Q[..., 8, 1] = 1e20, 0.0, -1e20
    K[..., 2], Q[..., 2] = 16.0, 0.0             # the same for every key: shifts all scores of a query
    shift = 300.0 / 1.4426950408889634 * d ** 0.5 / 16.0
    Q[:, :, 4:6, 2], Q[:, :, 6:8, 2] = shift, -shift
    out, lse = bd.basa_sparse_attn(Q, K, V, None, None, block, want_lse=True, attn_shape=shape)
    torch.cuda.synchronize()
    for h in range(hq):
        q, k, v = np64(Q[0, h]), np64(K[0, 0]), np64(V[0, 0])
        with np.errstate(over="ignore"):
            s = (q @ k.T / d ** 0.5).astype(np.float32).astype(np.float64)
        m = s.max(1, keepdims=True)
        p = np.exp(s - np.where(np.isinf(m), 0.0, m))
        l = p.sum(1, keepdims=True)
        check_output(np64(out[0, h]), p @ v / np.maximum(l, 1e-300), True, f"head {h}")
        got = lse[0, h].cpu().numpy()
        assert got[8] == -np.inf
        rest = np.arange(Lq) != 8
        np.testing.assert_allclose(got[rest], (m + np.log(np.maximum(l, 1e-300)))[rest, 0], rtol=1e-4, atol=3e-2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,Lk,causal", [(64, 300, False), (128, 4096, False), (128, 4096, True)])
def test_nan_of_a_query_reaches_its_output_row(dtype, d, Lk, causal):
    """Also where the list is split over workgroups that each saw no number (above 32 tiles in bf16, all sizes in f32)."""
    Lq = 200
    Q, K, V = _qkv(2, 1, Lq, Lk, d, dtype, seed=Lk)
    Q[0, 1, 77] = float("nan")
    out, lse = bd.basa_dense_attn(Q, K, V, 128, want_lse=True, causal=causal)
    torch.cuda.synchronize()
    nan = torch.zeros(2, Lq, dtype=torch.bool)
    nan[1, 77] = True
    assert torch.equal(torch.isnan(lse[0]).cpu(), nan)
    assert torch.equal(torch.isnan(out[0]).all(-1).cpu(), nan) and torch.equal(torch.isnan(out[0]).any(-1).cpu(), nan)


@pytest.mark.parametrize("d,L", [(64, 300), (64, 3000), (128, 700), (128, 5000)])
def test_f32_lse_of_large_scores(d, L):
    """Scores near 500 to 2000.  The result is a rounded fp32 number: half a unit in its last place (0.55 with the small
    terms).  The d additions behind the large product of a score round to its place, ulp / sqrt(12) each, sqrt(d) together,
    and 1 / sqrt(d) scales them; averaging over the L / e keys that count (scores of unit variance) leaves the standard
    deviation below, of which four cover 200 queries."""
    Q, K, V = _qkv(3, 1, 200, L, d, torch.float32, seed=d + L)
    K[..., 2], Q[..., 2] = 16.0, torch.tensor([300.0, -300.0, 1000.0], device=DEV)[None, :, None]
    _, lse = bd.basa_dense_attn(Q, K, V, 128, want_lse=True)
    torch.cuda.synchronize()
    for h in range(3):
        s = np64(Q[0, h]) @ np64(K[0, 0]).T / d ** 0.5
        m = s.max(1)
        ref = m + np.log(np.exp(s - m[:, None]).sum(1))
        ulp = lambda x: np.spacing(np.abs(x).astype(np.float32)).astype(np.float64)
        bound = 0.55 * ulp(ref) + 4.0 * ulp(ref * d ** 0.5) / 12 ** 0.5 / (L / np.e) ** 0.5
        assert (np.abs(lse[0, h].cpu().numpy() - ref) <= bound).all(), h


@pytest.mark.parametrize("d,block,L", [(64, 64, 300), (128, 128, 200), (128, 64, 4000)])
def test_small_calls_with_scores_outside_the_range_of_the_pass_without_running_maxima(d, block, L):
    """Scores near +300 and near -300 (log2 units): the 128-query shape has to repeat itself with running maxima
    (L = 4000 instead splits its lists, which always carry maxima)."""
    g = torch.Generator().manual_seed(d + L)
    u = torch.randn(d, generator=g)
    u /= u.norm()
    amp = (300.0 * d ** 0.5 / 1.4426950408889634) ** 0.5
    Q, K, V = (torch.randn(1, 3, L, d, generator=g) * 0.5 for _ in range(3))
    Q[0, :2] += amp * u
    K[0, 0] += amp * u
    K[0, 1] -= amp * u
    Q, K, V = (t.to(torch.bfloat16).to(DEV) for t in (Q, K, V))
    out, lse = bd.basa_dense_attn(Q, K, V, block, want_lse=True)
    torch.cuda.synchronize()
    for h in range(3):
        s = np64(Q[0, h]) @ np64(K[0, h]).T / d ** 0.5
        m = s.max(1, keepdims=True)
        p = np.exp(s - m)
        check_output(np64(out[0, h]), p @ np64(V[0, h]) / p.sum(1, keepdims=True), True, f"head {h}")
        np.testing.assert_allclose(lse[0, h].cpu().numpy(), m[:, 0] + np.log(p.sum(1)), rtol=1e-4, atol=3e-2)


@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("d,block", [(64, 64), (128, 128)])
@pytest.mark.parametrize("hq,Lq,Lk", [(2, 1, 1), (2, 64 * 33 - 5, 64 * 65 + 1), (4, 300, 20000), (90, 64 * 64 * 2, 64 * 129)])
def test_block_scores_of_small_maps(hq, Lq, Lk, d, block, beta):
    """The 32 x 32 tiles of small maps (2 to 540 tiles of 64 x 64)."""
    Q, K, _ = _qkv(hq, 2, Lq, Lk, d, torch.bfloat16, seed=Lq + d)
    sel = bd.basa_select(Q, K, block, 0.5, beta, bd.SORT_NONE, want_scores=True)
    torch.cuda.synchronize()
    for h in (0, hq - 1):
        mq, vq = o.block_stats(np64(Q[0, h]), block)
        mk, vk = o.block_stats(np64(K[0, h // (hq // 2)]), block)
        ref = o.baseline_logits(mq, mk)
        if beta:
            ref = ref + beta * o.diag_compensation(mq, vq, mk, vk)
        np.testing.assert_allclose(sel.scores[0, h].cpu().numpy(), ref, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("window", [0, 128, 1024, 9 * 128, 5120])
@pytest.mark.parametrize("heads,L", [(2, 1), (3, 255), (2, 257), (2, 1024), (2, 1025), (1, 4097), (2, 16385), (1, 70001),
                                     (8, 65536), (8, 65537)])
def test_norm_sort_around_the_tile_and_pass_sizes(heads, L, window):
    """Small tiles and ranked runs (2 to 69 of them, one to three passes), and past 2^19 words the large tiles."""
    g = torch.Generator(device=DEV).manual_seed(L)
    x = torch.randn((1, heads, L, 64), generator=g, device=DEV).to(torch.bfloat16)
    if L > 300:
        x[0, 0, 100:140] = x[0, 0, 200:240]              # exact ties
    perm = bd.basa_norm_sort(x, 64 if window % 128 else 128, window=window)
    torch.cuda.synchronize()
    for h in {0, heads - 1}:
        assert np.array_equal(perm[0, h].cpu().numpy(), o.norm_sort(np64(x[0, h]), window)), h


@pytest.mark.parametrize("dtype,d,block", [(torch.bfloat16, 128, 128), (torch.float32, 64, 64)])
@pytest.mark.parametrize("hq,hk,Lq,Lk", [(4, 2, 1, 9000), (4, 2, 2000, 70), (2, 2, 5000, 3000), (8, 4, 500, 131072)])
def test_sort_and_features_of_sequences_of_different_lengths(hq, hk, Lq, Lk, dtype, d, block):
    """Q and K share the launches although their tiles, passes and block counts differ (the last: too many words)."""
    Q, K, _ = _qkv(hq, hk, Lq, Lk, d, dtype, seed=Lq)
    sel = bd.basa_select(Q, K, block, 0.5, want_scores=True)
    torch.cuda.synchronize()
    for h in (0, hq - 1):
        q, k = np64(Q[0, h]), np64(K[0, h // (hq // hk)])
        ref = o.select(q, k, block, 0.5, 1.0)
        assert np.array_equal(sel.perm_q[0, h].cpu().numpy(), ref["perm_q"])
        assert np.array_equal(sel.perm_k[0, h // (hq // hk)].cpu().numpy(), ref["perm_k"])
        np.testing.assert_allclose(sel.scores[0, h].cpu().numpy(), ref["logits"], rtol=2e-5, atol=2e-5)


def test_causal_blocks_ordered_by_index_with_a_malformed_permutation():
    """Entries that are no index fall back to their position, repeated ones leave places of the block without a row:
    wrong rows, but nothing outside the tensors, and the other blocks come out right."""
    L, d, block = 700, 128, 128
    Q, K, V = _qkv(1, 1, L, L, d, torch.bfloat16, seed=9)
    pk = torch.arange(L, dtype=torch.int32)
    pk[:100] = torch.tensor([-7, 10 ** 6, 5, 5] * 25, dtype=torch.int32)
    cnt = torch.full((1, 1, 6), 1, dtype=torch.int32, device=DEV)
    cols = torch.tensor([0, 0, 0, 1, 1, 2], dtype=torch.int32, device=DEV).reshape(1, 1, 6, 1)
    for shape in (0, 3):
        out = bd.basa_sparse_attn(Q, K, V, cnt, cols, block, None, pk.reshape(1, 1, L).to(DEV), attn_shape=shape, causal=True)
        torch.cuda.synchronize()
        ref, _ = o.sparse_attention_causal(np64(Q[0, 0]), np64(K[0, 0]), np64(V[0, 0]), np.arange(L), np.arange(L),
                                           [[0], [0], [0], [1], [1], [2]], block, return_lse=True)
        check_output(np64(out[0, 0, 384:]), ref[384:], True, "blocks without a malformed entry")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("hq,hk,Lq,Lk,d,block", [(4, 2, 300, 140000, 64, 128), (2, 1, 1030, 70000, 128, 64), (16, 8, 8200, 8200, 128, 128)])
def test_tiles_of_listed_blocks_only(hq, hk, Lq, Lk, d, block, causal):
    """K and V large enough for the bitmaps of listed blocks: rows of different lengths, with invalid entries behind and
    among them, the last block listed by some; unlisted tiles of the workspace hold NaN."""
    Q, K, V = _qkv(hq, hk, Lq, Lk, d, torch.bfloat16, seed=Lk)
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    stride = max(2, n_k // 12)
    rng = np.random.default_rng(Lk)
    cols = np.full((1, hq, n_q, stride), n_k + 3)
    cnt = rng.integers(1, stride + 1, (1, hq, n_q))
    for idx in np.ndindex(cnt.shape):
        own = rng.choice(n_k, cnt[idx], replace=False)
        own[0] = n_k - 1 if idx[2] % 2 else own[0]
        own = np.unique(own)
        cols[idx][:cnt[idx]] = np.append(own, [n_k + 9] * (cnt[idx] - len(own)))
    t = lambda a: torch.from_numpy(a.astype(np.int32)).to(DEV)
    ws = torch.full((bd.attn_workspace_size(Q, K, bd.params(block, 0.5, causal=causal)),), 0xFF, dtype=torch.uint8, device=DEV)
    out = bd.basa_sparse_attn(Q, K, V, t(cnt), t(cols), block, ws=ws, causal=causal)
    torch.cuda.synchronize()
    ident_q, ident_k = np.arange(Lq), np.arange(Lk)
    for h in (0, hq - 1):
        kh = h // (hq // hk)
        k, v = np64(K[0, kh]), np64(V[0, kh])
        for g in (0, n_q // 2, n_q - 1):
            rows = ident_q[g * block:(g + 1) * block]
            keys = np.concatenate([ident_k[c * block:(c + 1) * block] for c in cols[0, h, g, :cnt[0, h, g]] if c < n_k])
            s = np64(Q[0, h])[rows] @ k[keys].T / d ** 0.5
            if causal:
                s = np.where(keys[None] <= rows[:, None] + (Lk - Lq), s, -np.inf)
            m = s.max(1, keepdims=True)
            p = np.exp(s - np.where(np.isinf(m), 0.0, m))
            ref = p @ v[keys] / np.maximum(p.sum(1, keepdims=True), 1e-300)
            check_output(np64(out[0, h])[rows], ref, True, f"head {h} block {g}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,d,block", [(torch.bfloat16, 128, 128), (torch.bfloat16, 64, 64), (torch.float32, 128, 128)])
def test_split_lists_with_several_batch_entries_and_less_workspace(dtype, d, block, causal):
    """Three entries in a token-major buffer, lists of up to 80 tiles: split as far as the workspace has room for partial
    rows (all of it, two parts per list, none).  Every entry against the oracle each time.  In bf16 the workspace shows
    in the bits: without room the lists stay whole, as those of attn_shape 3 are."""
    b, hq, hk, Lq, Lk = 3, 4, 2, 300, 5000
    g = torch.Generator(device=DEV).manual_seed(d + block)
    r = lambda h, L: torch.randn((b, L, h, d), generator=g, device=DEV).to(dtype).permute(0, 2, 1, 3)
    Q, K, V = r(hq, Lq), r(hk, Lk), r(hk, Lk)
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    lists = [_lists(hq, n_q, n_k, 70 + i, n_k) for i in range(b)]
    cnt, cols = torch.cat([x[0] for x in lists]), torch.cat([x[1] for x in lists])
    pq, pk = torch.cat([_perm(hq, Lq, 10 * i) for i in range(b)]), torch.cat([_perm(hk, Lk, 500 + 10 * i) for i in range(b)])
    call = lambda **kw: bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, want_lse=True, causal=causal, **kw)
    room = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device=DEV)
    full = bd.attn_workspace_size(Q, K, bd.params(block, causal=causal))
    least = 256
    if dtype == torch.bfloat16:
        with pytest.raises(bd.BasaError, match="too small: need") as e:
            call(ws=room(256))
        least = int(re.search(r"need (\d+) bytes", str(e.value)).group(1))
    two = least + 2 * b * hq * Lq * (4 * d + 8)
    assert least < two < full
    got = [call(ws=room(n)) for n in (full, two, least)]
    torch.cuda.synchronize()
    if dtype == torch.bfloat16:
        whole = call(attn_shape=3)
        assert torch.equal(got[2][0], whole[0]) and torch.equal(got[2][1], whole[1])
        assert not torch.equal(got[0][0], whole[0]) and not torch.equal(got[1][0], whole[0]) and not torch.equal(got[0][0], got[1][0])
    fn = o.sparse_attention_causal if causal else o.sparse_attention
    for i in range(b):
        for h in range(hq):
            args = (np64(Q[i, h]), np64(K[i, h // 2]), np64(V[i, h // 2]), pq[i, h].cpu().numpy(), pk[i, h // 2].cpu().numpy(),
                    [lists[i][3][0, h, j, :lists[i][2][0, h, j]] for j in range(n_q)], block)
            ref, ref_lse = fn(*args, return_lse=True)
            fin = np.isfinite(ref_lse)
            for out, lse in got:
                check_output(np64(out[i, h]), ref, dtype == torch.bfloat16, f"entry {i} head {h}")
                have = lse[i, h].cpu().numpy()
                assert np.array_equal(np.isfinite(have), fin)
                np.testing.assert_allclose(have[fin], ref_lse[fin], rtol=0, atol=2e-2 if dtype == torch.bfloat16 else 1e-4)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 64), (torch.float32, 128)])
@pytest.mark.parametrize("parts", [1, 2, 3, 4, 5, 8, 9, 17])
def test_adding_up_any_number_of_parts(parts, dtype, d):
    """Room for so many partial rows, lists long enough for all of them: the rows of the whole lists.  bf16: within the rounding of the
    outputs and of the probabilities, fp32: sixteen units of the last place of the values that a row averages."""
    h, Lq, Lk = 2, 70, 20000
    Q, K, V = _qkv(h, 1, Lq, Lk, d, dtype, seed=parts)
    n_k = -(-Lk // 64)
    cnt, cols, _, _ = _lists(h, -(-Lq // 64), n_k, 3, n_k)
    call = lambda n: bd.basa_sparse_attn(Q, K, V, cnt, cols, 64, want_lse=True, ws=torch.full((n,), 0xFF, dtype=torch.uint8, device=DEV))
    least = 256
    if dtype == torch.bfloat16:
        with pytest.raises(bd.BasaError, match="too small: need") as e:
            call(256)
        least = int(re.search(r"need (\d+) bytes", str(e.value)).group(1))
    (whole, lse), (out, lse_p) = call(least), call(least + parts * h * Lq * (4 * d + 8))
    bf = dtype == torch.bfloat16
    assert (out.float() - whole.float()).abs().max() <= (2.0 ** -7 * whole.float().abs().max() if bf else 2.0 ** -20 * V.abs().mean())
    torch.testing.assert_close(lse_p, lse, rtol=0, atol=4e-3 if bf else 1e-5)


@pytest.mark.parametrize("dtype,d,windows", [(torch.bfloat16, 128, (12416, 40960, 16384, 0)), (torch.float32, 64, (12416, 0))])
def test_norm_sort_of_many_words_with_runs_of_three_to_eighteen_tiles(dtype, d, windows):
    """Past 2^19 words: tiles of 4096, and the kernel that merges four of them in LDS (a ragged quad that is also the last
    pass, whole quads followed by ordinary passes, one run of 17.1 tiles), then segments that straddle tiles."""
    heads, L = 8, 70000 + 64
    g = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn((1, heads, L, d), generator=g, device=DEV).to(dtype)
    x[0, 0, 9000:9064] = x[0, 0, 100:164]                # exact ties across tiles
    x[0, 7, 4090:4100] = x[0, 7, 4080:4090]              # and around a tile edge
    assert heads * L > 1 << 19
    for kw in [dict(window=w) for w in windows] + [dict(segments=[0, 4095, 4097, 9000, 30001, 50000])]:
        perm = bd.basa_norm_sort(x, 128, **kw)
        torch.cuda.synchronize()
        for h in (0, 3, heads - 1):
            assert np.array_equal(perm[0, h].cpu().numpy(), o.norm_sort(np64(x[0, h]), **kw)), (kw, h)


@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,n_q,n_k", [(20, 500, 507), (20, 500, 513), (4, 130, 4000)])
def test_block_scores_on_both_sides_of_the_line_between_the_tile_sizes(hq, n_q, n_k, d, beta):
    """Ragged rows and columns: 1280 tiles of 64 x 64 (the small kernel's last), 1440, and 756 of few rows and many columns."""
    Q, K, _ = _qkv(hq, 2, 64 * n_q - 5, 64 * n_k - 9, d, torch.bfloat16, seed=n_k + d)
    sel = bd.basa_select(Q, K, 64, 0.5, beta, bd.SORT_NONE, want_scores=True)
    torch.cuda.synchronize()
    for h in (0, hq - 1):
        mq, vq = o.block_stats(np64(Q[0, h]), 64)
        mk, vk = o.block_stats(np64(K[0, h // (hq // 2)]), 64)
        ref = o.baseline_logits(mq, mk)
        if beta:
            ref = ref + beta * o.diag_compensation(mq, vq, mk, vk)
        np.testing.assert_allclose(sel.scores[0, h].cpu().numpy(), ref, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("block,Lq,Lk", [(128, 512, 2048), (128, 1100, 1920 + 70), (64, 600, 1000), (64, 512, 64), (128, 513, 129)])
@pytest.mark.parametrize("kind", ["disjoint", "one_has_all", "staggered", "single"])
def test_query_blocks_of_a_workgroup_at_different_tiles(kind, block, Lq, Lk):
    # 512-query workgroups, whose query blocks walk the tiles of the union at their own pace, against the 128-query ones,
    # which have no neighbours to wait for: every query takes the same tiles in the same order, so the bits agree
    Q, K, V = _qkv(2, 1, Lq, Lk, 128, torch.bfloat16, seed=Lq + Lk)
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    rows = {"disjoint": lambda g: [c for c in range(n_k) if c % 4 == g % 4] or [0],
            "one_has_all": lambda g: list(range(n_k)) if g % 4 == 2 else [n_k - 1 if g % 2 else 0],
            "staggered": lambda g: list(range(min(2 * (g % 4), n_k - 1), n_k)),
            "single": lambda g: [(5 * g) % n_k]}[kind]
    cnt_h = np.array([[[len(rows(g)) for g in range(n_q)]] * 2])
    cols_h = np.full((1, 2, n_q, n_k), -1)
    for g in range(n_q):
        cols_h[:, :, g, :len(rows(g))] = rows(g)
    t = lambda a: torch.from_numpy(a.astype(np.int32)).to(DEV)
    pq, pk = _perm(2, Lq, 3), _perm(1, Lk, 9)
    wide, lse_w = bd.basa_sparse_attn(Q, K, V, t(cnt_h), t(cols_h), block, pq, pk, want_lse=True, attn_shape=3)
    solo, lse_s = bd.basa_sparse_attn(Q, K, V, t(cnt_h), t(cols_h), block, pq, pk, want_lse=True)
    assert torch.equal(wide, solo) and torch.equal(lse_w, lse_s)
    ref = o.sparse_attention(np64(Q[0, 1]), np64(K[0, 0]), np64(V[0, 0]), pq[0, 1].cpu().numpy(), pk[0, 0].cpu().numpy(),
                             [rows(g) for g in range(n_q)], block)
    check_output(np64(wide[0, 1]), ref, True, kind)


def _three_part_call(Q, K, V, cnt, cols, block, pq, pk, **kw):
    """The call, and that it went to the kernel of three-part products (which alone lays out K and V for f32)."""
    bd.basa_profile_enable(True)
    try:
        out = bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, **kw)
        launches = bd.basa_profile_read()
    finally:
        bd.basa_profile_enable(False)
    assert any("gather" in n and c for n, (_, c) in launches.items()), launches
    return out


@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("Lq,Lk", [(4096, 4096), (4096 + 33, 2944 + 1), (3000, 4001), (8000, 97 * 32)])
def test_f32_attention_on_three_part_products(d, block, Lq, Lk):
    # Bound: the six part products leave 2^-25 of |q||k|, sums of up to Lk terms in fp32 (1e-5 with room), as for the
    # fp32 instruction; and no further from 64 bits than that kernel, whose result the small workspace gives, by half again.
    hq, hk = 8, 4
    Q, K, V = _qkv(hq, hk, Lq, Lk, d, torch.float32, seed=Lq + Lk + d)
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    cnt, cols, cnt_h, cols_h = _lists(hq, n_q, n_k, Lq + 3 * Lk, n_k)
    cnt[0, 5, 1] = 0                                      # a query block without a list: zero rows
    pq, pk = _perm(hq, Lq, 1), _perm(hk, Lk, 50)
    out, lse = _three_part_call(Q, K, V, cnt, cols, block, pq, pk, want_lse=True)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    plain = bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, ws=small)
    none = pq[0, 5, block:2 * block].long()
    assert not out[0, 5, none].any() and torch.all(lse[0, 5, none] == -float("inf"))
    for h in (0, 3):
        lists = [cols_h[0, h, g, :cnt_h[0, h, g]] for g in range(n_q)]
        ref, ref_lse = o.sparse_attention(np64(Q[0, h]), np64(K[0, h // 2]), np64(V[0, h // 2]), pq[0, h].cpu().numpy(),
                                          pk[0, h // 2].cpu().numpy(), lists, block, return_lse=True)
        check_output(np64(out[0, h]), ref, False, f"head {h}")
        err = lambda x: np.linalg.norm(np64(x[0, h]) - ref) / np.linalg.norm(ref)
        assert err(out) <= max(1.5 * err(plain), 3e-7)
        got, fin = lse[0, h].cpu().numpy(), np.isfinite(ref_lse)
        assert np.array_equal(np.isfinite(got), fin)
        np.testing.assert_allclose(got[fin], ref_lse[fin], rtol=0, atol=1e-5)


@pytest.mark.parametrize("where", ["k_minus", "k_plus", "v", "q_nan", "huge"])
@pytest.mark.parametrize("block", [64, 128])
def test_f32_three_part_products_leave_infinities_to_the_fp32_instruction(where, block):
    L, d, h = 4096, 128, 8
    Q, K, V = _qkv(h, h, L, L, d, torch.float32, seed=7)
    if where == "k_minus":                                # scores of -inf or NaN by the sign of one number of the query
        K[0, 1, 70, 5] = -float("inf")
    elif where == "k_plus":
        K[0, 1, 70] = float("inf")
    elif where == "v":
        V[0, 2, 4095, 3] = float("inf")
    elif where == "q_nan":
        Q[0, 3, 1000, 7] = float("nan")
    else:                                                 # rounds up past the largest bf16; finite in fp32
        V[0, 4, 17, 9] = 3.4e38
    out, lse = _three_part_call(Q, K, V, None, None, block, None, None, want_lse=True)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    ref, ref_lse = bd.basa_sparse_attn(Q, K, V, None, None, block, want_lse=True, ws=small)
    for a, b in ((out, ref), (lse, ref_lse)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
        fin = torch.isfinite(a) & torch.isfinite(b)
        assert torch.allclose(a[fin], b[fin], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("where", ["v", "v_subnormal", "v_large", "k", "q", "probabilities"])
@pytest.mark.parametrize("d,block", [(64, 64), (128, 128)])
def test_f32_three_part_products_keep_the_bits_of_small_numbers(where, d, block):
    # Parts of bf16 end at 2^-133: numbers whose 24 bits reach below that, as values, as keys or queries against large
    # partners, and as probabilities that alone make up a column of the result.  Bound: that of the products above, an error
    # of the fp32 instruction's by half again.
    L, h = 4096, 8
    Q, K, V = _qkv(h, h, L, L, d, torch.float32, seed=11)
    cols = slice(None)
    if where == "v":
        V *= 1e-36
    elif where == "v_subnormal":
        V *= 1e-20
        V *= 1e-19
    elif where == "v_large":
        V *= 1e30
    elif where == "k":
        Q, K = Q * 1e36, K * 1e-36
    elif where == "q":
        Q, K = Q * 1e-36, K * 1e36
    else:                                                 # key 0 takes all but 2^-124 of every row; key j alone fills column j
        Q *= 0.01
        Q[..., 0] = 32.0
        K[..., 0] = 0.0
        K[..., 0, :] = 0.0
        K[..., 0, 0] = 85.8 * d ** 0.5 / 32
        V.zero_()
        V[..., torch.arange(1, d), torch.arange(1, d)] = 1.0
        V[..., 0, 0] = 1.0
        cols = slice(1, None)
    out = _three_part_call(Q, K, V, None, None, block, None, None)
    plain = bd.basa_sparse_attn(Q, K, V, None, None, block, ws=torch.empty(256, dtype=torch.uint8, device=DEV))
    for i in (0, 5):
        q, k, v = (np64(x[0, i]) for x in (Q, K, V))
        s = q @ k.T / d ** 0.5
        w = np.exp(s - s.max(1, keepdims=True))
        ref = ((w / w.sum(1, keepdims=True)) @ v)[:, cols]
        err = lambda x: np.linalg.norm(np64(x[0, i])[:, cols] - ref) / np.linalg.norm(ref)
        assert err(out) <= max(1.5 * err(plain), 3e-7), (err(out), err(plain))


@pytest.mark.parametrize("dtype,d,block,hq,hk,lens,kw", [
    (torch.bfloat16, 128, 128, 4, 2, [1024, 1, 1025, 129, 64, 2050], {}),
    (torch.bfloat16, 64, 64, 4, 4, [63, 4096 + 1, 700, 65], dict(beta=0.0)),
    (torch.bfloat16, 128, 64, 2, 1, [8192 + 100, 300, 9000], dict(mass_target=0.6, min_keep=2)),     # two ranking passes
    (torch.bfloat16, 64, 128, 8, 2, [130 + 17 * i for i in range(15)], {}),                          # more than one launch holds
    (torch.bfloat16, 128, 128, 32, 32, [200, 9000, 500], {}),                                        # one that goes by itself
    (torch.bfloat16, 128, 128, 16, 16, [565, 7627, 1977, 3390, 4802, 6215], {}),                     # 512 queries to a workgroup
    (torch.bfloat16, 128, 64, 16, 4, [700, 7000, 4200, 6400, 5100, 300, 6900], {}),
    (torch.bfloat16, 64, 128, 32, 32, [3072, 2049, 4096, 3070], {}),                                 # words: one ranking pass
    (torch.bfloat16, 64, 128, 32, 32, [3072, 2049, 4096, 3073], {}),                                 # ... a cut merge, one part and two
    (torch.bfloat16, 64, 128, 32, 32, [4096, 3073, 2048, 1025, 4096, 3072, 4000, 3500], {}),         # ... of a large call
    (torch.bfloat16, 128, 64, 2, 2, [400, 300], dict(causal=True)),                                  # all by themselves
    (torch.bfloat16, 128, 64, 2, 2, [400, 300], dict(sort=bd.SORT_K)),
    (torch.float32, 64, 64, 2, 2, [400, 0, 300], {})])
def test_packed_batch_against_one_call_per_sequence(dtype, d, block, hq, hk, lens, kw):
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(lens) + d)
    T = sum(lens) + 3                                     # tokens behind the last sequence stay out of it
    q, k, v = (torch.randn((T, h, d), generator=g, device=DEV).to(dtype) for h in (hq, hk, hk))
    cu = np.cumsum([0] + lens).tolist()
    out = bd.ba_att_varlen(q, k, v, cu, block, 0.5, **kw)
    assert torch.equal(bd.ba_att_varlen(q, k, v, cu, block, 0.5, **kw)[:cu[-1]], out[:cu[-1]])
    view = lambda x, a, b: x[a:b].permute(1, 0, 2).unsqueeze(0)
    for a, b in zip(cu[:-1], cu[1:]):
        if a == b:
            continue
        want, _ = bd.ba_att(view(q, a, b), view(k, a, b), view(v, a, b), block, 0.5, **kw)
        got = view(out, a, b)
        if dtype == torch.float32:
            assert torch.equal(got, want)
        else:                                             # (lists split or not, shapes of workgroup: bf16 rounding of out)
            err = (got.float() - want.float()).norm() / want.float().norm()
            assert err < 4e-3 and (got.float() - want.float()).abs().max() < 2e-2, (a, b, err)


@pytest.mark.parametrize("heads,L,window,segments", [(64, 8193, 0, None), (33, 16384 + 1, 0, None), (20, 32768 + 5000, 0, None),
                                                     (400, 1500, 0, None), (40, 40000, 17408, None), (16, 50000, 0, [0, 3, 20000]),
                                                     (41, 51150, 0, None), (130, 4097, 0, None), (132, 5000, 0, None), (300, 2049, 0, None),
                                                     (131, 4096, 0, None), (18, 40000, 5120, None), (64, 9000, 8192, None),
                                                     (70, 9000, 2048, None), (128, 4096, 0, None), (101, 4001, 0, None)])
def test_sort_of_middling_calls_from_tiles_of_1024(heads, L, window, segments):
    Q, _, _ = _qkv(heads, 1, L, 64, 64, torch.bfloat16, seed=L)
    Q[0, 1] = Q[0, 1, :1]
    Q[0, 2, ::3] = Q[0, 2, :1]
    perm, keys = bd.basa_norm_sort(Q, 64, window=window, segments=segments, return_keys=True)
    bounds = segments + [L] if segments else list(range(0, L, window or L)) + [L]
    for a, b in zip(bounds[:-1], bounds[1:]):
        assert torch.equal(perm[0, :, a:b].long(), torch.sort(keys[0, :, a:b], dim=-1, stable=True).indices + a)


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 64), (torch.bfloat16, 128)])
@pytest.mark.parametrize("L,window", [(1025, 0), (1536, 0), (2047, 0), (2049, 0), (3584 + 1, 0), (4096, 0), (4097, 0), (5000, 1152),
                                      (5000, 4096), (3000, 512)])
def test_sort_tiles_of_512_tokens(dtype, d, L, window):
    Q, _, _ = _qkv(3, 1, L, 64, d, dtype, seed=L + d)
    Q[0, 1] = Q[0, 1, :1]                                 # all keys alike: index order
    Q[0, 2, ::7] = Q[0, 2, :1]
    perm, keys = bd.basa_norm_sort(Q, 64, window=window, return_keys=True)
    for a in range(0, L, window or L):
        b = min(a + (window or L), L)
        want = torch.sort(keys[0, :, a:b], dim=-1, stable=True).indices + a
        assert torch.equal(perm[0, :, a:b].long(), want)


def _tiles_laid_out(call):
    """What the call returns, and whether tiles of K and V were laid out for it."""
    bd.basa_profile_enable(True)
    try:
        out = call()
        torch.cuda.synchronize()
        return out, bd.basa_profile_read().get("gather_kernels", (0.0, 0))[1] > 0
    finally:
        bd.basa_profile_enable(False)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("Lq,Lk", [(3, 64), (100, 65), (1, 127), (257, 600), (64, 2049), (300, 6017), (40, 20000)])
@pytest.mark.parametrize("form", ["plain", "token-major", "no order", "broken order", "infinite last key"])
def test_attention_on_rows_of_k_and_v(d, block, Lq, Lk, form):
    """The 128-query shape without tiles, which calls of few queries take, against the 512-query one, which always lays them out:
    whole lists give the same bits, split ones (more than 32 tiles) the same within the rounding of bf16 outputs."""
    Q, K, V = _qkv(4, 2, Lq, Lk, d, torch.bfloat16, seed=Lk + d)
    if form == "token-major":
        K, V = (torch.cat([x.permute(0, 2, 1, 3), x.permute(0, 2, 1, 3)], 2).contiguous()[:, :, 1:3].permute(0, 2, 1, 3) for x in (K, V))
    n_q, n_k = -(-Lq // block), -(-Lk // block)
    cnt, cols, _, _ = _lists(4, n_q, n_k, Lk, n_k)
    pq, pk = _perm(4, Lq, 1), _perm(2, Lk, 50)
    if form == "no order":
        pq, pk = None, None
    elif form == "broken order":
        pk[0, 0, ::7] = Lk + 3
        pk[0, 1, 5::11] = -1
    elif form == "infinite last key":
        V[0, 0, int(pk[0, 0, Lk - 1])] = float("inf")
    (rows, lse), laid_out = _tiles_laid_out(lambda: bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, want_lse=True))
    assert not laid_out
    (tiles, lse_t), laid_out = _tiles_laid_out(lambda: bd.basa_sparse_attn(Q, K, V, cnt, cols, block, pq, pk, want_lse=True, attn_shape=3))
    assert laid_out
    if n_k * (block // 64) <= 32:
        assert torch.equal(rows.view(torch.int16), tiles.view(torch.int16)) and torch.equal(lse, lse_t)
        return
    fin = torch.isfinite(tiles.float())
    assert torch.equal(fin, torch.isfinite(rows.float()))
    diff = (rows.float() - tiles.float())[fin].abs()
    assert diff.max() <= 2.0 ** -7 * tiles.float()[fin].abs().max()      # a last place of the largest, rounded twice
    torch.testing.assert_close(lse, lse_t, rtol=0, atol=4e-3)             # (sums of probabilities rounded to 8 bits)


@pytest.mark.parametrize("stride,Lk,laid_out", [(2 ** 23 - 8, 256, False), (2 ** 23, 70, True), (2 ** 15, 2 ** 16, True), (2 ** 15 - 8, 2 ** 16, False)])
def test_rows_of_k_and_v_at_the_limits_of_their_offsets(stride, Lk, laid_out):
    """Tokens so far apart that the last one's offset takes all 32 bits, or more, where the call has to go by tiles."""
    far = torch.empty(stride * Lk, dtype=torch.bfloat16, device=DEV)
    Q, K0, V0 = _qkv(2, 2, 50, Lk, 64, torch.bfloat16, seed=Lk)
    K, V = (far.as_strided((1, 2, Lk, 64), (0, 64, stride, 1), 128 * i) for i in range(2))
    K.copy_(K0)
    V.copy_(V0)
    n_k = -(-Lk // 64)
    cnt, cols, _, _ = _lists(2, 1, n_k, Lk, n_k)
    pk = _perm(2, Lk, 9)
    call = lambda k, v: bd.basa_sparse_attn(Q, k, v, cnt, cols, 64, None, pk)
    want, near = _tiles_laid_out(lambda: call(K0, V0))
    got, apart = _tiles_laid_out(lambda: call(K, V))
    assert not near and apart == laid_out and torch.isfinite(want.float()).all()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 64), (torch.bfloat16, 128)])
@pytest.mark.parametrize("heads,L", [(128, 900), (129, 900), (16, 8000), (32, 4096), (33, 4096), (64, 2047), (65, 2047), (1, 1), (3, 5000)])
def test_sort_on_both_sides_of_eight_waves_to_a_tile(dtype, d, heads, L):
    x, _, _ = _qkv(heads, 1, L, 64, d, dtype, seed=L + d)
    x[0, heads // 2] = x[0, heads // 2, :1]
    perm, keys = bd.basa_norm_sort(x, 64, return_keys=True)
    assert torch.equal(perm[0].long(), torch.sort(keys[0], dim=-1, stable=True).indices)


# (from (64, 32768) on parts of 48 samples, before them of 32)
@pytest.mark.parametrize("heads,L", [(64, 8193), (16, 32768), (30, 32769), (41, 32767), (132, 5000), (6, 70000), (12, 33000), (64, 32768),
                                     (50, 35456), (80, 22500)])
@pytest.mark.parametrize("kind", ["spread", "few values", "ascending", "descending", "far outliers", "runs alike", "smallest last"])
def test_merge_cut_by_samples(heads, L, kind):
    """Parts whose bounds fall on few distinct keys, on runs that do not overlap at all, and far apart; the largest parts (runs that hold
    the same 1024 keys: 4206 words of 22500, in more slots than there are threads); a short last run below all others."""
    x, _, _ = _qkv(heads, 1, L, 64, 64, torch.float32 if kind == "runs alike" else torch.bfloat16, seed=L)
    ramp = torch.linspace(0.01, 3.0, L, device=DEV)[None, None, :, None]
    if kind == "few values":
        x = x[:, :, :1].expand(-1, -1, L, -1).contiguous()
        x[:, :, ::3] *= 2
        x[:, :, L // 2:L // 2 + 3000] = 0
    elif kind in ("ascending", "descending"):
        x = ((ramp if kind == "ascending" else ramp.flip(2)) * torch.ones_like(x)).to(x.dtype)
    elif kind == "runs alike":
        x = (1.0 + torch.arange(L, device=DEV) % 1024)[None, None, :, None] * torch.ones_like(x)
    elif kind == "smallest last":
        x[:, :, L // 1024 * 1024:] = 0
    elif kind == "far outliers":
        x[:, :, ::50] *= 1000
        x[:, :, 5::1000] = float("inf")
    perm, keys = bd.basa_norm_sort(x, 64, return_keys=True)
    assert torch.equal(perm[0].long(), torch.sort(keys[0], dim=-1, stable=True).indices)


def test_packed_batch_repeats_what_left_the_safe_range():
    # 512 queries to a workgroup, scores near +-600 in one sequence: its workgroups go to the pass with running maxima
    lens, h, d = [565, 7627, 1977, 3390, 4802, 6215], 16, 128
    cu = np.cumsum([0] + lens).tolist()
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    q, k, v = (torch.randn((cu[-1], h, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3))
    q[cu[3]:cu[4]] *= 50
    out = bd.ba_att_varlen(q, k, v, cu, 128, 0.5)
    assert torch.isfinite(out.float()).all()
    view = lambda x, a, b: x[a:b].permute(1, 0, 2).unsqueeze(0)
    for a, b in zip(cu[:-1], cu[1:]):
        want, _ = bd.ba_att(view(q, a, b), view(k, a, b), view(v, a, b), 128, 0.5)
        assert (view(out, a, b).float() - want.float()).norm() < 4e-3 * want.float().norm()


@pytest.mark.parametrize("hq,hk,Lq,Lk,d,sort,streams", [
    (16, 16, 25000, 28000, 128, bd.SORT_QK, True),        # 102 and 115 MB, sorted one after the other
    (16, 16, 15000, 20000, 128, bd.SORT_QK, False),       # 61 and 82 MB, likewise
    (16, 4, 30000, 30000, 128, bd.SORT_Q, False), (16, 4, 40000, 40000, 128, bd.SORT_K, True),
    (64, 64, 4096, 4096, 128, bd.SORT_QK, False), (75, 75, 4096, 4096, 128, bd.SORT_QK, False)])
def test_both_passes_over_the_rows_load_them_the_same_way(hq, hk, Lq, Lk, d, sort, streams):
    # one answer for a call: what the key pass leaves in the caches is there for the pooling pass, or neither pass goes by it
    from torch.profiler import ProfilerActivity, profile
    Q, K, _ = _qkv(hq, hk, Lq, Lk, d, torch.bfloat16)
    bd.basa_select(Q, K, 128, 0.5, sort=sort)
    torch.cuda.synchronize()
    names = []
    try:
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            bd.basa_select(Q, K, 128, 0.5, sort=sort)
            torch.cuda.synchronize()
        names = [e.name for e in prof.events()]
    except RuntimeError as e:                             # (of the profiler: the calls above and below run without it)
        pytest.skip(f"no profiler here: {e}")
    passes = [m.group(2) == "true" for n in names for m in [re.search(r"(norm_tile_sort|block_stats)_kernel<[^>]*, (true|false)>", n)] if m]
    if not passes:
        pytest.skip("the profiler reports no kernels here")
    assert len(passes) >= 2 and all(p == streams for p in passes), [n[:120] for n in names]


@pytest.mark.parametrize("kw", [{}, dict(causal=True), dict(mass_target=0.6, min_keep=2), dict(beta=0.0)])
@pytest.mark.parametrize("hq,hk,n_q,n_k,d", [(2, 1, 1, 1, 64), (3, 1, 9, 33, 64), (8, 2, 33, 64, 128), (2, 2, 40, 65, 128),
                                             (2, 1, 7, 128, 64), (32, 8, 65, 65, 64), (32, 32, 128, 127, 128), (33, 11, 128, 40, 64)])
def test_map_and_selection_in_one_launch_against_two(hq, hk, n_q, n_k, d, kw):
    """Strips of 8 and 16 rows and calls on both sides of their line: the lists, bitmaps and masses of the two launches."""
    Q, K, _ = _qkv(hq, hk, 64 * n_q - 5, 64 * n_k - 9, d, torch.bfloat16, seed=n_q + n_k)
    one, two = (bd.basa_select(Q, K, 64, 0.6, select_path=path, **kw) for path in (0, 1))
    torch.cuda.synchronize()
    for name in ("row_count", "mask_bits", "row_mass"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    listed = torch.arange(two.row_cols.shape[-1], device=DEV) < two.row_count[..., None]
    assert torch.equal(torch.where(listed, one.row_cols, -1), torch.where(listed, two.row_cols, -1))
