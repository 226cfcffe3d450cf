"""The walk of a prefix that only one member has, where it is answered from that member's tokens alone: members around a
wavefront's length, nested ones, prefixes that end with, before, behind or beside a member, vocabularies with no lists
at all.  Mask, rank range and membership against the oracle; the other callers of the walk against the mask."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_09135_amd import binding as ppv
from paper_2504_09135_amd import workloads as W

from gpu_helpers import DEV, assert_query_parity, to_dev, unpack_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [2, 31, 40, 1_000, 3_000])   # one-bit rows, no lists (V / 32 = 0), one word per lane, whole rows
@pytest.mark.parametrize("L", [1, 2, 62, 63, 64, 65, 66, 130])
def test_prefixes_of_one_member(L, V, dtype):
    rng = np.random.default_rng(L * 10_000 + V)
    n = 40
    rows = rng.integers(0, V, (n, L)).astype(np.int32)
    lens = np.where(np.arange(n) % 3 == 0, rng.integers(1, L + 1, n), L)
    rows[1::4] = rows[0::4][: len(rows[1::4])]           # some begin like another, and leave it (or end in it) somewhere
    for i in range(1, n, 4):
        rows[i, int(rng.integers(0, L))] = int(rng.integers(0, V))
    S = [rows[i, : lens[i]] for i in range(n)]
    offsets = np.cumsum([0] + [len(s) for s in S]).astype(np.int64)
    tokens = np.concatenate(S).astype(np.int32)
    stride = L + 2
    P, T = [], []
    for i in range(0, n, 3):
        for t in {0, 1, L // 2, lens[i] - 2, lens[i] - 1, lens[i], lens[i] + 1} | {62, 63, 64, 65}:
            if not 0 <= t <= stride:
                continue
            p = np.full(stride, W.PAD_TOKEN, np.int32)
            p[: lens[i]] = S[i]
            p[lens[i]:t] = rng.integers(0, V, max(0, t - lens[i]))
            for change in (None, t - 1, t // 2):
                q = p.copy()
                if change is not None and change >= 0:
                    q[change] = (q[change] + rng.integers(0, 3) - 1) % V
                P.append(np.where(np.arange(stride) < t, q, W.PAD_TOKEN))
                T.append(t)
    P, T = np.array(P, np.int32), np.array(T, np.int32)
    B = len(T)
    trie = oracle.Trie(tokens, offsets, V)
    index = ppv.ppv_build_index(tokens, offsets, V)
    assert_query_parity(index, trie, P, T)

    dP, dT = to_dev(P), to_dev(T)
    stride_l = -(-V // 8) * 8
    logits = torch.from_numpy(rng.standard_normal((B, stride_l)).astype(np.float32)).to(DEV).to(dtype)[:, :V]
    u = torch.from_numpy(rng.random(B, dtype=np.float32)).to(DEV)
    mask = torch.empty((B, index.n_words), dtype=torch.int32, device=DEV)
    ppv.ppv_next_token_mask(index, dP, dT, mask)
    ids = torch.empty((4, B), dtype=torch.int32, device=DEV)
    mass = torch.empty((4, B), dtype=torch.float32, device=DEV)
    ppv.constrained_sample(logits, mask, u, ids[0], mass[0])
    ppv.ppv_sample_next(index, dP, dT, logits, u, ids[1], mass[1])
    assert torch.equal(ids[1], ids[0]) and torch.allclose(mass[1], mass[0], rtol=1e-5, atol=1e-5)
    state = torch.empty((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
    begun = torch.empty(B, dtype=torch.uint8, device=DEV)
    ppv.ppv_decode_begin(index, dP, dT, state, begun)
    went = (begun != 0) & (dT < stride)
    after = []
    for k, st in ((2, None), (3, state)):   # one step without a cursor and one with
        rows_k, lens_k, active = dP.clone(), dT.clone(), begun.clone()
        ppv.ppv_decode_step(index, rows_k, lens_k, active, logits, u, ids[k], mass[k], None, st)
        after.append((rows_k, lens_k, active))
        assert torch.equal(ids[k][went], ids[0][went])
        assert torch.allclose(mass[k][went], mass[0][went], rtol=1e-5, atol=1e-5)
    for a, b in zip(*after):
        assert torch.equal(a, b)
    M = min(V, 20)
    got = torch.empty_like(mask)
    ppv.ppv_topm_mask(index, dP, dT, logits, M, got)
    ref = oracle.SortedArray(tokens, offsets, V).topm(P, T, logits.float().cpu().numpy(), M)
    assert np.array_equal(unpack_mask(got.cpu().numpy().view(np.uint32), V), ref.mask)
    index.free()
