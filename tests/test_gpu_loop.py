"""ppv_decode_loop against ppv_decode_step, bit for bit, where its launch shape changes: tiles per row around the number of
wavefronts, batches around 256, 512 and 1,024 rows, rows whose first tokens are filtered or far below the rest.  The rows go
through an image or a short list, long lists and chains of prefixes with one child each (counted, not assumed)."""
import numpy as np
import pytest
import torch

from paper_2504_09135_amd import binding as ppv

from gpu_helpers import DEV, tuning

pytestmark = pytest.mark.gpu


def make_set(V, L, rng, many_firsts):
    """Members of 3 .. L tokens.  many_firsts: the root has an image, and nearly every prefix below it one child (V large); else
    seven first tokens with some 400 continuations each, and chains below these."""
    n = 3_000
    S = rng.integers(0, V, (n, L)).astype(np.int32)
    if not many_firsts:
        S[:, 0] = S[:7, 0][S[:, 0] % 7]
    return S, rng.integers(3, L + 1, n)


def steps_in_chains(S, lens, P, taken):
    """Per row, the longest run of steps taken from prefixes with exactly one child."""
    children = {}
    for row, k in zip(S.tolist(), lens):
        for t in range(k):
            children.setdefault(tuple(row[:t]), set()).add(row[t])
    best = np.zeros(len(P), int)
    for b, row in enumerate(P.tolist()):
        run = 0
        for t in range(taken[b]):
            run = run + 1 if len(children[tuple(row[:t])]) == 1 else 0
            best[b] = max(best[b], run)
    return best


def check(V, B, dtype, L, waves=0, chains=True):
    rng = np.random.default_rng(V * 31 + B)
    S, n_tok = make_set(V, L, rng, many_firsts=B % 2 == 0)
    index = ppv.ppv_build_index(np.concatenate([row[:k] for row, k in zip(S, n_tok)]), np.cumsum([0, *n_tok]).astype(np.int64), V)
    g = torch.Generator(device=DEV).manual_seed(V + B)
    padded = -(-V // 8) * 8
    lg = torch.empty((L, B, padded), dtype=dtype, device=DEV)
    for s in range(L):
        lg[s] = torch.randn((B, padded), generator=g, device=DEV).mul_(2)
    tile = 1024 if dtype == torch.float32 else 2048
    first = torch.arange(padded, device=DEV) % tile < 32
    lg[1:, 1::5, first] = -torch.inf           # from the second step on, filtered where a tile's reference is looked for
    lg[1:, 2::5, first] = -1e9
    lg[1:, 3::5, first] -= 200                 # the rest far above it
    lg = lg[..., :V]
    un = torch.rand((L, B), generator=g, device=DEV)
    results = []
    for one_launch in (False, True):
        P = torch.full((B, L), 7, dtype=torch.int32, device=DEV)
        lens, act = torch.zeros(B, dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.uint8, device=DEV)
        state = torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
        lx = torch.zeros(B, device=DEV)
        ids = torch.full((L, B), -7, dtype=torch.int32, device=DEV)
        lz = torch.full((L, B), 7.0, device=DEV)
        ppv.ppv_decode_begin_empty(index, lens, state, act, lx)
        if one_launch:
            with tuning(ppv.PPV_TUNE_WAVES_PER_ROW, waves):
                ppv.ppv_decode_loop(index, P, lens, act, lg, un, ids, lz, lx, state=state)
        else:
            for s in range(L):
                ppv.ppv_decode_step(index, P, lens, act, lg[s], un[s], ids[s], lz[s], lx, state=state)
        torch.cuda.synchronize()
        results.append([x.cpu().numpy() for x in (P, lens, act, lx, ids, lz)])
    for a, b in zip(*results):
        assert np.array_equal(a, b, equal_nan=True)
    P, taken = results[0][:2]
    for kind in range(min(5, B)):              # the rows of each kind have gone below their first tokens
        assert (taken[kind::5] >= 3).mean() > 0.7, (kind, taken[kind::5])
    if chains:
        runs = steps_in_chains(S, n_tok, P, taken)
        assert (runs >= 2).mean() > 0.5, runs


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [200, 256, 257, 512, 513, 1_024, 1_025])
@pytest.mark.parametrize("tiles", [1, 2, 3, 5, 7, 15, 16, 18, 19])
def test_loop_gives_the_bits_of_its_steps(tiles, B, dtype):
    tile = 1024 if dtype == torch.float32 else 2048
    check(tiles * tile - 5, B, dtype, 7)


@pytest.mark.parametrize("tiles, B", [(47, 257), (47, 520), (48, 40), (48, 257), (48, 320), (48, 321), (48, 520), (48, 1_024), (49, 513),
                                      (95, 257), (95, 321), (95, 600), (96, 321), (96, 600), (97, 520)])
def test_long_rows(tiles, B):
    check(tiles * 1024 - 3, B, torch.float32, 6)


@pytest.mark.parametrize("waves", [1, 2, 8])
def test_more_tiles_to_a_wavefront_than_lanes(waves):
    check(130 * 1024 + 3, 3, torch.float32, 6, waves, chains=False)


@pytest.mark.parametrize("B", [1_025, 1_026])
def test_more_tiles_to_a_wavefront_than_lanes_in_large_batches(B):
    """(Batches above 1,024 rows run with two wavefronts a row: 65 tiles each.)"""
    check(129 * 1024 + 3, B, torch.float32, 4, chains=False)
