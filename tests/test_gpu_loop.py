"""ppv_decode_loop against ppv_decode_step, bit for bit, where its launch shape changes: tiles per row around the number of
wavefronts, batches around 256, 512 and 1,024 rows, rows whose first tokens are filtered or far below the rest."""
import numpy as np
import pytest
import torch

from paper_2504_09135_amd import binding as ppv

from gpu_helpers import DEV, tuning

pytestmark = pytest.mark.gpu


def make_index(V, L, rng):
    """Members that share little: below the first levels every prefix has one child."""
    n = 3_000
    S = rng.integers(0, V, (n, L)).astype(np.int32)
    S[:, 0] %= 7
    lens = rng.integers(1, L + 1, n)
    return ppv.ppv_build_index(np.concatenate([S[i, : lens[i]] for i in range(n)]), np.cumsum([0, *lens]).astype(np.int64), V)


def check(V, B, dtype, L, waves=0):
    rng = np.random.default_rng(V * 31 + B)
    index = make_index(V, L, rng)
    g = torch.Generator(device=DEV).manual_seed(V + B)
    padded = -(-V // 8) * 8
    lg = torch.empty((L, B, padded), dtype=dtype, device=DEV)
    for s in range(L):
        lg[s] = torch.randn((B, padded), generator=g, device=DEV).mul_(2)
    tile = 1024 if dtype == torch.float32 else 2048
    first = torch.arange(padded, device=DEV) % tile < 32
    lg[:, 1::5, first] = -torch.inf            # filtered where a tile's reference is looked for
    lg[:, 2::5, first] = -1e9
    lg[:, 3::5, first] -= 200                  # the rest far above it
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
    assert (results[0][1] > 0).any()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [200, 257, 513, 1_025])
@pytest.mark.parametrize("tiles", [1, 2, 3, 5, 7, 15, 16, 18, 19])
def test_loop_gives_the_bits_of_its_steps(tiles, B, dtype):
    tile = 1024 if dtype == torch.float32 else 2048
    check(tiles * tile - 5, B, dtype, 5)


@pytest.mark.parametrize("tiles, B", [(48, 40), (48, 320), (48, 321), (48, 520), (95, 257), (95, 321), (97, 520)])
def test_long_rows(tiles, B):
    check(tiles * 1024 + 1, B, torch.float32, 4)


@pytest.mark.parametrize("waves", [1, 2, 8])
def test_more_tiles_to_a_wavefront_than_lanes(waves):
    check(130 * 1024 + 3, 3, torch.float32, 4, waves)
