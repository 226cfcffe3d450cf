"""constrained_sample at the edges of its tiles: rows that end inside, at and behind a tile and a 16-byte group, one to five
tiles per wavefront, and tiles whose cheap reference (the largest of the first 16 bytes) is no use: nothing but -inf
there, tokens far above it, tokens far below it.  Sums and samples against double precision."""
import numpy as np
import pytest
import torch

from paper_2504_09135_amd import binding as ppv
from paper_2504_09135_amd import workloads as W

from gpu_helpers import CDF_BAND, DEV, LOGZ_TOL, to_dev, tuning

pytestmark = pytest.mark.gpu


def rows_for(V, tile, rng):
    """One row per kind of reference."""
    base = rng.normal(0, 2, size=(8, V)).astype(np.float32)
    base[1, ::tile] = -np.inf                                   # the very first token of each tile
    for at in range(0, V, tile):
        base[2, at:at + 8] = -np.inf                            # all of the first group
        base[3, at:at + 8] = -1e9                               # ... masked the other way
        base[4, at:at + 8] -= 100.0                             # the rest 100 above it: beyond the sums' range
        base[5, at:at + 8] += 60.0                              # the rest far below it
        base[6, at + (tile - 1) % min(tile, V - at)] = 90.0     # one token far above, at the tile's end
    base[7, :V - 1] = -np.inf                                   # tiles of nothing, and a single token at the row's end
    return base


@pytest.mark.parametrize("waves", [1, 2, 4, 16])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("over", [-9, -8, -1, 0, 1, 7, 8, 9])
@pytest.mark.parametrize("tiles", [1, 2, 5])
def test_row_ends_and_references(tiles, over, dtype, waves):
    tile = 1024 if dtype == "f32" else 2048
    V = tiles * tile + over
    rng = np.random.default_rng(V + waves)
    lg = rows_for(V, tile, rng)
    B = lg.shape[0]
    bits = W.f32_to_bf16_bits(lg)
    x = (W.bf16_bits_to_f32(bits) if dtype == "bf16" else lg).astype(np.float64)
    per = 8 if dtype == "bf16" else 4
    Vp = -(-V // per) * per
    buf = np.full((B, Vp), np.inf, np.float32)                  # behind the row's end: never looked at
    buf[:, :V] = lg
    if dtype == "bf16":
        raw = np.full((B, Vp), 0x7F80, np.uint16)
        raw[:, :V] = bits
        ld = to_dev(raw.view(np.int16)).view(torch.bfloat16)[:, :V]
    else:
        ld = to_dev(buf)[:, :V]
    for n_valid in (5, V // 2):                                 # a list, an image
        mask = np.zeros((B, V), np.uint8)
        for b in range(B):
            mask[b, rng.choice(V, n_valid, replace=False)] = 1
            mask[b, V - 1] = 1
        words = np.packbits(np.pad(mask, ((0, 0), (0, (-V) % 32))), axis=1, bitorder="little").view(np.int32)
        un = rng.random(B, dtype=np.float32)
        ids = torch.full((B,), -9, dtype=torch.int32, device=DEV)
        lzv = torch.zeros(B, device=DEV)
        lza = torch.zeros(B, device=DEV)
        with tuning(ppv.PPV_TUNE_WAVES_PER_ROW, waves):
            ppv.constrained_sample(ld, to_dev(words), to_dev(un), ids, lzv, lza)
        torch.cuda.synchronize()
        ids, lzv, lza = ids.cpu().numpy(), lzv.cpu().numpy(), lza.cpu().numpy()
        for b in range(B):
            top = x[b].max()
            za = np.exp(x[b] - top).sum()
            valid = np.flatnonzero(mask[b])
            vtop = x[b, valid].max()
            w = np.exp(x[b, valid] - vtop)
            cdf = np.cumsum(w) / w.sum()
            all_ref, val_ref = top + np.log(za), vtop + np.log(w.sum()) - top - np.log(za)
            tol = LOGZ_TOL["f32"]                               # (the reference has the rounded logits)
            assert abs(lza[b] - all_ref) <= tol * max(1.0, abs(all_ref)), (b, n_valid, lza[b], all_ref)
            assert abs(lzv[b] - val_ref) <= tol * max(1.0, abs(val_ref)), (b, n_valid, lzv[b], val_ref)
            at = int(np.searchsorted(cdf, un[b], side="right"))
            near = [i for i in (at - 1, at, at + 1) if 0 <= i < len(valid)]
            assert ids[b] in valid[near] and (ids[b] == valid[min(at, len(valid) - 1)] or
                                              np.abs(cdf - un[b]).min() < CDF_BAND), (b, n_valid, ids[b], valid[near])


@pytest.mark.parametrize("dtype,V", [("f32", 2_500), ("bf16", 9_000), ("bf16", 130_000)])
def test_one_token_far_above_the_rest_is_summed_exactly(dtype, V):
    """A token 40 T or more above every other: its tile has to be summed relative to it, which makes that sum 1 up to
    2e3 * exp(-40), 1 in fp32.  logZ_all is then that logit, and logZ_valid of a list without it the difference from the
    listed ones' log-sum: half an ulp each of two numbers below 128 (4e-6 each) and 1e-7 for a sum of five."""
    rng = np.random.default_rng(V)
    peaks = np.repeat([50.0, 55.0, 60.0, 65.0, 72.0], 16).astype(np.float32)   # (noise: below 9, as drawn)
    B = len(peaks)
    lg = rng.normal(0, 2, size=(B, V)).astype(np.float32).clip(-9, 9)
    at = rng.integers(0, V, B)
    lg[np.arange(B), at] = peaks
    bits = W.f32_to_bf16_bits(lg)
    x = (W.bf16_bits_to_f32(bits) if dtype == "bf16" else lg).astype(np.float64)
    mask = np.zeros((B, V), np.uint8)
    for b in range(B):
        mask[b, rng.choice(V, 5, replace=False)] = 1
        mask[b, at[b]] = 0
    words = np.packbits(np.pad(mask, ((0, 0), (0, (-V) % 32))), axis=1, bitorder="little").view(np.int32)
    row = -(-V // 8) * 8
    buf = np.zeros((B, row), np.float32)
    buf[:, :V] = lg
    ld = to_dev(W.f32_to_bf16_bits(buf).view(np.int16)).view(torch.bfloat16)[:, :V] if dtype == "bf16" else to_dev(buf)[:, :V]
    ids = torch.zeros(B, dtype=torch.int32, device=DEV)
    lzv, lza = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
    ppv.constrained_sample(ld, to_dev(words), to_dev(np.full(B, 0.5, np.float32)), ids, lzv, lza)
    assert np.array_equal(lza.cpu().numpy(), peaks)
    for b in range(B):
        w = x[b, mask[b] != 0]
        want = np.log(np.exp(w - w.max()).sum()) + w.max() - peaks[b]
        assert abs(float(lzv[b]) - want) <= 8.2e-6, (b, float(lzv[b]), want)


def filtered_rows(V, keep, rng, fill):
    """(rows, V) logits of which `keep` tokens per row are left, the others -inf or what stands for it."""
    lg = rng.normal(0, 2, size=(6, V)).astype(np.float32)
    for b in range(6):
        out = np.ones(V, bool)
        out[rng.choice(V, min(keep, V), replace=False)] = False
        lg[b, out] = fill
    lg[1, :min(V, 2_100)] = fill                                           # nothing left in the first tile
    lg[2] = fill                                                           # nothing left at all, or every token alike
    return lg


@pytest.mark.parametrize("fill,T", [(-np.inf, 1.0), (-np.inf, 0.3), (-1e9, 1.0), (-1e4, 1.0), (-1e4, 0.3)])
@pytest.mark.parametrize("dtype,V", [("f32", 1_023), ("f32", 9_004), ("bf16", 2_049), ("bf16", 32_000), ("bf16", 131_000)])
def test_filtered_rows(dtype, V, fill, T):
    """Rows of which a filter has left a few tokens (top-k, top-p), with a list of valid tokens: the reference is then the
    tile's exact maximum, also where it is all there is, and the tokens filtered out weigh exp(-3e3) or less, that is
    nothing.  Sums of at most 50 terms of 2^-24 relative error each, and logs of numbers below 64: 1e-5."""
    rng = np.random.default_rng(V)
    lg = filtered_rows(V, 50, rng, fill)
    B = len(lg)
    bits = W.f32_to_bf16_bits(lg)
    x = (W.bf16_bits_to_f32(bits) if dtype == "bf16" else lg).astype(np.float64) / T
    mask = np.zeros((B, V), np.uint8)
    for b in range(B):
        mask[b, rng.choice(V, 30, replace=False)] = 1
        left = np.flatnonzero(lg[b] > fill)
        mask[b, left[:3]] = 1
    words = np.packbits(np.pad(mask, ((0, 0), (0, (-V) % 32))), axis=1, bitorder="little").view(np.int32)
    row = -(-V // 8) * 8
    buf = np.zeros((B, row), np.float32)
    buf[:, :V] = lg
    ld = to_dev(W.f32_to_bf16_bits(buf).view(np.int16)).view(torch.bfloat16)[:, :V] if dtype == "bf16" else to_dev(buf)[:, :V]
    ids = torch.zeros(B, dtype=torch.int32, device=DEV)
    lzv, lza = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
    un = rng.random(B, dtype=np.float32)
    ppv.constrained_sample(ld, to_dev(words), to_dev(un), ids, lzv, lza, temperature=T)
    ids, lzv, lza = ids.cpu().numpy(), lzv.cpu().numpy(), lza.cpu().numpy()
    for b in range(B):
        m = x[b].max()
        valid = np.flatnonzero(mask[b])
        if m == -np.inf:
            assert ids[b] == -1 and lzv[b] == -np.inf and lza[b] == -np.inf
            continue
        want = np.log(np.exp(x[b] - m).sum()) + m
        assert abs(lza[b] - want) <= 1e-5 * max(1.0, abs(want)), (b, lza[b], want)
        e = np.exp(x[b, valid] - m)
        assert e.sum() > 0
        assert abs(lzv[b] - np.log(e.sum()) - (m - want)) <= 2e-5 * max(1.0, abs(want) / 64), (b, lzv[b])
        cdf = np.cumsum(e) / e.sum()
        at = int(np.searchsorted(cdf, un[b], side="right"))
        assert ids[b] == valid[min(at, len(valid) - 1)] or np.abs(cdf - un[b]).min() < CDF_BAND, (b, ids[b])


@pytest.mark.parametrize("fill", [-np.inf, -1e9])
@pytest.mark.parametrize("dtype,V,B", [("bf16", 32_000, 2_048), ("f32", 50_264, 384)])
def test_filtered_rows_take_no_second_pass(dtype, V, B, fill):
    """A batch of filtered rows takes as long as one of unfiltered rows (reading every tile twice took 1.6 to 1.9 times as
    long; what is wanted is 1, and half of the difference is left for noise)."""
    rng = np.random.default_rng(1)
    lg = rng.normal(0, 2, size=(B, V)).astype(np.float32)
    noise = to_dev(lg)
    few = torch.where(noise >= noise.topk(50, dim=1).values[:, -1:], noise, torch.full_like(noise, float(fill)))
    if dtype == "bf16":
        noise, few = noise.bfloat16(), few.bfloat16()
    mask = np.zeros((B, -(-V // 32) * 32), np.uint8)
    mask[np.arange(B)[:, None], rng.integers(0, V, (B, 20))] = 1
    words = to_dev(np.packbits(mask, axis=1, bitorder="little").view(np.int32))
    un = to_dev(rng.random(B, dtype=np.float32))
    ids = torch.zeros(B, dtype=torch.int32, device=DEV)
    lzv, lza = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
    best = {}
    for _ in range(12):
        for name, x in (("noise", noise), ("few", few)):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            ppv.constrained_sample(x, words, un, ids, lzv, lza)
            a.record()
            for _ in range(20):
                ppv.constrained_sample(x, words, un, ids, lzv, lza)
            b.record()
            torch.cuda.synchronize()
            best[name] = min(best.get(name, 1e9), a.elapsed_time(b))
    assert best["few"] < 1.4 * best["noise"], best


F32_MIN, BF16_MIN = float(np.finfo(np.float32).min), -3.3895313892515355e38   # (torch.finfo(torch.bfloat16).min)


def on_device(lg, dtype):
    """((rows, V) of dtype on the device, the same values in 64 bits)"""
    V = lg.shape[-1]
    buf = np.zeros(lg.shape[:-1] + (-(-V // 8) * 8,), np.float32)
    buf[..., :V] = lg
    if dtype == "f32":
        return to_dev(buf)[..., :V], lg.astype(np.float64)
    bits = W.f32_to_bf16_bits(buf)
    return to_dev(bits.view(np.int16)).view(torch.bfloat16)[..., :V], W.bf16_bits_to_f32(bits)[..., :V].astype(np.float64)


def check_row(x, valid, u, id, lzv, lza=None):
    """A row of logits over T in 64 bits, its valid tokens and its uniform against what was drawn.  A mass is a difference of
    two logarithms, each rounded to 2^-24 of itself, beside sums of 2^-24 a term: 2e-5 of the larger; beyond fp32 -inf."""
    top, vtop = x.max(), x[valid].max()
    all_ref = top + np.log(np.exp(x - top).sum())
    w = np.exp(x[valid] - vtop)
    val_ref = (vtop - top) + np.log(w.sum()) - np.log(np.exp(x - top).sum())
    for got, want, size in ((lza, all_ref, abs(all_ref)), (lzv, val_ref, max(abs(val_ref), min(abs(all_ref), 1e4)))):
        if got is None:
            continue
        if abs(want) >= 3.4e38:
            assert got == np.copysign(np.inf, want) or abs(got) > 3.39e38, (got, want)
        else:
            assert abs(float(got) - want) <= 2e-5 * max(1.0, size / 64), (got, want)
    cdf = np.cumsum(w) / w.sum()
    at = min(int(np.searchsorted(cdf, u, side="right")), len(valid) - 1)
    assert id == valid[at] or (id in valid and np.abs(cdf - u).min() < CDF_BAND), (id, valid[at])


FAR = [(-4e3, 1e-6), (-1e8, 1.0), (-1.2e9, 1.0), (-1e9, 0.3), (-1e10, 1.0), (-3e12, 1.0), (-1e30, 0.3), (BF16_MIN, 1.0), (BF16_MIN, 0.3), (F32_MIN, 1.0), (F32_MIN, 0.3)]


@pytest.mark.parametrize("fill,T", FAR)
@pytest.mark.parametrize("dtype,V", [("f32", 1_024), ("f32", 1_000), ("bf16", 2_047), ("f32", 9_004), ("bf16", 32_000), ("bf16", 131_000)])
def test_logits_of_any_size(dtype, V, fill, T):
    """Logits so far from 0 that their products with log2(e) / T are known to whole units only, or not at all: rows filtered
    with them, made of them, allowed only them; and the same above the rest of the row."""
    if dtype == "bf16" and fill < BF16_MIN:
        pytest.skip("no bf16 number")
    rng = np.random.default_rng(V)
    lg = np.concatenate([filtered_rows(V, 50, rng, fill), rng.normal(0, 2, size=(5, V)).astype(np.float32)])
    B = len(lg)
    step = np.spacing(np.float32(fill / 2))
    lg[9] = np.float32(-fill / 2) + step * rng.integers(0, 4, V).astype(np.float32)        # neighbours, all of them far from 0
    lg[10] = -lg[9]
    lg[6, rng.choice(V, 4, replace=False)] = -fill                         # far above the rest
    lg[7, rng.choice(V, V // 2, replace=False)] = fill
    lg[7, rng.choice(V, V // 8, replace=False)] = fill / 2
    lg[8, :: 256] = -fill                                                  # ... also where references are looked for
    lg[8, 5] = -fill / 2
    ld, x = on_device(lg, dtype)
    x = x / T
    for n_valid in (1, 30, min(200, V // 3), V // 3):                      # one token, lists of a slice and of several, an image
        mask = np.zeros((B, V), np.uint8)
        for b in range(B):
            mask[b, rng.choice(V, n_valid, replace=False)] = 1
            if b not in (3, 4, 7):
                mask[b, np.flatnonzero(lg[b] > fill)[:3]] = 1
        mask[3] &= lg[3] == np.float32(fill)                               # only what was filtered out
        mask[3, np.flatnonzero(lg[3] == np.float32(fill))[:2]] = 1
        mask[4] = 0
        mask[4, np.flatnonzero(lg[4] == np.float32(fill))[-n_valid:]] = 1
        words = np.packbits(np.pad(mask, ((0, 0), (0, (-V) % 32))), axis=1, bitorder="little").view(np.int32)
        un = rng.random(B, dtype=np.float32)
        ids = torch.full((B,), -9, dtype=torch.int32, device=DEV)
        lzv, lza = torch.zeros(B, device=DEV), torch.zeros(B, device=DEV)
        ppv.constrained_sample(ld, to_dev(words), to_dev(un), ids, lzv, lza, temperature=T)
        ids, lzv, lza = ids.cpu().numpy(), lzv.cpu().numpy(), lza.cpu().numpy()
        for b in range(B):
            check_row(x[b], np.flatnonzero(mask[b]), un[b], ids[b], lzv[b], lza[b])


@pytest.mark.parametrize("fill,T", FAR)
@pytest.mark.parametrize("dtype,V", [("f32", 1_000), ("bf16", 9_000), ("f32", 40_000)])
def test_decoding_under_logits_of_any_size(dtype, V, fill, T):
    """The same through the root's image, short lists, long lists and chains of the decoding calls: every step against 64
    bits, one launch per step and one for all bit for bit, ppv_sample_next beside them."""
    if dtype == "bf16" and fill < BF16_MIN:
        pytest.skip("no bf16 number")
    rng = np.random.default_rng(V + 1)
    n, L, B = 6_000, 5, 24
    S = rng.integers(0, V, (n, L)).astype(np.int32)
    S[:3_000, 0] = 1 + rng.integers(0, 4, 3_000)                           # four heavy first tokens
    S[:1_500, 1] = rng.integers(0, 30, 1_500)                              # ... with short lists below some
    index = ppv.ppv_build_index(S.reshape(-1), np.arange(n + 1, dtype=np.int64) * L, V)
    lg = np.concatenate([filtered_rows(V, 50, rng, fill) for _ in range(L * B // 6)]).reshape(L, B, V)
    lg[0, :, 1:5] = 9.0                                                    # (most rows go below the heavy tokens)
    lg[1, ::2, :30] = 8.0
    lg[2:, 3] = -fill                                                      # a row far above 0
    ld, x = on_device(lg, dtype)
    un = to_dev(rng.random((L, B), dtype=np.float32))
    runs = []
    for one_launch in (False, True):
        P = torch.full((B, L), 7, dtype=torch.int32, device=DEV)
        lens, act = torch.zeros(B, dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.uint8, device=DEV)
        state = torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
        lx, lz = torch.zeros(B, device=DEV), torch.full((L, B), 7.0, device=DEV)
        ids = torch.full((L, B), -7, dtype=torch.int32, device=DEV)
        ppv.ppv_decode_begin_empty(index, lens, state, act, lx)
        if one_launch:
            ppv.ppv_decode_loop(index, P, lens, act, ld, un, ids, lz, lx, state=state, temperature=T)
        else:
            for s in range(L):
                words = torch.zeros((B, index.n_words), dtype=torch.int32, device=DEV)
                nxt, mass = torch.zeros(B, dtype=torch.int32, device=DEV), torch.zeros(B, device=DEV)
                ppv.ppv_next_token_mask(index, P, lens, words)
                ppv.ppv_sample_next(index, P, lens, ld[s], un[s], nxt, mass, temperature=T)
                ppv.ppv_decode_step(index, P, lens, act, ld[s], un[s], ids[s], lz[s], lx, state=state, temperature=T)
                bits = np.unpackbits(words.cpu().numpy().view(np.uint8), axis=1, bitorder="little")[:, :V]
                for b in range(B):
                    for id, mass_of in ((ids[s, b], lz[s, b]), (nxt[b], mass[b])):
                        check_row(x[s, b] / T, np.flatnonzero(bits[b]), float(un[s, b]), int(id), float(mass_of))
        torch.cuda.synchronize()
        runs.append([t.cpu().numpy() for t in (P, lens, act, ids, lz, lx)])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
    assert (runs[0][1] == L).all()


@pytest.mark.parametrize("dtype,V", [("f32", 1024), ("f32", 997), ("f32", 260), ("f32", 3), ("bf16", 2048), ("bf16", 2041), ("bf16", 520)])
def test_rows_of_one_tile_find_their_token(dtype, V):
    """Rows of a single tile: one valid token at the edges of lanes, groups and the row, two in one lane, two at the ends of two groups, and
    rows that are valid throughout; mask bits behind the vocabulary are set and do not count."""
    per, group = (8, 512) if dtype == "bf16" else (4, 256)
    rng = np.random.default_rng(V)
    spots = sorted({p for p in (0, 1, per - 1, per, group - 1, group, 2 * group, V - 2, V - 1) if 0 <= p < V})
    sets = [[p] for p in spots] + [[p, p + 1] for p in spots if p + 1 < V] + [[spots[0], spots[-1]], list(range(V)), list(range(0, V, 7))]
    sets = sets + sets
    lg = rng.normal(0, 2, size=(len(sets), V)).astype(np.float32)
    un = np.concatenate([np.zeros(len(sets) // 2), np.full(len(sets) // 2, 1 - 2.0 ** -24)]).astype(np.float32)   # the first and the last
    un[len(sets) // 2 - 2:len(sets) // 2] = 0.5
    mask = np.ones((len(sets), -(-V // 32) * 32), np.uint8)
    mask[:, :V] = 0
    for b, s in enumerate(sets):
        mask[b, s] = 1
    dev, x = on_device(lg, dtype)
    ids = torch.full((len(sets),), -9, dtype=torch.int32, device=DEV)
    lzv, lza = torch.zeros(len(sets), device=DEV), torch.zeros(len(sets), device=DEV)
    ppv.constrained_sample(dev, to_dev(np.packbits(mask, axis=1, bitorder="little").view(np.int32)), to_dev(un), ids, lzv, lza)
    ids, lzv, lza = ids.cpu().numpy(), lzv.cpu().numpy(), lza.cpu().numpy()
    for b, s in enumerate(sets):
        check_row(x[b], np.array(s), un[b], ids[b], lzv[b], lza[b])
        if len(s) <= 2:
            assert ids[b] == (s[0] if un[b] == 0 else s[-1])


@pytest.mark.parametrize("dtype,V", [("f32", 1_024), ("f32", 777), ("bf16", 2_048), ("bf16", 1_500)])
@pytest.mark.parametrize("scale", [1.0, 1e8])
def test_one_tile_rows_under_an_image_are_the_decode_step_s(dtype, V, scale):
    """constrained_sample and ppv_sample_next have kernels of their own for rows of one tile, the first decode step has not: the same
    tokens and the same bits of the masses, for uniforms on the very edges between two tokens.  (Logits of 1e8 are taken apart differently
    from usual ones.)"""
    rng = np.random.default_rng(V)
    B, per = 2_000, 8
    first = np.sort(rng.choice(V, V // 2, replace=False)).astype(np.int32)
    index = ppv.ppv_build_index(first, np.arange(len(first) + 1, dtype=np.int64), V)
    lg = rng.normal(0, 2, size=(B, -(-V // per) * per)).astype(np.float32)
    if scale != 1.0:
        lg = (scale + np.round(lg) * 8).astype(np.float32)     # (neighbours at 1e8)
    ld = to_dev(lg)
    if dtype == "bf16":
        ld = ld.to(torch.bfloat16)
    ld = ld[:, :V]
    x = ld.float().cpu().numpy().astype(np.float64)[:, first]
    w = np.exp(x - x.max(1, keepdims=True))
    cdf = np.cumsum(w, 1) / w.sum(1, keepdims=True)
    un = cdf[np.arange(B), rng.integers(0, len(first) - 1, B)].astype(np.float32)
    un = to_dev(np.minimum(un, np.float32(1) - np.float32(2 ** -24)))
    P, lens = torch.zeros((B, 2), dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.int32, device=DEV)
    words = torch.zeros((B, index.n_words), dtype=torch.int32, device=DEV)
    ppv.ppv_next_token_mask(index, P, lens, words)
    got = []
    for name in ("step", "next", "sample"):
        ids, lz = torch.full((B,), -9, dtype=torch.int32, device=DEV), torch.zeros(B, device=DEV)
        if name == "step":
            act, state = torch.ones(B, dtype=torch.uint8, device=DEV), torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
            ppv.ppv_decode_first_step(index, P.clone(), lens.clone(), act, ld, un, ids, lz, torch.zeros(B, device=DEV), state=state)
        elif name == "next":
            ppv.ppv_sample_next(index, P, lens, ld, un, ids, lz)
        else:
            ppv.constrained_sample(ld, words, un, ids, lz)
        got.append((ids.cpu().numpy(), lz.cpu().numpy().view(np.int32)))
    for ids, lz in got[1:]:
        assert np.array_equal(ids, got[0][0]), np.flatnonzero(ids != got[0][0])[:8]
        assert np.array_equal(lz, got[0][1])
