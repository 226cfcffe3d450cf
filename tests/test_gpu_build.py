"""The index builder at the sizes where its steps change over: groups of equal first tokens at and beyond what is ordered
by counting, several rounds of them, vocabularies at and beyond 16 bits, uploads of several slots and more than the ring
holds, rows too long for the staging in LDS, more heavy prefixes than the index's block has room for, and prefixes that
leave a member behind the point where it is alone.  Everything against the oracle."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2504_09135_amd import binding as ppv
from paper_2504_09135_amd import workloads as W

from gpu_helpers import DEV, assert_query_parity, to_dev

pytestmark = pytest.mark.gpu


def csr(rows, lens):
    offsets = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offsets[1:])
    keep = np.arange(rows.shape[1])[None, :] < np.asarray(lens)[:, None]
    return np.ascontiguousarray(rows[keep], dtype=np.int32), offsets


def prefixes_of(tokens, offsets, V, rng, n, stride):
    """Prefixes of members: as they are, with a wrong token at any place, and beyond a member's end."""
    P = np.full((n, stride), W.PAD_TOKEN, np.int32)
    L = np.zeros(n, np.int32)
    who = rng.integers(0, len(offsets) - 1, n)
    for i, w in enumerate(who):
        row = tokens[offsets[w]:offsets[w + 1]][:stride]
        k = int(rng.integers(0, len(row) + 1))
        P[i, :k] = row[:k]
        kind = i % 4
        if kind == 1 and k:
            P[i, int(rng.integers(0, k))] = int(rng.integers(0, V))
        elif kind == 2 and k < stride:
            P[i, k] = int(rng.integers(0, V))
            k += 1
        elif kind == 3 and k:
            P[i, k - 1] = int(rng.integers(0, V))
        L[i] = k
    return P, L


def check(tokens, offsets, V, rng, n_prefixes=300, stride=None):
    trie = oracle.Trie(tokens, offsets, V)
    index = ppv.ppv_build_index(tokens, offsets, V)
    assert (index.n_distinct, index.l_max, index.n_prefixes) == (trie.n_members, trie.l_max, trie.n_nodes - 1)
    got_t, got_o = ppv.ppv_index_export(index)
    P, L = prefixes_of(tokens, offsets, V, rng, n_prefixes, stride or index.l_max + 2)
    assert_query_parity(index, trie, P, L)
    index.free()
    return got_t, got_o


@pytest.mark.parametrize("group", [2, 255, 512, 1024, 1025, 3000])
@pytest.mark.parametrize("V,stem,tail", [(300, 6, 3), (32_000, 4, 1), (70_000, 9, 6), (1_000, 40, 30)])
def test_groups_of_equal_first_tokens(group, V, stem, tail):
    """`group` rows that share their first `stem` tokens (and some that are duplicates, or end there), among others."""
    rng = np.random.default_rng(group * 7 + V)
    s = rng.integers(0, V, stem)
    rows = rng.integers(0, min(V, 40), (group + 500, stem + tail))
    rows[:group, :stem] = s
    lens = rng.integers(1, stem + tail + 1, group + 500)
    lens[:group] = rng.integers(stem, stem + tail + 1, group)
    rows[group // 2] = rows[0]
    lens[group // 2] = lens[0]
    order = rng.permutation(group + 500)
    tokens, offsets = csr(rows[order], lens[order])
    got_t, got_o = check(tokens, offsets, V, rng)
    rows_out = [tuple(got_t[a:b]) for a, b in zip(got_o[:-1], got_o[1:])]
    assert rows_out == sorted({tuple(tokens[a:b]) for a, b in zip(offsets[:-1], offsets[1:])})


@pytest.mark.parametrize("copies", [16, 17, 300, 1_024, 1_025])
@pytest.mark.parametrize("V,length", [(300, 23), (128_256, 18), (90, 400)])
def test_sets_with_many_copies_and_long_common_stems(copies, V, length):
    """Groups that stay together for several rounds: copies of whole rows, and rows that differ in their last token only."""
    rng = np.random.default_rng(copies + V)
    base = rng.integers(0, V, (5, length))
    rows = np.repeat(base, copies, axis=0)
    lens = np.full(len(rows), length)
    rows[copies:2 * copies, -1] = rng.integers(0, V, copies)              # a stem and its leaves
    rows[2 * copies:3 * copies, length // 2] = rng.integers(0, 3, copies)  # three branches half way, alike again behind it
    lens[3 * copies:4 * copies:2] = rng.integers(1, length + 1, len(lens[3 * copies:4 * copies:2]))
    rows = np.concatenate([rows, rng.integers(0, V, (400, length))])
    lens = np.concatenate([lens, rng.integers(1, length + 1, 400)])
    order = rng.permutation(len(rows))
    tokens, offsets = csr(rows[order], lens[order])
    got_t, got_o = check(tokens, offsets, V, rng)
    rows_out = [tuple(got_t[a:b]) for a, b in zip(got_o[:-1], got_o[1:])]
    assert rows_out == sorted({tuple(tokens[a:b]) for a, b in zip(offsets[:-1], offsets[1:])})


@pytest.mark.parametrize("V", [1, 2, 65_535, 65_536, 65_537, ppv.PPV_MAX_VOCAB])
def test_vocabularies_at_the_edges_of_the_packed_forms(V):
    rng = np.random.default_rng(V)
    rows = rng.integers(max(0, V - 50), V, (2_000, 7))
    rows[::3] = rng.integers(0, V, rows[::3].shape)
    tokens, offsets = csr(rows, rng.integers(1, 8, 2_000))
    check(tokens, offsets, V, rng)
    for bad in (V, -1):
        wrong = tokens.copy()
        wrong[len(wrong) // 2] = bad
        with pytest.raises(ppv.PPVError):
            ppv.ppv_build_index(wrong, offsets, V)


@pytest.mark.parametrize("n,L,V", [(131_071, 2, 500), (131_073, 2, 70_000), (600_000, 30, 70_000)])
def test_uploads_of_several_slots(n, L, V):
    """Around a slot of offsets, several slots of tokens, and 18M tokens (more slots than the ring has)."""
    rng = np.random.default_rng(n)
    rows = rng.integers(0, V, (n, L), dtype=np.int32)
    lens = np.full(n, L)
    tokens, offsets = csr(rows, lens)
    index = ppv.ppv_build_index(tokens, offsets, V)
    got_t, got_o = ppv.ppv_index_export(index)
    # row order by the radix-free route: numpy's lexicographic sort
    srt = rows[np.lexsort(rows.T[::-1])]
    keep = np.concatenate([[True], (srt[1:] != srt[:-1]).any(axis=1)])
    assert np.array_equal(got_t.reshape(-1, L), srt[keep]) and got_o[-1] == got_t.size
    index.free()
    for at in (0, n // 2, n - 1):
        broken = offsets.copy()
        broken[at + 1] = broken[at]                          # an empty sequence, in the first, a middle and the last slot
        with pytest.raises(ppv.PPVError):
            ppv.ppv_build_index(tokens, broken, V)
    wrong = tokens.copy()
    wrong[-1] = V
    with pytest.raises(ppv.PPVError):
        ppv.ppv_build_index(wrong, offsets, V)


@pytest.mark.parametrize("lens_of_64", [(1, 1), (64, 64), (1, 64), (65, 66), (200, 400)])
def test_rows_around_the_staging_in_lds(lens_of_64):
    """64 rows that fit their wavefront's LDS and 64 that do not, next to each other."""
    rng = np.random.default_rng(lens_of_64[1])
    a, b = lens_of_64
    lens = rng.integers(a, b + 1, 900)
    lens[:300] = 1 + lens[:300] // 8
    rows = rng.integers(0, 90, (900, int(lens.max())))
    rows[:, 0] = np.arange(900) // 13
    tokens, offsets = csr(rows, lens)
    check(tokens, offsets, 90, rng)


@pytest.mark.parametrize("heads", [250, 256, 257, 700])
def test_number_of_heavy_prefixes(heads):
    """`heads` second-level prefixes (and the root) with more than V / 32 children each."""
    V = 1_024
    rng = np.random.default_rng(heads)
    first = rng.choice(V, heads - 1, replace=False)
    rows = np.array([(f, c) for f in first for c in rng.choice(V, 40, replace=False)])
    tokens, offsets = csr(rows, np.full(len(rows), 2))
    check(tokens, offsets, V, rng)


def test_builds_one_after_another_reuse_memory():
    """Indices of different sizes built, queried and freed in turn, two of them alive at a time."""
    rng = np.random.default_rng(5)
    alive = []
    for k in range(12):
        n = int(rng.integers(10, 60_000))
        V = int(rng.integers(5, 90_000))
        rows = rng.integers(0, V, (n, 6), dtype=np.int32)
        tokens, offsets = csr(rows, rng.integers(1, 7, n))
        trie = oracle.Trie(tokens, offsets, V)
        index = ppv.ppv_build_index(tokens, offsets, V)
        P, L = prefixes_of(tokens, offsets, V, rng, 64, 8)
        alive.append((index, trie, P, L))
        for ix, t, p, l in alive:
            assert_query_parity(ix, t, p, l)
        if len(alive) == 2:
            alive.pop(int(rng.integers(0, 2)))[0].free()
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,ok", [(60_000, True), (61_400, False)])
def test_sets_beyond_the_limit_of_depths_times_rows_are_refused(n, ok):
    """One row of 70,000 tokens among rows of one token: accepted while depths x rows stay below 2^32 (4.2e9 and 4.298e9)."""
    long = np.arange(70_000, dtype=np.int32)
    tokens = np.concatenate([long, np.arange(1, n, dtype=np.int32)])
    offsets = np.concatenate([[0], 70_000 + np.arange(n)]).astype(np.int64)
    if not ok:
        with pytest.raises(ppv.PPVError, match="ERANGE"):
            ppv.ppv_build_index(tokens, offsets, 70_000)
        return
    index = ppv.ppv_build_index(tokens, offsets, 70_000)
    assert (index.n_distinct, index.l_max, index.n_prefixes) == (n, 70_000, 70_000 + n - 1)
    index.free()


def test_copies_do_not_count_towards_that_limit():
    """A row of 2^17 tokens among 2^21 rows of one token, nearly all of them copies: 2^32 (depth, 64 rows) pairs as given,
    6 rows of the index."""
    n, length = 1 << 21, 1 << 17
    rng = np.random.default_rng(3)
    tokens = np.concatenate([np.arange(n - 1, dtype=np.int32) % 5, rng.integers(0, 1_024, length).astype(np.int32)])
    offsets = np.append(np.arange(n), n - 1 + length).astype(np.int64)
    index = ppv.ppv_build_index(tokens, offsets, 1_024)
    assert (index.n_distinct, index.l_max) == (6, length)
    got_t, got_o = ppv.ppv_index_export(index)
    want = sorted([(t,) for t in range(5)] + [tuple(tokens[n - 1:].tolist())])
    assert [tuple(got_t[a:b].tolist()) for a, b in zip(got_o[:-1], got_o[1:])] == want
    index.free()


@pytest.mark.parametrize("V", [1_024, 256_000])
def test_a_small_set_holds_little_memory(V):
    """Room for images is laid out for the heavy prefixes that there can be, not for 256 of them (16 MB at V = 256,000)."""
    rng = np.random.default_rng(V)
    tokens, offsets = csr(rng.integers(0, V, (60, 5)), np.full(60, 5))
    index = ppv.ppv_build_index(tokens, offsets, V)
    assert index.device_bytes < 1_000_000
    index.free()


def test_builds_from_several_threads():
    """Threads that build, query and free sets of their own at the same time, each upload several slots long: they
    share the ring of pinned slots, the kept blocks and the pinned words."""
    sets = []
    for k in range(3):
        rng = np.random.default_rng(100 + k)
        V = (500, 70_000, 30_000)[k]
        n = 150_000 + 20_000 * k
        rows = rng.integers(0, V, (n, 6), dtype=np.int32)
        rows[:, 0] = rows[:, 0] % 50
        tokens, offsets = csr(rows, rng.integers(1, 7, n))
        trie = oracle.Trie(tokens, offsets, V)
        P, L = prefixes_of(tokens, offsets, V, rng, 128, 8)
        sets.append((tokens, offsets, V, trie, P, L))
    errors = []

    def work(k):
        try:
            tokens, offsets, V, trie, P, L = sets[k]
            for _ in range(6):
                index = ppv.ppv_build_index(tokens, offsets, V)
                assert (index.n_distinct, index.n_prefixes) == (trie.n_members, trie.n_nodes - 1)
                with torch.cuda.stream(torch.cuda.Stream()):
                    assert_query_parity(index, trie, P, L)
                index.free()
        except BaseException as e:   # noqa: BLE001 (reported by the test's own thread)
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_heavy_prefixes_with_large_numbers():
    """Few heavy prefixes (more than 1,024 children), some of them behind the first 2^20 prefixes: the images are laid out again."""
    V, heads = 200_000, 4
    rng = np.random.default_rng(11)
    base = np.array([(f, c % V, (f + c) % V) for f in range(V) for c in (f, f + 70_000, f + 140_000)], np.int32)
    stems = base[np.lexsort(base.T[::-1])][[10, -40, -20, -1]]              # low and high numbers at depth 3
    more = np.concatenate([np.column_stack([np.repeat(s[None], 1_500, 0), rng.choice(V, 1_500, replace=False)]) for s in stems])
    tokens = np.concatenate([base.ravel(), more.astype(np.int32).ravel()])
    offsets = np.concatenate([np.arange(len(base)) * 3, base.size + np.arange(len(more) + 1) * 4]).astype(np.int64)
    trie = oracle.Trie(tokens, offsets, V)
    index = ppv.ppv_build_index(tokens, offsets, V)
    assert index.n_prefixes == trie.n_nodes - 1 > (1 << 20)
    P = np.full((64, 5), W.PAD_TOKEN, np.int32)
    L = np.zeros(64, np.int32)
    for i in range(64):
        row = stems[i % heads] if i < 32 else base[rng.integers(0, len(base))]
        L[i] = 3 if i < 48 else rng.integers(0, 4)
        P[i, :L[i]] = row[:L[i]]
    assert_query_parity(index, trie, P, L)
    # the same rows through the sampler and a step with a cursor: one valid token, the same one
    lg, un = torch.randn((64, V), device=DEV), torch.rand(64, device=DEV)
    pd, ld = to_dev(P), to_dev(L)
    ids = torch.full((64,), -7, dtype=torch.int32, device=DEV)
    ppv.ppv_sample_next(index, pd, ld, lg, un, ids)
    state = torch.zeros((64, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
    active = torch.zeros(64, dtype=torch.uint8, device=DEV)
    ppv.ppv_decode_begin(index, pd, ld, state, active)
    active.fill_(1)
    step = torch.full((64,), -7, dtype=torch.int32, device=DEV)
    ppv.ppv_decode_step(index, pd, ld, active, lg, un, step, state=state)
    ids, step = ids.cpu().numpy(), step.cpu().numpy()
    assert np.array_equal(ids, step)
    children = {tuple(s): set(more[(more[:, :3] == s).all(axis=1), 3]) for s in stems}
    for i in range(32):
        assert ids[i] in children[tuple(P[i, :3])]
    index.free()
