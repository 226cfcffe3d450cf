"""Rows spread over several workgroups (small batches): every number of workgroups per row gives bit for bit the
result of one workgroup per row, which in turn is checked against the oracle.  The split is a launch detail
(PPV_TUNE_ROW_SPLIT forces it; the library picks it from the batch size and the row length otherwise)."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_2504_09135_amd import binding as ppv
from paper_2504_09135_amd import workloads as W

from gpu_helpers import DEV, check_sample_rows, logits_to_dev, to_dev, tuning
from test_gpu_parity import setup_case

pytestmark = pytest.mark.gpu

SPLITS = (1, 2, 4, 8, 16)


def pack(mask: np.ndarray) -> np.ndarray:
    B, V = mask.shape
    pad = (-V) % 32
    return np.packbits(np.pad(mask, ((0, 0), (0, pad))), axis=1, bitorder="little").view(np.uint32).view(np.int32)


def sample_all_splits(logits_dev, words_dev, un_dev, temperature=1.0, waves=0):
    """constrained_sample with 1, 2, ... workgroups per row; returns the unsplit result after checking that every
    split reproduces its bits."""
    B = logits_dev.shape[0]
    base = None
    for k in SPLITS:
        ids = torch.full((B,), -7, dtype=torch.int32, device=DEV)
        lzv = torch.full((B,), 3.0, dtype=torch.float32, device=DEV)
        lza = torch.full((B,), 3.0, dtype=torch.float32, device=DEV)
        with tuning(ppv.PPV_TUNE_ROW_SPLIT, k), tuning(ppv.PPV_TUNE_WAVES_PER_ROW, waves):
            ppv.constrained_sample(logits_dev, words_dev, un_dev, ids, lzv, lza, temperature=temperature)
        torch.cuda.synchronize()
        got = (ids.cpu().numpy(), lzv.cpu().numpy(), lza.cpu().numpy())
        if base is None:
            base = got
            continue
        assert np.array_equal(got[0], base[0]), (k, np.nonzero(got[0] != base[0])[0][:8])
        assert np.array_equal(got[1].view(np.int32), base[1].view(np.int32)), k
        assert np.array_equal(got[2].view(np.int32), base[2].view(np.int32)), k
    return base


@pytest.mark.parametrize("name", ["C2", "C5s", "C3s"])
def test_split_rows_on_the_workloads(name):
    cfg, S, trie, index = setup_case(name)
    pb = W.make_prefix_batch(cfg, S)
    logits = W.make_logits(cfg)
    un = W.make_uniforms(cfg)
    ref = trie.step(pb.prefixes, pb.lens, W.logits_as_f32(cfg, logits), un, threads=8)
    ids, lzv, lza = sample_all_splits(logits_to_dev(cfg, logits), to_dev(pack(ref.mask)), to_dev(un))
    check_sample_rows(cfg.dtype, ref, lambda b: ref.mask[b], un, ids, lzv, lza)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("waves", [0, 1, 2])
def test_split_rows_hand_made_masks(dtype, waves):
    """List rows of 0, 1, 63, 64, 65, 700 and 1,000 valid tokens, image rows, an image row whose valid mass lies far
    below the row maximum (the second pass over the row), rows with -inf tiles, a ragged last tile; several tiles per
    workgroup and fewer tiles than wavefronts."""
    V = 128_256                                               # the vocabulary of the paper's larger model (Table 1)
    rng = np.random.default_rng(31)
    counts = [0, 1, 63, 64, 65, 700, 1000, 1100, 5000, V // 2, 300, 40, 4000, 1]
    B = len(counts)
    lg = (rng.standard_normal((B, V)) * 2).astype(np.float32)
    mask = np.zeros((B, V), np.uint8)
    for b, c in enumerate(counts):
        mask[b, rng.choice(V, c, replace=False)] = 1
    lg[10, mask[10] == 1] -= 150.0                            # list row, mass ~ e^-150
    lg[12, mask[12] == 1] -= 60.0                             # image row, mass ~ e^-55: sums are redone
    lg[11, : V // 3] = -np.inf                                # whole tiles without a finite value
    lg[13, mask[13] == 1] = -np.inf                           # the only valid token has probability 0
    un = rng.random(B, dtype=np.float32)
    un[2], un[3] = 0.0, np.float32(1.0) - np.float32(2 ** -24)
    if dtype == "bf16":
        bits = W.f32_to_bf16_bits(lg)
        lf = W.bf16_bits_to_f32(bits)
        ld = to_dev(bits.view(np.int16)).view(torch.bfloat16)
    else:
        lf, ld = lg, to_dev(lg)
    ids, lzv, lza = sample_all_splits(ld, to_dev(pack(mask)), to_dev(un), waves=waves)
    ref = oracle.masked_sample(lf, mask, un, threads=8)
    check_sample_rows(dtype, ref, lambda b: mask[b], un, ids, lzv, lza)
    assert ids[0] == -1 and ids[13] == -1 and lzv[13] == -np.inf


def test_split_rows_with_temperature_and_a_second_smaller_call():
    """The scratch area is the same for one call after the other: a second, smaller call right after a larger one, at
    another temperature and on other rows, must not see any of it."""
    cfg, S, trie, index = setup_case("C2")
    pb = W.make_prefix_batch(cfg, S)
    for step, (rows, T) in enumerate([(slice(0, 64), 0.7), (slice(5, 22), 1.9), (slice(0, 64), 1.0)]):
        logits = W.make_logits(cfg, step=40 + step)[rows]
        un = W.make_uniforms(cfg, step=40 + step)[rows]
        P, L = pb.prefixes[rows], pb.lens[rows]
        ref = trie.step(P, L, W.logits_as_f32(cfg, logits), un, threads=8, temperature=T)
        ids, lzv, lza = sample_all_splits(logits_to_dev(cfg, logits), to_dev(pack(ref.mask)), to_dev(un), temperature=T)
        check_sample_rows(cfg.dtype, ref, lambda b: ref.mask[b], un, ids, lzv, lza)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_one_area_for_calls_of_every_kind(dtype):
    """Calls whose rows are of other kinds and numbers one after the other in one area: lists of 1, 64, 65 and 1,000 tokens, images and
    empty sets take each other's places, with listed weights and valid sums of 0, and each call gives the unsplit call's bits.  (That
    nothing of another call is taken: test_no_word_of_another_call_is_taken.)"""
    V = 50_001
    g = torch.Generator(device=DEV).manual_seed(8)
    counts = [0, 1, 64, 65, 1_000, 20_000]
    words = torch.zeros((len(counts), (V + 31) // 32), dtype=torch.int32)
    for i, n in enumerate(counts):
        m = np.zeros((1, V), np.uint8)
        m[0, np.random.default_rng(i).choice(V // 2, n, replace=False)] = 1   # (whole tiles without a valid token)
        words[i] = torch.from_numpy(pack(m)[0])
    for step, B in enumerate([12, 5, 16, 1, 12]):
        logits = torch.randn((B, -(-V // 8) * 8), generator=g, device=DEV).mul_(2).to(dtype)[:, :V]
        logits[::3] = logits[::3].sign() * -150   # listed weights of 0
        logits[::3, ::7] = 0
        un = torch.rand(B, generator=g, device=DEV)
        kinds = (torch.arange(B) + step) % len(counts)
        sample_all_splits(logits, words[kinds].to(DEV), un)


class Area:
    """The area that calls on the default stream meet in, or the fixed array: each row's count of workgroups that have arrived, then the
    words of all rows, a value and a call's mark each."""
    def __init__(self, fixed=False):
        self.fixed = fixed
        at, n, words = self.look_again(True)
        self.__cuda_array_interface__ = {"shape": (n // 4,), "typestr": "<i4", "data": (at, False), "version": 3}
        everything = torch.as_tensor(self, device=DEV)
        self.arrived, self.words = everything[:words // 4], everything[words // 4:].view(-1, 2)

    def look_again(self, on):
        """Whether calls from here on wait for a word that is not there when they first look."""
        at, n, words = C.c_void_p(), C.c_int64(), C.c_int64()
        torch.cuda.synchronize()
        lib = ppv.load_library()
        assert lib.ppv_split_area_for_tests(None, int(self.fixed), int(on), C.byref(at), C.byref(n), C.byref(words)) == 0
        return at.value, n.value, words.value

    def disturb(self, B, arrived):
        """As calls that overlap may leave it: words of a call, with plausible values, and workgroups of no call counted."""
        self.words[:, 0] = torch.tensor(1.5).view(torch.int32).item()
        self.words[:, 1] = 0x7FFFFFFF
        self.arrived[:B] = arrived
        torch.cuda.synchronize()


def sample_case(dtype, seed, V=100_000):
    """Rows of every kind: an empty set, lists of 1, 64, 65 and 1,000 tokens, an image."""
    counts = [0, 1, 64, 65, 1_000, 20_000] * 2
    words = torch.zeros((len(counts), (V + 31) // 32), dtype=torch.int32)
    for i, n in enumerate(counts):
        m = np.zeros((1, V), np.uint8)
        m[0, np.random.default_rng(100 * seed + i).choice(V, n, replace=False)] = 1
        words[i] = torch.from_numpy(pack(m)[0])
    g = torch.Generator(device=DEV).manual_seed(seed)
    logits = torch.randn((len(counts), V), generator=g, device=DEV).mul_(2).to(dtype)
    return logits, words.to(DEV), torch.rand(len(counts), generator=g, device=DEV)


def sample_bits(case, fixed):
    B = case[0].shape[0]
    ids = torch.full((B,), -7, dtype=torch.int32, device=DEV)
    lzv, lza = torch.full((B,), 3.0, device=DEV), torch.full((B,), 3.0, device=DEV)
    (ppv.constrained_sample_noalloc if fixed else ppv.constrained_sample)(*case, ids, lzv, lza)
    torch.cuda.synchronize()
    return torch.stack([ids, lzv.view(torch.int32), lza.view(torch.int32)], 1).cpu()


def cursor_step_bits(index, P, state, logits, un):
    """One step of every row from the given cursors; the buffers that it changes are the caller's copies."""
    B = P.shape[0]
    P, state = P.clone(), state.clone()
    lens, act = torch.ones(B, dtype=torch.int32, device=DEV), torch.ones(B, dtype=torch.uint8, device=DEV)
    ids = torch.full((B,), -7, dtype=torch.int32, device=DEV)
    lz, logx = torch.full((B,), 3.0, device=DEV), torch.zeros(B, device=DEV)
    ppv.ppv_decode_step(index, P, lens, act, logits, un, ids, lz, logx, state=state)
    torch.cuda.synchronize()
    return torch.cat([t.view(torch.int32).reshape(B, -1) for t in (P, lens, ids, lz, logx, state)], 1).cpu()


def cursor_case(dtype, V=100_000, B=12):
    """Rows one token into S: a few children each, then one."""
    rng = np.random.default_rng(5)
    S = np.concatenate([rng.integers(0, 40, (400, 1)), rng.integers(0, V, (400, 3))], axis=1).astype(np.int32)
    index = ppv.ppv_build_index(S.reshape(-1), np.arange(401, dtype=np.int64) * 4, V)
    P = torch.zeros((B, 4), dtype=torch.int32, device=DEV)
    P[:, 0] = to_dev(S[rng.integers(0, 400, B), 0])
    state = torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
    lens, act = torch.ones(B, dtype=torch.int32, device=DEV), torch.ones(B, dtype=torch.uint8, device=DEV)
    ppv.ppv_decode_begin(index, P, lens, state, act)
    g = torch.Generator(device=DEV).manual_seed(9)
    logits = torch.randn((B, V), generator=g, device=DEV).mul_(2).to(dtype)
    return index, P, state, logits, torch.rand(B, generator=g, device=DEV)


@pytest.mark.parametrize("kind", ["sample", "fixed", "cursor"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_no_word_of_another_call_is_taken(dtype, kind):
    """Whatever an area holds, and whichever workgroup its counts make the last of a row: a call's results are the unsplit call's bits.
    And calls in an area that is as it should be, with rows of every kind, leave it so: nothing of theirs in it, which is what a graph's
    replays start from."""
    fixed = kind == "fixed"
    case = cursor_case(dtype) if kind == "cursor" else sample_case(dtype, 1)
    run = (lambda: cursor_step_bits(*case)) if kind == "cursor" else (lambda: sample_bits(case, fixed))
    with tuning(ppv.PPV_TUNE_ROW_SPLIT, 1):
        want = run()
    area, B = Area(fixed), want.shape[0]
    for k in SPLITS[1:]:
        with tuning(ppv.PPV_TUNE_ROW_SPLIT, k):
            for arrived in (k - 1, 1, 16, 100, k - 1):
                area.disturb(B, arrived)
                for _ in range(3):
                    assert torch.equal(run(), want), (k, arrived)
            area.arrived[:] = 0
            area.words[:] = 0
            for _ in range(3):
                assert torch.equal(run(), want), k
                assert not area.arrived.any() and not area.words.any(), k


@pytest.mark.parametrize("fixed", [False, True])
def test_a_row_whose_words_do_not_arrive_says_so(fixed):
    """With no further look at a word that is not there yet, rows finished by the first workgroup to arrive are those of the unsplit
    call or have id -1 and masses that are NaN; the calls after that are as ever, whatever is left in the area."""
    case = sample_case(torch.bfloat16, 2)
    with tuning(ppv.PPV_TUNE_ROW_SPLIT, 1):
        want = sample_bits(case, fixed)
    area, B, said = Area(fixed), want.shape[0], 0
    for k in SPLITS[1:]:
        with tuning(ppv.PPV_TUNE_ROW_SPLIT, k):
            area.disturb(B, k - 1)
            area.look_again(False)
            try:
                got = sample_bits(case, fixed)
            finally:
                area.look_again(True)
            masses = got[:, 1:].contiguous().view(torch.float32)
            none = (got[:, 0] == -1) & masses.isnan().all(1)
            assert (none | (got == want).all(1)).all(), k
            said += int(none.sum())
            for _ in range(3):
                assert torch.equal(sample_bits(case, fixed), want), k
            area.arrived[:] = 0
            area.words[:] = 0
    assert said > 0


@pytest.mark.parametrize("use_state", [True, False])
def test_split_rows_in_the_decode_step(use_state):
    """The fused decode step with its rows split: the whole loop, every split, bit for bit the unsplit loop."""
    cfg, S, trie, index = setup_case("C3s")
    B, L = 48, index.l_max
    logits = torch.stack([logits_to_dev(cfg, W.make_logits(cfg, batch=B, step=300 + s)) for s in range(L)])
    un = torch.stack([to_dev(W.make_uniforms(cfg, batch=B, step=300 + s)) for s in range(L)])
    base = None
    for k in SPLITS:
        P = torch.full((B, L), W.PAD_TOKEN, dtype=torch.int32, device=DEV)
        lens = torch.zeros(B, dtype=torch.int32, device=DEV)
        act = torch.ones(B, dtype=torch.uint8, device=DEV)
        state = None
        logx = torch.zeros(B, dtype=torch.float32, device=DEV)
        if use_state:
            state = torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV)
            ppv.ppv_decode_begin(index, P, lens, state, act, logx)
        ids = torch.full((L, B), -5, dtype=torch.int32, device=DEV)
        lz = torch.full((L, B), 2.0, dtype=torch.float32, device=DEV)
        with tuning(ppv.PPV_TUNE_ROW_SPLIT, k):
            for s in range(L):
                ppv.ppv_decode_step(index, P, lens, act, logits[s], un[s], ids[s], lz[s], logx, state=state)
        torch.cuda.synchronize()
        got = [t.cpu().numpy() for t in (P, lens, act, ids, lz.view(torch.int32), logx.view(torch.int32))]
        if base is None:
            base = got
            assert not got[2].any() and (got[1] > 0).all()
            q = trie.query(got[0], got[1], want_mask=False)
            assert (q.member == 1).all()                       # every row ended on a member of S
            continue
        for a, b in zip(got, base):
            assert np.array_equal(a, b), k


@pytest.mark.parametrize("V,dtype", [(20_000, torch.float32), (50_001, torch.bfloat16)])
def test_split_rows_in_the_first_step(V, dtype):
    """Rows that start from the empty candidate, under the root's image or its list, in every split: bit for bit the
    unsplit step, whatever the buffers held."""
    rng = np.random.default_rng(V)
    g = torch.Generator(device=DEV).manual_seed(V)
    B, L = 9, 3
    logits = torch.randn((B, -(-V // 8) * 8), generator=g, device=DEV).mul_(2).to(dtype)[:, :V]
    un = torch.rand(B, generator=g, device=DEV)
    for n, firsts in ((4_000, V), (300, 20)):                      # an image, a list
        S = rng.integers(0, V, (n, L)).astype(np.int32)
        S[:, 0] = rng.integers(0, firsts, n)
        index = ppv.ppv_build_index(S.reshape(-1), np.arange(n + 1, dtype=np.int64) * L, V)
        base = None
        for k in SPLITS:
            P = torch.full((B, L), W.PAD_TOKEN, dtype=torch.int32, device=DEV)
            lens, act = torch.full((B,), 77, dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.uint8, device=DEV)
            state = torch.full((B, ppv.PPV_STATE_WORDS), -3, dtype=torch.int32, device=DEV)
            logx, lz = torch.full((B,), 5.0, device=DEV), torch.full((B,), 5.0, device=DEV)
            ids = torch.full((B,), -5, dtype=torch.int32, device=DEV)
            with tuning(ppv.PPV_TUNE_ROW_SPLIT, k):
                ppv.ppv_decode_first_step(index, P, lens, act, logits, un, ids, lz, logx, state=state)
            torch.cuda.synchronize()
            got = [t.cpu().numpy() for t in (P, lens, act, ids, lz, logx, state[:, :4].contiguous())]
            base = base or got
            assert (got[3] >= 0).all()
            for a, b in zip(got, base):
                assert np.array_equal(a, b), k


def test_split_rows_under_graph_capture():
    """A stream that is being captured cannot allocate its scratch area: without one the rows are simply not
    split; with one (the stream made a call before the capture) they are.  Replays equal the eager result."""
    cfg, S, trie, index = setup_case("C2")
    pb = W.make_prefix_batch(cfg, S)
    logits = logits_to_dev(cfg, W.make_logits(cfg))
    un = to_dev(W.make_uniforms(cfg))
    ref = trie.query(pb.prefixes, pb.lens)
    words = to_dev(pack(ref.mask))
    B = logits.shape[0]
    ids = torch.full((B,), -7, dtype=torch.int32, device=DEV)
    lzv = torch.zeros(B, dtype=torch.float32, device=DEV)
    ppv.constrained_sample(logits, words, un, ids, lzv)
    torch.cuda.synchronize()
    want = (ids.cpu().numpy().copy(), lzv.cpu().numpy().copy())
    for warm in (False, True):
        side = torch.cuda.Stream()
        if warm:
            with torch.cuda.stream(side):
                ppv.constrained_sample(logits, words, un, ids, lzv)
            side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ppv.constrained_sample(logits, words, un, ids, lzv)
        for _ in range(3):
            ids.fill_(-9)
            lzv.fill_(7.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(ids.cpu().numpy(), want[0])
            assert np.array_equal(lzv.cpu().numpy().view(np.int32), want[1].view(np.int32))


def first_step_buffers(B, L):
    return [torch.full((B, L), 7, dtype=torch.int32, device=DEV), torch.full((B,), 77, dtype=torch.int32, device=DEV),
            torch.zeros(B, dtype=torch.uint8, device=DEV), torch.full((B,), -5, dtype=torch.int32, device=DEV),
            torch.full((B,), 5.0, device=DEV), torch.full((B,), 5.0, device=DEV),
            torch.full((B, ppv.PPV_STATE_WORDS), -3, dtype=torch.int32, device=DEV)]


def first_step_setup(V, B, L, seeds):
    rng = np.random.default_rng(V)
    S = rng.integers(0, V, (4_000, L)).astype(np.int32)
    index = ppv.ppv_build_index(S.reshape(-1), np.arange(4_001, dtype=np.int64) * L, V)
    inputs = []
    for seed in seeds:
        g = torch.Generator(device=DEV).manual_seed(seed)
        inputs.append((torch.randn((B, V), generator=g, device=DEV).mul_(2), torch.rand(B, generator=g, device=DEV)))
    return index, inputs


def first_step(index, x, u, bufs, stream=None):
    P, lens, act, ids, lz, lx, state = bufs
    ppv.ppv_decode_first_step(index, P, lens, act, x, u, ids, lz, lx, state=state, stream=stream)


def split_call(name, index, x, u, bufs, words):
    """One call of each kind that splits rows, from the empty prefixes; repeatable."""
    P, lens, act, ids, lz, lx, state = bufs
    if name == "first":
        first_step(index, x, u, bufs)
    elif name == "sample":
        ppv.constrained_sample(x, words, u, ids, lz)
    else:
        lens.zero_()
        act.fill_(1)
        if name == "next":
            ppv.ppv_sample_next(index, P, lens, x, u, ids, lz)
        else:
            ppv.ppv_decode_step(index, P, lens, act, x, u, ids, lz)


@pytest.mark.parametrize("name", ["first", "step", "sample", "next"])
def test_graphs_side_by_side(name):
    """Graphs captured one after the other on one stream (more of them than areas lie ready), replayed on streams of their own
    at the same time, eager calls on the capture's stream beside them: each gives what it gives alone."""
    V, B, L, N = 64_000, 6, 3, 7
    index, inputs = first_step_setup(V, B, L, range(N + 1))
    words = torch.zeros((B, index.n_words), dtype=torch.int32, device=DEV)
    ppv.ppv_next_token_mask(index, torch.zeros((B, L), dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.int32, device=DEV), words)
    want = []
    for x, u in inputs:
        bufs = first_step_buffers(B, L)
        split_call(name, index, x, u, bufs, words)
        want.append([t.clone() for t in bufs[:6]])
    side = torch.cuda.Stream()
    got = [first_step_buffers(B, L) for _ in inputs]
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        split_call(name, index, *inputs[N], got[N], words)     # the stream has an area, captures to come have theirs
    torch.cuda.synchronize()
    graphs, streams = [], [torch.cuda.Stream() for _ in range(N)]
    for (x, u), bufs in zip(inputs[:N], got):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=side):
            for _ in range(10):
                split_call(name, index, x, u, bufs, words)
    for _ in range(5):
        for bufs in got:
            bufs[3].fill_(-9)
            bufs[4].fill_(9.0)
        torch.cuda.synchronize()
        for graph, stream in zip(graphs, streams):
            with torch.cuda.stream(stream):
                graph.replay()
        with torch.cuda.stream(side):
            for _ in range(10):
                split_call(name, index, *inputs[N], got[N], words)
        torch.cuda.synchronize()
        for k, (bufs, ref) in enumerate(zip(got, want)):
            for a, b in zip(bufs, ref):
                assert torch.equal(a, b), k


def test_more_rows_than_an_area_of_a_capture_has():
    """(128; only a forced split has more.)"""
    V, B, L = 20_000, 129, 3
    index, inputs = first_step_setup(V, B, L, (1,))
    want, got = first_step_buffers(B, L), first_step_buffers(B, L)
    with tuning(ppv.PPV_TUNE_ROW_SPLIT, 2):
        first_step(index, *inputs[0], want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            first_step(index, *inputs[0], got)
        graph.replay()
        torch.cuda.synchronize()
    for a, b in zip(got[:6], want):
        assert torch.equal(a, b)


def test_threads_with_the_per_thread_stream():
    """hipStreamPerThread is one handle for a stream in each thread: split rows of several threads do not meet."""
    import threading
    import types
    per_thread = types.SimpleNamespace(cuda_stream=2)     # the handle's value
    V, B, L, N = 64_000, 6, 3, 4
    index, inputs = first_step_setup(V, B, L, range(N))
    want = []
    for x, u in inputs:
        bufs = first_step_buffers(B, L)
        first_step(index, x, u, bufs)
        want.append(bufs)
    got = [first_step_buffers(B, L) for _ in inputs]
    torch.cuda.synchronize()
    failed = []

    def work(k):
        try:
            for _ in range(200):
                first_step(index, *inputs[k], got[k], stream=per_thread)
            torch.cuda.synchronize()                      # (the thread's stream ends with the thread)
        except Exception as e:                            # (an assertion in a thread would go unseen)
            failed.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(N)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed
    for bufs, ref in zip(got, want):
        for a, b in zip(bufs[:6], ref[:6]):
            assert torch.equal(a, b)
