"""What the Python calls accept and refuse: the shapes of `prefixes`, which the decoding calls take with further dimensions."""
import numpy as np
import pytest
import torch

from paper_2504_09135_amd import binding as ppv

from gpu_helpers import DEV, to_dev

pytestmark = pytest.mark.gpu

V, B, L = 500, 9, 6


def make_state(shape):
    return {"prefixes": torch.zeros(shape, dtype=torch.int32, device=DEV), "lens": torch.zeros(B, dtype=torch.int32, device=DEV),
            "state": torch.zeros((B, ppv.PPV_STATE_WORDS), dtype=torch.int32, device=DEV),
            "active": torch.ones(B, dtype=torch.uint8, device=DEV), "logx": torch.zeros(B, device=DEV)}


def decode(index, shape, how, logits, uniforms):
    s = make_state(shape)
    if how == "loop":
        ppv.ppv_decode_begin(index, s["prefixes"], s["lens"], s["state"], s["active"], s["logx"])
        ppv.ppv_decode_loop(index, s["prefixes"], s["lens"], s["active"], logits, uniforms, logx=s["logx"], state=s["state"])
    else:
        for k in range(len(logits)):
            if k == 0 and how == "first":
                ppv.ppv_decode_first_step(index, s["prefixes"], s["lens"], s["active"], logits[0], uniforms[0], logx=s["logx"],
                                          state=s["state"])
                continue
            if k == 0:
                ppv.ppv_decode_begin(index, s["prefixes"], s["lens"], s["state"], s["active"], s["logx"])
            ppv.ppv_decode_step(index, s["prefixes"], s["lens"], s["active"], logits[k], uniforms[k], logx=s["logx"], state=s["state"])
    return {k: v.cpu().reshape(B, -1).numpy() for k, v in s.items()}


@pytest.mark.parametrize("how", ["loop", "steps", "first"])
def test_prefixes_with_a_further_dimension(how):
    rng = np.random.default_rng(4)
    index = ppv.ppv_build_index(rng.integers(0, V, 200 * L, dtype=np.int32), np.arange(201, dtype=np.int64) * L, V)
    logits, uniforms = to_dev(rng.normal(0, 2, (L, B, V)).astype(np.float32)), to_dev(rng.random((L, B), dtype=np.float32))
    want = decode(index, (B, L), how, logits, uniforms)
    assert (want["lens"] == L).all()
    got = decode(index, (B, L, 1), how, logits, uniforms)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    s = make_state((B,))
    for call in (lambda: ppv.ppv_decode_begin(index, s["prefixes"], s["lens"], s["state"], s["active"]),
                 lambda: ppv.ppv_decode_step(index, s["prefixes"], s["lens"], s["active"], logits[0], uniforms[0]),
                 lambda: ppv.ppv_decode_loop(index, s["prefixes"], s["lens"], s["active"], logits, uniforms),
                 lambda: ppv.ppv_decode_begin_empty(index, s["lens"][0], s["state"], s["active"])):
        with pytest.raises(IndexError):
            call()
    mask = torch.zeros((B, index.n_words), dtype=torch.int32, device=DEV)
    for shape in ((B,), (B, L, 1)):
        with pytest.raises(ValueError):
            ppv.ppv_next_token_mask(index, torch.zeros(shape, dtype=torch.int32, device=DEV), s["lens"], mask)
    index.free()
