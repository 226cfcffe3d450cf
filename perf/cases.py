"""What this library is asked to do in use, as cases that can be timed and compared.

Every case goes through the public calls of paper_2504_09135_amd.binding, with the index, the buffers and (for the
replayed loop) the captured graph that a serving program holds on to.  `path` says which calls a pass makes:

  decode   the decoding loop of Algorithm 1 as README.md shows it, one call per decode step, launched eagerly
  replay   the same loop captured once in a HIP graph and replayed, as bench.py times it
  loop     the whole loop as one ppv_decode_loop call: distributions that are known up front (scoring, replay)
  disc     one round of DISC: 2K candidates per query through the decoding loop, then ppv_disc_select
  fused    ppv_sample_next: the next token of given prefixes
  pair     ppv_next_token_mask, then constrained_sample on its mask
  topm     ppv_topm_mask (Algorithm 2 with M candidates), then constrained_sample on its mask
  build    ppv_build_index from S in host memory, and the first mask call on the new index

Constraint sets, prefixes and logits are drawn as in paper_2504_09135_amd/workloads.py (Zipf tokens, or one codebook
per position; normal logits with sigma 2), but on the GPU, so that they are there in a fraction of a second.
"""
import math

import numpy as np
import torch

from paper_2504_09135_amd import binding as ppv

DEVICE = "cuda:0"
PAD_TOKEN = 0x7FFFFFF0      # fills prefix slots past a row's length; never a real token
SIGMA = 2.0
LOOPS = ("decode", "replay", "loop", "disc")
LOOP_BYTES = 4.2e9          # logits of all steps of a decoding loop, resident up front: at most this much
LOOP_READ_BYTES = 2.3e9     # ... and what the rows read of them before they are members of S
CALL_BYTES = 5.2e8          # logits of one single-step call


def new_case(path, n_seq, vocab, batch, dtype, len_lo, len_hi, tokens="zipf", **more):
    c = {"path": path, "n_seq": n_seq, "vocab": vocab, "batch": batch, "dtype": dtype, "len_lo": len_lo, "len_hi": len_hi,
         "tokens": tokens, "valid": 1.0, "temperature": 1.0, "M": 0, "lists": False, "K": 0}
    c.update(more)
    return c


def listed():
    return [
        # one interactive request, the vocabulary of the paper's larger model: latency alone
        dict(new_case("decode", 100_000, 128_256, 1, "bf16", 4, 16), name="decode B=1 V=128256"),
        # a small batch over item codes (configuration C1): the smallest rows, nothing but launches
        dict(new_case("decode", 1_000, 1_024, 16, "f32", 8, 8, "codes"), name="decode B=16 codes"),
        # the repository's headline loop (configuration C3), replayed from a graph as bench.py does
        dict(new_case("replay", 1_000_000, 32_000, 256, "bf16", 4, 32), name="replay B=256 V=32000"),
        # the same set under a large batch of candidates: throughput
        dict(new_case("decode", 1_000_000, 32_000, 2_048, "bf16", 4, 32), name="decode B=2048 V=32000"),
        # a fixed proposal scored in one launch: fp32 logits, the vocabulary of the paper's smaller model
        dict(new_case("loop", 300_000, 50_264, 384, "f32", 2, 12), name="loop B=384 V=50264 f32"),
        # DISC over a batch of queries, K = 4: 8 candidates each, then the selection
        dict(new_case("disc", 300_000, 50_264, 1_024, "bf16", 2, 16, K=4), name="disc Q=128 K=4"),
        # next tokens of a mixed batch of prefixes, some of them outside S (configuration C2)
        dict(new_case("fused", 100_000, 32_000, 64, "bf16", 2, 16, valid=0.9), name="fused B=64 V=32000"),
        # generative recommendation over four codebooks, a large batch (configuration C4)
        dict(new_case("pair", 3_000_000, 1_024, 4_096, "f32", 4, 4, "codes"), name="pair B=4096 codes"),
        # the paper's batch with an odd vocabulary (padded rows), fp32 logits and a temperature
        dict(new_case("pair", 1_000_000, 50_265, 128, "f32", 2, 16, valid=0.95, temperature=0.7), name="pair B=128 V=50265 f32"),
        # the largest vocabulary and batch (configuration C5)
        dict(new_case("pair", 1_000_000, 256_000, 1_024, "bf16", 2, 24, valid=0.95), name="pair B=1024 V=256000"),
        # Algorithm 2 as the paper ran it: M = 50, batch 128, then a token sampled from what is left
        dict(new_case("topm", 1_000_000, 128_256, 128, "bf16", 2, 16, valid=0.95, M=50), name="topm M=50 B=128 V=128256"),
        # a new constraint set arrives: the index, and the first batch that asks it
        dict(new_case("build", 1_000_000, 32_000, 256, "bf16", 4, 32), name="build 1M"),
    ]


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["decode", "replay", "loop", "disc", "fused", "pair", "topm", "build"])
    dtype = rng.choice(["f32", "bf16"])
    e = 4 if dtype == "f32" else 2
    codes = path != "build" and rng.random() < 0.2
    len_lo = rng.randint(1, 4)
    len_hi = rng.randint(max(4, len_lo + 1), 32)
    c = new_case(path, log_int(rng, 1_000, 1_000_000), log_int(rng, 8_000, 256_000), 0, dtype, len_lo, len_hi)
    if codes:
        len_hi = rng.randint(3, 8)
        c.update(tokens="codes", len_lo=len_hi, len_hi=len_hi, vocab=log_int(rng, 512, 8_192))
    row = c["vocab"] * e
    if path in LOOPS:
        mean_len = (c["len_lo"] + c["len_hi"]) / 2
        most = max(1, min(2_048, int(LOOP_BYTES / (row * c["len_hi"])), int(LOOP_READ_BYTES / (row * mean_len))))
        c["batch"] = log_int(rng, 1, most)
        if path == "disc":
            c["K"] = rng.randint(1, 5)
            c["batch"] = 2 * c["K"] * max(1, c["batch"] // (2 * c["K"]))     # 2K candidates per query
    else:
        c["batch"] = log_int(rng, 1, max(1, min(4_096, int(CALL_BYTES / row))))
        c["valid"] = rng.choice([1.0, 0.95, 0.8])
    if path == "topm":
        c["M"] = log_int(rng, 20, min(1_000, c["vocab"] // 4))
        c["lists"] = rng.random() < 0.5
    if path != "build" and rng.random() < 0.3:
        c["temperature"] = round(rng.uniform(0.5, 2.0), 2)
    return c


# ------------------------------------------------------------------------------------------ inputs
def constraint_set(c, g):
    """S as a padded matrix on the GPU with its lengths."""
    n, V, L = c["n_seq"], c["vocab"], c["len_hi"]
    lens = torch.randint(c["len_lo"], L + 1, (n,), generator=g, device=DEVICE)
    if c["tokens"] == "codes":      # position l has the tokens of codebook l
        per = V // L
        tok = torch.randint(0, per, (n, L), generator=g, device=DEVICE, dtype=torch.int32)
        tok += torch.arange(L, device=DEVICE, dtype=torch.int32) * per
    else:
        cdf = torch.arange(1, V + 1, device=DEVICE, dtype=torch.float64).pow(-1.1).cumsum(0)
        cdf /= cdf[-1].clone()
        u = torch.rand((n, L), generator=g, device=DEVICE, dtype=torch.float64)
        tok = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1).to(torch.int32)
    return tok, lens


def host_csr(tok, lens):
    inside = torch.arange(tok.shape[1], device=DEVICE)[None, :] < lens[:, None]
    offsets = np.zeros(tok.shape[0] + 1, dtype=np.int64)
    np.cumsum(lens.cpu().numpy(), out=offsets[1:])
    return tok[inside].cpu().numpy(), offsets


def prefix_batch(c, g, tok, lens):
    """Prefixes of random members, 0 .. length - 1 tokens long; a share 1 - valid of them with the last token replaced."""
    B, L, V = c["batch"], c["len_hi"], c["vocab"]
    who = torch.randint(0, tok.shape[0], (B,), generator=g, device=DEVICE)
    k = (torch.rand(B, generator=g, device=DEVICE, dtype=torch.float64) * lens[who]).to(torch.int64)
    bad = torch.rand(B, generator=g, device=DEVICE) >= c["valid"]
    k = torch.where(bad, k.clamp(min=1), k)
    rows = tok[who].clone()
    at = torch.arange(L, device=DEVICE)[None, :]
    other = torch.randint(0, V, (B,), generator=g, device=DEVICE, dtype=torch.int32)
    rows = torch.where(bad[:, None] & (at == k[:, None] - 1), other[:, None], rows)
    rows.masked_fill_(at >= k[:, None], PAD_TOKEN)
    return rows.contiguous(), k.to(torch.int32)


def random_logits(c, g, shape):
    """Normal logits; rows start on 16-byte boundaries (an odd vocabulary is padded, as a model's output buffer is)."""
    bf16 = c["dtype"] == "bf16"
    V = c["vocab"]
    per = 8 if bf16 else 4
    padded = -(-V // per) * per
    out = torch.empty(shape + (padded,), dtype=torch.bfloat16 if bf16 else torch.float32, device=DEVICE)
    for step in out.view(-1, shape[-1], padded):
        step.copy_(torch.randn(step.shape, generator=g, device=DEVICE).mul_(SIGMA))
    return out[..., :V]


def prepare(case, seed):
    c = dict(case)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    B, L = c["batch"], c["len_hi"]
    tok, lens = constraint_set(c, g)
    tokens, offsets = host_csr(tok, lens)
    st = {"case": c, "tokens": tokens, "offsets": offsets}

    def zeros(*shape, dtype=torch.int32):
        return torch.zeros(shape, dtype=dtype, device=DEVICE)

    if c["path"] not in LOOPS:
        st["prefixes"], st["lens"] = prefix_batch(c, g, tok, lens)
        st["mask"] = zeros(B, (c["vocab"] + 31) // 32)
        st["lo"], st["hi"], st["member"] = zeros(B), zeros(B), zeros(B, dtype=torch.uint8)
    del tok, lens
    if c["path"] == "build":
        return st
    st["index"] = ppv.ppv_build_index(tokens, offsets, c["vocab"])
    del st["tokens"], st["offsets"]
    st["ids"], st["logZ"], st["logZ_all"] = zeros(B), zeros(B, dtype=torch.float32), zeros(B, dtype=torch.float32)
    if c["path"] not in LOOPS:
        st["logits"] = random_logits(c, g, (B,))
        st["uniforms"] = torch.rand(B, generator=g, device=DEVICE)
        if c["lists"]:
            st["top_ids"], st["mask_V"] = zeros(B, c["M"]), zeros(B, c["M"], dtype=torch.uint8)
        return st
    st["all_logits"] = random_logits(c, g, (L, B))
    st["all_uniforms"] = torch.rand((L, B), generator=g, device=DEVICE)
    st["logits"], st["uniforms"] = list(st["all_logits"]), list(st["all_uniforms"])
    st["prefixes"] = torch.full((B, L), PAD_TOKEN, dtype=torch.int32, device=DEVICE)
    st["lens"], st["state"] = zeros(B), zeros(B, ppv.PPV_STATE_WORDS)
    st["active"], st["logx"] = zeros(B, dtype=torch.uint8), zeros(B, dtype=torch.float32)
    if c["path"] == "disc":
        Q = B // (2 * c["K"])
        st["accept_u"] = torch.rand((c["K"], Q), generator=g, device=DEVICE)
        st["resample_u"] = torch.rand(Q, generator=g, device=DEVICE)
        st["chosen"], st["n_draws"], st["accepted"] = zeros(Q), zeros(Q), zeros(Q, dtype=torch.uint8)
    if c["path"] == "replay":       # captured on a stream that has run the loop once
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            decode(st)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"], stream=side):
            decode(st)
    return st


# ------------------------------------------------------------------------------------------ passes
def decode(st):
    """Every row from the empty candidate to a member of S."""
    T = st["case"]["temperature"]
    step = ppv.ppv_decode_first_step
    for logits, u in zip(st["logits"], st["uniforms"]):
        step(st["index"], st["prefixes"], st["lens"], st["active"], logits, u, st["ids"], st["logZ"], st["logx"],
             state=st["state"], temperature=T)
        step = ppv.ppv_decode_step


def run(st):
    c = st["case"]
    path = c["path"]
    if path == "build":
        index = ppv.ppv_build_index(st["tokens"], st["offsets"], c["vocab"])
        ppv.ppv_next_token_mask(index, st["prefixes"], st["lens"], st["mask"], st["lo"], st["hi"], st["member"])
        sizes = (index.n_distinct, index.l_max, index.n_prefixes)
        index.free()
        return [st["mask"], st["lo"], st["hi"], st["member"], *sizes]
    index, T = st["index"], c["temperature"]
    if path in LOOPS:
        if path == "replay":
            st["graph"].replay()
        elif path == "loop":
            ppv.ppv_decode_begin_empty(index, st["lens"], st["state"], st["active"], st["logx"])
            ppv.ppv_decode_loop(index, st["prefixes"], st["lens"], st["active"], st["all_logits"], st["all_uniforms"], None,
                                None, st["logx"], state=st["state"], temperature=T)
        else:
            decode(st)
        out = [st["prefixes"], st["lens"], st["active"], st["logx"]]
        if path == "disc":
            ppv.ppv_disc_select(st["logx"].view(2 * c["K"], -1), c["K"], st["accept_u"], st["resample_u"], st["chosen"],
                                st["n_draws"], st["accepted"])
            out += [st["chosen"], st["n_draws"], st["accepted"]]
        return out
    if path == "fused":
        ppv.ppv_sample_next(index, st["prefixes"], st["lens"], st["logits"], st["uniforms"], st["ids"], st["logZ"],
                            temperature=T)
        return [st["ids"], st["logZ"]]
    out = [st["mask"], st["ids"], st["logZ"], st["logZ_all"]]
    if path == "pair":
        ppv.ppv_next_token_mask(index, st["prefixes"], st["lens"], st["mask"], st["lo"], st["hi"], st["member"])
        out += [st["lo"], st["hi"], st["member"]]
    else:
        ppv.ppv_topm_mask(index, st["prefixes"], st["lens"], st["logits"], c["M"], st["mask"], st.get("top_ids"),
                          st.get("mask_V"))
        if c["lists"]:
            out += [st["top_ids"], st["mask_V"]]
    ppv.constrained_sample(st["logits"], st["mask"], st["uniforms"], st["ids"], st["logZ"], st["logZ_all"], temperature=T)
    return out


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    row = c["vocab"] * (4 if c["dtype"] == "f32" else 2)
    mask = (c["vocab"] + 31) // 32 * 4
    mean_len = (c["len_lo"] + c["len_hi"]) / 2
    if c["path"] == "build":        # S read; S sorted, and 16 bytes for every prefix, written (nearly every token opens one)
        tokens = c["n_seq"] * mean_len
        return {"bytes": 4 * tokens + 8 * c["n_seq"] + 20 * tokens + c["batch"] * mask, "flops": 0}
    if c["path"] in LOOPS:          # a row reads logits until it is a member of S
        rows = c["batch"] * mean_len
        return {"bytes": rows * (row + 96), "flops": 4 * rows * c["vocab"]}
    rows = c["batch"]
    per_row = row + 96
    if c["path"] != "fused":
        per_row += mask
    if c["lists"]:
        per_row += 5 * c["M"]
    return {"bytes": rows * per_row, "flops": 4 * rows * c["vocab"]}


def tolerance(case):
    if case["path"] == "build":
        return "exact"
    # sums of fp32 exponentials; a uniform on the very edge between two tokens may fall on either side
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
