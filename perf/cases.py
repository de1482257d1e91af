"""Performance cases of the batched speculative verify step and its stages.

Each case is one call (or the call pair of one decoding step) that a serving
loop makes through the public entry points, on inputs made from a seed: whole
steps, a position of the draft chain, and the single stages with the sizes they
have inside steps of the shapes in ``paper_2512_22420_amd/workload.py``.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2512_22420_amd import binding as nb
from paper_2512_22420_amd import workload as W
from paper_2512_22420_amd.device import DeviceCache, DeviceModel, StepIO, Workspace, kv_append, model_desc, pack_weight, verify

LAYER_8B = "llama3-8b-layer"
LAYER_7B = "qwen2.5-7b-layer"
DRAFT_1B = "llama-1b-draft"
TINY = "tiny-f32"
SHAPES = {LAYER_8B: W.LLAMA8B_LAYER, LAYER_7B: dataclasses.replace(W.QWEN7B, name=LAYER_7B, n_layers=1),
          DRAFT_1B: W.LLAMA1B_DRAFT, TINY: W.TINY_F32}
POOLS = {LAYER_8B: W.LLAMA8B, LAYER_7B: W.QWEN7B}  # the whole stacks, for the pool migration


# --------------------------------------------------------------------------
# The cases
# --------------------------------------------------------------------------
def listed():
    return [
        # The smallest step: the fp32 model used to check a deployment (two
        # sequences, three drafts).  Launches and latency are all there is.
        {"name": "step_tiny_f32_b2_k3", "op": "step", "shape": TINY, "B": 2, "k": 3, "ctx": 40, "spread": 0.2},
        # The headline point of the benchmark: a small batch with five drafts
        # per sequence, bound by the weight stream.
        {"name": "step_8b_b8_k5", "op": "step", "shape": LAYER_8B, "B": 8, "k": 5, "ctx": 1024, "spread": 0.0},
        # A large batch of a size that requests come and go in (305 window
        # rows, mixed contexts): weights and matrix work about equally long.
        {"name": "step_8b_b61_k4", "op": "step", "shape": LAYER_8B, "B": 61, "k": 4, "ctx": 768, "spread": 0.5},
        # One position of the draft chain (a decode step of the 16-layer draft
        # with its KV append), run k+1 times per speculative step.
        {"name": "draft_1b_b8", "op": "draft", "shape": DRAFT_1B, "B": 8, "ctx": 1024, "spread": 0.0},
        # A layer's attention inputs (norm, QKV projection, RoPE, window K/V)
        # for a small window.
        {"name": "qkv_8b_b4_k3", "op": "qkv", "shape": LAYER_8B, "B": 4, "k": 3, "ctx": 1024, "spread": 0.5},
        # Verify attention of a layer at the large-batch grid's contexts.
        {"name": "attn_8b_b64_k4", "op": "attn", "shape": LAYER_8B, "B": 64, "k": 4, "ctx": 768, "spread": 0.5},
        # Verify attention with many long contexts and eight window rows (the
        # largest read of the cache; 56 query rows per KV head).
        {"name": "attn_7b_b256_k7", "op": "attn", "shape": LAYER_7B, "B": 256, "k": 7, "ctx": 2400, "spread": 0.35},
        # The down projection with its residual for a ragged small window (13 sequences, two drafts).
        {"name": "down_8b_m39", "op": "gemm", "shape": LAYER_8B, "gemm": "down", "M": 39},
        # The gate/up projection with its SwiGLU at a middle window (32
        # sequences, four drafts), between weight-bound and matrix-bound.
        {"name": "gate_up_8b_m160", "op": "gemm", "shape": LAYER_8B, "gemm": "gate_up", "M": 160},
        # The largest window of the 7B stack (256 sequences, seven drafts): matrix-bound.
        {"name": "gate_up_7b_m2048", "op": "gemm", "shape": LAYER_7B, "gemm": "gate_up", "M": 2048},
        # The acceptance test alone, from given logits of a middle batch.
        {"name": "accept_8b_b64_k4", "op": "accept", "shape": LAYER_8B, "B": 64, "k": 4},
        # The pool contraction of the 32-layer stack: its blocks above the
        # boundary move below it (the paper's 292 blocks).
        {"name": "migrate_8b_292", "op": "migrate", "shape": LAYER_8B, "moves": 292},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49))))))


def draw(rng):
    op = rng.choice(["step", "step", "tiny", "draft", "qkv", "attn", "attn", "gemm", "gemm", "gemm", "accept", "migrate"])
    shape = rng.choice([LAYER_8B, LAYER_7B])
    k = rng.randint(0, 7)
    spread = rng.choice([0.0, 0.3, 0.5])
    if op == "tiny":
        return {"op": "step", "shape": TINY, "B": rng.randint(1, 8), "k": k, "ctx": _log_int(rng, 8, 400), "spread": spread}
    if op == "step":
        return {"op": "step", "shape": LAYER_8B, "B": _log_int(rng, 1, 320 // (k + 1)), "k": k,
                "ctx": _log_int(rng, 128, 1024), "spread": spread}
    if op == "draft":
        return {"op": "draft", "shape": DRAFT_1B, "B": _log_int(rng, 1, 8), "ctx": _log_int(rng, 128, 1024), "spread": spread}
    if op == "qkv":
        return {"op": "qkv", "shape": shape, "B": _log_int(rng, 1, 768 // (k + 1)), "k": k, "ctx": _log_int(rng, 128, 4096),
                "spread": spread}
    if op == "attn":
        B = _log_int(rng, 1, 256)
        return {"op": "attn", "shape": shape, "B": B, "k": k,
                "ctx": _log_int(rng, 64, min(8192, (SHAPES[LAYER_7B].n_kv_heads * 256 * 2400) // (SHAPES[shape].n_kv_heads * B))),
                "spread": spread}
    if op == "gemm":
        gemm = rng.choice(["o", "gate_up", "down", "lm_head"])
        N, K, _ = _gemm_shape(SHAPES[shape], gemm)
        top = int(min(2048, 2048 * 37888 * 3584 / (N * K)))
        return {"op": "gemm", "shape": shape, "gemm": gemm, "M": _log_int(rng, 1, top)}
    if op == "accept":
        return {"op": "accept", "shape": shape, "B": _log_int(rng, 1, 320 // (k + 1)), "k": k}
    return {"op": "migrate", "shape": shape, "moves": _log_int(rng, 8, 292)}


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _bits(gen, shape, std):
    return W.device_normal_bf16(gen, shape, std)


def _rand(gen, shape):
    return torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32)


def _ids(gen, V, shape):
    return torch.randint(0, V, shape, generator=gen, device="cuda", dtype=torch.int32)


def _f32_or_bf16(t):
    """bf16 bit patterns as bfloat16, fp32 as it is (the same memory)."""
    return t.view(torch.bfloat16) if t.dtype == torch.int16 else t


def _contexts(case, seed):
    """Context lengths: all alike at spread 0, else lognormal about the median
    (the same lengths for every seed, in another order, so that a case is the
    same work for every seed)."""
    c, B = case["ctx"], case["B"]
    if not case["spread"]:
        return np.full(B, c, np.int32)
    x = W.ctx_lengths("lognormal", B, 0, median=c, sigma=case["spread"], lo=max(1, c // 6), hi=c * 8 // 3)
    return np.random.default_rng(seed).permutation(x)


def _weights(s, gen):
    """Random weights of the shape: bf16 bits (row-major), or fp32 for the tiny model."""
    if s.dtype == "bf16":
        return W.device_weights(s, gen)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * 0.02
    ones = torch.ones(s.d_model, device="cuda", dtype=torch.float32)
    return {"embed": rnd(s.vocab, s.d_model), "lm_head": rnd(s.vocab, s.d_model), "final_norm": ones,
            "layers": [{"attn_norm": ones, "ffn_norm": ones, "w_qkv": rnd(s.qkv_dim, s.d_model),
                        "w_o": rnd(s.d_model, s.n_heads * s.head_dim), "w_gate_up": rnd(2 * s.ffn_dim, s.d_model),
                        "w_down": rnd(s.d_model, s.ffn_dim)} for _ in range(s.n_layers)]}


def _cache(s, case, seed, k, gen):
    """A paged cache with shuffled blocks and room for the window of k+1 rows;
    the pages of all layers in one tensor each for K and V."""
    ctx = _contexts(case, seed)
    table, num_blocks, max_blocks = W.make_block_table(s, ctx, k, seed=seed)
    shape_k = (s.n_layers, num_blocks, s.n_kv_heads, s.block_size, s.head_dim)
    shape_v = (s.n_layers, num_blocks, s.n_kv_heads, s.head_dim, s.block_size)
    if s.dtype == "bf16":
        kp, vp = _bits(gen, shape_k, 0.5), _bits(gen, shape_v, 0.5)
    else:
        kp = torch.randn(shape_k, generator=gen, device="cuda", dtype=torch.float32) * 0.5
        vp = torch.randn(shape_v, generator=gen, device="cuda", dtype=torch.float32) * 0.5
    cache = DeviceCache({"k_pages": list(kp), "v_pages": list(vp), "block_table": table, "context_lens": ctx,
                         "num_blocks": num_blocks})
    return cache, kp, vp, ctx


def _drafts(s, B, k, gen):
    """Last tokens, k drafts with their distributions (softmax of N(0, 2^2), the
    drafts sampled from them) and uniforms."""
    d = {"last_tokens": _ids(gen, s.vocab, (B,)), "uniforms": _rand(gen, (B, k + 1))}
    probs = torch.softmax(2.0 * torch.randn((B * k, s.vocab), generator=gen, device="cuda", dtype=torch.float32), -1)
    # argmax(log q + Gumbel noise) is a draw from q
    noise = torch.empty_like(probs).exponential_(generator=gen)
    toks = (probs / noise).argmax(-1).to(torch.int32) if k else torch.zeros(0, dtype=torch.int32, device="cuda")
    d["draft_probs"], d["draft_tokens"] = probs.view(B, k, s.vocab), toks.view(B, k)
    return d


def _gemm_shape(s, gemm):
    HD = s.n_heads * s.head_dim
    return {"o": (s.d_model, HD, nb.NJ_GEMM_RESIDUAL), "gate_up": (2 * s.ffn_dim, s.d_model, nb.NJ_GEMM_SWIGLU),
            "down": (s.d_model, s.ffn_dim, nb.NJ_GEMM_RESIDUAL), "lm_head": (s.vocab, s.d_model, nb.NJ_GEMM_STORE)}[gemm]


def _inputs(case, seed):
    """The inputs of a case before any packing: shared by prepare() and exact()."""
    gen = _gen(seed)
    s = SHAPES[case["shape"]]
    op = case["op"]
    i = {"s": s}
    if op == "step":
        i["w"] = _weights(s, gen)
        i["cache"], i["kp"], i["vp"], i["ctx"] = _cache(s, case, seed, case["k"], gen)
        i["d"] = _drafts(s, case["B"], case["k"], gen)
    elif op == "draft":
        i["w"] = _weights(s, gen)
        i["cache"], i["kp"], i["vp"], i["ctx"] = _cache(s, case, seed, 0, gen)
        i["last"], i["u"] = _ids(gen, s.vocab, (case["B"],)), _rand(gen, (case["B"],))
    elif op == "qkv":
        M = case["B"] * (case["k"] + 1)
        i["h"] = torch.randn((M, s.d_model), generator=gen, device="cuda", dtype=torch.float32)
        i["g"] = torch.ones(s.d_model, dtype=torch.bfloat16, device="cuda").view(torch.int16)
        i["w"] = _bits(gen, (s.qkv_dim, s.d_model), 0.02)
        i["ctx"] = _contexts(case, seed)
    elif op == "attn":
        B, T = case["B"], case["k"] + 1
        i["cache"], i["kp"], i["vp"], i["ctx"] = _cache(s, case, seed, case["k"], gen)
        i["q"] = _bits(gen, (B * T, s.n_heads, s.head_dim), 1.0)
        wk = torch.zeros((B, s.n_kv_heads, 16, s.head_dim), dtype=torch.int16, device="cuda")
        wv = torch.zeros((B, s.n_kv_heads, s.head_dim, 16), dtype=torch.int16, device="cuda")
        wk[:, :, :T] = _bits(gen, (B, s.n_kv_heads, T, s.head_dim), 0.5)
        wv[..., :T] = _bits(gen, (B, s.n_kv_heads, s.head_dim, T), 0.5)
        i["wk"], i["wv"] = wk, wv
    elif op == "gemm":
        N, K, epi = _gemm_shape(s, case["gemm"])
        M = case["M"]
        if case["gemm"] == "down":  # SwiGLU activations
            a = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32)
            b = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32)
            i["x"] = (torch.nn.functional.silu(a) * b).to(torch.bfloat16).view(torch.int16)
        else:
            i["x"] = _bits(gen, (M, K), 1.0)
        i["w"] = _bits(gen, (N, K), 0.02)
        i["y"] = (torch.randn((M, N), generator=gen, device="cuda", dtype=torch.float32) if epi == nb.NJ_GEMM_RESIDUAL
                  else None)
    elif op == "accept":
        B, k = case["B"], case["k"]
        i["d"] = _drafts(s, B, k, gen)
        # the target agrees with the draft in part, as a draft model's does: half of the sequences follow it closely
        l = 1.2 * torch.randn((B, k + 1, s.vocab), generator=gen, device="cuda", dtype=torch.float32)
        l[: B // 2, :k] = torch.log(i["d"]["draft_probs"][: B // 2]) + 0.3 * l[: B // 2, :k]
        i["logits"] = l
    elif op == "migrate":
        s = i["s"] = POOLS[case["shape"]]
        n = 2 * case["moves"] + 8
        i["kp"] = _bits(gen, (s.n_layers, n, s.n_kv_heads, 16, s.head_dim), 0.5)
        i["vp"] = _bits(gen, (s.n_layers, n, s.n_kv_heads, s.head_dim, 16), 0.5)
        order = torch.randperm(n, generator=gen, device="cuda", dtype=torch.int64)
        lo, hi = order[order < n // 2], order[order >= n // 2]  # destinations below the boundary, sources above
        i["src"] = hi[: case["moves"]].to(torch.int32).contiguous()
        i["dst"] = lo[: case["moves"]].to(torch.int32).contiguous()
        i["n"] = n
    return i


class State:
    pass


def _buffer(nbytes):
    b = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    nb.workspace_init(b.data_ptr(), nbytes, _stream())
    return b


def prepare(case, seed):
    i = _inputs(case, seed)
    s, op = i["s"], case["op"]
    st = State()
    st.op, st.s, st.desc = op, s, model_desc(s)
    if op in ("step", "draft"):
        B, k = case["B"], case.get("k", 0)
        st.model = DeviceModel(s, i["w"])
        st.cache, st.kp, st.vp = i["cache"], i["kp"], i["vp"]
        st.ctx0 = st.cache.context_lens.clone()
        st.ws = Workspace(s, B, k, stream=_stream())
        if op == "step":
            st.io = StepIO(s, i["d"])
        else:
            st.B, st.last, st.u = B, i["last"], i["u"]
            st.token = torch.zeros(B, dtype=torch.int32, device="cuda")
            st.probs = torch.empty((B, s.vocab), dtype=torch.float32, device="cuda")
            st.accepted = torch.zeros(B, dtype=torch.int32, device="cuda")
    elif op == "qkv":
        st.B, st.k = case["B"], case["k"]
        st.h, st.g, st.w = i["h"], i["g"], pack_weight(i["w"])
        st.ctx = torch.from_numpy(i["ctx"]).cuda()
        st.q = torch.empty((st.B * (st.k + 1), s.n_heads, s.head_dim), dtype=torch.int16, device="cuda")
        st.wk = torch.empty((st.B, s.n_kv_heads, 16, s.head_dim), dtype=torch.int16, device="cuda")
        st.wv = torch.empty((st.B, s.n_kv_heads, s.head_dim, 16), dtype=torch.int16, device="cuda")
        st.ws = _buffer(nb.rmsnorm_rope_workspace_bytes(st.desc, st.B, st.k))
    elif op == "attn":
        st.B, st.k = case["B"], case["k"]
        st.cache, st.kp, st.vp = i["cache"], i["kp"], i["vp"]
        st.q, st.wk, st.wv = i["q"], i["wk"], i["wv"]
        st.out = torch.empty((st.B * (st.k + 1), s.n_heads * s.head_dim), dtype=torch.int16, device="cuda")
        st.ws = _buffer(nb.attn_workspace_bytes(st.desc, st.B, st.k))
    elif op == "gemm":
        st.N, st.K, st.epi = _gemm_shape(s, case["gemm"])
        st.M, st.x, st.w = case["M"], i["x"], pack_weight(i["w"])
        if st.epi == nb.NJ_GEMM_RESIDUAL:
            st.y = i["y"]
        elif st.epi == nb.NJ_GEMM_SWIGLU:
            st.y = torch.empty((st.M, st.N // 2), dtype=torch.int16, device="cuda")
        else:
            st.y = torch.empty((st.M, st.N), dtype=torch.float32, device="cuda")
        st.ws = _buffer(nb.gemm_workspace_bytes(nb.NJ_BF16, st.M, st.N, st.K, st.epi))
    elif op == "accept":
        st.B, st.k, st.logits = case["B"], case["k"], i["logits"]
        st.d = i["d"]
        st.accepted = torch.zeros(st.B, dtype=torch.int32, device="cuda")
        st.next = torch.zeros((st.B, st.k + 1), dtype=torch.int32, device="cuda")
        st.ws = _buffer(nb.accept_workspace_bytes(s.vocab, st.B, st.k))
    elif op == "migrate":
        st.kp, st.vp, st.src, st.dst, st.moves = i["kp"], i["vp"], i["src"], i["dst"], case["moves"]
        st.cache = DeviceCache({"k_pages": list(st.kp), "v_pages": list(st.vp), "num_blocks": i["n"],
                                "block_table": torch.zeros((1, 1), dtype=torch.int32, device="cuda"),
                                "context_lens": torch.zeros(1, dtype=torch.int32, device="cuda")})
        st.err = torch.zeros(1, dtype=torch.int32, device="cuda")
    return st


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------
def run(st):
    op, s = st.op, st.s
    if op == "step":
        # the append advances the context lengths: every pass starts from the same ones
        st.cache.context_lens.copy_(st.ctx0)
        verify(st.model, st.cache, st.io, st.ws)
        kv_append(st.model, st.cache, st.io, st.ws)
        out = {"logits": st.io.logits}
        if s.dtype != "bf16":
            out.update(accepted=st.io.accepted_len, next=st.io.next_tokens, ctx=st.cache.context_lens, k=st.kp, v=st.vp)
        elif st.io.k == 0:  # what is committed does not hang on the draw
            out.update(accepted=st.io.accepted_len, ctx=st.cache.context_lens, k=_f32_or_bf16(st.kp), v=_f32_or_bf16(st.vp))
        # With drafts in bf16 the accepted lengths and drawn tokens sit on
        # running sums over the whole vocabulary that any change of rounding
        # moves: the acceptance case compares them, on given logits.
        return out
    if op == "draft":
        c = st.cache
        c.context_lens.copy_(st.ctx0)
        nb.draft_step(st.desc, st.model.c, c.c, c.block_table.data_ptr(), c.max_blocks, c.context_lens.data_ptr(),
                      st.last.data_ptr(), st.u.data_ptr(), st.B, st.token.data_ptr(), 1, st.probs.data_ptr(), s.vocab,
                      st.ws.ptr, st.ws.nbytes, _stream())
        nb.kv_append(st.desc, c.c, c.block_table.data_ptr(), c.max_blocks, c.context_lens.data_ptr(), st.accepted.data_ptr(),
                     st.B, 0, st.ws.ptr, st.ws.nbytes, _stream())
        return {"probs": st.probs, "ctx": c.context_lens, "k": _f32_or_bf16(st.kp), "v": _f32_or_bf16(st.vp)}
    if op == "qkv":
        nb.rmsnorm_rope(st.desc, st.h.data_ptr(), st.g.data_ptr(), st.w.data_ptr(), st.ctx.data_ptr(), st.B, st.k,
                        st.q.data_ptr(), st.wk.data_ptr(), st.wv.data_ptr(), st.ws.data_ptr(), st.ws.numel(), _stream())
        return {"q": _f32_or_bf16(st.q), "k": _f32_or_bf16(st.wk), "v": _f32_or_bf16(st.wv)}
    if op == "attn":
        c = st.cache
        nb.attn_verify(st.desc, st.q.data_ptr(), st.kp.data_ptr(), st.vp.data_ptr(), c.num_blocks, st.wk.data_ptr(),
                       st.wv.data_ptr(), c.block_table.data_ptr(), c.max_blocks, c.context_lens.data_ptr(), st.B, st.k,
                       st.out.data_ptr(), st.ws.data_ptr(), st.ws.numel(), _stream())
        return {"out": _f32_or_bf16(st.out)}
    if op == "gemm":
        nb.gemm(nb.NJ_BF16, st.x.data_ptr(), st.w.data_ptr(), st.y.data_ptr(), st.M, st.N, st.K, st.epi, st.ws.data_ptr(),
                st.ws.numel(), _stream())
        return {"y": _f32_or_bf16(st.y)}
    if op == "accept":
        d = st.d
        nb.accept(st.desc, st.logits.data_ptr(), d["draft_tokens"].data_ptr(), d["draft_probs"].data_ptr(),
                  d["uniforms"].data_ptr(), st.B, st.k, st.accepted.data_ptr(), st.next.data_ptr(), st.ws.data_ptr(),
                  st.ws.numel(), _stream())
        return {"accepted": st.accepted, "next": st.next}
    nb.kv_migrate(st.desc, st.cache.c, st.src.data_ptr(), st.dst.data_ptr(), st.moves, st.err.data_ptr(), _stream())
    return {"k": st.kp, "v": st.vp, "err": st.err}


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    s, op = SHAPES[case["shape"]], case["op"]
    e = 2 if s.dtype == "bf16" else 4
    HD, KVD = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layer = s.qkv_dim * s.d_model + s.d_model * HD + 3 * s.ffn_dim * s.d_model
    if op in ("step", "draft"):
        B, k = case["B"], case.get("k", 0)
        M, kv = B * (k + 1), int(_contexts(case, 0).sum())
        params = s.n_layers * layer + s.vocab * s.d_model
        nbytes = params * e + M * s.d_model * e + s.n_layers * (kv + 2 * M) * KVD * 2 * e + M * s.vocab * 4
        nbytes += B * s.vocab * 4 if k else 0  # the draft distribution of the row that is drawn from
        flops = 2 * M * params + s.n_layers * 4 * (k + 1) * HD * (kv + B * (k + 2) / 2)
        return {"bytes": nbytes, "flops": flops}
    if op == "qkv":
        M = case["B"] * (case["k"] + 1)
        return {"bytes": s.qkv_dim * s.d_model * 2 + M * s.d_model * 4 + M * s.qkv_dim * 2,
                "flops": 2 * M * s.qkv_dim * s.d_model}
    if op == "attn":
        B, T = case["B"], case["k"] + 1
        kv = int(_contexts(case, 0).sum())
        return {"bytes": (kv + B * T) * KVD * 2 * 2 + 2 * B * T * HD * 2, "flops": 4 * T * HD * (kv + B * (T + 1) / 2)}
    if op == "gemm":
        N, K, epi = _gemm_shape(s, case["gemm"])
        M = case["M"]
        out = {nb.NJ_GEMM_RESIDUAL: 8 * N, nb.NJ_GEMM_SWIGLU: N, nb.NJ_GEMM_STORE: 4 * N}[epi]
        return {"bytes": N * K * 2 + M * K * 2 + M * out, "flops": 2 * M * N * K}
    if op == "accept":
        B, k = case["B"], case["k"]
        # every row's normaliser reads its logits; the draw reads one row of them and of the draft's distribution
        return {"bytes": (B * (k + 1) + (B if k else 0)) * s.vocab * 4, "flops": 4 * B * (k + 1) * s.vocab}
    s = POOLS[case["shape"]]
    return {"bytes": 2 * case["moves"] * s.n_layers * 2 * KVD * 16 * 2, "flops": 0}


def tolerance(case):
    op = case["op"]
    if op in ("migrate",):
        return "exact"
    if op == "accept":
        return {"rel": 0.0, "max": 0.0, "differ": 0.01}  # draws that sit on a boundary of a running sum
    if SHAPES[case["shape"]].dtype != "bf16":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if op == "draft":
        return {"rel": 0.03, "max": 0.5, "differ": 0.0}  # sixteen layers of bf16 activations
    if op == "step":
        return {"rel": 0.02, "max": 0.2, "differ": 0.0}  # one layer and the head, bf16 activations
    if op == "gemm" and case["gemm"] != "gate_up":
        return {"rel": 1e-5, "max": 1e-3}  # fp32 sums of bf16 products, fp32 results
    return {"rel": 1e-2, "max": 0.2}  # bf16 results


# --------------------------------------------------------------------------
# The same in 64 bits
# --------------------------------------------------------------------------
def _wide(t):
    return _f32_or_bf16(t).to(torch.float64)


def _norm64(h, g, eps):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * g


def _rope64(x, pos, theta):
    """x [M][heads][D], pos [M]: pair (j, j + D/2) turned by pos * theta^(-2j/D)."""
    D = x.shape[-1]
    j = torch.arange(D // 2, dtype=torch.float64, device="cuda")
    a = pos.to(torch.float64)[:, None] * torch.pow(torch.tensor(float(np.float32(theta)), dtype=torch.float64, device="cuda"), -2.0 * j / D)
    c, sn = torch.cos(a)[:, None], torch.sin(a)[:, None]
    x0, x1 = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([x0 * c - x1 * sn, x0 * sn + x1 * c], -1)


def _attn64(s, q, kp, vp, table, ctx, k_win, v_win):
    """q [M][H][D]; k_win, v_win [B][T][Hkv][D]; pages of one layer, any dtype.  -> [M][H*D]"""
    B, T = k_win.shape[:2]
    G = s.n_heads // s.n_kv_heads
    out = []
    for b in range(B):
        c = int(ctx[b])
        blocks = table[b, : (c + 15) // 16].long()
        kc = _wide(kp[blocks]).permute(1, 0, 2, 3).reshape(s.n_kv_heads, -1, s.head_dim)[:, :c]
        vc = _wide(vp[blocks]).permute(1, 0, 3, 2).reshape(s.n_kv_heads, -1, s.head_dim)[:, :c]
        kk = torch.cat([kc, k_win[b].permute(1, 0, 2)], 1)
        vv = torch.cat([vc, v_win[b].permute(1, 0, 2)], 1)
        qb = q[b * T: (b + 1) * T].view(T, s.n_kv_heads, G, s.head_dim).permute(1, 2, 0, 3).reshape(s.n_kv_heads, G * T, s.head_dim)
        sc = torch.matmul(qb, kk.transpose(1, 2).contiguous()).view(s.n_kv_heads, G, T, c + T) / math.sqrt(s.head_dim)
        mask = torch.arange(c + T, device="cuda")[None, :] > c + torch.arange(T, device="cuda")[:, None]
        p = torch.softmax(sc.masked_fill(mask, -math.inf), -1).view(s.n_kv_heads, G * T, c + T)
        ob = torch.matmul(p, vv).view(s.n_kv_heads, G, T, s.head_dim).permute(2, 0, 1, 3)
        out.append(ob.reshape(T, s.n_heads * s.head_dim))
    return torch.cat(out)


def _forward64(s, w, tokens, pos, kp, vp, table, ctx, B, T):
    """Logits [M][V] and the window's rotated keys and values [L][B][T][Hkv][D]."""
    h = _wide(w["embed"][tokens.long()])
    HD, KVD = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    eps = float(np.float32(s.rms_eps))
    ks, vs = [], []
    for l, lw in enumerate(w["layers"]):
        y = _norm64(h, _wide(lw["attn_norm"]), eps) @ _wide(lw["w_qkv"]).T
        q = _rope64(y[:, :HD].reshape(-1, s.n_heads, s.head_dim), pos, s.rope_theta)
        kw = _rope64(y[:, HD: HD + KVD].reshape(-1, s.n_kv_heads, s.head_dim), pos, s.rope_theta).view(B, T, s.n_kv_heads, s.head_dim)
        vw = y[:, HD + KVD:].reshape(B, T, s.n_kv_heads, s.head_dim)
        h = h + _attn64(s, q, kp[l], vp[l], table, ctx, kw, vw) @ _wide(lw["w_o"]).T
        y = _norm64(h, _wide(lw["ffn_norm"]), eps) @ _wide(lw["w_gate_up"]).T
        h = h + (torch.nn.functional.silu(y[:, : s.ffn_dim]) * y[:, s.ffn_dim:]) @ _wide(lw["w_down"]).T
        ks.append(kw)
        vs.append(vw)
    return _norm64(h, _wide(w["final_norm"]), eps) @ _wide(w["lm_head"]).T, torch.stack(ks), torch.stack(vs)


def _accept64(logits, d, B, k):
    """The acceptance rule: accepted lengths and tokens, from logits [B][k+1][V] in 64 bits."""
    acc = torch.zeros(B, dtype=torch.int32)
    nxt = torch.full((B, k + 1), -1, dtype=torch.int32)
    for b in range(B):
        p = torch.softmax(logits[b].to(torch.float64), -1)
        q = d["draft_probs"][b].to(torch.float64)
        u = d["uniforms"][b].to(torch.float64)
        n = 0
        while n < k:
            x = int(d["draft_tokens"][b, n])
            if not float(u[n]) * float(q[n, x]) < float(p[n, x]):
                break
            nxt[b, n] = x
            n += 1
        wts = torch.clamp(p[n] - q[n], min=0) if n < k else p[n]
        if float(wts.sum()) == 0.0:
            wts = p[n]
        c = torch.cumsum(wts, 0)
        nxt[b, n] = int(torch.searchsorted(c, u[k] * c[-1], right=True))
        acc[b] = n
    return acc, nxt


def _append64(pages, new, table, ctx, rows, dim_major):
    """The pages with window rows 0..rows[b]-1 of new [L][B][T][Hkv][D] at the sequences' ends."""
    out = _wide(pages).clone()
    for b in range(len(ctx)):
        for j in range(int(rows[b])):
            t = int(ctx[b]) + j
            block = int(table[b, t // 16])
            if dim_major:
                out[:, block, :, :, t % 16] = new[:, b, j]
            else:
                out[:, block, :, t % 16] = new[:, b, j]
    return out


def exact(case, seed):
    i = _inputs(case, seed)
    s, op = i["s"], case["op"]
    if op in ("step", "draft"):
        B, k = case["B"], case.get("k", 0)
        T, ctx, table = k + 1, i["ctx"], i["cache"].block_table
        tokens = torch.cat([i["d"]["last_tokens"][:, None], i["d"]["draft_tokens"]], 1) if op == "step" else i["last"][:, None]
        pos = (torch.from_numpy(ctx).cuda()[:, None] + torch.arange(T, device="cuda")).reshape(-1)
        logits, ks, vs = _forward64(s, i["w"], tokens.reshape(-1), pos, i["kp"], i["vp"], table, ctx, B, T)
        if op == "draft":
            ones = np.ones(B, np.int32)
            return {"probs": torch.softmax(logits, -1), "ctx": None, "k": _append64(i["kp"], ks, table, ctx, ones, False),
                    "v": _append64(i["vp"], vs, table, ctx, ones, True)}
        out = {"logits": logits.view(B, T, s.vocab)}
        if s.dtype != "bf16" or k == 0:
            acc, nxt = _accept64(out["logits"], i["d"], B, k)
            out.update(accepted=acc, ctx=torch.from_numpy(ctx + acc.numpy() + 1), k=_append64(i["kp"], ks, table, ctx, acc + 1, False),
                       v=_append64(i["vp"], vs, table, ctx, acc + 1, True))
            if s.dtype != "bf16":
                out["next"] = nxt
        return out
    if op == "qkv":
        B, T = case["B"], case["k"] + 1
        pos = (torch.from_numpy(i["ctx"]).cuda()[:, None] + torch.arange(T, device="cuda")).reshape(-1)
        HD, KVD = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
        y = _norm64(i["h"].double(), _wide(i["g"]), float(np.float32(s.rms_eps))) @ _wide(i["w"]).T
        q = _rope64(y[:, :HD].reshape(-1, s.n_heads, s.head_dim), pos, s.rope_theta)
        kr = _rope64(y[:, HD: HD + KVD].reshape(-1, s.n_kv_heads, s.head_dim), pos, s.rope_theta)
        k = torch.zeros((B, s.n_kv_heads, 16, s.head_dim), dtype=torch.float64, device="cuda")
        v = torch.zeros((B, s.n_kv_heads, s.head_dim, 16), dtype=torch.float64, device="cuda")
        k[:, :, :T] = kr.view(B, T, s.n_kv_heads, s.head_dim).permute(0, 2, 1, 3)
        v[..., :T] = y[:, HD + KVD:].reshape(B, T, s.n_kv_heads, s.head_dim).permute(0, 2, 3, 1)
        return {"q": q, "k": k, "v": v}
    if op == "attn":
        T = case["k"] + 1
        kw, vw = _wide(i["wk"])[:, :, :T].permute(0, 2, 1, 3), _wide(i["wv"])[..., :T].permute(0, 3, 1, 2)
        return {"out": _attn64(s, _wide(i["q"]), i["kp"][0], i["vp"][0], i["cache"].block_table, i["ctx"], kw, vw)}
    if op == "gemm":
        _, _, epi = _gemm_shape(s, case["gemm"])
        y = _wide(i["x"]) @ _wide(i["w"]).T
        if epi == nb.NJ_GEMM_RESIDUAL:
            y += i["y"].double()
        elif epi == nb.NJ_GEMM_SWIGLU:
            y = torch.nn.functional.silu(y[:, : s.ffn_dim]) * y[:, s.ffn_dim:]
        return {"y": y}
    if op == "accept":
        acc, nxt = _accept64(i["logits"], i["d"], case["B"], case["k"])
        return {"accepted": acc, "next": nxt}
    return None  # bytes moved, nothing computed
