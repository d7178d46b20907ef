"""The work that a program using this library has it do, as timed cases.

Six kinds of call sequences, each over the range of sizes in which it is used:

  encode    ba_encode_blocks: passages attended on their own, their keys kept for a cache
  reencode  ba_reencode_positions: cached keys of all layers turned to their place in a prompt
  final     ba_final_block_attention: the query block over its whole, contiguous context
  cached    ba_final_block_attention_cached: the same straight from a cache of blocks
  train     ba_block_attention_prompts and its backward: one attention layer of a fine-tune step
  request   encode, re-encode and final block one after the other: a prompt nothing of which is cached

``listed`` names the cases, ``draw`` makes further ones of the same ranges, ``prepare`` builds what a
program has in hand before the call, ``run`` makes one pass, ``work`` says what a pass cannot do
without, ``tolerance`` how far two correct implementations may differ.
"""
import math

import numpy as np
import torch

from paper_2409_15355_amd import binding as ba

LLAMA = {"n_q_heads": 32, "n_kv_heads": 8, "head_dim": 128, "rope_base": 500000.0}
SMALL = {"n_q_heads": 4, "n_kv_heads": 4, "head_dim": 64, "rope_base": 10000.0}
# head shapes a drawn case may have: the two above, and groups of four and two query heads per KV head
GEOMETRIES = [LLAMA, LLAMA, LLAMA, SMALL,
              {"n_q_heads": 8, "n_kv_heads": 2, "head_dim": 64, "rope_base": 10000.0},
              {"n_q_heads": 16, "n_kv_heads": 8, "head_dim": 128, "rope_base": 500000.0}]


def listed():
    return [
        # the smallest prompt: two passages of 128 tokens, one query head per KV head; launches and host work count
        {"name": "encode_tiny", "kind": "encode", **SMALL, "layout": "interleaved", "n_blocks": 2, "len_min": 128, "len_max": 128,
         "shape_seed": 1, "keep_keys": True},
        # a batch of eight prompts' retrieved passages, ragged, encoded once and their keys kept
        {"name": "encode_passages", "kind": "encode", **LLAMA, "layout": "interleaved", "n_blocks": 160, "len_min": 100, "len_max": 300,
         "shape_seed": 3, "keep_keys": True},
        # a whole 32,000-token prompt as one block: ordinary causal prefill, the largest call
        {"name": "encode_one_block", "kind": "encode", **LLAMA, "layout": "interleaved", "n_blocks": 1, "len_min": 32000,
         "len_max": 32000, "shape_seed": 5, "keep_keys": False},
        # the cached keys of 32 passages of 1,000 tokens moved to other places of the prompt, all layers
        {"name": "reencode_cache", "kind": "reencode", **LLAMA, "layout": "interleaved", "n_layers": 32, "n_blocks": 32,
         "len_min": 1000, "len_max": 1000, "shape_seed": 4, "mode": "shift", "dtype": "bf16"},
        # one prompt's ten passages in the pairing that Llama checkpoints store, all layers
        {"name": "reencode_prompt_half", "kind": "reencode", **LLAMA, "layout": "half", "n_layers": 32, "n_blocks": 10,
         "len_min": 200, "len_max": 200, "shape_seed": 2, "mode": "shift", "dtype": "bf16"},
        # a 256-token query block over 31 passages of 1,024 tokens: one layer of a long prompt
        {"name": "final_32k", "kind": "final", **LLAMA, "layout": "interleaved", "n_prompts": 1, "ctx_min": 31744, "ctx_max": 31744,
         "q_min": 256, "q_max": 256, "shape_seed": 5},
        # a 50-token question over the same length of context, as in the paper's time-to-first-token table
        {"name": "final_question_32k", "kind": "final", **LLAMA, "layout": "interleaved", "n_prompts": 1, "ctx_min": 31950,
         "ctx_max": 31950, "q_min": 50, "q_max": 50, "shape_seed": 6},
        # eight prompts of some 4,000 context tokens each, ragged, batched into one call
        {"name": "final_batch", "kind": "final", **LLAMA, "layout": "half", "n_prompts": 8, "ctx_min": 3400, "ctx_max": 4600,
         "q_min": 32, "q_max": 128, "shape_seed": 3},
        # a query block over 31 cached passages that stay at the positions they were encoded at
        {"name": "cached_32k", "kind": "cached", **LLAMA, "layout": "interleaved", "n_prompts": 1, "n_blocks": 31, "len_min": 1024,
         "len_max": 1024, "q_min": 256, "q_max": 256, "shape_seed": 5},
        # hundreds of small cached state blocks, none of them rewritten, and a short query
        {"name": "cached_small_blocks", "kind": "cached", **LLAMA, "layout": "interleaved", "n_prompts": 1, "n_blocks": 512,
         "len_min": 20, "len_max": 60, "q_min": 64, "q_max": 64, "shape_seed": 6},
        # forward and backward of eight prompts of 20 ragged passages and a query block
        {"name": "train_step", "kind": "train", **LLAMA, "layout": "interleaved", "n_prompts": 8, "n_blocks": 20, "len_min": 100,
         "len_max": 300, "q_min": 32, "q_max": 128, "shape_seed": 3},
        # ten passages of 200 tokens and a 64-token question, nothing cached: three calls in a row
        {"name": "request", "kind": "request", **LLAMA, "layout": "half", "n_blocks": 10, "len_min": 200, "len_max": 200, "q_min": 64,
         "q_max": 64, "shape_seed": 2},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _drawn(rng):
    case = {"kind": rng.choice(["encode", "reencode", "final", "cached", "train", "request"]), **rng.choice(GEOMETRIES)}
    case["layout"] = rng.choice(["interleaved", "half"])
    case["shape_seed"] = rng.randrange(1, 1 << 30)
    kind = case["kind"]
    if kind == "encode":
        mean = _log_int(rng, 32, 16000)
        n = _log_int(rng, 1, max(1, min(320, 33000 // mean)))
        case.update(n_blocks=n, len_min=max(1, mean // 2 + rng.randrange(3)), len_max=mean + mean // 2, keep_keys=rng.random() < 0.7)
    elif kind == "reencode":
        mean = _log_int(rng, 32, 2000)
        n = _log_int(rng, 1, max(1, min(96, 32000 // mean)))
        case.update(n_layers=_log_int(rng, 1, 32), n_blocks=n, len_min=max(1, mean // 2 + rng.randrange(3)), len_max=mean + mean // 2,
                    mode=rng.choice(["shift", "shift", "absolute"]), dtype=rng.choice(["bf16", "bf16", "f32"]))
    elif kind == "final":
        ctx = _log_int(rng, 500, 32000)
        n = _log_int(rng, 1, max(1, min(16, 64000 // ctx)))
        q = _log_int(rng, 1, 256)
        case.update(n_prompts=n, ctx_min=max(1, ctx // 2 + rng.randrange(3)), ctx_max=ctx + ctx // 2, q_min=max(1, q // 2), q_max=q + q // 2)
    elif kind == "cached":
        mean = _log_int(rng, 20, 2000)
        n = _log_int(rng, 4, max(4, min(600, 32000 // mean)))
        q = _log_int(rng, 1, 256)
        case.update(n_prompts=rng.choice([1, 1, 2, 4]) if n * mean <= 16000 else 1, n_blocks=n, len_min=max(1, mean // 2 + rng.randrange(3)),
                    len_max=mean + mean // 2, q_min=max(1, q // 2), q_max=q + q // 2)
    elif kind == "train":
        mean = _log_int(rng, 50, 800)
        blocks = _log_int(rng, 2, max(2, min(30, 8000 // mean)))
        prompts = _log_int(rng, 1, max(1, min(8, 33000 // (mean * blocks))))
        q = _log_int(rng, 8, 256)
        case.update(n_prompts=prompts, n_blocks=blocks, len_min=max(1, mean // 2 + rng.randrange(3)), len_max=mean + mean // 2,
                    q_min=max(1, q // 2), q_max=q + q // 2)
    else:
        mean = _log_int(rng, 50, 1000)
        n = _log_int(rng, 2, max(2, min(31, 16000 // mean)))
        q = _log_int(rng, 8, 256)
        case.update(n_blocks=n, len_min=max(1, mean // 2 + rng.randrange(3)), len_max=mean + mean // 2, q_min=max(1, q // 2), q_max=q + q // 2)
    return case


def draw(rng):
    """One more case of the ranges above, no dearer than the largest listed one."""
    most = [work(c) for c in listed()]
    flops, nbytes = max(w["flops"] for w in most), max(w["bytes"] for w in most)
    while True:
        case = _drawn(rng)
        w = work(case)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return case


# ---- shapes: the lengths of a case's blocks, contexts and query blocks ----------------------------------
def _shape(case):
    rng = np.random.Generator(np.random.Philox(case["shape_seed"]))

    def ints(lo, hi, n):
        return rng.integers(lo, hi + 1, n).astype(np.int32)

    kind = case["kind"]
    prompts = case.get("n_prompts", 1)
    s = {}
    if kind == "final":
        s["ctx"] = ints(case["ctx_min"], case["ctx_max"], prompts)
    else:
        s["blk"] = ints(case["len_min"], case["len_max"], prompts * case["n_blocks"])
        s["order"] = rng.permutation(len(s["blk"]))
    if "q_min" in case:
        s["q"] = ints(case["q_min"], case["q_max"], prompts)
    return s


def _cumulative(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def _heads(case):
    layout = ba.ROPE_HALF if case["layout"] == "half" else ba.ROPE_INTERLEAVED
    return ba.Heads(case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["rope_base"], rope_layout=layout)


def _causal_pairs(lens):
    lens = lens.astype(np.float64)
    return float((lens * (lens + 1) / 2).sum())


def _final_pairs(ctx, q):
    return float((ctx.astype(np.float64) * q).sum()) + _causal_pairs(q)


def work(case):
    s = _shape(case)
    hq, hkv, d = case["n_q_heads"], case["n_kv_heads"], case["head_dim"]
    kind, prompts = case["kind"], case.get("n_prompts", 1)
    if kind == "encode":
        t = float(s["blk"].sum())
        return {"bytes": 2 * d * t * (2 * hq + (3 if case["keep_keys"] else 2) * hkv), "flops": 4 * d * hq * _causal_pairs(s["blk"])}
    if kind == "reencode":
        n = float(s["blk"].sum()) * case["n_layers"] * hkv * d
        return {"bytes": 2 * n * (4 if case["dtype"] == "f32" else 2), "flops": 3 * n}
    if kind in ("final", "cached"):
        ctx = s["ctx"] if kind == "final" else s["blk"].reshape(prompts, -1).sum(axis=1)
        tq, tc = float(s["q"].sum()), float(ctx.sum())
        return {"bytes": 2 * d * (2 * hq * tq + 2 * hkv * (tq + tc)), "flops": 4 * d * hq * _final_pairs(ctx, s["q"])}
    ctx = s["blk"].reshape(prompts, -1).sum(axis=1)
    t, tq = float(s["blk"].sum()), float(s["q"].sum())
    pairs = _causal_pairs(s["blk"]) + _final_pairs(ctx, s["q"])
    if kind == "train":  # q, dO, o, dq and k, v, dk, dv once each, the log-sum-exps; 2 products forward, 5 backward
        return {"bytes": 2 * d * (t + tq) * (4 * hq + 4 * hkv) + 4 * hq * (t + tq), "flops": 14 * d * hq * pairs}
    # request: q, k, v and o of every token, the keys rotated twice
    return {"bytes": 2 * d * ((t + tq) * (2 * hq + 2 * hkv) + 2 * hkv * t), "flops": 4 * d * hq * pairs}


# ---- inputs -----------------------------------------------------------------------------------------------
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def randn(shape, dtype=torch.bfloat16):
        # projected activations and cached keys: standard normal, rounded to the tensor's type
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)

    def scratch(nbytes):
        return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")

    s = _shape(case)
    heads = _heads(case)
    hq, hkv, d = case["n_q_heads"], case["n_kv_heads"], case["head_dim"]
    kind, prompts = case["kind"], case.get("n_prompts", 1)
    st = {"kind": kind, "heads": heads}
    if kind == "encode":
        offs = _cumulative(s["blk"])
        t = int(offs[-1])
        st.update(offs=offs, q=randn((t, hq, d)), k=randn((t, hkv, d)), v=randn((t, hkv, d)))
        st["o"] = torch.empty_like(st["q"])
        st["k_local"] = torch.empty_like(st["k"]) if case["keep_keys"] else None
        st["ws"] = scratch(ba.ba_encode_blocks_workspace_bytes(heads, offs, ba.ROPE_APPLY, case["keep_keys"]))
    elif kind == "reencode":
        # blocks lie in the cache in the order they were encoded and go to the prompt in retrieval order
        order, lens = s["order"], s["blk"]
        src_off = _cumulative(lens)[:-1]
        dst_off = np.empty_like(src_off)
        dst_off[order] = _cumulative(lens[order])[:-1]
        dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        shape = (case["n_layers"], int(lens.sum()), hkv, d)
        k_src = torch.empty(shape, dtype=dtype, device="cuda")
        for layer in range(shape[0]):
            k_src[layer] = randn(shape[1:], dtype)
        st.update(k_src=k_src, k_dst=torch.empty_like(k_src), src_off=src_off, dst_off=dst_off, lens=lens,
                  mode=ba.REENC_ABSOLUTE if case["mode"] == "absolute" else ba.REENC_SHIFT)
    elif kind == "final":
        cu_ctx, cu_q = _cumulative(s["ctx"]), _cumulative(s["q"])
        tc, tq = int(cu_ctx[-1]), int(cu_q[-1])
        st.update(cu_ctx=cu_ctx, cu_q=cu_q, q=randn((tq, hq, d)), kc=randn((tc, hkv, d)), vc=randn((tc, hkv, d)),
                  kf=randn((tq, hkv, d)), vf=randn((tq, hkv, d)))
        st["o"] = torch.empty_like(st["q"])
        st["ws"] = scratch(ba.ba_final_block_attention_workspace_bytes(heads, cu_q, cu_ctx))
    elif kind == "cached":
        cu_q = _cumulative(s["q"])
        cu_blk = (np.arange(prompts + 1) * case["n_blocks"]).astype(np.int32)
        order, lens = s["order"], s["blk"]
        off = np.empty(len(lens), dtype=np.int32)
        off[order] = _cumulative(lens[order])[:-1]  # a prompt's blocks lie anywhere in the cache
        tc, tq = int(lens.sum()), int(cu_q[-1])
        st.update(cu_q=cu_q, cu_blk=cu_blk, off=off, lens=lens, q=randn((tq, hq, d)), kc=randn((tc, hkv, d)), vc=randn((tc, hkv, d)),
                  kf=randn((tq, hkv, d)), vf=randn((tq, hkv, d)))
        st["o"] = torch.empty_like(st["q"])
        st["ws"] = scratch(ba.ba_final_block_attention_cached_workspace_bytes(heads, cu_q, cu_blk, lens))
    elif kind == "train":
        blocks = np.concatenate([s["blk"].reshape(prompts, -1), s["q"][:, None]], axis=1)
        offs = _cumulative(blocks.reshape(-1))
        cu_blk = (np.arange(prompts + 1) * blocks.shape[1]).astype(np.int32)
        t = int(offs[-1])
        st.update(offs=offs, cu_blk=cu_blk, q=randn((t, hq, d)), k=randn((t, hkv, d)), v=randn((t, hkv, d)), d_out=randn((t, hq, d)))
        st.update(o=torch.empty_like(st["q"]), lse=torch.empty((t, hq), dtype=torch.float32, device="cuda"),
                  dq=torch.empty_like(st["q"]), dk=torch.empty_like(st["k"]), dv=torch.empty_like(st["v"]))
        st["ws"] = scratch(max(ba.ba_block_attention_prompts_workspace_bytes(heads, cu_blk, offs),
                               ba.ba_block_attention_prompts_backward_workspace_bytes(heads, cu_blk, offs)))
    else:
        offs, cu_q = _cumulative(s["blk"]), _cumulative(s["q"])
        t, tq = int(offs[-1]), int(cu_q[-1])
        cu_ctx = np.array([0, t], dtype=np.int32)
        st.update(offs=offs, cu_q=cu_q, cu_ctx=cu_ctx, start=offs[:-1].copy(), lens=s["blk"], q=randn((t, hq, d)), k=randn((t, hkv, d)),
                  v=randn((t, hkv, d)), qf=randn((tq, hq, d)), kf=randn((tq, hkv, d)), vf=randn((tq, hkv, d)))
        st.update(o=torch.empty_like(st["q"]), k_local=torch.empty_like(st["k"]), k_ctx=torch.empty_like(st["k"]),
                  of=torch.empty_like(st["qf"]))
        st["ws"] = scratch(max(ba.ba_encode_blocks_workspace_bytes(heads, offs, ba.ROPE_APPLY, True),
                               ba.ba_final_block_attention_workspace_bytes(heads, cu_q, cu_ctx)))
    return st


def run(st):
    kind, heads = st["kind"], st["heads"]
    if kind == "encode":
        ba.ba_encode_blocks(heads, st["q"], st["k"], st["v"], st["o"], st["k_local"], st["offs"], ba.ROPE_APPLY, st["ws"])
        return [st["o"]] if st["k_local"] is None else [st["o"], st["k_local"]]
    if kind == "reencode":
        ba.ba_reencode_positions(heads, st["k_src"], st["k_dst"], st["src_off"], st["dst_off"], st["lens"], None, st["dst_off"], st["mode"])
        return [st["k_dst"]]
    if kind == "final":
        ba.ba_final_block_attention(heads, st["q"], st["kc"], st["vc"], st["kf"], st["vf"], st["o"], None, st["cu_q"], st["cu_ctx"],
                                    None, ba.ROPE_APPLY, st["ws"])
        return [st["o"]]
    if kind == "cached":
        ba.ba_final_block_attention_cached(heads, st["q"], st["kc"], st["vc"], st["kf"], st["vf"], st["o"], None, st["cu_q"],
                                           st["cu_blk"], st["off"], st["lens"], None, None, None, st["ws"])
        return [st["o"]]
    if kind == "train":
        ba.ba_block_attention_prompts(heads, st["q"], st["k"], st["v"], st["o"], None, st["lse"], st["cu_blk"], st["offs"],
                                      ba.ROPE_APPLY, st["ws"])
        ba.ba_block_attention_prompts_backward(heads, st["q"], st["k"], st["v"], st["o"], st["lse"], st["d_out"], st["dq"], st["dk"],
                                               st["dv"], st["cu_blk"], st["offs"], st["ws"])
        return [st["o"], st["lse"], st["dq"], st["dk"], st["dv"]]
    ba.ba_encode_blocks(heads, st["q"], st["k"], st["v"], st["o"], st["k_local"], st["offs"], ba.ROPE_APPLY, st["ws"])
    ba.ba_reencode_positions(heads, st["k_local"], st["k_ctx"], st["start"], st["start"], st["lens"], None, st["start"])
    ba.ba_final_block_attention(heads, st["qf"], st["k_ctx"], st["v"], st["kf"], st["vf"], st["of"], None, st["cu_q"], st["cu_ctx"],
                                None, ba.ROPE_APPLY, st["ws"])
    return [st["o"], st["k_local"], st["k_ctx"], st["of"]]


def tolerance(case):
    """About four times what each path differs from itself in 64 bits, over the cases above: 2-norms 4e-8
    (re-encoded fp32 keys), 1.7e-3 (bf16 keys: one rounding), 2e-3 to 3.7e-3 (outputs and gradients of
    the attention steps: bf16 operands and probabilities, one rounding of the result); single elements
    5e-7, 4e-3 and 8e-2 of the larger of their size and the tensor's root mean square."""
    if case["kind"] == "reencode":
        return {"rel": 2e-7, "max": 2e-6} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1.4e-2, "max": 0.3}


# ---- the same in 64 bits, in plain torch --------------------------------------------------------------------
def _turn(x, pos, case):
    """x [tokens, heads, D] turned by the angles of the tokens' positions (a negative position turns back)."""
    d = x.shape[-1]
    freq = case["rope_base"] ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    angle = torch.as_tensor(pos, dtype=torch.float64, device=x.device)[:, None, None] * freq
    c, s = angle.cos(), angle.sin()
    if case["layout"] == "half":
        a, b = x[..., : d // 2], x[..., d // 2:]
        return torch.cat([c * a - s * b, s * a + c * b], dim=-1)
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([c * a - s * b, s * a + c * b], dim=-1).reshape(x.shape)


def _attend(q, k, v, first, d_out=None):
    """Causal attention of rotated q, whose first token is key `first`; with d_out also the log-sum-exps and gradients."""
    hq, hkv, d = q.shape[1], k.shape[1], q.shape[2]
    g = hq // hkv
    o, lse, dq = torch.zeros_like(q), q.new_zeros(q.shape[:2]), torch.zeros_like(q)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    for h in range(hkv):
        heads = slice(h * g, (h + 1) * g)
        step = max(16, (1 << 26) // max(1, len(k) * g))
        for r in range(0, len(q), step):
            n = min(step, len(q) - r)
            keys = first + r + n
            kh, vh = k[:keys, h], v[:keys, h]
            qh = q[r: r + n, heads].reshape(n * g, d)
            sc = (qh @ kh.T / math.sqrt(d)).view(n, g, keys)
            last = first + r + torch.arange(n, device=q.device)
            sc.masked_fill_(torch.arange(keys, device=q.device)[None, None, :] > last[:, None, None], -math.inf)
            norm = torch.logsumexp(sc, dim=-1)
            p = sc.sub_(norm[..., None]).exp_().view(n * g, keys)
            oh = p @ vh
            o[r: r + n, heads], lse[r: r + n, heads] = oh.view(n, g, d), norm
            if d_out is not None:
                gh = d_out[r: r + n, heads].reshape(n * g, d)
                ds = p * (gh @ vh.T - (gh * oh).sum(-1, keepdim=True)) / math.sqrt(d)
                dq[r: r + n, heads] = (ds @ kh).view(n, g, d)
                dk[:keys, h] += ds.T @ qh
                dv[:keys, h] += p.T @ gh
    return o, lse, dq, dk, dv


def exact(case, seed):
    """What `run` returns for these inputs, in 64 bits, without rounding anything on the way."""
    st, s = prepare(case, seed), _shape(case)
    kind = case["kind"]
    f = {n: t.double() for n, t in st.items() if n in ("q", "k", "v", "kc", "vc", "kf", "vf", "qf", "d_out")}
    pos = torch.arange(40000, dtype=torch.float64, device="cuda")  # longer than any prompt here

    def encode():
        o, kl = torch.empty_like(f["q"]), torch.empty_like(f["k"])
        for a, b in zip(st["offs"][:-1].tolist(), st["offs"][1:].tolist()):
            kl[a:b] = _turn(f["k"][a:b], pos[: b - a], case)
            o[a:b] = _attend(_turn(f["q"][a:b], pos[: b - a], case), kl[a:b], f["v"][a:b], 0)[0]
        return o, kl

    def final(q, kf, vf, k, v):
        n = len(k)
        at = pos[n: n + len(q)]
        return _attend(_turn(q, at, case), torch.cat([k, _turn(kf, at, case)]), torch.cat([v, vf]), n)[0]

    if kind == "encode":
        o, kl = encode()
        return [o] if st["k_local"] is None else [o, kl]
    if kind == "reencode":
        out = torch.empty(st["k_src"].shape, dtype=torch.float64, device="cuda")
        for a, b, n in zip(st["src_off"].tolist(), st["dst_off"].tolist(), s["blk"].tolist()):
            # shift: every key of a block by the block's new first position; absolute: by its own position
            at = b + pos[:n] if case["mode"] == "absolute" else torch.full((n,), float(b), dtype=torch.float64, device="cuda")
            for layer in range(case["n_layers"]):
                out[layer, b: b + n] = _turn(st["k_src"][layer, a: a + n].double(), at, case)
        return [out]
    if kind == "final":
        o = torch.empty_like(f["q"])
        for i in range(case["n_prompts"]):
            a, b = st["cu_q"][i: i + 2].tolist()
            c, e = st["cu_ctx"][i: i + 2].tolist()
            o[a:b] = final(f["q"][a:b], f["kf"][a:b], f["vf"][a:b], f["kc"][c:e], f["vc"][c:e])
        return [o]
    if kind == "cached":
        o = torch.empty_like(f["q"])
        for i in range(case["n_prompts"]):
            ks, vs, at = [], [], 0
            for blk in range(*st["cu_blk"][i: i + 2].tolist()):
                a, n = int(st["off"][blk]), int(st["lens"][blk])
                ks.append(_turn(f["kc"][a: a + n], torch.full((n,), float(at), dtype=torch.float64, device="cuda"), case))
                vs.append(f["vc"][a: a + n])
                at += n
            a, b = st["cu_q"][i: i + 2].tolist()
            o[a:b] = final(f["q"][a:b], f["kf"][a:b], f["vf"][a:b], torch.cat(ks), torch.cat(vs))
        return [o]
    if kind == "train":
        out = [torch.zeros_like(f["q"]), torch.zeros(st["lse"].shape, dtype=torch.float64, device="cuda")]
        out += [torch.zeros_like(f[n]) for n in ("q", "k", "v")]
        o, lse, dq, dk, dv = out
        for i in range(case["n_prompts"]):
            lo, hi = st["cu_blk"][i: i + 2].tolist()
            t0, t1 = int(st["offs"][lo]), int(st["offs"][hi])
            at = pos[: t1 - t0]
            q, k = _turn(f["q"][t0:t1], at, case), _turn(f["k"][t0:t1], at, case)
            for blk in range(lo, hi):
                a, b = st["offs"][blk: blk + 2].tolist()
                key0 = t0 if blk == hi - 1 else a  # only the last block sees the others
                got = _attend(q[a - t0: b - t0], k[key0 - t0: b - t0], f["v"][key0:b], a - key0, f["d_out"][a:b])
                o[a:b], lse[a:b], dq[a:b] = got[:3]
                dk[key0:b] += got[3]
                dv[key0:b] += got[4]
            dq[t0:t1], dk[t0:t1] = _turn(dq[t0:t1], -at, case), _turn(dk[t0:t1], -at, case)
        return out
    o, kl = encode()
    k_ctx = torch.empty_like(kl)
    for a, n in zip(st["start"].tolist(), st["lens"].tolist()):
        k_ctx[a: a + n] = _turn(kl[a: a + n], torch.full((n,), float(a), dtype=torch.float64, device="cuda"), case)
    return [o, kl, k_ctx, final(f["qf"], f["kf"], f["vf"], k_ctx, f["v"])]
