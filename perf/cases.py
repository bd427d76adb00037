"""The work a program gives this library, as measurable cases: decode steps on a filled cache and
appends of new tokens, over the sizes of the benchmark configurations (synth.WORKLOADS), their ragged
neighbours, both pack sizes, wide codes, paged arenas, repacking and both input types.

A case is a dict:
  op        "fused":  append one token, kv_decode_attention                      (one decode step)
            "steps":  append one token, kv_k_matvec, kv_softmax, kv_v_matvec     (the paper's three steps)
            "append": kv_compress_append of `new` tokens                         (prompt, chunk or block flush)
  batch, kv_heads, q_heads
  tokens    tokens the cache holds before the call (0: an empty cache, a prompt)
  new       tokens the call appends
  pack      16 or 8; k_rel, v_rel: relative quantization scales (below 1/15: wide chunks)
  dtype     "fp16" or "bf16" of the new tokens
  paged     chunks in pages of a shared pool
  repack    V-median repacking
"""
import math

import torch

from paper_2512_24449_amd import binding, synth

SM_SCALE = 1.0 / math.sqrt(synth.HEAD_DIM)
D = synth.HEAD_DIM
BLOCK = synth.BLOCK_TOKENS


def _case(name, op, batch, kv_heads, q_heads, tokens, new=1, pack=16, k_rel=0.1, v_rel=0.2, dtype="fp16",
          paged=False, repack=False):
    c = dict(op=op, batch=batch, kv_heads=kv_heads, q_heads=q_heads, tokens=tokens, new=new, pack=pack,
             k_rel=k_rel, v_rel=v_rel, dtype=dtype, paged=paged, repack=repack)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest decode step, the paper's way: one head, a short context with a ragged tail
        _case("steps_1x1_1k", "steps", 1, 1, 1, 1000),
        # interactive decoding of one sequence, 32 heads, an ordinary context just past a block edge
        _case("fused_1x32_4k", "fused", 1, 32, 32, 4100),
        # a small batch with grouped queries at the usual long context
        _case("fused_4x8x4_32k", "fused", 4, 8, 32, 32788),
        # one very long document, grouped queries, three steps
        _case("steps_1x8x4_128k", "steps", 1, 8, 32, 131079),
        # a serving batch of a 52-head model at 32 000 tokens: sustained streaming, one pass
        _case("fused_8x52_32k", "fused", 8, 52, 52, 32000),
        # the same through the three steps: the headline benchmark's decode step
        _case("steps_8x52_32k", "steps", 8, 52, 52, 32000),
        # packs of 8 tokens in pages of a pool shared with other sequences, an odd context length
        _case("fused_pack8_paged_4x8x4_10k", "fused", 4, 8, 32, 9999, pack=8, paged=True),
        # fine scales (20 levels): wide chunks in both tensors
        _case("fused_wide_2x32_8k", "fused", 2, 32, 32, 8190, pack=8, k_rel=0.05, v_rel=0.05),
        # an ordinary prompt of one sequence
        _case("prompt_1x32_4k", "append", 1, 32, 32, 0, new=4096),
        # the prompts of the serving batch in one call, the largest append
        _case("prompt_8x52_32k", "append", 8, 52, 52, 0, new=32000),
        # the decode-time append that completes a block: every stream of the batch is flushed
        _case("flush_8x52", "append", 8, 52, 52, 4095),
        # a ragged bf16 prompt into a paged, repacked cache
        _case("prompt_bf16_repack_paged_4x8_3k", "append", 4, 8, 32, 0, new=3001, dtype="bf16", paged=True,
              repack=True),
    ]


MOST_ROWS = 8 * 52 * 32000   # (batch, kv-head, token) rows of the largest listed case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["fused", "steps", "append", "append"])
    batch = rng.choice([1, 1, 2, 3, 4, 8])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 10, 32, 40, 52])
    group = rng.choice([1, 1, 2, 3, 4, 4, 8]) if kv_heads <= 10 else 1
    pack = rng.choice([16, 16, 16, 8])
    k_rel, v_rel = 0.1, 0.2
    if pack == 8:
        k_rel, v_rel = rng.choice([(0.1, 0.2), (0.05, 0.2), (0.1, 0.05), (0.05, 0.05)])
    elif rng.random() < 0.3:
        k_rel, v_rel = rng.choice([(0.1, 0.1), (0.2, 0.25), (0.07, 0.07)])
    repack = rng.random() < 0.15
    paged = rng.random() < 0.25
    dtype = rng.choice(["fp16", "fp16", "bf16"])
    most = min(131072, MOST_ROWS // (batch * kv_heads))
    if op == "append":
        if paged or rng.random() < 0.6:
            tokens, new = 0, _log(rng, 100, min(most, 40000))
        else:
            # a cache at work: what completes its tail, up to one block
            tokens = _log(rng, 200, min(most, 9000))
            new = rng.choice([BLOCK - tokens % BLOCK, rng.randint(1, BLOCK)])
    else:
        tokens, new = _log(rng, 200, most - 64), 1
        if paged:   # pages taken by a flush are not given back by a step that is run again
            tokens -= tokens % BLOCK == BLOCK - 1
    return _case(None, op, batch, kv_heads, kv_heads * group, tokens, new, pack, k_rel, v_rel, dtype, paged, repack)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float16


def _inputs(case, seed):
    total = case["tokens"] + case["new"]
    k, v, q = synth.make_kv(case["batch"], total, case["kv_heads"], case["q_heads"], seed, device="cuda:0")
    return k.to(_dtype(case)), v.to(_dtype(case)), q


def prepare(case, seed):
    k, v, q = _inputs(case, seed)
    held, total = case["tokens"], case["tokens"] + case["new"]
    wide = case["k_rel"] < 1 / 15 or case["v_rel"] < 1 / 15
    pool = None
    if case["paged"]:
        # what the cache can come to hold, at about the worst chunk size of its layout, and some pages more
        chunk = 10240 if wide else 5120
        chunks = 2 * (-(-total // BLOCK)) * case["batch"] * case["kv_heads"]
        pool = binding.PagePool(chunks // (binding.PAGE_BYTES // chunk) + 8)
        pool.pages.zero_()
    cache = binding.PackedKVCache(case["batch"], case["kv_heads"], case["q_heads"], total, k_rel_scale=case["k_rel"],
                                  v_rel_scale=case["v_rel"], pack_size=case["pack"], pool=pool,
                                  repack=binding.REPACK_V_MEDIAN if case["repack"] else binding.REPACK_NONE)
    # buffers that a case returns start from zeros, so that what no call has written is the same every time
    for name in ("k_arena", "v_arena", "k_index", "v_index", "k_token_meta", "v_token_meta", "k_tail", "v_tail",
                 "token_order"):
        cache.tensors[name].zero_()
    if pool is not None:   # the page lists: what the library has not written of them
        cache.kv_cache_release()
    if held:
        cache.kv_compress_append(k[:, :held].contiguous(), v[:, :held].contiguous())
    state = dict(op=case["op"], cache=cache, pool=pool, held=held, q=q,
                 k_new=k[:, held:].contiguous(), v_new=v[:, held:].contiguous())
    return state


def run(state):
    cache, op = state["cache"], state["op"]
    # the cache as it was before the call (host bookkeeping; an empty one gives its pages back), so that
    # the call can be repeated
    if state["held"]:
        cache.kv_cache_restore(state["held"])
    else:
        cache.kv_cache_release()
    cache.kv_compress_append(state["k_new"], state["v_new"])
    tails = {"k_tail": cache.view("k_tail", torch.float16), "v_tail": cache.view("v_tail", torch.float16)}
    if op == "fused":
        return dict(tails, out=cache.kv_decode_attention(state["q"], SM_SCALE))
    if op == "steps":
        p = cache.kv_softmax(cache.kv_k_matvec(state["q"], SM_SCALE))
        return dict(tails, p=p, out=cache.kv_v_matvec(p))
    out = dict(tails)
    names = ["k_index", "v_index", "k_token_meta", "v_token_meta"]
    for name in names:
        out[name] = cache.view(name, torch.int32)
    if state["pool"] is not None:
        out["pages"] = state["pool"].pages
    else:
        out["k_arena"], out["v_arena"] = cache.tensors["k_arena"], cache.tensors["v_arena"]
    if cache.tensors["token_order"].numel():
        out["token_order"] = cache.tensors["token_order"]
    return out


def _packed_bits(case, rel):
    """Packed bits per cached element on these inputs, as measured on the listed cases (2.5 to 2.8 for
    packs of 16, 2.6 to 2.9 for packs of 8, 4.3 to 5.5 for wide chunks)."""
    return 4.9 if rel < 1 / 15 else 2.6 if case["pack"] == 16 else 2.75


def work(case):
    b, h, hq = case["batch"], case["kv_heads"], case["q_heads"]
    held, new = case["tokens"], case["new"]
    if case["op"] == "append":
        # the new tokens in; packed blocks (and their token metadata) or tail tokens out
        tail0 = held % BLOCK
        packed = (tail0 + new) // BLOCK * BLOCK
        rest = (tail0 + new) - packed
        elems_in = 2.0 * b * h * D * (new + (tail0 if packed else 0))
        out_bytes = b * h * D * packed * (_packed_bits(case, case["k_rel"]) + _packed_bits(case, case["v_rel"])) / 8
        return {"bytes": 2 * elems_in + out_bytes + 8.0 * b * packed + 4.0 * b * h * D * rest,
                "flops": 4.0 * elems_in}
    total = held + new
    packed = total // BLOCK * BLOCK
    cached = b * h * D * packed * (_packed_bits(case, case["k_rel"]) + _packed_bits(case, case["v_rel"])) / 8
    cached += 4.0 * b * h * D * (total - packed) + 8.0 * b * packed
    rows = b * hq * (2.0 * D + 4.0 * D)
    if case["op"] == "steps":
        rows += 16.0 * b * hq * total   # scores out, in and out again as weights, in
    return {"bytes": cached + rows + 8.0 * b * h * D * new, "flops": 4.0 * b * hq * D * total}


def tolerance(case):
    if case["op"] == "append":
        return "exact"    # bytes, whole numbers and copies
    # about four times the error against exact(): up to 2.4e-5, and 4.3e-5 with four query heads per
    # kv-head, where the weights of the V product carry 16 bits instead of 20
    return {"rel": 2e-4 if case["q_heads"] >= 4 * case["kv_heads"] else 1e-4}


def _dequantized(x, rel, packed):
    """x: fp16 [B, T, H, D]; the first `packed` tokens as the cache holds them (token-wise scale and minimum in
    fp16, rounded codes), the others as they are; fp64, one batch element at a time."""
    levels = round(1.0 / rel)
    rel32 = torch.tensor(rel, dtype=torch.float32, device=x.device)
    y = x.double()
    if packed:
        t = x[:packed].float()
        flat = t.reshape(packed, -1)
        mn, mx = flat.min(1).values, flat.max(1).values
        scale = (rel32 * (mx - mn)).half().double().view(-1, 1, 1)
        mn = mn.view(-1, 1, 1)
        q = ((t - mn).double() / scale).float().double().round().clamp(0, levels)   # half to even
        y[:packed] = torch.where(scale > 0, q * scale, torch.zeros_like(q)) + mn.double()
    return y


def exact(case, seed):
    if case["op"] == "append":
        return None
    k, v, q = _inputs(case, seed)
    k, v = k.half(), v.half()
    b, h, hq = case["batch"], case["kv_heads"], case["q_heads"]
    g = hq // h
    total = case["tokens"] + case["new"]
    packed = total // BLOCK * BLOCK
    p_all = torch.empty(b, hq, total, dtype=torch.float64, device=k.device) if case["op"] == "steps" else None
    out = torch.empty(b, hq, D, dtype=torch.float64, device=k.device)
    for i in range(b):
        kd, vd = _dequantized(k[i], case["k_rel"], packed), _dequantized(v[i], case["v_rel"], packed)
        order = _storage_order(v[i], case["v_rel"], packed) if case["repack"] else None
        for j in range(hq):
            s = (kd[:, j // g] * q[i, j].double()).sum(1) * SM_SCALE
            p = torch.softmax(s, 0)
            out[i, j] = (p[:, None] * vd[:, j // g]).sum(0)
            if p_all is not None:
                p_all[i, j] = p if order is None else p[order]
        del kd, vd
    tails = {"k_tail": None, "v_tail": None}
    return dict(tails, out=out) if p_all is None else dict(tails, out=out, p=p_all)


def _storage_order(x, rel, packed):
    """V-median repacking: scores come out with the tokens of a block sorted by the lower median of their V codes."""
    total = x.shape[0]
    order = torch.arange(total, device=x.device)
    t = x[:packed].float().reshape(packed, -1)
    mn, mx = t.min(1).values, t.max(1).values
    scale = (torch.tensor(rel, dtype=torch.float32, device=x.device) * (mx - mn)).half().double()
    codes = ((t - mn[:, None]).double() / scale[:, None]).float().round().clamp(0, round(1.0 / rel))
    key = codes.sort(1).values[:, (t.shape[1] - 1) // 2].view(-1, BLOCK)
    sub = torch.sort(key, dim=1, stable=True).indices + BLOCK * torch.arange(key.shape[0], device=x.device)[:, None]
    order[:packed] = sub.reshape(-1)
    return order
