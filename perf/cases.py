"""The work that users of this framework have it do, as cases whose time is measured.

A case is one pass through the public entry points (`paper_2102_03161_amd.binding.Context`): a whole training
step at a freeze boundary k (frozen forward, forward + backward of the active blocks, gradient norms, update),
or the forward-only prefix alone.  `listed()` holds fixed cases from the smallest model to the largest,
`draw(rng)` gives further ones of the same ranges.

Fields of a case:
  arch, head       "vit" (pre-LN, class token) or "bert" (post-LN) with head "qa" (span) or "cls" (first token)
  dtype            "bf16" or "f32"
  L, D, H, F, S    blocks, width, heads, MLP width, tokens per sample; img / patch (ViT), vocab (BERT)
  n_out            classes (2 for the span head)
  B                samples in a batch; cap: the batch size that the context was created for (>= B)
  k                freeze boundary
  source           where the boundary activation comes from when k > 0: "recompute", "hbm" (cached rows in HBM)
                   or "host" (cached rows in pinned host memory, the next batch prefetched during the step)
  micro            micro-batches accumulated into one update
  optimizer        "adamw" or "sgdm"
  mode             "step", or "prefix" (pt_frozen_forward alone)
"""
import math

import numpy as np
import torch

from paper_2102_03161_amd import binding

CHUNK = 1024        # every tensor starts at a multiple of this many elements of the parameter / state arenas
LN_EPS = {"vit": 1e-6, "bert": 1e-12}

TINY = dict(L=2, D=64, H=4, F=256)
SMALL = dict(L=4, D=256, H=4, F=1024)
BASE = dict(L=12, D=768, H=12, F=3072)
LARGE = dict(L=24, D=1024, H=16, F=4096)


def _case(name, arch, size, dtype="bf16", **over):
    c = dict(arch=arch, head="cls" if arch == "vit" else "qa", dtype=dtype, img=0, patch=0, vocab=0, n_out=2, k=0, source="recompute",
             micro=1, optimizer="adamw", mode="step", **size)
    if name:
        c["name"] = name
    c.update(over)
    if arch == "vit":
        c["S"] = (c["img"] // c["patch"]) ** 2 + 1
    c.setdefault("cap", c["B"])
    return c


def _vit_base(name, **over):
    return _case(name, "vit", BASE, **dict(dict(img=224, patch=16, n_out=1000, B=64), **over))


def listed():
    return [
        # The smallest model in fp32, as used for checks and debugging: launch and synchronisation latency.
        _case("vit_tiny_f32_b4", "vit", TINY, dtype="f32", img=32, patch=8, n_out=10, B=4, optimizer="sgdm"),
        # A small bf16 model on a handful of odd-length sequences: few tokens, every tile ragged.
        _case("bert_small_b3_s77", "bert", SMALL, vocab=30522, S=77, B=3),
        # The headline configuration: a full ViT-B/16 step, nothing frozen.
        _vit_base("vit_b16_b64_k0"),
        # The usual state after some epochs: half the blocks frozen, their output served from the cache in HBM.
        _vit_base("vit_b16_b64_k6_cached", k=6, source="hbm"),
        # The pass that fills or bypasses the cache: front end and six frozen blocks, forward only.
        _vit_base("vit_b16_b64_prefix6", k=6, mode="prefix"),
        # The last, partial batch of an epoch.
        _vit_base("vit_b16_b7_k3", k=3, B=7, cap=64),
        # Late phase of a freeze schedule: three active blocks, rows from pinned host memory.
        _vit_base("vit_b16_b128_k9_host", k=9, B=128, source="host"),
        # fp32 mode at full width (debugging a run's precision, small fine-tuning batches).
        _vit_base("vit_b16_f32_b8_k0", dtype="f32", B=8),
        # Span QA, nothing frozen.
        _case("bert_base_qa_b32_k0", "bert", BASE, vocab=30522, S=384, B=32),
        # Sequence classification on short sequences, the embeddings and the lowest block frozen.
        _case("bert_base_cls_b64_s128_k1", "bert", BASE, vocab=30522, S=128, B=64, head="cls", k=1),
        # Ragged batch and sequence, a recomputed frozen prefix, two micro-batches per update, momentum SGD.
        _case("bert_base_qa_b13_s203_acc2", "bert", BASE, vocab=30522, S=203, B=13, k=4, micro=2, optimizer="sgdm"),
        # The largest configuration: BERT-large on 32768 tokens.
        _case("bert_large_cls_b64_s512_k1", "bert", LARGE, vocab=30522, S=512, B=64, head="cls", k=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    arch = rng.choice(["vit", "bert"])
    size = dict(rng.choice([TINY, SMALL, dict(L=12, D=384, H=6, F=1536), BASE, BASE, LARGE]))
    if size["D"] == SMALL["D"]:
        size["L"] = rng.randint(2, 8)
    over = dict(optimizer="sgdm" if rng.random() < 0.2 else "adamw")
    if arch == "vit":
        patch = 8 if size["D"] == TINY["D"] else 16
        over.update(img=patch * rng.randint(4, 22), patch=patch, n_out=_logint(rng, 2, 1000))
        S = (over["img"] // patch) ** 2 + 1
    else:
        S = over["S"] = _logint(rng, 16, 512)
        over.update(vocab=30522, head=rng.choice(["qa", "qa", "cls"]))
        if over["head"] == "cls":
            over["n_out"] = rng.randint(2, 10)
        else:      # deep span QA is chaotic in bf16: two correct runs of 24 blocks are 3e-2 apart, of 12 blocks 1e-2
            size["L"] = min(size["L"], 12)
    L = size["L"]
    over["k"] = 0 if rng.random() < 0.4 and over.get("head") != "cls" else rng.randint(1, L - 1)
    if over["k"]:
        over["source"] = rng.choice(["recompute", "recompute", "hbm", "hbm", "host"])
    if rng.random() < 0.15:
        over["micro"] = rng.randint(2, 4)
    if over["k"] and over["source"] == "recompute" and rng.random() < 0.3:
        over.update(mode="prefix", micro=1)
    # as many samples as stay well below the largest listed case in work (fp32 runs at a fraction of bf16's rate)
    one = _case("", arch, size, dtype=dtype, B=1, **over)
    most = int((3e11 if dtype == "f32" else 2e13) / work(one)["flops"])
    B = _logint(rng, 1, max(1, min(256, most, (1 << 16) // S)))
    if arch == "bert":
        over["vocab"] = _logint(rng, 64, min(32000, 64 + 16 * B * S))
    return _case("", arch, size, dtype=dtype, B=B, **over)


class _State:
    pass


def _config(c):
    w = dict(arch=c["arch"], dtype=c["dtype"], L=c["L"], D=c["D"], H=c["H"], F=c["F"], S=c["S"], n_out=c["n_out"], img=c["img"],
             patch=c["patch"], chans=3 if c["arch"] == "vit" else 0, vocab=c["vocab"], max_pos=max(512, c["S"]) if c["arch"] == "bert" else 0,
             ln_eps=LN_EPS[c["arch"]], B=c["cap"], optimizer=c["optimizer"],
             head="cls" if c["arch"] == "bert" and c["head"] == "cls" else "default")
    n = c["B"] * c["micro"]
    tier = dict(cache_slots=n) if c["source"] == "hbm" else dict(host_slots=n, window_slots=4 * c["cap"]) if c["source"] == "host" else {}
    return binding.make_config(w, grad_accum=c["micro"] > 1, **tier)


def prepare(case, seed):
    c, s = case, _State()
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    s.case, s.ctx = c, binding.Context(_config(c))
    ctx = s.ctx
    # weights N(0, 0.02), LayerNorm gains around 1; bf16 runs start from bf16-representable masters
    tensors = ctx.tensors()
    sizes = [int(np.prod(shape)) for _, _, shape, _, _ in tensors]
    flat = torch.empty(sum(sizes), device="cuda").normal_(0.0, 0.02, generator=gen)
    at, offset, group_at = 0, 0, {}
    for (tid, name, shape, group, _), n in zip(tensors, sizes):
        if name.endswith("_g"):
            flat[at:at + n] += 1.0
        first, _ = group_at.get(group, (offset, 0))
        offset += -(-n // CHUNK) * CHUNK
        group_at[group] = (first, offset)
        at += n
    if c["dtype"] == "bf16":
        flat = flat.to(torch.bfloat16).float()
    host, at = flat.cpu().numpy(), 0
    for (tid, _, shape, _, _), n in zip(tensors, sizes):
        ctx.write_tensor(tid, binding.KIND_PARAM, host[at:at + n].reshape(shape))
        at += n
    # batches resident on the GPU: images N(0, 1) or uniform token ids, uniform labels
    s.batches = []
    B, S = c["B"], c["S"]
    for j in range(c["micro"]):
        if c["arch"] == "vit":
            x = torch.empty(B, 3, c["img"], c["img"], device="cuda").normal_(generator=gen)
            if c["dtype"] == "bf16":
                x = x.to(torch.bfloat16).float()
        else:
            x = torch.randint(0, c["vocab"], (B, S), generator=gen, device="cuda", dtype=torch.int32)
        span = c["head"] == "qa"
        y = torch.randint(0, S if span else c["n_out"], (B, 2) if span else (B,), generator=gen, device="cuda", dtype=torch.int32)
        s.batches.append((x, y, np.arange(j * B, (j + 1) * B) if c["source"] != "recompute" else None))
    if c["k"]:
        ctx.set_freeze_boundary(c["k"])
    for x, _, ids in s.batches:      # the epoch that filled the cache
        if ids is not None:
            ctx.frozen_forward(x, ids)
    # learning rates of the first steps of a linear warm-up: the passes of one state all see nearly the same weights
    s.hp = dict(lr=1e-7, weight_decay=0.01) if c["optimizer"] == "adamw" else dict(lr=1e-4, momentum=0.9)
    if c["mode"] == "prefix":
        return s
    # what a step leaves behind, as views of the context's arenas: the master weights, the gradient of every
    # active layer and its moments (of two layers together where there are more than 12 blocks)
    params, state = ctx.arenas[0].view(torch.float32), ctx.arenas[1].view(torch.float32)
    part = -(-offset * 4 // 256) * 64
    s.out = {"weights": params[:offset]}
    L, k, pair = c["L"], c["k"], -(-c["L"] // 12)
    for lo, hi in ([] if k else [(0, 0)]) + [(1 + l, min(l + pair, L)) for l in range(k, L, pair)] + [(L + 1, L + 1)]:
        for i in range(1, 3 if c["optimizer"] == "adamw" else 2):
            s.out["moment%d_%02d" % (i, lo)] = state[i * part + group_at[lo][0]:i * part + group_at[hi][1]]
    for group, (lo, hi) in group_at.items():
        if group > c["k"] or c["k"] == 0:
            s.out["gradient%02d" % group] = state[lo:hi]
    return s


def run(state):
    s, ctx, micro = state, state.ctx, state.case["micro"]
    if s.case["mode"] == "prefix":
        c = s.case
        at = ctx.frozen_forward(s.batches[0][0]) - ctx.arenas[2].data_ptr()
        dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        n = c["B"] * c["S"] * c["D"]
        return ctx.arenas[2][at:at + n * dt.itemsize].view(dt).view(c["B"], c["S"], c["D"])
    host = s.case["source"] == "host"
    for j, (x, y, ids) in enumerate(s.batches):
        hk = ctx.frozen_forward(x, ids)
        if host:                                   # stage the next batch's rows while this one trains
            ctx.cache_prefetch(s.batches[(j + 1) % micro][2])
        ctx.active_fwd_bwd(hk, y, want_loss=False)
        if micro > 1:
            ctx.accumulate_grads(first=j == 0)
    if micro > 1:
        ctx.finish_accumulation(want_loss=False)
    ctx.layer_grad_norms_begin()
    ctx.optimizer_step(**s.hp)
    out = dict(s.out)
    out["norms"] = ctx.layer_grad_norms_end()      # the freeze rule and the training log read these on the host
    return out


def work(case):
    c = case
    L, D, F, S, k, n = c["L"], c["D"], c["F"], c["S"], c["k"], c["B"] * c["micro"]
    block = 2.0 * S * (4 * D * D + 2 * D * F) + 4.0 * S * S * D
    # under a first-token head the top block needs keys and values of every token, the rest for one row per sample
    first = c["head"] == "cls" and S >= 4
    top = 2.0 * S * 2 * D * D + 2.0 * (2 * D * D + 2 * D * F) + 4.0 * S * D if first else block
    patch = 3 * c["patch"] ** 2
    front = 2.0 * (S - 1) * patch * D if c["arch"] == "vit" else 0.0
    head = 2.0 * D * c["n_out"] * (1 if first else S)
    front_params = patch * D + (2 + S) * D if c["arch"] == "vit" else (c["vocab"] + max(512, S) + 2) * D
    block_params = 4 * D * D + 2 * D * F + 9 * D + F
    x_bytes = n * 3.0 * c["img"] ** 2 * 4 if c["arch"] == "vit" else n * S * 4.0
    e = 2 if c["dtype"] == "bf16" else 4
    rows = float(n * S * D * e)
    if c["mode"] == "prefix":
        return {"flops": n * (front + k * block), "bytes": x_bytes + (front_params + k * block_params) * e + rows}
    cached = k and c["source"] != "recompute"
    flops = 3.0 * ((L - k - 1) * block + top + head) + (0.0 if cached else (front if k else 2 * front) + k * block)
    active = (L - k) * block_params + (D + 1) * c["n_out"] + (0 if k else front_params)
    # per active parameter: weight and moments read and written, the gradient written, the bf16 copy written
    per = (7 if c["optimizer"] == "adamw" else 5) * 4 + (2 if e == 2 else 0)
    byts = active * per + (rows if cached else x_bytes + (front_params + k * block_params) * e * (1 if k else 0))
    return {"flops": n * flops, "bytes": float(byts)}


def tolerance(case):
    # bf16: activations and the operands of every product are rounded to 8 bits at each stage of each block, and
    # one rounding that falls the other way changes all that follow: gradients of two runs whose front ends differ
    # in the last bit of 1 % of the weights are 0.3 to 2.3e-2 apart (2-norm; single elements up to 0.8 of the rms).
    # f32: a batch in another order moves them by 1 to 7e-6.
    return {"rel": 3e-2, "max": 0.99} if case["dtype"] == "bf16" else {"rel": 3e-5}
