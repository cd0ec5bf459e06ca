"""The library's work that is timed and compared, case by case.

Each case is one call (or the few calls that belong together) that a program
using the library makes: decode steps over a value-only cache, prompt prefill,
cross-attention, and the forward and backward of training. The sizes are those
of this repository's workloads and tests (32 heads x 128 at d_model 4096, the
paper's testbed layer of 12 query heads over 2 value heads, the small fp32
layer), or lie between them.

A case is a dict; "kind" selects the calls:

  decode    keyless_decode_append, contiguous bf16 cache (one serving step)
  ragged    keyless_decode, contiguous cache, ragged lengths
  paged     keyless_decode, paged cache in random block order, ragged lengths
  step      keyless_decode_project + keyless_decode: a layer's whole decode step
  latent    keyless_latent_decode over one shared latent
  prefill   keyless_prefill_packed (bf16) or keyless_prefill (fp32, raw weights)
  cross     keyless_cross_attention_packed
  attn      keyless_attention_forward + keyless_attention_backward
  layer     a training step's layer: projections, attention, and every gradient
"""

import math

import torch

from paper_2606_21848_amd import binding as kb

BF16, F32 = "bf16", "f32"
DTYPES = {BF16: torch.bfloat16, F32: torch.float32}
DEV = "cuda"

# (d_model, query heads, value groups, d_head)
TESTBED = (1536, 12, 2, 128)   # the paper's decode testbed: 12 heads over 2 value heads
LARGE = (4096, 32, 32, 128)    # the prefill workload's layer
LARGE_GQA = (4096, 32, 8, 128)  # the paged workload's heads
MEDIUM = (1024, 8, 8, 128)     # the paper's GPT-2 heads
TINY = (256, 4, 4, 64)         # the small fp32 layer


def _case(kind, dtype, dims, **more):
    d_model, H, G, d = dims
    return dict(kind=kind, dtype=dtype, d_model=d_model, H=H, G=G, d=d, **more)


def listed():
    return [
        # One token of one layer at batch 1 over a 2048-row cache: the paper's
        # decode setting, and the smallest call of all.
        dict(_case("decode", BF16, TESTBED, B=1, L=2048), name="decode_b1"),
        # fp32 serving of a small model: a few sequences of uneven length.
        dict(_case("ragged", F32, (512, 8, 8, 64), B=6, L=2048, lo=5, hi=1500), name="decode_f32"),
        # A serving batch over a paged cache with lengths of 1k to 32k rows.
        dict(_case("paged", BF16, LARGE_GQA, B=64, L=32768, lo=1024, hi=32768), name="paged_b64"),
        # A layer's decode step at batch 8: projections, append and decode.
        dict(_case("step", BF16, LARGE, B=8, L=4096), name="step_b8"),
        # Decode over a latent cache that all 32 heads share.
        dict(_case("latent", BF16, (4096, 32, 1, 128), B=32, L=16384), name="latent_b32"),
        # The small fp32 layer's prompt, from raw weights.
        dict(_case("prefill", F32, TINY, B=1, N=128), name="prefill_f32"),
        # A user's prompt of odd length through a 1.5B-model layer.
        dict(_case("prefill", BF16, TESTBED, B=1, N=517), name="prompt_517"),
        # A long prompt through a large layer.
        dict(_case("prefill", BF16, LARGE, B=1, N=8192), name="prefill_8k"),
        # Cross-attention of decoder tokens to encoder outputs.
        dict(_case("cross", BF16, LARGE, B=4, N=1024, Nb=4096), name="cross_4x1k"),
        # Long-context training: the attention's forward and backward.
        dict(_case("attn", BF16, LARGE, B=1, N=8192), name="attn_8k"),
        # A bf16 training step of a grouped layer on two sequences of 1000 tokens.
        dict(_case("layer", BF16, TESTBED, B=2, N=1000), name="layer_bf16"),
        # The same in fp32, the precision of the paper's 12-layer training.
        dict(_case("layer", F32, MEDIUM, B=1, N=512), name="layer_f32"),
    ]


def _log(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], odd ones included."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("decode", "ragged", "paged", "step", "latent", "prefill", "prefill", "cross",
                       "attn", "layer", "layer"))
    if kind == "decode":
        dims = rng.choice((TESTBED, MEDIUM, LARGE, LARGE_GQA))
        B = _log(rng, 1, 32)
        L = _log(rng, 128, min(32768, 2 ** 17 // (B * max(1, dims[2] // 8))))
        return _case(kind, BF16, dims, B=B, L=L)
    if kind == "ragged":
        dims = rng.choice((TINY, (512, 8, 8, 64), (1024, 16, 4, 64), MEDIUM))
        hi = _log(rng, 64, 8192)
        return _case(kind, rng.choice((F32, F32, BF16)), dims, B=_log(rng, 1, 24), L=hi + 100, lo=1,
                     hi=hi)
    if kind == "paged":
        dims = rng.choice((TESTBED, LARGE_GQA, (4096, 32, 2, 128)))
        hi = _log(rng, 256, 32768)
        return _case(kind, BF16, dims, B=_log(rng, 2, 64), L=(hi + 15) // 16 * 16,
                     lo=max(1, hi // rng.choice((2, 8, 32))), hi=hi)
    if kind == "step":
        return _case(kind, BF16, rng.choice((TESTBED, MEDIUM, LARGE, LARGE_GQA)), B=_log(rng, 1, 32),
                     L=_log(rng, 128, 4096))
    if kind == "latent":
        H = rng.choice((16, 32))
        return _case(kind, BF16, (4096, H, 1, 128), B=_log(rng, 1, 32), L=_log(rng, 256, 16384))
    if kind == "prefill":
        if rng.random() < 0.35:
            dims = rng.choice((TINY, (512, 8, 8, 64), MEDIUM))
            return _case(kind, F32, dims, B=rng.choice((1, 2)), N=_log(rng, 16, 600))
        dims = rng.choice((TESTBED, MEDIUM, LARGE, LARGE_GQA))
        B = rng.choice((1, 1, 2, 4))
        return _case(kind, BF16, dims, B=B, N=_log(rng, 32, 8192 // B))
    if kind == "cross":
        return _case(kind, BF16, rng.choice((TESTBED, MEDIUM, LARGE)), B=rng.choice((1, 2, 4)),
                     N=_log(rng, 32, 1024), Nb=_log(rng, 64, 4096))
    if kind == "attn":
        dims = rng.choice((TESTBED, MEDIUM, LARGE, LARGE_GQA))
        B = rng.choice((1, 1, 2, 4))
        return _case(kind, BF16, dims, B=B, N=_log(rng, 128, 8192 // B))
    if rng.random() < 0.5:
        dims = rng.choice((TINY, (512, 8, 8, 64), MEDIUM))
        return _case(kind, F32, dims, B=rng.choice((1, 2)), N=_log(rng, 32, 700))
    dims = rng.choice((TESTBED, MEDIUM, LARGE_GQA))
    B = rng.choice((1, 2, 4))
    return _case(kind, BF16, dims, B=B, N=_log(rng, 64, 4096 // B))


class _Draw:
    """Normal tensors in the case's dtype, made on the GPU from the seed."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))
        self.dtype = dtype

    def normal(self, *shape, std=1.0):
        t = torch.empty(shape, dtype=self.dtype, device=DEV)
        t.normal_(0.0, std, generator=self.gen)
        return t

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi + 1, (n,), generator=self.gen, device=DEV, dtype=torch.int32)


def _weights(c, r):
    std = 1.0 / math.sqrt(c["d_model"])
    H, G, d = c["H"], c["G"], c["d"]
    return (r.normal(c["d_model"], H * d, std=std), r.normal(H, d, d, std=1.0 / math.sqrt(d)),
            r.normal(c["d_model"], G * d, std=std))


def _decode_buffers(s, c):
    """The output and workspace that a serving loop keeps."""
    s["out"] = torch.empty((c["B"], c["H"], c["d"]), dtype=s["q"].dtype, device=DEV)
    s["ws"] = torch.empty(max(kb.decode_workspace_bytes(s["vc"], c["B"], c["H"]), 256),
                          dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c = case
    kind, dtype = c["kind"], DTYPES[c["dtype"]]
    B, H, G, d, dm = c["B"], c["H"], c["G"], c["d"], c["d_model"]
    r = _Draw(seed, dtype)
    s = dict(kind=kind, dtype=c["dtype"], H=H, G=G)
    if kind in ("decode", "step"):
        s["cache"] = r.normal(B, G, c["L"], d)
        s["vc"] = kb.ValueCache(s["cache"])
        s["before"] = torch.full((B,), c["L"] - 1, dtype=torch.int32, device=DEV)
        s["lengths"] = s["before"] + 1
        if kind == "decode":
            s["q"], s["v_new"] = r.normal(B, H, d), r.normal(B, G, d)
        else:
            s["x"] = r.normal(B, dm)
            s["packed"] = kb.keyless_pack_weights(*_weights(c, r), H, G)
            s["q"] = torch.empty((B, H, d), dtype=dtype, device=DEV)
        _decode_buffers(s, c)
    elif kind == "ragged":
        s["cache"] = r.normal(B, G, c["L"], d)
        s["vc"] = kb.ValueCache(s["cache"])
        s["lengths"] = r.ints(c["lo"], c["hi"], B)
        s["q"] = r.normal(B, H, d)
        _decode_buffers(s, c)
    elif kind == "paged":
        bs = 16
        lengths = r.ints(c["lo"], c["hi"], B)
        nblk = ((lengths + bs - 1) // bs).tolist()
        used = sum(nblk)
        width = (c["L"] + bs - 1) // bs
        perm = torch.randperm(used, generator=r.gen, device=DEV).to(torch.int32)
        table = torch.full((B, width), used, dtype=torch.int32, device=DEV)
        at = 0
        for b, n in enumerate(nblk):
            table[b, :n] = perm[at:at + n]
            at += n
        s["cache"] = r.normal(used + 1, G, bs, d)
        s["table"], s["lengths"] = table, lengths
        s["vc"] = kb.ValueCache(s["cache"], table)
        s["q"] = r.normal(B, H, d)
        _decode_buffers(s, c)
    elif kind == "latent":
        s["cache"] = r.normal(B, G, c["L"], 128)
        s["vc"] = kb.ValueCache(s["cache"])
        s["lengths"] = torch.full((B,), c["L"], dtype=torch.int32, device=DEV)
        s["q"] = r.normal(B, H, d)
        s["W_post"] = r.normal(H, 128, d, std=1.0 / math.sqrt(d))
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = torch.empty(kb.latent_decode_workspace_bytes(s["vc"], B, H, d), dtype=torch.uint8,
                              device=DEV)
    elif kind == "prefill":
        s["x"] = r.normal(B, c["N"], dm)
        s["w"] = _weights(c, r)
        if c["dtype"] == BF16:  # an inference program packs its weights once
            s["packed"] = kb.keyless_pack_weights(*s["w"], H, G)
    elif kind == "cross":
        s["xa"], s["xb"] = r.normal(B, c["N"], dm), r.normal(B, c["Nb"], dm)
        s["w"] = _weights(c, r)
        s["packed"] = kb.keyless_pack_weights(*s["w"], H, G)
    elif kind == "attn":
        s["q"], s["v"], s["dout"] = (r.normal(B, c["N"], H, d), r.normal(B, c["N"], G, d),
                                     r.normal(B, c["N"], H, d))
    elif kind == "layer":
        s["x"] = r.normal(B, c["N"], dm)
        s["w"] = _weights(c, r)
        s["dout"] = r.normal(B, c["N"], H, d)
    else:
        raise ValueError(kind)
    return s


def run(state):
    s = state
    kind, H, G = s["kind"], s["H"], s["G"]
    if kind == "decode":
        out = kb.keyless_decode_append(s["q"], s["v_new"], s["vc"], s["before"], out=s["out"],
                                       workspace=s["ws"])
        return dict(out=out, cache=s["cache"])
    if kind in ("ragged", "paged"):
        return dict(out=kb.keyless_decode(s["q"], s["vc"], s["lengths"], out=s["out"],
                                          workspace=s["ws"]))
    if kind == "step":
        q = kb.keyless_decode_project(s["x"], s["packed"], H, G, cache=s["vc"],
                                      lengths_before=s["before"], q_routed_out=s["q"])
        out = kb.keyless_decode(q, s["vc"], s["lengths"], out=s["out"], workspace=s["ws"])
        return dict(out=out, q=q, cache=s["cache"])
    if kind == "latent":
        return dict(out=kb.keyless_latent_decode(s["q"], s["W_post"], s["vc"], s["lengths"],
                                                 out=s["out"], workspace=s["ws"]))
    if kind == "prefill":
        if s["dtype"] == BF16:
            out, q, v = kb.keyless_prefill_packed(s["x"], s["packed"], H, G, return_qv=True)
        else:
            out, q, v = kb.keyless_prefill(s["x"], *s["w"], H, G, return_qv=True)
        return dict(out=out, q=q, v=v)
    if kind == "cross":
        out, q, v = kb.keyless_cross_attention_packed(s["xa"], s["xb"], s["packed"], H, G,
                                                      return_qv=True)
        return dict(out=out, q=q, v=v)
    if kind == "attn":
        q = s["q"]
        o32 = torch.empty(q.shape, dtype=torch.float32, device=q.device)
        out, lse = kb.keyless_attention_forward(q, s["v"], out_f32=o32)
        dq, dv = kb.keyless_attention_backward(q, s["v"], out, s["dout"], lse, out_f32=o32)
        return dict(out=out, lse=lse, dq=dq, dv=dv)
    # layer: the forward keeps q~, v, the fp32 output and the log-sum-exp for the backward.
    x, w = s["x"], s["w"]
    _, q, v = kb.keyless_prefill(x, *w, H, G, return_qv=True)
    o32 = torch.empty(q.shape, dtype=torch.float32, device=q.device)
    out, lse = kb.keyless_attention_forward(q, v, out_f32=o32)
    dq, dv = kb.keyless_attention_backward(q, v, out, s["dout"], lse, out_f32=o32)
    grads = kb.keyless_weight_gradients(x, *w, dq, dv, H, G)
    return dict(out=out, q=q, v=v, dq=dq, dv=dv, **grads)


def work(case):
    c = case
    kind = c["kind"]
    e = 2 if c["dtype"] == BF16 else 4
    B, H, G, d, dm = c["B"], c["H"], c["G"], c["d"], c["d_model"]
    if kind in ("decode", "step", "ragged", "paged", "latent"):
        rows = B * (c["L"] if kind in ("decode", "step", "latent") else (c["lo"] + c["hi"]) / 2)
        nbytes = rows * G * d * e + 2 * B * H * d * e + (B * G * d * e if kind == "decode" else 0)
        flops = 4 * rows * H * d
        if kind == "step":
            nbytes += (H + G) * d * dm * e + B * dm * e + B * G * d * e
            flops += 2 * B * dm * (H + G) * d
        if kind == "latent":
            nbytes += H * 128 * d * e
            flops += 4 * B * H * 128 * d
        return dict(bytes=nbytes, flops=flops)
    N, Nb = c["N"], c.get("Nb", c["N"])
    weights = (H + G) * d * dm
    pairs = N * Nb if kind == "cross" else N * (N + 1) // 2
    qo, vv = B * N * H * d, B * Nb * G * d
    attend = 4 * B * H * d * pairs
    if kind in ("prefill", "cross"):
        x = B * N * dm + (B * Nb * dm if kind == "cross" else 0)
        project = 2 * dm * (qo + vv)
        if c["dtype"] == F32:
            weights += H * d * d
            project += 2 * dm * H * d * d
        return dict(bytes=e * (x + weights + 2 * qo + vv), flops=project + attend)
    backward = 10 * B * H * d * pairs
    if kind == "attn":
        return dict(bytes=e * (4 * qo + 2 * vv) + 4 * B * H * N, flops=attend + backward)
    # X W^Q, X W^V, dQ~ W^R^T, Q^T dQ~, X^T dQ, X^T dV, dQ W^Q^T, dV W^V^T and the routing fold.
    grads = 2 * dm * (3 * qo + 2 * vv) + 4 * qo * d
    forward = 2 * dm * (qo + vv) + 2 * dm * H * d * d
    return dict(bytes=e * (2 * B * N * dm + 2 * (weights + H * d * d) + 4 * qo + 2 * vv),
                flops=forward + attend + backward + grads)


def tolerance(case):
    # bf16: every output is rounded to bf16 (2^-9 each, about 1.7e-3 in the
    # 2-norm) and the values it is formed from (weights, q~, v, P, dS) once more.
    # fp32: sums of a few hundred to a few thousand terms; the gradients, at the
    # end of the chain, are about 1.3e-6 from 64 bits.
    if case["dtype"] == BF16:
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 5e-6, "max": 2e-4}


def _attend64(q, v, scale, mask):
    """out, lse of one head in 64 bits: q [N, d], v [Nk, d]."""
    z = (q @ v.T) * scale
    if mask is not None:
        z.masked_fill_(mask, float("-inf"))
    lse = torch.logsumexp(z, 1)
    z.sub_(lse[:, None]).exp_()
    return z @ v, lse, z



def exact(case, seed):
    c = case
    s = prepare(case, seed)
    kind, H, G, d, B = c["kind"], c["H"], c["G"], c["d"], c["B"]
    R, f = H // G, torch.float64
    scale = 1.0 / math.sqrt(d)
    if kind in ("decode", "step", "ragged", "paged", "latent"):
        got = {}
        cache = s["cache"]
        if kind == "step":
            p = s["packed"].to(f)
            qv = s["x"].to(f) @ p.T
            q, vn = qv[:, :H * d].reshape(B, H, d), qv[:, H * d:].reshape(B, G, d)
            got["q"] = q
        else:
            q = s["q"].to(f)
            vn = s["v_new"].to(f) if kind == "decode" else None
        if vn is not None:
            cache = cache.clone()
            cache[:, :, -1] = vn.to(cache.dtype)
            got["cache"] = cache
        if kind == "latent":
            W = s["W_post"].to(f)
            q = torch.stack([q[:, h] @ W[h].T for h in range(H)], 1)
        out = torch.empty((B, H, cache.shape[3]), dtype=f, device=DEV)
        for b in range(B):
            n = int(s["lengths"][b])
            if kind == "paged":
                blocks = s["table"][b, :(n + 15) // 16].long()
                rows = cache[blocks].permute(1, 0, 2, 3).reshape(G, -1, d)[:, :n]
            else:
                rows = cache[b, :, :n]
            for g in range(G):
                v = rows[g].to(f)
                if vn is not None:
                    v[n - 1] = vn[b, g]
                out[b, g * R:(g + 1) * R] = torch.softmax((q[b, g * R:(g + 1) * R] @ v.T) * scale, 1) @ v
        if kind == "latent":
            out = torch.stack([out[:, h] @ W[h] for h in range(H)], 1)
        return dict(out=out, **got)
    N, Nb = c["N"], c.get("Nb", c["N"])
    mask = None
    if kind != "cross":
        mask = torch.ones((N, N), dtype=torch.bool, device=DEV).triu_(1)
    got = {}
    if kind == "attn":
        q, v = s["q"].to(f), s["v"].to(f)
    else:
        xa = (s["xa"] if kind == "cross" else s["x"]).to(f).reshape(-1, c["d_model"])
        xb = s["xb"].to(f).reshape(-1, c["d_model"]) if kind == "cross" else xa
        WQ, WR, WV = (w.to(f) for w in s["w"])
        WQR = torch.cat([WQ[:, h * d:(h + 1) * d] @ WR[h] for h in range(H)], 1)
        q, v = (xa @ WQR).reshape(B, N, H, d), (xb @ WV).reshape(B, Nb, G, d)
        got["q"], got["v"] = q, v
    out = torch.empty((B, N, H, d), dtype=f, device=DEV)
    back = kind in ("attn", "layer")
    if back:
        dout = s["dout"].to(f)
        dq, dv = torch.empty_like(q), torch.zeros_like(v)
    lses = torch.empty((B, H, N), dtype=f, device=DEV)
    for b in range(B):
        for h in range(H):
            qh, vh = q[b, :, h].contiguous(), v[b, :, h // R].contiguous()
            o, lse, p = _attend64(qh, vh, scale, mask)
            out[b, :, h], lses[b, h] = o, lse
            if back:
                g = dout[b, :, h].contiguous()
                ds = (g @ vh.T).sub_((g * o).sum(1)[:, None]).mul_(p).mul_(scale)
                dq[b, :, h] = ds @ vh
                dv[b, :, h // R] += p.T @ g + ds.T @ qh
    got["out"] = out
    if back:
        got["dq"], got["dv"] = dq, dv
    if kind == "attn":
        got["lse"] = lses
    if kind == "layer":
        dqf, dvf = dq.reshape(-1, H, d), dv.reshape(-1, G * d)
        dQ = torch.cat([dqf[:, h] @ WR[h].T for h in range(H)], 1)
        Q = (xa @ WQ).reshape(-1, H, d)
        got["dW_Q"], got["dW_V"] = xa.T @ dQ, xa.T @ dvf
        got["dW_R"] = torch.stack([Q[:, h].T @ dqf[:, h] for h in range(H)])
        got["dX"] = (dQ @ WQ.T + dvf @ WV.T).reshape(B, N, -1)
    return got
