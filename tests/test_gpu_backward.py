"""GPU parity of the backward pass (Section 2.3, Eqs. 5 and 6) against the CPU
oracle: the attention forward's log-sum-exp, the attention gradients dQ~ and dV
(both of its terms), and the weight and input gradients."""

import numpy as np
import pytest
import torch

from oracle import keyless as K
from paper_2606_21848_amd import binding as kb
from tests.parity import assert_parity, rowwise_rel, say, to64
from workloads import configs, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"

# N spans one query tile, ragged tails of the 64-row staged tiles and of the
# 128-row work tiles, and a single row.
# Gradient rows can cancel to zero (dQ~ of the first causal row is exactly 0):
# such rows are compared against 1% of the tensor's largest row.
FLOOR = 1e-2

SHAPES = [(2, 200, 4, 2, 128), (1, 77, 2, 2, 64), (2, 1, 4, 1, 128), (1, 300, 8, 2, 64),
          (1, 385, 4, 4, 128)]


def _qvd(B, N, H, G, dk, seed, dtype):
    Qr = synth.normal((B, N, H, dk), seed, 1, 1.0, dtype)
    V = synth.normal((B, N, G, dk), seed, 2, 1.0, dtype)
    dO = synth.normal((B, N, H, dk), seed, 3, 1.0, dtype)
    return Qr, V, dO


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,N,H,G,dk", SHAPES[:3])
def test_attention_forward_lse(lib, dtype, causal, B, N, H, G, dk):
    say(f"attention forward + lse dtype={dtype} causal={causal} B={B} N={N} H={H} G={G} dk={dk}")
    Qr, V, _ = _qvd(B, N, H, G, dk, 71, dtype)
    out, lse = kb.keyless_attention_forward(Qr.to(DEV), V.to(DEV), causal=causal)
    torch.cuda.synchronize()
    ref_lse = K.attention_logsumexp(to64(Qr), to64(V), H, G, dk, causal=causal)
    # out against the oracle's attention of the same routed queries and values
    ref_out = np.zeros((B, N, H, dk))
    q64, v64 = to64(Qr), to64(V)
    for b in range(B):
        for i in range(N):
            seen = i + 1 if causal else N
            for h in range(H):
                ref_out[b, i, h] = K.decode_one(q64[b, i, h], v64[b, :seen, h // (H // G)])
    assert_parity(out, ref_out, dtype, "output")
    # lse is a per-row scalar: compare with an absolute bar scaled like the rows.
    err = np.max(np.abs(lse.cpu().numpy() - ref_lse))
    assert err <= (1e-4 if dtype == torch.float32 else 2e-2), f"lse error {err:.3e}"


@pytest.mark.parametrize("keep_f32", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,N,H,G,dk", SHAPES)
def test_attention_backward_matches_oracle(lib, dtype, causal, B, N, H, G, dk, keep_f32):
    """Both ways of forming rowsum(P * dP): from the forward's fp32 output
    (keep_f32) and, without it, from P and dP in the dQ~ kernel."""
    say(f"attention backward dtype={dtype} causal={causal} B={B} N={N} H={H} G={G} dk={dk} "
        f"keep_f32={keep_f32}")
    Qr, V, dO = _qvd(B, N, H, G, dk, 72, dtype)
    q, v, g = Qr.to(DEV), V.to(DEV), dO.to(DEV)
    o32 = torch.empty((B, N, H, dk), dtype=torch.float32, device=DEV) if keep_f32 else None
    out, lse = kb.keyless_attention_forward(q, v, causal=causal, out_f32=o32)
    dq, dv = kb.keyless_attention_backward(q, v, out, g, lse, causal=causal, out_f32=o32)
    torch.cuda.synchronize()
    ref_dq, ref_dv = K.keyless_attention_backward(to64(Qr), to64(V), to64(dO), H, G, dk,
                                                  causal=causal)
    # Where every dQ~ row cancels (a single causal row), the scale of dV stands in.
    scale = FLOOR * max(np.abs(ref_dq).max(), np.abs(ref_dv).max())
    assert_parity(dq, ref_dq, dtype, "dQ~", FLOOR, scale)
    assert_parity(dv, ref_dv, dtype, "dV", FLOOR, scale)


@pytest.mark.parametrize("keep_f32", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,N,H,G,dk", [(40, 77, 8, 2, 64), (60, 200, 4, 4, 128), (300, 1, 4, 1, 128)])
def test_attention_of_many_sequences(lib, causal, B, N, H, G, dk, keep_f32):
    """Enough query tiles to fill the chip, so that the forms with whole workgroups
    per query tile run, on short ragged sequences."""
    say(f"attention of many sequences B={B} N={N} H={H} G={G} dk={dk} causal={causal} {keep_f32}")
    Qr, V, dO = _qvd(B, N, H, G, dk, 76, torch.bfloat16)
    q, v, g = Qr.to(DEV), V.to(DEV), dO.to(DEV)
    o32 = torch.empty((B, N, H, dk), dtype=torch.float32, device=DEV) if keep_f32 else None
    out, lse = kb.keyless_attention_forward(q, v, causal=causal, out_f32=o32)
    dq, dv = kb.keyless_attention_backward(q, v, out, g, lse, causal=causal, out_f32=o32)
    torch.cuda.synchronize()
    # A score is off by at most 2^-9 tau sum |q v| (q~ rounded to bf16 once more),
    # 0.014 for 128 products of N(0, 1) pairs.
    ref_lse = K.attention_logsumexp(to64(Qr), to64(V), H, G, dk, causal=causal)
    assert np.abs(to64(lse) - ref_lse).max() <= 2e-2
    refs = K.keyless_attention_backward(to64(Qr), to64(V), to64(dO), H, G, dk, causal=causal)
    # Over tens of thousands of rows some dQ~ cancel to a small part of their terms,
    # whose bf16 rounding then shows in that row. So here by the 2-norm of the
    # tensor: q~, P, dS and the result are each rounded by at most 2^-9 of
    # themselves, 4 x 2^-9 = 7.8e-3 in all (a row of one value has dQ~ = 0).
    for got, ref, what in zip((dq, dv), refs, ("dQ~", "dV")):
        off = np.linalg.norm(to64(got) - ref)
        assert off <= 7.8e-3 * np.linalg.norm(refs[1] if N == 1 else ref), what
    if keep_f32:
        assert torch.equal(o32.to(torch.bfloat16), out)


@pytest.mark.parametrize("B,N,H,G,dk", [(1, 255, 4, 1, 64), (2, 193, 6, 2, 128), (1, 700, 3, 3, 128)])
def test_attention_backward_split_sums(lib, B, N, H, G, dk):
    """dV from the fp32 partial sums of several workgroups, and from one workgroup
    per tile when the workspace holds only the row sums: both at the oracle's."""
    say(f"split dV sums B={B} N={N} H={H} G={G} dk={dk}")
    Qr, V, dO = _qvd(B, N, H, G, dk, 75, torch.bfloat16)
    q, v, g = Qr.to(DEV), V.to(DEV), dO.to(DEV)
    rows = -(-B * N * H * 4 // 256) * 256
    assert kb._lib.keyless_attention_backward_workspace_size_for(B, N, H, G, dk, kb.KL_BF16) > rows
    for causal in (True, False):
        out, lse = kb.keyless_attention_forward(q, v, causal=causal)
        _, ref_dv = K.keyless_attention_backward(to64(Qr), to64(V), to64(dO), H, G, dk,
                                                 causal=causal)
        for ws in (None, torch.empty(rows, dtype=torch.uint8, device=DEV)):
            _, dv = kb.keyless_attention_backward(q, v, out, g, lse, causal=causal, workspace=ws)
            torch.cuda.synchronize()
            assert_parity(dv, ref_dv, torch.bfloat16, "dV", FLOOR)


def test_attention_backward_is_deterministic(lib):
    B, N, H, G, dk = 1, 700, 8, 2, 128
    say("attention backward determinism")
    Qr, V, dO = (t.to(DEV) for t in _qvd(B, N, H, G, dk, 73, torch.bfloat16))
    out, lse = kb.keyless_attention_forward(Qr, V)
    first = kb.keyless_attention_backward(Qr, V, out, dO, lse)
    for _ in range(2):
        again = kb.keyless_attention_backward(Qr, V, out, dO, lse)
        torch.cuda.synchronize()
        assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,N,d,H,G,dk", [(2, 130, 256, 4, 2, 64), (1, 64, 128, 2, 1, 128)])
def test_layer_backward_matches_oracle(lib, dtype, B, N, d, H, G, dk):
    """x -> routed queries and values -> attention -> dO: every gradient of the
    layer (dX, dW^Q, dW^R of Eq. 5, dW^V of Eq. 6) against the oracle."""
    say(f"layer backward dtype={dtype} B={B} N={N} d={d} H={H} G={G} dk={dk}")
    x = synth.normal((B, N, d), 74, 1, 1.0, dtype)
    W_Q = synth.normal((d, H * dk), 74, 2, d ** -0.5, dtype)
    W_R = synth.normal((H, dk, dk), 74, 3, dk ** -0.5, dtype)
    W_V = synth.normal((d, G * dk), 74, 4, d ** -0.5, dtype)
    dO = synth.normal((B, N, H, dk), 74, 5, 1.0, dtype)
    xs, wq, wr, wv, g = (t.to(DEV) for t in (x, W_Q, W_R, W_V, dO))
    _, qr, v = kb.keyless_prefill(xs, wq, wr, wv, H, G, return_qv=True)
    out, lse = kb.keyless_attention_forward(qr, v)
    dq, dv = kb.keyless_attention_backward(qr, v, out, g, lse)
    grads = kb.keyless_weight_gradients(xs, wq, wr, wv, dq, dv, H, G)
    torch.cuda.synchronize()
    ref = K.keyless_backward(to64(x), to64(W_Q), to64(W_R), to64(W_V), to64(dO), H, G, dk)
    # The attention backward against the oracle's, on the routed queries and
    # values the GPU's attention consumed (the same bits, copied back).
    ref_dq, ref_dv = K.keyless_attention_backward(to64(qr), to64(v), to64(dO), H, G, dk)
    assert_parity(dq, ref_dq, dtype, "dQ~", FLOOR)
    assert_parity(dv, ref_dv, dtype, "dV", FLOOR)
    # End to end against the float64 oracle of the whole layer: the fp32 path
    # meets its bar; the bf16 path also rounds the folded weights, the routed
    # queries and the values once each, which moves dQ~ by about the bf16 bar
    # (the softmax backward's dP - rowsum subtraction amplifies it), so there the
    # figure is reported, not asserted.
    e2e_dq = rowwise_rel(dq, ref["dQr"], FLOOR)
    e2e_dv = rowwise_rel(dv, ref["dV"], FLOOR)
    say(f"  end to end against the float64 layer oracle: dQ~ {e2e_dq:.3e}, dV {e2e_dv:.3e}")
    if dtype == torch.float32:
        assert_parity(dq, ref["dQr"], dtype, "dQ~ end to end", FLOOR)
        assert_parity(dv, ref["dV"], dtype, "dV end to end", FLOOR)
    assert_parity(grads["dW_R"], ref["dW_R"], dtype, "dW^R (Eq. 5)", FLOOR)
    assert_parity(grads["dW_V"].T, ref["dW_V"].T, dtype, "dW^V (Eq. 6)", FLOOR)
    assert_parity(grads["dW_Q"].T, ref["dW_Q"].T, dtype, "dW^Q", FLOOR)
    assert_parity(grads["dX"], ref["dX"], dtype, "dX", FLOOR)
    # The projection gradients against the oracle's on the attention gradients
    # the GPU produced (the same bits).
    same = K.keyless_projection_gradients(to64(x), to64(W_Q), to64(W_R), to64(W_V), to64(dq),
                                          to64(dv), H, G, dk)
    assert_parity(grads["dW_R"], same["dW_R"], dtype, "dW^R, same inputs", FLOOR)
    assert_parity(grads["dW_V"].T, same["dW_V"].T, dtype, "dW^V, same inputs", FLOOR)
    assert_parity(grads["dW_Q"].T, same["dW_Q"].T, dtype, "dW^Q, same inputs", FLOOR)
    assert_parity(grads["dX"], same["dX"], dtype, "dX, same inputs", FLOOR)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,N,d,H,G,dk", [(2, 130, 256, 4, 2, 64), (1, 100, 200, 2, 2, 64),
                                          (3, 33, 320, 4, 4, 128), (1, 1, 64, 2, 1, 64)])
def test_weight_gradients_match_oracle(lib, dtype, B, N, d, H, G, dk):
    """keyless_weight_gradients on given attention gradients against the oracle
    on the same inputs: token counts that are not multiples of 64 (padded for
    the contractions over tokens), d_model that is not (padded for dW^R),
    grouped values, and a single token."""
    say(f"weight gradients dtype={dtype} B={B} N={N} d={d} H={H} G={G} dk={dk}")
    x = synth.normal((B, N, d), 92, 1, 1.0, dtype)
    W_Q = synth.normal((d, H * dk), 92, 2, d ** -0.5, dtype)
    W_R = synth.normal((H, dk, dk), 92, 3, dk ** -0.5, dtype)
    W_V = synth.normal((d, G * dk), 92, 4, d ** -0.5, dtype)
    dq = synth.normal((B, N, H, dk), 92, 5, 1.0, dtype)
    dv = synth.normal((B, N, G, dk), 92, 6, 1.0, dtype)
    grads = kb.keyless_weight_gradients(*(t.to(DEV) for t in (x, W_Q, W_R, W_V, dq, dv)), H, G)
    torch.cuda.synchronize()
    ref = K.keyless_projection_gradients(to64(x), to64(W_Q), to64(W_R), to64(W_V), to64(dq),
                                         to64(dv), H, G, dk)
    assert_parity(grads["dW_R"], ref["dW_R"], dtype, "dW^R (Eq. 5)", FLOOR)
    assert_parity(grads["dW_V"].T, ref["dW_V"].T, dtype, "dW^V (Eq. 6)", FLOOR)
    assert_parity(grads["dW_Q"].T, ref["dW_Q"].T, dtype, "dW^Q", FLOOR)
    assert_parity(grads["dX"], ref["dX"], dtype, "dX", FLOOR)


def test_weight_gradients_128_wide_tiles(lib):
    """Products whose outputs take the 128-wide GEMM tiles (one term, two terms)."""
    B, N, d, H, G, dk = 2, 901, 1472, 22, 2, 64
    say("weight gradients, 128-wide tiles")
    x, dq, dv = (synth.normal(s, 93, i) for i, s in enumerate(((B, N, d), (B, N, H, dk), (B, N, G, dk))))
    W_Q = synth.normal((d, H * dk), 93, 4, d ** -0.5)
    W_R = synth.normal((H, dk, dk), 93, 5, dk ** -0.5)
    W_V = synth.normal((d, G * dk), 93, 6, d ** -0.5)
    got = kb.keyless_weight_gradients(*(t.to(DEV) for t in (x, W_Q, W_R, W_V, dq, dv)), H, G)
    torch.cuda.synchronize()
    ref = K.keyless_projection_gradients(*(to64(t) for t in (x, W_Q, W_R, W_V, dq, dv)), H, G, dk)
    for name, g in got.items():
        assert_parity(g, ref[name], torch.bfloat16, name, FLOOR)


@pytest.mark.parametrize("wanted", [("dW_Q",), ("dW_V",), ("dW_R",), ("dX",), ("dW_Q", "dX"),
                                    ("dW_R", "dW_V")])
def test_weight_gradients_subsets(lib, wanted):
    """Any of the four outputs may be skipped (NULL): each requested subset is
    bit-equal to the same outputs of the full call, and skipped ones are not
    written."""
    B, N, d, H, G, dk = 1, 192, 256, 4, 2, 64
    say(f"weight gradients subset {wanted}")
    bf = torch.bfloat16
    x, W_Q, W_R, W_V = (synth.normal(sh, 93, i + 1, sc, bf).to(DEV) for i, (sh, sc) in enumerate(
        [((B, N, d), 1.0), ((d, H * dk), d ** -0.5), ((H, dk, dk), dk ** -0.5),
         ((d, G * dk), d ** -0.5)]))
    dq = synth.normal((B, N, H, dk), 93, 5, 1.0, bf).to(DEV)
    dv = synth.normal((B, N, G, dk), 93, 6, 1.0, bf).to(DEV)
    full = kb.keyless_weight_gradients(x, W_Q, W_R, W_V, dq, dv, H, G)
    outs = {k: torch.full_like(v, 7.0) for k, v in full.items()}
    ws = torch.empty(kb._lib.keyless_weight_gradients_workspace_size(B, N, d, H, G, dk, kb.KL_BF16),
                     dtype=torch.uint8, device=DEV)
    ptr = lambda k: kb._ptr(outs[k]) if k in wanted else None
    kb._check(kb._lib.keyless_weight_gradients(
        kb._ptr(x), kb._ptr(W_Q), kb._ptr(W_R), kb._ptr(W_V), kb._ptr(dq), kb._ptr(dv), B, N, d, H,
        G, dk, kb.KL_BF16, ptr("dW_Q"), ptr("dW_R"), ptr("dW_V"), ptr("dX"), kb._ptr(ws),
        ws.numel(), kb._stream(x)))
    torch.cuda.synchronize()
    for k in full:
        if k in wanted:
            assert torch.equal(outs[k], full[k]), f"{k} differs from the full call"
        else:
            assert bool((outs[k] == 7.0).all()), f"{k} was written although not requested"


def test_weight_gradients_full_size_sampled(lib):
    """keyless_weight_gradients at the size the benchmark times (8192 tokens,
    d_model 4096, 32 + 32 heads x 128, bf16): the weight gradients of two query
    heads and two value groups over every token, and dX on sampled tokens,
    against the oracle on the same inputs. Each of those depends only on its own
    heads (or its own token), so the oracle runs on that slice."""
    B, N, d, H, G, dk = 1, 8192, 4096, 32, 32, 128
    say(f"weight gradients full size B={B} N={N} d={d} H={H} G={G} dk={dk}")
    bf = torch.bfloat16
    x = synth.normal((B, N, d), 91, 1, 1.0, bf)
    W_Q = synth.normal((d, H * dk), 91, 2, d ** -0.5, bf)
    W_R = synth.normal((H, dk, dk), 91, 3, dk ** -0.5, bf)
    W_V = synth.normal((d, G * dk), 91, 4, d ** -0.5, bf)
    dq = synth.normal((B, N, H, dk), 91, 5, 1.0, bf)
    dv = synth.normal((B, N, G, dk), 91, 6, 1.0, bf)
    grads = kb.keyless_weight_gradients(*(t.to(DEV) for t in (x, W_Q, W_R, W_V, dq, dv)), H, G)
    torch.cuda.synchronize()
    heads = [0, H - 1]
    qcols = np.concatenate([np.arange(h * dk, (h + 1) * dk) for h in heads])
    ref = K.keyless_projection_gradients(to64(x), to64(W_Q)[:, qcols], to64(W_R)[heads],
                                         to64(W_V)[:, qcols], to64(dq)[:, :, heads],
                                         to64(dv)[:, :, heads], len(heads), len(heads), dk)
    assert_parity(grads["dW_Q"][:, qcols].T, ref["dW_Q"].T, bf, "dW^Q, two heads", FLOOR)
    assert_parity(grads["dW_R"][heads], ref["dW_R"], bf, "dW^R (Eq. 5), two heads", FLOOR)
    assert_parity(grads["dW_V"][:, qcols].T, ref["dW_V"].T, bf, "dW^V (Eq. 6), two groups", FLOOR)
    rows = sorted(set([0, N - 1] + synth.uniform_int(14, 1, N - 2, 91, 7).tolist()))
    refx = K.keyless_projection_gradients(to64(x)[:, rows], to64(W_Q), to64(W_R), to64(W_V),
                                          to64(dq)[:, rows], to64(dv)[:, rows], H, G, dk)
    assert_parity(grads["dX"][:, rows], refx["dX"], bf, "dX, sampled tokens", FLOOR)


def test_backward_full_size_sampled(lib):
    """The measured backward workload (8192 tokens, 32 heads x 128, causal, the
    routed queries and values of the prefill workload's layer): 24 sampled dQ~
    rows anywhere and the dV rows of the last 48 positions against the oracle."""
    say("backward full size")
    c = configs.backward_bf16(device=DEV)
    o32 = torch.empty(c["q"].shape, dtype=torch.float32, device=DEV)
    out, lse = kb.keyless_attention_forward(c["q"], c["v"], out_f32=o32)
    dq, dv = kb.keyless_attention_backward(c["q"], c["v"], out, c["dout"], lse, out_f32=o32)
    torch.cuda.synchronize()
    assert torch.isfinite(dq.float()).all() and torch.isfinite(dv.float()).all()
    N = c["N"]
    rq = sorted(set([0, N - 1] + synth.uniform_int(22, 1, N - 2, 8, 50).tolist()))
    rv = list(range(N - 48, N))
    ref_dq, ref_dv = K.keyless_attention_backward_rows(to64(c["q"]), to64(c["v"]), to64(c["dout"]),
                                                      c["H"], c["G"], c["d_head"], rq, rv)
    assert_parity(dq[0, rq], ref_dq, torch.bfloat16, "sampled dQ~ rows", FLOOR)
    assert_parity(dv[0, rv], ref_dv, torch.bfloat16, "last dV rows", FLOOR)
