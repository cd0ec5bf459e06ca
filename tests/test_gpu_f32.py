"""GPU parity of the fp32 matrix-core kernels (the GEMM in fp32 arithmetic, the
fp32 attention forward and backward) at the edges of their tiles and in every
way they load an operand, against the CPU oracle."""

import numpy as np
import pytest
import torch

from oracle import keyless as K
from paper_2606_21848_amd import binding as kb
from tests.parity import assert_parity, rowwise_rel, say, to64
from workloads import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
F32 = torch.float32


def _shifted(t):
    """The same values at an address that is only 4-byte aligned."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,H,dk", [(33, 2, 64), (1021, 16, 128), (4093, 16, 128)])
def test_fold_tiles(lib, dtype, d, H, dk):
    """One shape per output tile (32, 64 and 128 wide), ragged rows."""
    say(f"fold d={d} H={H} dk={dk} {dtype}")
    W_Q = synth.normal((d, H * dk), 31, 1, d ** -0.5, dtype)
    W_R = synth.normal((H, dk, dk), 31, 2, dk ** -0.5, dtype)
    got = kb.keyless_fold_routing(W_Q.to(DEV), W_R.to(DEV))
    torch.cuda.synchronize()
    assert_parity(got, K.fold_routing(to64(W_Q), to64(W_R), H, dk), dtype, "fold")


@pytest.mark.parametrize("shift", [False, True])
@pytest.mark.parametrize("N,d,H,G,dk", [(16, 64, 4, 4, 64), (17, 102, 2, 1, 128), (131, 63, 6, 2, 64)])
def test_layer_f32(lib, N, d, H, G, dk, shift):
    """Prefill and every gradient of the fp32 layer: d_model that is no multiple
    of 4 (element loads) or of the k-step, and operands without 16-byte
    alignment (element loads, and the vector-ALU attention)."""
    say(f"fp32 layer N={N} d={d} H={H} G={G} dk={dk} shift={shift}")
    B = 2
    x = synth.normal((B, N, d), 32, 1, 1.0, F32)
    W_Q = synth.normal((d, H * dk), 32, 2, d ** -0.5, F32)
    W_R = synth.normal((H, dk, dk), 32, 3, dk ** -0.5, F32)
    W_V = synth.normal((d, G * dk), 32, 4, d ** -0.5, F32)
    dO = synth.normal((B, N, H, dk), 32, 5, 1.0, F32)
    put = _shifted if shift else (lambda t: t.to(DEV))
    xs, wq, wr, wv = (put(t) for t in (x, W_Q, W_R, W_V))
    outs = [put(torch.zeros(B, N, n, dk)) for n in (H, H, G)]
    out, q, v = kb.keyless_prefill(xs, wq, wr, wv, H, G, return_qv=True, out=outs[0],
                                   q_routed_out=outs[1], v_out=outs[2])
    torch.cuda.synchronize()
    O, Qr, V = K.keyless_prefill(to64(x), to64(W_Q), to64(W_R), to64(W_V), H, G, dk)
    assert_parity(out, O, F32, "out")
    assert_parity(q, Qr, F32, "q")
    assert_parity(v, V, F32, "v")
    q, v = q.clone(), v.clone()
    out, lse = kb.keyless_attention_forward(q, v)
    dq, dv = kb.keyless_attention_backward(q, v, out, dO.to(DEV), lse)
    grads = kb.keyless_weight_gradients(xs, wq, wr, wv, put(dq), put(dv), H, G)
    torch.cuda.synchronize()
    ref = K.keyless_projection_gradients(to64(x), to64(W_Q), to64(W_R), to64(W_V), to64(dq),
                                         to64(dv), H, G, dk)
    for name, g in grads.items():
        assert_parity(g, ref[name], F32, name, 1e-2)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,N,H,G,dk", [(2, 1, 4, 2, 64), (1, 4, 3, 1, 128), (1, 5, 2, 2, 128),
                                        (2, 8, 2, 2, 64), (1, 9, 4, 4, 64),
                                        (1, 15, 2, 2, 64), (2, 16, 4, 2, 128), (1, 17, 3, 1, 128),
                                        (1, 129, 2, 2, 128), (2, 250, 4, 1, 64)])
def test_attention_f32(lib, causal, B, N, H, G, dk):
    """Whole and ragged 16-row blocks, fewer and more of them than waves; the
    most rows that the forward leaves to the vector ALU, and one more."""
    say(f"fp32 attention B={B} N={N} H={H} G={G} dk={dk} causal={causal}")
    q, v, g = (synth.normal((B, N, n, dk), 33, i, 1.0, F32) for i, n in enumerate((H, G, H)))
    o32 = torch.empty((B, N, H, dk), dtype=F32, device=DEV)
    out, lse = kb.keyless_attention_forward(q.to(DEV), v.to(DEV), causal=causal, out_f32=o32)
    dq, dv = kb.keyless_attention_backward(q.to(DEV), v.to(DEV), out, g.to(DEV), lse, causal=causal)
    torch.cuda.synchronize()
    assert torch.equal(out, o32)
    ref_lse = K.attention_logsumexp(to64(q), to64(v), H, G, dk, causal=causal)
    assert rowwise_rel(lse, ref_lse) <= 1e-4
    rq, rv = K.keyless_attention_backward(to64(q), to64(v), to64(g), H, G, dk, causal=causal)
    scale = 1e-2 * max(np.abs(rq).max(), np.abs(rv).max())
    assert_parity(dq, rq, F32, "dQ~", 1e-2, scale)
    assert_parity(dv, rv, F32, "dV", 1e-2, scale)


def test_attention_backward_f32_above_one_grid(lib):
    """More 16-row blocks than a grid takes (65535): both kernels run in several
    launches. Rows on both sides of the seam, the first and the last ones against
    their sums in 64 bits (lse, out and dout are inputs: any finite values do). A
    sum of n terms of either sign is off by about sqrt(n) 2^-24 of itself, 6e-5."""
    N, d = 16 * 65535 + 35, 64
    say(f"fp32 backward of {N} rows")
    gen = torch.Generator(device=DEV).manual_seed(5)
    q, v, o, g = (torch.randn((1, N, 1, d), generator=gen, device=DEV) for _ in range(4))
    lse = torch.full((1, 1, N), 13.0, device=DEV)
    dq, dv = kb.keyless_attention_backward(q, v, o, g, lse)
    torch.cuda.synchronize()
    say("fp32 backward done")
    q, v, o, g, dq, dv = (t.view(N, d) for t in (q, v, o, g, dq, dv))
    dd = (o.double() * g.double()).sum(1)
    for r in (0, 33, N // 2, 16 * 65535 - 1, 16 * 65535, 16 * 65535 + 16, N - 1):
        vr, qr, gr = v[r].double(), q[r].double(), g[r].double()
        V = v[:r + 1].double()
        ref = (torch.exp(V @ qr / 8 - 13) * (V @ gr - dd[r])) @ V / 8
        assert (dq[r].double() - ref).norm() <= 1e-3 * ref.norm(), f"dQ~ {r}"
        Q, G = q[r:].double(), g[r:].double()
        P = torch.exp(Q @ vr / 8 - 13)
        ref = P @ G + (P * (G @ vr - dd[r:])) @ Q / 8
        assert (dv[r].double() - ref).norm() <= 1e-3 * ref.norm(), f"dV {r}"


def test_unseen_rows_do_not_reach_a_row_f32(lib):
    """Causal rows before an infinite value row, and value rows after a query row
    with a NaN gradient, keep their results (a block that holds such a row is summed
    in another order)."""
    N, H, dk = 40, 2, 64
    say("fp32 attention, non-finite rows out of sight")
    q, v, g = (synth.normal((1, N, H, dk), 34, i, 1.0, F32).to(DEV) for i in range(3))
    out, lse = kb.keyless_attention_forward(q, v)
    dq, dv = kb.keyless_attention_backward(q, v, out, g, lse)
    at = 21  # inside the second block
    v2, g2 = v.clone(), g.clone()
    v2[:, at, :, 5] = float("inf")
    g2[:, at, :, 7] = float("nan")
    out2, lse2 = kb.keyless_attention_forward(q, v2)
    dq2, _ = kb.keyless_attention_backward(q, v2, out, g, lse)
    _, dv3 = kb.keyless_attention_backward(q, v, out, g2, lse)
    torch.cuda.synchronize()
    for a, b in ((out2, out), (dq2, dq)):
        torch.testing.assert_close(a[:, :at], b[:, :at], rtol=1e-5, atol=1e-6)
    torch.testing.assert_close(lse2[:, :, :at], lse[:, :, :at], rtol=1e-6, atol=1e-6)
    torch.testing.assert_close(dv3[:, at + 1:], dv[:, at + 1:], rtol=1e-5, atol=1e-6)
    assert not torch.isfinite(out2[:, at:, :, 5]).any()
    assert torch.isnan(dv3[:, :at + 1, :, 7]).all()
