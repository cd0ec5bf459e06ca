"""GPU parity of the fp32 matrix-core kernels (the GEMM in fp32 arithmetic, the
fp32 attention forward and backward) at the edges of their tiles and in every
way they load an operand, against the CPU oracle."""

import pytest
import torch

from oracle import keyless as K
from paper_2606_21848_amd import binding as kb
from tests.parity import assert_parity, say, to64
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
