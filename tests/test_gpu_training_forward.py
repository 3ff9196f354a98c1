"""A training step's own forward, layer by layer, against code that it does not share: the outputs
bit for bit against the forward entry point (its wide kernel above 4096 rows) and against the
64 x 64 product kernel (operands without a unit stride) on the exported activations, and each
hidden activation against GELU in float64 of that product's pre-activation."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _product(sg, A, W, b):
    """A W + b on the 64 x 64 kernel: every second element of wider buffers."""
    import torch
    M, K = A.shape
    N = W.shape[1]
    A2 = torch.zeros((M, 2 * K), device="cuda", dtype=torch.bfloat16)
    A2[:, ::2] = A
    W2 = torch.zeros((K, 2 * N), device="cuda", dtype=torch.bfloat16)
    W2[:, ::2] = W
    return sg.gemm_bf16(A2, (2 * K, 2), W2, (2 * N, 2), M, N, K, bias=b)


def _assert_gelu(h, pre):
    """h, a BF16 value, is a rounding of GELU(pre) in the tanh form: within half a BF16 ulp of the
    float64 value plus the float32 evaluation's error (a few 2^-24 of |pre|)."""
    import torch
    x = pre.double()
    ref = 0.5 * x * (1.0 + torch.tanh(0.7978845608 * (x + 0.044715 * x ** 3)))
    # half an ulp of the binade of |ref| rounded up by the evaluation's error: 2^-8 |ref| at most
    bound = ref.abs() * 2.0 ** -8 + 16.0 * 2.0 ** -24 * x.abs() + 1e-37
    bad = (h.double() - ref).abs() > bound
    assert not bool(bad.any()), int(bad.sum())


@pytest.mark.parametrize("B", [37, 4096, 4111, 8192, 8193, 16399])
def test_training_forward_layer_by_layer(B):
    import torch
    import paper_2607_25388_amd.sgtp as sg
    m = sg.Mlp(max(B, 64), seed=B % 89)
    try:
        rng = np.random.default_rng(B)
        p = m.get_params()
        P = sg.mlp_unpack(p)
        for nm in ("b1", "b2", "b3"):
            P[nm][...] = 0.2 * rng.standard_normal(P[nm].shape)
        P["W3"][...] *= 5.0
        m.set_params(p)
        assert all(np.shares_memory(P[nm], p) for nm in P)
        T = {k: torch.as_tensor(np.ascontiguousarray(v)).cuda() for k, v in P.items()}
        X = torch.as_tensor(rng.standard_normal((B, 50)).astype(np.float32)).cuda()
        U = torch.as_tensor(np.stack([rng.uniform(-8, 4, (B, 50)), rng.uniform(-0.4, 0.4, (B, 50))], -1)
                            .astype(np.float32)).cuda()
        print(f"training forward, {B} rows", flush=True)
        m.grad(X, U, 1.5, 0.08)
        h1, h2, out = (m.workspace(k)[:B] for k in ("h1", "h2", "out"))
        fwd = m.forward(X)
        bf = {k: T[k].to(torch.bfloat16) for k in ("W1", "W2", "W3")}
        o = _product(sg, h2.to(torch.bfloat16), bf["W3"], T["b3"])
        torch.cuda.synchronize()
        bits = lambda t: t.contiguous().view(torch.int32)
        assert torch.equal(bits(out[:, :200].float()), bits(fwd))
        assert torch.equal(bits(out[:, :200].float()), bits(o))
        _assert_gelu(h1, _product(sg, X.to(torch.bfloat16), bf["W1"], T["b1"]))
        _assert_gelu(h2, _product(sg, h1.to(torch.bfloat16), bf["W2"], T["b2"]))
    finally:
        m.close()
