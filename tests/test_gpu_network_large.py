"""The network's large-tile product and wide forward pass: bit for bit against the kernels of
small sizes (same blocks of 32 k in the same order), and the product within the accumulation
bound of its float64 value, at the edges of the tiles, with every operand layout, odd leading
dimensions and misaligned bases."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _operand(rows, cols, along_rows, pad, offset, gen):
    """BF16 operand of logical shape [rows][cols] and its element strides: unit stride along
    the columns, or (along_rows) along the rows; `pad` extra elements between lines."""
    import torch
    lines, length = (cols, rows) if along_rows else (rows, cols)
    ld = length + pad
    buf = torch.zeros(lines * ld + offset + 8, device="cuda", dtype=torch.bfloat16)
    v = buf[offset:offset + lines * ld].view(lines, ld)
    v[:, :length] = torch.randn((lines, length), generator=gen, device="cuda").to(torch.bfloat16)
    t = buf[offset:]
    logical = v[:, :length].T if along_rows else v[:, :length]
    return t, ((1, ld) if along_rows else (ld, 1)), logical


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (16, 16, 32), (127, 129, 33), (128, 128, 64), (129, 127, 65), (5, 300, 200),
                                   (257, 256, 96), (300, 200, 1000), (5000, 3000, 40), (57, 57345, 7)])
@pytest.mark.parametrize("a_rows,b_rows,pad", [(False, False, 0), (False, True, 1), (True, False, 3), (True, True, 8)])
def test_large_tile_product(M, N, K, a_rows, b_rows, pad):
    import torch
    import paper_2607_25388_amd.sgtp as sg
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    print(f"case {M} {N} {K} {a_rows} {b_rows} {pad}", flush=True)
    A, sa, LA = _operand(M, K, a_rows, pad, pad & 1, g)
    B, sb, LB = _operand(K, N, b_rows, pad, pad & 1, g)
    bias = torch.randn(N, generator=g, device="cuda") if pad else None
    C = torch.full((M, N + pad), float("nan"), device="cuda")
    sg.gemm_bf16(A, sa, B, sb, M, N, K, bias=bias, out=C)
    # the 64 x 64 kernel: operands without a unit stride
    A2 = torch.zeros((M, 2 * K), device="cuda", dtype=torch.bfloat16)
    A2[:, ::2] = LA
    B2 = torch.zeros((K, 2 * N), device="cuda", dtype=torch.bfloat16)
    B2[:, ::2] = LB
    R = torch.empty((M, N), device="cuda")
    sg.gemm_bf16(A2, (2 * K, 2), B2, (2 * N, 2), M, N, K, bias=bias, out=R)
    torch.cuda.synchronize()
    assert torch.equal(C[:, :N].contiguous().view(torch.int32), R.view(torch.int32))
    assert pad == 0 or torch.isnan(C[:, N:]).all()  # nothing beyond the columns
    a, b = LA.double().cpu(), LB.double().cpu()
    if M * N * K > 2e8:
        a, C, R = a[::50], C[::50], R[::50]
    ref, mag = a @ b, a.abs() @ b.abs()
    if bias is not None:
        ref, mag = ref + bias.double().cpu(), mag + bias.double().cpu().abs()
    n = K + 1
    bound = mag * (n * 2.0 ** -24 / (1 - n * 2.0 ** -24)) + 1e-30
    assert bool(((C[:, :N].double().cpu() - ref).abs() <= bound).all())


@pytest.mark.parametrize("B,ld", [(4097, 200), (5000, 203), (8192, 256), (16383, 200), (16384, 200), (16401, 204)])
def test_wide_forward_matches_the_planning_forward(B, ld):
    import torch
    import paper_2607_25388_amd.sgtp as sg
    m = sg.Mlp(B, seed=B % 97)
    try:
        p = m.get_params()
        p[-200:] = np.linspace(-1.0, 1.0, 200)  # biases that show a misplaced column
        p[12800:13056] = np.linspace(-0.5, 0.5, 256)
        m.set_params(p)
        X = torch.randn((B, 50), generator=torch.Generator(device="cuda").manual_seed(B), device="cuda")
        out = torch.full((B + 1, ld), float("nan"), device="cuda")
        print(f"case {B} {ld}", flush=True)
        m.forward(X, out=out[:B])
        ref = torch.cat([m.forward(X[a:a + 4096]) for a in range(0, B, 4096)])
        torch.cuda.synchronize()
        assert torch.equal(out[:B, :200].contiguous().view(torch.int32), ref.view(torch.int32))
        assert torch.isnan(out[:B, 200:]).all() and torch.isnan(out[B]).all()
    finally:
        m.close()
