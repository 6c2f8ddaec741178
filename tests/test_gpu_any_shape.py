"""The GEMM kernels for shapes and storage types outside the 256-wide bf16 tiles, at the edges of their own tiles,
against float64 products of the same stored operands (plain PyTorch).

Bars: a result is a sum of `n` exact products accumulated in fp32 and rounded once to bf16, so per element
|diff| <= 2^-8 (1 + 2^-8) |ref| + n 2^-23 sum |a b| (bf16 has a significand of 8 bits: rounding to nearest moves a value
by at most 2^-8 of itself); where the result is kept in fp32 the first term is 2^-23 |ref|.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2401_13920_amd import locmoe as lm
    assert torch.cuda.is_available(), "these tests need the MI355X"
    lm.lib()
    return torch, lm


def segments(torch, rows):
    off = [0]
    for n in rows:
        off.append(off[-1] + n)
    i32 = dict(dtype=torch.int32, device="cuda")
    return off, torch.tensor(off, **i32), torch.tensor(list(range(len(rows)))[::-1], **i32)  # rank r holds expert E-1-r


def storage(torch, dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


def rows_with_nan_tail(torch, n, extra, cols, dtype, gen):
    """[n + extra, cols]: random rows, then rows that no kernel may use (NaN)."""
    t = torch.full((n + extra, cols), float("nan"), device="cuda")
    t[:n] = torch.randn(n, cols, generator=gen, device="cuda")
    return t.to(dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,h", [(8, 8), (128, 128), (120, 264), (136, 1000), (1600, 40)])
def test_weight_gradients_of_any_shape(env, d, h, dtype):
    torch, lm = env
    rows = [0, 1, 31, 32, 33, 97]
    E, K, C = len(rows), sum(rows), 100
    print(f"[wgrad] d={d} h={h} {dtype} rows={rows}", flush=True)
    if d % E:
        E_d = d * E      # (the descriptor wants d % E == 0; the GEMMs do not care)
        d = E_d
    gen = torch.Generator(device="cuda").manual_seed(d * 7 + h)
    off, seg, be = segments(torch, rows)
    xd = storage(torch, dtype)
    desc = lm.make_desc(600, d, E, 1, h, C, dtype)
    send = rows_with_nan_tail(torch, K, 40, d, xd, gen)
    dout = rows_with_nan_tail(torch, K, 40, d, xd, gen)
    H = rows_with_nan_tail(torch, K, 40, h, torch.bfloat16, gen)
    dZ = rows_with_nan_tail(torch, K, 40, h, torch.bfloat16, gen)
    dW_in = torch.full((E, h, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dW_out = torch.full((E, d, h), float("nan"), dtype=torch.bfloat16, device="cuda")
    lm.locmoe_expert_ffn_wgrad(desc, send, H, dout, dZ, seg, be, dW_in, dW_out)
    torch.cuda.synchronize()
    for r in range(E):
        e, a, z = E - 1 - r, off[r], off[r + 1]
        for got, P, Q in ((dW_in[e], dZ, send), (dW_out[e], dout, H)):
            p, q = P[a:z].double(), Q[a:z].double()
            ref = p.T @ q
            bound = 2.0 ** -8 * (1 + 2.0 ** -8) * ref.abs() + (z - a) * 2.0 ** -23 * (p.abs().T @ q.abs())
            assert ((got.double() - ref).abs() <= bound).all(), (r, z - a)
