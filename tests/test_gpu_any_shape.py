"""The GEMM kernels for shapes and storage types outside the 256-wide bf16 tiles, at the edges of their own tiles,
against float64 products of the same stored operands (plain PyTorch).

Bars: a result is a sum of `n` exact products accumulated in fp32 and rounded once to bf16, so per element
|diff| <= 2^-8 (1 + 2^-8) |ref| + n 2^-23 sum |a b| (bf16 has a significand of 8 bits: rounding to nearest moves a value
by at most 2^-8 of itself); where the result is kept in fp32 the first term is 2^-23 |ref|.
"""
import random

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


# fp32 storage with enough tiles for the wide ones (three per compute unit): remainders along both axes, and rows at the
# edges of a step
@pytest.mark.parametrize("d,h", [(1032, 3080), (2040, 1544)])
def test_weight_gradients_of_wide_tiles(env, d, h):
    torch, lm = env
    rows = [33, 0, 1, 97, 32, 64, 31, 2] * 3
    E, K = len(rows), sum(rows)
    print(f"[wgrad wide] d={d} h={h} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d + h)
    off, seg, be = segments(torch, rows)
    desc = lm.make_desc(600, d, E, 1, h, 100, "f32")
    send, dout = (rows_with_nan_tail(torch, K, 40, d, torch.float32, gen) for _ in range(2))
    H, dZ = (rows_with_nan_tail(torch, K, 40, h, torch.bfloat16, gen) for _ in range(2))
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


# 2 experts: tiles of 128 x 128.  24: with fp32 storage tiles of 256 columns of the bf16 operand (three per compute unit); each
# axis has a last tile that is not full, with infinities in it
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,d,h", [([40, 33], 136, 264), ([40, 33] + [0] * 22, 1032, 3080)])
def test_weight_gradients_of_infinities(env, rows, d, h, dtype):
    """An infinite or NaN operand gives what the products give: inf where 1.0 * inf, NaN only where 0 * inf or inf - inf.
    The other operand's values (small whole numbers) have few significant bits."""
    torch, lm = env
    E, K, C = len(rows), sum(rows), 40
    print(f"[wgrad inf] {dtype} d={d} h={h}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    off, seg, be = segments(torch, rows)
    ints = lambda cols, t: torch.randint(-3, 4, (K, cols), generator=gen, device="cuda").to(t)
    send, dout = (ints(d, storage(torch, dtype)) for _ in range(2))
    H, dZ = (ints(h, torch.bfloat16) for _ in range(2))
    inf = float("inf")
    for t, r, c, v in ((H, 3, 5, inf), (H, 20, 130, -inf), (H, 50, 263, inf), (H, 51, 263, -inf), (dZ, 7, 100, -inf),
                       (dZ, 45, 0, float("nan")), (dZ, 72, 200, inf), (send, 2, 17, inf), (send, 60, 135, -inf),
                       (dout, 11, 64, inf), (dout, 3, 70, -inf)):
        t[r, c] = v
    for t, r, c, v in ((H, 5, h - 1, inf), (H, 41, h - 70, -inf), (dZ, 9, h - 1, inf), (dZ, 61, h - 140, float("nan")),
                       (send, 30, d - 1, inf), (dout, 44, d - 2, -inf)):
        t[r, c] = v
    desc = lm.make_desc(600, d, E, 1, h, C, dtype)
    dW_in = torch.empty((E, h, d), dtype=torch.bfloat16, device="cuda")
    dW_out = torch.empty((E, d, h), dtype=torch.bfloat16, device="cuda")
    lm.locmoe_expert_ffn_wgrad(desc, send, H, dout, dZ, seg, be, dW_in, dW_out)
    torch.cuda.synchronize()
    for r in range(E):
        e, a, z = E - 1 - r, off[r], off[r + 1]
        if a == z:
            assert not dW_in[e].any() and not dW_out[e].any()
            continue
        for got, P, Q in ((dW_in[e], dZ, send), (dW_out[e], dout, H)):
            ref = torch.zeros(P.shape[1], Q.shape[1], dtype=torch.float64, device="cuda")
            for k in range(a, z):
                ref += P[k].double()[:, None] * Q[k].double()[None, :]
            assert ref.isinf().any()
            # finite sums are whole numbers below 2^9: exact in fp32, rounded once to bf16
            assert torch.equal(got.double().nan_to_num(12345.0), ref.to(torch.bfloat16).double().nan_to_num(12345.0)), r


def gelu(torch, v):
    return 0.5 * v * torch.erfc(-v * 2.0 ** -0.5)


def gelu_grad(torch, v):
    return 0.5 * torch.erfc(-v * 2.0 ** -0.5) + v * torch.exp(-0.5 * v * v) * (2.0 * torch.pi) ** -0.5


# (8, 8): one partial tile and k-step; 128/64-column tiles with and without remainders; k remainders of 8 and 56; the
# last one has enough tiles for the 128-column kernel in both directions (6 x 86 >= 512)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,h", [(48, 8), (120, 264), (192, 128), (384, 1000), (264, 11000), (11016, 72)])
def test_expert_ffn_of_any_shape(env, d, h, dtype):
    check_expert_ffn(env, d, h, dtype, [0, 1, 16, 17, 128, 259], 300)


# few rows per segment and few experts with packed weights: the narrow tiles of ffn_gemm_any (128 x 32), K = 256 .. 1280, segments
# at the edges of its row subtiles; 64 experts: its wider ones
@pytest.mark.parametrize("rows", [[0, 1, 15, 16], [32, 17, 0, 5], [64, 0, 33, 48, 1, 63, 2, 16], [65, 0, 64, 1], [33] * 64])
@pytest.mark.parametrize("d,h", [(768, 256), (256, 768), (512, 1280)])
def test_expert_ffn_of_few_rows(env, d, h, rows):
    check_expert_ffn(env, d, h, "bf16", rows, max(rows), packed=True)


def ffn_outputs(env, d, h, rows, T, C, dtype="bf16", packed=True):
    """H, Z, out, dZ and dsend with a descriptor of T tokens and capacity C."""
    torch, lm = env
    E, K = len(rows), sum(rows)
    print(f"[ffn T, C] d={d} h={h} T={T} C={C} {dtype} packed={packed} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d * 3 + h)
    off, seg, be = segments(torch, rows)
    xd = storage(torch, dtype)
    desc = lm.make_desc(T, d, E, 1, h, C, dtype, w_packed=packed)
    send, dout = (rows_with_nan_tail(torch, K, 0, d, xd, gen) for _ in range(2))
    W_in = (torch.randn(E, h, d, generator=gen, device="cuda") * d ** -0.5).to(torch.bfloat16)
    W_out = (torch.randn(E, d, h, generator=gen, device="cuda") * h ** -0.5).to(torch.bfloat16)
    L_in, L_out, Lt_in, Lt_out = W_in, W_out, torch.empty_like(W_out), torch.empty_like(W_in)
    if packed:
        L_in, L_out = torch.empty_like(W_in), torch.empty_like(W_out)
        lm.locmoe_pack_weights(desc, W_in, W_out, L_in, L_out)
        lm.locmoe_pack_weights_t(desc, W_in, W_out, Lt_in, Lt_out)
    else:
        lm.locmoe_transpose_weights(desc, W_in, W_out, Lt_in, Lt_out)
    H, Z, dZ = (torch.full((K, h), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    out, dsend = (torch.full((K, d), float("nan"), dtype=xd, device="cuda") for _ in range(2))
    lm.locmoe_expert_ffn_in_save(desc, send, seg, be, L_in, H, Z)
    lm.locmoe_expert_ffn_out(desc, H, seg, be, L_out, out)
    lm.locmoe_expert_ffn_dgrad(desc, dout, Z, seg, be, Lt_out, Lt_in, dZ, dsend)
    torch.cuda.synchronize()
    return dict(H=H, Z=Z, out=out, dZ=dZ, dsend=dsend)


# an element is one sum over K in one order, whichever kernel the capacity and the token count select
@pytest.mark.parametrize("rows", [[16, 1, 15, 0], [32, 17, 0, 5, 31, 16, 1, 2], [48, 33, 0, 47], [64, 0, 33, 48, 1, 63, 2, 16]])
@pytest.mark.parametrize("d,h", [(768, 256), (256, 2048), (512, 1280)])
def test_bits_do_not_depend_on_capacity_or_token_count(env, d, h, rows):
    ref = ffn_outputs(env, d, h, rows, 600, 300)
    for T, C in ((600, max(rows)), (max(rows), 300)):
        got = ffn_outputs(env, d, h, rows, T, C)
        for name in ref:
            assert env[0].equal(got[name], ref[name]), name


# the stream of weights (ffn_gemm_few) in its two forms, with every epilogue: rows at the edges of its 16-row subtiles,
# segments without rows, and segments longer than min(C, T), which it walks in passes.  The same bits as the persistent
# kernel and the row-major one give.
@pytest.mark.parametrize("rows,C", [([16, 1, 15, 0, 9, 2, 16, 8], 16), ([0, 16, 17, 130, 64, 33, 1, 32], 16),
                                    ([32, 17, 0, 5, 31, 16, 1, 2], 32), ([32, 33, 0, 65, 31, 130, 64, 1], 32)])
def test_few_rows_kernel(env, rows, C):
    torch, lm = env
    d, h, rows = 768, 2048, rows * 16
    E = len(rows)
    for second in (False, True):
        for cap, kernel in ((C, "ffn_gemm_few"), (1000, "ffn_gemm_dma_persistent")):
            assert lm.ffn_kernel(lm.make_desc(E * cap, d, E, 1, h, cap, w_packed=True), second, not second) == kernel
    got = ffn_outputs(env, d, h, rows, E * C, C)
    for ref in (ffn_outputs(env, d, h, rows, E * 1000, 1000), ffn_outputs(env, d, h, rows, E * C, C, packed=False)):
        for name in ref:
            assert torch.equal(got[name], ref[name]), name


# segments may hold more rows than min(C, T) (rows of other ranks' tokens): seg_off decides
@pytest.mark.parametrize("T,C", [(600, 16), (600, 32), (600, 64), (16, 300)])
def test_few_rows_kernel_covers_longer_segments(env, T, C):
    rows = [17, 0, 130, 64, 65, 16, 1, 33]
    ref, got = ffn_outputs(env, 256, 512, rows, 600, 300), ffn_outputs(env, 256, 512, rows, T, C)
    for name in ref:
        assert env[0].equal(got[name], ref[name]), name


def spread(E, top, every=1):
    """Rows per expert, 0 .. top, only every `every`-th expert with any; the longest and lengths of one and none are there."""
    r = random.Random(E)
    rows = [r.randint(0, top) if e % every == 0 else 0 for e in range(E)]
    rows[0], rows[every % E], rows[-1] = top, 1, 0
    return rows


# (packed, kernels of the first and second GEMM, E, d, h, T, C, rows).  test_ffn_kernel_choice.py checks without a GPU that
# the shapes reach these kernels.
KERNEL_SHAPES = [
    # the persistent kernel: uneven and empty segments; a list so short that its m-tiles are cut to 64 rows; the most experts it
    # takes; the shortest K (four double steps) and the shortest N; three m-tiles per segment; more tiles per XCD than
    # work-groups, also of segments without rows
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 8, 1536, 4096, 3200, 400, [400, 0, 257, 256, 1, 129, 64, 300]),
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 64, 2048, 2048, 2080, 65, spread(64, 65, 8)),
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 512, 1024, 768, 16640, 65, spread(512, 65, 2)),
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 256, 256, 8192, 8320, 65, spread(256, 65, 3)),
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 16, 1024, 1024, 48000, 3000, spread(16, 700)),
    (True, "ffn_gemm_dma_persistent", "ffn_gemm_dma_persistent", 128, 768, 4096, 4160, 65, spread(128, 65)),
    # one tile per work-group: expert counts that are no multiple of 8, or above 512
    (True, "ffn_gemm_dma", "ffn_gemm_dma", 4, 3072, 4096, 4000, 1000, [1000, 0, 333, 257]),
    (True, "ffn_gemm_dma", "ffn_gemm_dma", 12, 1536, 8192, 4200, 700, spread(12, 700)),
    (True, "ffn_gemm_dma", "ffn_gemm_dma", 1024, 1024, 512, 33280, 65, spread(1024, 65, 2)),
    # every tile shape of ffn_gemm_any, in lists of up to 64 segments and of more; weight tiles that end in the next block of
    # 256 packed columns, or past the last column
    (True, "ffn_gemm_any<128, 32>", "ffn_gemm_any<128, 32>", 8, 256, 512, 1200, 150, [150, 0, 1, 97, 128, 129, 33, 16]),
    (True, "ffn_gemm_any<160, 160>", "ffn_gemm_any<128, 64>", 32, 256, 2304, 5152, 161, [161, 0, 160, 1, 130, 96, 65, 32] * 4),
    (True, "ffn_gemm_any<160, 160>", "ffn_gemm_any<192, 128>", 64, 512, 1280, 9600, 150, [150, 33, 149, 0, 64, 150, 128, 17] * 8),
    (True, "ffn_gemm_any<192, 128>", "ffn_gemm_any<192, 128>", 128, 256, 768, 17920, 140, [140, 0, 139, 1, 96, 97, 15, 129] * 16),
    (False, "ffn_gemm_any<128, 32>", "ffn_gemm_any<128, 32>", 8, 256, 512, 1200, 150, [150, 0, 1, 97, 128, 129, 33, 16]),
    (False, "ffn_gemm_any<160, 160>", "ffn_gemm_any<128, 64>", 32, 256, 2304, 5152, 161, [161, 0, 160, 1, 130, 96, 65, 32] * 4),
    (False, "ffn_gemm_any<192, 128, dealt>", "ffn_gemm_any<192, 128>", 128, 256, 768, 17920, 140,
     [140, 0, 139, 1, 96, 97, 15, 129] * 16),
    (False, "ffn_gemm_any<192, 128>", "ffn_gemm_any<192, 128>", 128, 512, 256, 24704, 193, spread(128, 193)),
    (False, "ffn_gemm_any<192, 128, dealt>", "ffn_gemm_any<192, 128>", 128, 256, 2048, 24704, 193, spread(128, 193, 2)),
    (False, "ffn_gemm_any<192, 64, dealt>", "ffn_gemm_any<160, 160>", 48, 768, 256, 6192, 400, spread(48, 129)),
]


def other_tiles(lm, first, second, E, d, h):
    """T and C with which the row-major kernel takes other tiles, in both GEMMs if there are such."""
    def same(tc):
        desc = lm.make_desc(tc[0], d, E, 1, h, tc[1])
        return (lm.ffn_kernel(desc) == first) + (lm.ffn_kernel(desc, True) == second)
    best = min(((600, 3000), (8, 8), (E * 100, 100), (E * 600, 600), (E * 4000, 4000)), key=same)
    assert same(best) < 2
    return best


@pytest.mark.parametrize("packed,first,second,E,d,h,T,C,rows", KERNEL_SHAPES)
def test_each_kernel_gives_the_same_bits(env, packed, first, second, E, d, h, T, C, rows):
    """H, Z, out and both data gradients, bit for bit as the row-major kernel with another tile shape makes them (which
    check_expert_ffn above holds against the formulas in float64)."""
    torch, lm = env
    desc = lm.make_desc(T, d, E, 1, h, C, w_packed=packed)
    for i, name in enumerate((first, second)):
        assert lm.ffn_kernel(desc, bool(i), i == 0) == lm.ffn_kernel(desc, bool(i)) == name
    other = other_tiles(lm, first, second, E, d, h)
    ref, got = ffn_outputs(env, d, h, rows, *other, packed=False), ffn_outputs(env, d, h, rows, T, C, packed=packed)
    for name in ref:
        assert torch.equal(got[name], ref[name]), name


# row-major weights: a work-group per weight tile (min(C, T) <= 128) and lists of tiles, shorter and longer than the grid
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,C", [(600, 64), (60, 3000), (260, 3000)])
def test_row_major_kernel_covers_longer_segments(env, T, C, dtype):
    rows = [17, 0, 1300, 64, 193, 16, 400, 33]
    ref, got = (ffn_outputs(env, 264, 520, rows, *tc, dtype, packed=False) for tc in ((6000, 3000), (T, C)))
    for name in ref:
        assert env[0].equal(got[name], ref[name]), name


# more segments than a wave has lanes, empty ones among them, weight tiles that divide by 8 and that do not; a list that
# fills the chip once in tiles of 128 rows, one that does not, and a long one
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,h,rows", [(280, 264, [0, 300, 1, 193, 192, 0, 129] * 10), (1024, 1024, [0, 256, 129, 0] * 32),
                                      (64, 8200, [200, 0, 131, 600]), (1032, 2048, [1000, 0, 30, 385]),
                                      (264, 20000, [0, 777, 0, 0, 0, 0, 0, 193])])
def test_row_major_lists_of_tiles(env, d, h, rows, dtype):
    check_expert_ffn(env, d, h, dtype, rows, max(rows))


# rows of more than 2^32 / 768 values (5.6 M), and so long that a tile's rows span more than 4 GiB.  The operands are zero
# but for a few columns (the first and the last ones among them), so that the sums have few terms.
@pytest.mark.parametrize("dtype,d,rows", [("bf16", 5_600_008, 17), ("bf16", 11_200_008, 192), ("f32", 8_400_008, 128)])
def test_expert_ffn_of_very_long_rows(env, dtype, d, rows):
    torch, lm = env
    print(f"[ffn long rows] d={d} {dtype} rows={rows}", flush=True)
    h, n = 8, 300
    gen = torch.Generator(device="cuda").manual_seed(d)
    cols = torch.cat([torch.arange(8, device="cuda"), torch.randint(8, d - 8, (n - 16,), generator=gen, device="cuda"),
                      torch.arange(d - 8, d, device="cuda")]).unique()
    xd = storage(torch, dtype)
    off, seg, be = segments(torch, [rows])
    desc = lm.make_desc(rows, d, 1, 1, h, rows, dtype)
    send = torch.zeros(rows, d, dtype=xd, device="cuda")
    send[:, cols] = torch.randn(rows, len(cols), generator=gen, device="cuda").to(xd)
    W_in = torch.zeros(1, h, d, dtype=torch.bfloat16, device="cuda")
    W_in[:, :, cols] = torch.randn(1, h, len(cols), generator=gen, device="cuda").to(torch.bfloat16)
    W_out = torch.randn(1, d, h, generator=gen, device="cuda").to(torch.bfloat16)
    H, Z = (torch.full((rows, h), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    out = torch.full((rows, d), float("nan"), dtype=xd, device="cuda")
    lm.locmoe_expert_ffn_in_save(desc, send, seg, be, W_in, H, Z)
    lm.locmoe_expert_ffn_out(desc, H, seg, be, W_out, out)
    torch.cuda.synchronize()
    b16, u = 2.0 ** -8 * (1 + 2.0 ** -8), 2.0 ** -23
    x, w = send[:, cols].to(torch.bfloat16).double(), W_in[0, :, cols].double()
    ref, bound = x @ w.T, len(cols) * u * (x.abs() @ w.abs().T)
    assert ((Z.double() - ref).abs() <= b16 * ref.abs() + 1.01 * bound).all()
    for r in range(rows):
        hr = H[r].double()
        ref, bound = W_out[0].double() @ hr, h * u * (W_out[0].double().abs() @ hr.abs())
        assert ((out[r].double() - ref).abs() <= (b16 if dtype == "bf16" else u) * ref.abs() + 1.01 * bound).all(), r


def test_expert_ffn_of_very_many_columns(env):
    """8 experts of 2^28 columns: 2^24 tiles of 128, more than one launch dimension takes."""
    torch, lm = env
    E, d, h = 8, 8, 1 << 28
    print(f"[ffn many columns] E={E} d={d} h={h}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    off, seg, be = segments(torch, [1] * E)
    desc = lm.make_desc(E, d, E, 1, h, 1, "bf16")
    send = torch.randn(E, d, generator=gen, device="cuda").to(torch.bfloat16)
    W_in = torch.empty(E, h, d, dtype=torch.bfloat16, device="cuda")
    for e in range(E):
        W_in[e].normal_(0.0, 1.0, generator=gen)
    H = torch.full((E, h), float("nan"), dtype=torch.bfloat16, device="cuda")
    lm.locmoe_expert_ffn_in(desc, send, seg, be, W_in, H)
    torch.cuda.synchronize()
    b16, u, step = 2.0 ** -8 * (1 + 2.0 ** -8), 2.0 ** -23, 1 << 24
    for r in range(E):
        x = send[r].double()
        for n in range(0, h, step):
            w = W_in[E - 1 - r, n:n + step].double()
            z, zb = (w * x).sum(1), d * u * (w * x).abs().sum(1)
            hr = gelu(torch, z)
            bound = 1.01 * (b16 * hr.abs() + 5e-5 * hr.abs() + 7e-6 + 1.13 * zb)
            assert ((H[r, n:n + step].double() - hr).abs() <= bound).all(), (r, n)


def check_expert_ffn(env, d, h, dtype, rows, C, packed=False):
    """H, Z, out and the data gradients; GeLU's polynomial is within 5e-5 |ref| + 7e-6 (its derivative within 5e-5)."""
    torch, lm = env
    E, K = len(rows), sum(rows)
    print(f"[ffn] d={d} h={h} {dtype} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d * 5 + h)
    off, seg, be = segments(torch, rows)
    xd = storage(torch, dtype)
    desc = lm.make_desc(600, d, E, 1, h, C, dtype)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    send = rows_with_nan_tail(torch, K, 40, d, xd, gen)
    dout = rows_with_nan_tail(torch, K, 40, d, xd, gen)
    W_in = (torch.randn(E, h, d, generator=gen, device="cuda") * d ** -0.5).to(torch.bfloat16)
    W_out = (torch.randn(E, d, h, generator=gen, device="cuda") * h ** -0.5).to(torch.bfloat16)
    H, Z, dZ = (torch.full((K + 40, h), float("nan"), **bf) for _ in range(3))
    H2 = torch.empty_like(H)
    out, dsend = (torch.full((K + 40, d), float("nan"), dtype=xd, device="cuda") for _ in range(2))
    Wt_in, Wt_out = W_in.transpose(1, 2).contiguous(), W_out.transpose(1, 2).contiguous()
    L_in, L_out = W_in, W_out  # in the layout that the kernels read
    if packed:
        desc.w_packed = 1
        L_in, L_out = torch.empty_like(W_in), torch.empty_like(W_out)
        lm.locmoe_pack_weights(desc, W_in, W_out, L_in, L_out)
        lm.locmoe_pack_weights_t(desc, W_in, W_out, Wt_in, Wt_out)
    lm.locmoe_expert_ffn_in_save(desc, send, seg, be, L_in, H, Z)
    lm.locmoe_expert_ffn_in(desc, send, seg, be, L_in, H2)
    lm.locmoe_expert_ffn_out(desc, H, seg, be, L_out, out)
    lm.locmoe_expert_ffn_dgrad(desc, dout, Z, seg, be, Wt_out, Wt_in, dZ, dsend)
    torch.cuda.synchronize()
    assert torch.equal(H[:K], H2[:K])
    for t in (H, Z, dZ, out, dsend):
        assert t[K:].isnan().all()  # nothing past the last segment is written
    b16, u = 2.0 ** -8 * (1 + 2.0 ** -8), 2.0 ** -23
    ulp = b16 if dtype == "bf16" else u
    for r in range(E):
        e, a, z = E - 1 - r, off[r], off[r + 1]
        s, do = send[a:z].to(torch.bfloat16).double(), dout[a:z].to(torch.bfloat16).double()
        zr, zb = s @ W_in[e].double().T, d * u * (s.abs() @ W_in[e].double().abs().T)
        hr = gelu(torch, zr)
        assert ((Z[a:z].double() - zr).abs() <= b16 * zr.abs() + 1.01 * zb).all(), r
        assert ((H[a:z].double() - hr).abs() <= 1.01 * (b16 * hr.abs() + 5e-5 * hr.abs() + 7e-6 + 1.13 * zb)).all(), r
        hs = H[a:z].double()
        orf, ob = hs @ W_out[e].double().T, h * u * (hs.abs() @ W_out[e].double().abs().T)
        assert ((out[a:z].double() - orf).abs() <= ulp * orf.abs() + 1.01 * ob).all(), r
        gr = gelu_grad(torch, Z[a:z].double())
        dh, hb = do @ W_out[e].double(), d * u * (do.abs() @ W_out[e].double().abs())
        assert ((dZ[a:z].double() - dh * gr).abs() <= 1.01 * (b16 * (dh * gr).abs() + 5e-5 * dh.abs() + 1.13 * hb)).all(), r
        dz = dZ[a:z].double()
        dr, db = dz @ W_in[e].double(), h * u * (dz.abs() @ W_in[e].double().abs())
        assert ((dsend[a:z].double() - dr).abs() <= ulp * dr.abs() + 1.01 * db).all(), r
