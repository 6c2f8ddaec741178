"""Which kernel a GEMM of the expert FFN goes to, asked of the library's own rule (which the launches follow) for 256
compute units, without a GPU.  The GPU tests that are meant for one kernel ask the same way, so that a change of the rule
cannot take their shapes away unseen."""
import pytest

from paper_2401_13920_amd import locmoe as lm
from test_gpu_any_shape import KERNEL_SHAPES, other_tiles


def kernels(T, d, E, h, C, dtype="bf16", packed=True):
    desc = lm.make_desc(T, d, E, 1, h, C, dtype, w_packed=packed)
    return [lm.ffn_kernel(desc, second, keeps_z) for second, keeps_z in ((False, False), (False, True), (True, False))]


# up to 32 rows per segment and four waves per compute unit: a stream of weights (the tiles of 256 columns take 1.05 to 1.5
# times as long, whatever the spread of the tokens); up to 64 rows never those tiles
@pytest.mark.parametrize("T,d,E,h,C", [(192, 1024, 64, 4096, 6), (700, 1024, 64, 4096, 16), (700, 2048, 32, 8192, 17),
                                       (700, 2048, 32, 8192, 22), (2000, 1024, 128, 2816, 32), (5000, 512, 256, 1024, 20)])
def test_few_rows_go_to_the_stream_of_weights(T, d, E, h, C):
    assert kernels(T, d, E, h, C) == ["ffn_gemm_few"] * 3


@pytest.mark.parametrize("T,d,E,h,C", [(700, 2048, 32, 8192, 44), (2000, 2048, 32, 8192, 63), (2000, 2048, 64, 8192, 64),
                                       (5000, 1024, 128, 2816, 40), (192, 4096, 8, 16384, 48), (700, 2560, 20, 10240, 35)])
def test_no_wide_tiles_up_to_64_rows(T, d, E, h, C):
    assert all(k.startswith("ffn_gemm_any") for k in kernels(T, d, E, h, C))


# above, the small tiles only where they are expected to be a tenth faster.  Uneven tokens made the first four lose 6 to 22 %
# of what the tiles of 256 columns take
@pytest.mark.parametrize("T,d,E,h,C,second", [(192, 4096, 8, 16384, 192, False), (700, 4096, 8, 16384, 175, False),
                                              (12000, 2048, 4, 8192, 12000, True), (700, 2560, 16, 10240, 700, True),
                                              (65536, 4096, 64, 16384, 501, True), (32768, 2048, 32, 8192, 1280, False)])
def test_wide_tiles_unless_the_small_ones_win_clearly(T, d, E, h, C, second):
    assert kernels(T, d, E, h, C)[2 * second] == ("ffn_gemm_dma_persistent" if E % 8 == 0 else "ffn_gemm_dma")


@pytest.mark.parametrize("T,d,E,h,C", [(8192, 1024, 16, 4096, 255), (2000, 2048, 4, 8192, 500), (2000, 768, 12, 3072, 334),
                                       (8192, 1024, 16, 4096, 640)])
def test_small_tiles_for_small_layers(T, d, E, h, C):
    assert kernels(T, d, E, h, C)[2].startswith("ffn_gemm_any")


# row-major weights: the dealt tiles unless another shape is expected faster.  Uneven tokens made the first three lose 22 to 41 % to
# tiles that an even spread gains 6 to 16 % with
@pytest.mark.parametrize("T,d,E,h,C,second,bn", [(700, 1024, 16, 4096, 700, True, 64), (700, 768, 6, 3072, 234, False, 64),
                                                 (5000, 1536, 12, 4096, 834, False, 128), (32768, 2048, 8, 8192, 4096, True, 128)])
def test_row_major_tiles_are_dealt(T, d, E, h, C, second, bn):
    assert kernels(T, d, E, h, C, packed=False)[2 * second] == f"ffn_gemm_any<192, {bn}, dealt>"


# the second line's shapes lose 12 to 85 % to the dealt tiles, whatever the spread of the tokens
@pytest.mark.parametrize("T,d,E,h,C,second,kernel", [
    (5003, 1600, 40, 6400, 157, True, "160, 160"), (12000, 1024, 16, 4096, 750, True, "192, 128"), (12000, 1024, 64, 2736, 188, True, "192, 128"),
    (12000, 512, 4, 2048, 3000, True, "192, 128"), (32768, 768, 6, 3072, 5462, True, "192, 128"), (32768, 2560, 16, 6832, 4096, False, "160, 160"),
    (12000, 768, 96, 3072, 125, True, "160, 160"), (12000, 640, 20, 1712, 1200, False, "160, 160")])
def test_row_major_tiles_in_runs(T, d, E, h, C, second, kernel):
    assert kernels(T, d, E, h, C, packed=False)[2 * second] == f"ffn_gemm_any<{kernel}>"


# capacities at the even share, narrow outputs or short segments
@pytest.mark.parametrize("T,d,E,h,C", [(294, 1600, 40, 3200, 8), (4096, 1024, 16, 4096, 320)])
def test_row_major_tiles_of_64_columns_in_runs(T, d, E, h, C):
    assert kernels(T, d, E, h, C, packed=False)[2] == "ffn_gemm_any<128, 64>"


def test_row_major_tiles_of_64_columns_dealt_where_128_rows_make_more_tiles():
    assert kernels(1097, 4096, 8, 10928, 172, packed=False)[2] == "ffn_gemm_any<192, 64, dealt>"


@pytest.mark.parametrize("packed,first,second,E,d,h,T,C,rows", KERNEL_SHAPES)
def test_shapes_reach_the_kernels_they_are_meant_for(packed, first, second, E, d, h, T, C, rows):
    assert len(rows) == E and max(rows) <= min(C, T) and min(rows) == 0
    assert kernels(T, d, E, h, C, packed=packed) == [first, first, second]


def test_every_kernel_has_a_shape():
    packed = {k for p, a, b, *_ in KERNEL_SHAPES if p for k in (a, b)}
    plain = {k for p, a, b, *_ in KERNEL_SHAPES if not p for k in (a, b)}
    tiles = {f"ffn_gemm_any<{t}>" for t in ("192, 128", "160, 160", "128, 64", "128, 32")}
    assert packed == tiles | {"ffn_gemm_dma", "ffn_gemm_dma_persistent"}  # (ffn_gemm_few: its own test)
    assert plain == tiles | {"ffn_gemm_any<192, 128, dealt>", "ffn_gemm_any<192, 64, dealt>"}


@pytest.mark.parametrize("packed,first,second,E,d,h,T,C,rows", KERNEL_SHAPES)
def test_shapes_have_other_tiles_to_be_compared_with(packed, first, second, E, d, h, T, C, rows):
    other_tiles(lm, first, second, E, d, h)
