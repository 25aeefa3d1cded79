"""The choice of kernels on the CPU, at shapes where both sides were measured (us beside each case: this choice / the others;
tile shapes: of the product, on packed weights)."""
import pytest

from tests.plan_util import plan, plan_f32

T256, T256N, T128, T128X2, T128N = 256256, 256128, 128256, 128257, 128128
W256, W256H, W256G, W128, W128H = 256258, 256259, 256260, 128258, 128259     # four-wave kernel: cached, with the hint, by group


@pytest.mark.parametrize("T,d,f,E,k,C,residual,which,kernel", [
    # room for few more than 128 rows, or for many more than there are: 256 x 128 tiles where 256 x 256 ones are too few
    (832, 4096, 16384, 8, 1, 130, False, 1, T256N),      # 224 / 260 (128 x 256), 243 (256 x 256)
    (682, 4096, 16384, 8, 1, 256, False, 1, T256N),      # 214 / 253, 235
    (2080, 2048, 8192, 16, 1, 130, False, 1, T256N),     # 126 / 138, 136
    (4160, 1024, 4096, 32, 1, 130, False, 1, T256N),     # 66 / 71, 76
    (800, 4096, 4096, 2, 1, 1200, False, 1, T256N),      # 68 / 110, 80
    (2000, 520, 2080, 16, 1, 156, False, 0, W256),       # 20 / 25 in two rounds of 256 x 128
    # rows that fill their tiles: as before
    (4001, 1024, 4096, 32, 2, 251, False, 1, W128),      # 80 / 93 (256 x 256)
    (8192, 1024, 4096, 32, 1, 256, True, 0, W256G),
    (16384, 4096, 16384, 64, 2, 640, False, 0, W256G),
    (1500, 1024, 4096, 16, 1, 117, False, 1, T128N),     # 50 / 58 (128 x 256)
    # two products in a launch, the experts' with few more than 128 rows: not two small tiles per compute unit
    (1664, 2048, 8192, 16, 1, 130, True, 0, W256G),      # 137 / 215
    (3328, 1024, 4096, 32, 1, 130, True, 0, W256G),      # 84 / 116
])
def test_tile_shape(T, d, f, E, k, C, residual, which, kernel):
    assert plan(T, d, f, E, k, C, residual, packed=True)[0][which] == kernel


@pytest.mark.parametrize("T,d,f,E,k,C,residual,which,kernel", [
    # packed weights, 256 columns: the four-wave kernel; weights of more than 128 MB that one row tile reads get the hint
    (8192, 1024, 4096, 64, 1, 128, True, 0, W128H), (8192, 1024, 4096, 64, 1, 128, True, 1, W256G), (8192, 1024, 4096, 64, 1, 128, True, 2, W256),
    (4001, 1024, 4096, 32, 2, 251, False, 0, W256H), (4001, 1024, 2048, 32, 2, 251, False, 0, W256),
    # a pair of products of which one has groups of at most 128 rows: us with 128 / 256 rows
    (2069, 1024, 4096, 32, 1, 97, True, 1, W128),        # 69 / 82
    (979, 1024, 2048, 16, 1, 77, True, 0, W128),         # 24 / 31
    (2870, 1024, 2048, 64, 1, 68, True, 0, W256G),       # 71 / 66
    (300, 256, 32, 64, 1, 300, True, 1, W128),
    # two tiles per compute unit chosen: K up to 512 (four waves with 128, 256 rows / here), beyond it 128 or 256 rows
    (9585, 256, 1024, 128, 2, 300, False, 0, T128X2),    # 36, 48 / 32
    (13866, 512, 2048, 16, 1, 1084, True, 0, T128X2),    # 85, 75 / 76
    (12000, 1024, 4096, 16, 1, 800, False, 0, W256),     # 125 / 112
    (16384, 1024, 4096, 64, 1, 260, False, 0, W128),     # 203 / 224
    (16384, 2048, 8192, 64, 1, 300, False, 0, W128),     # 680 / 748
    (6466, 2048, 8192, 16, 1, 809, False, 0, W128),      # 147 / 213 (skewed routing)
])
def test_four_wave_kernel(T, d, f, E, k, C, residual, which, kernel):
    assert plan(T, d, f, E, k, C, residual, packed=True)[0][which] == kernel


@pytest.mark.parametrize("T,d,f,E,C,packed,kernel", [
    # inner dimension off 32, few experts: the streaming kernel with K split for the second product (layer / on tiles)
    (124, 1000, 4000, 2, 156, False, 864),       # 78 / 92
    (102, 2008, 8032, 1, 128, False, 864),       # 116 / 161
    (102, 2008, 8032, 1, 128, True, 864),        # 110 / 148
    # many rows or many tiles, and whole stages
    (800, 1000, 4000, 1, 1000, False, T128N),    # 97 / 120 (streaming)
    (1280, 1000, 4000, 4, 400, False, T128N),    # 99 / 137
    (409, 1000, 1000, 4, 128, False, T128N),     # 54 / 63
    (3200, 1000, 4000, 16, 250, True, T128N), (124, 1024, 4096, 2, 156, False, T128N),
])
def test_ragged_inner_dimension(T, d, f, E, C, packed, kernel):
    assert plan(T, d, f, E, 1, C, False, packed)[0][1] == kernel


@pytest.mark.parametrize("T,d,f,E,C,packed,which,kernel", [
    # first product beyond 48 K columns: the few-weights kernel while some experts are missed, the streaming one (116) when not
    (64, 2048, 8192, 128, 1, True, 0, 4), (64, 2048, 8192, 64, 4, True, 0, 4), (64, 2048, 8192, 32, 8, True, 0, 4),
    (128, 2048, 8192, 8, 16, True, 0, 116), (64, 2048, 8192, 16, 8, True, 0, 116), (96, 2048, 8192, 8, 12, True, 0, 116),
    (96, 2048, 8192, 12, 16, True, 0, 4),
    # second product: many rows per expert, few columns per work-group, long K: streaming with K split
    (64, 2048, 8192, 1, 64, True, 1, 864), (256, 2048, 8192, 4, 64, True, 1, 864), (48, 4096, 16384, 2, 24, True, 1, 832),
    (64, 1024, 4096, 1, 64, True, 1, 864), (32, 2048, 8192, 2, 16, False, 1, 816),
    (128, 2048, 8192, 32, 8, True, 1, 2), (16, 2048, 8192, 64, 1, True, 1, 2), (128, 4096, 16384, 8, 16, True, 1, 4),
    (2, 2048, 8192, 8, 1, False, 1, 2), (64, 128, 512, 1, 64, True, 1, 1), (12, 4096, 16384, 8, 2, True, 1, 2),
    (32, 1024, 4096, 2, 32, True, 1, 1), (4, 1024, 4096, 1, 4, False, 1, 2),
])
def test_few_rows(T, d, f, E, C, packed, which, kernel):
    assert plan(T, d, f, E, 1, C, False, packed)[0][which] == kernel


@pytest.mark.parametrize("T,d,f,E,k,C,packed,which,kernel", [
    # few rows per expert, beyond 48 K columns of a first product with K = 1024: the few-weights kernel (us, streaming / here, even and skewed)
    (16, 1024, 4096, 64, 1, 1, True, 0, 4),              # layer 57.6 / 53.4, 38.8 / 22.7
    (64, 1024, 4096, 128, 1, 1, True, 0, 4),             # 141 / 139, 42.6 / 28.5
    (180, 1024, 4096, 128, 1, 2, True, 0, 4),            # 280 / 261, 88 / 44, with the second product
    # ... the streaming kernel where the tokens reach most of few experts, or with plain weights
    (64, 1024, 4096, 32, 1, 4, True, 0, 116), (20, 1024, 4096, 64, 1, 1, False, 0, 116),
    # second product, waves enough for the streaming kernel without a split
    (64, 2048, 8192, 64, 1, 2, True, 1, 1),              # 453 / 423, 136 / 70
    (96, 2048, 8192, 128, 1, 2, True, 1, 1),             # 729 / 664, 203 / 85
    (180, 1024, 4096, 128, 1, 2, True, 1, 1),
    # ... not with few of the experts, nor with more rows per expert
    (64, 2048, 8192, 128, 1, 1, True, 1, 116), (90, 2048, 8192, 64, 1, 3, True, 1, 116),
    # K below 8192: up to 256 rows
    (100, 1024, 4096, 64, 2, 7, True, 1, 1),             # 180 / 174, 50 / 43
])
def test_few_rows_per_expert(T, d, f, E, k, C, packed, which, kernel):
    assert plan(T, d, f, E, k, C, False, packed)[0][which] == kernel


@pytest.mark.parametrize("T,d,f,E,k,C,residual,kernels", [
    # fp32: both products of a narrow FFN; the next ones beyond
    (256, 64, 256, 8, 1, 32, True, ["ffn"] * 4), (2500, 64, 228, 32, 1, 1024, False, ["ffn", "ffn"]),
    (2500, 64, 228, 32, 1, 1025, False, ["tile", "tile_narrow"]), (100, 68, 256, 3, 1, 40, False, ["rows32", "rows32"]), (100, 64, 260, 3, 1, 16, False, ["rows16", "rows16"]),
    # at most 512 tiles of 32 x 64: split from K = 512 on, four waves beyond 256 tiles that have rows
    (1024, 512, 2048, 8, 1, 128, False, ["split2", "rows_split8"]), (300, 512, 2048, 4, 1, 75, True, ["rows_split4", "rows_split8", "rows_split4", "rows_split8"]),
    (300, 508, 508, 4, 1, 75, False, ["rows32", "rows32"]), (300, 516, 508, 4, 1, 16, False, ["rows16", "rows16"]),
    (2048, 512, 2048, 8, 1, 256, False, ["split1", "rows_split4"]), (1024, 512, 2048, 8, 1, 256, False, ["split2", "rows_split8"]),
    # more of them: split from K = 160 (more than 256 tiles of 64 x 128 that have rows) and 256 on, more than 64 columns
    (1536, 512, 2048, 8, 2, 480, False, ["split1", "split2"]), (16000, 156, 1024, 8, 1, 2000, False, ["tile", "split1"]), (16000, 160, 1024, 8, 1, 2000, False, ["split1", "split1"]),
    (4000, 192, 256, 8, 1, 600, False, ["tile", "rows32"]), (4096, 64, 1024, 8, 1, 2100, False, ["tile", "tile_narrow"]),
    (1000, 16777216, 512, 1, 1, 1000, False, ["rows_split8", "rows32"]),      # columns beyond a buffer descriptor's offsets
])
def test_f32_kernels(T, d, f, E, k, C, residual, kernels):
    assert plan_f32(T, d, f, E, k, C, residual) == kernels
