"""Host-only checks of which kernels the plans pick, asked of the planning code itself: the shapes that GPU tests use to reach a
kernel have to reach it, and the rules that were measured have to hold where they were measured."""
import pytest

import test_few_rows_gpu
import test_mid_tiles_gpu
import test_padded_shapes_gpu
import test_row_kernels_gpu
import test_small_workspaces_gpu
import test_special_values_gpu
import test_tile_bias_gpu
from paper_2509_14279_amd import api
from routes import route


# N, and the pitch of dZ where both gradients run in 128 x 128 tiles: whole lines of 64 elements where those add at most an eighth
# (57: not padded, no room for more)
@pytest.mark.parametrize("op", ["block", "relu"])
@pytest.mark.parametrize("M,K,N,pitch", [(3001, 771, 1537, 1600), (20067, 773, 824, 832), (1024, 777, 513, 576), (1025, 776, 520, 576),
                                         (2500, 1000, 300, 320), (9000, 100, 264, 264), (3000, 200, 71, 72), (2000, 500, 57, 57),
                                         (4097, 130, 8, 8), (1024, 512, 640, 640)])
def test_pitch_of_the_gradient(op, M, K, N, pitch):
    forward, gradients, ldz = route(op, "bf16", M, K, N)
    assert gradients.startswith("mid"), gradients
    if not (op == "relu" and forward.startswith("padded")):      # (the padded product's masking epilogue writes whole tiles)
        assert int(ldz) == pitch


# few rows whose width is even but no multiple of 8: the few-row kernel takes 27, 30, 35, 19 and 17 us, 128 x 128 tiles 43, 40, 45, 23
# and 20
@pytest.mark.parametrize("M,D,H", [(21, 3924, 3698), (36, 3114, 3032), (17, 3754, 3369), (117, 1634, 1428), (1, 718, 8352)])
def test_gate_products_of_few_even_rows(M, D, H):
    assert route("ffn", "bf16", M, D, H)[0] == "few rows"


def forward(op, shapes):
    return [route(op, "bf16", *s)[0] for s in shapes]


# the tests of infinite and very large biases, of infinities in X, of the smallest workspaces and of parity on the large tiles: each
# form of the forward product is among the shapes of each
@pytest.mark.parametrize("op", ["block", "relu"])
def test_forward_products_of_the_large_tiles(op):
    large = forward(op, test_padded_shapes_gpu.LARGE)
    assert set(large) == {"tiled", "padded", "tiled split", "padded split"}
    assert {m % 256 == 0 for (m, _, _), f in zip(test_padded_shapes_gpu.LARGE, large) if f == "tiled split"} == {True, False}
    assert {k % 128 == 0 for (_, k, _), f in zip(test_padded_shapes_gpu.LARGE, large) if f == "padded"} == {True, False}
    special = forward(op, test_special_values_gpu.SHAPES)
    assert set(special) >= set(large) | {"mid", "mid split", "few rows", "generic"}
    assert set(forward(op, [s[1:] for s in test_small_workspaces_gpu.SHAPES if s[0] == "bf16"])) >= set(large)
    assert set(forward(op, test_mid_tiles_gpu.SHAPES)) >= {"mid", "mid split"}
    assert set(forward(op, test_tile_bias_gpu.EVERY)) == set(large) | {"mid", "mid split", "few rows", "generic"}


@pytest.mark.parametrize("op", ["block", "relu"])
def test_gradients(op):
    large = {route(op, "bf16", *s)[1] for s in test_padded_shapes_gpu.LARGE}
    assert large >= {"pair padded-x", "pair padded extra", "pair extra", "tiled and tiled padded-x"}
    mid = {route(op, "bf16", *s)[1] for s in test_mid_tiles_gpu.SHAPES}
    assert mid >= {"mid", "mid dx-split", "mid dw-split", "mid dx-split dw-split"}


# dZ read by one to four columns of tiles: 128 x 128 ones were up to 11 % slower here (whole backward passes, 104 to 115, 105 to 116,
# 139 to 152, 134 to 147 us)
@pytest.mark.parametrize("M,K,N", [(8857, 216, 3592), (7336, 152, 4488), (6656, 381, 5808), (35638, 248, 1128)])
def test_gradients_of_few_columns_and_a_large_dz(M, K, N):
    assert not route("block", "bf16", M, K, N)[1].startswith("mid")


def test_blocked_gradients():
    narrow = [s for s in test_row_kernels_gpu.BLOCKED if "blocked" in route("block", "bf16", *s)[1]]
    assert narrow == test_row_kernels_gpu.BLOCKED[1:]
    assert min(n for _, _, n in narrow) <= 512 < max(n for _, _, n in narrow) <= 1024


def test_feed_forward_products():
    expected = {"padded | padded", "padded | padded split", "tiled | tiled", "tiled | tiled split", "tiled | mid"}
    for shapes in (test_padded_shapes_gpu.LARGE_FFN, test_special_values_gpu.FFN):
        assert {" | ".join(route("ffn", "bf16", *s)) for s in shapes} >= expected
    assert "mid | tiled split" in {" | ".join(route("ffn", "bf16", *s)) for s in test_padded_shapes_gpu.LARGE_FFN}


# from 16384 rows on the activation passes to the down product in blocks, whose weights are then copied into such blocks; an activation
# that comes as rows gains nothing from the copy, and the workspace has no room for it
@pytest.mark.parametrize("M,D,H,gate,down", [(16384, 4096, 11008, "tiled", "tiled from blocks"), (16384, 1024, 4096, "tiled", "tiled from blocks"),
                                             (16385, 512, 1024, "mid", "tiled"), (32805, 256, 512, "mid", "tiled")])
def test_the_down_products_copy_goes_with_the_blocked_activation(M, D, H, gate, down):
    assert route("ffn", "bf16", M, D, H) == [gate, down]
    rows = (M + 255) // 256 * 256
    tails = 2 * (256 * D * 2 + 256)
    assert api.fdl_llama_ffn_workspace_bytes("bf16", M, D, H) <= rows * H * 2 + (D * H * 2 if "blocks" in down else 0) + tails


def test_long_reductions_of_few_rows():
    assert {route("relu", "bf16", *s)[0] for s in test_few_rows_gpu.LINES} == {"few rows"}
    assert {tuple(route("ffn", "bf16", *s)) for s in test_few_rows_gpu.LINES_FFN} <= {("few rows", "few rows"), ("few rows", "mid split")}
    assert sum(route("ffn", "bf16", *s)[1] == "few rows" for s in test_few_rows_gpu.LINES_FFN) >= 12


# fp32 gradients in 32 x 32 tiles, unless a long reduction of few of them is one wavefront's chain (whole calls, us, so / in split 64 x 64
# tiles: 42.8 / 35.5, 35.5 / 29.8, 31.5 / 28.1, 30.6 / 27.2; and where they are faster 20.5 / 25.5, 36.6 / 44.3, 36.5 / 43.3, 44.6 / 49.6)
@pytest.mark.parametrize("op", ["block", "relu"])
@pytest.mark.parametrize("M,K,N,tiles", [(24, 512, 1024, 64), (26, 512, 1024, 64), (1016, 88, 48, 64), (27, 256, 1024, 64),
                                         (256, 256, 256, 32), (300, 300, 700, 32), (1000, 200, 300, 32), (256, 512, 1024, 32)])
def test_small_fp32_gradients(op, M, K, N, tiles):
    assert route(op, "f32", M, K, N)[1] == f"{tiles} x {tiles}"
