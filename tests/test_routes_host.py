"""Host-only checks of which kernels the plans pick, asked of the planning code itself: the shapes that GPU tests use to reach a
kernel have to reach it, and the rules that were measured have to hold where they were measured."""
import pytest

from routes import route


# N, and the pitch of dZ where both gradients run in 128 x 128 tiles: whole lines of 64 elements where those add at most an eighth
# (57: not padded, no room for more)
@pytest.mark.parametrize("op", ["block", "relu"])
@pytest.mark.parametrize("M,K,N,pitch", [(3001, 771, 1537, 1600), (20067, 473, 824, 832), (1024, 777, 513, 576), (1025, 776, 520, 576),
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
