"""GPU parity of the tile kernels at the row counts where a tile, a chunk or a segment begins,
ends or has one row too many, over the head dimensions whose kernels split work differently.

The bounds are derived, not the suite's general tolerances, where those leave room: an fp32 output
is a sum of at most N + 2 d products, each rounded to 2^-24 of its size (and every partial sum
again), so it is off by a few times sqrt(N + 2 d) 2^-24 of the largest output, and never by more
than (N + 2 d) 2^-23."""
import pytest

from test_gpu_dkdv import run as run_shape
import test_gpu_dkdv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    yield b
    b.cottn_tune_segments(0)


ROWS = [1, 31, 32, 33, 64, 65, 97, 161]
DIMS = [(32, 32), (64, 64), (128, 128), (32, 128), (128, 32), (64, 128), (128, 64)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dk,dv", DIMS)
def test_f32(cottn, oracle, monkeypatch, causal, dk, dv):
    for i, N in enumerate(ROWS):
        monkeypatch.setitem(test_gpu_dkdv.TOL, "f32", (N + 2 * max(dk, dv)) * 2.0 ** -23)
        run_shape(cottn, oracle, causal, 2, 2, N, dk, dv, "f32", seed=1200 + dk + dv + N,
                  segments=[0, 1, 2, 3][i % 4], saved=i % 2 == 1)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("dk,dv", [(64, 128), (128, 64)])
def test_16bit_wide_rectangles(cottn, oracle, dtype, dk, dv):
    """The backward takes these in steps of 32 rows with two waves per row group."""
    for i, N in enumerate(ROWS):
        run_shape(cottn, oracle, True, 2, 2, N, dk, dv, dtype, seed=1300 + dk + N,
                  segments=[0, 1, 2][i % 3], saved=i % 2 == 1)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_16bit_widest(cottn, oracle, dtype):
    """128 x 128: 64-row steps with two waves per row group."""
    for i, N in enumerate(ROWS):
        run_shape(cottn, oracle, True, 2, 2, N, 128, 128, dtype, seed=1350 + N,
                  segments=[0, 1, 2][i % 3], saved=i % 2 == 1)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("dk,dv", DIMS)
def test_bidirectional_by_unit(cottn, oracle, dtype, dk, dv):
    """A (batch, head) per workgroup in 128-row steps: edges of a step, and the most rows for few, for
    many (160) and for very many (192) of them."""
    wide = dk == 128 and dv == 128
    for i, (B, H, N) in enumerate([(2, 2, 1), (2, 3, 127), (2, 2, 128), (8, 8, 129) if wide else (1, 2, 129),
                                   (8, 8, 256) if wide else (2, 2, 256), (20, 8, 257), (16, 12, 513)]):
        if N > 256 and (dk, dv) not in ((32, 32), (64, 64)):
            continue
        run_shape(cottn, oracle, False, B, H, N, dk, dv, dtype, seed=1600 + dk + dv + N, saved=i % 2 == 1)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d,segments", [(64, 5), (64, 24), (64, 25), (128, 10), (128, 11), (32, 17)])
def test_segment_totals_added_in_place_or_carried(cottn, oracle, causal, d, segments):
    """Up to a number of segments the kernels add the segment totals up themselves, beyond it a
    launch of its own does: both sides of the line, and batches of totals that do not divide."""
    N = 64 * segments - 10
    run_shape(cottn, oracle, causal, 1, 2, N, d, d, "bf16", seed=1400 + d + segments, segments=segments, saved=True)
    run_shape(cottn, oracle, causal, 1, 1, 32 * segments - 5, d, d, "f32", seed=1500 + d + segments,
              segments=segments, saved=False)
