"""GPU parity of the tile kernels at the row counts where a tile, a chunk or a segment begins,
ends or has one row too many, over the head dimensions whose kernels split work differently.

Where the suite's general tolerances leave room the bounds are tighter: an fp32 output is a sum of at
most N + 2 d products, each rounded to 2^-24 of its size (and every partial sum again), which is off by a
few times sqrt(N + 2 d) 2^-24 of the sum of the products' sizes.  Measured against the largest output,
which may be smaller than that sum where terms cancel, (N + 2 d) 2^-23 is an empirical bound: for these
values the error stays below a tenth of it."""
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
    for i, (B, H, N) in enumerate([(2, 2, 1), (2, 3, 127), (2, 2, 128), (12, 8, 129) if wide else (1, 2, 129),
                                   (12, 8, 256) if wide else (2, 2, 256), (20, 8, 257), (16, 12, 513)]):
        if N > 256 and (dk, dv) not in ((32, 32), (64, 64)):
            continue
        cottn.profile_start()
        run_shape(cottn, oracle, False, B, H, N, dk, dv, dtype, seed=1600 + dk + dv + N, saved=i % 2 == 1)
        names = {"fwd_bidir_unit_" + dtype, "bwd_bidir_unit_" + dtype}
        # (32 x 32 beyond 512 rows is split in any case)
        assert names <= set(cottn.profile_stop()) or (N > 512 and dk == 32), (B, H, N)


def _sums_launched(cottn):
    """Whether a launch of its own added up segment totals since profile_start()."""
    return bool({"fwd_state_carry", "bwd_state_carry", "bidir_combine"} & set(cottn.profile_stop()))


# (d, segments, whether a launch of its own adds the totals up): both sides of each line, at two units
@pytest.mark.parametrize("d,segments,launch", [(64, 5, False), (64, 18, False), (64, 19, True), (64, 25, True), (128, 4, False),
                                               (128, 5, True), (128, 11, True), (32, 17, False)])
def test_causal_totals_added_in_place_or_carried(cottn, oracle, d, segments, launch):
    """Up to a number of segments the scans add the segment totals up themselves, beyond it a launch of
    its own does: both sides of the line, batches of totals that do not divide, states handed over or not."""
    for dtype, rows, saved in (("bf16", 64, True), ("f16", 64, False), ("f32", 32, True), ("f32", 32, False)):
        cottn.profile_start()
        run_shape(cottn, oracle, True, 1, 2, rows * segments - 5, d, d, dtype, seed=1400 + d + segments,
                  segments=segments, saved=saved)
        assert cottn.cottn_segments(cottn.OP_FWD_CAUSAL, 1, 2, rows * segments - 5, d, 0, cottn.COTTN_F32 if dtype == "f32"
                                    else cottn.COTTN_BF16) == segments
        assert _sums_launched(cottn) == launch


@pytest.mark.parametrize("dtype,segments,launch", [("f32", 10, False), ("f32", 11, True), ("bf16", 7, False), ("f16", 8, True)])
def test_causal_totals_of_sixteen_units(cottn, oracle, dtype, segments, launch):
    """With the units the line of 128 x 128 moves further in fp32 than in 16 bits."""
    rows = 32 if dtype == "f32" else 64
    cottn.profile_start()
    run_shape(cottn, oracle, True, 2, 8, rows * segments - 5, 128, 128, dtype, seed=1450 + segments, segments=segments,
              saved=segments % 2 == 0)
    assert _sums_launched(cottn) == launch


# (width, units, segments, steps of a segment, whether carry launches add up): both sides of the same lines with so
# many rows before the last segment that no call forms its state from them
@pytest.mark.parametrize("d,units,segments,steps,carry", [(64, 2, 5, 2, False), (64, 2, 18, 2, False), (64, 2, 19, 2, True),
                                                          (128, 2, 4, 5, False), (128, 2, 5, 2, True), (128, 16, 7, 2, False),
                                                          (128, 16, 8, 2, True), (32, 2, 17, 2, False)])
def test_causal_totals_of_long_segments(cottn, oracle, d, units, segments, steps, carry):
    for dtype, saved in (("bf16", True), ("f16", False)):
        N = 64 * steps * segments - 5
        cottn.profile_start()
        run_shape(cottn, oracle, True, 2, units // 2, N, d, d, dtype, seed=1460 + d + segments, segments=segments, saved=saved)
        names = set(cottn.profile_stop())
        assert "fwd_segment_state_" + dtype in names
        assert ("fwd_state_carry" in names) == carry and ("bwd_state_carry" in names) == carry


# fp32 steps are 32 rows; at 128 x 128 and 16 units the line lies further, and two segments of any length start from
# their own prefix up to 224 rows
@pytest.mark.parametrize("d,units,segments,steps,carry", [(64, 2, 5, 3, False), (64, 2, 18, 2, False), (64, 2, 19, 2, True),
                                                          (128, 2, 4, 1, False), (128, 16, 10, 1, False), (128, 16, 11, 1, True)])
def test_causal_totals_of_long_segments_f32(cottn, oracle, d, units, segments, steps, carry):
    N = 32 * steps * segments - 5
    cottn.profile_start()
    run_shape(cottn, oracle, True, 2, units // 2, N, d, d, "f32", seed=1480 + d + segments, segments=segments, saved=False)
    names = set(cottn.profile_stop())
    assert "fwd_segment_state_f32" in names
    assert ("fwd_state_carry" in names) == carry and ("bwd_state_carry" in names) == carry


@pytest.mark.parametrize("d,segments,launch", [(64, 5, False), (64, 24, False), (64, 25, True), (128, 10, False),
                                               (128, 11, True), (32, 17, False)])
def test_bidirectional_totals_added_in_place_or_combined(cottn, oracle, d, segments, launch):
    for dtype, rows, saved in (("bf16", 128, True), ("f16", 128, False), ("f32", 64, True), ("f32", 64, False)):
        cottn.profile_start()
        run_shape(cottn, oracle, False, 1, 1, rows * segments - 5, d, d, dtype, seed=1500 + d + segments,
                  segments=segments, saved=saved)
        assert cottn.cottn_segments(cottn.OP_FWD_BIDIR, 1, 1, rows * segments - 5, d, 0, cottn.COTTN_F32 if dtype == "f32"
                                    else cottn.COTTN_BF16) == segments
        assert _sums_launched(cottn) == launch


@pytest.mark.parametrize("segments", [1, 3])
@pytest.mark.parametrize("dk,dv", [(32, 32), (64, 64), (128, 128), (64, 128), (128, 32)])
def test_f32_beyond_256_workgroups(cottn, oracle, monkeypatch, dk, dv, segments):
    """The waves of the fp32 scans swap their row groups from workgroup to workgroup of a compute unit,
    every 256 of them: results and states of both kinds."""
    N = 70
    monkeypatch.setitem(test_gpu_dkdv.TOL, "f32", (N + 2 * max(dk, dv)) * 2.0 ** -23)
    run_shape(cottn, oracle, True, 53, 5, N, dk, dv, "f32", seed=1700 + dk + dv, segments=segments, saved=True)
