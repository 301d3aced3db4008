"""Which kernel variant the rules of launch.h choose, on both sides of their lines and for the shapes that the GPU tests
of a variant list: the compiler evaluates the rules (no GPU, nothing is run)."""
import shutil
import subprocess

import pytest

from paper_2409_18747_amd import build
from test_gpu_two_to_a_cu import FROM_TOTALS

pytestmark = pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="needs the compiler")


def holds(tmp_path, rules):
    src = tmp_path / "rules.hip"
    src.write_text('#include "%s/launch.h"\nusing namespace cottn;\n' % build.CSRC
                   + "".join('static_assert(%s, "%s");\n' % (r, r) for r in rules))
    run = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-fsyntax-only", str(src)],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr


def test_value_parts(tmp_path):
    """Four parts up to 64 rows and two beyond at up to 128 units of 128 wide keys, two up to 256 of narrower ones."""
    rules = ["value_parts(%d, %d, 128) == %d" % (u, n, 1 if u > 128 else 4 if n <= 64 else 2)
             for u in (1, 2, 6, 127, 128, 129, 130, 258, 512) for n in (1, 5, 32, 33, 63, 64, 65, 129, 2048)]
    rules += ["value_parts(%d, %d, %d) == %d" % (u, n, dk, 1 if u > 256 else 2)
              for u in (1, 130, 256, 257, 258) for n in (1, 64, 65, 500) for dk in (32, 64)]
    holds(tmp_path, rules)


def test_two_to_a_compute_unit(tmp_path):
    rules = ["%stwo_to_a_cu_%s(%d)" % ("" if yes else "!", scan, w)
             for scan, line in (("forward", [(256, 0), (257, 1), (640, 1), (641, 0), (768, 0), (769, 1)]),
                                ("dq", [(256, 0), (257, 1), (512, 1), (513, 0), (768, 0), (769, 1)]),
                                ("dkdv", [(256, 0), (257, 1), (700, 1), (5000, 1)])) for w, yes in line]
    # the GPU test of segments that start from totals: no state of their own forming
    for units, N, G in FROM_TOTALS:
        chunks = (N + 63) // 64
        rows = (chunks + G - 1) // G * 64
        assert -(-chunks // (rows // 64)) == G
        rules += ["two_to_a_cu_forward(%d)" % (units * G), "two_to_a_cu_dkdv(%d)" % (units * G),
                  "!own_prefix(%d, %d, %d, 128, 128, false)" % (units, G, rows), "causal_totals_in_place(%d, %d, 128, 128, false)" % (units, G)]
    holds(tmp_path, rules)


def test_own_prefix(tmp_path):
    """(units, segments, rows of a segment, widths, fp32): the last that the forward takes, and the dQ scan, and the next."""
    rules = []
    for units, G, rows, dk, dv, f32, forward, dq in [
            (10, 10, 64, 64, 64, 0, 1, 1), (10, 11, 64, 64, 64, 0, 0, 0), (40, 4, 128, 64, 64, 0, 1, 1), (40, 5, 128, 64, 64, 0, 0, 0),
            (120, 4, 192, 64, 64, 0, 1, 0), (120, 4, 256, 64, 64, 0, 0, 0), (10, 16, 64, 32, 32, 0, 1, 1), (10, 17, 64, 32, 32, 0, 0, 0),
            (2, 13, 64, 64, 128, 0, 1, 1), (2, 14, 64, 64, 128, 0, 0, 0), (2, 13, 64, 128, 64, 0, 0, 0), (100, 2, 320, 128, 128, 0, 1, 1),
            (60, 4, 256, 128, 128, 0, 1, 0), (60, 4, 320, 128, 128, 0, 0, 0), (2, 7, 32, 64, 64, 1, 1, 1), (2, 8, 32, 64, 64, 1, 0, 0),
            (100, 2, 224, 64, 128, 1, 1, 1), (100, 2, 256, 64, 128, 1, 0, 0), (100, 1, 64, 64, 64, 0, 0, 0)]:
        args = "%d, %d, %d, %d, %d, %s" % (units, G, rows, dk, dv, "true" if f32 else "false")
        rules += ["own_prefix(%s) == %s" % (args, "true" if forward else "false"), "own_prefix_dq(%s) == %s" % (args, "true" if dq else "false")]
    holds(tmp_path, rules)


def test_own_prefix_by_sets(tmp_path):
    """Four steps at a time at 32 x 32, and in the 16-bit forward at 64 x 32, up to 256 workgroups."""
    rules = ["prefix_by_sets(256)", "!prefix_by_sets(257)"]
    for dk in (32, 64, 128):
        for dv in (32, 64, 128):
            for f32 in (False, True):
                for forward in (False, True):
                    four = (dk, dv) == (32, 32) or ((dk, dv) == (64, 32) and forward and not f32)
                    rules.append("prefix_sets_built(%d, %d, %s, %s) == %d" % (dk, dv, str(f32).lower(), str(forward).lower(), 4 if four else 1))
    holds(tmp_path, rules)


def test_quotients_of_kernel_arguments(tmp_path):
    """Divisor and quotient: around multiples of small and large divisors, up to the largest row numbers and indexes."""
    rules = []
    for n in (1, 2, 3, 7, 8, 12, 13, 96, 641, 777, 1000, 4096, 65535, 65537, 16777216, 1073741823, 2147483647):
        xs = {0, 1, n - 1, n, 2147483647, 2147483646, 2147483647 // n * n, 2147483647 // n * n - 1, 536870912, 1234567890}
        xs |= {k * n + e for k in (1, 2, 3, 1000003) for e in (-1, 0, 1)}
        rules += ["quotient(%d, Divisor(%d)) == %d" % (x, n, x // n) for x in sorted(xs) if 0 <= x <= 2147483647]
    holds(tmp_path, rules + ["Divisor(0) == 0"])


def test_states_at_once(tmp_path):
    """Up to two tiles a wave take six stored states at once, five to eight four, but not where sixteen waves hold 64 x 64."""
    rules = ["states_at_once(%d) == %d" % (t, n) for t, n in ((1, 3), (4, 3), (5, 2), (8, 2), (9, 1), (16, 1))]
    for waves in (4, 8, 15, 16):
        for tiles, elements, n in ((1, 64 * 64, 6 if waves < 16 else 3), (2, 64 * 64, 6 if waves < 16 else 3), (1, 32 * 32, 6),
                                   (4, 64 * 64, 3), (8, 64 * 128, 4 if waves < 16 else 2), (8, 128 * 128, 2), (16, 128 * 128, 1)):
            rules.append("states_at_once_of_many(%d, %d, %d) == %d" % (tiles, elements, waves, n))
    holds(tmp_path, rules)


def test_argument_bytes(tmp_path):
    """As the compiler lays kernel arguments out (that those of the forward scan stay within 128 bytes is asserted at its launch)."""
    holds(tmp_path, ["argument_bytes<void*, int, void*>() == 24", "argument_bytes<int, Divisor, int>() == 16", "argument_bytes<>() == 0",
                     "argument_bytes<const float*, Divisor, int, const int*, int>() == 36",
                     "(SUM_TOTALS | SCALE_PER_UNIT | STREAM_Q | STREAM_KV) == 15"])
