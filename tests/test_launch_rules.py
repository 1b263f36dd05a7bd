"""The rules by which the host picks kernels and divides work, called through the library's own functions.  No GPU needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_08358_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not available")


def _run(tmp_path, body):
    """Compiles a main() around `body` against the library's headers and library, runs it and returns what it prints."""
    src, exe, lib = tmp_path / "rules.hip", tmp_path / "rules", os.path.dirname(CSRC)
    src.write_text('#include <stdio.h>\n#include "mar_split.h"\nint main() {\n' + body + "\nreturn 0;\n}\n")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe), "-L", lib,
                        "-lmarius_hip", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split()


def test_one_workgroup_sorts_less_where_nothing_runs_beside_it(tmp_path):
    """One workgroup takes longer over 9,000 to 16,384 rows than the launches it replaces: in the pipeline and above 256 floats,
    where its own time counts, half as many rows."""
    out = _run(tmp_path, """for (int alone = 0; alone < 2; ++alone) for (int dk : {16, 256, 260, 400}) printf("%d ", mar_sort_one_limit(dk, alone));""")
    assert [int(x) for x in out] == [16384, 16384, 8192, 8192] + [8192] * 4


def test_shares_of_an_evaluation_cover_every_tile_once(tmp_path):
    """Units of one or two tiles are never cut into shares (their borders could not be moved to a unit's); in all others the
    shares follow one another from the first tile to the last, and no piece of a unit is a single tile."""
    out = _run(tmp_path, """
  MarDims d = {};
  d.dk = 400; d.bilinear = 1;
  long taken = 0, bad = 0;
  for (int ntiles = 1; ntiles <= 70; ++ntiles) for (long units : {30L, 257L, 684L, 2048L, 9001L}) for (int sy : {1, 2, 4, 64}) {
    const int tps = (ntiles + sy - 1) / sy;
    if (!mar_plan_shares(d, units, ntiles, sy, tps)) continue;
    ++taken;
    const int64_t tiles = (int64_t)units * ntiles, share = tiles / MAR_SHARES;
    const int32_t rest = (int32_t)(tiles % MAR_SHARES);
    if (ntiles < 3 || sp_share_border(share, rest, ntiles, 0) != 0 || sp_share_border(share, rest, ntiles, MAR_SHARES) != tiles) ++bad;
    for (int p = 0; p < MAR_SHARES; ++p) {
      const int64_t at = sp_share_border(share, rest, ntiles, p), end = sp_share_border(share, rest, ntiles, p + 1);
      if (end < at) ++bad;
      for (int64_t t = at; t < end;) {
        const int64_t unit_end = (t / ntiles + 1) * ntiles, piece = (unit_end < end ? unit_end : end) - t;
        if (piece < 2) ++bad;
        t += piece;
      }
    }
  }
  printf("%ld %ld", taken, bad);""")
    assert int(out[0]) > 100 and out[1] == "0", out


def test_sizes_of_the_row_order_tests(tmp_path):
    """The batches that are meant to fill one workgroup's sort exactly, or to be just beyond it, do."""
    from test_gpu_row_order import ROWS
    sizes = list(ROWS)
    out = _run(tmp_path, """
  const int c[][4] = {%s};
  for (auto& k : c) {
    MarDims d = {};
    d.bilinear = 1; d.dim = k[0]; d.dk = (k[0] + 3) & ~3; d.B = k[1]; d.C = k[2]; d.S = k[1] / k[2]; d.N = k[3];
    const int sr = mar_stripe_rows(d, 2);
    int32_t sy, tps;
    mar_plan_parts(d, 2, 2L * d.C * ((d.N + sr - 1) / sr), d.S, &sy, &tps);
    printf("%%ld ", 3L * d.B + 2L * d.C * d.N * sy);
  }""" % ", ".join("{%d, %d, %d, %d}" % k for k in sizes))
    assert [int(x) for x in out] == [ROWS[k] for k in sizes]


def test_sizes_of_the_shared_evaluation_tests(tmp_path):
    """The evaluations that are meant to be cut into shares are: not on dense operands as a whole, each chunk alone is."""
    from test_gpu_operand_split import SHARED
    out = _run(tmp_path, """
  const int c[][4] = {%s};
  for (auto& k : c) {
    MarDims d = {};
    d.bilinear = 1; d.dim = k[0]; d.dk = (k[0] + 3) & ~3; d.C = k[1]; d.S = k[2]; d.N = k[3]; d.B = d.C * d.S;
    MarBatch b = {};
    b.n = d.B - d.S / 2; b.nchunks = (b.n + d.S - 1) / d.S;
    const int sr = mar_stripe_rows(d, 3), ntiles = (d.N + 31) / 32;
    const long units = 2L * b.nchunks * ((d.S + sr - 1) / sr);
    int32_t sy, tps;
    mar_plan_parts(d, 3, units, d.N, &sy, &tps);
    MarBatch one = {};
    one.n = d.S;
    printf("%%d%%d%%d ", (int)mar_eval_dense(d, b), (int)mar_plan_shares(d, units, ntiles, sy, tps), (int)mar_eval_dense(d, one));
  }""" % ", ".join("{%d, %d, %d, %d}" % k for k in SHARED))
    assert out == ["011"] * len(SHARED), out


def plan(tmp_path, configs, fields):
    """What the library plans for configurations (nodes, relations, dim, model, batch, chunks, negatives): the printed C expressions of d."""
    out = _run(tmp_path, """
  const long c[][7] = {%s};
  for (auto& k : c) {
    mar_config cfg = {k[0], (int32_t)k[1], (int32_t)k[2], (int32_t)k[3], (int32_t)k[4], (int32_t)k[5], (int32_t)k[6], 0, 0.1f, 1e-10f, 0.001f, 0, 0, 0};
    MarDims d = {};
    if (mar_check_config(&cfg, &d)) return 1;
    printf("%s ", %s);
  }""" % (", ".join("{%s}" % ", ".join(map(str, k)) for k in configs), " ".join(["%ld"] * len(fields)), ", ".join("(long)(%s)" % f for f in fields)))
    out = [int(x) for x in out]
    return [tuple(out[i:i + len(fields)]) for i in range(0, len(out), len(fields))]


def test_smallest_steps_stay_on_the_callers_stream(tmp_path):
    """Also those that cannot carry the row order because their ids have more than 27 bits, up to 4,096 gradient rows."""
    big = (1 << 27) + 1000
    got = plan(tmp_path, [(big, 3, 4, 0, 200, 2, 50), (big, 3, 4, 0, 1000, 1, 90), (10_000, 3, 300, 0, 1280, 128, 1), (10_000, 10, 50, 0, 1000, 10, 100)],
               ("d.n_pos_max <= 4096", "d.order_rides", "d.one_stream"))
    assert got == [(1, 0, 1), (0, 0, 0), (1, 0, 0), (0, 1, 1)], got


def test_sizes_of_the_one_workgroup_tests(tmp_path):
    """Steps with ids above 27 bits: none carries its order, those up to 16,384 gradient rows are sorted by one workgroup."""
    from test_gpu_row_order import ONE_WORKGROUP
    sizes = list(ONE_WORKGROUP)
    got = plan(tmp_path, [((1 << 27) + 1000, 3, 4, 0) + k for k in sizes], ("d.n_pos_max", "d.order_rides", "d.n_pos_max <= d.sort_one", "d.one_stream"))
    assert got == [(n, 0, int(n <= 16384), int(n <= 4096)) for n in (ONE_WORKGROUP[k] for k in sizes)], got


def test_lines_of_the_carried_order(tmp_path):
    from test_gpu_carried_order import RIDES
    got = plan(tmp_path, [(V, 5, dim, model, B, C, N) for model, V, dim, B, C, N in RIDES], ("d.order_rides",))
    assert [bool(x) for x, in got] == list(RIDES.values()), dict(zip(RIDES, got))


def test_transe_on_images_where_their_padding_leaves_a_gain(tmp_path):
    """All of at least 2e8 pairs x columns: chunks of few edges or few negatives, and few stripes of wide rows, stay on dense operands; what the tests of the images
    mean to run on them does."""
    from test_gpu_dist_images import SHAPES
    wide = [(372, 3 * 875, 3, 345), (397, 2140, 4, 319)]     # few stripes of rows above 256 floats
    dense = [(20, 50), (50, 100), (55, 644), (42, 361), (722, 29), (1000, 50), (1000, 64), (100, 50)]
    images = [(272, 564), (70, 703), (94, 566), (209, 144), (696, 185), (1000, 65), (65, 1000), (1000, 1000)]
    chunks = lambda S, N: -(-2_000_000 // (S * N))            # of 100 floats: 2e8
    sizes = [(100, S * chunks(S, N), chunks(S, N), N) for S, N in dense + images]
    sizes = wide + sizes + list(SHAPES) + [(100, 23_000, 230, 100), (100, 4_000, 2, 600), (100, 2_400, 4, 1000)]
    got = plan(tmp_path, [(5_000, 5, dim, 2, B, C, N) for dim, B, C, N in sizes], ("(double)d.B * d.N * d.dk >= 2.0e8", "d.dist_img"))
    assert all(g[0] for g in got)
    assert [g[1] for g in got] == [0] * len(wide + dense) + [1] * (len(sizes) - len(wide + dense)), list(zip(sizes, got))


def test_splits_of_the_last_round_on_images_and_on_dense_operands(tmp_path):
    """Parts of the stripes beyond the last whole round: of TransE's images in both passes, of its dense form in the first."""
    from test_gpu_dist_images import SPLIT
    got = plan(tmp_path, [(20_000, 7, dim, 2, B, C, N) for dim, B, C, N in SPLIT], ("d.dist_img", "d.rem1.k", "d.rem2.k"))
    assert got == [(1, k, k) for k in SPLIT.values()], got
    got = plan(tmp_path, [(30_000, 3, dim, model, 21_504, 48, 128) for model, dim in ((2, 36), (2, 100), (0, 100), (1, 100))],
               ("d.bilinear || d.dist_img", "d.rem1.k", "d.rem2.k"))
    assert got == [(0, 2, 1)] + 3 * [(1, 1, 1)], got
