"""TransE's training passes on images and 16-bit products against the oracle: every instantiation's widths (whole and half-filled last
blocks, rows of no whole 16 bytes), chunks that fill no stripe, tile or part, negatives that coincide with their target or nearly do,
rows of different size, and the line between images and dense operands."""
import numpy as np
import pytest

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu
TRANSE = 2


# dim, edges, chunks, negatives: at least 2e8 pairs x columns
SHAPES = ((17, 11_000, 11, 1001), (50, 5_005, 5, 911), (75, 3_003, 3, 1000), (96, 2_431, 11, 1003), (100, 4_440, 37, 801), (110, 2_000, 1, 1100),
          (128, 2_010, 10, 999), (131, 2_100, 3, 1000), (249, 1_602, 2, 733), (300, 3_000, 4, 600), (400, 1_005, 15, 700))


@pytest.mark.parametrize("dim,B,C,N", SHAPES)
def test_one_step(dim, B, C, N):
    assert B * N * ((dim + 3) // 4 * 4) >= 2e8
    print("case", dim, B, flush=True)
    print(check_step(run_step_both(TRANSE, 4000, 7, dim, B, C, N, B - B // (3 * C), seed=dim, std=0.3)), flush=True)


@pytest.mark.parametrize("B", (1_999, 2_000))
def test_beside_the_line(B):
    """100 floats, 1,000 negatives: 1,999 edges on dense operands, 2,000 on images."""
    print("case", B, flush=True)
    print(check_step(run_step_both(TRANSE, 3000, 3, 100, B, 1, 1000, B, seed=B, std=0.2)), flush=True)


@pytest.mark.parametrize("dim,level", ((100, 0.0), (128, 0.0), (100, 1e-3), (128, 1e-4), (53, 3e-2), (400, 0.0)))
def test_negatives_at_or_near_the_target(dim, level):
    """Relation 0 is zero, so that the operand of its edges is the endpoint's own row: negatives at that row (distance 0: no
    gradient) or `level` of its norm away.  Row bar as in test_transe_negatives_that_nearly_coincide_with_the_target: the direction
    of a pair at `level` is known to 2^-23 / level."""
    rng = np.random.default_rng(dim + int(1 / max(level, 1e-5)))
    V, R, B, C, N = 3000, 4, 4_000, 5, 1000
    S = B // C
    ne, re_ = (rng.standard_normal((V, dim)) * 0.2).astype(np.float32), (rng.standard_normal((R, dim)) * 0.2).astype(np.float32)
    re_[0] = 0.0
    spare = V - 500
    src, dst = (rng.integers(0, spare, B).astype(np.int32) for _ in range(2))
    rel = rng.integers(0, R, B).astype(np.int32)
    neg_src, neg_dst = (rng.integers(0, spare, (C, N)).astype(np.int32) for _ in range(2))
    for c in range(C):
        for k in range(40):
            e = c * S + 19 * k
            rel[e] = 0
            for neg, end, slot in ((neg_dst, src, 25 * k), (neg_src, dst, 25 * k + 3)):
                if level == 0.0:
                    neg[c, slot] = end[e]
                else:
                    d = rng.standard_normal(dim)
                    ne[spare] = ne[end[e]] + d / np.linalg.norm(d) * level * np.linalg.norm(ne[end[e]])
                    neg[c, slot] = spare
                    spare += 1
    out = run_step_both(TRANSE, V, R, dim, B, C, N, B, seed=0, tables=(ne, re_), ids=(src, rel, dst, neg_src, neg_dst))
    print(check_step(out, row_rel=max(1e-4, 2.0 ** -23 / level) if level else None), flush=True)


@pytest.mark.parametrize("low", (1e-2, 1e-3))
def test_rows_of_different_size(low):
    """Half of the rows `low` of the others' size, in blocks of their own and mixed, two of them zero.  (A small row beside a large
    one is no near pair, but two small ones are distances of `low` apart whose weights meet operands of size 1 in the sums: an error
    of 2^-24 / low, in fp32 instructions as well.)"""
    rng = np.random.default_rng(3)
    V, R, dim, B, C, N = 2000, 3, 100, 2_000, 2, 1000
    ne, re_ = rng.standard_normal((V, dim)) * 0.3, rng.standard_normal((R, dim)) * 0.3
    ne[::2] *= low
    ne[4] = ne[6] = 0.0
    re_[1] *= low
    ids = [rng.integers(0, k, B).astype(np.int32) for k in (V, R, V)] + [rng.integers(0, V, (C, N)).astype(np.int32) for _ in range(2)]
    ids[3][0, :320] = 2 * rng.integers(0, V // 2, 320)      # whole blocks of small rows
    out = run_step_both(TRANSE, V, R, dim, B, C, N, B, seed=1, tables=(ne.astype(np.float32), re_.astype(np.float32)), ids=tuple(ids))
    print(check_step(out), flush=True)
