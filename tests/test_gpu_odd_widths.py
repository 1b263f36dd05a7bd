"""Steps on rows of no whole 16 bytes, the narrowest included: the chain rule reads such rows 16 bytes at a time from any multiple of 4
bytes, their last columns with those before them."""
import numpy as np
import pytest

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", (2, 3, 5, 6, 7, 63, 66, 131, 255, 258, 399))
def test_one_step(dim):
    # (a row of one column is one sum of terms of either sign, whose rounding has no bound against the sum: the test below)
    for model, B, C, N in ((0, 90, 3, 40), (2, 90, 3, 40), (3, 700, 2, 300)):
        print("case", dim, model, flush=True)
        print(check_step(run_step_both(model, 500, 4, dim, B, C, N, B - 11, seed=dim, std=0.3)), flush=True)


@pytest.mark.parametrize("model,B,C,N", ((0, 90, 3, 40), (2, 90, 3, 40), (3, 700, 2, 300)))
def test_rows_of_one_column(model, B, C, N):
    """The same step on rows of two columns, the second of zeros: adding zeros changes no sum, so outputs are the same bits."""
    V, R = 500, 4
    rng = np.random.default_rng(model)
    ids = [rng.integers(0, k, B).astype(np.int32) for k in (V, R, V)] + [rng.integers(0, V, (C, N)).astype(np.int32) for _ in range(2)]
    ne, re_ = (rng.standard_normal((k, 1)).astype(np.float32) * np.float32(0.3) for k in (V, R))
    one, two = (run_step_both(model, V, R, d, B, C, N, B, seed=0, tables=tables, ids=ids)["gpu"]
                for d, tables in ((1, (ne, re_)), (2, tuple(np.concatenate([t, np.zeros_like(t)], 1) for t in (ne, re_)))))
    for k in ("pos", "lse_dst", "lse_src", "uniq_nodes", "uniq_rels"):
        assert np.array_equal(one[k], two[k]), k
    for k in ("G", "node_emb", "node_state", "rel_emb", "rel_state"):
        assert np.array_equal(one[k][:, 0], two[k][:, 0]), k
