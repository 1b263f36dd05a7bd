"""The row-sorted order of the gradient rows (radix sort by unified id, segment borders read off the sorted ids) for every
number of sort passes and both tile sizes, and the step with and without the outputs that need ranks."""
import numpy as np
import pytest
import torch

import paper_2101_08358_amd as mar

from parity_util import run_step_both, check_step, run_step_device_tables

pytestmark = pytest.mark.gpu


# ids of 9, 10, 19 bits: one, two and three passes; batches of one tile, several small tiles, large tiles
@pytest.mark.parametrize("V,B,C,N", ((300, 64, 1, 32), (509, 3000, 3, 200), (700, 1500, 3, 400), (400_000, 600, 2, 100), (400_000, 30_000, 10, 700)))
def test_passes_and_tile_sizes(V, B, C, N):
    rng = np.random.default_rng(V + B)
    hot = lambda m: np.where(rng.random(m) < 0.4, rng.integers(0, 3, m), rng.integers(0, V, m)).astype(np.int32)
    ids = (hot(B), rng.integers(0, 2, B).astype(np.int32), hot(B), hot(C * N).reshape(C, N), hot(C * N).reshape(C, N))
    print("case", V, B, flush=True)
    print(check_step(run_step_both(0, V, 2, 8, B, C, N, B, seed=1, std=0.2, ids=ids)), flush=True)


def test_four_passes():
    """2^27 + 1000 nodes of 4 floats: ids of 28 bits."""
    rng = np.random.default_rng(28)
    V, R, B, C, N = (1 << 27) + 1000, 3, 2000, 4, 200
    draw = lambda m: np.where(rng.random(m) < 0.3, V - 1 - rng.integers(0, 4, m), rng.integers(0, V, m)).astype(np.int32)
    ids = (draw(B), rng.integers(0, R, B).astype(np.int32), draw(B), draw(C * N).reshape(C, N), draw(C * N).reshape(C, N))
    out = run_step_device_tables(0, V, R, 4, B, C, N, ids, seed=2, std=0.2)
    assert out["gpu"]["untouched_ok"]
    print(check_step(out), flush=True)


# edges, chunks, negatives -> gradient rows (tests/test_launch_rules.py asks the library)
ONE_WORKGROUP = {(200, 2, 50): 1400, (1000, 1, 9): 3144, (2720, 1, 2): 8192, (2721, 1, 2): 8195, (5456, 1, 1): 16384, (5457, 1, 1): 16387}


@pytest.mark.parametrize("B,C,N", ONE_WORKGROUP)
def test_four_passes_in_one_workgroup(B, C, N):
    """Steps with ids above 27 bits cannot carry their row order: one workgroup sorts it, in 8 or 16 rounds, on the caller's stream (up
    to 4,096 gradient rows) or on the second one; just beyond 16,384 rows launches do."""
    rng = np.random.default_rng(B)
    V, R = (1 << 27) + 1000, 3
    draw = lambda m: np.where(rng.random(m) < 0.3, V - 1 - rng.integers(0, 4, m), rng.integers(0, V, m)).astype(np.int32)
    ids = (draw(B), rng.integers(0, R, B).astype(np.int32), draw(B), draw(C * N).reshape(C, N), draw(C * N).reshape(C, N))
    print("case", B, flush=True)
    out = run_step_device_tables(0, V, R, 4, B, C, N, ids, seed=2, std=0.2)
    assert out["gpu"]["untouched_ok"]
    print(check_step(out), flush=True)


@pytest.mark.parametrize("dim,R", ((16, 1), (100, 2), (400, 700)))
def test_the_step_is_the_same_without_debug_outputs(dim, R):
    """Ranks are formed only for the outputs that need them; tables and loss have the same bits either way.  One relation
    row that all 20,000 edges touch spans 79 workgroups of the reduce."""
    V, B, C, N = 5000, 20_000, 4, 256
    rng = np.random.default_rng(dim)
    ids = [torch.from_numpy(rng.integers(0, k, B).astype(np.int32)).to("cuda:0") for k in (V, R, V)]
    ne, re_ = rng.standard_normal((V, dim)).astype(np.float32) * 0.2, rng.standard_normal((R, dim)).astype(np.float32) * 0.2
    got = []
    for with_dbg in (False, True):
        tr = mar.Trainer(V, R, dim, 0, B, C, N, seed=4, node_emb=ne, rel_emb=re_)
        for i in range(3):
            tr.sample_negatives(i, ids[0], ids[2])
            dbg, keep = tr.make_debug(B) if with_dbg else (None, None)
            tr.train_batch(*ids, dbg)
            torch.cuda.synchronize()
        torch.cuda.synchronize()
        got.append([x.cpu().numpy().copy() for x in (tr.node_emb, tr.node_state, tr.rel_emb, tr.rel_state, tr.loss)])
        tr.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


# dim, edges, chunks, negatives of each -> gradient rows: three an edge, and for each of the 2 C N negatives one per part of pass 2
# (tests/test_launch_rules.py asks the library)
ROWS = {(8, 1, 1, 1): 5, (8, 320, 1, 64): 1600, (8, 1500, 1, 16): 4756, (12, 2720, 1, 2): 8192, (12, 2721, 1, 2): 8195, (8, 900, 9, 100): 9900,
        (8, 1600, 16, 90): 16320, (8, 5456, 1, 1): 16384, (8, 5457, 1, 1): 16387, (260, 2400, 1, 62): 8192, (260, 2401, 1, 62): 8195}


@pytest.mark.parametrize("dim,B,C,N", ROWS)
def test_orders_that_one_workgroup_sorts(dim, B, C, N):
    """Batches up to, exactly at and just beyond what one workgroup holds in 8 and in 16 rounds (8,192 and 16,384 rows).  With these
    ids, of at most 27 bits, steps carry the order along; k_sort_one itself: test_four_passes_in_one_workgroup.  Hot ids among them, one, two and three passes.  (Wide rows with 62 negatives: with one, the loss is
    sum(-2 f + f' + f'') of scores that nearly cancel, and its rounding, 2^-24 sum(2 |f| + |f'| + |f''|), was 1.3e-4 of it.)"""
    for V in (200, 100_000, 300_000):
        rng = np.random.default_rng(V + B)
        hot = lambda m: np.where(rng.random(m) < 0.4, rng.integers(0, 3, m), rng.integers(0, V, m)).astype(np.int32)
        ids = (hot(B), rng.integers(0, 2, B).astype(np.int32), hot(B), hot(C * N).reshape(C, N), hot(C * N).reshape(C, N))
        print("case", V, dim, B, flush=True)
        print(check_step(run_step_both(0, V, 2, dim, B, C, N, B, seed=1, std=0.2, ids=ids)), flush=True)
