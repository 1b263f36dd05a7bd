"""Row order carried along by the step's own launches: beside passes that leave it slots and passes that do not, with one, two and three
passes over the ids, with the ranks of the debug outputs and without, against the oracle and against itself; and sizes at both sides of
the lines to the second stream (RIDES; tests/test_launch_rules.py asks the library)."""
import numpy as np
import pytest
import torch

import paper_2101_08358_amd as mar

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu


def _ids(rng, V, R, B, C, N):
    hot = lambda m: np.where(rng.random(m) < 0.4, rng.integers(0, 3, m), rng.integers(0, V, m)).astype(np.int32)
    return hot(B), rng.integers(0, R, B).astype(np.int32), hot(B), hot(C * N).reshape(C, N), hot(C * N).reshape(C, N)


# model, nodes, dim, edges, chunks, negatives -> whether the step carries its order: a pass that fills the chip but for 32 workgroups
# (long: each takes several tiles), ranks over 70 tiles, TransE on dense operands and on images, 72,000 rows and more that fit beside
# both passes; then, each after one that does, rows of one workgroup a CU with two and three sort passes, more than 72 x 1,024 rows beside
# passes that fill the chip, rows above 256 floats that do not fit
RIDES = {(1, 14_951, 100, 6_000, 6, 1000): True, (0, 300, 24, 9_030, 7, 333): True, (0, 400_000, 76, 5_005, 7, 211): True,
         (2, 5_000, 40, 3_000, 5, 200): True, (2, 5_000, 100, 2_500, 5, 900): True, (3, 600_000, 16, 24_000, 1, 20): True,
         (0, 300_000, 8, 24_000, 1, 16): True, (0, 300_000, 8, 25_000, 1, 16): True,
         (0, 200_000, 132, 4_992, 8, 483): True, (0, 300_000, 132, 4_992, 8, 483): False,
         (0, 100_000, 140, 15_000, 15, 250): False,
         (3, 14_951, 32, 26_000, 13, 150): True, (3, 14_951, 32, 20_000, 40, 200): False,
         (0, 10_000, 300, 1_200, 120, 10): True, (0, 10_000, 300, 1_280, 128, 10): False}


@pytest.mark.parametrize("model,V,dim,B,C,N", RIDES)
def test_one_step(model, V, dim, B, C, N):
    rng = np.random.default_rng(B + N)
    print("case", model, V, dim, B, flush=True)
    print(check_step(run_step_both(model, V, 5, dim, B, C, N, B, seed=1, std=0.2, ids=_ids(rng, V, 5, B, C, N))), flush=True)


@pytest.mark.parametrize("V,dim,B,C,N", ((14_951, 100, 10_000, 10, 1000), (400_000, 50, 5_000, 5, 300), (300, 33, 2_000, 4, 100)))
def test_the_same_bits_with_and_without_ranks_and_under_capture(V, dim, B, C, N):
    """Two batches, the second shorter: the counts' places follow the batch.  Then the step as a graph, replayed between eager steps."""
    rng = np.random.default_rng(V)
    ids = [torch.from_numpy(x.reshape(-1)).to("cuda:0") for x in _ids(rng, V, 6, B, C, N)]
    ne, re_ = (rng.standard_normal((k, dim)).astype(np.float32) * 0.2 for k in (V, 6))
    got = []
    for mode in ("plain", "ranks", "graph"):
        tr = mar.Trainer(V, 6, dim, 0, B, C, N, seed=4, node_emb=ne, rel_emb=re_)
        tr.neg_src.copy_(ids[3]); tr.neg_dst.copy_(ids[4])
        short = [x[:B - B // C - 7].contiguous() for x in ids[:3]]
        dbg, keep = tr.make_debug(B) if mode == "ranks" else (None, None)
        torch.cuda.synchronize()
        if mode == "graph":
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=st):
                    mar.mar_train_batch(tr.ctx, *ids[:3], B, tr.neg_src, tr.neg_dst, tr.loss, None, st)
            torch.cuda.synchronize()
        for _ in range(2):
            if mode == "graph":
                g.replay()
            else:
                tr.train_batch(*ids[:3], dbg)
            torch.cuda.synchronize()
            tr.train_batch(*short, dbg)
            torch.cuda.synchronize()
        got.append([x.cpu().numpy().copy() for x in (tr.node_emb, tr.node_state, tr.rel_emb, tr.rel_state, tr.loss)])
        tr.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
