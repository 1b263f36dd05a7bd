"""TransE on images where the rows of a table share an offset: distances are those without it, so gradients are as exact and a step
takes no longer.  With degenerate batches for the estimate of that offset: few nodes, many chunks, a row of infinities
or NaN among the sampled ones."""
import numpy as np
import pytest
import torch

import paper_2101_08358_amd as mar

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu
TRANSE = 2


def _tables(rng, V, R, dim, offset):
    ne = (rng.standard_normal((V, dim)) * 0.2 + offset).astype(np.float32)
    return ne, (rng.standard_normal((R, dim)) * 0.2).astype(np.float32)


# dim, offset, offsets of either sign, and how far off relation gradients are when nothing but the operands s + r and d - r is rounded
# to fp32 (the same step in 64 bits with and without that rounding)
@pytest.mark.parametrize("dim,offset,negative,rounding", ((100, 5.0, False, 2.5e-7), (400, 1.0, False, 1.0e-6), (53, -3.0, False, 1.2e-7),
                                                          (130, 1.0, True, 1.0e-6)))
def test_gradients_with_an_offset(dim, offset, negative, rounding):
    """Relation gradients, where the error sums over edges: the operands' rounding, and what the passes lose without an offset (2e-7,
    here with a factor of 2).  (With the offset left in: 1.4e-6, 3.4e-6, 5.5e-6 and 1.8e-6; fp32 instructions: 4.0e-6, 1.5e-6, 3.3e-6
    and 1.5e-6.)"""
    rng = np.random.default_rng(dim)
    V, R, B, C, N = 3000, 4, 4_000, 5, 1000
    ne, re_ = _tables(rng, V, R, dim, offset)
    if negative:
        ne[:, ::2] *= -1.0
    print("case", dim, offset, flush=True)
    out = run_step_both(TRANSE, V, R, dim, B, C, N, B, seed=dim, tables=(ne, re_))
    print(check_step(out), flush=True)
    res, un = out["ora"]["res"], out["ora"]["res"].uniq_nodes.size
    err = np.linalg.norm(out["gpu"]["G"][un:] - res.G_rels) / np.linalg.norm(res.G_rels)
    print("relation gradients", err, flush=True)
    assert err <= rounding + 4e-7, err


def test_a_step_takes_no_longer_with_an_offset():
    """5 +- 0.3 against 0 +- 0.3: the same pairs and distances (3.4 times as long while nearly all of them counted as near)."""
    V, R, dim, B, C, N = 14_951, 50, 100, 10_000, 10, 1000
    us = []
    for offset in (0.0, 5.0):
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(1)
        ne = torch.randn((V, dim), generator=gen, device="cuda:0") * 0.3 + offset
        re_ = torch.randn((R, dim), generator=gen, device="cuda:0") * 0.3
        tr = mar.Trainer(V, R, dim, TRANSE, B, C, N, 0, 1e-6, 1e-10, 0.001, 3, node_emb=ne, rel_emb=re_)
        ids = [torch.randint(0, k, (B,), generator=gen, device="cuda:0", dtype=torch.int32) for k in (V, R, V)]
        times = []
        for i in range(60):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            tr.sample_negatives(i, ids[0], ids[2])
            a.record()
            tr.train_batch(*ids)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        tr.close()
        us.append(1e3 * float(np.median(times[20:])))
    print("us a step without and with the offset", us, flush=True)
    assert us[1] <= 1.5 * us[0], us


@pytest.mark.parametrize("V,B,C,N", ((3, 4_000, 2, 600), (9, 4_000, 2, 600), (2000, 23_000, 230, 100)))
def test_small_tables_and_many_chunks(V, B, C, N):
    """The eight rows are few different ones; more chunks than rows."""
    dim, R = 100, 3
    rng = np.random.default_rng(V + N)
    print("case", V, B, N, flush=True)
    ids = (rng.integers(0, V, B).astype(np.int32), rng.integers(0, R, B).astype(np.int32), rng.integers(0, V, B).astype(np.int32),
           rng.integers(0, V, (C, N)).astype(np.int32), rng.integers(0, V, (C, N)).astype(np.int32))
    print(check_step(run_step_both(TRANSE, V, R, dim, B, C, N, B, seed=V, std=0.3, ids=ids)), flush=True)


@pytest.mark.parametrize("bad", (np.inf, np.nan, 3e38))
def test_sampled_rows_that_are_no_numbers(bad):
    """One such row among the negatives that the offset is estimated from: rows of other edges and negatives keep their values."""
    rng = np.random.default_rng(5)
    V, R, dim, B, C, N = 3000, 4, 100, 2_400, 4, 1000
    ne, re_ = _tables(rng, V, R, dim, 1.0)
    ids = [rng.integers(1, V, B).astype(np.int32), rng.integers(0, R, B).astype(np.int32), rng.integers(1, V, B).astype(np.int32)]
    neg = [rng.integers(1, V, (C, N)).astype(np.int32) for _ in range(2)]
    neg[1][0, N - 1] = 0                                    # chunk 0, destination side
    ne[0] = bad
    got = []
    for row in (None, 1.0):
        tab = ne.copy()
        if row is not None:
            tab[0] = row
        tr = mar.Trainer(V, R, dim, TRANSE, B, C, N, seed=0, node_emb=tab, rel_emb=re_)
        t = [torch.from_numpy(x).to(tr.device) for x in ids]
        tr.neg_src.copy_(torch.from_numpy(neg[0].reshape(-1))); tr.neg_dst.copy_(torch.from_numpy(neg[1].reshape(-1)))
        dbg, keep = tr.make_debug(B)
        tr.train_batch(*t, dbg)
        torch.cuda.synchronize()
        got.append([keep[k].cpu().numpy()[:B].copy() for k in ("pos", "lse_dst", "lse_src")])
        tr.close()
    S = B // C
    assert np.array_equal(got[0][0], got[1][0])
    for k, sel in ((1, slice(S, B)), (2, slice(0, B))):
        assert np.isfinite(got[0][k][sel]).all()
        assert np.max(np.abs(got[0][k][sel] - got[1][k][sel])) <= 1e-6 * np.max(np.abs(got[1][k][sel]))
