"""The fp32 contraction on f16 hi + lo operands with block exponents: the edges of its instantiations, tiles and stripes,
rows of very different size in one block, and evaluation's close comparisons."""
import numpy as np
import pytest
import torch

import paper_2101_08358_amd as mar

from parity_util import run_step_both, check_step

pytestmark = pytest.mark.gpu

DISTMULT, COMPLEX, DOT = 0, 1, 3


@pytest.mark.parametrize("dim", (30, 32, 33, 64, 65, 96, 97, 112, 113, 129, 192, 193, 257))
def test_width_at_the_edges_of_the_instantiations(dim):
    print("case", dim, flush=True)
    print(check_step(run_step_both(DISTMULT, 3000, 5, dim, 260, 2, 100, 260, seed=dim, std=0.3)), flush=True)


@pytest.mark.parametrize("model,S,N", ((DOT, 31, 33), (DISTMULT, 32, 32), (COMPLEX, 127, 129), (DISTMULT, 129, 31), (DOT, 1, 1), (COMPLEX, 257, 385)))
def test_chunk_and_candidate_counts_at_tile_and_stripe_edges(model, S, N):
    print("case", model, S, N, flush=True)
    for n in (3 * S, 2 * S + 1):
        print(check_step(run_step_both(model, 4000, 3, 52, 3 * S, 3, N, n, seed=S + N, std=0.2)), flush=True)


def test_rows_of_different_size_in_one_block():
    """Rows 2^-12 .. 1 of the largest in every 16-row block: each keeps its bits (a block's values hold 23 bits down to
    2^-17 of its largest), so the usual bars hold for every row of the gradient."""
    V, R, dim, B, C, N = 2000, 3, 100, 512, 2, 256
    rng = np.random.default_rng(5)
    size = np.exp2(-rng.integers(0, 13, V)).astype(np.float32)
    ne = (rng.standard_normal((V, dim)) * 0.3).astype(np.float32) * size[:, None]
    out = run_step_both(DOT, V, R, dim, B, C, N, B, seed=9, tables=(ne, np.zeros((R, dim), np.float32)))
    print(check_step(out), flush=True)


def _chain(q, y):
    """fp32 dot product as a chain of fused multiply-adds in the order of the fp32 matrix instructions (products are exact
    in float64, every step is rounded to float32)."""
    d = q.shape[-1]
    chain = 48 if d <= 52 else (96 if d <= 100 else 400)
    order = [16 * b + 4 * g + i for b in range((min(chain, d) + 15) // 16) for i in range(4) for g in range(4)]
    s = np.zeros(np.broadcast_shapes(q.shape[:-1], y.shape[:-1]), np.float32)
    for k in [k for k in order if k < d] + list(range(chain, d)):
        s = (q[..., k].astype(np.float64) * y[..., k] + s).astype(np.float32)
    return s


@pytest.mark.parametrize("dim", (17, 52, 56, 100, 128, 400))
@pytest.mark.parametrize("special", (False, True))
def test_ranks_are_those_of_the_fp32_chain(dim, special):
    """Every node is a candidate, so each edge meets its own endpoint, whose score differs from the positive's by rounding
    only; with `special` the table holds infinities, a NaN, a huge and a zero row."""
    V, S, C = 333, 70, 2
    rng = np.random.default_rng(dim)
    ne = (rng.standard_normal((V, dim)) * 0.3).astype(np.float32)
    if special:
        ne[3, 0], ne[5, dim // 2], ne[7, 1], ne[11] = np.inf, np.nan, -np.inf, 0.0
        ne[9] *= np.float32(1e12)
    src, dst = rng.integers(16, V, S * C).astype(np.int32), rng.integers(16, V, S * C).astype(np.int32)
    tr = mar.Trainer(V, 1, dim, DOT, S * C, C, V, device="cuda:0", node_emb=ne, rel_emb=np.zeros((1, dim), np.float32))
    every = torch.arange(V, dtype=torch.int32, device=tr.device).repeat(C)
    pos = torch.zeros(S * C, device=tr.device)
    ranks = torch.zeros(2 * S * C, dtype=torch.int32, device=tr.device)
    d_src, d_dst = torch.from_numpy(src).to(tr.device), torch.from_numpy(dst).to(tr.device)
    mar.mar_eval_scores(tr.ctx, d_src, d_src, d_dst, S * C, every, every, pos, ranks[:S * C], ranks[S * C:])
    torch.cuda.synchronize()
    p, r = pos.cpu().numpy(), ranks.cpu().numpy()
    tr.close()
    with np.errstate(all="ignore"):
        for got, q in ((r[:S * C], ne[src]), (r[S * C:], ne[dst])):
            want = 1 + (_chain(q[:, None, :], ne[None, :, :]) > p[:, None]).sum(1)
            assert np.array_equal(got, want), (dim, special, int((got != want).sum()))


@pytest.mark.parametrize("small", (0.3, 1e-3, 1e-5))
@pytest.mark.parametrize("where", ("negatives", "edges"))
def test_a_block_of_zero_rows_beside_others(small, where):
    """Sixteen aligned zero rows among the negatives (first pass) or the edges' destinations (second pass), the other rows of
    the same operand being small and those of the other operand so large that scores are of order 1.  Zero rows carry
    nothing: the softmax reference that the others' weights are formed against must not be theirs.  Every gradient row
    within 1e-4 of its own largest entry."""
    V, dim, B, C, N = 3000, 64, 512, 2, 200
    rng = np.random.default_rng(3)
    ne = rng.standard_normal((V, dim)) * small                   # 0 .. 15 zero, 16 .. 1999 small, 2000 .. large
    ne[:16] = 0
    ne[2000:] *= 0.25 / small ** 2
    src, dst = rng.integers(2000, V, B).astype(np.int32), rng.integers(16, 2000, B).astype(np.int32)
    neg_src, neg_dst = rng.integers(2000, V, (C, N)).astype(np.int32), rng.integers(16, 2000, (C, N)).astype(np.int32)
    if where == "negatives":
        neg_dst[:, 64:80] = np.arange(16)
    else:
        dst[32:48] = np.arange(16)
    out = run_step_both(DOT, V, 1, dim, B, C, N, B, seed=9, ids=(src, np.zeros(B, np.int32), dst, neg_src, neg_dst),
                        tables=(ne.astype(np.float32), np.zeros((1, dim), np.float32)))
    G = out["ora"]["res"].G_nodes
    top = np.abs(G).max(1)
    err = np.abs(out["gpu"]["G"][:G.shape[0]] - G).max(1)[top > 0] / top[top > 0]
    print("worst row %.1e" % err.max(), flush=True)
    assert err.max() <= 1e-4


def _above(q, y, p):
    """Candidates whose score, the fp32 chain of `_chain`, is above the edge's: q [edges, d], y [candidates, d], p [edges]."""
    d = q.shape[1]
    chain = 48 if d <= 52 else (96 if d <= 100 else 400)
    order = [16 * b + 4 * g + i for b in range((min(chain, d) + 15) // 16) for i in range(4) for g in range(4)]
    q, y = (torch.from_numpy(np.ascontiguousarray(x.T)).to("cuda:0").double() for x in (q, y))
    s = torch.zeros((q.shape[1], y.shape[1]), device="cuda:0")
    for k in [k for k in order if k < d] + list(range(chain, d)):
        s = (q[k][:, None] * y[k][None, :] + s).float()
    return (s > torch.from_numpy(p).to("cuda:0")[:, None]).sum(1).cpu().numpy()


def _dot_ranks(ne, src, dst, C, neg_src, neg_dst):
    """Ranks under the Dot score through the library, and those of the fp32 chain."""
    V, dim = ne.shape
    n, N = src.size, neg_src.shape[1]
    tr = mar.Trainer(V, 1, dim, DOT, n, C, N, device="cuda:0", node_emb=ne, rel_emb=np.zeros((1, dim), np.float32))
    d_src, d_dst, d_ns, d_nd = (torch.from_numpy(np.ascontiguousarray(x).reshape(-1)).to(tr.device) for x in (src, dst, neg_src, neg_dst))
    pos = torch.zeros(n, device=tr.device)
    ranks = torch.zeros(2 * n, dtype=torch.int32, device=tr.device)
    mar.mar_eval_scores(tr.ctx, d_src, d_src, d_dst, n, d_ns, d_nd, pos, ranks[:n], ranks[n:])
    torch.cuda.synchronize()
    got, p = ranks.cpu().numpy().reshape(2, n), pos.cpu().numpy()
    tr.close()
    want = np.ones((2, n), np.int64)
    for c in range(C):
        e = slice(c * (n // C), (c + 1) * (n // C))
        for k, (q, neg) in enumerate(((ne[src], neg_dst), (ne[dst], neg_src))):
            want[k, e] += _above(q[e], ne[neg[c]], p[e])
    return got, want


# Two chunks of 1,100 edges against some 1,000 candidates run on the images; small evaluations on dense fp32 operands.
S_IMG = 1100


@pytest.mark.parametrize("n,N", ((2 * 48, 64), (2 * S_IMG, 960)))
@pytest.mark.parametrize("dim", (36, 100, 260))
def test_ranks_when_positive_scores_leave_the_range(dim, n, N):
    """Rows of 1e20 with one sign each: the positive score of an edge between rows of different sign is -inf, which no
    candidate whose score is -inf too outscores."""
    rng = np.random.default_rng(dim)
    V, C = 400, 2
    sign = np.where(rng.random(V) < 0.5, -1, 1)
    ne = (sign[:, None] * rng.uniform(0.5e20, 2e20, (V, dim))).astype(np.float32)
    src, dst = (rng.integers(0, V, n).astype(np.int32) for _ in range(2))
    neg = [rng.integers(0, V, (C, N)).astype(np.int32) for _ in range(2)]
    got, want = _dot_ranks(ne, src, dst, C, *neg)
    assert np.array_equal(got, want), int((got != want).sum())


@pytest.mark.parametrize("n,N", ((2 * 64, 300), (2 * S_IMG, 960)))
@pytest.mark.parametrize("size", (2.0 ** -60, 2.0 ** -95, 2.0 ** -110))
def test_ranks_of_edges_with_tiny_rows(size, n, N):
    """Edges from tiny rows to rows of ordinary size: the tiny operand's block exponent ends at its limit and the scaled
    values keep fewer bits, so more comparisons are close."""
    rng = np.random.default_rng(8)
    V, dim, C = 600, 100, 2
    ne = (rng.standard_normal((V, dim)) * 0.3).astype(np.float32)
    ne[:200] *= np.float32(size)
    src, dst = rng.integers(0, 200, n).astype(np.int32), rng.integers(200, V, n).astype(np.int32)
    neg = [rng.integers(200, V, (C, N)).astype(np.int32) for _ in range(2)]
    got, want = _dot_ranks(ne, src, dst, C, *neg)
    assert np.array_equal(got, want), int((got != want).sum())


@pytest.mark.parametrize("n,V", ((2 * 64, 300), (2 * S_IMG, 990)))
@pytest.mark.parametrize("model", (DISTMULT, DOT))
def test_ranks_with_rows_of_very_different_size_in_one_block(model, n, V):
    """Rows 2^-40 .. 1 of the largest among edges and candidates (DistMult: the relation rows too), some of them zero, every
    node a candidate: each rank is the one of the fp32 chain."""
    rng = np.random.default_rng(model)
    R, dim, C = 9, 100, 2
    ne, re_ = (rng.standard_normal((k, dim)).astype(np.float32) * np.exp2(-rng.integers(0, 41, (k, 1))).astype(np.float32) for k in (V, R))
    ne[rng.random(V) < 0.05], re_[0] = 0, 0
    src, dst = (rng.integers(0, V, n).astype(np.int32) for _ in range(2))
    rel = rng.integers(0, R, n).astype(np.int32)
    tr = mar.Trainer(V, R, dim, model, n, C, V, device="cuda:0", node_emb=ne, rel_emb=re_)
    tr.neg_src = tr.neg_dst = torch.arange(V, dtype=torch.int32, device=tr.device).repeat(C)
    pos, rd, rs = (x.cpu().numpy() for x in tr.eval_scores(*(torch.from_numpy(x).to(tr.device) for x in (src, rel, dst))))
    tr.close()
    r = re_[rel] if model == DISTMULT else np.float32(1)
    for got, q in ((rd, ne[src] * r), (rs, r * ne[dst])):
        want = 1 + _above(q, ne, pos)
        assert np.array_equal(got, want), int((got != want).sum())


@pytest.mark.parametrize("dim,N", ((20, 961), (50, 1000), (75, 965), (99, 992), (100, 1000), (128, 991), (190, 964), (256, 970), (400, 997), (100, 70)))
@pytest.mark.parametrize("ties", ("one node", "equal rows", "all", "two edges", "not finite"))
def test_ranks_where_most_comparisons_are_close(dim, N, ties):
    """More close comparisons than an edge keeps one by one: candidates that are the edge's own endpoint again and again
    (counted), rows equal to it under other ids (whole tiles settled), every row of the table equal, two edges of a tile
    only, and rows with infinities and NaN.  Ranks are those of the fp32 chain; candidate counts end inside a tile."""
    rng = np.random.default_rng(dim)
    V, n, C = 300, 2 * (S_IMG if N > 70 else 70), 2
    ne = (rng.standard_normal((V, dim)) * 0.3).astype(np.float32)
    if ties == "equal rows":
        ne[20:150] = ne[20]
    if ties == "all":
        ne[:] = ne[0]
    if ties == "not finite":
        ne[30, 0], ne[31, dim // 2], ne[160, 1], ne[161] = np.inf, np.nan, -np.inf, 0.0
    src, dst = (rng.integers(20, 150, n).astype(np.int32) for _ in range(2))
    if ties == "one node":
        dst[:], src[n // 2:] = 25, 26
    neg = [np.where(rng.random((C, N)) < 0.6, rng.integers(20, 150, (C, N)), rng.integers(0, V, (C, N))).astype(np.int32) for _ in range(2)]
    if ties in ("one node", "two edges"):
        neg[0][rng.random((C, N)) < 0.5], neg[1][rng.random((C, N)) < 0.5] = 26, 25
    if ties == "two edges":
        ne[200:] = ne[25]
        src[[3, 19]], dst[[3, 19]] = 26, 25
    got, want = _dot_ranks(ne, src, dst, C, *neg)
    assert np.array_equal(got, want), int((got != want).sum())


@pytest.mark.parametrize("model", (DISTMULT, COMPLEX, DOT))
@pytest.mark.parametrize("dim", (18, 50, 64, 98, 100, 126, 200, 256, 330, 400))
def test_small_and_large_evaluations_rank_alike(model, dim):
    """Two chunks of 1,100 edges against 1,000 candidates are above the line of dense fp32 operands, one of them (a short
    batch in the same context) and a part of one below it: the same edges have the same ranks and scores, bit for bit."""
    rng = np.random.default_rng(dim + model)
    V, R, C, N = 3000, 7, 2, 1000
    B = C * S_IMG
    ne, re_ = ((rng.standard_normal((k, dim)) * 0.3).astype(np.float32) for k in (V, R))
    ids = [torch.from_numpy(rng.integers(0, k, B).astype(np.int32)).to("cuda:0") for k in (V, R, V)]
    tr = mar.Trainer(V, R, dim, model, B, C, N, device="cuda:0", node_emb=ne, rel_emb=re_)
    tr.sample_negatives(0)
    tr.neg_dst[5:700:9] = ids[2][:78]                      # edges' own endpoints among the candidates
    got = []
    for n in (B, S_IMG, 333):
        pos, rd, rs = tr.eval_scores(*(x[:n] for x in ids))
        torch.cuda.synchronize()
        got.append([x.cpu().numpy()[:333].copy() for x in (pos, rd, rs)])
    tr.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)


# Above the line of dense operands, and cut into equal shares (tests/test_launch_rules.py asks the library): dim, chunks, edges and
# candidates of each.
SHARED = ((400, 19, 1000, 997), (393, 33, 500, 340), (260, 34, 500, 338))


@pytest.mark.parametrize("dim,C,S,N", ((4, 3, 1100, 1000), (24, 3, 1100, 1000), (28, 3, 1100, 1000), (104, 3, 1100, 1000), (105, 3, 1100, 1000),
                                       (112, 3, 1100, 1000), (124, 3, 1100, 1000), (392, 3, 1100, 1000)) + SHARED)
def test_chunks_evaluated_together_rank_as_each_alone(dim, C, S, N):
    """A chunk alone takes the fp32 instructions, all together the operand images: rows whose last columns fill a whole, half or
    quarter step, and (the last three) tiles cut into shares that end inside a stripe, with stripes of the last chunk empty."""
    print("case", dim, C, S, N, flush=True)
    rng = np.random.default_rng(dim)
    V, R, B, n = 3000, 5, C * S, C * S - S // 2
    ne, re_ = ((rng.standard_normal((k, dim)) * 0.3).astype(np.float32) for k in (V, R))
    ids = [torch.from_numpy(rng.integers(0, k, n).astype(np.int32)).to("cuda:0") for k in (V, R, V)]
    tr = mar.Trainer(V, R, dim, DISTMULT, B, C, N, device="cuda:0", node_emb=ne, rel_emb=re_)
    tr.sample_negatives(0)
    tr.neg_dst[3:N:7] = ids[2][:len(range(3, N, 7))]       # edges' own endpoints among the candidates
    all_ = tr.eval_scores(*ids)
    one = mar.Trainer(V, R, dim, DISTMULT, S, 1, N, device="cuda:0", node_emb=ne, rel_emb=re_)
    for c in (0, 1, C // 2, C - 2, C - 1):
        one.neg_src, one.neg_dst = tr.neg_src[c * N:(c + 1) * N].clone(), tr.neg_dst[c * N:(c + 1) * N].clone()
        at = slice(c * S, min((c + 1) * S, n))
        alone = one.eval_scores(*(x[at].clone() for x in ids))
        for a, b in zip(all_, alone):
            assert torch.equal(a[at], b), (dim, c, int((a[at] != b).sum()))
    torch.cuda.synchronize()
    tr.close()
    one.close()


@pytest.mark.parametrize("dim", (1, 16, 17, 20, 21, 25, 32, 33, 49, 52, 53, 56, 57, 64, 65, 81, 84, 85, 88, 89, 96, 97, 100, 101, 108))
def test_narrow_rows_by_the_columns_of_their_last_step(dim):
    """Rows up to 112 floats: at most 4 columns of the last step share one instruction, 5 to 8 two, more take three."""
    test_chunks_evaluated_together_rank_as_each_alone(dim, 2, 1100, 1000)


@pytest.mark.parametrize("dim", (8, 24, 25, 56, 57, 104, 105, 120, 121, 184, 248, 392, 393))
def test_step_where_the_last_columns_fill_half_a_block_or_a_little_more(dim):
    """Up to 8 columns of the last block share their instructions (hi and lo parts side by side), from 9 on they do not."""
    print("case", dim, flush=True)
    print(check_step(run_step_both(DISTMULT, 2000, 3, dim, 130, 1, 70, 130, seed=dim, std=0.3)), flush=True)


def test_close_comparisons_cost_about_as_much_as_others():
    """Candidates drawn by degree hold an edge's own endpoint many times, and rows may be equal: both evaluations within 6
    times that of candidates without ties (1.3 and 3.2 times here; one comparison after the other 20 to 60 times)."""
    V, dim, n, C, N = 20_000, 100, 20_000, 20, 1000
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    ne = torch.randn((V, dim), generator=g, device="cuda:0") * 0.3
    src, dst = (torch.randint(0, V, (n,), generator=g, device="cuda:0", dtype=torch.int32) for _ in range(2))
    neg = torch.randint(0, V, (C * N,), generator=g, device="cuda:0", dtype=torch.int32)
    half = torch.rand(n, generator=g, device="cuda:0") < 0.5
    popular = [torch.where(half, torch.zeros_like(x), x) for x in (src, dst, neg)]
    equal = ne.clone()
    equal[::2] = ne[0]

    def best(table, s, d, k):
        tr = mar.Trainer(V, 1, dim, DOT, n, C, N, device="cuda:0", node_emb=table, rel_emb=torch.zeros((1, dim), device="cuda:0"))
        tr.neg_src = tr.neg_dst = k
        pos, ranks = torch.zeros(n, device="cuda:0"), torch.zeros(2 * n, dtype=torch.int32, device="cuda:0")
        got = []
        for _ in range(8):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            mar.mar_eval_scores(tr.ctx, s, s, d, n, k, k, pos, ranks[:n], ranks[n:])
            ev[1].record()
            torch.cuda.synchronize()
            got.append(ev[0].elapsed_time(ev[1]))
        tr.close()
        return min(got)

    plain, tied, equal_rows = best(ne, src, dst, neg), best(ne, *popular), best(equal, src, dst, neg)
    print("ms: %.3f, popular node %.3f, equal rows %.3f" % (plain, tied, equal_rows), flush=True)
    assert max(tied, equal_rows) <= 6 * plain
