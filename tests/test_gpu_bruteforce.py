"""GPU exhaustive filtered k-NN (Def. 2) against the oracle's exhaustive
search, through the C ABI."""
import numpy as np
import pytest

import oracle
import paper_2608_16491_amd as F
import workloads
from tests.parity import assert_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cuda(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a)).to(dtype=dtype, device="cuda")


def _run(X, attr, Q, lo, hi, k):
    perm = np.argsort(attr, kind="stable").astype(np.int32)
    srt = attr[perm]
    Xr = X[perm]
    n, d = X.shape
    ENC = -np.ones((n, 1, 1), np.int32)
    ix = F.Index.from_arrays(Xr, srt, perm, ENC).upload(0)
    ids, ds, cert = F.bruteforce(ix, _cuda(Q, torch.float32), _cuda(lo, torch.float64),
                                 _cuda(hi, torch.float64), k)
    torch.cuda.synchronize()
    o_ids, o_d = oracle.exact(Xr, srt, perm, Q, lo, hi, k)
    return ids.cpu().numpy(), ds.cpu().numpy(), cert.cpu().numpy(), o_ids, o_d


def test_bruteforce_tiny():
    print("[gpu] bruteforce tiny", flush=True)
    w = workloads.make("tiny")
    ids, ds, cert, o_ids, o_d = _run(w.X, w.attr, w.Q, w.lo, w.hi, 10)
    assert (cert == 1).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


@pytest.mark.parametrize("k", [1, 10, 100])
def test_bruteforce_mixture(k):
    print(f"[gpu] bruteforce mixture k={k}", flush=True)
    w = workloads.make("c2", n=40000, nq=200)
    ids, ds, cert, o_ids, o_d = _run(w.X, w.attr, w.Q, w.lo, w.hi, k)
    assert np.isin(cert, (1, 2)).all() and (cert == 1).mean() > 0.99
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


@pytest.mark.parametrize("d", [200, 1030])
def test_bruteforce_wide_rows(d):
    # rows wider than 128 floats take the chunk loop with the query read per
    # chunk (d = 200: 14 steps of 16 dimensions; d = 1030: 66 steps)
    print(f"[gpu] bruteforce wide rows d={d}", flush=True)
    rng = np.random.default_rng(d)
    n, nq = 3000, 48
    X = rng.standard_normal((n, d)).astype(np.float32)
    attr = rng.permutation(n).astype(np.float64)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    sig = np.array([0.01, 0.1, 0.5, 1.0])[np.arange(nq) % 4]
    lo, hi = workloads.ranges_for_selectivity(rng, sig, n)
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, 10)
    assert np.isin(cert, (1, 2)).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


def test_bruteforce_edges():
    rng = np.random.default_rng(1)
    n, d = 2000, 40
    X = rng.standard_normal((n, d)).astype(np.float32)
    attr = rng.integers(0, 300, n).astype(np.float64)      # duplicate attribute values
    Q = rng.standard_normal((9, d)).astype(np.float32)
    lo = np.array([0, 5, np.nan, 7, 299, 100, 50, -5, 10], np.float64)
    hi = np.array([299, 5, 3, 2, 400, 100.5, 60, 1e9, 10], np.float64)
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, 25)
    assert (cert == 1).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)
    assert (ids[2] == -1).all() and (ids[3] == -1).all()


@pytest.mark.parametrize("k", [1, 10, 100, 256])
def test_bruteforce_uncertified_rows_are_exact(k):
    # Vectors with large norms close to each other (coordinates 1000 +- 0.01):
    # the fp32 approximation |q|^2 + |x|^2 - 2 q.x errs by ~u |x|^2, far more
    # than the gaps between distances, so the margin test certifies almost
    # nothing and the rows come from the exhaustive exact pass.  A tenth of
    # the vectors are duplicates of others (exact ties, broken by rank).  The
    # coordinates are multiples of the fp32 ulp at 1000, so every fp64 sum is
    # exact and both sides agree bit for bit.
    print(f"[gpu] bruteforce, uncertified rows, k={k}", flush=True)
    rng = np.random.default_rng(3)
    n, d, nq = 20000, 32, 48
    X = (1000.0 + 0.01 * rng.standard_normal((n, d))).astype(np.float32)
    src = rng.choice(n, 2000, replace=False)
    X[src[1000:]] = X[src[:1000]]
    attr = rng.permutation(n).astype(np.float64)
    Q = (1000.0 + 0.01 * rng.standard_normal((nq, d))).astype(np.float32)
    cnt = np.array([n, 1, 7, 300, 4095, 4096, 4097, 9000] * (nq // 8))
    lo = rng.integers(0, n - cnt + 1).astype(np.float64)
    hi = lo + cnt - 1
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, k)
    assert np.isin(cert, (1, 2)).all() and (cert == 2).sum() >= nq // 2
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


@pytest.mark.parametrize("n,d,nq,k", [(1, 5, 3, 4), (15, 32, 33, 10), (257, 33, 1, 33), (1536, 64, 32, 64), (1537, 96, 31, 65),
                                      (24575, 20, 70, 10), (24576, 128, 65, 129), (24592, 130, 17, 1), (393216, 16, 40, 10),
                                      (393472, 16, 40, 10)])
def test_bruteforce_sampling_passes(n, d, nq, k):
    # sizes around those at which a further sampling pass is added (1,536 and
    # 24,576 and 393,216 rows at k <= 64; half a tile, a tile and a bit more
    # of queries; every number of list entries re-ranked; both row paths)
    print(f"[gpu] bruteforce passes n={n} d={d} nq={nq} k={k}", flush=True)
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    attr = rng.permutation(n).astype(np.float64)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    lo, hi = workloads.ranges_for_selectivity(rng, np.exp2(-8.0 * rng.random(nq)), n)
    lo[0], hi[0] = 0, n - 1
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, k)
    assert (cert == 1).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("period", [16, 256])
def test_bruteforce_rows_in_a_pattern(period, near):
    # one block of 16 ranks in each 16 or 256 lies nearer to the queries than the
    # others, or farther: a sample in step with the pattern would give
    # thresholds that let every other row into the list, which overflows and
    # leaves the query to the exact pass (slow); a drawn one certifies them all
    print(f"[gpu] bruteforce, one block of {period} nearer={near}", flush=True)
    rng = np.random.default_rng(5)
    n, d, nq, k = 20000, 24, 40, 10
    X = rng.standard_normal((n, d)).astype(np.float32)
    odd = (np.arange(n) // 16) % period == 0
    X[odd != near] += 6.0      # the others, or those blocks, far away
    attr = np.arange(n, dtype=np.float64)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    cnt = np.array([n, 12000, 300, 40] * (nq // 4))
    lo = rng.integers(0, n - cnt + 1).astype(np.float64)
    hi = lo + cnt - 1
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, k)
    assert (cert == 1).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


def test_bruteforce_overflowing_list():
    # 5,000 rows at one distance, the smallest: every threshold lets them all
    # into the list (2,048 entries), so the exact pass answers, ties by rank
    print("[gpu] bruteforce, 5000 equal rows", flush=True)
    rng = np.random.default_rng(6)
    n, d, nq, k = 20000, 24, 8, 10
    X = rng.standard_normal((n, d)).astype(np.float32) + 4.0
    X[rng.permutation(n)[:5000]] = 0.5
    attr = rng.permutation(n).astype(np.float64)
    Q = (0.1 * rng.standard_normal((nq, d))).astype(np.float32)
    lo, hi = np.zeros(nq), np.full(nq, n - 1.0)
    hi[::2] = n // 40      # 125 or so of them: certified
    ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, hi, k)
    assert (cert[1::2] == 2).all()
    assert_parity(ids, ds, o_ids, o_d, max_residual=0)


def test_bruteforce_workspace_is_bounded():
    # the largest k has lists four times as long as the smallest: a batch
    # of any size is done in parts that take at most about 0.3 GB, which the
    # pool keeps (1.07 GB at once before); rows on both sides of the parts' ends
    print("[gpu] bruteforce workspace: n=3000 d=32 nq=16384 k=256", flush=True)
    rng = np.random.default_rng(7)
    n, d, nq, k = 3000, 32, 16384, 256
    X = rng.standard_normal((n, d)).astype(np.float32)
    attr = rng.permutation(n).astype(np.float64)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    lo, hi = workloads.ranges_for_selectivity(rng, np.exp2(-3.0 * rng.random(nq)), n)
    perm = np.argsort(attr, kind="stable").astype(np.int32)
    ix = F.Index.from_arrays(X[perm], attr[perm], perm, -np.ones((n, 1, 1), np.int32)).upload(0)
    dQ, dlo, dhi = _cuda(Q, torch.float32), _cuda(lo, torch.float64), _cuda(hi, torch.float64)
    F.bruteforce(ix, dQ[:32], dlo[:32], dhi[:32], k)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    ids, ds, cert = F.bruteforce(ix, dQ, dlo, dhi, k)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 400 << 20    # 34 MB of it the results
    for s in (0, 4032, 8064, 12096, 16352):
        rows = slice(s, s + 32)
        o_ids, o_d = oracle.exact(X[perm], attr[perm], perm, Q[rows], lo[rows], hi[rows], k)
        assert_parity(ids[rows].cpu().numpy(), ds[rows].cpu().numpy(), o_ids, o_d, max_residual=0)


@pytest.mark.parametrize("d", [129, 960])
@pytest.mark.parametrize("nq", [1, 16, 17, 32, 45])
def test_bruteforce_wide_rows_half_tiles(d, nq):
    # rows above 128 values multiply only the halves of a tile of 32 queries
    # that hold queries near the blocks: batches that fill one half, both, and
    # spill into a second tile; short ranges far apart, so that most blocks meet
    # the intervals of one half or of none
    print(f"[gpu] bruteforce wide rows, half tiles d={d} nq={nq}", flush=True)
    rng = np.random.default_rng(d + nq)
    n = 5000
    X = rng.standard_normal((n, d)).astype(np.float32)
    attr = rng.permutation(n).astype(np.float64)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    for cnt in (n, 300, 40):
        lo = rng.integers(0, n - cnt + 1, nq).astype(np.float64)
        ids, ds, cert, o_ids, o_d = _run(X, attr, Q, lo, lo + cnt - 1, 10)
        assert (cert == 1).all()
        assert_parity(ids, ds, o_ids, o_d, max_residual=0)
