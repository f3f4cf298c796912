"""GPU parity of the graph-construction entry points (exact kNN, medoid,
alpha pruning + repair) against the CPU oracle: bit-exact ids."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_15986_amd import synth
from tests.common import int_index, say, tiny_index

pytestmark = pytest.mark.gpu


def _ann():
    from paper_2506_15986_amd import ann
    return ann


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_gt_knn_fp64_engine_tiny_exact():
    ix = tiny_index()
    say("case: gt_knn fp64 tiny")
    ids, dist = _ann().ann_gt_knn(_dev(ix["base"]), _dev(ix["q"]), 10)
    torch.cuda.synchronize()
    assert (ids.cpu().numpy() == ix["truth"]).all()
    assert (dist.cpu().numpy() == ix["truth_d2"].astype(np.float32)).all()


def test_gt_knn_int8_engine_exact():
    ix = int_index()
    say("case: gt_knn int8 20k")
    ids, dist = _ann().ann_gt_knn(_dev(ix["base"]), _dev(ix["q"]), 10)
    torch.cuda.synchronize()
    assert (ids.cpu().numpy() == ix["truth"]).all()
    assert (dist.cpu().numpy() == ix["truth_d2"].astype(np.float32)).all()


@pytest.mark.parametrize("n,nq,d,k,ints", [(1000, 77, 32, 13, False), (999, 65, 64, 130, True),
                                             (300, 1, 96, 300, False), (257, 200, 128, 5, True)])
def test_gt_knn_ragged_shapes(n, nq, d, k, ints):
    r = np.random.default_rng(n + nq)
    if ints:
        base = r.integers(0, 256, size=(n, d)).astype(np.float32)
        q = r.integers(0, 256, size=(nq, d)).astype(np.float32)
    else:
        base = (np.rint(r.normal(size=(n, d)) * 2 ** 12) / 2 ** 12).astype(np.float32)
        q = (np.rint(r.normal(size=(nq, d)) * 2 ** 12) / 2 ** 12).astype(np.float32)
    say("case: gt_knn n=%d nq=%d d=%d k=%d ints=%s" % (n, nq, d, k, ints))
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q), k)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (ids.cpu().numpy() == ref_ids).all()
    assert (dist.cpu().numpy()[ref_ids >= 0] == ref_d2[ref_ids >= 0].astype(np.float32)).all()


@pytest.mark.parametrize("n,nq,d,k,vmax", [
    (70_000, 300, 32, 10, 255),      # 17 column slices merged per row
    (20_000, 50, 256, 100, 255),     # widest rows, 4 slices
    (9_000, 700, 96, 300, 255),      # 2 slices of 301 kept entries
    (130, 600, 64, 200, 255),        # k above n: -1 padded
    (5_000, 3, 128, 1024, 255),      # largest k
    (20_000, 64, 160, 50, 3),        # values 0..3: long runs of equal distances
])
def test_int8_engine_slices_and_ties(n, nq, d, k, vmax):
    r = np.random.default_rng(n + d)
    base = r.integers(0, vmax + 1, size=(n, d)).astype(np.float32)
    q = r.integers(0, vmax + 1, size=(nq, d)).astype(np.float32)
    say("case: int8 kNN n=%d nq=%d d=%d k=%d values 0..%d" % (n, nq, d, k, vmax))
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q), k)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (ids.cpu().numpy() == ref_ids).all()
    ok = ref_ids >= 0
    assert (dist.cpu().numpy()[ok] == ref_d2[ok].astype(np.float32)).all()
    assert np.isinf(dist.cpu().numpy()[~ok]).all()


@pytest.mark.parametrize("k", [64, 65, 192, 193, 448, 449])
@pytest.mark.parametrize("d,vmax", [(32, 0), (64, 1), (96, 255)])
def test_int8_engine_list_cuts(k, d, vmax):
    # the edges of the lists' sizes (128, 256, 512 and larger), with all
    # distances equal, with many equal ones and with hardly any
    r = np.random.default_rng(k + d)
    base = r.integers(0, vmax + 1, size=(4001, d)).astype(np.float32)
    q = r.integers(0, vmax + 1, size=(70, d)).astype(np.float32)
    say("case: int8 kNN list cuts k=%d d=%d values 0..%d" % (k, d, vmax))
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q), k)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (ids.cpu().numpy() == ref_ids).all()
    assert (dist.cpu().numpy() == ref_d2.astype(np.float32)).all()


def test_int8_engine_exclude_self_with_duplicates():
    # rows repeated several times: the row's own column is dropped, its
    # duplicates stay (distance 0, by id)
    r = np.random.default_rng(11)
    base = r.integers(0, 256, size=(3000, 64)).astype(np.float32)
    base[1000:1040] = base[5]
    say("case: int8 kNN exclude_self with 41 copies of one row")
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(base), 60, exclude_self=True)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, base, 60, exclude_self=True)
    assert (ids.cpu().numpy() == ref_ids).all()
    assert (dist.cpu().numpy() == ref_d2.astype(np.float32)).all()


@pytest.mark.parametrize("n,d,k,vmax", [
    (70_000, 32, 20, 255),
    (70_000, 128, 128, 255),      # the graph build's shape: 128 dimensions, K = 128
    (66_000, 64, 30, 3),          # values 0..3: long runs of equal distances
])
def test_int8_all_pairs_in_cluster_order(n, d, k, vmax):
    # all pairs over one buffer of at least 65,536 rows run with rows and
    # columns grouped by their nearest sample row: every row's result equals
    # the pass in id order (a second buffer holding the same data) and, on a
    # sample of rows, the oracle's
    r = np.random.default_rng(n + d + vmax)
    base = r.integers(0, vmax + 1, size=(n, d)).astype(np.float32)
    base[500:530] = base[77]                     # duplicates of one row
    x = _dev(base)
    say("case: int8 all pairs in cluster order n=%d d=%d k=%d values 0..%d" % (n, d, k, vmax))
    ids, dist = _ann().ann_gt_knn(x, x, k, exclude_self=True)
    ids2, dist2 = _ann().ann_gt_knn(x, x.clone(), k, exclude_self=True)
    torch.cuda.synchronize()
    ids, dist, ids2, dist2 = ids.cpu().numpy(), dist.cpu().numpy(), ids2.cpu().numpy(), dist2.cpu().numpy()
    assert (ids == ids2).all()
    assert (dist.view(np.uint32) == dist2.view(np.uint32)).all()
    rows = np.concatenate([np.arange(0, n, n // 300), np.arange(500, 530), [77, n - 1]])
    ref_ids, ref_d2 = oracle.knn(base, base[rows], k + 1)
    for t, row in enumerate(rows):
        keep = [j for j in range(k + 1) if ref_ids[t, j] != row][:k]
        assert (ids[row] == ref_ids[t, keep]).all(), row
        assert (dist[row] == ref_d2[t, keep].astype(np.float32)).all(), row


def test_gt_knn_duplicates_tie_by_id_and_exclude_self():
    r = np.random.default_rng(3)
    base = r.integers(0, 4, size=(500, 32)).astype(np.float32)   # many exact ties
    base[100:110] = base[7]
    say("case: gt_knn ties")
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(base), 20, exclude_self=True)
    torch.cuda.synchronize()
    ref_ids, _ = oracle.knn(base, base, 20, exclude_self=True)
    assert (ids.cpu().numpy() == ref_ids).all()


def _real_points(kind, n, nq, d):
    # values on a dyadic grid, so that the FP64 distances are exact
    r = np.random.default_rng(n + d)
    x = np.rint(r.normal(size=(n + nq, d)) * 2 ** 10) / 2 ** 10
    if kind == "copies":            # more equal rows than a list can hold
        x[r.permutation(n)[:900]] = x[n]
    elif kind == "tight":           # groups far narrower than their distance from the centre
        x = x / 4 + r.integers(-900, 901, size=(12, d))[r.integers(0, 12, n + nq)]
    elif kind == "large":
        x = x * 2.0 ** 60
    elif kind == "small":
        x = x * 2.0 ** -60
    elif kind == "flat":            # one wide dimension beside narrow ones
        x[:, 0] *= 2 ** 8
        x[:, 1:] = np.rint(x[:, 1:] * 2 ** 4) / 2 ** 10
    elif kind == "outlier":
        x[n // 2] = 2.0 ** 12
    elif kind == "infinite":
        x[n // 3, 0] = np.inf
    x = x.astype(np.float32)
    return x[:n], x[n:]


@pytest.mark.parametrize("n,nq,d,k,kind", [
    (3_000, 300, 100, 10, "normal"),       # ragged rows, columns and dimensions
    (6_000, 1_025, 20, 64, "normal"),      # one row past a workgroup's 256 four times
    (70_000, 3, 96, 100, "normal"),        # the rows' lists merged over column slices
    (2_000, 300, 130, 1024, "normal"),     # largest k
    (60, 3_000, 200, 100, "normal"),       # k above n: -1 padded
    (4_000, 500, 64, 30, "copies"),
    (5_000, 600, 48, 128, "tight"),
    (3_000, 300, 68, 12, "large"),
    (3_000, 300, 68, 12, "small"),
    (3_000, 300, 68, 12, "flat"),
    (3_000, 300, 68, 12, "outlier"),
    (3_000, 300, 68, 12, "infinite"),
])
def test_real_valued_knn_matches_oracle(n, nq, d, k, kind):
    base, q = _real_points(kind, n, nq, d)
    say("case: real-valued kNN n=%d nq=%d d=%d k=%d %s" % (n, nq, d, k, kind))
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q), k)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (ids == ref_ids).all()
    ok = ref_ids >= 0
    assert (dist[ok] == ref_d2[ok].astype(np.float32)).all()
    assert np.isinf(dist[~ok]).all()


@pytest.mark.parametrize("n,d,k,kind", [(6_000, 100, 64, "normal"), (3_000, 36, 20, "copies"),
                                        (9_001, 96, 128, "tight")])
def test_real_valued_all_pairs_match_oracle(n, d, k, kind):
    base, _ = _real_points(kind, n, 1, d)
    say("case: real-valued all pairs n=%d d=%d k=%d %s" % (n, d, k, kind))
    x = _dev(base)
    ids, dist = _ann().ann_gt_knn(x, x, k, exclude_self=True)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    rows = np.arange(0, n, max(1, n // 400))
    ref_ids, ref_d2 = oracle.knn(base, base[rows], k + 1)
    for t, row in enumerate(rows):
        # the row itself is first, except among copies of it, where ids order
        keep = [j for j in range(k + 1) if ref_ids[t, j] != row][:k]
        assert (ids[row] == ref_ids[t, keep]).all(), row
        assert (dist[row] == ref_d2[t, keep].astype(np.float32)).all(), row


def test_medoid_matches_oracle():
    ix = tiny_index()
    say("case: medoid")
    assert _ann().ann_medoid(_dev(ix["base"])) == ix["medoid"]
    ii = int_index()
    assert _ann().ann_medoid(_dev(ii["base"])) == ii["medoid"]


def test_build_graph_tiny_bit_exact():
    ix = tiny_index()
    say("case: build_graph tiny")
    g, med, (nf, nr) = _ann().ann_build_graph(_dev(ix["base"]), 64, 16, 1.2)
    torch.cuda.synchronize()
    assert med == ix["medoid"]
    assert (nf, nr) == (ix["nf"], ix["nr"])
    assert (g.cpu().numpy() == ix["graph"]).all()


def test_build_graph_int_bit_exact():
    ix = int_index()
    say("case: build_graph int 20k")
    g, med, (nf, nr) = _ann().ann_build_graph(_dev(ix["base"]), 64, 32, 1.2)
    torch.cuda.synchronize()
    assert med == ix["medoid"]
    assert (nf, nr) == (ix["nf"], ix["nr"])
    assert (g.cpu().numpy() == ix["graph"]).all()


def test_build_graph_small_alpha_variants():
    w = synth.scaled(synth.WORKLOADS["tiny"], n=1200)
    base = synth.base(w)
    for alpha, K, R in ((1.0, 24, 8), (2.0, 40, 12)):
        say("case: build_graph alpha=%.1f K=%d R=%d" % (alpha, K, R))
        ref, med, nf, nr, _, _ = oracle.build_graph(base, K, R, alpha)
        g, gm, (gf, gr) = _ann().ann_build_graph(_dev(base), K, R, alpha)
        torch.cuda.synchronize()
        assert gm == med and (gf, gr) == (nf, nr)
        assert (g.cpu().numpy() == ref).all()


@pytest.mark.parametrize("n,d,k,kind", [
    (1_500, 8, 10, "infinite query"),     # no first thresholds: lists that fill
    (1_500, 8, 10, "overflow"),           # finite, but x - c is beyond FP32
    (12_000, 16, 1000, "infinite query"),
    (5_000, 16, 10, "infinite query"),    # first thresholds
    (5_000, 16, 10, "overflow"),
    (1_500, 8, 10, "infinite base"),
])
def test_knn_of_values_beyond_fp16_products_matches_oracle(n, d, k, kind):
    # large finite values (few bits, so that FP64 sums are exact) beside an
    # infinity or of both signs near the largest float: products that are
    # infinite in the FP16 estimates, distances that FP64 tells apart
    r = np.random.default_rng(n + d)
    base = (r.integers(1, 256, size=(n, d)) * 2.0 ** 100).astype(np.float32)
    q = (r.integers(1, 256, size=(40, d)) * 2.0 ** 100).astype(np.float32)
    if kind == "infinite query":
        q[::3, 1] = np.inf
    elif kind == "infinite base":
        base[::7, 2] = np.inf
    else:
        base = (r.integers(192, 256, size=(n, d)) * 2.0 ** 120).astype(np.float32)
        q = -base[:40]
    say("case: kNN beyond FP16 products n=%d d=%d k=%d %s" % (n, d, k, kind))
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q), k)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (ids.cpu().numpy() == ref_ids).all()
    with np.errstate(over="ignore"):
        assert (dist.cpu().numpy() == ref_d2.astype(np.float32)).all()


@pytest.mark.parametrize("n,nq,d,k,kind", [
    (5_000, 600, 49, 128, "tight"),        # the second level's columns: odd rows,
    (3_000, 300, 130, 12, "flat"),         # ... two and a half stages of dimensions,
    (70_000, 3, 97, 50, "tight"),          # ... several column slices
])
def test_real_valued_second_level_matches_oracle(n, nq, d, k, kind):
    test_real_valued_knn_matches_oracle(n, nq, d, k, kind)


@pytest.mark.parametrize("n,nq,d,k", [
    (249, 1, 31, 10), (250, 1, 31, 10),    # the last shape of the plain engine, the first of the shortlist
    (109, 8, 6, 64), (110, 8, 6, 64), (109, 9, 6, 64), (64, 1, 300, 3), (1, 1, 1, 1), (3, 8, 5, 7),
])
def test_real_valued_knn_of_few_rows(n, nq, d, k):
    test_real_valued_knn_matches_oracle(n, nq, d, k, "normal")


@pytest.mark.parametrize("exclude", [False, True])
@pytest.mark.parametrize("n,d,k,kind", [(16_385, 20, 30, "normal"), (16_384, 33, 16, "tight"),
                                        (20_011, 36, 20, "copies"), (20_011, 100, 64, "tight")])
def test_real_valued_all_pairs_in_group_order(n, d, k, kind, exclude):
    # from 16,384 rows on, all pairs go through in the order of their groups
    base, _ = _real_points(kind, n, 1, d)
    say("case: real-valued all pairs in group order n=%d d=%d k=%d %s" % (n, d, k, kind))
    x = _dev(base)
    ids, dist = _ann().ann_gt_knn(x, x, k, exclude_self=exclude)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(0, n, max(1, n // 300)), [n - 1]]))
    ref_ids, ref_d2 = oracle.knn(base, base[rows], k + 1)
    for t, row in enumerate(rows):
        keep = [j for j in range(k + 1) if not exclude or ref_ids[t, j] != row][:k]
        assert (ids[row] == ref_ids[t, keep]).all(), row
        assert (dist[row] == ref_d2[t, keep].astype(np.float32)).all(), row


def test_real_valued_knn_in_batches_of_rows():
    # more query rows than go through at a time (2^18): half of them have
    # neighbours, the others equal more columns than a list holds and pass
    # both levels on to the FP64 engine, more of them than a batch too
    n, nq, d, k = 2_000, 600_001, 21, 8
    base, q = _real_points("copies", n, 300, d)
    r = np.random.default_rng(2)
    pick = np.where(r.random(nq) < 0.5, 0, r.integers(1, 300, nq))
    say("case: real-valued kNN in batches of rows")
    ids, dist = _ann().ann_gt_knn(_dev(base), _dev(q)[_dev(pick)].contiguous(), k)
    torch.cuda.synchronize()
    ref_ids, ref_d2 = oracle.knn(base, q, k)
    assert (q[0] == base).all(1).sum() > 512 and (pick == 0).sum() > 2 ** 18
    assert (ids.cpu().numpy() == ref_ids[pick]).all()
    assert (dist.cpu().numpy() == ref_d2.astype(np.float32)[pick]).all()


def test_real_valued_all_pairs_in_batches_of_rows():
    n, d, k = 300_001, 12, 10
    base, _ = _real_points("normal", n, 1, d)
    say("case: real-valued all pairs in batches of rows")
    x = _dev(base)
    ids, dist = _ann().ann_gt_knn(x, x, k)
    torch.cuda.synchronize()
    rows = np.concatenate([np.arange(0, n, 3_001), [n - 1]])
    ref_ids, ref_d2 = oracle.knn(base, base[rows], k)
    assert (ids.cpu().numpy()[rows] == ref_ids).all()
    assert (dist.cpu().numpy()[rows] == ref_d2.astype(np.float32)).all()


def test_real_valued_knn_of_more_rows_than_a_launch_of_wavefronts():
    # 2^26 rows of one wavefront each are 2^32 threads
    n, d, k = 2 ** 26 + 1_001, 4, 5
    say("case: real-valued kNN among %d rows" % n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    base = torch.randn((n, d), generator=gen, device="cuda")
    q = torch.cat([torch.randn((2, d), generator=gen, device="cuda"), base[-1:] + 1e-3])
    ids, dist = _ann().ann_gt_knn(base, q, k)
    for t in range(3):
        d2 = ((base.double() - q[t].double()) ** 2).sum(1)
        v, i = torch.topk(d2, k, largest=False)
        assert torch.equal(ids[t].long(), i)
        # one rounding to FP32, after FP64 sums in another order
        assert torch.allclose(dist[t].double(), v, rtol=2.0 ** -23, atol=0)


def _start_size(n, rows, dim, k):
    """The bytes that a kNN call took when it held the int8 and the FP64 engine alone."""
    ru = lambda x: (x + 255) // 256 * 256
    c = 2
    while c < k + 64:
        c *= 2
    kp, cap = k + 1, 64
    while cap < kp + 64 or (cap < 512 and cap < 2 * kp + 64):
        cap *= 2
    blocks = (rows + 255) // 256
    s = max(1, min(-(-2048 // blocks), max(n // 4096, 1), max(4096 // kp, 1)))
    sl = (-(-n // s) + 63) // 64 * 64
    slices = -(-n // sl)
    b = ru(rows * slices * cap * 8) + ru(rows * slices * 4) + ru(n * dim) + ru(n * 4) + ru(rows * dim) + ru(rows * 4)
    if rows == n and n >= 65536:
        b += 2 * ru(n * 4) + ru(256 * dim) + 3 * ru(257 * 4) + ru((n + 255) // 256 * 4)
    return max(ru(rows * c * 16) + 256, b + 256) + 256


@pytest.mark.parametrize("n,nq,d,k,ints", [
    (9_000, 700, 96, 10, False), (50_000, 50_000, 32, 16, True), (50_000, 50_000, 32, 16, False),
    (70_000, 70_000, 64, 64, True), (150_000, 5, 260, 10, False), (400, 3, 9, 1024, False),
])
def test_knn_takes_the_smaller_workspace(n, nq, d, k, ints):
    # a buffer for the int8 and the FP64 engine alone is enough for either
    # data, less is refused, and the results are the same
    ann = _ann()
    r = np.random.default_rng(n)
    x = r.integers(0, 256, size=(n, d)) if ints else np.rint(r.normal(size=(n, d)) * 2 ** 10) / 2 ** 10
    base = _dev(x.astype(np.float32))
    q = base if nq == n else base[torch.randperm(n, device="cuda")[:nq]] + 0.25
    ref = ann.ann_gt_knn(base, q, k)
    nb = _start_size(n, nq, d, k)
    say("case: kNN in the smaller workspace n=%d nq=%d d=%d k=%d" % (n, nq, d, k))
    ids, dist = torch.empty_like(ref[0]), torch.empty_like(ref[1])
    buf = torch.full((nb + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    call = lambda size: ann._lib.ann_gt_knn(ann._ptr(base), n, d, ann._ptr(q), nq, k, 0, ann._ptr(ids),
                                            ann._ptr(dist), ann._ptr(buf), size, ann._stream())
    assert call(nb) == ann.ANN_OK
    torch.cuda.synchronize()
    assert torch.equal(ids, ref[0]) and torch.equal(dist, ref[1])
    assert bool((buf[nb:] == 0x5A).all())
    if nq < n:      # all pairs in group order take a little less
        assert call(nb - 1) == ann.ANN_EINVAL


@pytest.mark.parametrize("ints,d", [(True, 32), (False, 20)])
def test_group_candidates_of_a_smaller_group_with_more_slices(ints, d):
    # 65,000 rows go through in more column slices than 70,000: the workspace,
    # sized for the larger group, serves both
    ann = _ann()
    n, first, K = 135_000, 70_000, 8
    r = np.random.default_rng(d)
    x = r.integers(0, 256, size=(n, d)) if ints else np.rint(r.normal(size=(n, d)) * 2 ** 10) / 2 ** 10
    base = _dev(x.astype(np.float32))
    lab = (torch.arange(n, device="cuda") >= first).to(torch.int32)[:, None].contiguous()
    cand = torch.empty((n, K), dtype=torch.int32, device="cuda")
    cd2 = torch.empty((n, K), dtype=torch.float64, device="cuda")
    say("case: candidates of two groups, d=%d" % d)
    ann.ann_group_candidates(base, K, lab, 2, 0, 2, cand, cd2)
    for a, b in ((0, first), (first, n)):
        part = base[a:b].contiguous()
        ids, dist = ann.ann_gt_knn(part, part, K, exclude_self=True)
        assert torch.equal(cand[a:b], ids + a)
        assert torch.equal(cd2[a:b].float(), dist)


def _repair_points(which):
    r = np.random.default_rng(17)
    if which == "equal points":
        # groups of equal points larger than the candidate lists: most
        # bridges need a full scan, and all of them want the same few nodes
        base = r.integers(0, 40, size=(900, 8))
        base[r.permutation(900)[:600]] = base[:3].repeat(200, 0)
        return base, 24, 12, 1.2
    if which == "islands":
        # far groups no larger than the lists, wider than one staged block of
        # dimensions; R at its largest
        cen = r.integers(0, 4000, size=(60, 136))
        return cen[r.integers(0, 60, 1300)] + r.integers(-3, 4, size=(1300, 136)), 64, 64, 1.0
    if which == "line":
        # points on a line, one candidate each: chains, and full scans for the rest
        return r.permutation(701)[:, None] * np.array([[1, 0, 0]]), 1, 3, 1.2
    i = np.arange(3001)
    if which == "line in order":
        # the medoid's label has to travel 1,500 edges each way
        return i[:, None] * np.array([[1, 0, 0, 0]]), 4, 4, 1.0
    if which == "lines apart":
        # ... in three lines, ids against, along and across the order
        x = np.concatenate([i[:1000][::-1], i[:1000] + 20000, r.permutation(1001) + 60000])
        return x[:, None] * np.array([[1, 0, 0, 0]]), 4, 4, 1.0
    if which == "one way":
        # spacings that grow: the candidates all lie on one side, so the
        # edges do too
        x = np.rint(np.cumsum(1.02 ** np.arange(700)))
        return x[:, None] * np.array([[1, 0]]), 3, 4, 1.0
    # "ring": two candidates each, so labels travel along one long chain
    a = np.arange(1024) * (2 * np.pi / 1024)
    base = np.rint(np.stack([np.cos(a), np.sin(a), 0 * a, 0 * a], 1) * 4096)
    return base[r.permutation(1024)], 2, 4, 1.0


@pytest.mark.parametrize("which", ["equal points", "islands", "line", "ring", "line in order",
                                   "lines apart", "one way"])
def test_build_graph_repair_bit_exact(which):
    base, K, R, alpha = _repair_points(which)
    base = np.ascontiguousarray(base, np.float32)
    say("case: repair, %s" % which)
    ref, med, nf, nr, _, _ = oracle.build_graph(base, K, R, alpha)
    assert nf > 0 or which in ("ring", "line in order", "one way")
    g, gm, (gf, gr) = _ann().ann_build_graph(_dev(base), K, R, alpha)
    torch.cuda.synchronize()
    assert gm == med and (gf, gr) == (nf, nr)
    assert (g.cpu().numpy() == ref).all()


@pytest.mark.parametrize("n,d,K,R,alpha,kind", [
    (700, 6, 9, 5, 1.2, "grid"),        # rows that are no float4s; a list that is no whole group
    (700, 20, 30, 32, 1.0, "small"),    # many exact ties a2 d2 == dpc; as few candidates as R allows
    (900, 128, 33, 32, 1.1, "grid"),    # the row a lane holds in registers, all of it
    (600, 300, 70, 64, 1.2, "grid"),    # more than it holds
    (600, 36, 24, 16, 1.2, "huge"),     # squares beyond FP32
    (600, 36, 24, 16, 1.2, "tiny"),     # ... and below it
])
def test_build_graph_prune_bit_exact(n, d, K, R, alpha, kind):
    r = np.random.default_rng(n + d)
    if kind == "small":
        base = r.integers(0, 3, size=(n, d)).astype(np.float32)
    else:
        base = (np.rint(r.normal(0, 1, size=(n, d)) * 256) / 256).astype(np.float32)
        base *= np.float32({"huge": 2.0 ** 70, "tiny": 2.0 ** -80}.get(kind, 1.0))
    say("case: prune n=%d d=%d K=%d R=%d %s" % (n, d, K, R, kind))
    ref, med, nf, nr, _, _ = oracle.build_graph(base, K, R, alpha)
    g, gm, (gf, gr) = _ann().ann_build_graph(_dev(base), K, R, alpha)
    torch.cuda.synchronize()
    assert gm == med and (gf, gr) == (nf, nr)
    assert (g.cpu().numpy() == ref).all()


def test_build_graph_partitioned_bit_exact():
    # candidates among the members of each point's home group (k-means
    # clusters, a second group for a third of the points, repeats, a home
    # group of one point, a small group), then prune / medoid / full-scan
    # repair; bit-exact against the oracle composition
    ann = _ann()
    ix = int_index()
    base = ix["base"]
    n = base.shape[0]
    K, R = 64, 32
    say("case: partitioned graph build, n=%d K=%d R=%d" % (n, K, R))
    km = oracle.kmeans_hubs(base, 4, 10, synth.kmeans_init(ix["w"], n, 4))
    groups = np.full((n, 2), -1, np.int32)
    groups[:, 0] = km["assign"]
    r = np.random.default_rng(3)
    sel = r.random(n) < 0.33
    groups[sel, 1] = r.integers(0, 4, int(sel.sum()))
    groups[7] = [4, -1]
    groups[100:110, 0] = 5
    groups[200:300, 1] = 5
    G = 6
    ref, med, nf, nr, _, _ = oracle.build_graph_grouped(base, groups, K, R, 1.2)
    g, m, br = ann.ann_build_graph_partitioned(_dev(base), K, R, 1.2, _dev(groups), G)
    torch.cuda.synchronize()
    assert m == med
    assert br == (nf, nr)
    assert (g.cpu().numpy() == ref).all()
    # the same build through the split entry points, a few groups per call
    say("case: group candidates in chunks + graph from candidates")
    bd, gd = _dev(base), _dev(groups)
    cand = torch.full((n, K), -7, dtype=torch.int32, device=bd.device)
    cd2 = torch.zeros((n, K), dtype=torch.float64, device=bd.device)
    for g0, g1 in ((0, 2), (2, 2), (2, 5), (5, 6)):
        ann.ann_group_candidates(bd, K, gd, G, g0, g1, cand, cd2)
    rc, rd = oracle.knn_in_home_group(base, groups, K)
    torch.cuda.synchronize()
    assert (cand.cpu().numpy() == rc).all()
    assert (cd2.cpu().numpy() == rd).all()
    g2, m2, br2 = ann.ann_graph_from_candidates(bd, cand, cd2, R, 1.2)
    torch.cuda.synchronize()
    assert m2 == med and br2 == (nf, nr)
    assert (g2.cpu().numpy() == ref).all()


def _merge_inputs(n, d, aw, bw, seed):
    r = np.random.default_rng(seed)
    base = (np.rint(r.normal(size=(n, d)) * 2 ** 10) / 2 ** 10).astype(np.float32)
    base[n // 2:n // 2 + 5] = base[3]            # equal distances, told apart by id
    a = r.integers(-1, n, size=(n, aw)).astype(np.int32)
    b = r.integers(-1, n, size=(n, bw)).astype(np.int32)
    if aw and bw:
        b[:, :min(aw, bw) // 2] = a[:, :min(aw, bw) // 2]   # repeats across the lists
    if aw:
        a[::7, 0] = np.arange(0, n, 7)                      # the row's own id
    return base, a, b


def _d2_rows(base, ids):
    # FP64 squared distances of row i to ids[i]; exact on this grid
    diff = base[np.maximum(ids, 0)].astype(np.float64) - base[:, None, :].astype(np.float64)
    return np.where(ids >= 0, (diff * diff).sum(-1), np.inf)


@pytest.mark.parametrize("n,d,aw,bw", [(300, 40, 37, 20), (129, 8, 0, 5), (200, 72, 300, 128),
                                       (64, 16, 900, 124), (97, 128, 1, 0)])
def test_merge_candidates_matches_oracle(n, d, aw, bw):
    say("case: merge_candidates n=%d d=%d aw=%d bw=%d" % (n, d, aw, bw))
    base, a, b = _merge_inputs(n, d, aw, bw, n + aw)
    ids, d2 = _ann().ann_merge_candidates(_dev(base), _dev(a) if aw else None,
                                          _dev(b) if bw else None)
    torch.cuda.synchronize()
    ea = a if aw else np.zeros((n, 0), np.int32)
    eb = b if bw else np.zeros((n, 0), np.int32)
    ref_ids, ref_d2 = oracle.merge_candidates(ea, _d2_rows(base, ea), eb, _d2_rows(base, eb))
    assert (ids.cpu().numpy() == ref_ids).all()
    assert (d2.cpu().numpy() == ref_d2).all()


def test_merge_candidates_rejects_ids_out_of_range():
    ann = _ann()
    base, a, b = _merge_inputs(100, 8, 10, 10, 5)
    a[17, 3] = 100
    say("case: merge_candidates id out of range")
    with pytest.raises(RuntimeError):
        ann.ann_merge_candidates(_dev(base), _dev(a), _dev(b))
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,d,knn_k,L,R,path", [(3000, 32, 32, 40, 16, 0),
                                                (2000, 64, 64, 100, 24, 0),
                                                (2500, 32, 16, 16, 24, 64)])
def test_nsg_graph_bit_exact(n, d, knn_k, L, R, path):
    from paper_2506_15986_amd import gate
    r = np.random.default_rng(n)
    if path:
        # uniform data: here the expanded nodes change about a fifth of the rows
        base = r.integers(0, 256, size=(n, d))
    else:
        cen = r.integers(30, 220, size=(12, d))
        base = np.clip(cen[r.integers(0, 12, n)] + r.integers(-25, 26, size=(n, d)), 0, 255)
    base = base.astype(np.float32)
    say("case: nsg graph n=%d d=%d knn_k=%d L=%d R=%d path=%d" % (n, d, knn_k, L, R, path))
    ix = gate.build_index_nsg(_dev(base), knn_k, R, L, path=path)
    g, m, nf, nr, _, _ = oracle.build_graph_nsg(base, knn_k, L, R, path=path)
    assert ix.medoid == m
    assert ix.bridges == (nf, nr)
    assert (ix.graph.cpu().numpy() == g).all()


def test_merge_candidates_single_point_and_self_only():
    base = np.array([[0.5, -1.0, 2.0, 0.25]], np.float32)
    a = np.array([[0, -1, 0]], np.int32)
    b = np.array([[-1, 0]], np.int32)
    say("case: merge_candidates n=1")
    ids, d2 = _ann().ann_merge_candidates(_dev(base), _dev(a), _dev(b))
    torch.cuda.synchronize()
    assert ids.cpu().numpy().tolist() == [[-1] * 5]
    assert np.isinf(d2.cpu().numpy()).all()
