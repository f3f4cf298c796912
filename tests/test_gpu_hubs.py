"""GPU parity of hub selection (Lloyd k-means + Definition 3) and of the hub
topology features against the CPU oracle."""
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


@pytest.mark.parametrize("which,nh", [("tiny", 64), ("int", 64), ("tiny", 7)])
def test_select_hubs_bit_exact(which, nh):
    ix = tiny_index() if which == "tiny" else int_index()
    base = ix["base"]
    init = synth.kmeans_init(ix["w"], base.shape[0], nh)
    say("case: select_hubs %s nh=%d" % (which, nh))
    ref = oracle.kmeans_hubs(base, nh, 20, init)
    hub, cen, asg, steps = _ann().ann_select_hubs(_dev(base), nh, 20, _dev(init))
    torch.cuda.synchronize()
    assert steps == ref["steps"]
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


@pytest.mark.parametrize("seed", [0, 2**63 + 11])
def test_select_hubs_from_a_seed_bit_exact(seed):
    # the library's seeded start (SplitMix64 + Floyd's sampling) is the
    # oracle's: the same centroids, assignment and hubs
    ix = int_index()
    base = ix["base"]
    nh = 48
    say("case: select_hubs from seed %d" % seed)
    init = oracle.hub_init_ids(base.shape[0], nh, seed)
    ref = oracle.kmeans_hubs(base, nh, 20, init)
    hub, cen, asg, steps = _ann().ann_select_hubs(_dev(base), nh, 20, seed=seed)
    torch.cuda.synchronize()
    assert steps == ref["steps"]
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


@pytest.mark.parametrize("case", ["repeated", "wide", "odd_dim"])
def test_select_hubs_bit_exact_special_shapes(case):
    # repeated: 5 distinct rows behind 3,000 points and 64 centroids, so many
    # centroids coincide (exact ties, shortlists longer than their capacity:
    # the all-centroid fallback); wide: 960 dimensions (30 LDS stages per
    # pass) on the 2^-14 grid; odd_dim: 6 dimensions (no float4 rows: the
    # FP64 assignment kernel)
    r = np.random.default_rng(31)
    if case == "repeated":
        rows = r.integers(0, 256, size=(5, 64)).astype(np.float32)
        base = rows[r.integers(0, 5, size=3000)]
        nh = 64
    elif case == "wide":
        w = synth.scaled(synth.WORKLOADS["gist1m"], n=2000)
        base = synth.base(w)
        nh = 40
    else:
        base = (np.rint(r.normal(0, 4, size=(3000, 6)) * 2 ** 12) / 2 ** 12).astype(np.float32)
        nh = 24
    init = r.choice(base.shape[0], nh, replace=False).astype(np.int32)
    say("case: select_hubs %s" % case)
    ref = oracle.kmeans_hubs(base, nh, 20, init)
    hub, cen, asg, steps = _ann().ann_select_hubs(_dev(base), nh, 20, _dev(init))
    torch.cuda.synchronize()
    assert steps == ref["steps"]
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


@pytest.mark.parametrize("case,n,dim,nh,iters", [
    ("ints", 5000, 20, 33, 6),        # one fragment of 32 dimensions, part of it
    ("ints", 5000, 64, 100, 6),       # two
    ("offset", 4000, 96, 70, 6),      # three, far from the origin
    ("ints", 3001, 200, 64, 5),       # eight
    ("ints", 2000, 400, 40, 4),       # sixteen
    ("ints", 1500, 1000, 24, 4),      # thirty-two
    ("ints", 900, 128, 1, 3),         # a single centroid
    ("outlier", 4000, 128, 65, 5),    # a point beyond FP16's range
    ("tight", 40000, 32, 64, 3),      # sixteen near centroids in each far place:
                                      # more points left than the class search takes
    ("tight", 3000, 32, 64, 3),       # ... and fewer
    ("ints", 17000, 4, 16400, 2),     # more centroids than the FP16 products take
])
def test_select_hubs_bit_exact_assignment_paths(case, n, dim, nh, iters):
    r = np.random.default_rng(n + dim)
    if case == "ints":
        base = r.integers(0, 256, size=(n, dim)).astype(np.float32)
    elif case == "offset":
        base = (3000 + np.rint(r.normal(0, 40, size=(n, dim)) * 256) / 256).astype(np.float32)
    elif case == "outlier":
        base = r.integers(0, 256, size=(n, dim)).astype(np.float32)
        base[17] = 2.0 ** 27
    else:
        place = 2000.0 * r.integers(-1, 2, size=(4, dim))
        base = (place[r.integers(0, 4, size=n)] +
                np.rint(r.normal(0, 1, size=(n, dim)) * 256) / 256).astype(np.float32)
    init = r.choice(n, nh, replace=False).astype(np.int32)
    say("case: select_hubs %s n=%d dim=%d nh=%d" % (case, n, dim, nh))
    ref = oracle.kmeans_hubs(base, nh, iters, init)
    hub, cen, asg, steps = _ann().ann_select_hubs(_dev(base), nh, iters, _dev(init))
    torch.cuda.synchronize()
    assert steps == ref["steps"]
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


def test_select_hubs_empty_cluster():
    x = np.zeros((8, 4), np.float32)
    x[:, 0] = [0, 0, 10, 11, 0, 0, 10, 11]
    x[4:, 1] = 0.5
    init = np.array([0, 1, 2], np.int32)
    say("case: select_hubs empty cluster")
    ref = oracle.kmeans_hubs(x, 3, 5, init)
    hub, cen, asg, steps = _ann().ann_select_hubs(_dev(x), 3, 5, _dev(init))
    torch.cuda.synchronize()
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


def test_hub_features_match_oracle():
    ix = tiny_index()
    base, g, med = ix["base"], ix["graph"], ix["medoid"]
    nh = 64
    init = synth.kmeans_init(ix["w"], base.shape[0], nh)
    km = oracle.kmeans_hubs(base, nh, 20, init)
    say("case: hub features tiny")
    ref, ref_ws = oracle.hub_features(base, g, med, km["hub_ids"], km["assign"], km["centroids"])
    raw, _ = oracle.hub_features(base, g, med, km["hub_ids"], km["assign"], km["centroids"],
                                 standardize=False)
    ann = _ann()
    args = (_dev(base), _dev(g), med, _dev(km["hub_ids"]), _dev(km["assign"]),
            _dev(km["centroids"]))
    f, wsz = ann.ann_hub_features(*args)
    fr, _ = ann.ann_hub_features(*args, standardise=False)
    torch.cuda.synchronize()
    assert (wsz.cpu().numpy() == ref_ws).all()
    assert np.allclose(fr.cpu().numpy(), raw, rtol=1e-5, atol=1e-6)
    assert np.allclose(f.cpu().numpy(), ref, rtol=0, atol=1e-4)


@pytest.mark.parametrize("case,n,dim,nh,iters", [
    ("ints", 5000, 20, 900, 4),        # the FP16 products, one fragment, part of it
    ("ints", 5000, 64, 300, 5),        # two
    ("offset", 4000, 96, 200, 5),      # three, far from the origin
    ("outlier", 4000, 128, 150, 5),    # four; a point beyond FP16's range
    ("tight", 140000, 32, 64, 3),      # more points left than the class search takes
    ("ints", 3000, 64, 256, 4),        # the last shape of the FP32 kernel alone
    ("ints", 3000, 64, 257, 4),        # ... and the first past it
    ("ints", 6400, 8, 100, 4),         # sums by atomics: 64 points a cluster,
    ("ints", 6401, 8, 100, 4),         # by the sort: more
])
def test_select_hubs_dispatch_lines(case, n, dim, nh, iters):
    test_select_hubs_bit_exact_assignment_paths(case, n, dim, nh, iters)


@pytest.mark.parametrize("m", [2, 3, 4, 5])
def test_select_hubs_equal_centroids(m):
    # every centroid starts m times over, in lanes of their own: a point has m
    # open candidates (up to four are decided in one list, five go to the
    # class search) and takes the first
    r = np.random.default_rng(m)
    # (more than 16,384 centroid values: the FP16 products)
    n, dim, places = 4000, 64, 140
    base = r.integers(0, 256, size=(n, dim)).astype(np.float32)
    init = r.choice(n, m * places, replace=False).astype(np.int32)
    for j in range(m):
        base[init[j * places:(j + 1) * places]] = base[init[:places]]
    say("case: select_hubs, %d equal centroids" % m)
    for iters in (1, 3):
        ref = oracle.kmeans_hubs(base, m * places, iters, init)
        hub, cen, asg, steps = _ann().ann_select_hubs(_dev(base), m * places, iters, _dev(init))
        torch.cuda.synchronize()
        assert steps == ref["steps"]
        assert (asg.cpu().numpy() == ref["assign"]).all()
        assert (cen.cpu().numpy() == ref["centroids"]).all()
        assert (hub.cpu().numpy() == ref["hub_ids"]).all()


def test_select_hubs_more_open_points_than_a_quarter_of_int32():
    # every centroid twice: all of 2^29 + 77 points are open (four lanes each
    # decide them) and join the first of the two, as without the copies
    n, places = 2 ** 29 + 77, 16
    say("case: select_hubs, %d open points" % n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    base = torch.randint(0, 256, (n, 4), generator=gen, device="cuda", dtype=torch.float32)
    init = torch.arange(places, dtype=torch.int32, device="cuda") * 1000
    twice = torch.cat([init, init + 1])
    base[twice[places:].long()] = base[init.long()]
    _, _, one, _ = _ann().ann_select_hubs(base, places, 1, init)
    _, _, two, _ = _ann().ann_select_hubs(base, 2 * places, 1, twice)
    assert torch.equal(one, two)


@pytest.mark.parametrize("n,dim,R,h,wcap", [
    (900, 6, 64, 3, 1),       # the hub alone; rows that are no float4 rows
    (900, 6, 64, 4, 17),      # the cap falls inside the first batch of nodes
    (3000, 20, 64, 5, 1000),  # the cap falls inside a full batch, 64-wide rows
    (3000, 20, 7, 250, 4096), # no cap: the walk ends by itself, odd row length
    (5000, 33, 48, 5, 4096),  # the largest cap crossed
])
def test_hub_features_walk_edges(n, dim, R, h, wcap):
    # whole numbers of the walk exactly, features as closely as FP64 sums in
    # another order allow once rounded to FP32 (2^-24 relative, and 1e-6 of
    # the unit-scale features)
    rng = np.random.default_rng(n + R)
    base = (np.rint(rng.normal(0, 40, size=(n, dim)))).astype(np.float32)
    g = rng.integers(0, n, size=(n, R)).astype(np.int32)
    for v in range(n):   # distinct neighbours, no self edge, rows of any length
        row = np.unique(g[v][g[v] != v])[:rng.integers(0, R + 1)]
        g[v] = -1
        g[v, :row.size] = rng.permutation(row)
    nh = 40
    hubs = rng.choice(n, nh, replace=False).astype(np.int32)
    asg = rng.integers(0, nh, size=n).astype(np.int32)
    cen = rng.normal(0, 30, size=(nh, dim))
    say("case: hub features walk n=%d R=%d h=%d wcap=%d" % (n, R, h, wcap))
    ref, ref_ws = oracle.hub_features(base, g, 5, hubs, asg, cen, h=h, wcap=wcap,
                                      standardize=False)
    f, ws = _ann().ann_hub_features(_dev(base), _dev(g), 5, _dev(hubs), _dev(asg), _dev(cen),
                                    h=h, wcap=wcap, standardise=False)
    torch.cuda.synchronize()
    assert (ws.cpu().numpy() == ref_ws).all()
    assert np.allclose(f.cpu().numpy(), ref, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("which,k,levels,lam,iters", [
    ("int", 8, 2, 1.0, 5),       # integers 0..255, 64 clusters
    ("tiny", 4, 3, 0.5, 4),      # grid data, 64 clusters over 3 rounds
    ("tiny", 16, 1, 0.0, 6),     # no size term: Lloyd from spaced members
    ("int", 4, 2, 1e9, 2),       # a dominant size term: exact balance
])
def test_hbkm_hubs_bit_exact(which, k, levels, lam, iters):
    ann = _ann()
    ix = int_index() if which == "int" else tiny_index()
    base = ix["base"]
    say("case: HBKM %s k=%d levels=%d lambda=%g iters=%d" % (which, k, levels, lam, iters))
    hub, cen, asg = ann.ann_select_hubs_hbkm(_dev(base), k, levels, lam, iters)
    torch.cuda.synchronize()
    ref = oracle.hbkm_hubs(base, k, levels, lam, iters)
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()


def test_hbkm_more_clusters_than_distinct_points():
    # 64 clusters of 80 points with only 20 distinct rows: empty children and
    # the empty-cluster hub rule
    ann = _ann()
    r = np.random.default_rng(9)
    rows = r.integers(0, 256, size=(20, 32)).astype(np.float32)
    base = rows[r.integers(0, 20, size=80)]
    say("case: HBKM with repeated rows, 64 clusters")
    hub, cen, asg = ann.ann_select_hubs_hbkm(_dev(base), 8, 2, 0.0, 3)
    torch.cuda.synchronize()
    ref = oracle.hbkm_hubs(base, 8, 2, 0.0, 3)
    assert (asg.cpu().numpy() == ref["assign"]).all()
    assert (cen.cpu().numpy() == ref["centroids"]).all()
    assert (hub.cpu().numpy() == ref["hub_ids"]).all()
    assert len(set(hub.cpu().numpy().tolist())) == 64
