"""The candidate passes over ranges of keys (Alg. 1's dictionary, Alg. 3's second layer) against the
oracle's estimates, exactly, where they can go wrong: dictionaries below one 256-key block and with a
ragged last one, several units of blocks, every hash and filter form (d 1..9, widths that are powers of
two and not, Count-Min), few hot counters, many (most keys reach the exact test) and too many for a
filter, super-items that straddle blocks, and both sides of the line below which no filter is built."""
import numpy as np
import pytest

import oracle
import paper_1711_00975_amd as csk

pytestmark = pytest.mark.gpu

THETA = 10


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _counters(d, w, share, variant, seed):
    """A share of the counters is hot (|M| >= THETA, both signs for Count Sketch), the rest is noise."""
    rng = np.random.default_rng(seed)
    M = rng.integers(-THETA + 1, THETA, (d, w))
    big = rng.integers(THETA, 1000, (d, w)) * (1 if variant else rng.choice([-1, 1], (d, w)))
    M = np.where(rng.random((d, w)) < share, big, np.abs(M) if variant else M).astype(np.int32)
    if share > 0.01:
        M.flat[:3] = (2**31 - 1, -2**31, THETA)
    return M


def _check(s, M, T, keys, variant, theta):
    est = oracle.estimate(M, T, keys, variant).astype(np.int64)
    sel = est >= theta
    u, e = keys[sel], est[sel]
    order = np.lexsort((u, -e))
    kg, eg, rc = s.topk(max(len(u), 1) + 1)
    assert len(kg) == len(u)
    assert np.array_equal(kg.cpu().numpy().view(np.uint64), u[order])
    assert np.array_equal(eg.cpu().numpy(), e[order])


FORMS = [(5, 1 << 14, 0), (5, 1 << 16, 0), (5, 1 << 16, 1), (5, 3 * 9973, 0), (5, 3 * 9973, 1), (1, 1 << 14, 0),
         (3, 50_021, 0), (4, 1 << 15, 1), (6, 1 << 16, 0), (6, 70_001, 0), (8, 1 << 14, 0), (8, 1 << 17, 1), (9, 1 << 14, 0)]


@pytest.mark.parametrize("d,w,variant", FORMS)
@pytest.mark.parametrize("share", [0.002, 0.2, 0.95])
@pytest.mark.parametrize("G,group", [(6, 1), (100, 1), (101, 7), (64, 1)])
def test_dictionary(d, w, variant, share, G, group):
    print("dictionary", d, w, variant, share, G, group, flush=True)
    seed = 5
    M, T = _counters(d, w, share, variant, d * w + G), oracle.hash_tables(seed, d)
    keys = np.arange((G**3 + group - 1) // group, dtype=np.uint64)
    s = csk.Sketch(d, w, seed, variant, 1 << 20, group)
    try:
        s.set_counters(_dev(M))
        for theta in (THETA, 700):
            s.clear_candidates()
            s.collect_dictionary(1.0, float(G), theta)
            _check(s, M, T, keys, variant, theta)
    finally:
        s.close()


@pytest.mark.parametrize("d,w", [(5, 1 << 16), (5, 200_003), (8, 1 << 16)])
def test_dictionary_of_several_units(d, w):
    print("units", d, w, flush=True)
    G, seed = 300, 5      # 27 M keys: eight blocks a unit, byte 3 in use
    M, T = _counters(d, w, 0.01, 0, w), oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed, 0, 1 << 20)
    try:
        s.set_counters(_dev(M))
        s.collect_dictionary(1.0, float(G), THETA)
        _check(s, M, T, np.arange(G**3, dtype=np.uint64), 0, THETA)
    finally:
        s.close()


def _line(d, w):
    return (1 << 19) + w // 10


@pytest.mark.parametrize("d,w,variant", [f for f in FORMS if f[0] in (1, 3, 5, 6, 9)])
@pytest.mark.parametrize("share", [0.002, 0.2, 0.95])
@pytest.mark.parametrize("group,side", [(1000, 0), (1000, 1), (777, 1), (64, 1), (1, 0)])
def test_children(d, w, variant, share, group, side):
    print("children", d, w, variant, share, group, side, flush=True)
    G, seed = 120, 6
    n = (G**3 + group - 1) // group
    m = min(n, _line(d, w) // group + side)
    rng = np.random.default_rng(m)
    supers = np.unique(np.concatenate([[0, n - 1], rng.choice(n, m, replace=False)]))[-m:]   # the ragged last one too
    cell = np.minimum(supers * group, G**3 - 1)
    pos = ((np.stack([cell // (G * G), cell // G % G, cell % G], 1) + 0.5)).astype(np.float32)
    M, T = _counters(d, w, share, variant, d * w), oracle.hash_tables(seed, d)
    keys = (supers[:, None] * group + np.arange(group)[None, :]).ravel()
    keys = keys[keys < G**3].astype(np.uint64)
    coarse, fine = csk.Sketch(5, 1 << 14, 9, 0, 1 << 21, group), csk.Sketch(d, w, seed, variant, 1 << 21)
    try:
        coarse.collect(_dev(pos), 1.0, float(G))
        fine.collect(_dev(pos[:0]), 1.0, float(G))
        fine.set_counters(_dev(M))
        fine.clear_candidates()
        fine.collect_children(coarse, THETA)
        _check(fine, M, T, keys, variant, THETA)
    finally:
        coarse.close()
        fine.close()


@pytest.mark.parametrize("d,w,variant", [(5, 1 << 18, 0), (5, 70_001, 0), (3, 1 << 18, 0), (8, 1 << 18, 1)])
@pytest.mark.parametrize("items,group,like", [(1, 300_000, 300), (10, 30_000, 300), (7, 999, 7), (3, 1_000_000, 3000),
                                              (100, 40_000, 4000)])
def test_children_of_few_large_super_items(d, w, variant, items, group, like):
    # as many children in few super-items as in many, directly and through the filter: the same keys as by
    # the oracle, and not much slower than the `like` super-items of 1000
    import time
    import torch
    G, L, theta, seed = 1000, 100.0, 600, 5
    rng = np.random.default_rng(items * group + d)
    M = rng.integers(0, 599, (d, w))
    hot = rng.random((d, w)) < 0.02
    M = np.where(hot, rng.integers(600, 2000, (d, w)), M)
    M = (M if variant else M * rng.choice([-1, 1], (d, w))).astype(np.int32)
    fine = csk.Sketch(d, w, seed, variant, 1 << 21)
    try:
        def children(n, of):
            """Time of the children of n random super-items of so many keys, and the super-items."""
            coarse = csk.Sketch(d, w, 9, variant, 1 << 16, group=of)
            try:
                at = rng.choice(G ** 3 // of, n, replace=False).astype(np.int64) * of
                c = np.stack([at // G ** 2, at // G % G, at % G], 1)
                coarse.collect(_dev(((c + 0.5) * (L / G)).astype(np.float32)), L / G, L)
                best = float("inf")
                for _ in range(4):
                    fine.clear_candidates()
                    torch.cuda.synchronize()
                    t = time.perf_counter()
                    fine.collect_children(coarse, theta)
                    torch.cuda.synchronize()
                    best = min(best, time.perf_counter() - t)
                return best * 1e6, at
            finally:
                coarse.close()

        fine.update(_dev(np.zeros((1, 3), dtype=np.float32)), L / G, L)     # latches the mesh
        fine.set_counters(_dev(M))
        usual, _ = children(like, 1000)
        took, at = children(items, group)
        print(f"children of {like} x 1000: {usual:.0f} us, of {items} x {group}: {took:.0f} us", flush=True)
        keys = (at[:, None] + np.arange(group)).ravel().astype(np.uint64)
        keys = keys[keys < G ** 3]
        est = oracle.estimate(M, oracle.hash_tables(seed, d), keys, variant)
        keys, est = keys[est >= theta], est[est >= theta]
        order = np.lexsort((keys, -est.astype(np.int64)))
        kg, eg, _ = fine.topk(len(keys) + 1)
        assert np.array_equal(kg.cpu().numpy().view(np.uint64), keys[order])
        assert np.array_equal(eg.cpu().numpy(), est[order])
        assert took < 2 * usual + 50
    finally:
        fine.close()
