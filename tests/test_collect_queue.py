"""The candidate pass with its per-wave queues, against the oracle's estimates, exactly, where it can go
wrong: every form of the filter for float and packed streams and odd widths, few hot counters, dense
filters, too many for one (every particle reaches the exact test), more new keys in a workgroup than it
holds back, a set that fills up, both sides of the short-stream rule, and a batch of all of these."""
import numpy as np
import pytest

import oracle
import paper_1711_00975_amd as csk

pytestmark = pytest.mark.gpu

L, DELTA, THETA = 100.0, 0.1, 10


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _stream(n, seed):
    """Half of the particles in 60^3 cells (about two each at n = 9e5), a tenth in one cell, wrapped ones."""
    rng = np.random.default_rng(seed)
    pos = np.where((rng.random(n) < 0.5)[:, None], rng.uniform(0, L, (n, 3)), rng.uniform(40, 46, (n, 3)))
    pos[rng.random(n) < 0.1] = 7.77
    pos = pos.astype(np.float32)
    pos[rng.choice(n, n // 100, replace=False), 1] = np.float32(-3.0)
    return pos


def _counters(d, w, share, variant, seed):
    rng = np.random.default_rng(seed)
    M = rng.integers(-THETA + 1, THETA, (d, w))
    big = rng.integers(THETA, 1000, (d, w)) * (1 if variant else rng.choice([-1, 1], (d, w)))
    return np.where(rng.random((d, w)) < share, big, np.abs(M) if variant else M).astype(np.int32)


def _want(M, T, keys, theta, variant):
    u = np.unique(keys)
    e = oracle.estimate(M, T, u, variant).astype(np.int64)
    u, e = u[e >= theta], e[e >= theta]
    order = np.lexsort((u, -e))
    return u[order], e[order]


def _check(s, want):
    kg, eg, _ = s.topk(len(want[0]) + 1)
    assert np.array_equal(kg.cpu().numpy().view(np.uint64), want[0])
    assert np.array_equal(eg.cpu().numpy(), want[1])


@pytest.mark.parametrize("d,w,variant", [(5, 1 << 16, 0), (5, 70_001, 0), (5, 70_001, 1), (5, (1 << 24) + 5, 0),
                                         (2, 1 << 16, 0), (4, 50_021, 1), (6, 1 << 16, 0), (8, 1 << 16, 0),
                                         (8, 99_991, 0)])
@pytest.mark.parametrize("share", [0.001, 0.3, 0.97])
@pytest.mark.parametrize("packed", [False, True])
def test_collect_forms(d, w, variant, share, packed):
    print("queue", d, w, variant, share, packed, flush=True)
    if w > 1 << 24:
        share /= 100     # about 1e5 and 1e6 hot counters
    n, seed = 1_300_003 if w <= 1 << 20 else (1 << 20) + 7, 5
    pos = _stream(n, d + w)
    words = oracle.pack(pos, L)
    keys = oracle.keys_packed(words, DELTA, L) if packed else oracle.keys(pos, DELTA, L)
    M, T = _counters(d, w, share, variant, d * w), oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed, variant, 1 << 21)
    try:
        s.set_counters(_dev(M))
        for theta in (THETA, 600):
            s.clear_candidates()
            if packed:
                s.collect_packed(_dev(words.view(np.int64)), DELTA, L, theta)
            else:
                s.collect(_dev(pos), DELTA, L, theta)
            _check(s, _want(M, T, keys, theta, variant))
    finally:
        s.close()


@pytest.mark.parametrize("w", [1 << 14, 1 << 20])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_the_short_rule(w, over):
    n, seed = (1 << 19) + w // 32 + over, 5
    pos = _stream(n, n)
    M, T = _counters(5, w, 0.2, 0, w), oracle.hash_tables(seed, 5)
    s = csk.Sketch(5, w, seed, 0, 1 << 20)
    try:
        s.set_counters(_dev(M))
        s.collect(_dev(pos), DELTA, L, THETA)
        _check(s, _want(M, T, oracle.keys(pos, DELTA, L), THETA, 0))
    finally:
        s.close()


@pytest.mark.parametrize("n", [200_000, 1_300_003])
@pytest.mark.parametrize("cap", [300, 5000])
def test_a_set_that_fills_up(n, cap):
    print("full", n, cap, flush=True)
    seed = 5
    pos = _stream(n, n + cap)
    M, T = _counters(5, 1 << 16, 0.97, 0, cap), oracle.hash_tables(seed, 5)
    s = csk.Sketch(5, 1 << 16, seed, 0, cap)
    try:
        s.set_counters(_dev(M))
        s.collect(_dev(pos), DELTA, L, THETA)
        with pytest.raises(csk.CskError) as ei:
            s.topk(10)
        assert ei.value.code == csk.CSK_E_CAPACITY
        s.clear_candidates()
        s.collect(_dev(pos[:cap]), DELTA, L, THETA)    # fits: the set is whole again
        _check(s, _want(M, T, oracle.keys(pos[:cap], DELTA, L), THETA, 0))
    finally:
        s.close()


def test_a_batch_of_them():
    import torch
    shapes = [(700_001, 1 << 16, 0.3), (90_000, 1 << 14, 0.97), (1_300_003, 1 << 17, 0.97), (5, 1 << 15, 0.5)]
    sk = [csk.Sketch(5, w, 20 + i, 0, 1 << 20) for i, (_, w, _) in enumerate(shapes)]
    try:
        pos = [_stream(max(n, 100), 70 + i)[:n] for i, (n, _, _) in enumerate(shapes)]
        b = csk.Batch(sk, [n for n, _, _ in shapes], DELTA, L)
        try:
            Ms = [_counters(5, w, share, 0, w) for _, w, share in shapes]
            for s, M in zip(sk, Ms):
                s.set_counters(_dev(M))
            b.collect([_dev(p) for p in pos], [THETA] * len(sk))
            torch.cuda.synchronize()
        finally:
            b.close()
        for i, (s, M, p) in enumerate(zip(sk, Ms, pos)):
            _check(s, _want(M, oracle.hash_tables(20 + i, 5), oracle.keys(p, DELTA, L), THETA, 0))
    finally:
        for s in sk:
            s.close()


@pytest.mark.parametrize("n", [1 << 19, 1 << 24])
def test_a_set_that_is_full_ends_the_look_ups(n):
    # once a key was refused (the error) no other can get in: the rest of the stream costs its hashes,
    # not a walk through the whole table per particle
    import time
    import torch
    print("full table", n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    pos = torch.rand((n, 3), generator=gen, device="cuda") * L
    same = torch.full((n, 3), 12.34, device="cuda")
    s = csk.Sketch(5, 1 << 14, 5, 0, 1 << 12)
    try:
        def seconds(p):
            best = float("inf")
            for _ in range(3):
                s.clear_candidates()
                torch.cuda.synchronize()
                t = time.perf_counter()
                s.collect(p, DELTA, L)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            return best

        one = seconds(same)
        kg, _, _ = s.topk(10)
        assert len(kg) == 1
        took = seconds(pos)
        with pytest.raises(csk.CskError) as ei:
            s.topk(10)
        assert ei.value.code == csk.CSK_E_CAPACITY
        print(f"{n} particles: one cell {one * 1e6:.0f} us, a full set {took * 1e6:.0f} us", flush=True)
        assert took < 5 * one + 2e-3
    finally:
        s.close()


@pytest.mark.parametrize("d,w", [(5, 1 << 16), (2, 5000), (9, 1 << 16)])
@pytest.mark.parametrize("cells", [1, 64])
def test_short_streams_of_few_cells(d, w, cells):
    # a key that all particles share is claimed by a few of them: in the time of a stream of many cells
    import time
    import torch
    n = 1 << 17
    rng = np.random.default_rng(cells)
    c = rng.uniform(0, L, (cells, 3)).astype(np.float32)[rng.integers(0, cells, n)]
    spread = rng.uniform(0, L, (n, 3)).astype(np.float32)
    M, T = _counters(d, w, 0.97, 0, d), oracle.hash_tables(5, d)
    s = csk.Sketch(d, w, 5, 0, 1 << 20)
    try:
        s.set_counters(_dev(M))

        def microseconds(p):
            best = float("inf")
            for _ in range(5):
                s.clear_candidates()
                torch.cuda.synchronize()
                t = time.perf_counter()
                s.collect(p, DELTA, L, csk.INT32_MIN)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            return best * 1e6

        usual, few = microseconds(_dev(spread)), microseconds(_dev(c))
        print(f"d={d}: {n} particles of many cells {usual:.0f} us, of {cells} {few:.0f} us", flush=True)
        _check(s, _want(M, T, oracle.keys(c, DELTA, L), csk.INT32_MIN, 0))
        if d <= 8:      # more rows take the general kernel
            assert few < 2 * usual + 50
    finally:
        s.close()


@pytest.mark.parametrize("n", [1 << 16, 1 << 19])
def test_particles_outside_of_short_streams_are_latched_in_passing(n):
    # half of the particles outside: reported, skipped, and in the time of a stream that is all inside
    import time
    import torch
    d, w, seed = 2, 5000, 5
    rng = np.random.default_rng(n)
    pos = rng.uniform(0, L, (n, 3)).astype(np.float32)
    out = pos.copy()
    out[::2, 0] = np.nan
    s = csk.Sketch(d, w, seed, 0, 1 << 21)
    try:
        def microseconds(call):
            best = float("inf")
            for _ in range(5):
                s.reset()
                torch.cuda.synchronize()
                t = time.perf_counter()
                call()
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            return best * 1e6

        for call in (s.update, lambda *a: s.collect(*a, 1 << 20)):
            inside, outside = _dev(pos), _dev(out)
            usual = microseconds(lambda: call(inside, DELTA, L))
            s.check()
            took = microseconds(lambda: call(outside, DELTA, L))
            with pytest.raises(csk.CskError) as ei:
                s.check()
            assert ei.value.code == csk.CSK_E_DOMAIN
            print(f"{n} particles: all inside {usual:.0f} us, half outside {took:.0f} us", flush=True)
            assert took < 1.5 * usual + 20
        s.reset()
        s.update(_dev(out), DELTA, L)
        with pytest.raises(csk.CskError):
            s.check()
        M, skipped = oracle.sketch(out, d, w, seed, DELTA, L, threads=8)
        assert skipped == n // 2 and np.array_equal(s.counters().cpu().numpy(), M)
    finally:
        s.close()


def _line(w):
    """The most particles that the short form of the candidate pass takes (d <= 8)."""
    return min(1 << 20, (1 << 19) + w // 32)


@pytest.mark.parametrize("d,w,group,variant", [(1, 1 << 14, 1, 0), (5, 3 * 9973, 1, 1), (8, 1 << 15, 1, 0),
                                               (8, 1 << 15, 1, 1), (3, 1 << 24, 1, 0), (5, 1 << 25, 1, 0),
                                               (5, 1 << 14, 8, 0), (5, 30_011, 1000, 1), (2, 5000, 64, 0)])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("packed", [False, True])
def test_both_sides_of_the_short_rule_for_every_stream(d, w, group, variant, over, packed):
    # on one side one thread tests a particle against every row's counter; on the other the filter and the
    # queues, or for grouped items the general kernel
    print("short rule", d, w, group, variant, over, packed, flush=True)
    n, seed = _line(w) + over, 7
    rng = np.random.default_rng(n + d)
    pos = _stream(n, n + d)
    if not packed:
        pos[rng.choice(n, 20, replace=False), 2] = np.float32(np.nan)   # outside the domain
    words = oracle.pack(pos, L)
    keys = oracle.keys_packed(words, DELTA, L) if packed else oracle.keys(pos, DELTA, L)
    keys = keys[keys != np.uint64(2**64 - 1)] // np.uint64(group)
    M, T = _counters(d, w, 0.05 if w <= 1 << 20 else 0.001, variant, d * w), oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed, variant, 1 << 21, group)
    try:
        s.set_counters(_dev(M))
        for theta in (THETA, 600, -5):
            if theta < 0 and group == 1 and d != 5:
                continue
            s.clear_candidates()
            if packed:
                s.collect_packed(_dev(words.view(np.int64)), DELTA, L, theta)
            else:
                s.collect(_dev(pos), DELTA, L, theta)
                with pytest.raises(csk.CskError) as ei:
                    s.check()
                assert ei.value.code == csk.CSK_E_DOMAIN
            _check(s, _want(M, T, keys, theta, variant))
    finally:
        s.close()


@pytest.mark.parametrize("d,w", [(5, 1 << 16), (5, 70_001), (2, 5000), (8, 100_003)])
def test_long_streams_of_one_cell(d, w):
    # a key that all particles share is claimed once a workgroup: in the time of a stream of 2^16 cells
    import time
    import torch
    n = 1 << 22
    rng = np.random.default_rng(d)
    one = np.full((n, 3), 12.34, dtype=np.float32)
    spread = rng.uniform(0, L, (1 << 16, 3)).astype(np.float32)[rng.integers(0, 1 << 16, n)]
    M, T = _counters(d, w, 0.97, 0, d), oracle.hash_tables(5, d)
    s = csk.Sketch(d, w, 5, 0, 1 << 20)
    try:
        s.set_counters(_dev(M))

        def microseconds(p):
            best = float("inf")
            for _ in range(5):
                s.clear_candidates()
                torch.cuda.synchronize()
                t = time.perf_counter()
                s.collect(p, DELTA, L, csk.INT32_MIN)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            return best * 1e6

        usual, few = microseconds(_dev(spread)), microseconds(_dev(one))
        print(f"d={d}: {n} particles of many cells {usual:.0f} us, of one {few:.0f} us", flush=True)
        _check(s, _want(M, T, oracle.keys(one, DELTA, L), csk.INT32_MIN, 0))
        assert few < 2 * usual + 50
    finally:
        s.close()
