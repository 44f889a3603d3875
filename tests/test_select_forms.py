"""The top-k selection and the candidate pass of short streams against the oracle, exactly, where they
can go wrong: one block and many (8192 candidates and their neighbours), k at the sizes where the
placement changes, ties at the threshold down to the last key bit, estimates of the whole 32-bit
range, several selections of one handle and replays of a graph, a full candidate list, and both
sides of the short-stream rule of the candidate pass for every kind of stream."""
import numpy as np
import pytest

import oracle
import paper_1711_00975_amd as csk

pytestmark = pytest.mark.gpu

L, DELTA = 100.0, 0.1


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _cells(n, seed):
    """n particles in n distinct cells of the 1000^3 mesh, at the cells' centres."""
    rng = np.random.default_rng(seed)
    key = rng.choice(1 << 29, n, replace=False).astype(np.int64)
    c = np.stack([key % 1000, key // 1000 % 1000, key // 10**6], 1)
    return ((c + 0.5) * DELTA).astype(np.float32)


def _counters(kind, d, w, seed):
    rng = np.random.default_rng(seed)
    if kind == "ties":
        return rng.integers(3, 5, (d, w)).astype(np.int32)
    if kind == "near":
        return rng.integers(-60000, 60000, (d, w)).astype(np.int32)
    M = rng.integers(-2**31, 2**31, (d, w)).astype(np.int32)     # whole range
    M.flat[:4] = (-2**31, 2**31 - 1, 0, -1)
    return M


@pytest.mark.parametrize("n", [1, 63, 8192, 8193, 70_001])
@pytest.mark.parametrize("kind", ["ties", "near", "wide"])
@pytest.mark.parametrize("variant", [0, 1])
def test_select_against_the_oracle(n, kind, variant):
    import torch
    print("select", n, kind, variant, flush=True)
    d, w, seed = 5, 1 << 14, 3
    pos, T = _cells(n, n), oracle.hash_tables(seed, d)
    M = _counters(kind, d, w, n + variant)
    keys = oracle.keys(pos, DELTA, L)
    s = csk.Sketch(d, w, seed, variant)
    try:
        s.set_counters(_dev(M))
        for theta in (csk.INT32_MIN, 4):
            s.clear_candidates()
            s.collect(_dev(pos), DELTA, L, theta)
            ko, eo = oracle.topk_keys(M, T, keys, theta, n + 5, variant)
            for k in sorted({0, 1, min(n, 1024), 1025, n // 2, max(n - 1, 0), n, n + 5}):
                kg, eg, rc = s.topk(k)
                assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko[:k]), (theta, k)
                assert np.array_equal(eg.cpu().numpy(), eo[:k]), (theta, k)
                partial = theta != csk.INT32_MIN and k > len(ko)
                assert rc == (csk.CSK_W_INCOMPLETE if partial else csk.CSK_OK), (theta, k)
        # the same in a graph, its replays between eager work
        k = min(n, 1500)
        ok, oe = torch.empty(k, dtype=torch.int64, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
        out = torch.zeros(2, dtype=torch.int32, device="cuda")
        s.topk_async(k, ok, oe, out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            s.topk_async(k, ok, oe, out)
        for rep in range(3):
            s.topk(1)
            ok.zero_(), oe.zero_(), out.zero_()
            g.replay()
            torch.cuda.synchronize()
            m = min(k, len(ko))
            assert int(out[0]) == m, rep
            assert np.array_equal(ok[:m].cpu().numpy().view(np.uint64), ko[:m]), rep
            assert np.array_equal(oe[:m].cpu().numpy(), eo[:m]), rep
    finally:
        s.close()


@pytest.mark.parametrize("G", [4096, 4097, 9000])
def test_ties_up_to_the_highest_key_bits(G):
    # 2^36 cells, the most whose keys' top digit pass is left out, and more
    d, w, seed, n = 5, 1 << 14, 3, 20_000
    rng = np.random.default_rng(G)
    c = rng.integers(0, G, (n, 3))
    c[: n // 2] = G - 1 - rng.integers(0, 3, (n // 2, 3)) * rng.integers(0, G // 3, (n // 2, 3))   # up to the last cell
    pos = (c + 0.5).astype(np.float32)
    M, T = _counters("ties", d, w, G), oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed)
    try:
        s.set_counters(_dev(M))
        s.collect(_dev(pos), 1.0, float(G))
        ko, eo = oracle.topk_keys(M, T, oracle.keys(pos, 1.0, float(G)), csk.INT32_MIN, n)
        for k in (1, 700, 5000, len(ko) - 1, len(ko)):
            kg, eg, _ = s.topk(k)
            assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko[:k]), k
            assert np.array_equal(eg.cpu().numpy(), eo[:k]), k
    finally:
        s.close()


@pytest.mark.parametrize("n", [255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("kind", ["ties", "near", "wide"])
def test_candidates_ranked_outright(n, kind):
    # at most 512 candidates are ranked without a selection, unless k is above 1024
    d, w, seed = 5, 1 << 14, 3
    pos, T = _cells(n, n), oracle.hash_tables(seed, d)
    M = _counters(kind, d, w, n)
    ko, eo = oracle.topk_keys(M, T, oracle.keys(pos, DELTA, L), csk.INT32_MIN, n)
    s = csk.Sketch(d, w, seed)
    try:
        s.set_counters(_dev(M))
        s.collect(_dev(pos), DELTA, L)
        for k in (1, 64, 255, 256, n - 1, n, 1024, 1025):
            kg, eg, _ = s.topk(k)
            assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko[:k]), k
            assert np.array_equal(eg.cpu().numpy(), eo[:k]), k
    finally:
        s.close()


def test_few_candidates_after_many():
    # one block selects, the rank kernel places (k > 1024): nothing is left of the selection before
    d, w, seed = 5, 1 << 14, 3
    T = oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed)
    try:
        for n, kind in [(70_001, "near"), (5000, "near"), (70_001, "wide"), (4000, "ties"), (3000, "near")]:
            pos, M = _cells(n, n), _counters(kind, d, w, n)
            s.set_counters(_dev(M))
            s.clear_candidates()
            s.collect(_dev(pos), DELTA, L)
            kg, eg, _ = s.topk(2500)
            ko, eo = oracle.topk_keys(M, T, oracle.keys(pos, DELTA, L), csk.INT32_MIN, 2500)
            assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko), (n, kind)
            assert np.array_equal(eg.cpu().numpy(), eo), (n, kind)
    finally:
        s.close()


def test_a_full_candidate_list_is_an_error_and_clears():
    d, w, seed = 5, 1 << 14, 3
    pos, T = _cells(300, 9), oracle.hash_tables(seed, d)
    M = _counters("near", d, w, 5)
    s = csk.Sketch(d, w, seed, 0, 256)
    try:
        s.set_counters(_dev(M))
        s.collect(_dev(pos), DELTA, L)
        with pytest.raises(csk.CskError) as ei:
            s.topk(10)
        assert ei.value.code == csk.CSK_E_CAPACITY
        s.clear_candidates()
        s.collect(_dev(pos[:256]), DELTA, L)
        kg, eg, rc = s.topk(256)
        ko, eo = oracle.topk_keys(M, T, oracle.keys(pos[:256], DELTA, L), csk.INT32_MIN, 256)
        assert rc == csk.CSK_OK
        assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko) and np.array_equal(eg.cpu().numpy(), eo)
    finally:
        s.close()


def _line(d, w):
    """The most particles that the short form of the candidate pass takes."""
    return ((5 << 18) + d * w // 21) // d


@pytest.mark.parametrize("d,w,group,variant", [(1, 1 << 14, 1, 0), (5, 1 << 14, 1, 0), (5, 3 * 9973, 1, 1),
                                               (8, 1 << 15, 1, 0), (5, 1 << 14, 8, 0), (9, 1 << 14, 1, 0)])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("packed", [False, True])
def test_collect_on_both_sides_of_the_short_rule(d, w, group, variant, over, packed):
    print("short rule", d, w, group, variant, over, packed, flush=True)
    n, seed = min(_line(d, w), 1 << 20) + over, 7
    rng = np.random.default_rng(n)
    pos = np.where((rng.random(n) < 0.5)[:, None], rng.uniform(0, L, (n, 3)), rng.uniform(40, 40.6, (n, 3)))
    pos = pos.astype(np.float32)
    pos[rng.choice(n, 50, replace=False), 1] = np.float32(-3.0)     # wraps
    if not packed:
        pos[rng.choice(n, 20, replace=False), 2] = np.float32(np.nan)   # outside the domain
    words = oracle.pack(pos, L)
    keys = oracle.keys_packed(words, DELTA, L) if packed else oracle.keys(pos, DELTA, L)
    keys = keys // np.uint64(group)
    T = oracle.hash_tables(seed, d)
    s = csk.Sketch(d, w, seed, variant, 1 << 21, group)
    try:
        if packed:
            s.update_packed(_dev(words.view(np.int64)), DELTA, L)
        else:
            s.update(_dev(pos), DELTA, L)
            with pytest.raises(csk.CskError) as ei:     # reports the skipped particles and clears the latch
                s.check()
            assert ei.value.code == csk.CSK_E_DOMAIN
        M = s.counters().cpu().numpy()
        if group == 1 and not packed:
            Mo, skipped = oracle.sketch(pos, d, w, seed, DELTA, L, variant=variant, threads=8)
            assert skipped == 20 and np.array_equal(M, Mo)
        for theta in (1, 900):
            s.clear_candidates()
            if packed:
                s.collect_packed(_dev(words.view(np.int64)), DELTA, L, theta)
            else:
                s.collect(_dev(pos), DELTA, L, theta)
                with pytest.raises(csk.CskError) as ei:
                    s.check()
                assert ei.value.code == csk.CSK_E_DOMAIN
            ko, eo = oracle.topk_keys(M, T, keys, theta, 3000, variant)
            kg, eg, _ = s.topk(3000)
            assert np.array_equal(kg.cpu().numpy().view(np.uint64), ko), theta
            assert np.array_equal(eg.cpu().numpy(), eo), theta
    finally:
        s.close()
