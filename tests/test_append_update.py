"""The append bin kernel and the short-stream update against the oracle, bit for bit, where they
can go wrong: streams of one piece of 1024 particles and its neighbours, many flushes per
workgroup with a ragged end, bins that hold half a 64-byte piece in registers (w = 2^24), the
narrowest rows, structure order and a single cell (repeated cells, full buffers, full regions),
particles outside the domain, split accumulates, and both sides of the short-stream rule."""
import numpy as np
import pytest

import oracle
import paper_1711_00975_amd as csk

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _stream(n, L, seed, order):
    rng = np.random.default_rng(seed)
    if order == "one cell":
        return np.full((n, 3), 0.3 * L, dtype=np.float32)
    nclump = 40
    which = rng.integers(0, nclump, n)
    if order == "sorted":
        which = np.sort(which)
    centres = rng.uniform(0, L, (nclump, 3))
    clump = centres[which] + rng.normal(0, 0.002 * L, (n, 3))
    pos = np.where((rng.random(n) < 0.7)[:, None], clump, rng.uniform(0, L, (n, 3)))
    pos = np.mod(pos, L).astype(np.float32)
    pos[pos >= L] = 0.0
    if order == "outside":
        bad = rng.choice(n, max(1, n // 50), replace=False)
        pos[bad, rng.integers(0, 3, bad.size)] = rng.choice(
            np.array([np.nan, np.inf, 2 * L, -3 * L], dtype=np.float32), bad.size)
        wrap = rng.choice(n, max(1, n // 20), replace=False)   # inside [-L, 2L): wrapped, not skipped
        pos[wrap] = np.where(np.isfinite(pos[wrap]) & (np.abs(pos[wrap]) < L), pos[wrap] - np.float32(L), pos[wrap])
    return pos


def _check(n, d, w, L, delta, variant, order, max_wg, mode=None):
    print("append", n, d, w, L, delta, variant, order, max_wg, flush=True)
    pos = _stream(n, L, 17 + n % 97, order)
    mode = csk.CSK_UPDATE_BINNED if mode is None else mode
    s = csk.Sketch(d, w, 5, variant)
    try:
        s.set_update_plan(mode, max_wg)
        p = _dev(pos)
        s.update(p, delta, L)
        s.update(p[: n // 3], delta, L)          # a second call adds to the first
        if order == "outside":
            with pytest.raises(csk.CskError) as ei:
                s.check()
            assert ei.value.code == csk.CSK_E_DOMAIN
        M = s.counters().cpu().numpy()
    finally:
        s.close()
    Mo, _ = oracle.sketch(pos, d, w, 5, delta, L, variant=variant, threads=8)
    M2, _ = oracle.sketch(pos[: n // 3], d, w, 5, delta, L, variant=variant, threads=8)
    assert np.array_equal(M, Mo + M2)


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2049, 40_961])
def test_pieces_of_1024(n):
    _check(n, 5, 1 << 16, 100.0, 0.1, 0, "mixed", 0)


@pytest.mark.parametrize("d,w,L,delta,variant", [
    (5, 1 << 24, 1000.0, 0.25, 0),        # 2560 bins: half a piece waits in registers
    (5, (1 << 24) - 77, 1000.0, 0.25, 1), # the same on the row tables (or without the append kernel)
    (5, 1 << 23, 1000.0, 0.25, 0),        # 1280 bins, five per thread
    (6, 1 << 21, 100.0, 0.1, 0),
    (8, 3 * (1 << 20) + 5, 250.0, 250.0 / 768, 1),
    (8, 1 << 15, 100.0, 0.1, 0),          # 16-bit packed fields: no slice bits
    (7, 999, 3000.0, 0.5, 1),
    (4, 1000, 100.0, 0.4, 0),             # four key bytes
    (3, 1 << 18, 128.0, 0.125, 0),
    (2, 3, 100.0, 0.1, 0),
    (1, 1, 100.0, 0.1, 0),                # one counter: every token in one bin
])
@pytest.mark.parametrize("order", ["mixed", "sorted"])
def test_widths_with_many_flushes(d, w, L, delta, variant, order):
    _check(150_001, d, w, L, delta, variant, order, 3)


@pytest.mark.parametrize("d,w", [(5, 1 << 24), (5, 1 << 16), (8, 100_003)])
def test_one_cell(d, w):
    _check(200_003, d, w, 100.0, 0.1, 0, "one cell", 2)


@pytest.mark.parametrize("L,delta", [(1000.0, 0.25), (100.0, 0.1), (123.456, 0.123456)])
def test_outside_the_domain(L, delta):
    _check(60_001, 5, 1 << 20, L, delta, 0, "outside", 0)
    _check(3_001, 5, 1 << 20, L, delta, 0, "outside", 0, mode=csk.CSK_UPDATE_AUTO)


@pytest.mark.parametrize("d,w", [(5, 1 << 14), (3, 100_000), (1, 1 << 15)])
def test_split_accumulate(d, w):
    _check(1_500_001, d, w, 100.0, 0.1, 0, "mixed", 0)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("order", ["mixed", "one cell"])
def test_both_sides_of_the_short_stream_rule(order, variant):
    # n d <= 2^19 + d w / 21 goes straight to the counters
    d, w = 5, 1 << 16
    edge = ((1 << 19) + d * w // 21) // d
    for n in (255, 257, edge, edge + 1):
        _check(n, d, w, 100.0, 0.1, variant, order, 0, mode=csk.CSK_UPDATE_AUTO)


@pytest.mark.parametrize("w", [1 << 22, 99_991])
def test_packed_stream(w):
    n, d, L, delta = 200_001, 5, 1000.0, 0.25
    print("append packed", w, flush=True)
    pos = _stream(n, L, 3, "mixed")
    s = csk.Sketch(d, w, 5)
    try:
        s.set_update_plan(csk.CSK_UPDATE_BINNED, 2)
        s.update_packed(csk.pack_positions(_dev(pos), L), delta, L)
        M = s.counters().cpu().numpy()
    finally:
        s.close()
    keys = oracle.keys_packed(oracle.pack(pos, L), delta, L)
    assert np.array_equal(M, oracle.sketch_keys(keys, d, w, 5))


@pytest.mark.parametrize("d,w", [(1, 1), (1, 1000), (2, 3), (1, 1 << 15)])
def test_buffers_full_to_the_end_of_lds(d, w):
    # one or two bins of 4096 tokens, the last of LDS, full at every flush
    _check(300_001, d, w, 100.0, 0.1, 0, "mixed", 2)


@pytest.mark.parametrize("d,w", [(5, 1 << 16), (2, 5000)])
def test_direct_update_of_few_cells(d, w):
    # up to 2^20 particles one thread takes a particle and row, above it a particle: with 64 cells the adds
    # meet on few counters, and the first must not be the slower by more than a fifth
    import time
    import torch
    rng = np.random.default_rng(d)
    pos = rng.uniform(0, 100, (64, 3)).astype(np.float32)[rng.integers(0, 64, (1 << 20) + 1)]
    s = csk.Sketch(d, w, 5)
    try:
        s.set_update_plan(csk.CSK_UPDATE_DIRECT, 0)
        took = {}
        for n in (1 << 20, (1 << 20) + 1):
            p = _dev(pos[:n])
            took[n] = float("inf")
            for _ in range(8):
                s.reset()
                torch.cuda.synchronize()
                t = time.perf_counter()
                s.update(p, 0.1, 100.0)
                torch.cuda.synchronize()
                took[n] = min(took[n], time.perf_counter() - t)
            Mo, _ = oracle.sketch(pos[:n], d, w, 5, 0.1, 100.0, threads=8)
            assert np.array_equal(s.counters().cpu().numpy(), Mo), n
        print("direct update of 64 cells:", {n: f"{t * 1e6:.0f} us" for n, t in took.items()}, flush=True)
        assert took[1 << 20] < 1.2 * took[(1 << 20) + 1]
    finally:
        s.close()


@pytest.mark.parametrize("n,d,w", [(3_000_000, 5, 1 << 16), (3_000_000, 5, 1 << 14), (4_900_000, 5, 1 << 16), (1_200_001, 9, 40_000)])
def test_noalloc_update_shares_its_few_slices(n, d, w):
    # the general form of the update, slices shared by several workgroups as far as the fixed scratch has
    # room for their parts (none at 4.9 million): the same counters, and with room in about the time of
    # csk_sketch_update
    import time
    import torch
    pos = _stream(n, 100.0, 5, "mixed")
    s = csk.Sketch(d, w, 5)
    try:
        s.set_update_plan(csk.CSK_UPDATE_BINNED, 0)
        s.set_update_tiling(csk.CSK_BIN_GENERAL, 0, 0, 0)
        p = _dev(pos)

        def seconds(call):
            best = float("inf")
            for _ in range(5):
                s.reset()
                torch.cuda.synchronize()
                t = time.perf_counter()
                call(p, 0.1, 100.0)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            return best

        usual, took = seconds(s.update), seconds(s.update_noalloc)
        print(f"n={n} d={d} w={w}: update {usual * 1e6:.0f} us, without allocation {took * 1e6:.0f} us", flush=True)
        Mo, _ = oracle.sketch(pos, d, w, 5, 0.1, 100.0, threads=8)
        assert np.array_equal(s.counters().cpu().numpy(), Mo)
        if n <= 3_000_000:
            assert took < 1.3 * usual
    finally:
        s.close()


# ---- full regions: the append kernel's plan, and a stream that overfills one region of a workgroup

def _append_plan(n, d, w, max_wg, words, kb):
    """Particles of the fullest workgroup, region capacity, buffer tokens, granule, particles a flush: as
    plan_append() lays them out (words per table entry, key bytes looked up)."""
    Pr = (w + 32767) // 32768
    P = d * Pr
    fixed = 256 * words * kb * 4 + 4 * (P + 64) + 2 * P + 15 & ~15
    ring = min(((160 * 1024 - fixed - 16) // (2 * P)) & ~7, 4096)
    granule = 16 if ring < 48 else 32
    if granule == 16:
        assert ring >= 24
        ring = 24
    per_iter = 1024.0 * min(1.0, 32768 / w)
    pp = 8
    while pp > 2 and pp * per_iter + 2.5 * (pp * per_iter) ** 0.5 + granule - 1 > ring:
        pp //= 2
    pieces = -(-n // 1024)
    nwg = min(pieces, max_wg)
    per_wg = -(-pieces // nwg) * 1024
    cap = min(-(-per_wg * min(w, 32768) * 13 // (w * 10)) + 64, per_wg)
    return per_wg, -(-cap // 32) * 32, ring, granule, 1024 * pp


def _cells_of_one_slice(count, d, w, seed, L, G):
    """Centres of `count` cells whose row-0 buckets lie in the first slice."""
    T = oracle.hash_tables(seed, d)[0].astype(np.int64)
    rng = np.random.default_rng(w)
    got = np.zeros((0, 3), dtype=np.int64)
    while len(got) < count:
        c = rng.integers(0, G, (200_000, 3))
        key = (c[:, 0] * G + c[:, 1]) * G + c[:, 2]
        h = T[0][key & 255]
        for b in range(1, 6):
            h = h ^ T[b][(key >> (8 * b)) & 255]
        got = np.concatenate([got, c[((h & 0x7FFFFFFF) * w) >> 31 < min(w, 32768)]])
    return ((got[:count] + 0.5) * (L / G)).astype(np.float32)


@pytest.mark.parametrize("d,w,G,words,variant", [
    (5, 1 << 24, 1000, 4, 0),             # half a piece waits in registers when the region fills
    (5, 1 << 20, 1000, 4, 0),
    (8, 3 * (1 << 20) + 5, 768, 8, 1),    # row tables
    (4, 1 << 20, 1000, 4, 0),
    (5, 1 << 23, 1000, 4, 0),
])
@pytest.mark.parametrize("n", [200_704, 200_003])
def test_full_regions(d, w, G, words, variant, n):
    # 96 cells in random order: a wave has each less than twice, so next to none goes to the counters
    # straight away, and all of row 0 falls into one bin, far above its region
    print("full regions", d, w, n, flush=True)
    L, max_wg, seed = 250.0, 2, 5
    cells = _cells_of_one_slice(96, d, w, seed, L, G)
    which = np.random.default_rng(n).integers(0, len(cells), n)
    per_wg, cap, ring, granule, flush = _append_plan(n, d, w, max_wg, words, 4)
    waves = which[:n // 64 * 64].reshape(-1, 64)
    like = (waves == waves[:, :1]).sum(1) + (waves == waves[:, 29:30]).sum(1)
    assert np.mean(like < 8) > 0.9     # these waves append everything
    wait = region = 0                  # the fullest bin: what its buffer takes between two flushes
    for _ in range(per_wg // flush):
        wait = min(ring, wait + int(0.9 * flush))
        region += wait // granule * granule
        wait %= granule
    assert region > 1.1 * cap
    s = csk.Sketch(d, w, seed, variant)
    try:
        s.set_update_plan(csk.CSK_UPDATE_BINNED, max_wg)
        pos = cells[which]
        s.update(_dev(pos), L / G, L)
        s.update(_dev(pos[: n // 2]), L / G, L)
        M = s.counters().cpu().numpy()
    finally:
        s.close()
    Mo, _ = oracle.sketch(pos, d, w, seed, L / G, L, variant=variant, threads=8)
    M2, _ = oracle.sketch(pos[: n // 2], d, w, seed, L / G, L, variant=variant, threads=8)
    assert np.array_equal(M, Mo + M2)
