"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values.  Its `kind` names the calls of one pass:

  update   one snapshot into fresh counters, and the counters out: what a checkpoint, or one
           rank's share before the sketches are summed, takes (reset, update, counters)
  step     one snapshot to its heaviest cells (reset, update, collect, top-k)
  batch    many sub-volumes at once, each to its own heaviest cells (the Batch calls)
  routed   the learned router in front of the sketch (RoutedStep)
  query    estimates of a list of cell keys from a filled sketch
  search   every cell of the mesh against a filled sketch (full search), then the top-k
  layers   the two-layer search: heavy super-cells first, then the cells inside them
  train    minibatch training of the router's model

Streams are Plummer halos with masses ~ M^-1.9 over a uniform background, drawn on the GPU
from the seed; `order` "mixed" interleaves the halos as a random draw does, "halo" keeps the
particles of a halo together as a snapshot sorted by structure does.  `chunks` > 1 hands the
stream over in that many calls, as a program that reads a snapshot file by file would.
"""
import math

import numpy as np
import torch

import paper_1711_00975_amd as csk
from paper_1711_00975_amd.router import RoutedStep, Router, rest_width

SCALE_RADIUS = 0.2        # Plummer scale radius, Mpc/h
DRAW_CHUNK = 1 << 25      # particles drawn at a time
COUNT_MIN = csk.CSK_VARIANT_COUNT_MIN
SKETCH = csk.CSK_VARIANT_COUNT_SKETCH


def listed():
    return [
        # The smallest call: a serving loop that looks at a few thousand particles at a time.
        # Latency and launches are all there is.
        dict(name="tiny_step", kind="step", n=4093, L=100.0, G=1000, d=5, w=1 << 14, k=100, halos=8,
             m_lo=100.0, m_hi=1e4, f_bg=0.5, order="mixed", chunks=1, packed=False, variant="sketch", wait=False),
        # One sub-volume snapshot of 2^20 particles, the benchmark's small workload: as the
        # counters a rank hands on, and as a whole step.
        dict(name="small_update", kind="update", n=1 << 20, L=100.0, G=1000, d=5, w=1 << 16, halos=256,
             m_lo=100.0, m_hi=1e4, f_bg=0.9, order="mixed", chunks=1, packed=False, variant="sketch"),
        dict(name="small_step", kind="step", n=1 << 20, L=100.0, G=1000, d=5, w=1 << 16, k=100, halos=256,
             m_lo=100.0, m_hi=1e4, f_bg=0.9, order="mixed", chunks=1, packed=False, variant="sketch", wait=True),
        # Nothing a power of two: more rows, a width and a mesh that take the general forms, a
        # ragged stream in structure order, and the Count-Min variant.
        dict(name="ragged_update", kind="update", n=12_345_677, L=250.0, G=768, d=8, w=3 * (1 << 20) + 5,
             halos=3001, m_lo=50.0, m_hi=1e5, f_bg=0.3, order="halo", chunks=3, packed=False, variant="min"),
        # The paper's packed stream (three coordinates in 64 bits), read in file-sized pieces
        # into counters that stay in the last-level cache.
        dict(name="packed_update", kind="update", n=1 << 27, L=1000.0, G=4000, d=5, w=1 << 22, halos=1 << 17,
             m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed", chunks=4, packed=True, variant="sketch"),
        # The headline configuration: 2^30 particles resident in HBM, w = 2^24, top 10^4.
        dict(name="scale_step", kind="step", n=1 << 30, L=1000.0, G=4000, d=5, w=1 << 24, k=10_000,
             halos=1 << 20, m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed", chunks=1, packed=False,
             variant="sketch", wait=True),
        # 64 sub-volumes of 2^14 .. 2^22 particles at once, widths that follow their sizes.
        dict(name="batch_step", kind="batch", count=64, lo=14, hi=22, L=100.0, G=1000, d=5, f_bg=0.9),
        # The learned router before a narrower sketch of the same total memory.
        dict(name="routed_step", kind="routed", n=1 << 27, L=1000.0, G=4000, d=5, w=1 << 22, k=10_000,
             halos=1 << 18, m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed"),
        # Counts of a halo catalogue's cells read back from the sketch.
        dict(name="query", kind="query", n=1 << 24, L=1000.0, G=4000, d=5, w=1 << 24, m=1_000_003,
             halos=1 << 15, m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed", variant="sketch"),
        # The paper's full search over every cell of the mesh, occupied or not.
        dict(name="full_search", kind="search", n=1 << 26, L=500.0, G=2000, d=5, w=1 << 22, k=10_000,
             halos=1 << 16, m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed"),
        # The paper's two-layer search with super-cells of 1000 keys.
        dict(name="layered_search", kind="layers", n=1 << 26, L=500.0, G=2000, d=5, w=1 << 22, k=10_000,
             group=1000, halos=1 << 16, m_lo=50.0, m_hi=1e6, f_bg=0.3, order="mixed"),
        # Some minibatches of the router's training (forward, backward, Adam).
        dict(name="router_train", kind="train", rows=4096, steps=8, lr=2e-3),
    ]


def _log_size(rng, lo, hi):
    """A size spread over the logarithm of [2^lo, 2^hi], odd more often than not."""
    n = int(2.0 ** rng.uniform(lo, hi))
    return n | 1 if rng.random() < 0.7 else n


def _mesh(rng):
    # the three floor paths: G / L a power of two, exact in binary64, and general
    return rng.choice([(1000.0, 4000), (500.0, 2000), (128.0, 1024), (100.0, 1000), (100.0, 250), (250.0, 768),
                       (70.0, 511)])


def _width(rng, lo, hi):
    if rng.random() < 0.6:
        return 1 << rng.randint(lo, hi)
    return _log_size(rng, lo, hi)


def draw(rng):
    kind = rng.choices(["update", "step", "batch", "routed", "query", "search", "layers", "train"],
                       [5, 6, 2, 1, 2, 1, 1, 1])[0]
    L, G = _mesh(rng)
    halo = dict(m_lo=rng.choice([50.0, 100.0]), m_hi=rng.choice([1e4, 1e5, 1e6]), f_bg=round(rng.uniform(0.1, 0.9), 2),
                order=rng.choice(["mixed", "mixed", "halo"]))
    if kind in ("update", "step"):
        n = _log_size(rng, 10, 27)
        c = dict(kind=kind, n=n, L=L, G=G, d=rng.choice([3, 4, 5, 5, 5, 5, 6, 8]),
                 w=_width(rng, max(12, n.bit_length() - 8), 23),
                 halos=max(1, n >> rng.randint(9, 14)), chunks=rng.choice([1, 1, 1, 2, 5]),
                 packed=rng.random() < 0.2, variant=rng.choice(["sketch", "sketch", "sketch", "min"]), **halo)
        if kind == "step":
            c.update(k=max(1, min(10_000, n >> rng.randint(7, 11))), wait=rng.random() < 0.6)
        return c
    if kind == "batch":
        lo = rng.randint(12, 15)
        return dict(kind=kind, count=rng.randint(2, 64), lo=lo, hi=lo + rng.randint(2, 6), L=100.0, G=1000, d=5,
                    f_bg=halo["f_bg"])
    if kind == "routed":
        n = _log_size(rng, 21, 26)
        return dict(kind=kind, n=n, L=500.0, G=2000, d=5, w=1 << rng.randint(19, 22), k=rng.choice([500, 1000, 2000]),
                    halos=n >> 9, **halo)
    if kind == "query":
        return dict(kind=kind, n=_log_size(rng, 16, 23), L=L, G=G, d=rng.choice([3, 5, 5, 8]), w=_width(rng, 14, 24),
                    m=_log_size(rng, 8, 23), halos=1000, variant=rng.choice(["sketch", "sketch", "min"]), **halo)
    if kind in ("search", "layers"):
        G = rng.choice([255, 500, 700, 1000, 1500])
        c = dict(kind=kind, n=_log_size(rng, 20, 24), L=G / 4.0, G=G, d=5, w=_width(rng, 18, 22),
                 k=rng.choice([100, 500, 1000]), halos=4000, **halo)
        if kind == "layers":
            c["group"] = rng.choice([64, 1000, 1000, 777])
        return c
    return dict(kind="train", rows=_log_size(rng, 8, 12), steps=rng.randint(1, 12), lr=rng.choice([1e-3, 2e-3]))


# ------------------------------------------------------------------ inputs

def _stream(c, seed):
    """float32 [n][3] positions in [0, L)."""
    g = torch.Generator(device="cuda").manual_seed(1 + 7919 * seed)

    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)

    n, L, h = c["n"], c["L"], c["halos"]
    e = 1.0 - 1.9
    a, b = c["m_lo"] ** e, c["m_hi"] ** e
    mass = (a + rand(h) * (b - a)) ** (1.0 / e)
    centre = rand(h, 3) * L
    cum = torch.cumsum(mass, 0) / mass.sum()
    pos = torch.empty((n, 3), dtype=torch.float32, device="cuda")
    for at in range(0, n, DRAW_CHUNK):
        m = min(DRAW_CHUNK, n - at)
        u = rand(m)
        if c["order"] == "halo":   # this piece of the snapshot, halo by halo
            u = (torch.sort(u).values * m + at) / n
        j = torch.searchsorted(cum, u).clamp_(max=h - 1)
        del u
        r = SCALE_RADIUS / torch.sqrt((rand(m) * 1.01 ** -1.5) ** (-2.0 / 3.0) - 1.0)
        ct = 2.0 * rand(m) - 1.0
        st = torch.sqrt(torch.clamp(1.0 - ct * ct, min=0.0))
        phi = 2.0 * math.pi * rand(m)
        bg = torch.rand(m, generator=g, device="cuda") < c["f_bg"]
        for axis, off in enumerate((r * st * torch.cos(phi), r * st * torch.sin(phi), r * ct)):
            x = torch.where(bg, rand(m) * L, centre[:, axis][j] + off)
            x = torch.remainder(x, L).float()
            pos[at:at + m, axis] = torch.where(x >= L, torch.zeros_like(x), x)
    return pos


def _variant(c):
    return COUNT_MIN if c.get("variant") == "min" else SKETCH


def _candidates(c):
    """Room for every cell of a small stream; the library's default, or twice that, for a large one."""
    if c["n"] <= 1 << 18:
        return max(1 << 14, 8 * c["k"], c["n"])
    return csk.CSK_DEFAULT_CANDIDATES if c["n"] <= 1 << 26 else 2 * csk.CSK_DEFAULT_CANDIDATES


def _pieces(stream, chunks):
    step = -(-stream.shape[0] // chunks)
    return [stream[i:i + step] for i in range(0, stream.shape[0], step)]


def _add(s, pieces, packed, delta, L):
    for p in pieces:
        (s.update_packed if packed else s.update)(p, delta, L)


def _collect(s, pieces, packed, delta, L, theta):
    for p in pieces:
        (s.collect_packed if packed else s.collect)(p, delta, L, theta)


def _calibrate(k, attempt, top=1 << 22):
    """The threshold a program settles on before its steps: halved until k cells pass, and the
    last one that the candidate set held when there is no room for as many as pass."""
    theta = top
    while theta > 0:
        try:
            if attempt(theta) >= k:
                return theta
        except csk.CskError as e:
            if e.code != csk.CSK_E_CAPACITY:
                raise
            return 2 * theta
        theta //= 2
    return csk.INT32_MIN


def prepare(case, seed):
    c = case
    if c["kind"] == "train":
        return _prepare_train(c, seed)
    if c["kind"] == "batch":
        return _prepare_batch(c, seed)
    st = dict(case=c, L=c["L"], delta=c["L"] / c["G"])
    delta, L = st["delta"], c["L"]
    pos = _stream(c, seed)
    if c["kind"] == "routed":
        return _prepare_routed(st, pos, seed)
    stream = csk.pack_positions(pos, L) if c.get("packed") else pos
    if c["kind"] in ("update", "step"):
        st["pieces"] = _pieces(stream, c["chunks"])
        st["sketch"] = s = csk.Sketch(c["d"], c["w"], 1, _variant(c), _candidates(c) if c["kind"] == "step" else 1 << 14)
        if c["kind"] == "step":
            def attempt(theta):
                s.clear_candidates()
                _collect(s, st["pieces"], c["packed"], delta, L, theta)
                return s.topk(c["k"])[0].numel()
            _add(s, st["pieces"], c["packed"], delta, L)
            st["theta"] = _calibrate(c["k"], attempt)
            st["keys"] = torch.zeros(c["k"], dtype=torch.int64, device="cuda")
            st["est"] = torch.zeros(c["k"], dtype=torch.int32, device="cuda")
            st["out"] = torch.zeros(2, dtype=torch.int32, device="cuda")
        return st
    if c["kind"] == "query":
        st["sketch"] = s = csk.Sketch(c["d"], c["w"], 1, _variant(c), 1 << 14)
        s.update(pos, delta, L)
        # cells of the stream, and as many that may be empty
        g = torch.Generator(device="cuda").manual_seed(5 + 104_729 * seed)
        half = c["m"] // 2
        at = torch.randint(c["n"], (half,), generator=g, device="cuda")
        seen = csk.cell_keys(pos[at].contiguous(), delta, L)
        other = torch.randint(c["G"] ** 3, (c["m"] - half,), generator=g, device="cuda")
        st["keys"] = torch.cat([seen, other])
        return st
    # search and layers: the counters of the stream, and thresholds that let enough pass
    st["sketch"] = s = csk.Sketch(c["d"], c["w"], 1, max_candidates=1 << 20)
    s.update(pos, delta, L)

    def attempt(theta):
        s.clear_candidates()
        s.collect(pos, delta, L, theta)
        return s.topk(c["k"])[0].numel()
    st["theta"] = _calibrate(c["k"], attempt)
    if c["kind"] == "layers":
        st["coarse"] = q = csk.Sketch(c["d"], c["w"], 2, max_candidates=1 << 20, group=c["group"])
        q.update(pos, delta, L)

        def attempt1(theta):
            q.clear_candidates()
            q.collect_dictionary(delta, L, theta)
            return q.topk(min(3 * c["k"], c["G"] ** 3 // c["group"] // 2))[0].numel()
        st["theta1"] = _calibrate(min(3 * c["k"], c["G"] ** 3 // c["group"] // 2), attempt1)
    return st


def _sub_volumes(c, seed):
    rng = np.random.default_rng(11 + seed)
    out = []
    for i in range(c["count"]):
        u = float(rng.random()) if c["count"] > 2 else float(i)
        n = int(2.0 ** (c["lo"] + (c["hi"] - c["lo"]) * u))
        w = 1 << (14 + int(round(6.0 * u)))
        out.append(dict(n=n, L=c["L"], G=c["G"], d=c["d"], w=w, k=max(1, w // 100), halos=max(1, n >> 12),
                        m_lo=100.0, m_hi=1e4, f_bg=c["f_bg"], order="mixed"))
    return out


def _prepare_batch(c, seed):
    vols = _sub_volumes(c, 0)   # the shapes stay; the particles change with the seed
    delta, L = c["L"] / c["G"], c["L"]
    pos = [_stream(v, seed * 64 + i) for i, v in enumerate(vols)]
    sk = [csk.Sketch(v["d"], v["w"], 1, max_candidates=max(1 << 14, 8 * v["k"], min(v["n"], 1 << 18))) for v in vols]
    b = csk.Batch(sk, [v["n"] for v in vols], delta, L, 2048)
    ks = [v["k"] for v in vols]
    keys, est = (torch.zeros(sum(ks), dtype=t, device="cuda") for t in (torch.int64, torch.int32))
    outs = torch.zeros((len(vols), 2), dtype=torch.int32, device="cuda")
    b.update(pos)
    thetas = []
    for s, p, k in zip(sk, pos, ks):
        def attempt(theta):
            s.clear_candidates()
            s.collect(p, delta, L, theta)
            return s.topk(k)[0].numel()
        thetas.append(_calibrate(k, attempt, 1 << 12))
    return dict(case=c, batch=b, pos=pos, ks=ks, thetas=thetas, keys=keys, est=est, outs=outs,
                key_list=list(keys.split(ks)), est_list=list(est.split(ks)), out_list=list(outs.unbind(0)))


def _prepare_routed(st, pos, seed):
    c = st["case"]
    r = Router(st["delta"], c["L"], delta_c=4 * st["delta"])
    # a model that has learned to follow the cell's own count, with some noise on every weight
    p = np.random.default_rng(seed).normal(0, 0.02, csk.N_PARAMS).astype(np.float32)
    p[0 * 32 + 13] = 1.0                    # W1: the cell itself
    p[64 * 32 + 64 + 0] = 1.0               # W2
    p[64 * 32 + 64 + 64 * 64 + 64] = 1.0    # w3
    r.mlp.set_params(p)
    rest = csk.Sketch(c["d"], rest_width(c["w"], c["d"], r.table_slots), 1, max_candidates=1 << 21)
    step = RoutedStep(r, rest, c["k"])

    def attempt(theta):
        step.run(pos, theta)
        keys, est, partial = step.result()
        # a table key is always a candidate, so the k-th value decides
        return c["k"] if keys.numel() == c["k"] and int(est[-1]) >= theta else 0
    st.update(pos=pos, step=step, theta=_calibrate(c["k"], attempt))
    return st


def _prepare_train(c, seed):
    g = torch.Generator(device="cuda").manual_seed(3 + 15_485_863 * seed)
    n = c["rows"] * c["steps"]
    # log-counts of a clustered 1 % sample: mostly small, the centre cell the largest
    x = torch.zeros((n, csk.FEAT), dtype=torch.float32, device="cuda")
    level = -torch.log1p(-torch.rand((n, 1), generator=g, device="cuda")) * 1.5
    x[:, :27] = torch.log1p(torch.floor(level * torch.rand((n, 27), generator=g, device="cuda") * 4.0))
    y = ((x[:, 13] + 0.2 * x[:, :27].mean(1)) > 1.9).float()
    m = csk.MLP(seed=1 + seed % 1000, max_batch=c["rows"])
    return dict(case=c, mlp=m, init=m.params(), x=list(x.split(c["rows"])), y=list(y.split(c["rows"])),
                loss=torch.zeros((c["steps"], 1), dtype=torch.float32, device="cuda"))


# ------------------------------------------------------------------ one pass

def run(state):
    st, c = state, state["case"]
    kind = c["kind"]
    if kind == "batch":
        b = st["batch"]
        b.reset()
        b.update(st["pos"])
        b.collect(st["pos"], st["thetas"])
        b.topk(st["ks"], st["key_list"], st["est_list"], st["out_list"])
        return st["keys"], st["est"], st["outs"]
    if kind == "train":
        m = st["mlp"]
        m.set_params(st["init"])
        for x, y, loss in zip(st["x"], st["y"], st["loss"]):
            m.train_step(x, y, c["lr"], loss)
        return m.params(), st["loss"]
    delta, L = st["delta"], st["L"]
    if kind == "routed":
        step = st["step"]
        step.run(st["pos"], st["theta"])
        return step.keys, step.est, step.out
    s = st["sketch"]
    if kind == "query":
        return s.query(st["keys"])
    if kind == "search":
        s.clear_candidates()
        s.collect_dictionary(delta, L, st["theta"])
        return s.topk(c["k"])
    if kind == "layers":
        q = st["coarse"]
        q.clear_candidates()
        q.collect_dictionary(delta, L, st["theta1"])
        s.clear_candidates()
        s.collect_children(q, st["theta"])
        return s.topk(c["k"])
    s.reset()
    _add(s, st["pieces"], c["packed"], delta, L)
    if kind == "update":
        return s.counters()
    _collect(s, st["pieces"], c["packed"], delta, L, st["theta"])
    if c["wait"]:
        return s.topk(c["k"])
    s.topk_async(c["k"], st["keys"], st["est"], st["out"])
    return st["keys"], st["est"], st["out"]


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Positions and counters once each, the results once; hashing and comparing as operations
    (a handful per particle and row)."""
    c, kind = case, case["kind"]
    if kind == "train":
        p = csk.N_PARAMS
        return {"bytes": c["steps"] * c["rows"] * (32 + 1) * 4 + 2 * p * 4, "flops": c["steps"] * c["rows"] * 6 * (32 * 64 + 64 * 64 + 64)}
    if kind == "batch":
        vols = _sub_volumes(c, 0)
        return {"bytes": sum(12 * v["n"] + 4 * v["d"] * v["w"] + 12 * v["k"] for v in vols),
                "flops": sum(10 * v["d"] * v["n"] for v in vols)}
    table = 4 * c["d"] * c["w"]
    if kind == "query":
        # a counter is a transaction of its own in a table that no cache holds
        return {"bytes": c["m"] * (8 + 4) + min(table, 4 * c["d"] * c["m"]), "flops": 10 * c["d"] * c["m"]}
    if kind in ("search", "layers"):
        cells = c["G"] ** 3
        keys = cells if kind == "search" else cells // c["group"] + 3 * c["k"] * c["group"]
        return {"bytes": table * (1 if kind == "search" else 2) + 12 * c["k"], "flops": 10 * c["d"] * keys}
    b = (8 if c.get("packed") else 12) * c["n"] + table + 12 * c.get("k", 0)
    return {"bytes": b, "flops": 10 * c["d"] * c["n"]}


# ------------------------------------------------------------------ the same results in plain torch

def _tables(d, seed):
    """T[row][byte][value], two 32-bit words per SplitMix64 draw, low half first."""
    k = np.arange(1, d * 6 * 128 + 1, dtype=np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + k * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    t = np.stack([z & np.uint64(0xFFFFFFFF), z >> np.uint64(32)], 1).reshape(d, 6, 256)
    return torch.from_numpy(t.astype(np.int64)).cuda()


def _cell_keys(pos, L, G, packed):
    key = torch.zeros(pos.shape[0], dtype=torch.int64, device="cuda")
    for axis in range(3):
        g = 1 << 21 if packed else G
        t = pos[:, axis].double() * g        # exact, and so is i * L below
        i = torch.floor(t / L)
        i -= (t < i * L).double()
        i += (t >= (i + 1) * L).double()
        i = torch.remainder(i, g).long()
        key = key * G + ((i * G) >> 21 if packed else i)
    return key


def _rows(keys, T, w, cm):
    """(bucket, sign) of every row."""
    for t in T:
        h = t[0][keys & 255]
        for b in range(1, 6):
            h = h ^ t[b][(keys >> (8 * b)) & 255]
        yield ((h & 0x7FFFFFFF) * w) >> 31, torch.ones_like(h) if cm else 1 - 2 * (h >> 31)


def _counters(c, pos, T):
    M = torch.zeros((c["d"], c["w"]), dtype=torch.int64, device="cuda")
    for p in pos.split(DRAW_CHUNK):
        keys = _cell_keys(p, c["L"], c["G"], c.get("packed"))
        for r, (b, sg) in enumerate(_rows(keys, T, c["w"], c.get("variant") == "min")):
            M[r].index_add_(0, b, sg)
    return M


def _estimates(keys, M, T, w, cm):
    v = torch.stack([M[r][b] * sg for r, (b, sg) in enumerate(_rows(keys, T, w, cm))])
    return v.amin(0) if cm else torch.sort(v, 0).values[(len(T) - 1) // 2]


def _best(keys, est, k):
    if keys.numel() > 4 * k:                     # everything at or above the k-th estimate
        kth = torch.topk(est, k).values[-1]
        keys, est = keys[est >= kth], est[est >= kth]
    at = torch.argsort(keys)
    keys, est = keys[at], est[at]
    at = torch.argsort(-est, stable=True)[:k]
    return keys[at], est[at]


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "train":
        return _exact_train(c, seed)
    if kind == "batch":
        keys, est, outs = [], [], []
        for i, v in enumerate(_sub_volumes(c, 0)):
            a, b = _exact_step(v, seed * 64 + i)
            keys.append(torch.nn.functional.pad(a, (0, v["k"] - a.numel())))
            est.append(torch.nn.functional.pad(b, (0, v["k"] - b.numel())))
            outs.append(None)
        return torch.cat(keys), torch.cat(est), None
    if kind == "routed" or kind == "layers":
        return None              # what is admitted, and what the first layer lets through, decide
    if kind == "update":
        return _counters(c, _stream(c, seed), _tables(c["d"], 1)).to(torch.int32)
    if kind == "step":
        keys, est = _exact_step(c, seed)
        if not c["wait"]:        # buffers of k entries
            keys, est = (torch.nn.functional.pad(t, (0, c["k"] - t.numel())) for t in (keys, est))
        return keys, est.to(torch.int32), None
    pos = _stream(c, seed)
    T = _tables(c["d"], 1)
    M = _counters(c, pos, T)
    if kind == "query":
        g = torch.Generator(device="cuda").manual_seed(5 + 104_729 * seed)
        half = c["m"] // 2
        at = torch.randint(c["n"], (half,), generator=g, device="cuda")
        seen = _cell_keys(pos[at], c["L"], c["G"], False)
        other = torch.randint(c["G"] ** 3, (c["m"] - half,), generator=g, device="cuda")
        return _estimates(torch.cat([seen, other]), M, T, c["w"], c["variant"] == "min").to(torch.int32)
    best = None
    for lo in range(0, c["G"] ** 3, DRAW_CHUNK):
        keys = torch.arange(lo, min(lo + DRAW_CHUNK, c["G"] ** 3), device="cuda")
        est = _estimates(keys, M, T, c["w"], False)
        if best is not None:
            go = est >= best[1][-1]
            keys, est = torch.cat([best[0], keys[go]]), torch.cat([best[1], est[go]])
        best = _best(keys, est, c["k"])
    return best[0], best[1].to(torch.int32), None


def _exact_step(c, seed):
    pos = _stream(c, seed)
    T = _tables(c["d"], 1)
    M = _counters(c, pos, T)
    keys = torch.cat([_cell_keys(p, c["L"], c["G"], c.get("packed")) for p in pos.split(DRAW_CHUNK)])
    del pos
    keys = torch.unique(keys)
    est = torch.cat([_estimates(p, M, T, c["w"], c.get("variant") == "min") for p in keys.split(DRAW_CHUNK)])
    return _best(keys, est, c["k"])


def _exact_train(c, seed):
    st = _prepare_train(c, seed)
    p = torch.from_numpy(st["init"]).cuda().double()
    at = np.cumsum([0, 64 * 32, 64, 64 * 64, 64, 64, 1])
    mom, var = torch.zeros_like(p), torch.zeros_like(p)
    losses = []
    for t, (x, y) in enumerate(zip(st["x"], st["y"]), 1):
        q = p.clone().requires_grad_(True)
        W1, b1, W2, b2, w3, b3 = (q[a:b] for a, b in zip(at[:-1], at[1:]))
        h = torch.relu(x.double() @ W1.view(64, 32).T + b1)
        h = torch.relu(h @ W2.view(64, 64).T + b2)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(h @ w3 + b3, y.double())
        g, = torch.autograd.grad(loss, q)
        losses.append(loss.detach())
        mom, var = 0.9 * mom + 0.1 * g, 0.999 * var + 0.001 * g * g
        p = p - c["lr"] * (mom / (1 - 0.9 ** t)) / (torch.sqrt(var / (1 - 0.999 ** t)) + 1e-8)
    return p, torch.stack(losses).view(-1, 1)
