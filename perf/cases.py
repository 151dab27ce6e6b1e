"""What a user of the library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points on inputs made from a seed
on the GPU: walks (the uniform, dense and tiny workloads of `trajgen`, with
regular or per-walk start times) or particles of two approaching Plummer
spheres (its merger workload).  Record order inside a result is unspecified,
so a search's records are read the way a consumer that goes through them entry
by entry does: ordered by (e_seg, q_seg); trajectory-level results come ordered
from the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1410_2698_amd as tds

FIELDS = ("xs", "ys", "zs", "ts", "xe", "ye", "ze", "te")
INF = math.inf

WALK = {"data": "walk", "step": "uniform5", "box": 1000.0, "walls": False, "start": 0.0}
DENSE = {"data": "walk", "step": "normal", "box": 50.0, "walls": True, "start": 0.0}
TINY = {"data": "walk", "step": "normal", "box": 100.0, "walls": False, "start": 0.0}
MERGER = {"data": "merger"}


def listed():
    return [
        # one trajectory asked of a resident database, host memory in and out:
        # the smallest call, where latency counts
        dict(WALK, name="request", path="request", traj=2500, pts=401, q_traj=1, q_pts=202, d=25.0),
        # requests that arrived together, each a trajectory with its own
        # distance and window, through the captured batcher
        dict(WALK, name="batcher", path="batcher", traj=2500, pts=401, requests=32),
        # the small worked configuration: launches and latency
        dict(TINY, name="tiny", path="search", traj=2000, pts=50, q_traj=100, q_pts=50, d=5.0,
             precision="fp32", window=False),
        # odd sizes and irregular start times, searched in a window
        dict(WALK, name="ragged", path="search", traj=1237, pts=302, q_traj=83, q_pts=173, d=17.0,
             start=100.0, precision="fp32", window=True),
        # the uniform database asked at three distances in one batch
        dict(WALK, name="uniform_batch", path="batch", traj=2500, pts=401, q_traj=500, q_pts=401,
             d=1.0, d2=5.0, d3=25.0),
        # the dense box: many records per query
        dict(DENSE, name="dense", path="search", traj=10000, pts=101, q_traj=1000, q_pts=101, d=2.0,
             precision="fp32", window=False),
        # the plain form, every candidate pair in FP64
        dict(WALK, name="uniform_fp64", path="search", traj=2500, pts=401, q_traj=50, q_pts=401,
             d=5.0, precision="fp64", window=False),
        # stars close to the query stars at a small distance: few records from
        # a clustered database
        dict(MERGER, name="merger_near", path="search", traj=200000, pts=20, q_traj=2000, q_pts=20,
             d=0.1, precision="fp32", window=False),
        # when and which stars pass within the distance of the query stars:
        # the largest search and its trajectory-level result
        dict(MERGER, name="merger", path="merge", traj=200000, pts=20, q_traj=2000, q_pts=20, d=0.5),
        # every trajectory against every other, trajectory-level result
        dict(WALK, name="self_join", path="join", traj=2500, pts=401, d=25.0),
        # the index of a new database
        dict(WALK, name="build", path="build", traj=2503, pts=400, bins=0),
        # the fixed spatial grid
        dict(WALK, name="grid", path="grid", traj=2500, pts=401, q_traj=500, q_pts=401, d=5.0, cells=50),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


SCALE = {1000.0: 25.0, 50.0: 2.0, 100.0: 6.0}  # largest distance asked in each box


def draw(rng):
    while True:  # cases that have something to find
        c = _draw(rng)
        if c["path"] == "build" or _expected(c) >= 60:
            return c


def _draw(rng):
    path = rng.choice(["request", "batcher", "search", "search", "search", "batch", "merge", "join",
                       "build", "grid"])
    if path == "merge" or (path == "search" and rng.random() < 0.3):
        c = dict(MERGER, path=path, traj=2 * _log(rng, 5000, 100000), pts=rng.randint(5, 20),
                 q_traj=2 * _log(rng, 50, 1000), d=round(rng.uniform(0.02, 0.12 if path == "search" else 0.5), 4))
        c["q_pts"] = c["pts"]
        if path == "search":
            c.update(precision="fp32", window=rng.random() < 0.3)
        return c
    kind = rng.choice([WALK, WALK, DENSE, TINY])
    pts = rng.randint(20, 401)
    traj = max(20, min(10000, _log(rng, 20000, 1000000) // pts))
    c = dict(kind, path=path, traj=traj, pts=pts, start=rng.choice([0.0, 0.0, 100.0]))
    if path == "build":
        c["bins"] = pts + rng.randint(0, 100)
        return c
    if path == "batcher":
        return dict(c, requests=rng.randint(1, 64), start=0.0)
    c["d"] = round(rng.uniform(0.04, 1.0) * SCALE[kind["box"]], 3)
    if path == "join":
        c["d"] = round(c["d"] / (1.0 if kind is WALK else 4.0), 3)
        return c
    c["q_pts"] = rng.randint(6, pts)
    if path == "request":
        c["q_traj"] = 1
        return c
    c["q_traj"] = min(1000, max(1, _log(rng, 200, 200000) // c["q_pts"]))
    if path == "batch":
        c.update(d2=round(c["d"] * 0.3, 3), d3=round(c["d"] * 0.7, 3))
    elif path == "grid":
        c["cells"] = rng.choice([20, 50])
    else:
        fp64 = rng.random() < 0.2
        if fp64:
            c["q_traj"] = max(1, c["q_traj"] // 10)
        c.update(precision="fp64" if fp64 else "fp32", window=rng.random() < 0.3)
    return c


# ------------------------------------------------------------------ sizes

def _queries(c):
    """Query segments of one pass."""
    if c["path"] == "join":
        return c["traj"] * (c["pts"] - 1)
    if c["path"] == "batcher":
        return c["requests"] * (c["pts"] + 4) // 2
    return c["q_traj"] * (c["q_pts"] - 1)


def _pairs_in_time(c):
    """About how many pairs of segments overlap in time."""
    step = 2.0 if c.get("start") else 1.0
    share = 0.5 if c["path"] in ("join", "batcher") else 0.6 if c.get("window") else 1.0
    return share * _queries(c) * c["traj"] * min(1.0, step * (c["pts"] - 1) / (c["pts"] - 1 + c.get("start", 0.0)))


def _near(c, d):
    """About what part of them comes within d."""
    if c["data"] == "merger":
        return min(1.0, 0.023 * (d / 0.5) ** 2.2)
    return min(1.0, 4.19 * (d + (0.3 if c["step"] == "normal" else 2.0)) ** 3 / c["box"] ** 3)


def _distances(c):
    return [c[k] for k in ("d", "d2", "d3") if k in c] or [0.6 * SCALE[c["box"]]]


def _expected(c):
    """About how many records a pass finds."""
    return _pairs_in_time(c) * sum(_near(c, d) for d in _distances(c))


def _room(c):
    """Records that the case's result arrays hold, the same for every seed."""
    return int((1.4 if c["data"] == "merger" else 2.0) * _expected(c)) + 8192


def _slices(c):
    """(offset, records) of each distance's part of the result array."""
    near = [_near(c, d) for d in _distances(c)]
    size = [2048 + int((_room(c) - 2048 * len(near)) * x / sum(near)) for x in near]
    return [(sum(size[:i]), n) for i, n in enumerate(size)]


def work(case):
    c = case
    n = c["traj"] * (c["pts"] - 1)
    if c["path"] == "build":
        # end points, times and ids in; a 64-byte record, two ids and the order out
        return {"bytes": n * (68 + 72 + 4), "flops": 6 * n}
    results = _expected(c)
    flops = 95.0 * results + (74.0 * _pairs_in_time(c) if c.get("precision") == "fp64" else 0.0)
    # the entries of the times that the queries cover: end points, times and id
    read = 68 * min(n, 2 * c["traj"] * c.get("q_pts", c["pts"])) + 68 * _queries(c) * len(_distances(c))
    merged = 24 * results if c["path"] in ("merge", "join") else 0
    return {"bytes": read + 32 * results + merged, "flops": flops}


# ------------------------------------------------------------------ inputs

def _segments(pos, times):
    """Polylines (n, pts, 3) at times (n, pts) -> segments, trajectory-major."""
    n, pts, _ = pos.shape
    s = {k: pos[:, :-1, a].reshape(-1).contiguous() for a, k in enumerate(("xs", "ys", "zs"))}
    s.update({k: pos[:, 1:, a].reshape(-1).contiguous() for a, k in enumerate(("xe", "ye", "ze"))})
    s["ts"], s["te"] = times[:, :-1].reshape(-1).contiguous(), times[:, 1:].reshape(-1).contiguous()
    s["traj"] = torch.arange(n, dtype=torch.int32, device="cuda").repeat_interleave(pts - 1)
    return s


def _walks(c, n, pts, g, first=0.0):
    """Random walks of the case's process with unit steps from time `first`,
    plus a start of its own in [0, start) for each walk."""
    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)
    if c["step"] == "normal":
        step = torch.randn(n, pts - 1, 3, generator=g, device="cuda", dtype=torch.float64)
    else:
        step = rand(n, pts - 1, 3) * 10.0 - 5.0
    p = torch.cat([rand(n, 1, 3) * c["box"], step], dim=1).cumsum(1)
    if c["walls"]:  # mirrored at the walls of the box
        p = p.remainder(2.0 * c["box"])
        p = torch.where(p > c["box"], 2.0 * c["box"] - p, p)
    t = first + torch.arange(pts, device="cuda", dtype=torch.float64).expand(n, pts)
    if c["start"]:
        t = t + rand(n, 1) * c["start"]
    return _segments(p, t)


def _merger(c, counts, g):
    """Particles of two Plummer spheres (G = M = a = 1, 6 apart, impact
    parameter 1, 1.5 times the parabolic speed), integrated by leapfrog in the
    field of the two centres; snapshots every 0.5.  One set of segments for
    each number of particles in `counts`."""
    n, pts = sum(counts), c["pts"]

    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)

    def directions():
        z, a = rand(n) * 2.0 - 1.0, rand(n) * (2.0 * math.pi)
        s = (1.0 - z * z).sqrt()
        return torch.stack([s * a.cos(), s * a.sin(), z])
    m = (rand(n) * (1000.0 / 101.0 ** 1.5)).clamp_min(1e-12)
    r = 1.0 / (m ** (-2.0 / 3.0) - 1.0).sqrt()
    q, todo = torch.empty_like(r), torch.arange(n, device="cuda")
    for _ in range(64):  # speeds by rejection; a quarter is accepted each time
        x, y = rand(todo.numel()), rand(todo.numel()) * 0.1
        ok = y < x * x * (1.0 - x * x) ** 3.5
        q[todo] = x
        todo = todo[~ok]
        if todo.numel() == 0:
            break
    speed = q * math.sqrt(2.0) * (1.0 + r * r) ** -0.25
    x, v = directions() * r, directions() * speed
    half = torch.arange(n, device="cuda") % 2 == 0
    v0 = 1.5 * math.sqrt(4.0 / 6.0) / 2.0
    centre = [[-3.0, -0.5, 0.0], [3.0, 0.5, 0.0]]
    cvel = [[v0, 0.0, 0.0], [-v0, 0.0, 0.0]]
    for a in range(3):
        x[a] += torch.where(half, centre[0][a], centre[1][a])
        v[a] += torch.where(half, cvel[0][a], cvel[1][a])

    def field(centre):
        f = torch.zeros_like(x)
        for k in range(2):
            d = x - torch.tensor(centre[k], dtype=torch.float64).to("cuda", non_blocking=True)[:, None]
            r2 = d.square().sum(0) + 1.0
            f -= d * r2.pow(-1.5)
        return f

    def pull(centre):
        d = [centre[0][a] - centre[1][a] for a in range(3)]
        f = (sum(t * t for t in d) + 1.0) ** -1.5
        return [[-t * f for t in d], [t * f for t in d]]
    per, dt = 25, 0.02
    f, cf = field(centre), pull(centre)
    snaps = [x.t().clone()]
    for _ in range(pts - 1):
        for _ in range(per):
            v.add_(f, alpha=0.5 * dt)
            x.add_(v, alpha=dt)
            cvel = [[cvel[k][a] + 0.5 * dt * cf[k][a] for a in range(3)] for k in range(2)]
            centre = [[centre[k][a] + dt * cvel[k][a] for a in range(3)] for k in range(2)]
            f, cf = field(centre), pull(centre)
            v.add_(f, alpha=0.5 * dt)
            cvel = [[cvel[k][a] + 0.5 * dt * cf[k][a] for a in range(3)] for k in range(2)]
        snaps.append(x.t().clone())
    pos = torch.stack(snaps, dim=1)
    t = 0.5 * torch.arange(pts, device="cuda", dtype=torch.float64).expand(n, pts)
    out, at = [], 0
    for k in counts:
        out.append(_segments(pos[at:at + k], t[at:at + k]))
        at += k
    return out


def _requests(c, g):
    """Requests over the walks' database: a walk of 5 segments up to the whole
    length each, a window inside it and a distance of its own; host memory."""
    u = torch.rand(c["requests"], 5, generator=g, device="cuda", dtype=torch.float64).cpu().numpy()
    most = c["pts"] - 1
    out = []
    for a in u:
        n = min(5, most) + int(a[0] * (most - min(5, most) + 1))
        first = int(a[1] * (most - n + 1))
        s = {k: v.cpu().numpy() for k, v in _walks(c, 1, n + 1, g, float(first)).items()}
        s["traj"] = s["traj"].astype(np.uint32)
        t0 = first + a[2] * n
        t1 = first + n - a[3] * 0.999 * (first + n - t0)
        out.append((s, (0.04 + 0.96 * a[4]) * SCALE[c["box"]], float(t0), float(t1)))
    return out


def _inputs(c, seed):
    """(database, queries): the case's segments on the GPU, a function of the
    seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if c["data"] == "merger":
        return tuple(_merger(c, [c["traj"], c["q_traj"]], g))
    D = _walks(c, c["traj"], c["pts"], g)
    if c["path"] == "batcher":
        return D, _requests(c, g)
    if "q_traj" not in c:
        return D, None
    first = float((c["pts"] - c["q_pts"]) // 2)
    return D, _walks(c, c["q_traj"], c["q_pts"], g, first)


def _window(c):
    """The search window: everything, or the middle 60 % of the time covered."""
    if not c.get("window"):
        return -INF, INF
    span = (c["pts"] - 1) * (0.5 if c["data"] == "merger" else 1.0) + c.get("start", 0.0)
    return 0.2 * span, 0.8 * span


def _buffer(records, words=4):
    return torch.empty(records, words, dtype=torch.int64, device="cuda")


def prepare(case, seed):
    c = case
    D, Q = _inputs(c, seed)
    s = {"case": c, "D": D, "Q": Q}
    if c["path"] == "build":
        return s
    idx, room = tds.Index(D), _room(c)
    s.update(index=idx, window=_window(c), room=room)
    if c["path"] == "request":
        s["Q"] = {k: v.cpu().numpy() for k, v in Q.items()}
        s["Q"]["traj"] = s["Q"]["traj"].astype(np.uint32)
        return s
    if c["path"] == "batcher":
        n = sum(len(r[0]["xs"]) for r in Q)
        s["batcher"] = tds.Batcher(idx, max(n, 64), len(Q), len(Q) * 8192)
        return s
    s["out"] = _buffer(room)
    if c["path"] in ("merge", "join"):
        s["merged"] = _buffer(room, 3)
        return s
    s["sorted"] = _buffer(room)
    if c["path"] == "batch":
        nq, (t0, t1) = Q["xs"].numel(), s["window"]
        s["Q"] = {k: torch.cat([v, v, v]) for k, v in Q.items()}
        s["requests"] = [(i * nq, nq, d, t0, t1, a, b) for i, (d, (a, b)) in enumerate(zip(_distances(c), _slices(c)))]
    elif c["path"] == "grid":
        s["grid"] = tds.FSG(idx, c["cells"], c["cells"], c["cells"])
    return s


# ------------------------------------------------------------------ one pass

def _typed(w):
    """ids and times of records or intervals: whole numbers in all but the
    last two words, then t_lo and t_hi."""
    k = w.shape[1] - 2
    return {"ids": w[:, :k].view(torch.int32), "times": w[:, k:].view(torch.float64)}


def _ordered(src, n, to):
    """The n records of src by (e_seg, q_seg) in the result array, zeros after
    them.  A record's first word is e_seg, q_seg from the high half down."""
    torch.index_select(src[:n], 0, torch.sort(src[:n, 0])[1], out=to[:n])
    to[n:].zero_()
    return _typed(to)


def _host_records(c, r):
    ids, times = np.zeros((_room(c), 4), np.uint32), np.zeros((_room(c), 2))
    for a, k in enumerate(("q_seg", "e_seg", "q_traj", "e_traj")):
        ids[:len(r), a] = r[k]
    for a, k in enumerate(("t_lo", "t_hi")):
        times[:len(r), a] = r[k]
    return {"ids": ids, "times": times}


def _done(status):
    if status != 0:
        raise RuntimeError("status %d" % status)


def _merged(s, n):
    out, to = s["out"], s["merged"]
    st, k = tds.merge_trajectories_raw(out.data_ptr(), n, True, to.data_ptr(), to.shape[0], True)
    _done(st)
    to[k:].zero_()
    return _typed(to)


def run(state):
    s, c = state, state["case"]
    path = c["path"]
    if path == "build":
        with tds.Index(s["D"], num_bins=c["bins"]) as idx:
            return idx.export()
    idx, (t0, t1) = s["index"], s["window"]
    if path == "request":
        return _host_records(c, tds.sort_records(idx.search(s["Q"], c["d"], t0, t1)))
    if path == "batcher":
        got, _, st = s["batcher"].run(s["Q"])
        _done(st)
        return _host_records(c, np.concatenate([tds.sort_records(r) for r in got]))
    out, at = s["out"], dict(out_ptr=s["out"].data_ptr(), out_on_device=True)
    if path == "batch":
        st, n, _ = idx.search_batch_raw(s["Q"], s["requests"], out_capacity=out.shape[0], **at)
        _done(st)
        return [_ordered(out[r[5]:r[5] + r[6]], k, s["sorted"][r[5]:r[5] + r[6]]) for r, k in zip(s["requests"], n)]
    at["capacity"] = out.shape[0]
    if path == "join":
        st, n, _ = idx.self_join_raw(c["d"], t0, t1, **at)
    elif path == "grid":
        st, n, _ = s["grid"].search_raw(s["Q"], c["d"], t0, t1, **at)
    else:
        st, n, _ = idx.search_raw(s["Q"], c["d"], t0, t1, precision=c.get("precision", "fp32"), **at)
    _done(st)
    return _merged(s, n) if path in ("merge", "join") else _ordered(out, n, s["sorted"])


# ------------------------------------------------------------------ the same in 64 bits

def _motion(s):
    p = torch.stack([s["xs"], s["ys"], s["zs"]])
    v = (torch.stack([s["xe"], s["ye"], s["ze"]]) - p) / (s["te"] - s["ts"])
    return p, v


def _pairs(D, Q, d, t0, t1, unit, skip=None):
    """Every (query, entry) pair that overlaps in time inside the window and
    comes within d of each other: positions q, e and the interval's ends.
    Segments last `unit`, so a query meets entries of its own, the previous
    and the next step only."""
    pe, ve = _motion(D)
    pq, vq = _motion(Q)
    ke, kq = (D["ts"] / unit).floor().long(), (Q["ts"] / unit).floor().long()
    eo, qo = torch.argsort(ke), torch.argsort(kq)
    ke, kq = ke[eo].contiguous(), kq[qo].contiguous()
    steps = torch.unique(kq)
    near = torch.searchsorted(ke, torch.stack([steps - 1, steps + 2], 1).contiguous()).tolist()
    own = torch.searchsorted(kq, torch.stack([steps, steps + 1], 1).contiguous()).tolist()
    found = []
    for (e0, e1), (q0, q1) in zip(near, own):
        e = eo[e0:e1]
        if e.numel() == 0:
            continue
        part = max(1, 50_000_000 // e.numel())
        for a0 in range(q0, q1, part):
            q = qo[a0:min(q1, a0 + part)]
            a = torch.maximum(Q["ts"][q].clamp_min(t0)[:, None], D["ts"][e][None])
            b = torch.minimum(Q["te"][q].clamp_max(t1)[:, None], D["te"][e][None])
            i, j = (a < b).nonzero(as_tuple=True)
            if skip is not None:
                k = skip(q[i], e[j])
                i, j = i[k], j[k]
            if i.numel() == 0:
                continue
            a, b = a[i, j], b[i, j]
            i, j = q[i], e[j]
            da = [(pq[x][i] + vq[x][i] * (a - Q["ts"][i])) - (pe[x][j] + ve[x][j] * (a - D["ts"][j])) for x in range(3)]
            db = [(pq[x][i] + vq[x][i] * (b - Q["ts"][i])) - (pe[x][j] + ve[x][j] * (b - D["ts"][j])) for x in range(3)]
            w = [vq[x][i] - ve[x][j] for x in range(3)]
            c0 = sum(x * x for x in da) - d * d
            c1 = sum(x * x for x in db) - d * d
            aa = sum(x * x for x in w)
            bb = sum(x * y for x, y in zip(da, w))
            disc = bb * bb - aa * c0
            T = b - a
            hit = (c0 <= 0) | (c1 <= 0) | ((aa > 0) & (bb < 0) & (-bb < aa * T) & (disc >= 0))
            i, j, a, b, c0, c1, aa, bb, disc, T = (x[hit] for x in (i, j, a, b, c0, c1, aa, bb, disc, T))
            root = disc.clamp_min(0).sqrt()
            qq = torch.where(bb >= 0, -bb - root, -bb + root)
            r1, r2 = qq / aa, torch.where(qq != 0, c0 / qq, 0.0)
            lo = torch.where(c0 <= 0, a, a + torch.minimum(torch.minimum(r1, r2).clamp_min(0), T))
            hi = torch.where(c1 <= 0, b, a + torch.minimum(torch.maximum(r1, r2).clamp_min(0), T))
            still = aa == 0
            found.append((i, j, torch.where(still, a, lo), torch.where(still, b, hi)))
    if not found:
        z = torch.zeros(0, dtype=torch.long, device="cuda")
        return z, z, z.double(), z.double()
    return tuple(torch.cat(x) for x in zip(*found))


def _times(lo, hi, room):
    t = torch.zeros(room, 2, dtype=torch.float64, device="cuda")
    t[:lo.numel(), 0], t[:lo.numel(), 1] = lo, hi
    return {"ids": None, "times": t}


def _in_order(q, e, lo, hi, room, by_query=False):
    k = torch.argsort((q << 32) | e if by_query else (e << 32) | q)
    return _times(lo[k], hi[k], room)


def _joined(qt, et, lo, hi, room):
    """Maximal intervals of each trajectory pair, by (q_traj, e_traj, t_lo)."""
    o = torch.argsort(lo)
    o = o[torch.argsort((qt[o].long() << 32) | et[o].long(), stable=True)]
    pair, lo, hi = ((qt.long() << 32) | et.long())[o], lo[o], hi[o]
    run_of = torch.unique_consecutive(pair, return_inverse=True)[1]
    ends, rank = torch.unique(hi, return_inverse=True)
    most = torch.cummax(run_of * ends.numel() + rank, 0)[0]
    reach = ends[most % ends.numel()]
    head = torch.ones_like(pair, dtype=torch.bool)
    head[1:] = (pair[1:] != pair[:-1]) | (lo[1:] > reach[:-1])
    last = torch.cat([head[1:], head.new_ones(1)])
    return _times(lo[head], reach[last], room)


def exact(case, seed):
    c = case
    D, Q = _inputs(c, seed)
    unit = 0.5 if c["data"] == "merger" else 1.0
    t0, t1 = _window(c)
    if c["path"] == "build":
        tmin, tmax = D["ts"].min(), D["te"].max()
        m = c["bins"] or max(1, min(65535, int(((tmax - tmin) / (D["te"] - D["ts"]).mean()).round())))
        b = ((D["ts"] - tmin) / ((tmax - tmin) / m)).floor().long().clamp(0, m - 1)
        lo = torch.full((m,), INF, dtype=torch.float64, device="cuda").scatter_reduce(0, b, D["ts"], "amin")
        hi = torch.full((m,), -INF, dtype=torch.float64, device="cuda").scatter_reduce(0, b, D["te"], "amax")
        return {"order": None, "bin_first": None, "min_ts": lo, "max_te": hi, "cmax_te": torch.cummax(hi, 0)[0]}
    room = _room(c)
    if c["path"] == "batcher":
        got = []
        for r, d, a, b in Q:
            x = {k: torch.from_numpy(v.astype(np.int32) if k == "traj" else v).cuda() for k, v in r.items()}
            q, e, lo, hi = _pairs(D, x, d, a, b, unit)
            k = torch.argsort((q << 32) | e)
            got.append((lo[k], hi[k]))
        return _times(*(torch.cat(x) for x in zip(*got)), room)
    if c["path"] == "batch":
        return [_in_order(*_pairs(D, Q, d, t0, t1, unit), k) for d, (_, k) in zip(_distances(c), _slices(c))]
    if c["path"] == "join":
        other = lambda q, e: (D["traj"][q] != D["traj"][e]) & (q < e)  # noqa: E731
        q, e, lo, hi = _pairs(D, D, c["d"], t0, t1, unit, other)
        return _joined(D["traj"][q], D["traj"][e], lo, hi, room)
    q, e, lo, hi = _pairs(D, Q, c["d"], t0, t1, unit)
    if c["path"] == "merge":
        return _joined(Q["traj"][q], D["traj"][e], lo, hi, room)
    return _in_order(q, e, lo, hi, room, c["path"] == "request")
