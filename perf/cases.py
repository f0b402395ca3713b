"""Timed cases of the STA engine: what its users call, over the range of sizes they call it at.

A case is a dict of plain values.  `kind` names the use:

* ``step``     a placer's or optimiser's full timing step: the smoothed forward sweep, then the
               backward sweep with every per-pin output (arrival, slew, required time, slack)
               and the gradient of the smoothed TNS;
* ``forward``  a timing query: the forward sweep with per-pin arrivals, slews and smoothed
               arrivals, no backward;
* ``sta``      plain STA without differentiation: unsmoothed forward, required times and slacks;
* ``grad``     the loss term of a differentiable placer: ``smoothed_tns`` / ``smoothed_wns``
               and its backward through autograd, every buffer allocated by the call;
* ``ckpt``     a gradient step under per-level checkpointing, for callers short of memory;
* ``serve``    a burst of requests to the serving loop (host coordinates in, host results out).

Designs are drawn like the repository's generator draws its workloads (1-4 inputs a cell, 70 %
of nets with 2-3 pins and a Pareto tail up to 500, level distances geometric), with sinks
placed around their driver so that most loads and slews lie inside the library's tables.
Every call gets its netlist and constraints as host arrays, as a user's program has them.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2603_28381_amd import Graph, Server, smoothed_tns, smoothed_wns

GAMMA = 10.0
R_UM, C_UM = 0.1, 0.2
AXIS = 7
NO_EXACT_ABOVE = 6_000_000          # pins x snapshots beyond which the 64-bit reference is too slow


def _case(name, kind, pins, snaps=1, inner=False, designs=1, trees=False, fanin=4, canonical=False, wns=False,
          capture=False, requests=0):
    c = dict(kind=kind, pins=pins, snaps=snaps, inner=inner, designs=designs, trees=trees, fanin=fanin,
             canonical=canonical, wns=wns, capture=capture, requests=requests)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A block of a thousand gates inside an interactive loop: launches and latency only.
        _case("step_4k", "step", 4_000),
        # Sign-off style STA of a small block, with cells of up to 8 inputs.
        _case("sta_20k_fanin8", "sta", 20_011, fanin=8),
        # A partition of a chip in a timing-driven placer.
        _case("step_63k", "step", 63_000),
        # Slack query of a whole mid-size design (the 0.8M-pin workload's size).
        _case("forward_806k", "forward", 806_000),
        # Timing loss of a differentiable placer on it, through autograd.
        _case("grad_806k", "grad", 806_000),
        # Full step of a superblue-size design, canonical order: the headline workload's size.
        _case("step_2500k", "step", 2_500_000, canonical=True),
        # Full step with RC trees instead of stars.
        _case("step_trees_400k", "step", 400_000, trees=True),
        # Gradient step of the 0.8M-pin size in reduced memory.
        _case("ckpt_806k", "ckpt", 806_000, canonical=True),
        # A few placement candidates evaluated together, snapshot-outer layout.
        _case("snap8_100k", "step", 100_000, snaps=8, canonical=True),
        # Many placement candidates of the 0.8M-pin size, one wave lane per snapshot.
        _case("snap64_806k", "step", 806_000, snaps=64, inner=True, canonical=True),
        # Eight designs of different sizes in one captured batch.
        _case("batch8_600k", "step", 600_000, designs=8, canonical=True, capture=True),
        # A burst of slack and gradient requests to resident designs.
        _case("serve_8req", "serve", 120_000, designs=2, requests=8),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    fanin = 8 if rng.random() < 0.2 else 4
    canonical, wns = rng.random() < 0.5, rng.random() < 0.3
    use = rng.choice(["step", "step", "grad", "grad", "forward", "sta", "trees", "ckpt", "outer", "inner", "inner",
                      "batch"])
    if use == "outer":
        snaps = rng.randint(2, 12)
        return _case("", "step", size(5_000, 1_000_000 // snaps), snaps, canonical=canonical, wns=wns, fanin=fanin)
    if use == "inner":
        snaps = rng.choice([32, 48, 64, 64, 96])
        return _case("", "step", size(10_000, 20_000_000 // snaps), snaps, inner=True, canonical=canonical, wns=wns,
                     fanin=fanin)
    if use == "batch":
        return _case("", "step", size(50_000, 800_000), designs=rng.randint(2, 12), canonical=canonical,
                     capture=rng.random() < 0.5)
    if use == "trees":
        return _case("", "step", size(4_000, 800_000), trees=True, canonical=canonical, fanin=fanin)
    return _case("", use, size(4_000, 1_500_000), canonical=canonical and use != "grad", fanin=fanin,
                 wns=wns and use in ("step", "grad", "ckpt"))


# ------------------------------------------------------------------------------- designs
@functools.lru_cache(maxsize=2)
def _library(fanin_max):
    """Eight cell types of each fanin; mildly curved delay and slew tables on log axes."""
    rng = np.random.default_rng([7, fanin_max])
    fan = np.repeat(np.arange(1, fanin_max + 1), 8)
    off = np.concatenate([[0], np.cumsum(fan)])
    n = int(off[-1])
    slew = np.geomspace(5.0, 500.0, AXIS).astype(np.float32)
    load = np.geomspace(1.0, 200.0, AXIS).astype(np.float32)
    s, ld = slew.astype(np.float64)[:, None], load.astype(np.float64)[None, :]
    tab = np.empty((n, 4, AXIS, AXIS))
    for q, (a, b, c, k) in enumerate([((10, 30), (.05, .3), (.2, 1.), .15)] * 2 + [((3, 10), (.02, .15), (.5, 2.), .1)] * 2):
        u = lambda r: rng.uniform(*r, size=(n, 1, 1))  # noqa: E731
        tab[:, q] = u(a) + u(b) * s + u(c) * ld + k * np.sqrt(s * ld) + rng.normal(0, 0.1, (n, AXIS, AXIS))
    return dict(n_cell_types=len(fan), arc_offsets=off.astype(np.int32),
                arc_unate=np.where(rng.random(n) < 0.5, 1, -1).astype(np.int8), slew_axis=slew, load_axis=load,
                tables=tab.astype(np.float32))


@functools.lru_cache(maxsize=24)
def _design(pins, fanin_max, trees, salt):
    """A netlist of about `pins` pins: host arrays, as a user's program reads them from disk."""
    rng = np.random.default_rng([11, pins, fanin_max, salt])
    gates = max(16, int(round(pins / (3.85 if fanin_max <= 4 else 5.9))))
    levels = min(gates, max(2, int(round(12.0 * (pins / 4000.0) ** 0.31))))
    n_pi = max(8, gates // 100)
    N = n_pi + gates
    lev = np.concatenate([np.zeros(n_pi, np.int64), 1 + np.arange(gates) * levels // gates])   # nets by level
    start = np.searchsorted(lev, np.arange(levels + 2))
    u = rng.random(N)
    tail = np.clip(np.floor(2.5 * rng.random(N) ** (-1 / 1.5)), 4, 500)
    fan = np.where(u < 0.7, rng.integers(2, 4, N), tail).astype(np.int64) - 1
    if fanin_max > 4:
        fan = fan * 2
    # Each level's free fanout slots, taken in random order; a level that runs out widens its nets.
    pool, used = [], np.zeros(levels + 1, np.int64)
    for l in range(levels + 1):
        pool.append(rng.permutation(np.repeat(np.arange(start[l], start[l + 1]), fan[start[l]:start[l + 1]])))
    k = rng.integers(1, fanin_max + 1, gates)
    off = np.concatenate([[0], np.cumsum(k)])
    A = int(off[-1])
    gate = np.repeat(np.arange(gates), k)
    first = np.zeros(A, bool)
    first[off[:-1] + rng.integers(0, 1 << 30, gates) % k] = True          # this input sets the gate's level
    glev = lev[n_pi:][gate]
    src_lev = np.where(first, glev - 1, np.maximum(0, glev - rng.geometric(0.5, A)))
    src = np.empty(A, np.int64)
    order = np.argsort(src_lev, kind="stable")
    cut = np.searchsorted(src_lev[order], np.arange(levels + 2))
    for l in range(levels + 1):
        want = order[cut[l]:cut[l + 1]]
        if len(want):
            got = pool[l][:len(want)]
            used[l] = len(got)
            more = rng.integers(start[l], start[l + 1], len(want) - len(got))
            src[rng.permutation(want)] = np.concatenate([got, more])
    ep = np.concatenate([pool[l][used[l]:] for l in range(levels + 1)])
    ends = np.zeros(N, bool)
    ends[src] = ends[ep] = True
    ep = np.concatenate([ep, np.flatnonzero(~ends)])                       # no net without a sink
    P = N + A + len(ep)
    net = np.concatenate([np.arange(N), src, ep])
    kind = np.concatenate([np.where(np.arange(N) < n_pi, 0, 2), np.full(A, 1), np.where(rng.random(len(ep)) < .2, 3, 4)])
    pid, nid, cid = rng.permutation(P), rng.permutation(N), rng.permutation(gates)
    by = np.lexsort((rng.random(P), np.arange(P) >= N, nid[net]))
    cnt = np.bincount(nid[net], minlength=N)
    noff = np.concatenate([[0], np.cumsum(cnt)])
    inv = np.argsort(cid)
    coff = np.concatenate([[0], np.cumsum(k[inv])])
    slot = np.repeat(off[:-1][inv] - coff[:-1], k[inv]) + np.arange(A)
    pk = np.empty(P, np.int8)
    pk[pid] = kind
    cap = np.zeros(P, np.float32)
    cap[pid[N:]] = rng.uniform(1.0, 5.0, P - N)
    net_pins = pid[by]
    nl = dict(n_pins=P, n_nets=N, n_cells=gates, net_offsets=noff.astype(np.int32), net_pins=net_pins.astype(np.int32),
              cell_type=((k[inv] - 1) * 8 + rng.integers(0, 8, gates)).astype(np.int32),
              cell_in_offsets=coff.astype(np.int32), cell_in_pins=pid[N + slot].astype(np.int32),
              cell_out_pin=pid[n_pi + inv].astype(np.int32), pin_cap=cap, pin_kind=pk, pin_parent=None)
    if trees:                                             # a binary heap over each net's pins
        nn = np.repeat(np.arange(N), cnt)
        pos = np.arange(P) - noff[nn]
        par = np.full(P, -1, np.int32)
        par[net_pins[pos > 0]] = net_pins[noff[nn[pos > 0]] + (pos[pos > 0] - 1) // 2]
        nl["pin_parent"] = par
    net_level = np.empty(N, np.int64)
    net_level[nid] = lev
    cons = dict(t_clk=50.0 * levels, setup=5.0, hold=2.0, pi_at=0.0, pi_slew=10.0, r_per_um=R_UM, c_per_um=C_UM)
    # Every pin's driver, to place sinks around it.
    drv = np.empty(P, np.int64)
    drv[net_pins] = np.repeat(net_pins[noff[:-1]], cnt)
    return dict(nl=nl, lib=_library(fanin_max), cons=cons, net_level=net_level, driver=drv)


def _designs(case):
    """The netlists of a case: one, or a batch's or a server's, of sizes a factor of ten apart."""
    n = case["designs"]
    w = np.geomspace(1.0, 10.0, n) if n > 1 else np.ones(1)
    return [_design(max(1000, int(case["pins"] * f / w.sum())), case["fanin"], case["trees"], i) for i, f in enumerate(w)]


def _batch_cons(ds):
    """Batched graphs share their constraints: those of the deepest design."""
    return max((d["cons"] for d in ds), key=lambda c: c["t_clk"])


def _order(ds):
    """Canonical pin order of the designs together: nets by (level, pins, id), pins net by net."""
    base = np.concatenate([[0], np.cumsum([d["nl"]["n_pins"] for d in ds])])
    pins = np.concatenate([d["nl"]["net_pins"].astype(np.int64) + b for d, b in zip(ds, base)])
    cnt = np.concatenate([np.diff(d["nl"]["net_offsets"]) for d in ds]).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(cnt)])
    nets = np.lexsort((np.arange(len(cnt)), cnt, np.concatenate([d["net_level"] for d in ds])))
    c = cnt[nets]
    return pins[np.repeat(off[:-1][nets] - np.concatenate([[0], np.cumsum(c)[:-1]]), c) + np.arange(len(pins))]


def _place(ds, seed, snaps, device):
    """x, y [snaps, pins] by original pin id: drivers over the die, sinks around their driver;
    snapshots differ from the first by a few um."""
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 1009 + 17)
    xy = []
    for d in ds:
        P = d["nl"]["n_pins"]
        drv = torch.from_numpy(d["driver"]).to(device)
        side = 1.5 * math.sqrt(P)
        own = torch.rand(2, P, device=device, generator=g) * side
        off = torch.randn(2, P, device=device, generator=g) * 15.0
        sink = (drv != torch.arange(P, device=device)).float()
        xy.append(own[:, drv] + off * sink)
    base = torch.cat(xy, 1)
    out = base[:, None, :].repeat(1, snaps, 1)
    if snaps > 1:
        for s in range(1, snaps):
            out[:, s] += torch.randn(base.shape, device=device, generator=g) * 3.0
    return out[0].contiguous(), out[1].contiguous()


def _graph(d, cons):
    g = Graph(d["nl"], d["lib"], cons)
    g.levelize()
    return g


# ------------------------------------------------------------------------------- states
def prepare(case, seed):
    ds = _designs(case)
    st = dict(case=case)
    if case["kind"] == "serve":
        srv = Server(8 << 30, max_slots=2, max_merge=4)
        x, y = (t[0].cpu().numpy() for t in _place(ds, seed, 1, "cuda"))
        ids, lo, reqs = [], 0, []
        rng = np.random.default_rng([13, int(seed)])
        for d in ds:
            P = d["nl"]["n_pins"]
            ids.append(srv.add_design(_graph(d, d["cons"]), x[lo:lo + P], y[lo:lo + P]))
            reqs.append((x[lo:lo + P], y[lo:lo + P]))
            lo += P
        todo = []
        for i in range(case["requests"]):            # every other request asks for the gradient on new coordinates
            j = (i // 2) % len(ds)
            if i % 2:
                a, b = reqs[j]
                todo.append((ids[j], True, a + rng.normal(0, 2, len(a)).astype(np.float32),
                             b + rng.normal(0, 2, len(b)).astype(np.float32)))
            else:
                todo.append((ids[j], False, None, None))
        st.update(server=srv, todo=todo)
        return st
    cons = _batch_cons(ds)
    graphs = [_graph(d, cons) for d in ds]
    g = graphs[0] if len(ds) == 1 else Graph.batch(graphs)
    g.levelize()
    S = case["snaps"]
    if S > 1:
        g.set_snapshots(S)
        if case["inner"]:
            g.set_snapshot_layout(True)
    if case["kind"] == "ckpt":
        g.set_checkpointing(-1)
    g.upload()
    x, y = _place(ds, seed, S, "cuda")
    if case["canonical"]:
        perm = torch.from_numpy(g.levelization()["pin_perm"].astype(np.int64)).cuda()
        x, y = x[:, perm], y[:, perm]
    x, y = (t.t() if case["inner"] else t for t in (x, y))
    x, y = (t.reshape(-1).contiguous() if S == 1 else t.contiguous() for t in (x, y))
    st.update(graph=g, x=x, y=y)
    kind = case["kind"]
    if kind == "grad":
        x.requires_grad_(True)
        y.requires_grad_(True)
        return st
    st["state"] = g.new_state()
    st["scalars"] = torch.empty(((S,) if S > 1 else ()) + ((len(ds), 4) if len(ds) > 1 else (4,)), dtype=torch.float64,
                                device="cuda")
    P = g.n_pins
    shape = (lambda *t: ((P, S) if case["inner"] else (S, P)) + t) if S > 1 else (lambda *t: (P,) + t)
    new = lambda *t: torch.empty(shape(*t), device="cuda")  # noqa: E731
    if kind == "forward":
        st["out"] = dict(at=new(4), slew=new(4), atg=new(2))
    else:
        st["work"] = g.new_workspace()
        names = {"step": ("at", "slew", "rat", "slack", "dx", "dy"), "sta": ("at", "slew", "rat", "slack"),
                 "ckpt": ("dx", "dy")}[kind]
        st["out"] = {k: new() if k in ("dx", "dy") else new(4) for k in names}
    return st


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit(d, grad, x, y, GAMMA) for d, grad, x, y in state["todo"]]
        got = [srv.wait(t) for t in tickets]
        return [{k: r[k] for k in ("scalars", "dx", "dy") if k in r} for r in got]
    g, x, y = state["graph"], state["x"], state["y"]
    if kind == "grad":
        x.grad = y.grad = None
        loss = (smoothed_wns if case["wns"] else smoothed_tns)(x, y, g, GAMMA)
        loss.backward()
        return dict(loss=loss.detach(), dx=x.grad, dy=y.grad)
    smooth = kind != "sta"
    fwd = g.forward(x, y, gamma=GAMMA, smooth=smooth, canonical=case["canonical"], state=state["state"],
                    scalars=state["scalars"], capture=case["capture"], out=state["out"] if kind == "forward" else None)
    if kind == "forward":
        return dict(state["out"], scalars=state["scalars"])
    g.backward(x, y, fwd, rat=kind != "ckpt", grad=smooth, wns=case["wns"], pins=kind != "ckpt",
               workspace=state["work"], out=state["out"], capture=case["capture"])
    return dict(state["out"], scalars=state["scalars"] if smooth else state["scalars"][..., :2])


def work(case):
    """Coordinates, netlist and library read once, every output written once; about 120 operations
    a pin for the forward sweep and 180 for the backward one."""
    pins = float(sum(d["nl"]["n_pins"] for d in _designs(case)))
    S, kind = case["snaps"], case["kind"]
    if kind == "serve":
        per, each = case["requests"] / 2 / case["designs"], 8.0 + 8.0
        return dict(bytes=pins * per * (2 * 12.0 + each), flops=pins * per * 420.0)
    topo = pins * (16.0 + (4.0 if case["trees"] else 0.0) + (0.0 if case["canonical"] else 4.0))
    out = {"step": 72.0, "forward": 40.0, "sta": 64.0, "grad": 8.0, "ckpt": 8.0}[kind]
    ops = {"forward": 120.0, "sta": 200.0}.get(kind, 300.0)
    return dict(bytes=topo + pins * S * (8.0 + out), flops=pins * S * ops)


# ------------------------------------------------------------------------- 64-bit reference
def _wires(d, x, y, dev):
    """Wire delay and impulse of every pin, root load of every net (Eq. 1-3), in float64."""
    nl = d["nl"]
    P, N = nl["n_pins"], nl["n_nets"]
    off = torch.from_numpy(nl["net_offsets"].astype(np.int64)).to(dev)
    pins = torch.from_numpy(nl["net_pins"].astype(np.int64)).to(dev)
    net = torch.empty(P, dtype=torch.int64, device=dev)
    net[pins] = torch.repeat_interleave(torch.arange(N, device=dev), off[1:] - off[:-1])
    cp = torch.from_numpy(nl["pin_cap"].astype(np.float64)).to(dev)
    drv = torch.from_numpy(d["driver"]).to(dev)
    r, c = d["r"], d["c"]
    if nl["pin_parent"] is None:
        ln = (x - x[drv]).abs() + (y - y[drv]).abs()
        dly = 1e-3 * r * ln * (cp + 0.5 * c * ln)
        return net, dly, dly, torch.zeros(N, dtype=x.dtype, device=dev).index_add(0, net, cp + c * ln)
    par = torch.from_numpy(nl["pin_parent"].astype(np.int64)).to(dev)
    up = torch.where(par < 0, torch.arange(P, device=dev), par)
    ln = (x - x[up]).abs() + (y - y[up]).abs()
    res = 1e-3 * r * ln
    cap = (cp + 0.5 * c * ln).index_add(0, up, 0.5 * c * ln)
    depth, at = torch.zeros(P, dtype=torch.int64, device=dev), torch.arange(P, device=dev)
    while bool((up[at] != at).any()):
        depth += up[at] != at
        at = up[at]
    lay = [torch.nonzero((depth == k) & (par >= 0)).flatten() for k in range(1, int(depth.max()) + 1)]

    def total(v):                                   # a node's value plus its children's totals
        for i in reversed(lay):
            v = v.index_add(0, up[i], v[i])
        return v

    def path(v):                                    # sum of v from below the driver down to each pin
        s = torch.zeros_like(v)
        for i in lay:
            s = s.index_copy(0, i, s[up[i]] + v[i])
        return s

    load = total(cap)
    dly = path(res * load)
    arg = 2.0 * path(res * total(cap * dly)) - dly * dly
    imp = torch.where(arg > 0, arg, torch.ones_like(arg)).sqrt() * (arg > 0)
    return net, dly, imp, load[pins[off[:-1]]]


def _reference(d, x, y, smooth, wns, want_rat, want_grad, cons=None):
    """STA of one placement in float64 by plain torch operations; the gradient by autograd."""
    dev = x.device
    nl, lib, cons = d["nl"], d["lib"], cons or d["cons"]
    d = dict(d, r=float(np.float32(cons["r_per_um"])), c=float(np.float32(cons["c_per_um"])))
    P, N, C = nl["n_pins"], nl["n_nets"], nl["n_cells"]
    T = lambda a: torch.from_numpy(np.asarray(a).astype(np.int64)).to(dev)  # noqa: E731
    x = x.double().detach().requires_grad_(want_grad)
    y = y.double().detach().requires_grad_(want_grad)
    net, dly, imp, load = _wires(d, x, y, dev)
    off, cin = T(nl["cell_in_offsets"]), T(nl["cell_in_pins"])
    out_net = net[T(nl["cell_out_pin"])]
    ctype, aoff, una = T(nl["cell_type"]), T(lib["arc_offsets"]), T(lib["arc_unate"])
    tab = torch.from_numpy(lib["tables"].astype(np.float64)).to(dev)
    ax, ay = (torch.from_numpy(lib[k].astype(np.float64)).to(dev) for k in ("slew_axis", "load_axis"))
    lev = T(d["net_level"])
    F = int((off[1:] - off[:-1]).max())
    j = torch.arange(F, device=dev)
    has = j[None] < (off[1:] - off[:-1])[:, None]                          # [C, F]
    pin = cin[(off[:-1, None] + j[None]).clamp(max=len(cin) - 1)]
    arc = (aoff[ctype][:, None] + j[None]).clamp(max=int(aoff[-1]) - 1)
    at = torch.full((N, 4), cons["pi_at"], dtype=torch.float64, device=dev)
    sl = torch.full((N, 4), cons["pi_slew"], dtype=torch.float64, device=dev)
    ag = torch.full((N, 2), cons["pi_at"], dtype=torch.float64, device=dev)
    clev, order = torch.sort(lev[out_net], stable=True)
    cut = torch.searchsorted(clev, torch.arange(int(lev.max()) + 2, device=dev)).tolist()
    k4 = torch.arange(4, device=dev)
    kept = []
    inf = float("inf")
    for l in range(1, len(cut) - 1):
        c = order[cut[l]:cut[l + 1]]
        n, p, a, h = out_net[c], pin[c], arc[c], has[c]
        tp = torch.where(una[a][..., None] > 0, k4 % 2, 1 - k4 % 2)       # [c, F, 4] input transition
        kin = 2 * (k4 // 2) + tp
        s = net[p]
        w, im = dly[p][..., None], imp[p][..., None]
        ain = torch.gather(at[s], 2, kin) + w
        sin = (torch.gather(sl[s], 2, kin) ** 2 + im ** 2).sqrt()
        xi = torch.bucketize(sin.detach(), ax[1:-1], right=True)
        yl = load[n][:, None, None].expand_as(sin)
        yi = torch.bucketize(yl.detach().contiguous(), ay[1:-1], right=True)
        tx = (sin - ax[xi]) / (ax[xi + 1] - ax[xi])
        ty = (yl - ay[yi]) / (ay[yi + 1] - ay[yi])

        def look(q):
            aa = a[..., None].expand_as(xi)
            v = lambda i, m: tab[aa, q, i, m]  # noqa: E731
            return ((1 - tx) * (1 - ty) * v(xi, yi) + tx * (1 - ty) * v(xi + 1, yi) + (1 - tx) * ty * v(xi, yi + 1) +
                    tx * ty * v(xi + 1, yi + 1))

        t4 = (k4 % 2).expand_as(xi)
        dl, so = look(t4), look(2 + t4)
        miss = ~h[..., None]
        late = (k4 >= 2)
        cand = torch.where(miss, torch.where(late, -inf, inf), (ain + dl).detach())
        na = torch.where(late, cand.amax(1), cand.amin(1))
        so = torch.where(miss, torch.where(late, -inf, inf), so)
        ns = torch.where(late, so.max(1).values, so.min(1).values)
        at = at.detach().index_copy(0, n, na)
        sl = sl.index_copy(0, n, ns)
        if smooth:
            gin = torch.gather(ag[s], 2, tp[..., 2:]) + w
            g = torch.where(miss, -inf, (gin + dl[..., 2:]) / GAMMA)
            ag = ag.index_copy(0, n, GAMMA * torch.logsumexp(g, 1))
        kept.append((n, p, h, kin, dl.detach()))
    sink = torch.ones(P, dtype=torch.bool, device=dev)
    sink[torch.from_numpy(d["driver"]).to(dev)] = False
    kind = torch.from_numpy(nl["pin_kind"]).to(dev)
    ep = torch.nonzero(kind >= 3).flatten()
    rl, re = cons["t_clk"] - cons["setup"], cons["hold"]
    o = {}
    atp, imd, dd = at[net] + dly.detach()[:, None], imp.detach()[:, None], dly.detach()[:, None]
    atp = torch.where(sink[:, None], atp, at[net])
    o["at"] = atp
    o["slew"] = torch.where(sink[:, None], (sl.detach()[net] ** 2 + imd ** 2).sqrt(), sl.detach()[net])
    worst = (rl - atp[ep][:, 2:]).amin(1)
    sc = [worst.amin().clamp(max=0.0), worst.clamp(max=0.0).sum()]
    if smooth:
        agp = ag[net] + torch.where(sink, dly, torch.zeros_like(dly))[:, None]
        o["atg"] = agp.detach()
        se = -GAMMA * torch.logsumexp(-(rl - agp[ep]) / GAMMA, 1)
        tns = -(GAMMA * torch.logaddexp(torch.zeros_like(se), -se / GAMMA)).sum()
        wn = -GAMMA * torch.logsumexp(torch.cat([torch.zeros(1, dtype=torch.float64, device=dev), -se / GAMMA]), 0)
        sc += [wn.detach(), tns.detach()]
        if want_grad:
            o["dx"], o["dy"] = torch.autograd.grad(wn if wns else tns, (x, y))
    o["scalars"] = torch.stack(sc)
    if want_rat:
        late = (k4 >= 2)
        rat = torch.where(late, inf, -inf).double().repeat(P, 1)
        rat[ep] = torch.tensor([re, re, rl, rl], dtype=torch.float64, device=dev)
        pins = torch.nonzero(sink).flatten()
        plev, po = torch.sort(lev[net[pins]], stable=True)
        pins = pins[po]
        pcut = torch.searchsorted(plev, torch.arange(int(lev.max()) + 2, device=dev)).tolist()
        drv = T(d["driver"])
        root = T(nl["net_pins"])[T(nl["net_offsets"])[:-1]]
        for l in range(len(cut) - 2, -1, -1):
            p = pins[pcut[l]:pcut[l + 1]]
            v = rat[p] - dd[p]
            i = drv[p][:, None].expand(-1, 2)
            e = rat[:, :2].scatter_reduce(0, i, v[:, :2], "amax")
            f = rat[:, 2:].scatter_reduce(0, i, v[:, 2:], "amin")
            rat = torch.cat([e, f], 1)
            if l:
                n, q, h, kin, dl = kept[l - 1]
                ro = rat[root[n]][:, None, :] - dl
                back = torch.empty_like(ro).scatter_(2, kin, ro)
                rat[q[h]] = back[h]
        o["rat"] = rat
        o["slack"] = torch.where(late, rat - atp, atp - rat)
    return o


def exact(case, seed):
    S, kind = case["snaps"], case["kind"]
    if case["pins"] * S > NO_EXACT_ABOVE or kind == "serve":
        return None
    ds = _designs(case)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    x, y = _place(ds, seed, S, dev)
    cons = _batch_cons(ds)
    smooth = kind != "sta"
    grad = kind in ("step", "grad", "ckpt")
    snaps = []
    for s in range(S):
        parts, lo = [], 0
        for d in ds:
            P = d["nl"]["n_pins"]
            parts.append(_reference(d, x[s, lo:lo + P], y[s, lo:lo + P], smooth, case["wns"], kind in ("step", "sta"),
                                    grad, cons))
            lo += P
        o = {k: torch.cat([p[k] for p in parts]) for k in parts[0] if k != "scalars"}
        o["scalars"] = torch.stack([p["scalars"] for p in parts]) if len(ds) > 1 else parts[0]["scalars"]
        if case["canonical"]:
            perm = torch.from_numpy(_order(ds)).to(dev)
            o = {k: v if k == "scalars" else v[perm] for k, v in o.items()}
        snaps.append(o)
    if kind == "grad":
        o = snaps[0]
        return dict(loss=o["scalars"][2 if case["wns"] else 3], dx=o["dx"], dy=o["dy"])
    names = {"step": ("at", "slew", "rat", "slack", "dx", "dy"), "forward": ("at", "slew", "atg"),
             "sta": ("at", "slew", "rat", "slack"), "ckpt": ("dx", "dy")}[kind]
    if S == 1:
        return {k: snaps[0][k] for k in names + ("scalars",)}
    return {k: torch.stack([o[k] for o in snaps], 1 if case["inner"] and k != "scalars" else 0)
            for k in names + ("scalars",)}
