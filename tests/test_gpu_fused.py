"""Fused backward level kernel, which runs past the split levels' rule (nets a level over all snapshots):
against the split form of the same designs alone, bit for bit, over every lane mapping of its cell step,
cells of 5-8 inputs, whole-workgroup nets with a third pass of sinks, snapshots and batches."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gen.netlist import make_design, scaled_spec
from paper_2603_28381_amd import Graph
from tests._designs import fanout_design, wide_dag

pytestmark = pytest.mark.gpu

LINE = 16384          # nets a level beyond which every backward is fused, checkpointed or not
DESIGNS = {"wide": lambda: wide_dag(n_levels=9, gates_per_level=60, n_pi=16, seed=7),
           "fanout": lambda: fanout_design(via_cell=True),
           "tail": lambda: make_design(scaled_spec(30_000, cfg_id=81, box_um=400.0))}
KINDS = [dict(rat=True, grad=True), dict(rat=False, grad=True, pins=False), dict(rat=True, grad=False)]


def _copies(d, n):
    """n placements of d, a few um apart."""
    rng = np.random.default_rng(5)
    x, y = (np.repeat(v[None], n, 0) for v in (d.x, d.y))
    x[1:] += rng.normal(0, 3, x[1:].shape).astype(np.float32)
    y[1:] += rng.normal(0, 3, y[1:].shape).astype(np.float32)
    return x, y


def _backward(g, x, y, canonical, kind, levels, fused):
    """The outputs of one step, whose backward ran in the form asked for."""
    x, y = (torch.tensor(v, device="cuda") for v in (x, y))
    f = g.forward(x, y, canonical=canonical)
    g.profile(True)
    o = g.backward(x, y, f, **kind)
    ran = g.profile_read()
    g.profile(False)
    assert (ran["bwd_level"][0], ran["expand"][0]) == ((levels, 0) if fused else (levels - 1, 1))
    return {k: v.cpu().numpy() for k, v in o.items()}


@pytest.mark.parametrize("stride", [0, 4])
@pytest.mark.parametrize("canonical", [False, True])
@pytest.mark.parametrize("form", ["snapshots", "batch"])
@pytest.mark.parametrize("design", list(DESIGNS))
def test_fused_levels_equal_split_levels_bitwise(design, form, canonical, stride):
    d = DESIGNS[design]()
    one = Graph.from_design(d)
    L = one.levelize()
    n = LINE * L // d.n_nets + 2
    xs, ys = _copies(d, n)
    if form == "snapshots":
        many = Graph.from_design(d)
        many.levelize()
        many.set_snapshots(n)
    else:
        many = Graph.batch([one] * n)
        many.levelize()
    many.set_checkpointing(stride)
    order = one.levelization()["pin_perm"]
    if form == "snapshots":
        xm, ym = (v[:, order] for v in (xs, ys)) if canonical else (xs, ys)
        member = lambda v, s: v[s]  # noqa: E731
    else:
        perm = many.levelization()["pin_perm"]
        xm, ym = (v.reshape(-1)[perm] for v in (xs, ys)) if canonical else (v.reshape(-1) for v in (xs, ys))

        def member(v, s):
            if not canonical:
                return v[s * d.n_pins:(s + 1) * d.n_pins]
            w = np.empty_like(v)
            w[perm] = v                                 # by (member, pin of the design)
            return w[s * d.n_pins:(s + 1) * d.n_pins][order]

    for sweep in (2, 3, 4, 5, 6):
        one.set_schedule(sweep, 2, 64)
        many.set_schedule(sweep, 2, 64)
        for kind in KINDS:
            print(f"fused: {design} {form} x{n} sweep {sweep} canonical {canonical} stride {stride} {kind}", flush=True)
            got = _backward(many, xm, ym, canonical, kind, L, fused=True)
            for s in (0, n - 1):
                x1, y1 = (v[s][order] for v in (xs, ys)) if canonical else (xs[s], ys[s])
                ref = _backward(one, x1, y1, canonical, kind, L, fused=False)
                assert set(ref) == set(got)
                for k in ref:
                    assert np.array_equal(member(got[k], s), ref[k], equal_nan=True), (sweep, kind, s, k)
