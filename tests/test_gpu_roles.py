"""Backward sweep split by role: under checkpointing, against the fused level kernel, its passes without
required times or without the gradient; and RC-tree chunks at the edges of their packing."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

from gen.netlist import jitter, make_design, scaled_spec
from oracle import sta_oracle as O
from paper_2603_28381_amd import Graph
from tests._designs import fanout_design, wide_dag
from tests.test_gpu_parity import GAMMA, check_grad, check_values, gpu_run

pytestmark = pytest.mark.gpu

KINDS = [dict(rat=True, grad=True), dict(rat=False, grad=True), dict(rat=True, grad=False)]


def _sweep(g, x, y, wns=False, pins=True, **kind):
    f = g.forward(x, y, gamma=GAMMA)
    o = g.backward(x, y, f, wns=wns, pins=pins, **kind)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in o.items()}


@pytest.mark.parametrize("design", ["tail", "wide", "fanout"])
@pytest.mark.parametrize("kind", range(3))
def test_split_levels_under_checkpointing_equal_plain_bitwise(design, kind):
    # One segment (every slot shared), several, and one per level: heavy-tailed nets (every class and
    # whole workgroups), cells of 5-8 inputs, a net of over 512 sinks.
    d = {"tail": lambda: make_design(scaled_spec(30_000, cfg_id=81, box_um=400.0)),
         "wide": lambda: wide_dag(n_levels=9, gates_per_level=70, n_pi=16, seed=5),
         "fanout": lambda: fanout_design(via_cell=True)}[design]()
    g = Graph.from_design(d)
    g.levelize()
    x, y = torch.tensor(d.x, device="cuda"), torch.tensor(d.y, device="cuda")
    print(f"roles: {design} {KINDS[kind]}", flush=True)
    plain = _sweep(g, x, y, wns=kind == 1, **KINDS[kind])
    for stride in (1000, 3, 1):
        g.set_checkpointing(stride)
        got = _sweep(g, x, y, wns=kind == 1, **KINDS[kind])
        assert set(got) == set(plain)
        for k in plain:
            assert np.array_equal(got[k], plain[k], equal_nan=True), (stride, k)


@pytest.mark.parametrize("kind,S", [(0, 24), (1, 40), (2, 24)])
def test_snapshots_past_the_split_rule_equal_one_call_bitwise(kind, S):
    # Enough snapshots that a level's nets pass the line of the fused kernel, which one does not.
    d = make_design(scaled_spec(60_000, cfg_id=82, box_um=500.0))
    snaps = [jitter(d, 3.0, stream=s) for s in range(S)]
    g = Graph.from_design(d)
    L = g.levelize()
    line = 16384 if kind == 1 else 10000
    assert S * d.n_nets // L > line > d.n_nets // L
    alone = {}
    for s in (0, S - 1):
        alone[s] = _sweep(g, torch.tensor(snaps[s][0], device="cuda"), torch.tensor(snaps[s][1], device="cuda"), **KINDS[kind])
    g.set_snapshots(S)
    x = torch.tensor(np.stack([a for a, _ in snaps]), device="cuda")
    y = torch.tensor(np.stack([b for _, b in snaps]), device="cuda")
    many = _sweep(g, x, y, **KINDS[kind])
    for s, ref in alone.items():
        for k in ref:
            assert np.array_equal(many[k][s], ref[k], equal_nan=True), (s, k)


@pytest.mark.parametrize("S", [1, 5, 64])
def test_snapshot_lane_passes_equal_the_full_sweep_bitwise(S):
    # S = 1: the same kernels under one thread per net.
    d = make_design(scaled_spec(12_000, cfg_id=83, box_um=300.0))
    g = Graph.from_design(d)
    g.levelize()
    if S == 1:
        g.set_schedule(2, 2, 64, level_scheme="thread")
        x, y = torch.tensor(d.x, device="cuda"), torch.tensor(d.y, device="cuda")
    else:
        g.set_snapshots(S)
        g.set_snapshot_layout(True)
        snaps = [jitter(d, 3.0, stream=s) for s in range(S)]
        x = torch.tensor(np.stack([a for a, _ in snaps], 1), device="cuda")
        y = torch.tensor(np.stack([b for _, b in snaps], 1), device="cuda")
    full = _sweep(g, x, y, **KINDS[0])
    for kind in KINDS[1:]:
        part = _sweep(g, x, y, pins=kind["rat"], **kind)
        for k in part:
            assert np.array_equal(part[k], full[k], equal_nan=True), (kind, k)


@pytest.mark.parametrize("pins", [255, 256, 257, 512, 1023, 1024, 1025])
def test_tree_chunk_packing_edges(pins):
    # One net of `pins` pins (a chunk of its own from 257 on, the fallback kernel from 1025) as a
    # binary heap, among the small nets of its buffers.
    from gen.netlist import heap_trees
    d = heap_trees(fanout_design(n_sinks=pins - 1, via_cell=True))
    assert np.diff(d.net_offsets).max() == pins
    got = gpu_run(d)
    ref = O.run(d, gamma=GAMMA, grad="tns")
    check_values(d, got, ref)
    check_grad(got, ref, 1e-3, 1e-6)


@pytest.mark.parametrize("form", ["split", "lanes", "fused"])
def test_profile_counts_levels_apart_from_the_output_pass(form):
    # Split levels and snapshot lanes: a launch a level above 0, then one output pass of all nets.  The
    # fused kernel (past the nets a level of the split rule): a launch a level, outputs within.
    d = make_design(scaled_spec(60_000, cfg_id=82, box_um=500.0))
    g = Graph.from_design(d)
    L = g.levelize()
    S = {"split": 1, "lanes": 2, "fused": 24}[form]
    if S > 1:
        g.set_snapshots(S)
    if form == "lanes":
        g.set_snapshot_layout(True)
    x, y = (torch.tensor(np.repeat(v[None], S, 0) if S > 1 else v, device="cuda") for v in (d.x, d.y))
    if form == "lanes":
        x, y = x.t().contiguous(), y.t().contiguous()
    g.profile(True)
    _sweep(g, x, y, **KINDS[0])
    got = g.profile_read()
    g.profile(False)
    assert got["fwd_level"][0] == L - 1 and got["ep_seed"][0] == 1
    assert (got["bwd_level"][0], got["expand"][0]) == ((L, 0) if form == "fused" else (L - 1, 1))


@pytest.mark.parametrize("stride", [5, 8, 1000])
def test_checkpointed_segments_launch_once_a_level(stride):
    # A segment's outputs ride with its lowest level: no launch more than the fused kernel's, whose level 0
    # the last output pass replaces.
    d = make_design(scaled_spec(30_000, cfg_id=84, box_um=400.0))
    g = Graph.from_design(d)
    L = g.levelize()
    g.set_checkpointing(stride)
    x, y = torch.tensor(d.x, device="cuda"), torch.tensor(d.y, device="cuda")
    f = g.forward(x, y, gamma=GAMMA)
    g.profile(True)
    g.backward(x, y, f, pins=False)
    ran = g.profile_read()
    g.profile(False)
    assert ran["ep_seed"][0] <= 1 + -(-(L - 1) // stride)
    assert (ran["bwd_level"][0], ran["expand"][0]) == (L - 1, 1)


STREAM = 120 << 20        # output bytes beyond which canonical output passes write streaming stores


@pytest.mark.parametrize("names,per_pin", [(("at", "slew", "atg"), 40), (("slew",), 16)])
def test_forward_outputs_streamed_and_plain_equal_bitwise(names, per_pin):
    # Snapshots on both sides of the line in canonical order, and in original order, always plain.
    d = make_design(scaled_spec(30_000, cfg_id=85, box_um=400.0))
    n = STREAM // (per_pin * d.n_pins)
    g = Graph.from_design(d)
    g.levelize()
    perm = g.levelization()["pin_perm"]
    ref = None
    for S, canonical in ((1, True), (n, True), (n + 1, True), (n + 1, False)):
        g.set_snapshots(S)
        x, y = ((v[perm] if canonical else v)[None].repeat(S, 0) for v in (d.x, d.y))
        x, y = (torch.tensor(v[0] if S == 1 else v, device="cuda") for v in (x, y))
        out = {k: torch.full(((S,) if S > 1 else ()) + (d.n_pins, 2 if k == "atg" else 4), float("nan"), device="cuda")
               for k in names}
        g.forward(x, y, gamma=GAMMA, canonical=canonical, out=out)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy().reshape(S, d.n_pins, -1)[[0, S - 1]] for k, v in out.items()}
        if not canonical:
            got = {k: v[:, perm] for k, v in got.items()}
        ref = ref or got
        for k in names:
            assert np.array_equal(got[k], ref[k][[0, -1]], equal_nan=True), (S, canonical, k)


@pytest.mark.slow
def test_backward_outputs_streamed_and_plain_equal_bitwise():
    # 134 MB of outputs of deep, narrow levels, which stay split also under checkpointing: streamed
    # in canonical order by the output pass and by a segment's lowest level, plain in original order.
    d = make_design(dataclasses.replace(scaled_spec(2_100_000, cfg_id=86, box_um=3000.0), n_levels=112))
    assert 64 * d.n_pins > STREAM
    g = Graph.from_design(d)
    L = g.levelize()
    assert d.n_nets // L < 6000
    perm = g.levelization()["pin_perm"]
    plain = _sweep(g, torch.tensor(d.x, device="cuda"), torch.tensor(d.y, device="cuda"))
    x, y = torch.tensor(d.x[perm], device="cuda"), torch.tensor(d.y[perm], device="cuda")
    for stride in (0, 16):
        g.set_checkpointing(stride)
        f = g.forward(x, y, gamma=GAMMA, canonical=True)
        g.profile(True)
        o = g.backward(x, y, f)
        ran = g.profile_read()
        g.profile(False)
        assert (ran["bwd_level"][0], ran["expand"][0]) == (L - 1, 1)
        for k, v in o.items():
            assert np.array_equal(v.cpu().numpy(), plain[k][perm], equal_nan=True), (stride, k)


@pytest.mark.parametrize("S", [8, 9])
def test_tree_chunks_of_both_sizes_equal_one_call_bitwise(S):
    # 31k pins alone and in 8 snapshots (below 2^18) take the small chunks, in 9 the large; one net
    # between the two sizes, one over the largest (the fallback kernel).
    from gen.netlist import heap_trees
    designs = [heap_trees(make_design(scaled_spec(27_000, cfg_id=87, box_um=300.0)))]
    designs += [heap_trees(fanout_design(n_sinks=n, via_cell=True, n_buf=20)) for n in (299, 1030)]
    one = Graph.batch([Graph.from_design(d) for d in designs])
    one.levelize()
    P = sum(d.n_pins for d in designs)
    assert 8 * P <= 1 << 18 < 9 * P
    many = Graph.batch([Graph.from_design(d) for d in designs])
    many.levelize()
    many.set_snapshots(S)
    x, y = (np.concatenate([getattr(d, k) for d in designs]).astype(np.float32) for k in "xy")
    ref = _sweep(one, torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"))
    got = _sweep(many, *(torch.tensor(v[None].repeat(S, 0), device="cuda") for v in (x, y)))
    for k in ref:
        for s in (0, S - 1):
            assert np.array_equal(got[k][s], ref[k], equal_nan=True), (s, k)
