"""Host-side checks of libsta (no GPU): exported ABI, bit-exact levelization, input validation."""
from __future__ import annotations

import ctypes
import os
import re

import numpy as np
import pytest

from gen.netlist import CFG0, CFG1, make_design, tiny_spec
from oracle import sta_oracle as O
from paper_2603_28381_amd import sta as S
from tests._designs import PIN_CELL_IN, PIN_CELL_OUT, PIN_FF_D, PIN_PI, PIN_PO, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _header_functions():
    txt = open(os.path.join(ROOT, "include", "sta.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(sta_[a-z_]+)\s*\(", txt)))


def test_library_loads_and_exports_every_declared_function():
    lib = S.load_library()
    names = _header_functions()
    assert len(names) >= 10
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(S.EXPORTED)
    assert lib.sta_version() == 1


def _levelization_matches(d):
    g = S.Graph.from_design(d)
    L = g.levelize()
    got = g.levelization()
    ref = O.levelize(d)
    assert L == ref.n_levels
    for k in ("level", "level_offsets", "net_perm", "pin_perm"):
        assert np.array_equal(got[k], getattr(ref, k)), k
    info = g.info()
    assert info["n_endpoints"] == len(np.nonzero((d.pin_kind == 3) | (d.pin_kind == 4))[0])
    assert info["n_pi_nets"] == int(ref.level_offsets[1])
    g.close()


@pytest.mark.parametrize("seed", range(5))
def test_levelization_bit_exact_tiny(seed):
    _levelization_matches(make_design(tiny_spec(8 + 5 * seed, 2 + seed, n_pi=3, seed=seed)))


def test_levelization_bit_exact_cfg0():
    _levelization_matches(make_design(CFG0))


@pytest.mark.slow
def test_levelization_bit_exact_cfg1():
    _levelization_matches(make_design(CFG1))


def _small():
    # PI 0 -> {0, 1}; cell 0 (type 0, 1 input): in 1 -> out 2; net {2, 3}; 3 is a PO.
    return dict(nets=[[0, 1], [2, 3]], cells=[(0, [1], 2)], kinds=[PIN_PI, PIN_CELL_IN, PIN_CELL_OUT, PIN_PO],
                caps=[0, 1, 0, 1], x=[0, 1, 2, 3], y=[0, 0, 0, 0])


def _expect(code, **over):
    kw = _small()
    kw.update(over)
    d = build(**kw)
    with pytest.raises(S.StaError) as e:
        g = S.Graph.from_design(d)
        g.levelize()
    assert e.value.code == code


def test_valid_small_graph_builds():
    g = S.Graph.from_design(build(**_small()))
    assert g.levelize() == 2
    g.close()


def test_rejects_driver_not_first():
    _expect(S.STA_E_INVALID, nets=[[1, 0], [2, 3]])


def test_rejects_pin_in_two_nets():
    _expect(S.STA_E_INVALID, nets=[[0, 1], [2, 1]], kinds=[PIN_PI, PIN_CELL_IN, PIN_CELL_OUT, PIN_PO])


def test_rejects_wrong_fanin_for_type():
    _expect(S.STA_E_INVALID, cells=[(8, [1], 2)])      # type 8 has two arcs


def test_rejects_cell_type_out_of_range():
    _expect(S.STA_E_INVALID, cells=[(99, [1], 2)])


def test_rejects_cell_input_of_wrong_kind():
    _expect(S.STA_E_INVALID, kinds=[PIN_PI, PIN_PO, PIN_CELL_OUT, PIN_PO])


def test_rejects_negative_cap():
    _expect(S.STA_E_INVALID, caps=[0, -1, 0, 1])


def test_rejects_cycle():
    d = build([[0, 1], [2, 3], [4, 5]], [(8, [1, 5], 2), (0, [3], 4)],
              [PIN_PI, PIN_CELL_IN, PIN_CELL_OUT, PIN_CELL_IN, PIN_CELL_OUT, PIN_CELL_IN],
              [0, 1, 0, 1, 0, 1], [0, 1, 2, 3, 4, 5], [0] * 6)
    g = S.Graph.from_design(d)
    with pytest.raises(S.StaError) as e:
        g.levelize()
    assert e.value.code == S.STA_E_CYCLE


def test_levelization_state_errors():
    g = S.Graph.from_design(build(**_small()))
    with pytest.raises(S.StaError) as e:
        g.levelization()
    assert e.value.code == S.STA_E_STATE
    assert g.info()["n_levels"] == 0
    g.levelize()
    assert g.info()["fwd_state_bytes"] > 0 and g.info()["bwd_workspace_bytes"] > 0


def test_schedule_roundtrip_and_validation():
    g = S.Graph.from_design(make_design(tiny_spec(20, 3, n_pi=3, seed=1)))
    with pytest.raises(S.StaError) as e:
        g.set_schedule(4, 2, 64)
    assert e.value.code == S.STA_E_STATE          # not levelized yet
    g.levelize()
    assert g.schedule() == dict(sweep_group_log2=2, flat_group_log2=2, heavy_sinks=64, rc_scheme=S.STA_RC_GROUPS,
                                fwd_cell_lanes=16, level_scheme=S.STA_LEVEL_GROUPS, lane_block=512)
    g.set_schedule(5, 3, 32)
    assert g.schedule() == dict(sweep_group_log2=5, flat_group_log2=3, heavy_sinks=32, rc_scheme=S.STA_RC_GROUPS,
                                fwd_cell_lanes=16, level_scheme=S.STA_LEVEL_GROUPS, lane_block=512)
    g.set_schedule(5, 3, 32, "groups", 4)
    assert g.schedule()["fwd_cell_lanes"] == 4
    g.set_schedule(5, 3, 32, "groups", 8)
    assert g.schedule()["fwd_cell_lanes"] == 8
    g.set_schedule(5, 3, 32, "cte")
    assert g.schedule()["rc_scheme"] == S.STA_RC_CTE
    g.set_schedule(5, 3, 32, "thread", 16, "groups", 1024)
    assert g.schedule()["lane_block"] == 1024
    g.set_schedule(5, 3, 32, "thread")
    assert g.schedule()["rc_scheme"] == S.STA_RC_THREAD
    for bad in ((1, 2, 64), (7, 2, 64), (4, 1, 64), (4, 7, 64), (4, 2, 0), (4, 2, 65), (4, 2, 64, 3),
                (4, 2, 64, -1), (4, 2, 64, 0, 2), (4, 2, 64, 0, 0), (4, 2, 64, 0, 12), (4, 2, 64, 0, 32),
                (4, 2, 64, 0, 16, 3), (4, 2, 64, 0, 16, -1), (4, 2, 64, 0, 16, 0, 128), (4, 2, 64, 0, 16, 0, 768),
                (4, 2, 64, 0, 16, 0, 2048)):
        with pytest.raises(S.StaError) as e:
            g.set_schedule(*bad)
        assert e.value.code == S.STA_E_INVALID
    assert g.schedule() == dict(sweep_group_log2=5, flat_group_log2=3, heavy_sinks=32, rc_scheme=S.STA_RC_THREAD,
                                fwd_cell_lanes=16, level_scheme=S.STA_LEVEL_GROUPS, lane_block=512)
    g.set_schedule(5, 3, 32, "thread", 16, "thread")
    assert g.schedule()["level_scheme"] == S.STA_LEVEL_THREAD
    for call in (lambda: g.set_snapshots(2), lambda: g.set_checkpointing(-1), lambda: g.set_snapshot_layout(True)):
        with pytest.raises(S.StaError) as e:      # one snapshot, no checkpointing, lane groups for snapshot lanes
            call()
        assert e.value.code == S.STA_E_INVALID
    g.set_schedule(5, 3, 32, "cte", 16, "cte")
    assert g.schedule()["level_scheme"] == S.STA_LEVEL_CTE
    for call in (lambda: g.set_snapshots(2), lambda: g.set_checkpointing(-1), lambda: g.set_snapshot_layout(True)):
        with pytest.raises(S.StaError) as e:      # the CTE level kernels: the same restrictions
            call()
        assert e.value.code == S.STA_E_INVALID
    g.set_schedule(5, 3, 32, "thread", 16, "groups")
    g.set_snapshots(2)
    for lv in ("thread", "cte"):
        with pytest.raises(S.StaError) as e:
            g.set_schedule(5, 3, 32, "thread", 16, lv)
        assert e.value.code == S.STA_E_INVALID
    g.close()
    from gen.netlist import heap_trees
    t = S.Graph.from_design(heap_trees(make_design(tiny_spec(20, 3, n_pi=3, seed=1))))
    t.levelize()
    with pytest.raises(S.StaError) as e:                # RC trees: lane groups only
        t.set_schedule(2, 2, 64, "cte", 16, "cte")
    assert e.value.code == S.STA_E_INVALID
    t.close()


def _members():
    from gen.netlist import scaled_spec
    return [make_design(tiny_spec(30, 4, n_pi=4, seed=3)), make_design(scaled_spec(3_000, cfg_id=44, box_um=300.0)),
            make_design(tiny_spec(12, 2, n_pi=2, seed=4))]


def test_batch_levels_and_pin_map_match_members():
    ds = _members()
    gs = [S.Graph.from_design(d) for d in ds]
    b = S.Graph.batch(gs + [gs[0]])
    with pytest.raises(S.StaError) as e:
        b.batch_pin_map()
    assert e.value.code == S.STA_E_STATE
    L = b.levelize()
    members = ds + [ds[0]]
    refs = [O.levelize(d) for d in members]
    assert L == max(r.n_levels for r in refs)
    info = b.info()
    assert info["n_designs"] == 4
    assert info["n_pins"] == sum(d.n_pins for d in members)
    assert info["n_endpoints"] == sum(int(((d.pin_kind == 3) | (d.pin_kind == 4)).sum()) for d in members)
    dsg, pin = b.batch_pin_map()
    # a bijection onto (design, pin)
    flat = np.cumsum([0] + [d.n_pins for d in members])[dsg] + pin
    assert np.array_equal(np.sort(flat), np.arange(info["n_pins"]))
    # every net keeps the level it has in its own design
    lv = b.levelization()
    pperm_b = lv["pin_perm"]          # canonical pin -> union pin id
    pin_off = np.cumsum([0] + [d.n_pins for d in members])
    assert np.array_equal(pin_off[dsg] + pin, pperm_b)
    level_of_net = lv["level"]
    union_net_of_pin = np.concatenate([np.repeat(np.arange(d.n_nets), np.diff(d.net_offsets))[np.argsort(d.net_pins)]
                                       + sum(m.n_nets for m in members[:i]) for i, d in enumerate(members)])
    net_off = np.cumsum([0] + [d.n_nets for d in members])
    for i, (d, r) in enumerate(zip(members, refs)):
        drivers = d.net_pins[d.net_offsets[:-1]]
        assert np.array_equal(level_of_net[union_net_of_pin[pin_off[i] + drivers]], r.level), i
    assert union_net_of_pin.shape[0] == info["n_pins"] and net_off[-1] == info["n_nets"]
    b.close()
    for g in gs:
        g.close()


def test_batch_rejects_mismatched_constraints():
    from gen.netlist import Constraints
    d0 = build(**_small())
    kw = _small()
    d1 = build(**kw, cons=Constraints(t_clk=500.0))
    with pytest.raises(S.StaError) as e:
        S.Graph.batch([S.Graph.from_design(d0), S.Graph.from_design(d1)])
    assert e.value.code == S.STA_E_INVALID


def _expected_checkpoint_counts(d, k):
    """Kept nets and record slots of checkpointing with stride k, from the netlist itself."""
    lv = O.levelize(d)
    N, lvl, L = d.n_nets, lv.level, lv.n_levels
    net_of_pin = np.empty(d.n_pins, np.int64)
    net_of_pin[d.net_pins] = np.repeat(np.arange(N), np.diff(d.net_offsets))
    reader_level = lvl[net_of_pin[d.cell_out_pin]]                      # level of each cell
    cell_of_input = np.repeat(np.arange(d.n_cells), np.diff(d.cell_in_offsets))
    maxc = np.full(N, -1)
    np.maximum.at(maxc, net_of_pin[d.cell_in_pins], reader_level[cell_of_input])
    seg_end = np.where(lvl == 0, 1, 1 + k * ((lvl - 1) // k + 1))
    kept = (lvl == 0) | (maxc >= seg_end)      # endpoints' nets too go in segment buffers
    seg = (lvl - 1) // k
    widest = max([int(np.count_nonzero(~kept & (lvl >= 1) & (seg == j))) for j in range((L - 2) // k + 1)] + [0])
    return int(kept.sum()), int(kept.sum()) + widest


def _expected_sink_slots(d, k):
    """Backward workspace slots under checkpointing with stride k, from the netlist: a net keeps
    its sinks' slots when it sits at level 0, or one of its sinks feeds neither a cell nor is
    an endpoint, or feeds a cell of another segment; the other nets of a segment share a
    buffer (an endpoint is seeded right before its segment's levels)."""
    lv = O.levelize(d)
    N, lvl, L = d.n_nets, lv.level, lv.n_levels
    net_of_pin = np.empty(d.n_pins, np.int64)
    net_of_pin[d.net_pins] = np.repeat(np.arange(N), np.diff(d.net_offsets))
    cell_level = lvl[net_of_pin[d.cell_out_pin]]
    reader = np.full(d.n_pins, -1)
    reader[d.cell_in_pins] = np.repeat(cell_level, np.diff(d.cell_in_offsets))
    seg = lambda l: np.where(l == 0, -1, (l - 1) // k)
    sinks = np.ones(d.n_pins, bool)
    sinks[d.net_pins[d.net_offsets[:-1]]] = False                     # drivers
    is_ep = (d.pin_kind == PIN_FF_D) | (d.pin_kind == PIN_PO)
    own = lvl[net_of_pin]
    out = sinks & ((own == 0) | ((reader < 0) & ~is_ep) | ((reader >= 0) & (seg(np.maximum(reader, 0)) != seg(own))))
    kept = np.zeros(N, bool)
    kept[net_of_pin[out]] = True
    n_sinks = np.diff(d.net_offsets) - 1
    per_seg = [int(n_sinks[~kept & (lvl >= 1) & ((lvl - 1) // k == j)].sum()) for j in range((L - 2) // k + 1)]
    return int(n_sinks[kept].sum()) + max(per_seg + [0])


@pytest.mark.parametrize("k", [1, 3, 100])
def test_checkpoint_segments_backward_workspace(k):
    d = make_design(CFG0)
    g = S.Graph.from_design(d)
    g.levelize()
    up = lambda b: -(-b // 256) * 256                                 # pieces start 256-aligned
    plain = g.info()["bwd_workspace_bytes"]
    state = g.info()["fwd_state_bytes"]
    assert plain == up(32 * d.n_pins)
    g.set_checkpointing(k)
    slots = _expected_sink_slots(d, k)
    sinks = d.n_pins - d.n_nets
    assert slots == sinks if k == 100 else slots < sinks              # one segment: no reuse
    assert g.info()["bwd_workspace_bytes"] == up(32 * max(slots, 1))
    # the wire values (8 bytes per sink slot instead of per pin) follow the same slots
    recs = g.checkpointing()["record_slots"]
    assert g.info()["fwd_state_bytes"] == state - (up(64 * d.n_nets) - up(64 * recs)) \
        - (up(8 * d.n_pins) - up(8 * max(slots, 1)))
    g.set_checkpointing(0)
    assert g.info()["bwd_workspace_bytes"] == plain
    assert g.info()["fwd_state_bytes"] == state
    g.close()


@pytest.mark.parametrize("k", [1, 2, 3, 5, 100])
def test_checkpoint_frontier_counts(k):
    d = make_design(CFG0)
    g = S.Graph.from_design(d)
    with pytest.raises(S.StaError) as e:
        g.set_checkpointing(k)
    assert e.value.code == S.STA_E_STATE
    L = g.levelize()
    full = g.info()["fwd_state_bytes"]
    assert g.checkpointing() == dict(stride_levels=0, record_slots=d.n_nets, kept_nets=d.n_nets)
    g.set_checkpointing(k)
    kept, slots = _expected_checkpoint_counts(d, k)
    assert g.checkpointing() == dict(stride_levels=k, record_slots=slots, kept_nets=kept)
    assert g.info()["fwd_state_bytes"] <= full - 64 * (d.n_nets - slots) + 256
    g.set_checkpointing(-1)
    assert g.checkpointing()["stride_levels"] == int(np.ceil(np.sqrt(L - 1)))
    g.set_checkpointing(0)
    assert g.info()["fwd_state_bytes"] == full
    g.close()


def test_tune_cache_lookup_before_any_tuning():
    g = S.Graph.from_design(make_design(tiny_spec(20, 3, n_pi=3, seed=1)))
    with pytest.raises(S.StaError) as e:
        g.tune_cached()                              # not levelized
    assert e.value.code == S.STA_E_STATE
    g.levelize()
    before = g.schedule()
    assert g.tune_cached() is None                   # nothing tuned in this bucket yet
    assert g.schedule() == before
    g.close()


def test_server_rejects_bad_configuration():
    lib = S.load_library()
    h = S._P()
    for cfg in ((0, 4, 16), (1 << 30, 0, 16), (1 << 30, 65, 16), (1 << 30, 4, 0),
                (1 << 30, 4, 16, 3), (1 << 30, 4, 16, -1), (1 << 30, 4, 16, 128)):   # max_merge: 0 or 2^k <= 64
        c = S.StaServerConfig(*cfg)
        assert lib.sta_server_create(ctypes.byref(c), ctypes.byref(h)) == S.STA_E_INVALID
    assert lib.sta_submit(None, None, None) == S.STA_E_INVALID
    assert lib.sta_poll(None, 1, None) == S.STA_E_INVALID
    assert lib.sta_release(None, 1) == S.STA_E_INVALID
    assert lib.sta_server_set_max_merge(None, 2) == S.STA_E_INVALID
    lib.sta_server_destroy(None)


def test_snapshots_scale_per_call_buffers():
    g = S.Graph.from_design(make_design(tiny_spec(20, 3, n_pi=3, seed=2)))
    g.levelize()
    one = g.info()
    assert one["n_snapshots"] == 1
    g.set_snapshots(5)
    five = g.info()
    assert five["n_snapshots"] == 5
    assert five["fwd_state_bytes"] == 5 * one["fwd_state_bytes"]
    assert five["bwd_workspace_bytes"] == 5 * one["bwd_workspace_bytes"]
    for bad in (0, -1, 65536):
        with pytest.raises(S.StaError) as e:
            g.set_snapshots(bad)
        assert e.value.code == S.STA_E_INVALID
    g.close()


def test_levelization_bit_exact_wide_cells():
    from tests._designs import wide_dag
    _levelization_matches(wide_dag(seed=5))


def test_placement_loop_pin_cell_maps():
    # The placement loop's gather of pin gradients to cells (built on the host).
    import torch
    from paper_2603_28381_amd import TimingDescent
    d = make_design(tiny_spec(40, 5, n_pi=4, seed=7))
    g = S.Graph.from_design(d)
    g.levelize()
    td = TimingDescent(g, d.x, d.y, d.cell_in_offsets, d.cell_in_pins, d.cell_out_pin, device="cpu")
    idx, cell = td.idx.numpy(), td.cell.numpy()
    P, C = d.n_pins, d.n_cells
    for c in range(C):
        pins = [d.cell_out_pin[c]] + list(d.cell_in_pins[d.cell_in_offsets[c]:d.cell_in_offsets[c + 1]])
        assert sorted(p for p in idx[c] if p != P) == sorted(pins)
        assert all(cell[p] == c for p in pins)
    owned = np.zeros(P, bool)
    owned[d.cell_out_pin] = True
    owned[d.cell_in_pins] = True
    assert np.all(cell[~owned] == C)
    # pin gradients gathered per cell equal a plain loop
    gp = torch.arange(P, dtype=torch.float32) * 0.5 + 1.0
    got = torch.cat([gp, torch.zeros(1)])[td.idx].sum(1).numpy()
    for c in range(C):
        pins = [d.cell_out_pin[c]] + list(d.cell_in_pins[d.cell_in_offsets[c]:d.cell_in_offsets[c + 1]])
        assert got[c] == pytest.approx(float(sum(gp[p] for p in pins)))
    g.close()


def test_rc_tree_parents_validated():
    from dataclasses import replace
    from gen.netlist import heap_trees
    d = heap_trees(make_design(tiny_spec(30, 4, n_pi=3, seed=5, fanout_p=0.25, fanout_cap=8)))
    g = S.Graph.from_design(d)          # a valid tree per net
    g.levelize()
    star = S.Graph.from_design(replace(d, pin_parent=None))
    star.levelize()
    # the tree passes keep 32 bytes per pin in the state and 40 in the workspace
    assert g.info()["fwd_state_bytes"] >= star.info()["fwd_state_bytes"] + 32 * d.n_pins
    assert g.info()["bwd_workspace_bytes"] >= star.info()["bwd_workspace_bytes"] + 40 * d.n_pins
    g.close()
    star.close()
    off, pins = d.net_offsets, d.net_pins
    big = int(np.argmax(np.diff(off)))
    drv, s1, s2 = pins[off[big]], pins[off[big] + 1], pins[off[big] + 2]
    other = pins[off[(big + 1) % d.n_nets] + 1]
    for what, edit in (("driver with a parent", {drv: s1}), ("parent in another net", {s1: other}),
                       ("self parent", {s1: s1}), ("cycle", {s1: s2, s2: s1}), ("out of range", {s1: d.n_pins})):
        pp = d.pin_parent.copy()
        for k, v in edit.items():
            pp[k] = v
        with pytest.raises(S.StaError) as e:
            S.Graph.from_design(replace(d, pin_parent=pp))
        assert e.value.code == S.STA_E_INVALID, what


def test_rc_tree_batch_with_star_member_levelizes():
    from gen.netlist import heap_trees
    a = heap_trees(make_design(tiny_spec(30, 4, n_pi=3, seed=6)))
    b = make_design(tiny_spec(20, 3, n_pi=2, seed=7))
    g = S.Graph.batch([S.Graph.from_design(a), S.Graph.from_design(b)])
    g.levelize()
    assert g.info()["n_designs"] == 2
    g.close()


@pytest.mark.slow
def test_backward_refuses_a_sink_workspace_of_4_gib():
    # One net of 2^27 pins: 32 bytes a pin are 4 GiB, which 32-bit byte offsets do not reach; with
    # checkpointing its 2^27 - 1 sinks have the slots, 32 bytes below.
    P = 1 << 27
    kind = np.full(P, PIN_PO, np.int8)
    kind[0] = PIN_PI
    lib = make_design(tiny_spec(8, 2, n_pi=2, seed=1)).lib
    g = S.Graph(dict(n_pins=P, n_nets=1, n_cells=0, net_offsets=[0, P], net_pins=np.arange(P, dtype=np.int32),
                     cell_type=[], cell_in_offsets=[0], cell_in_pins=[], cell_out_pin=[],
                     pin_cap=np.zeros(P, np.float32), pin_kind=kind),
                dict(n_cell_types=lib.n_cell_types, arc_offsets=lib.arc_offsets, arc_unate=lib.arc_unate,
                     slew_axis=lib.slew_axis, load_axis=lib.load_axis, tables=lib.tables),
                dict(t_clk=100.0, setup=5.0, hold=2.0, pi_at=0.0, pi_slew=10.0, r_per_um=0.1, c_per_um=0.2))
    g.levelize()
    assert g.info()["bwd_workspace_bytes"] == 1 << 32

    def backward():                                  # no buffers: refused before they matter
        return S.load_library().sta_backward(g.handle, None, None, None, None, 0, 10.0, None), \
            S.load_library().sta_last_error().decode()

    code, why = backward()
    assert code == S.STA_E_INVALID and "4 GiB" in why
    g.set_checkpointing(1)
    assert "4 GiB" not in backward()[1]
    g.close()
