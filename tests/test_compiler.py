"""Host compiler (libmpk) against the task-graph oracle: dependency sets bit-exact, structure
invariants, launch-mode labels, generic DAG passes, error handling.  No GPU needed."""
import os
import random
import re

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

import paper_2512_22219_amd as M
from oracle import tgraph as TG
from synth import gen as G
from tests import graph_util as GU

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "mpk.h")).read()
    declared = set(re.findall(r"\b(mpk_[a-z_]+)\s*\(", hdr))
    assert declared == set(M.binding.SYMBOLS), declared ^ set(M.binding.SYMBOLS)
    L = M.lib()
    for name in declared:
        assert hasattr(L, name), name


def test_public_header_is_plain_c(tmp_path):
    """The boundary is a C ABI: the header must compile as C99 on its own."""
    import subprocess
    src = tmp_path / "t.c"
    src.write_text('#include "mpk.h"\nint main(void) { mpk_compile_options o = {0}; mpk_serve_config c = {0}; '
                   '(void)o; (void)c; return (int)MPK_OK; }\n')
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", "-pedantic", "-I", os.path.join(ROOT, "include"),
                           "-fsyntax-only", str(src)])


def host_graph(shape, **kw):
    kw.setdefault("host_only", 1)
    return M.compile_graph(shape, None, None, **kw)


CASES = [
    ("C1", {}, dict(fusion=0)),
    ("C1", {}, dict(fusion=7)),
    ("C1", dict(batch=3), dict(fusion=0, n_workers=16, attn_chunks=3)),
    ("C1", dict(batch=2), dict(fusion=7, n_workers=7, attn_chunks=5, tiles_pointwise=3)),
    ("C1", dict(batch=2), dict(fusion=3, n_workers=24, tiles_lm_head=100)),
    ("C2", dict(n_layers=2), dict(fusion=0)),
    ("C2", dict(n_layers=2), dict(fusion=7)),
    ("C3", dict(n_layers=1), dict(fusion=7)),
    ("C1", dict(batch=2), dict(fusion=31, n_workers=24, attn_chunks=3)),
    ("C1", dict(batch=2), dict(fusion=31, n_workers=24, attn_chunks=3, no_attn_balance=1)),
    ("C1", dict(batch=3), dict(fusion=15, n_workers=24, attn_chunks=2)),   # rope unfused: a dealt chunk task waits for every row's rope tasks
    ("C2", dict(n_layers=2), dict(fusion=31)),
    # mixture-of-experts blocks
    ("C1", dict(batch=2, ffn=0, n_experts=8, top_k=2, expert_ffn=64), dict(fusion=0, n_workers=12)),
    ("C1", dict(batch=3, ffn=0, n_experts=16, top_k=4, expert_ffn=32), dict(fusion=31, n_workers=24, tiles_moe=10)),
    ("C4", dict(n_layers=1), dict(fusion=31)),
    # batch > 4 with a long down-projection input: decomposed along the input as well
    ("C3", dict(n_layers=2), dict(fusion=31)),
    ("C1", dict(batch=8, ffn=8192), dict(fusion=31, n_workers=32)),
    # greedy sampling as an operator of the graph (multi-token launch)
    ("C1", dict(batch=3), dict(fusion=31, n_workers=24, greedy_loop=1)),
    ("C1", {}, dict(fusion=0, greedy_loop=1)),
    ("C1", dict(batch=2), dict(fusion=31, greedy_loop=1, tiles_sampling=5, tiles_lm_head=7)),   # sampling tasks that share a row
    # serving graphs (Section 6.1): the serving task first, every embedding task behind it
    ("C1", dict(batch=3), dict(fusion=31, greedy_loop=1, kv_page_size=16, kv_pages=40, serving=1)),
    ("C1", dict(batch=8), dict(fusion=31, greedy_loop=1, kv_page_size=32, kv_pages=64, serving=1, n_workers=40)),
    # QKV heads cut unevenly, 3 tiles of 43, 43, 42 rows per head: 80 heads (the 70B shape) and 48 heads
    # (the 8B shape with 240 tiles per linear operator)
    ("C5", dict(n_layers=1), dict(fusion=31)),
    ("C2", dict(n_layers=1), dict(fusion=31, tiles_linear=240)),
    # column tiles sized by the speed of the worker that runs them (workers by index mod 8)
    ("C1", dict(batch=2), dict(fusion=31, n_workers=24, worker_weight_permille=[1300, 700] * 4)),
    ("C1", dict(batch=3), dict(fusion=0, n_workers=16, worker_weight_permille=[1300, 700, 1000, 1000] * 2)),
    ("C2", dict(n_layers=2), dict(fusion=31, worker_weight_permille=[1047, 955] * 4)),
]


@pytest.mark.parametrize("base,variant,opts", CASES)
def test_dependency_sets_bit_exact_and_structure(base, variant, opts):
    shape = G.small_variant(base, **variant)
    g = host_graph(shape, **opts)
    ex = g.export()
    GU.check_structure(ex)
    C = GU.attn_chunks_of(ex, shape)
    ops, deg = GU.oracle_ops_and_degrees(shape, ex, opts.get("fusion", 0), C, not opts.get("no_attn_balance", 0))
    want = TG.producer_sets(ops, deg)
    got = GU.compiled_producer_sets(ex)
    assert TG.canonical_bytes(got) == TG.canonical_bytes(want)
    st_ = g.stats()
    assert st_["n_pair_deps"] == sum(len(p) for per in want for p in per)
    assert st_["n_tasks"] == len(ex.tasks) and st_["n_events"] == len(ex.events)


def closure_by_op_tile(psets):
    memo = {}

    def go(k):
        if k in memo:
            return memo[k]
        acc = set()
        for p in psets[k[0]][k[1]]:
            acc.add(p)
            acc |= go(p)
        memo[k] = acc
        return acc
    return {(o, t): go((o, t)) for o in range(len(psets)) for t in range(len(psets[o]))}


@pytest.mark.parametrize("base,variant,opts", CASES[:5] + CASES[8:12] + [c for c in CASES if c[2].get("serving")])
def test_transitive_reduction_keeps_closures(base, variant, opts):
    shape = G.small_variant(base, **variant)
    g = host_graph(shape, transitive_reduction=1, **opts)
    ex = g.export()
    GU.check_structure(ex)
    C = GU.attn_chunks_of(ex, shape)
    ops, deg = GU.oracle_ops_and_degrees(shape, ex, opts.get("fusion", 0), C, not opts.get("no_attn_balance", 0))
    want = TG.producer_sets(ops, deg)
    got = GU.compiled_producer_sets(ex)
    assert closure_by_op_tile(got) == closure_by_op_tile(want)
    # every kept pair is one of the oracle's direct pairs
    for o in range(len(want)):
        for t in range(len(want[o])):
            assert set(got[o][t]) <= set(want[o][t])
    assert g.stats()["n_dummy_tasks"] <= host_graph(shape, **opts).stats()["n_dummy_tasks"]


def test_simulated_execution_respects_oracle_producers():
    """Random legal interleavings of the compiled graph in the runtime simulator: every task's
    brute-force producers are finished before it runs, nothing deadlocks; and a dropped trigger
    or an out-of-order AOT queue is detected."""
    shape = G.small_variant("C1", batch=2)
    for opts in (dict(fusion=0), dict(fusion=7, transitive_reduction=1),
                 dict(fusion=7, n_sched_wgs=2)):
        g = host_graph(shape, n_workers=6, attn_chunks=3, **opts)
        ex = g.export()
        C = GU.attn_chunks_of(ex, shape)
        ops, deg = GU.oracle_ops_and_degrees(shape, ex, opts["fusion"], C, not opts.get("no_attn_balance", 0))
        want = TG.producer_sets(ops, deg)
        lin = {(int(t["op"]), int(t["tile"])): i for i, t in enumerate(ex.tasks)
               if t["op"] != GU.DUMMY}
        producers = [set() for _ in ex.tasks]
        for (o, tl), i in lin.items():
            producers[i] = {lin[p] for p in want[o][tl]}
        tasks, events, queues = GU.sim_inputs(ex)
        n_sched = int(ex.header["n_sched_wgs"]) * 4
        for seed in range(40):
            log, hops = TG.simulate(tasks, events, queues, n_sched, random.Random(seed), producers)
            assert len(log) == len(tasks)
        if opts.get("n_sched_wgs"):
            assert any(t["jit"] for t in tasks)
            assert all(hops[i] == (2 if tasks[i]["jit"] else 1) for i in range(len(tasks)))
        victim = next(i for i, t in enumerate(tasks) if t["trig"] != int(ex.header["terminal_event"]))
        with pytest.raises(TG.Deadlock):
            TG.simulate(tasks, events, queues, n_sched, random.Random(0), producers, drop_trigger=victim)
        bad = [list(q) for q in queues]
        w = next(w for w, q in enumerate(bad) if len(q) >= 2)
        bad[w][0], bad[w][-1] = bad[w][-1], bad[w][0]
        with pytest.raises((TG.Deadlock, AssertionError)):
            for seed in range(5):
                TG.simulate(tasks, events, bad, n_sched, random.Random(seed), producers)


def test_launch_mode_labels_follow_the_barrier_rule():
    """Attention is JIT; an operator downstream of a JIT operator stays JIT unless each of its
    tasks waits for all tasks of that operator (Section 5.2).  Recomputed from the oracle sets."""
    shape = G.small_variant("C1", batch=2)
    for fusion in (0, 7):
        g = host_graph(shape, n_workers=8, attn_chunks=3, n_sched_wgs=1, fusion=fusion)
        ex = g.export()
        ops, deg = GU.oracle_ops_and_degrees(shape, ex, fusion, 3)
        want = TG.producer_sets(ops, deg)
        jit = []
        for oi, op in enumerate(ops):
            if op.kind == TG.K_ATTN_PARTIAL:
                jit.append(1)
                continue
            j = 0
            for ps in want[oi]:
                per = {}
                for (po, pt) in ps:
                    per[po] = per.get(po, 0) + 1
                for po, n in per.items():
                    if jit[po] and n != deg[po][0] * deg[po][1]:
                        j = 1
            jit.append(j)
        assert list(ex.ops["jit"]) == jit
        names = [o.name for o in ops]
        assert jit[names.index("L0.attn_merge")] == 1 and jit[names.index("L0.o_proj")] == 0
        # with no scheduler every task is pre-enqueued
        ex0 = host_graph(shape, n_workers=8, attn_chunks=3, fusion=fusion).export()
        assert not ex0.tasks["jit"].any()


def test_fully_fused_8b_graph_has_no_fork_join_and_five_events_per_layer():
    """With every fusion, head-aligned QKV tiles and transitive reduction the compiled graph of
    the 8B shape is purely sequential: no dummy tasks (Section 6.5 reports none for its LLM
    graphs) and one event per operator."""
    shape = G.small_variant("C2", n_layers=3)
    g = host_graph(shape, fusion=31, transitive_reduction=1)
    s = g.stats()
    assert s["n_dummy_tasks"] == 0
    assert s["n_ops"] == 1 + 5 * 3 + 1
    ex = g.export()
    qkv = [o for o in ex.ops if o["kind"] == M.binding.OP_LINEAR and o["cols"] == 6144][0]
    # every one of the 48 heads is cut into the same number of tiles, so none straddles a head;
    # 4 per head here: the projection is small, and 64 workers stay free for the attention tasks
    assert int(qkv["tc"]) == 48 * 4
    # start and terminal events, the LM head's event, and per layer one event each for qkv, the
    # 8 attention groups, o_proj, gate_up and down
    assert s["n_events"] == 2 + 1 + 3 * (1 + 8 + 1 + 1 + 1)


def test_no_dummies_when_nothing_forks_and_paper_style_stats():
    """A purely sequential fused graph needs no normalization (Section 6.5: no fork/join groups in
    the compiled LLM graphs); event storage after linearization is 8 bytes per event."""
    shape = G.small_variant("C1", n_kv_heads=4)      # one query head per KV head
    g = host_graph(shape, fusion=7, transitive_reduction=1, attn_chunks=1, n_workers=8,
                   tiles_linear=4)
    s = g.stats()
    assert s["successor_bytes_linearized"] == 8 * s["n_events"]
    assert s["successor_bytes_unlinearized"] >= 4 * (s["n_tasks"] - 1)
    assert s["n_events_fused"] < s["n_pair_deps"]


# ------------------------------------------------------------------ generic DAG entry point
def export_as_sets(ex):
    real_in = GU.real_in_sets(ex)
    prod = {}
    for i, t in enumerate(ex.tasks):
        if t["op"] == GU.DUMMY:
            continue
        prod[int(t["tile"])] = {int(ex.tasks["tile"][p]) for p in real_in[int(t["dep_event"])]}
    return prod


def test_compile_dag_fig4_example():
    names = ["Q", "K", "V", "X", "A1", "A2", "O1", "O2", "O3", "O4", "R"]
    ix = {n: i for i, n in enumerate(names)}
    pairs = []
    for a in ("A1", "A2"):
        pairs += [(ix[s], ix[a]) for s in ("Q", "K", "V")]
        pairs += [(ix[a], ix[o]) for o in ("O1", "O2", "O3", "O4")] + [(ix[a], ix["R"])]
    pairs += [(ix["X"], ix["R"])]
    g = M.compile_dag(len(names), pairs, n_workers=4)
    s, ex = g.stats(), g.export()
    assert s["n_pair_deps"] == 17 and s["n_events_fused"] == 3 and s["n_dummy_tasks"] == 2
    GU.check_structure(ex)
    # the event that launches O1..O4 stores them as one range of four
    o_pos = sorted(i for i, t in enumerate(ex.tasks) if t["op"] != GU.DUMMY and names[t["tile"]].startswith("O"))
    assert o_pos == list(range(o_pos[0], o_pos[0] + 4))
    e = int(ex.tasks["dep_event"][o_pos[0]])
    assert (int(ex.events["first"][e]), int(ex.events["last"][e])) == (o_pos[0], o_pos[0] + 4)
    prod = export_as_sets(ex)
    assert prod[ix["R"]] == {ix["A1"], ix["A2"], ix["X"]} and prod[ix["O3"]] == {ix["A1"], ix["A2"]}


@st.composite
def random_dag(draw):
    n = draw(st.integers(2, 16))
    pairs = set()
    for b in range(1, n):
        for a in draw(st.lists(st.integers(0, b - 1), max_size=4)):
            pairs.add((a, b))
    return n, sorted(pairs)


@settings(max_examples=100, deadline=None)
@given(random_dag())
def test_compile_dag_matches_oracle_passes(gr):
    n, pairs = gr
    if not pairs:
        return
    g = M.compile_dag(n, pairs, n_workers=3)
    ex, s = g.export(), g.stats()
    GU.check_structure(ex)
    ev = TG.predecessor_set_fusion(TG.successor_set_fusion(TG.pair_events(pairs)))
    n_ev, n_tasks, dummies = TG.normalize(ev, list(range(n)))
    assert s["n_events_fused"] == len(ev)
    assert s["n_dummy_tasks"] == len(dummies)
    assert s["n_events"] == len(n_ev) + 2            # + start and terminal events
    want = {}
    for a, b in pairs:
        want.setdefault(b, set()).add(a)
    got = export_as_sets(ex)
    for t in range(n):
        assert got.get(t, set()) == want.get(t, set())


# ------------------------------------------------------------------ error handling
def test_error_paths():
    s = G.CONFIGS["C1"]
    with pytest.raises(M.MpkError) as e:
        host_graph(G.small_variant("C1", head_dim=48))
    assert e.value.status == M.binding.MPK_ERR_UNSUPPORTED
    with pytest.raises(M.MpkError) as e:
        host_graph(G.small_variant("C1", hidden=0))
    assert e.value.status == M.binding.MPK_ERR_INVALID_ARG
    with pytest.raises(M.MpkError) as e:
        host_graph(s, fusion=1 << 9)
    assert e.value.status == M.binding.MPK_ERR_INVALID_ARG
    with pytest.raises(M.MpkError) as e:
        host_graph(G.small_variant("C1", n_q_heads=3))
    assert e.value.status == M.binding.MPK_ERR_UNSUPPORTED
    cfg = M.binding.model_config(s)
    cfg.struct_size = 4
    import ctypes as C
    h = C.c_void_p()
    o = M.binding.compile_options(host_only=1)
    assert M.lib().mpk_compile(C.byref(cfg), None, None, C.byref(o), C.byref(h)) == M.binding.MPK_ERR_INVALID_ARG
    assert b"struct_size" in M.lib().mpk_last_error()
    # a host-only graph refuses to run
    g = host_graph(s)
    assert M.lib().mpk_decode_step(g._h, 1, 1, 1, None) == M.binding.MPK_ERR_INVALID_ARG
    with pytest.raises(M.MpkError):
        M.compile_dag(3, [(0, 5)])


def test_kv_batch_option_is_validated_and_leaves_the_graph_alone():
    """kv_batch only changes where a layer's cache starts: same task graph; below batch = error."""
    s = G.small_variant("C1", batch=2)
    a = host_graph(s, fusion=31).export()
    b = host_graph(s, fusion=31, kv_batch=8).export()
    assert np.array_equal(a.tasks, b.tasks) and np.array_equal(a.events, b.events)
    with pytest.raises(M.MpkError) as e:
        host_graph(s, kv_batch=1)
    assert e.value.status == M.binding.MPK_ERR_INVALID_ARG


def test_moe_error_paths_and_graph_shape():
    moe = dict(ffn=0, n_experts=8, top_k=2, expert_ffn=64)
    for bad, status in ((dict(top_k=9), M.binding.MPK_ERR_INVALID_ARG),
                        (dict(top_k=0), M.binding.MPK_ERR_INVALID_ARG),
                        (dict(expert_ffn=60), M.binding.MPK_ERR_UNSUPPORTED),
                        (dict(expert_ffn=24), M.binding.MPK_ERR_UNSUPPORTED),
                        (dict(n_experts=1024, top_k=8), M.binding.MPK_ERR_UNSUPPORTED),
                        (dict(n_experts=64, top_k=32), M.binding.MPK_ERR_UNSUPPORTED),
                        (dict(batch=16, n_experts=64, top_k=16, hidden=264), M.binding.MPK_ERR_UNSUPPORTED)):
        with pytest.raises(M.MpkError) as e:
            host_graph(G.small_variant("C1", **{**moe, **bad}))
        assert e.value.status == status, bad
    with pytest.raises(M.MpkError) as e:      # dense model with stray MoE fields
        host_graph(G.small_variant("C1", top_k=2))
    assert e.value.status == M.binding.MPK_ERR_INVALID_ARG
    g = host_graph(G.small_variant("C1", batch=2, **moe), fusion=31, n_workers=12, tiles_moe=7)
    ex = g.export()
    kinds = [int(o["kind"]) for o in ex.ops if o["layer"] == 0]
    assert kinds == [M.binding.OP_LINEAR, M.binding.OP_ATTN_PARTIAL, M.binding.OP_LINEAR, M.binding.OP_LINEAR,
                     M.binding.OP_ROUTER, M.binding.OP_EXPERT, M.binding.OP_EXPERT, M.binding.OP_COMBINE]
    per_op = {int(o["kind"]): int(o["n_tasks"]) for o in ex.ops if o["layer"] == 0}
    assert per_op[M.binding.OP_ROUTER] == 1 and per_op[M.binding.OP_EXPERT] == 7
    st_ = g.stats()
    s = G.small_variant("C1", batch=2, **moe)
    assert st_["expert_bytes"] == 3 * s.expert_ffn * s.hidden * 2
    # the selection read-back needs a device graph
    with pytest.raises(M.MpkError) as e:
        g.moe_active()
    assert e.value.status == M.binding.MPK_ERR_INVALID_ARG
    # hybrid launch labels the expert stages just-in-time and combine ahead-of-time again
    gj = host_graph(G.small_variant("C1", batch=2, **moe), fusion=31, n_workers=12, n_sched_wgs=1)
    jit = {int(o["kind"]): int(o["jit"]) for o in gj.export().ops if o["layer"] == 0}
    assert jit[M.binding.OP_EXPERT] == 1 and jit[M.binding.OP_COMBINE] == 0 and jit[M.binding.OP_ROUTER] == 0


def test_weighted_column_tiles_follow_the_worker_speeds():
    """worker_weight_permille: a linear operator's column tiles are proportional to the speed of
    the worker (index mod 8) that runs each of them; operators that are not eligible (the head-
    aligned QKV projection) keep the even split; the weights [1000] * 8 change nothing."""
    shape = G.small_variant("C2", n_layers=2)
    even = host_graph(shape, fusion=31).export()
    same = host_graph(shape, fusion=31, worker_weight_permille=[1000] * 8).export()
    assert not even.col_begin and not same.col_begin
    ex = host_graph(shape, fusion=31, worker_weight_permille=[1047, 955] * 4).export()
    assert ex.header["version"] == 2 and ex.col_begin
    worker_of = {(int(t["op"]), int(t["tile"])): int(t["worker"]) for t in ex.tasks if t["op"] != M.binding.TASK_DUMMY_OP}
    seen_kinds = set()
    for oi, op in enumerate(ex.ops):
        if oi not in ex.col_begin:
            continue
        b = ex.col_begin[oi].astype(np.int64)
        assert b[0] == 0 and b[-1] == op["cols"] and len(b) == op["tc"] + 1 and (np.diff(b) > 0).all()
        size = np.diff(b)
        fast = np.array([worker_of[(oi, i)] % 2 == 0 for i in range(int(op["tc"]))])
        # sizes follow 1047 : 955 to within the rounding of a boundary (one column either way)
        ideal = op["cols"] / op["tc"]
        assert np.all(np.abs(size[fast] - ideal * 1.047 / 1.001) <= 1.01) and np.all(np.abs(size[~fast] - ideal * 0.955 / 1.001) <= 1.01)
        seen_kinds.add(int(op["kind"]))
    assert seen_kinds == {TG.K_LINEAR, TG.K_GATEUP}     # O, down, LM head; the fused gate/up projection
    qkv = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_LINEAR and op["cols"] == (shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim]
    assert qkv and all(oi not in ex.col_begin for oi in qkv)
    # batch 3 and more runs on the matrix cores, whose tiles are made of 16-row blocks: left alone
    big = host_graph(G.small_variant("C3", n_layers=1), fusion=31, worker_weight_permille=[1047, 955] * 4).export()
    assert not big.col_begin


def test_lds_page_preload_makes_the_preloaded_tiles_larger():
    """Batch 1, all ahead-of-time: a worker that runs a QKV task and then waits through the
    attention phase pre-loads the first 16 weight rows per compute unit of its gate/up task into
    LDS pages; the gate/up tiles of those workers are 8 columns (16 rows) larger than the tiles of
    the workers that ran attention, so that all have the same amount left to stream.  8B shape:
    192 tiles of 50 columns and 64 of 42; switched off, the split is even again.  (Pages need the worker's tasks back to back, i.e. the graph
    without fork/join dummies that transitive reduction gives; its closures are compared with the
    oracle's, over these uneven tiles, in test_transitive_reduction_keeps_closures.)"""
    shape = G.small_variant("C2", n_layers=2)
    g = host_graph(shape, fusion=31, transitive_reduction=1)
    ex = g.export()
    gateup = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_GATEUP]
    assert gateup and all(oi in ex.col_begin for oi in gateup) and len(ex.col_begin) == len(gateup)
    worker_of = {(int(t["op"]), int(t["tile"])): int(t["worker"]) for t in ex.tasks if t["op"] != M.binding.TASK_DUMMY_OP}
    attn_workers = {worker_of[(oi, i)] for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_ATTN_PARTIAL
                    for i in range(int(op["n_tasks"]))}
    assert len(attn_workers) == 64
    for oi in gateup:
        size = np.diff(ex.col_begin[oi].astype(np.int64))
        ran_attention = np.array([worker_of[(oi, i)] in attn_workers for i in range(len(size))])
        assert set(size[~ran_attention]) == {50} and set(size[ran_attention]) == {42}
        assert size.sum() == shape.ffn
    assert g.stats()["lds_bytes"] == 160 * 1024
    off = host_graph(shape, fusion=31, transitive_reduction=1, no_lds_pages=1)
    assert not off.export().col_begin and off.stats()["lds_bytes"] < 160 * 1024
    # nothing of it with scheduler workgroups, per-operator launches, batch > 1 or pre-loading off
    for kw in (dict(n_sched_wgs=1), dict(launch_mode=1), dict(no_preload=1)):
        assert not host_graph(shape, fusion=31, transitive_reduction=1, **kw).export().col_begin
    assert not host_graph(G.small_variant("C2", n_layers=2, batch=2), fusion=31, transitive_reduction=1).export().col_begin


@pytest.mark.parametrize("tiles_per_expert,n_tasks", [(96, 256), (128, 256), (96, 37), (2, 9), (5, 1), (40, 512)])
def test_expert_tasks_share_the_active_tiles_disjointly_in_order_and_completely(tiles_per_expert, n_tasks):
    """Section 6.4, tasks re-balanced at run time: for every number of active experts the shares
    of the expert tasks are consecutive ranges that start at tile 0, end at the last tile and
    leave no gap; an expert boundary inside a share costs the task tiles (it is charged like 8),
    so shares differ by no more than that charge plus rounding, and a share that crosses no
    boundary is never smaller than one that does."""
    from paper_2512_22219_amd.binding import moe_task_share
    for n_active in [0, 1, 2, 3, 7, 82, 128]:
        total = n_active * tiles_per_expert
        at = 0
        sizes, crossing = [], []
        for task in range(n_tasks):
            first, last = moe_task_share(n_active, tiles_per_expert, n_tasks, task)
            assert first == at and last >= first, (n_active, task, first, last, at)
            at = last
            sizes.append(last - first)
            # expert boundaries strictly inside the share (a tile on each side of them)
            crossing.append(0 if last == first else (last - 1) // tiles_per_expert - first // tiles_per_expert)
        assert at == total
        if n_active:
            cost = [s + 8 * c for s, c in zip(sizes, crossing)]
            assert max(cost) - min(cost) <= 8 + 2, (n_active, max(cost), min(cost))
    with pytest.raises(M.MpkError):
        moe_task_share(3, tiles_per_expert, n_tasks, n_tasks)
    with pytest.raises(M.MpkError):
        moe_task_share(3, 0, n_tasks, 0)


@pytest.mark.parametrize("batch,n_kv,head_dim,max_seq,chunks", [
    (9, 16, 128, 4096, 2), (16, 12, 128, 2048, 2), (13, 16, 128, 1536, 2),   # many long rows: something for the length deal to move
    (8, 24, 128, 2048, 1), (13, 16, 64, 2048, 1), (4, 48, 128, 4096, 1),     # 16384 rows or fewer, or short rows
    (16, 16, 128, 4096, 1), (16, 24, 128, 4096, 1),                          # a pair for every worker, and more
    (8, 16, 128, 4096, 2), (5, 24, 64, 1352, 2), (1, 8, 128, 1088, 8),       # as many tasks as workers hold
])
def test_default_number_of_attention_chunks(batch, n_kv, head_dim, max_seq, chunks):
    s = G.small_variant("C1", batch=batch, n_layers=1, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=head_dim, max_seq=max_seq)
    ex = host_graph(s, fusion=31, transitive_reduction=1, n_workers=256).export()
    attn = [op for op in ex.ops if op["kind"] == TG.K_ATTN_PARTIAL]
    assert [int(op["n_tasks"]) for op in attn] == [batch * n_kv * chunks]


@pytest.mark.parametrize("batch,chunks", [(1, 16), (2, 16)])
def test_size_of_the_projections_does_not_change_the_attention_chunks(batch, chunks):
    """A chunk's length is part of the order in which a row's attention is added up: 128 cached positions
    of the largest sequence where there are workers enough, whatever else the model does."""
    for hidden in (256, 8192):
        s = G.small_variant("C5", n_layers=1, hidden=hidden, ffn=1024, vocab=1000, batch=batch)
        ex = host_graph(s, fusion=31, transitive_reduction=1, n_workers=256).export()
        attn = [op for op in ex.ops if op["kind"] == TG.K_ATTN_PARTIAL]
        assert [int(op["n_tasks"]) for op in attn] == [batch * 8 * chunks]


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5])
def test_worker_speeds_resize_the_tiles_of_the_vector_body_only(batch):
    """Batch 3 and more runs on the matrix cores, whose tasks are made of 16-row blocks (and of jobs of 512 rows)."""
    s = G.small_variant("C2", n_layers=1, batch=batch, ffn=8192)
    ex = host_graph(s, fusion=31, worker_weight_permille=[1047, 955] * 4).export()
    assert bool(ex.col_begin) == (batch <= 2)


def test_only_graphs_of_the_static_entry_point_give_up_sharded_counters_for_its_scratch_array():
    """700 small layers at batch 4: with every event's counters on 17 lines of their own the scratch of a step
    exceeds the 32 MiB array, so the plain graph keeps its narrow events unsharded; a graph that
    mpk_decode_step_static refuses anyway has no reason to."""
    s = G.small_variant("C1", batch=4, n_layers=700, max_seq=136)

    def sharded(**kw):
        ev = host_graph(s, fusion=31, transitive_reduction=1, n_workers=256, **kw).export().events
        has_producers = ev["required"] > 0
        return int(((ev["flags"] & 2) != 0)[has_producers].sum()), int(has_producers.sum())

    n, total = sharded()
    assert 0 < n < total
    for kw in (dict(greedy_loop=1), dict(kv_page_size=8, kv_pages=80), dict(debug_flags=M.binding.DEBUG_TRACE)):
        n, total = sharded(**kw)
        assert n == total


@pytest.mark.parametrize("head_dim,grp", [(64, 1), (64, 8), (128, 4), (128, 8)])
@pytest.mark.parametrize("page,max_seq", [(0, 1024), (8, 1 << 17)])
def test_lds_of_attention_tasks(head_dim, grp, page, max_seq):
    """Queries, eight wavefronts' partial outputs (a row of d + 4 per term group and head), maxima and sums, the
    appended rows and their scores, page numbers; at least 84 KB, so that one worker fits a compute unit."""
    s = G.small_variant("C1", n_layers=1, head_dim=head_dim, n_q_heads=grp, n_kv_heads=1, max_seq=max_seq)
    kw = dict(kv_page_size=page, kv_pages=100) if page else {}
    terms = 2 if grp == 8 else 3
    floats = grp * head_dim + 8 * terms * grp * (head_dim + 4) + 16 * grp + 2 * head_dim + 24 + (max_seq // page if page else 0)
    assert host_graph(s, fusion=31, n_workers=256, **kw).stats()["lds_bytes"] == max(84 * 1024, 4 * (floats + 1024 + 48))


@pytest.mark.parametrize("n_active,tiles,n_tasks", [(8, 96, 256), (1, 1, 1), (0, 96, 256), (128, 96, 256), (512, 16375, 512),
                                                    (512, 16376, 512), (512, 16377, 512), (512, 1 << 20, 512)])
def test_expert_shares_are_the_same_in_32_and_in_64_bits(n_active, tiles, n_tasks):
    """The split is worked out in 32 bits where the products fit them (experts x (tiles + 8) x tasks up to
    2^32 - 1: 512 experts of 16375 tiles for 512 tasks, not 16376), in 64 above: the same shares."""
    from paper_2512_22219_amd.binding import moe_task_share
    period = tiles + 8

    def at(task):
        q, r = divmod(n_active * period * task // n_tasks, period)
        return q * tiles + min(r, tiles)

    for task in range(n_tasks):
        assert moe_task_share(n_active, tiles, n_tasks, task) == (at(task), at(task + 1))


def _marks(shape, **opts):
    """Export and task forms of a graph for 256 workers."""
    g = host_graph(shape, **{**dict(n_workers=256), **opts})
    return g.export(), g.task_forms()


@pytest.mark.parametrize("kw,opts", [
    (dict(), dict(tiles_linear=2)), (dict(batch=2), dict(tiles_linear=2)),       # 128 outputs a task of 256 inputs
    (dict(hidden=512, batch=2), dict(n_workers=15)), (dict(hidden=512, batch=2), dict(n_workers=14)),
    (dict(hidden=1032, n_q_heads=2, n_kv_heads=1, batch=2), dict(tiles_linear=1)),     # more outputs than threads
    (dict(ffn=0, n_experts=16, top_k=4, expert_ffn=64), dict(n_workers=11)),     # every layer's residual is unmarked
    (dict(ffn=0, n_experts=16, top_k=4, expert_ffn=64, batch=2), dict(tiles_linear=3)),
    (dict(hidden=4096, n_q_heads=16, batch=2), dict(tiles_linear=2)),            # 1024 inputs: every wavefront has some
])
def test_unmarked_residuals_are_read_only_by_wavefronts_that_have_seen_the_input(kw, opts):
    """Thread i of 512 loads the residual of outputs i, i + 512, ...; wavefront w has looked at an input word only if the
    input is longer than 128 w.  A task for which the two do not match has to keep its event."""
    ex, forms = _marks(G.small_variant("C1", **kw), fusion=31, transitive_reduction=1, **opts)
    resid = (forms["marks"] & M.binding.FORM_RESIDUAL) != 0
    assert resid.any()
    for f in forms[resid]:
        if f["marks"] & M.binding.FORM_RESIDUAL_MARKED or not f["marks"] & M.binding.FORM_INPUT_MARKED:
            continue
        loads = {i % 512 // 64 for i in range(int(f["outputs"]))}
        assert all(128 * w < f["inputs"] for w in loads), f


@pytest.mark.parametrize("kw,workers,packs,larger", [
    (dict(hidden=2048, n_q_heads=16, ffn=8192), 24, False, 8),     # 5 MB of weights a worker and layer: three weight buffers, no packing
    (dict(hidden=2048, n_q_heads=16, ffn=4096), 24, True, 16),     # 2.8 MB: two rows to a row of a page, twice the rows in it
    (dict(hidden=512, ffn=4096, vocab=4093, n_q_heads=8, n_kv_heads=8), 5, False, None),   # 3.2 MB, half of it the output head
])
def test_pages_are_sized_for_the_rows_the_kernel_set_packs(kw, workers, packs, larger):
    """A page takes 16 rows of half a block, or as many times more as share a row of it; the tiles that find theirs
    in a page are larger by that, in columns of a gate/up pair."""
    ex, forms = _marks(G.small_variant("C1", **kw), fusion=31, transitive_reduction=1, n_workers=workers)
    packed = forms["packed"][forms["inputs"] > 0]
    assert (packed.max() > 1) == packs and packed.min() == 1
    gateup = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_GATEUP and oi in ex.col_begin]
    assert bool(gateup) == (larger is not None)
    for oi in gateup:
        size = np.unique(np.diff(ex.col_begin[oi].astype(np.int64)))
        assert larger <= size.max() - size.min() <= larger + 1


_DENSE = "0 4 5 13 5 15 5 5 15 5 15 1"   # embedding; QKV, attention, O, gate/up, down of two layers; head
_EVENTS = "0 0 0 8 0 8 0 0 8 0 8 0"


@pytest.mark.parametrize("kw,opts,want", [
    (dict(), {}, _DENSE),
    (dict(batch=2, hidden=2048, n_q_heads=16, n_kv_heads=2, max_seq=2624), {}, _DENSE),
    (dict(qk_norm=True), dict(greedy_loop=1), _DENSE + " 0"),
    (dict(batch=2), dict(serving=1, greedy_loop=1, kv_page_size=32, kv_pages=16), "0 " + _DENSE + " 0"),
    # the router's task reads all of the expert tasks' and the combine's input: those may go by events
    (dict(n_experts=16, top_k=4, ffn=0, expert_ffn=64), {}, "0 4 5 13 1 0 0 0 0 4 5 13 1 0 0 0 0 0"),
    # operators in between that know no marks; an event that tasks of several kinds wait for
    (dict(batch=2), dict(fusion=30), "0 0 4 5 9 0 4 9 0 4 5 9 0 4 9 0 0"),
    (dict(batch=2), dict(fusion=29), "0 4 5 1 0 4 1 0 4 5 1 0 4 1 0 0"),
    (dict(batch=2), dict(fusion=27), "0 4 5 13 1 0 12 5 5 15 1 0 12 1"),
    (dict(batch=2), dict(fusion=15), "0 0 0 0 12 5 15 1 0 0 12 5 15 1"),
    (dict(batch=2), dict(transitive_reduction=0), "0 4 5 9 0 8 0 0 8 0 12 1"),
    # a residual that nothing vouches for
    (dict(batch=2), dict(tiles_linear=2), "0 0 0 12 5 15 5 5 15 5 15 1"),
    # never: matrix-core bodies, hybrid and per-operator launches, the loop kernel's graphs
    (dict(batch=3), {}, _EVENTS), (dict(), dict(n_sched_wgs=1), _EVENTS), (dict(), dict(launch_mode=1), _EVENTS),
    (dict(), dict(greedy_loop=2), _EVENTS + " 0"),
])
def test_which_operators_go_by_the_words_of_their_input(kw, opts, want):
    """Marks of every operator in order (1 input, 2 residual, 4 output marked, 8 has a residual); all tasks of an
    operator are alike."""
    ex, forms = _marks(G.small_variant("C1", **kw), **{**dict(fusion=31, transitive_reduction=1), **opts})
    marks = [np.unique(forms["marks"][ex.tasks["op"] == oi] & 15) for oi in range(len(ex.ops))]
    assert all(len(m) == 1 for m in marks)
    assert " ".join(str(m[0]) for m in marks) == want


@pytest.mark.parametrize("kw,opts", [
    (dict(batch=2, max_seq=1024), {}), (dict(batch=2, max_seq=1024, n_q_heads=8, n_kv_heads=8), dict(n_workers=5)),
    (dict(batch=2, max_seq=1024, n_kv_heads=1), dict(n_workers=37, attn_chunks=7)), (dict(max_seq=2624), dict(n_workers=1)),
    (dict(batch=2, max_seq=1024, n_q_heads=3, n_kv_heads=3, head_dim=128), dict(transitive_reduction=0, n_workers=11, attn_chunks=6)),
    (dict(batch=2, max_seq=1024), dict(tiles_linear=5, attn_chunks=4)),      # projection tiles that straddle heads
])
def test_attention_tasks_of_a_head_are_in_the_order_of_their_chunks(kw, opts):
    """A marked sequence's last chunk merges and waits for the words of the others, wherever the lengths deal them: no
    worker may have any of those behind it.  So a head's tasks come in order of (sequence, chunk), and every
    worker's list in linearized order."""
    ex, forms = _marks(G.small_variant("C1", **kw), **{**dict(fusion=31, transitive_reduction=1), **opts})
    for w in range(len(ex.aot_off) - 1):
        mine = ex.aot[ex.aot_off[w]:ex.aot_off[w + 1]].astype(np.int64)
        assert (np.diff(mine) > 0).all()
    for oi, op in enumerate(ex.ops):
        if op["kind"] != TG.K_ATTN_PARTIAL:
            continue
        at = np.flatnonzero(ex.tasks["op"] == oi)
        place = np.empty(len(at), np.int64)
        place[ex.tasks["tile"][at]] = at
        B, n_kv = int(op["tb"]), int(kw.get("n_kv_heads", 2))
        per_head = place.reshape(B, n_kv, -1).transpose(1, 0, 2).reshape(n_kv, -1)   # [head][sequence, chunk]
        assert (np.diff(per_head, axis=1) > 0).all()


def test_activation_bytes_count_the_copies_of_marked_tensors():
    """Whole lines of 64 floats: every tensor once, in a graph with marks the marked ones twice more.  Tiny model at batch 1,
    one chunk a head: QKV, partials and merged attention, O, gate/up, down of two layers."""
    s = G.small_variant("C1")
    plain = host_graph(s, fusion=31, transitive_reduction=1, n_workers=256, launch_mode=1).stats()["act_bytes"]
    marked = host_graph(s, fusion=31, transitive_reduction=1, n_workers=256).stats()["act_bytes"]
    layer = sum(-(-n // 64) * 64 for n in (8 * 64, 4 * (64 + 2), 4 * 64, 256, 688, 256))
    assert marked - plain == 2 * 4 * 2 * layer


PAGE_CHAINS = [(dict(hidden=2056, ffn=152), 5), (dict(hidden=2056, ffn=144, n_layers=3), 5), (dict(hidden=2600, ffn=320, qk_norm=True), 13),
               (dict(hidden=256, ffn=688), 5)]


@pytest.mark.parametrize("kw,workers", PAGE_CHAINS)
def test_no_task_both_uses_its_pages_and_fills_them_for_the_next(kw, workers):
    """Few workers: a gate/up task short enough to fill its successor's pages and long enough to have some itself."""
    ex, forms = _marks(G.small_variant("C1", **kw), fusion=31, transitive_reduction=1, n_workers=workers)
    nxt, ready = (forms["marks"] & M.binding.FORM_PAGE_NEXT) != 0, (forms["marks"] & M.binding.FORM_PAGE_READY) != 0
    assert ready.any() and nxt.sum() == ready.sum() and not (nxt & ready).any()
    for w in range(workers):   # ... and every page is filled by the task before
        mine = ex.aot[ex.aot_off[w]:ex.aot_off[w + 1]]
        assert np.array_equal(nxt[mine][:-1], ready[mine][1:])


@pytest.mark.parametrize("kw,tr,tiles", [
    (dict(hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128), 1, 192),          # the workers without one of 64 attention tasks
    (dict(hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128), 0, 256),          # ... would cut the 256 tiles of the residual across
    (dict(hidden=2048, n_q_heads=16, n_kv_heads=8, head_dim=128, batch=2), 1, 128),
    (dict(hidden=2048, n_q_heads=16, n_kv_heads=8, head_dim=128, batch=2), 0, 128),   # two of them each
    (dict(hidden=2048, n_q_heads=32, n_kv_heads=4, head_dim=128, ffn=0, n_experts=128, top_k=8, expert_ffn=768), 0, 224),   # 8 combine tasks
])
def test_o_projection_beside_attention_does_not_cut_its_residual_across(kw, tr, tiles):
    """Without transitive reduction, more pairs of an O projection task and a residual tile are more dummy tasks in its way."""
    ex, forms = _marks(G.small_variant("C1", max_seq=1088, **kw), fusion=31, transitive_reduction=tr)
    attn = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_ATTN_PARTIAL]
    assert int(ex.ops[attn[1] + 1]["n_tasks"]) == tiles      # (behind layer 0's, whose residual is the embedding)


@pytest.mark.parametrize("kw,fusion,pages", [
    (dict(hidden=2048, ffn=8192, n_q_heads=32, n_kv_heads=8), 31, False),    # 64 rows a gate/up task, two a row: two half blocks
    (dict(hidden=2048, ffn=8192, n_q_heads=32, n_kv_heads=8), 7, True),
    (dict(hidden=1536, ffn=8960, n_q_heads=16, head_dim=128), 31, True),     # 70 rows
    (dict(hidden=768, ffn=12288, n_q_heads=16, n_kv_heads=4), 31, False),    # 96 rows, four a row
    (dict(hidden=768, ffn=12288, n_q_heads=16, n_kv_heads=4), 7, True),
    (dict(hidden=4096, ffn=6144, n_q_heads=32, n_kv_heads=8), 31, True),     # 48 rows, one a row
    (dict(hidden=4096, ffn=6016, n_q_heads=32, n_kv_heads=8), 31, False),    # 47
])
def test_rows_from_which_on_tasks_have_pages(kw, fusion, pages):
    ex, forms = _marks(G.small_variant("C1", max_seq=1088, **kw), fusion=fusion, transitive_reduction=1)
    gateup = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_GATEUP]
    for oi in gateup:
        assert (forms["marks"][ex.tasks["op"] == oi] & M.binding.FORM_PAGE_READY).any() == pages


RESIZED = [   # gate/up tiles larger by the rows they find in pages, and tiles of other operators that read parts of them
    (dict(hidden=504, ffn=2024, n_kv_heads=4), dict(fusion=15, n_workers=32, attn_chunks=2, tiles_linear=7)),   # ... let tasks of other operators qualify
    (dict(hidden=504, ffn=2024, n_kv_heads=4), dict(fusion=31, n_workers=32, attn_chunks=2, tiles_linear=7)),   # ... make other dependencies
    (dict(hidden=1640, ffn=1760, n_q_heads=8, n_kv_heads=4, vocab=2958), dict(fusion=27, n_workers=8)),
]


@pytest.mark.parametrize("variant,opts", RESIZED)
def test_pages_whose_tile_sizes_change_the_graph(variant, opts):
    shape = G.small_variant("C1", **variant)
    test_dependency_sets_bit_exact_and_structure("C1", variant, opts)
    ex, forms = _marks(shape, **opts)
    nxt, ready = (forms["marks"] & M.binding.FORM_PAGE_NEXT) != 0, (forms["marks"] & M.binding.FORM_PAGE_READY) != 0
    for w in range(opts["n_workers"]):
        mine = ex.aot[ex.aot_off[w]:ex.aot_off[w + 1]]
        assert np.array_equal(nxt[mine][:-1], ready[mine][1:]) and not (nxt & ready).any()
    # tiles are of even size where no task has pages
    assert ready.any() == bool(ex.col_begin)


def own_routing(shape, **opts):
    """Whether first-stage expert tasks work the routing out by themselves: the answers there are in a graph."""
    ex, forms = _marks(shape, fusion=31, transitive_reduction=1, **opts)
    own = (forms["marks"] & M.binding.FORM_OWN_ROUTING) != 0
    kind = np.array([-1 if t["op"] == GU.DUMMY else ex.ops[t["op"]]["kind"] for t in ex.tasks])
    first = np.zeros(len(own), bool)
    stages = [oi for oi, op in enumerate(ex.ops) if op["kind"] == TG.K_EXPERT]
    for oi in stages[::2]:
        first |= ex.tasks["op"] == oi
    assert not own[~first].any() and (kind[first] == TG.K_EXPERT).all() and first.any()
    return set(own[first].tolist())


@pytest.mark.parametrize("batch", [1, 2, 3, 8, 16])
def test_expert_tasks_that_work_the_routing_out_by_themselves(batch):
    kw = dict(batch=batch, hidden=272, ffn=0, top_k=2, expert_ffn=64)
    for experts in (2, 64, 127, 128, 129, 512):
        s = G.small_variant("C1", n_experts=experts, **kw)
        assert own_routing(s) == {experts <= 128}
        assert own_routing(s, launch_mode=M.binding.LAUNCH_PER_OP) == {False}
    s = G.small_variant("C1", n_experts=16, **kw)
    assert own_routing(s, n_workers=24, tiles_moe=10) == {True}       # several tasks a worker
    assert own_routing(s, n_workers=24, n_sched_wgs=1) == {False}     # hybrid launch: handed out when their event is active
    assert own_routing(s, n_workers=24, n_sched_wgs=1, force_aot=1) == {True}
    assert own_routing(s, greedy_loop=2) == own_routing(s, serving=1, greedy_loop=1, kv_page_size=32, kv_pages=64) == {True}
