"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs.  Schedules must match bit-exactly; every node value, node gradient and parameter
gradient must agree within 1e-4 relative to the largest magnitude of its tensor."""
import sys

import numpy as np
import pytest

from oracle import schedule as S
from oracle.interp import Oracle
from paper_1705_07860_amd import workloads as wl
from tests.helpers import rel_err, segment_rel_err

pytestmark = pytest.mark.gpu

TOL = 1e-4   # max_i |gpu_i - ref_i| <= TOL * max_i |ref_i| per tensor (fp32 path vs fp64 oracle)


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run_gpu(p, g, mode, launch=0, arena=2 << 30, n_nodes=None, fuse=2, labels=None):
    """The arena starts as NaN, so that rows which nobody writes do not hold what an earlier run of the same graph left there."""
    import torch
    from paper_1705_07860_amd import binding as ob
    c = ob.Context(arena_bytes=arena, mode=mode, launch=launch)
    c._arena.fill_(255)
    torch.cuda.synchronize()      # (the context has a stream of its own)
    c.set_fusion(int(fuse))
    pids = c.params_create(p)
    assert pids == list(range(len(p.mats)))
    c.param_grad_zero()
    c.add_bulk(g)
    if labels is not None:
        c.set_manual_batches(labels)
    root = g.root if n_nodes is None else n_nodes - 1
    c.forward(root)
    return c, root


def check_against_oracle(c, p, g, o, root, tol=TOL, what=""):
    n = o.n
    total = int(o.v_off[-1])
    vals = c.all_read(0, total)      # (also when the values lie in several evaluation stages)
    ev = segment_rel_err(vals, o.val[:total], o.v_off)
    say(f"  {what} values: worst tensor rel err {ev:.2e}")
    assert ev <= tol
    c.backward(root)
    grads = c.all_read(1, total)
    eg = segment_rel_err(grads, o.grad[:total], o.v_off)
    say(f"  {what} node gradients: worst tensor rel err {eg:.2e}")
    assert eg <= tol
    worst = 0.0
    for pid, m in enumerate(p.mats):
        got = c.param_grad_read(pid, m.shape)
        e = rel_err(got, o.param_grad(pid))
        worst = max(worst, e)
        assert e <= tol, (p.names[pid], e)
    say(f"  {what} parameter gradients: worst tensor rel err {worst:.2e}")
    loss = c.value_read(root, 1)[0]
    assert abs(loss - o.value(root)[0]) <= tol * abs(o.value(root)[0])


# ------------------------------------------------------------------ scheduler stages

@pytest.mark.parametrize("name", ["rnn", "tagger", "tagger_char", "tree", "parser"])
def test_schedule_bit_exact(name, workload_cache):
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    say(f"schedule {name}: n={g.n} E={g.n_edges}")
    c, root = run_gpu(p, g, ob.OB_BYDEPTH)
    depth = c.debug_read(ob.OB_DBG_DEPTH)
    assert np.array_equal(depth.astype(np.int64), S.depths(g))
    succ_off = c.debug_read(ob.OB_DBG_SUCC_OFF).astype(np.int64)
    succ_edge = c.debug_read(ob.OB_DBG_SUCC_EDGE).astype(np.int64)
    ref_edge = np.argsort(g.in_idx, kind="stable")
    assert np.array_equal(succ_edge, ref_edge)
    assert np.array_equal(np.diff(succ_off), np.bincount(g.in_idx, minlength=g.n))
    bo, ids, bd, sig = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo)
    assert np.array_equal(ids, rids)
    assert np.array_equal(bd, rbd)
    st = c.stats()
    say(f"  steps={st['n_steps']} slots={st['n_slots']} batches={st['n_batches']} sched {st['ms_schedule']:.3f} ms "
        f"fwd {st['ms_forward']:.3f} ms launches(sched)={st['n_launch_sched']}")
    c.close()


@pytest.mark.parametrize("name", ["rnn", "tagger", "tagger_char", "tree", "parser"])
def test_agenda_schedule_bit_exact_and_parity(name, workload_cache):
    """Agenda-based batching (Section 3.2): the GPU schedule equals the reference agenda schedule
    bit for bit, and values and gradients still match the oracle."""
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    c, root = run_gpu(p, g, ob.OB_BYAGENDA)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbs = S.by_agenda(g)
    assert np.array_equal(bo, rbo)
    assert np.array_equal(ids, rids)
    assert np.array_equal(bd, rbs)
    st = c.stats()
    say(f"agenda {name}: batches={st['n_batches']} slots={st['n_slots']} sched {st['ms_schedule']:.3f} ms")
    check_against_oracle(c, p, g, o, root, what=f"{name}/agenda")
    c.close()


@pytest.mark.parametrize("seed", range(6))
def test_agenda_schedule_random_dags(seed):
    from paper_1705_07860_amd import binding as ob
    p, g = wl.random_dag(700 + seed, n_nodes=30 + 40 * seed, dim=4 + 2 * (seed % 3))
    c, root = run_gpu(p, g, ob.OB_BYAGENDA, arena=64 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbs = S.by_agenda(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbs)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    check_against_oracle(c, p, g, o, root, what=f"agenda dag{seed}")
    c.close()


@pytest.mark.parametrize("seed", range(6))
def test_schedule_bit_exact_random_dags(seed):
    from paper_1705_07860_amd import binding as ob
    p, g = wl.random_dag(500 + seed, n_nodes=30 + 40 * seed, dim=4 + 2 * (seed % 3))
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    check_against_oracle(c, p, g, o, root, what=f"dag{seed}")
    c.close()


@pytest.mark.parametrize("seed", range(8))
def test_random_dags_with_wider_rows(seed):
    """Rows of 16 .. 64 elements take the float4 paths and larger weights make some predictions
    confident: a PICK_NLS value close to zero (and the gradients behind it) must still be right
    relative to its own size, which the kernels get from log1p of the sum without the maximum and
    from the label's gradient as minus the sum of the other probabilities."""
    from paper_1705_07860_amd import binding as ob
    dim = (16, 32, 48, 64)[seed % 4]
    p, g = wl.random_dag(920 + seed, n_nodes=60 + 25 * (seed % 7), dim=dim)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=256 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    check_against_oracle(c, p, g, o, root, what=f"wide dag{seed} (dim {dim})")
    c.close()


def test_nobatch_schedule_is_one_node_per_batch(workload_cache):
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache("rnn")
    c, root = run_gpu(p, g, ob.OB_NOBATCH, arena=64 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.no_batching(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, root, what="rnn/nobatch")
    c.close()


# ------------------------------------------------------------------ values and gradients

def expected_uncopied_concats(g, bo, ids):
    """Which CONCAT batches of a schedule need no copy, from the rule alone (plain loops over the graph): at most
    four pieces, each a multiple of four wide; every reader of every node is a matrix product; and in every batch
    of products that reads one, all CONCAT operands have the piece widths of the lowest CONCAT batch among them.
    Returns (number of batches, number of elements)."""
    bo, ids = np.asarray(bo), np.asarray(ids)
    batch_of = np.empty(g.n, np.int64)
    for b in range(len(bo) - 1):
        batch_of[ids[bo[b]:bo[b + 1]]] = b
    pieces = lambda v: tuple(int(g.out_dim[u]) for u in g.in_idx[g.in_off[v]:g.in_off[v + 1]])
    cat_batches = [b for b in range(len(bo) - 1) if g.op[ids[bo[b]]] == wl.OP_CONCAT]
    ok = {b: len(pieces(ids[bo[b]])) <= 4 and all(w % 4 == 0 for w in pieces(ids[bo[b]])) for b in cat_batches}
    readers = {}                                      # product batch -> CONCAT operand nodes
    for v in range(g.n):
        for u in g.in_idx[g.in_off[v]:g.in_off[v + 1]]:
            if g.op[u] == wl.OP_CONCAT:
                if g.op[v] == wl.OP_MATVEC:
                    readers.setdefault(int(batch_of[v]), []).append(int(u))
                else:
                    ok[int(batch_of[u])] = False
    for mb, cats in readers.items():
        ref = min(int(batch_of[u]) for u in cats)
        if not ok[ref] or any(pieces(u) != pieces(ids[bo[ref]]) for u in cats):
            for u in cats:
                ok[int(batch_of[u])] = False
    good = [b for b in cat_batches if ok[b]]
    return len(good), int(sum((bo[b + 1] - bo[b]) * g.out_dim[ids[bo[b]]] for b in good))


@pytest.mark.parametrize("name", ["rnn", "tagger", "tagger_char", "tree", "parser"])
def test_values_and_gradients_by_depth(name, workload_cache):
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    say(f"parity {name}: n={g.n}")
    c, root = run_gpu(p, g, ob.OB_BYDEPTH)
    st = c.stats()
    bo, ids, _, _ = c.schedule_read()
    n_cat = int(np.sum(g.op[np.asarray(ids)[np.asarray(bo[:-1])]] == wl.OP_CONCAT))
    want = expected_uncopied_concats(g, bo, ids)
    say(f"  {n_cat} CONCAT batches, {want[0]} of them ({want[1]} elements) need no copy; "
        f"{st['n_view_batches']} SLICE batches are views")
    assert (st["n_uncopied_batches"], st["uncopied_floats"]) == want
    assert st["n_view_batches"] == int(np.sum(g.op[np.asarray(ids)[np.asarray(bo[:-1])]] == wl.OP_SLICE))
    check_against_oracle(c, p, g, o, root, what=name)
    st = c.stats()
    say(f"  sched {st['ms_schedule']:.3f} ms fwd {st['ms_forward']:.3f} ms bwd {st['ms_backward']:.3f} ms "
        f"(param grads {st['ms_param_grads']:.3f}) launches fwd={st['n_launch_fwd']} bwd={st['n_launch_bwd']}")
    # the backward step kernel alone: everything but the root kernel and the (at most three) deferred parameter kernels
    assert 0 < st["n_launch_bwd_steps"] <= st["n_launch_bwd"] - 2 and st["n_launch_bwd"] - st["n_launch_bwd_steps"] <= 4
    assert st["n_depth_retries"] == 0
    c.close()


@pytest.mark.parametrize("name", ["rnn", "tagger", "parser"])
def test_without_launch_fusion(name, workload_cache):
    """One launch per depth level (fusion off) gives the same schedule and the same numbers."""
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=False)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    st = c.stats()
    assert st["n_slots"] == st["n_steps"]
    check_against_oracle(c, p, g, o, root, what=f"{name}/nofuse")
    c.close()


@pytest.mark.parametrize("name", ["rnn", "tagger_char", "tree"])
def test_early_placement_and_launch_plan_invariants(name, workload_cache):
    """Fusion level 1 (every batch launched as early as possible) and level 2 (as late as possible)
    keep the schedule, give the same numbers (so no batch ran before a producer), and produce
    launch plans in which every batch appears in exactly one chain and the slots are ordered."""
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    rbo, rids, rbd = S.by_depth(g)
    slots = {}
    for level in (1, 2):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level)
        bo, ids, bd, _ = c.schedule_read()
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
        ch = c.debug_read(ob.OB_DBG_CHAINS).reshape(-1, 12)
        st = c.stats()
        assert int(ch[:, 1].sum()) == st["n_batches"]                      # members partition the batches
        assert np.array_equal(ch[:, 0], np.concatenate([[0], np.cumsum(ch[:, 1])[:-1]]))
        assert np.all(np.diff(ch[:, 2].astype(np.int64)) >= 0) and int(ch[-1, 2]) == st["n_slots"] - 1
        slots[level] = st["n_slots"]
        check_against_oracle(c, p, g, o, root, what=f"{name}/placement{level}")
        c.close()
    assert slots[1] == slots[2]     # both placements keep the longest dependency path


@pytest.mark.parametrize("rows,H,q", [(20, 32, 2), (37, 16, 2), (16, 64, 1), (45, 8, 4)])
def test_small_gated_cells_at_every_fusion_level(rows, H, q):
    """Cells whose matrix product has q = 1, 2 or 4 segments of H columns, with a row count that
    leaves a ragged last tile: h' = z * h + tanh(n) style cells over `rows` chains, three steps.
    Every launch-fusion level gives bit-identical results and matches the oracle."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(rows * 100 + H)
    pb = wl.ParamBuilder(rng, std=0.3)
    W = pb.add("W", q * H, H)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    hs = [gb.input(rng.standard_normal(H)) for _ in range(rows)]
    for _step in range(3):
        for i in range(rows):
            s_ = gb.add((gb.input(rng.standard_normal(q * H)), gb.matvec(W, -1, hs[i])))
            if q == 1:
                hs[i] = gb.tanh(s_)
            elif q == 2:
                z = gb.sigmoid(gb.slice(s_, 0, H))
                hs[i] = gb.add((gb.cmult(z, hs[i]), gb.tanh(gb.slice(s_, H, 2 * H))))
            else:
                i_, f_, o_ = (gb.sigmoid(gb.slice(s_, k * H, (k + 1) * H)) for k in range(3))
                c_ = gb.add((gb.cmult(f_, hs[i]), gb.cmult(i_, gb.tanh(gb.slice(s_, 3 * H, 4 * H)))))
                hs[i] = gb.cmult(o_, gb.tanh(c_))
    root = gb.add([gb.sqnorm(h) for h in hs])
    g = gb.finish(root, rows)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(o.v_off[-1])
    out = {}
    for level in (0, 1, 2):
        c, _ = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level, arena=128 << 20)
        st = c.stats()
        vals = c.all_read(0, total)
        c.backward(g.root)
        out[level] = (vals, c.all_read(1, total), c.param_grad_read(W, p.mats[W].shape), st["n_launch_fwd"])
        c.close()
    say(f"  rows {rows} H {H} q {q}: forward launches {out[0][3]} / {out[1][3]} / {out[2][3]}")
    assert out[2][3] <= out[0][3]
    for k in range(3):
        assert np.array_equal(out[0][k], out[2][k]) and np.array_equal(out[1][k], out[2][k])
    c, root_ = run_gpu(p, g, ob.OB_BYDEPTH, fuse=2, arena=128 << 20)
    check_against_oracle(c, p, g, o, root_, what=f"gated cells q={q}")
    c.close()


def _state_recurrence(H, rows, steps, late=False):
    """Cells whose gates do not depend on the output of the step before (only their states are carried on), so that the cells of
    all steps hang together by component-wise operations.  late: row r begins behind r operations of its own."""
    rng = np.random.default_rng(H + rows)
    pb = wl.ParamBuilder(rng, std=0.4)
    W, b = pb.add("W", 4 * H, H), pb.add("b", 4 * H, 1)
    p = pb.done()
    g = wl.GraphBuilder(p)
    losses = []
    for r in range(rows):
        c = g.input(rng.standard_normal(H))
        for _ in range(r if late else 0):
            c = g.tanh(c)
        for _ in range(steps):
            s = g.add((g.matvec(W, b, g.input(rng.standard_normal(H))), g.input(rng.standard_normal(4 * H))))
            i, f, o, cand = (g.slice(s, k * H, (k + 1) * H) for k in range(4))
            c = g.add((g.cmult(g.sigmoid(f), c), g.cmult(g.sigmoid(i), g.tanh(cand))))
            losses.append(g.sqnorm(g.cmult(g.sigmoid(o), g.tanh(c))))
    return p, g.finish(g.add(losses), rows)


def _cell_graph(H, nf, sums, rows, odd, seed=5):
    """Steps of gated cells with nf forget gates over `rows` rows; sums: the gates are slices of a sum of two rows (of one row
    otherwise).  odd: what keeps a row's cell from being one, or is unusual and must not."""
    rng = np.random.default_rng(seed)
    pb = wl.ParamBuilder(rng, std=0.4)
    D = (3 + nf) * H
    W, U, b = pb.add("W", D, H), pb.add("U", D, H), pb.add("b", D, 1)
    p = pb.done()
    g = wl.GraphBuilder(p)
    hs = [g.input(rng.standard_normal(H)) for _ in range(rows)]
    cs = [[g.input(rng.standard_normal(H)) for _ in range(max(nf, 1))] for _ in range(rows)]
    losses = []
    at = list(rng.permutation(3 + nf))          # the gates' places in the sum
    for step in range(3):
        for r in range(rows):
            s = g.matvec(U, b, hs[r])
            if sums:
                s = g.add((g.matvec(W, -1, g.input(rng.standard_normal(H))), s))
            sl = [g.slice(s, int(k) * H, (int(k) + 1) * H) for k in at]
            i, cand, o = g.sigmoid(sl[0]), g.tanh(sl[1]), g.sigmoid(sl[2])
            f = [g.sigmoid(x) for x in sl[3:]]
            terms = [g.cmult(cs[r][k], f[k]) if odd == "swapped" else g.cmult(f[k], cs[r][k]) for k in range(nf)]
            terms.insert(min(nf, 1), g.cmult(cand, i) if odd == "swapped" else g.cmult(i, cand))
            c = g.add(terms) if nf else terms[0]
            tc = g.tanh(c)
            h = g.cmult(tc, o) if odd == "swapped" else g.cmult(o, tc)
            if odd == "gate read" and r == rows - 1:
                losses.append(g.sqnorm(i))
            if odd == "state read" and r % 2 == 0:
                losses.append(g.sqnorm(c))
            if odd == "output read":
                losses.append(g.sqnorm(g.add((h, h))))
            cs[r] = [c] + [g.input(rng.standard_normal(H)) for _ in range(nf - 1)] if nf else cs[r]
            hs[r] = h
            if odd in ("four readers", "five readers"):
                losses += [g.sqnorm(g.tanh(h)), g.sqnorm(g.sigmoid(h)), g.sqnorm(g.cmult(h, g.input(rng.standard_normal(H))))]
            if odd == "five readers":
                losses.append(g.sqnorm(g.add((h, g.input(rng.standard_normal(H))))))
            if odd == "three readers":
                losses.append(g.sqnorm(g.tanh(h)))
                losses.append(g.sqnorm(g.sigmoid(h)))
    root = g.add(losses + [g.sqnorm(h) for h in hs] + [g.sqnorm(g.tanh(c[0])) for c in cs])
    return p, g.finish(root, rows)


@pytest.mark.parametrize("H,nf,sums,rows,odd,cells", [
    (2, 1, True, 3, "", True), (25, 1, True, 9, "", True), (64, 1, True, 5, "swapped", True), (65, 1, True, 6, "three readers", True),
    (100, 2, True, 7, "", True), (128, 0, False, 4, "", True), (130, 0, True, 5, "swapped", True), (192, 2, False, 3, "", True),
    (256, 1, True, 16, "output read", True), (300, 1, True, 3, "", True), (20, 2, True, 21, "swapped", True),
    (32, 1, True, 6, "four readers", True), (32, 1, True, 6, "five readers", False),
    (32, 1, True, 6, "gate read", False), (32, 1, True, 6, "state read", False), (1, 1, True, 4, "", False)])
def test_gated_cells(H, nf, sums, rows, odd, cells):
    """LSTM and tree-LSTM cells are worked row by row from one record: bit for bit what one launch per level gives, in one
    evaluation and in two, and within tolerance of the oracle; a chain with a cell that is read in other ways is not, nor one with
    more than four readers of an output."""
    from paper_1705_07860_amd import binding as ob
    p, g = _cell_graph(H, nf, sums, rows, odd)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(o.v_off[-1])
    out = {}
    for level in (0, 1, 2):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level, arena=128 << 20)
        kinds = c.debug_read(ob.OB_DBG_CHAINS).reshape(-1, 12)[:, 3]
        n_cells = int(np.sum(kinds == 3))
        say(f"  level {level}: {n_cells} chains of cells of {kinds.size} chains")
        if level != 1:      # (placed early, what reads an output joins its chain; the last step's may be joined in any case)
            assert (n_cells >= 2 if cells else n_cells == 0) if level else n_cells == 0, kinds
        c.backward(root)
        out[level] = [c.all_read(0, total), c.all_read(1, total)] + [c.param_grad_read(k, m.shape) for k, m in enumerate(p.mats)]
        if level == 2:
            for cut in (None, g.n * 2 // 3):      # in one evaluation, and in two: gradients arrive from the second one
                c.graph_new()
                c.param_grad_zero()
                c.add_bulk(g)
                if cut:
                    c.forward(cut)
                c.forward(g.root)
                check_against_oracle(c, p, g, o, g.root, what=f"cells {H} {nf} {odd} {'in two stages' if cut else ''}")
        c.close()
    for k in range(len(out[0])):
        assert np.array_equal(out[0][k], out[1][k]) and np.array_equal(out[0][k], out[2][k]), k


@pytest.mark.parametrize("H,rows", [(36, 9), (1040, 2)])
def test_gradients_of_products_are_there_when_asked_for(H, rows):
    """A product with one reader that passes its gradient on has no row of its own written by the backward pass: nodes asked
    for by themselves (rows of more than 4 096 elements come in two pieces), all at once, and again after another backward pass on
    other values, also of two evaluations."""
    import torch
    from paper_1705_07860_amd import binding as ob
    for cut in (False, True):
        out = []
        for seed in (3, 4):
            p, g = _cell_graph(H, 1, True, rows, "")
            g.payload[:] = np.random.default_rng(seed).standard_normal(g.payload.size).astype(np.float32)
            out.append((p, g, Oracle(g, p, "f64")))
        c = ob.Context(arena_bytes=512 << 20)
        c._arena.fill_(255)
        torch.cuda.synchronize()
        c.params_create(out[0][0])
        for p, g, o in out:
            o.forward()
            o.backward(g.root)
            total = int(o.v_off[-1])
            products = np.nonzero(g.op == wl.OP_MATVEC)[0]
            c.graph_new()
            c.param_grad_zero()
            c.add_bulk(g)
            if cut:
                c.forward(g.n * 2 // 3)
            c.forward(g.root)
            c.backward(g.root)
            alone = [c.grad_read(int(v), int(g.out_dim[v])) for v in products]
            every = c.all_read(1, total)
            assert segment_rel_err(every, o.grad[:total], o.v_off) <= TOL
            for v, row in zip(products, alone):
                lo, hi = int(o.v_off[v]), int(o.v_off[v + 1])
                assert np.array_equal(row.view(np.uint32), every[lo:hi].view(np.uint32))
                assert np.array_equal(c.grad_read(int(v), hi - lo).view(np.uint32), row.view(np.uint32))
        c.close()


@pytest.mark.parametrize("H,cells", [(956, True), (972, False)])
def test_gated_cells_of_rows_on_both_sides_of_what_a_chain_may_hold(H, cells):
    """A chain becomes one of cells if a group of all its rows fits the LDS copy of an interpreted one: 17 H floats for a cell
    with one forget gate whose sum is its own, of 16 384.  Wider cells are interpreted, with the same bits."""
    from paper_1705_07860_amd import binding as ob
    p, g = _cell_graph(H, 1, True, 2, "")
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(o.v_off[-1])
    out = []
    for level in (0, 2):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level, arena=1 << 30)
        kinds = c.debug_read(ob.OB_DBG_CHAINS).reshape(-1, 12)[:, 3]
        assert bool(np.any(kinds == 3)) == (cells and level > 0)
        check_against_oracle(c, p, g, o, root, what=f"cells of {H} columns, level {level}")
        out.append([c.all_read(0, total), c.all_read(1, total)] + [c.param_grad_read(k, m.shape) for k, m in enumerate(p.mats)])
        c.close()
    for x, y in zip(*out):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


@pytest.mark.parametrize("mode", ["agenda", "manual by agenda", "manual by depth"])
@pytest.mark.parametrize("graph", ["cells", "swapped", "state carried on", "behind products", "uneven"])
def test_gated_cells_in_agenda_and_manual_plans(graph, mode):
    """Batches that were put together by other rules than depth: chains of cells occur there too, and their values and gradients
    have the bits of a launch per batch.  "state carried on" and "uneven" (rows start their steps at different depths):
    the cells of all steps hang together by their states, so that an output and a cell that reads its state may come into one
    batch; no chain there is one of cells alone."""
    from paper_1705_07860_amd import binding as ob
    if graph == "cells":
        p, g = _cell_graph(64, 1, True, 7, "")
    elif graph == "swapped":
        p, g = _cell_graph(20, 2, True, 11, "swapped")
    elif graph == "state carried on":
        p, g = _state_recurrence(24, 6, 5)
    elif graph == "uneven":
        p, g = _state_recurrence(40, 9, 4, late=True)
    else:
        p, g, _ = _cells_behind_products(32, 32, 21, 2, "sum")
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(o.v_off[-1])
    labels = None
    if mode != "agenda":
        labels = labels_of(*(S.by_agenda if mode == "manual by agenda" else S.by_depth)(g)[:2])
    out = {}
    for level in (0, 1, 2):
        c, root = run_gpu(p, g, ob.OB_BYAGENDA if mode == "agenda" else ob.OB_MANUAL, fuse=level, arena=256 << 20, labels=labels)
        kinds = c.debug_read(ob.OB_DBG_CHAINS).reshape(-1, 12)[:, 3]
        check_against_oracle(c, p, g, o, root, what=f"{graph}/{mode}/level {level}")
        if level == 2 and graph == "behind products":
            st = c.stats()
            say(f"  {st['n_launch_fwd']} forward launches of {st['n_slots']} slots")
            assert st["n_launch_fwd"] < st["n_slots"]
        out[level] = [int(np.sum(kinds == 3)), c.all_read(0, total), c.all_read(1, total)] + [c.param_grad_read(k, m.shape) for k, m in enumerate(p.mats)]
        c.close()
    say(f"  {graph}/{mode}: chains of cells {[out[k][0] for k in out]}")
    if graph in ("cells", "behind products"):
        assert out[1][0] >= 2 and out[2][0] >= 2
    for level in (1, 2):
        for x, y in zip(out[0][1:], out[level][1:]):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


def _cells_behind_products(H, K, rows, dirs, first, steps=4):
    """Steps of LSTM cells over `rows` rows, one less from step to step, and `dirs` directions; also the last node of every step."""
    rng = np.random.default_rng(H + rows)
    pb = wl.ParamBuilder(rng, std=0.3)
    U = [pb.add(f"U{k}", 4 * H, K) for k in range(dirs)]
    b = [pb.add(f"b{k}", 4 * H, 1) if k != 1 else -1 for k in range(dirs)]
    E = pb.add("E", K, H) if K != H else None
    p = pb.done()
    g = wl.GraphBuilder(p)
    at = rng.permutation(4)
    h = [[g.input(rng.standard_normal(K)) for _ in range(dirs)] for _ in range(rows)]
    c = [[g.input(rng.standard_normal(H)) for _ in range(dirs)] for _ in range(rows)]
    losses, ends = [], []
    for step in range(steps):
        for r in range(rows - step):          # (rows end one by one: the operand rows are not evenly spaced)
            r = r if step < 2 else r + 1
            for k in range(dirs):
                x = g.input(rng.standard_normal(4 * H))
                y = g.matvec(U[k], b[k], h[r][k])
                s = g.add((x, y) if first == "sum" else (y, x))
                sl = [g.slice(s, int(q) * H, (int(q) + 1) * H) for q in at]
                i, f, o, cand = g.sigmoid(sl[0]), g.sigmoid(sl[1]), g.sigmoid(sl[2]), g.tanh(sl[3])
                c[r][k] = g.add((g.cmult(f, c[r][k]), g.cmult(i, cand)))
                out = g.cmult(o, g.tanh(c[r][k]))
                h[r][k] = out if E is None else g.matvec(E, -1, out)
                if step == steps - 1:
                    losses.append(g.sqnorm(out))
        ends.append(len(g.op) - 1)
    return p, g.finish(g.add(losses), rows), ends


@pytest.mark.parametrize("H,K,rows,dirs,first", [(1, 1, 5, 1, "sum"), (2, 7, 31, 2, "sum"), (8, 8, 32, 1, "product"), (9, 9, 33, 2, "product"),
                                                (100, 100, 70, 2, "sum"), (256, 256, 40, 3, "sum"), (33, 600, 6, 1, "sum")])
def test_cells_behind_products_in_one_launch(H, K, rows, dirs, first):
    """Cells that add rows of the products before them to others run in the products' launch, the products of all directions
    together, in tiles of 32 rows and eight columns of each gate: values and gradients have the bits of a launch per batch.
    K: what the products read, the outputs themselves or (K != H) another product of them."""
    from paper_1705_07860_amd import binding as ob
    p, gr, _ = _cells_behind_products(H, K, rows, dirs, first)
    o = Oracle(gr, p, "f64")
    o.forward()
    o.backward(gr.root)
    out = {}
    for level in (2, 1, 0):
        ctx, root = run_gpu(p, gr, ob.OB_BYDEPTH, fuse=level, arena=512 << 20)
        check_against_oracle(ctx, p, gr, o, root, what=f"cells behind products {H} {rows} level {level}")
        total = int(gr.out_dim.sum())
        out[level] = [ctx.all_read(0, total), ctx.all_read(1, total)] + [ctx.param_grad_read(q, m.shape) for q, m in enumerate(p.mats)]
        st = ctx.stats()
        if level > 0 and H > 1:       # (a single column is no cell; a step whose products have other work beside them keeps its two launches)
            assert st["n_launch_fwd"] < st["n_slots"], (level, st["n_launch_fwd"], st["n_slots"])
        ctx.close()
    for level in (1, 2):
        for x, y in zip(out[0], out[level]):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


@pytest.mark.parametrize("H,rows,dirs,reader", [(2, 3, 1, ""), (16, 16, 1, "late"), (17, 17, 2, "late"), (40, 49, 1, "beside"), (33, 261, 1, "late"),
                                                (64, 292, 2, ""), (256, 20, 1, "both")])
def test_cells_worked_in_the_tiles_of_the_products_behind_them(H, rows, dirs, reader):
    """Backward, cells whose outputs are a product's operands are worked in the tiles of the product's dX (of 16 x 16, from 256 rows
    on 32 x 32), the others of their slot (rows end one by one) beside them: the bits of a launch per batch.  reader: what else reads the
    outputs; with a component-wise reader or a second product beside the first the two slots keep their launches."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(H + rows)
    pb = wl.ParamBuilder(rng, std=0.3)
    U = [pb.add(f"U{k}", 4 * H, H) for k in range(dirs)]
    Q = pb.add("Q", 4 * H, H)
    p = pb.done()
    g = wl.GraphBuilder(p)
    h = [[g.input(rng.standard_normal(H)) for _ in range(dirs)] for _ in range(rows)]
    c = [[g.input(rng.standard_normal(H)) for _ in range(dirs)] for _ in range(rows)]
    losses, outs = [], []
    for step in range(4):
        for r in range(rows - step):
            for k in range(dirs):
                x = g.input(rng.standard_normal(4 * H))
                if reader == "both":
                    x = g.matvec(Q, -1, h[r][k])
                s = g.add((x, g.matvec(U[k], -1, h[r][k])))
                if reader == "beside" and step:
                    s = g.add((s, g.concat([g.tanh(h[r][k])] * 4)))
                i, f, o, cand = (g.slice(s, q * H, (q + 1) * H) for q in range(4))
                c[r][k] = g.add((g.cmult(g.sigmoid(f), c[r][k]), g.cmult(g.sigmoid(i), g.tanh(cand))))
                h[r][k] = g.cmult(g.sigmoid(o), g.tanh(c[r][k]))
                outs.append(h[r][k])
    if reader == "late":
        losses = [g.sqnorm(g.tanh(v)) for v in outs]
    else:
        losses = [g.sqnorm(g.tanh(v)) for row in h for v in row]
    gr = g.finish(g.add(losses), rows)
    o = Oracle(gr, p, "f64")
    o.forward()
    o.backward(gr.root)
    total = int(gr.out_dim.sum())
    out = []
    for level in (0, 1, 2):
        ctx, root = run_gpu(p, gr, ob.OB_BYDEPTH, fuse=level, arena=512 << 20)
        check_against_oracle(ctx, p, gr, o, root, what=f"cells before products {H} {rows} level {level}")
        out.append([ctx.all_read(0, total), ctx.all_read(1, total)] + [ctx.param_grad_read(q, m.shape) for q, m in enumerate(p.mats)])
        st = ctx.stats()
        ctx.close()
    say(f"  {st['n_launch_bwd_steps']} backward launches of {st['n_slots']} slots")
    assert (st["n_launch_bwd_steps"] < st["n_slots"]) == (reader in ("", "late")), (st["n_launch_bwd_steps"], st["n_slots"])
    for level in (1, 2):
        for x, y in zip(out[0], out[level]):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


def _states_through_matrices(H, rows, reads):
    """Two LSTM steps whose cells share their batches; rows then go on through their output h, or (a decoder started from an encoder's
    state) through their state c and a fresh state, and end a step later.  reads, for the rows that go on through c: what h is read by
    ("late": a loss at the end, "unread", "also": a product of the same slot); "all": every row goes on through c."""
    rng = np.random.default_rng(H + rows)
    pb = wl.ParamBuilder(rng, std=0.3)
    U, V, Q = pb.add("U", 4 * H, H), pb.add("V", 4 * H, H), pb.add("Q", 4 * H, H)
    p = pb.done()
    g = wl.GraphBuilder(p)
    losses = []
    for r in range(rows):
        h, c = g.input(rng.standard_normal(H)), g.input(rng.standard_normal(H))
        late = []
        for step in range(4):
            through_c = step == 2 and (r % 3 == 1 or reads == "all")
            if through_c:
                x = g.matvec(Q, -1, h) if reads == "also" else g.input(rng.standard_normal(4 * H))
                if reads == "late":
                    late.append(h)
                s = g.add((x, g.matvec(V, -1, c)))
                c = g.input(rng.standard_normal(H))
            else:
                s = g.add((g.input(rng.standard_normal(4 * H)), g.matvec(U, -1, h)))
            i, f, o, cand = (g.slice(s, q * H, (q + 1) * H) for q in range(4))
            c = g.add((g.cmult(g.sigmoid(f), c), g.cmult(g.sigmoid(i), g.tanh(cand))))
            h = g.cmult(g.sigmoid(o), g.tanh(c))
        losses += [g.sqnorm(g.tanh(v)) for v in late + [h]]
    return p, g.finish(g.add(losses), rows)


@pytest.mark.parametrize("H,rows,reads", [(20, 7, "late"), (20, 7, "unread"), (16, 9, "also"), (64, 33, "all"), (33, 400, "late"), (40, 270, "all")])
def test_products_that_read_the_state_of_a_cell(H, rows, reads):
    """A product of the slot behind a cell may read the cell's state c instead of its output h: its dX is no gradient of h, and the cell
    must not be worked in its tiles.  Against the oracle, and the bits of a launch per batch, in every batching mode."""
    from paper_1705_07860_amd import binding as ob
    p, g = _states_through_matrices(H, rows, reads)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(g.out_dim.sum())
    bo, ids, _ = S.by_depth(g)
    labels = np.zeros(g.n, np.int64)
    labels[ids] = np.repeat(np.arange(len(bo) - 1), np.diff(bo))
    for mode in (ob.OB_BYDEPTH, ob.OB_BYAGENDA, ob.OB_MANUAL):
        out = []
        for level in (0, 1, 2):
            c, root = run_gpu(p, g, mode, fuse=level, arena=512 << 20, labels=labels if mode == ob.OB_MANUAL else None)
            check_against_oracle(c, p, g, o, root, what=f"states through matrices {H} {rows} {reads} mode {mode} level {level}")
            out.append([c.all_read(0, total), c.all_read(1, total)] + [c.param_grad_read(q, m.shape) for q, m in enumerate(p.mats)])
            c.close()
        for level in (1, 2):
            for x, y in zip(out[0], out[level]):
                assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


def _products_of_one_slot(K, rows, slices, m=21):
    """`rows` products with 200 to a matrix, half of them behind an operation more: one slot if they are placed late, two if not."""
    rng = np.random.default_rng(K + rows)
    pb = wl.ParamBuilder(rng, std=0.3)
    E = pb.add("E", 50, K)
    Ws = [pb.add(f"W{j}", m, K) for j in range(-(-rows // 200))]
    p = pb.done()
    g = wl.GraphBuilder(p)
    losses = []
    for r in range(rows):
        j = r // 200
        x = g.tanh(g.lookup(E, r % 50))
        y = g.matvec(Ws[j], -1, g.tanh(x) if j % 2 else x)
        losses.append(g.sqnorm(g.tanh(g.slice(y, 3, m - 1) if slices else y)))
    return p, g.finish(g.add(losses), rows)


@pytest.mark.parametrize("K,rows,m", [(64, 8191, 21), (64, 8192, 21), (33, 15887, 21), (33, 15888, 21), (128, 4095, 260), (128, 4096, 260),
                                      (64, 16400, 21)])
@pytest.mark.parametrize("slices", [True, False])
def test_dx_tiles_on_both_sides_of_a_large_slot(K, rows, m, slices):
    """A slot with 524 288 elements of dX and more has the larger dX tiles whatever its batches are (of 200 rows and fewer here, which
    otherwise have the smaller ones), in graphs with slices (in which a plan looks for gated cells) and without: ragged in rows and
    columns, against the oracle, and with the bits of the unfused plan, whose slots of half the size have the smaller tiles (but
    for the last shape, where they are large enough, too)."""
    from paper_1705_07860_amd import binding as ob
    p, gr = _products_of_one_slot(K, rows, slices, m)
    o = Oracle(gr, p, "f64")
    o.forward()
    o.backward(gr.root)
    total = int(gr.out_dim.sum())
    out = []
    for level in (0, 2):
        c, root = run_gpu(p, gr, ob.OB_BYDEPTH, fuse=level, arena=1 << 30)
        check_against_oracle(c, p, gr, o, root, what=f"dX of {rows} x {K} slices {slices} level {level}")
        edge = 32 if rows * K // (1 if level else 2) >= 524288 else 16
        batches = [200] * (rows // 200) + [rows % 200]
        assert c.stats()["n_tiles_bwd_dx"] == sum(-(-b // edge) * -(-K // edge) for b in batches)
        out.append([c.all_read(1, total)] + [c.param_grad_read(q, x.shape) for q, x in enumerate(p.mats)])
        c.close()
    for x, y in zip(*out):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


@pytest.mark.parametrize("rows,m,K,grid", [(20, 256, 40, True), (64, 128, 33, True), (128, 64, 130, True), (255, 32, 256, True), (96, 96, 96, False),
                                           (250, 48, 64, True), (512, 256, 20, True), (300, 200, 48, False), (700, 100, 16, False), (1, 1, 1, False),
                                           (290, 70, 300, False)])
def test_order_of_product_tiles(rows, m, K, grid):
    """Two products of each shape in one slot: every tile is there once, in whichever order, and (grid: the XCDs divide the product evenly)
    the tiles that workgroups eight apart take, one XCD's, are some rows times some columns of tiles."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(rows)
    pb = wl.ParamBuilder(rng, std=0.3)
    E, Ws = pb.add("E", 50, K), [pb.add(f"W{j}", m, K) for j in range(2)]
    p = pb.done()
    g = wl.GraphBuilder(p)
    gr = g.finish(g.add([g.sqnorm(g.tanh(g.matvec(Ws[r % 2], -1, g.lookup(E, r % 50)))) for r in range(2 * rows)]), rows)
    c, root = run_gpu(p, gr, ob.OB_BYDEPTH, arena=256 << 20)
    tiles = c.debug_read(ob.OB_DBG_TILES_FWD).reshape(-1, 40)
    o = Oracle(gr, p, "f64")
    o.forward()
    o.backward(gr.root)
    check_against_oracle(c, p, gr, o, root, what=f"tiles of {rows} x {m} x {K}")     # (dX: a tile that is missing leaves NaN)
    c.close()
    edge = 64 if rows >= 256 else 32
    ntr, ntn = -(-rows // edge), -(-m // edge)
    products = tiles[tiles[:, 0] == wl.OP_MATVEC]
    assert len(products) == 2 * ntr * ntn
    for pos0 in np.unique(products[:, 4]):
        t = products[products[:, 4] == pos0, 17].astype(int)
        assert sorted(t) == list(range(ntr * ntn))
        for x in range(8 if grid else 0):
            mine = t[x::8]
            assert mine.size == np.unique(mine // ntn).size * np.unique(mine % ntn).size


def test_dx_tiles_of_a_large_slot_do_not_depend_on_the_arena():
    """The tables for gated cells are left out where an arena has no room for them; the larger dX tiles are not."""
    from paper_1705_07860_amd import binding as ob
    p, g = _products_of_one_slot(32, 16400, True, m=6)
    tiles = []
    for arena in (_smallest_arena(p, g, 2, most=512 << 20), 1 << 30):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=arena)
        tiles.append(c.stats()["n_tiles_bwd_dx"])
        c.close()
    assert tiles == [82 * 7] * 2, tiles


@pytest.mark.parametrize("rows", [257, 258, 259, 260])
def test_cells_behind_products_of_256_rows(rows):
    """From 256 rows on, products of 64 columns and more are worked in larger tiles and keep a launch of their own; narrower
    ones do not.  Six steps of `rows` rows and fewer, of which the second to the fifth may be one launch."""
    from paper_1705_07860_amd import binding as ob
    for H in (15, 16):
        p, g, _ = _cells_behind_products(H, H, rows, 1, "sum", steps=6)
        o = Oracle(g, p, "f64")
        o.forward()
        o.backward(g.root)
        total = int(o.v_off[-1])
        out = []
        for level in (0, 2):
            c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level, arena=512 << 20)
            check_against_oracle(c, p, g, o, root, what=f"{rows} rows, H {H}, level {level}")
            st = c.stats()
            out.append([c.all_read(0, total), c.all_read(1, total)] + [c.param_grad_read(k, m.shape) for k, m in enumerate(p.mats)])
            c.close()
        say(f"  rows {rows}, H {H}: {st['n_launch_fwd']} launches of {st['n_slots']} slots")
        assert st["n_slots"] - st["n_launch_fwd"] == sum(H < 16 or rows - step < 256 for step in (1, 2, 3, 4))
        for x, y in zip(*out):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))


@pytest.mark.parametrize("H,rows,first", [(24, 37, "sum"), (64, 33, "product")])
def test_cells_behind_products_in_a_later_evaluation(H, rows, first):
    """The same where the graph is evaluated a step or two at a time: the later evaluations, whose first products read copies of
    earlier outputs, run products and cells together too, and gradients arrive from the evaluations behind them."""
    from paper_1705_07860_amd import binding as ob
    p, g, ends = _cells_behind_products(H, H, rows, 1, first, steps=6)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for cuts in ((ends[0],), (ends[1],), (ends[0], ends[2])):
        c, _ = run_gpu(p, g, ob.OB_BYDEPTH, arena=512 << 20, n_nodes=cuts[0] + 1)
        for cut in cuts[1:] + (g.root,):
            c.forward(cut)
            st = c.stats()
            say(f"  up to node {cut}: stage {st['n_stages']}, {st['n_launch_fwd']} launches of {st['n_slots']} slots")
            assert st["n_stages"] > 1 and st["n_launch_fwd"] < st["n_slots"]
        check_against_oracle(c, p, g, o, g.root, what=f"cells behind products cut at {cuts}")
        c.close()


@pytest.mark.parametrize("seed", range(950, 964))
def test_random_dags_of_400_nodes(seed):
    """Unstructured graphs of 400 nodes, consecutive seeds, nothing left out: some of these graphs
    hold softmax rows so confident that their loss is below 1e-20 (seed 953: 9.5e-25), and values
    and gradients still agree with the reference to 1e-4 of their own size at every fusion level."""
    from paper_1705_07860_amd import binding as ob
    dim = (32, 64)[seed % 2]
    p, g = wl.random_dag(seed, n_nodes=400, dim=dim)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for level in (2, 0):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=level, arena=256 << 20)
        check_against_oracle(c, p, g, o, root, what=f"dag {seed} level {level}")
        c.close()


@pytest.mark.parametrize("name", ["tagger", "tree"])
def test_hipgraph_launch_matches(name, workload_cache):
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, launch=ob.OB_LAUNCH_GRAPH)
    check_against_oracle(c, p, g, o, root, what=f"{name}/hipgraph")
    st = c.stats()
    say(f"  graph build {st['ms_graph_build']:.3f} ms fwd {st['ms_forward']:.3f} bwd {st['ms_backward']:.3f}")
    c.close()


def test_nobatch_matches_on_a_small_tagger():
    from paper_1705_07860_amd import binding as ob
    p = wl.tagger_params()
    g = wl.tagger_minibatch(p, seed=31, lengths=[3, 6, 1])
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_NOBATCH, arena=512 << 20)
    check_against_oracle(c, p, g, o, root, what="tagger3/nobatch")
    c.close()


def test_runs_are_bit_identical(workload_cache):
    """No atomics on floating point anywhere: two runs give the same bits."""
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache("tree")
    outs = []
    for _ in range(2):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH)
        total = int(o.v_off[-1])
        c.backward(root)
        outs.append((c.all_read(0, total).copy(), c.all_read(1, total).copy(),
                     [c.param_grad_read(i, m.shape).copy() for i, m in enumerate(p.mats)]))
        c.close()
    assert np.array_equal(outs[0][0], outs[1][0])
    assert np.array_equal(outs[0][1], outs[1][1])
    for a, b in zip(outs[0][2], outs[1][2]):
        assert np.array_equal(a, b)


# ------------------------------------------------------------------ edge cases

def test_edge_cases_single_node_and_prefix_forward():
    from paper_1705_07860_amd import binding as ob
    p = wl.rnn_params()
    # a one-node graph
    c = ob.Context(arena_bytes=16 << 20)
    c.params_create(p)
    x = c.add_input(np.arange(1, 2, dtype=np.float32))
    c.forward(x)
    assert c.value_read(x, 1)[0] == 1.0
    c.backward(x)
    assert c.grad_read(x, 1)[0] == 1.0
    # extending an evaluated graph keeps what is evaluated; the next forward evaluates the new node only
    y = c.add_input(np.full(1, 2.5, dtype=np.float32))
    assert c.value_read(x, 1)[0] == 1.0
    with pytest.raises(ob.ObError) as e:
        c.value_read(y, 1)                           # no value yet
    assert e.value.code == -1
    c.forward(y)
    assert c.value_read(x, 1)[0] == 1.0 and c.value_read(y, 1)[0] == 2.5
    st = c.stats()
    assert (st["n_stages"], st["n_nodes"], st["n_proxies"]) == (2, 1, 0)
    with pytest.raises(ob.ObError) as e:
        c.grad_read(x, 1)                            # the gradient of the shorter graph is gone
    assert e.value.code == -6
    c.backward(y)                                    # over the two evaluation stages as they are
    assert c.stats()["n_stages"] == 2
    assert c.grad_read(y, 1)[0] == 1.0 and c.grad_read(x, 1)[0] == 0.0
    # graph_new starts over; forward of a prefix evaluates only ids <= node
    c.graph_new()
    g = wl.rnn_minibatch(p, seed=5, lengths=[2, 4])
    c.add_bulk(g)
    first_sq = int(np.nonzero(g.op == wl.OP_SQNORM)[0][0])
    c.forward(first_sq)
    o = Oracle(g, p, "f64", n_nodes=first_sq + 1)
    o.forward()
    o.backward(first_sq)
    total = int(o.v_off[-1])
    assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL
    c.param_grad_zero()
    c.backward(first_sq)
    assert segment_rel_err(c.all_read(1, total), o.grad[:total], o.v_off) <= TOL
    with pytest.raises(ob.ObError) as e:
        c.backward(first_sq - 1)                     # not a scalar
    assert e.value.code == -4
    with pytest.raises(ob.ObError) as e:
        c.value_read(g.n - 1, 1)                     # beyond the evaluated prefix
    assert e.value.code == -1
    with pytest.raises(ob.ObError) as e:
        c.value_read(0, 3)                           # capacity too small
    assert e.value.code == -3
    c.close()


def _wide_sum_graph(n_leaves=60500):
    """A sum over more than 60 000 one-element leaves (some behind a tanh): a node of that arity
    takes the scheduler off its partitioned depth pass onto the single-workgroup one."""
    p = wl.Params([], [])
    rng = np.random.default_rng(77)
    gb = wl.GraphBuilder(p)
    xs = [gb.input(rng.standard_normal(1)) for _ in range(n_leaves)]
    ts = [gb.tanh(x) for x in xs[:200]]
    ss = [gb.sigmoid(t) for t in ts[:50]]
    root = gb.add(ss + ts[50:] + xs[200:])
    return p, gb.finish(root, 1)


@pytest.mark.parametrize("mode", ["depth", "agenda"])
def test_single_workgroup_depth_pass_on_a_very_wide_sum(mode):
    """The fallback depth pass (taken for nodes with 60 000 or more operands) leaves everything the
    later stages read intact: schedule bit-exact and values / gradients right in depth and in
    agenda mode."""
    from paper_1705_07860_amd import binding as ob
    p, g = _wide_sum_graph()
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH if mode == "depth" else ob.OB_BYAGENDA, arena=1 << 30)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = (S.by_depth if mode == "depth" else S.by_agenda)(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    assert c.stats()["n_depth_retries"] == 0
    check_against_oracle(c, p, g, o, root, what=f"wide sum/{mode}")
    c.close()


@pytest.mark.parametrize("name,mode", [("tagger", "depth"), ("parser", "agenda")])
def test_depth_pass_that_gives_up_is_repeated_with_the_single_workgroup_pass(name, mode, workload_cache):
    """With no idle polls allowed, every id range of the partitioned depth pass that has to wait for
    a lower range gives up at once (all kernels still end normally).  The library then schedules
    again with the single-workgroup pass instead of reporting a cycle, and the result is the same
    schedule."""
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache(name)
    c = ob.Context(arena_bytes=2 << 30, mode=ob.OB_BYDEPTH if mode == "depth" else ob.OB_BYAGENDA)
    c.debug_set(ob.OB_DBG_SET_DEPTH_SPIN, 0)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(g.root)
    st = c.stats()
    say(f"  {name}/{mode}: depth retries {st['n_depth_retries']}")
    assert st["n_depth_retries"] == 1
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = (S.by_depth if mode == "depth" else S.by_agenda)(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, g.root, what=f"{name}/{mode} after a depth retry")
    c.close()


@pytest.mark.parametrize("graph", ["rnn", "cells", "dag 1024", "dag 2048", "sums"])
def test_small_plan_that_gives_up_is_repeated_with_the_single_workgroup_pass(graph, workload_cache):
    """The same for graphs that are planned in one launch.  A node that was given up on takes its id as its step there, and the
    stages behind it plan what comes of that before the host sees the error: with a wave that finds nothing to do at its
    first look giving up, for graphs of both sides of a thread's second node, lists of twelve operands and gated cells."""
    from paper_1705_07860_amd import binding as ob
    if graph == "rnn":
        p, g, _ = workload_cache("rnn")
    elif graph == "cells":
        p, g = _cell_graph(20, 1, True, 12, "")
    elif graph == "sums":
        p, g = _sum_recurrences(1, 100, 12)
    else:
        p, g = _dag_of(int(graph[4:]), 7, 6)
    assert 64 < g.n <= 2048 and g.n_edges <= 4096
    o = Oracle(g, p, "f64")
    o.forward()
    if g.out_dim[g.root] == 1:
        o.backward(g.root)
    c = ob.Context(arena_bytes=256 << 20, mode=ob.OB_BYDEPTH)
    c.debug_set(ob.OB_DBG_SET_DEPTH_SPIN, 0)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(g.root)
    assert c.stats()["n_depth_retries"] == 1
    for got, want in zip(c.schedule_read(), S.by_depth(g)):
        assert np.array_equal(got, want)
    check_against_oracle(c, p, g, o, g.root, what=f"{graph} after a depth retry")
    c.close()


def test_backward_from_a_one_row_matrix_product_with_one_consumer():
    """A prefix backward whose root is a 1-element MATVEC node with exactly one plain consumer: the
    root's gradient is the seed, not the (zero) gradient row of its consumer."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(5)
    pb = wl.ParamBuilder(rng, std=0.5)
    W1 = pb.add("W1", 8, 6)
    w = pb.add("w", 1, 8)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    x = gb.input(rng.standard_normal(6))
    h = gb.tanh(gb.matvec(W1, -1, x))
    y = gb.matvec(w, -1, h)                      # 1 element, one consumer below
    z = gb.add((y, gb.input(np.ones(1))))
    g = gb.finish(z, 1)
    o = Oracle(g, p, "f64", n_nodes=y + 1)
    o.forward()
    o.backward(y)
    c = ob.Context(arena_bytes=64 << 20)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(z)
    c.backward(y)
    for v in (y, h, x):
        assert rel_err(c.grad_read(v, int(g.out_dim[v])), o.node_grad(v)) <= TOL, v
    for pid, m in enumerate(p.mats):
        assert rel_err(c.param_grad_read(pid, m.shape), o.param_grad(pid)) <= TOL
    assert c.grad_read(z, 1)[0] == 0.0           # not an ancestor of the root
    c.close()


def test_rows_with_differing_consumers_four_columns_at_a_time():
    """Batches whose rows have different consumer edges (so no tile of them is uniform) and whose width is a
    multiple of 4 take the backward routine that works four columns per thread straight from the edge list:
    slices at bounds that are not multiples of 4 (a range may cut the four columns), views as operands of
    tanh / sigmoid / products, labels among the four columns, fan-out that differs from row to row."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(77)
    pb = wl.ParamBuilder(rng, std=0.4)
    W = pb.add("W", 8, 12)
    E = pb.add("E", 11, 12)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for i in range(23):
        x = gb.lookup(E, i % 11) if i % 3 else gb.input(rng.standard_normal(12))      # 12 wide
        s = gb.slice(x, 3, 11)                          # 8 wide, bounds not multiples of 4
        t = gb.tanh(s)
        parts = [gb.sqnorm(t)]
        if i % 2:
            parts.append(gb.sqnorm(gb.cmult(gb.sigmoid(s), t)))     # one more consumer of s and of t on odd rows
        if i % 3 == 0:
            parts.append(gb.pick_nls(s, i % 8))                      # a label among s's columns
        if i % 4 == 1:
            parts.append(gb.sqnorm(gb.slice(x, 0, 4)))               # another range of the same row
        y = gb.matvec(W, -1, x)                         # 8 wide
        if i % 5:
            parts.append(gb.pick_nls(y, i % 8))
        if i % 2 == 0:
            parts.append(gb.sqnorm(gb.add((y, s))))
        losses += parts
    g = gb.finish(gb.add(losses), 23)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for mode, fuse in ((ob.OB_BYDEPTH, 2), (ob.OB_BYDEPTH, 0), (ob.OB_BYAGENDA, 2)):
        c, root_ = run_gpu(p, g, mode, fuse=fuse, arena=128 << 20)
        check_against_oracle(c, p, g, o, root_, what=f"differing consumers/{mode}/fuse {fuse}")
        c.close()


@pytest.mark.parametrize("other", ["none", "tanh", "cmult", "slice", "odd offset", "sqnorm"])
def test_consumer_lists_of_every_length_read_four_at_a_time(other):
    """Rows whose lists of consumers differ are read four edges at a time: lists of 1 to 24 plain edges with one of another kind at each
    place, and lists of that kind alone, the bits of a launch per batch."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(24)
    pb = wl.ParamBuilder(rng, std=0.4)
    E = pb.add("E", 50, 8)
    p = pb.done()
    g = wl.GraphBuilder(p)
    losses = []

    def reader(x, kind):
        y = g.input(rng.standard_normal(8))
        if kind == "tanh":
            z = g.tanh(x)
        elif kind == "cmult":
            z = g.cmult(y, x)
        elif kind == "slice":
            z = g.slice(x, 1, 7)
        elif kind == "odd offset":
            z = g.concat((g.slice(y, 0, 3), x))
        elif kind == "sqnorm":
            losses.append(g.sqnorm(x))
            return
        else:
            z = g.add((x, y))
        losses.append(g.sqnorm(z))

    for r in range(49):
        x = g.lookup(E, r)
        for k in range(1 + r % 24):
            reader(x, other if r >= 24 and (k == (5 * r) % (1 + r % 24) or r >= 45) else "add")
    gr = g.finish(g.add(losses), 1)
    o = Oracle(gr, p, "f64")
    o.forward()
    o.backward(gr.root)
    out = []
    for level in (0, 2):
        c, root = run_gpu(p, gr, ob.OB_BYDEPTH, fuse=level, arena=128 << 20)
        check_against_oracle(c, p, gr, o, root, what=f"lists with {other} level {level}")
        out.append(c.param_grad_read(E, (50, 8)))
        c.close()
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))


@pytest.mark.parametrize("mode", ["depth", "agenda", "nobatch"])
def test_slices_are_views_of_their_operand_rows(mode):
    """SLICE nodes are never copied: readers are pointed at the range of the operand's row.  Covers
    slices of slices, ranges that are not multiples of 4, slices of leaves and of matrix products,
    slices read by every kind of consumer (including the per-row reductions, which need the slice's
    own values in the backward pass), a slice as the operand of a shared-weight product (its rows
    feed the weight gradient), fan-out from one row into overlapping slices, and reading a slice's
    value and gradient back."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(8)
    pb = wl.ParamBuilder(rng, std=0.4)
    W = pb.add("W", 12, 10)
    b = pb.add("b", 12, 1)
    U = pb.add("U", 5, 6)
    E = pb.add("E", 9, 10)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for i in range(7):
        x = gb.input(rng.standard_normal(10)) if i % 2 else gb.lookup(E, i)
        y = gb.matvec(W, b, x)                       # 12
        s1 = gb.slice(y, 1, 11)                      # 10, unaligned
        s2 = gb.slice(s1, 2, 8)                      # 6: slice of a slice = y[3:9)
        s3 = gb.slice(y, 4, 12)                      # overlaps s1
        s4 = gb.slice(x, 3, 9)                       # slice of a leaf
        t = gb.tanh(s2)
        m = gb.cmult(gb.sigmoid(s4), s2)
        z = gb.matvec(U, -1, s2)                     # a view as GEMM operand (dW reads its rows)
        cat = gb.concat((s3, t, gb.slice(s3, 0, 4)))
        losses += [gb.sqnorm(s1), gb.pick_nls(s3, i % 8), gb.sqnorm(gb.add((m, t))), gb.pick_nls(z, i % 5),
                   gb.sqnorm(cat), gb.sqnorm(gb.slice(cat, 5, 9))]
    root = gb.add(losses)
    g = gb.finish(root, 7)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    m_ = {"depth": ob.OB_BYDEPTH, "agenda": ob.OB_BYAGENDA, "nobatch": ob.OB_NOBATCH}[mode]
    for fuse in ((2, 0) if mode == "depth" else (2,)):
        c, root_ = run_gpu(p, g, m_, fuse=fuse, arena=128 << 20)
        check_against_oracle(c, p, g, o, root_, what=f"slice views/{mode}/fuse {fuse}")
        for v in np.nonzero(g.op == wl.OP_SLICE)[0][:9]:
            assert rel_err(c.value_read(int(v), int(g.out_dim[v])), o.value(int(v))) <= TOL
            assert rel_err(c.grad_read(int(v), int(g.out_dim[v])), o.node_grad(int(v))) <= TOL
        st = c.stats()
        c.close()
    say(f"  slice views/{mode}: {st['n_batches']} batches, {st['n_tiles_fwd']} forward tiles")


def _concat_graph(rows, H, seed=21):
    """Rows of a small network in which CONCAT nodes of every kind feed shared matrices: two, three and four
    pieces (leaves, component-wise results, views, a piece used twice), a batch of products that mixes
    CONCAT operands with plain ones, a single-piece CONCAT, a piece that starts off a 16-byte boundary, and
    the cases that must still be copied (five pieces, a piece width that is no multiple of 4, a CONCAT that
    something other than a product reads, two piece structures into one batch of products)."""
    rng = np.random.default_rng(seed)
    pb = wl.ParamBuilder(rng, std=0.3)
    M = max(H, 12)
    E = pb.add("E", 9, H)
    Wy = pb.add("Wy", 2 * H + 4, H)
    by = pb.add("by", 2 * H + 4, 1)
    W1 = pb.add("W1", M, H)
    W2 = pb.add("W2", M, 2 * H)
    b2 = pb.add("b2", M, 1)
    W2c = pb.add("W2c", M, 2 * H)
    W2n = pb.add("W2n", M, 3 * H + 4)
    W3 = pb.add("W3", M, 3 * H)
    W3b = pb.add("W3b", M, 3 * H)
    W4 = pb.add("W4", M, 4 * H)
    b4 = pb.add("b4", M, 1)
    W5 = pb.add("W5", M, 5 * H)
    W6 = pb.add("W6", M, 16)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses, kinds = [], {k: [] for k in ("c1", "c2", "c3", "c4", "cu", "c5", "c6", "cn", "cd")}
    for i in range(rows):
        a = gb.tanh(gb.lookup(E, i % 9))
        b = gb.input(rng.standard_normal(H))
        y = gb.matvec(Wy, by, b)                      # 2H + 4
        s = gb.slice(y, 4, 4 + H)                     # a view, 16-byte aligned
        su = gb.slice(y, 2, 2 + H)                    # a view that starts off a 16-byte boundary
        c1 = gb.concat((a,))
        c2 = gb.concat((a, b)) if i % 2 == 0 else gb.input(rng.standard_normal(2 * H))
        c3 = gb.concat((a, s, b))
        c4 = gb.concat((a, b, s, a))
        cu = gb.concat((su, a))
        c5 = gb.concat((a, b, a, b, a))
        c6 = gb.concat((gb.slice(y, 0, 6), gb.slice(y, 6, 16)))
        cn = gb.concat((b, y))                        # also read by a tanh: copied
        cd = gb.concat((a, gb.slice(y, 0, 2 * H))) if i % 2 else gb.concat((gb.slice(y, 0, 2 * H), a))
        for k, v in (("c1", c1), ("c3", c3), ("c4", c4), ("cu", cu), ("c5", c5), ("c6", c6), ("cn", cn), ("cd", cd)):
            kinds[k].append(v)
        if i % 2 == 0:
            kinds["c2"].append(c2)
        outs = [gb.matvec(W1, -1, c1), gb.matvec(W2, b2, c2), gb.matvec(W3, -1, c3), gb.matvec(W4, b4, c4),
                gb.matvec(W2c, -1, cu), gb.matvec(W5, -1, c5), gb.matvec(W6, -1, c6), gb.matvec(W2n, -1, cn),
                gb.matvec(W3b, -1, cd)]
        losses += [gb.sqnorm(t) for t in outs[:-2]] + [gb.pick_nls(outs[-2], i % M), gb.pick_nls(outs[-1], (3 * i) % M)]
        losses.append(gb.sqnorm(gb.tanh(cn)))
    root = gb.add(losses)
    return p, gb.finish(root, rows), kinds


@pytest.mark.parametrize("mode,rows,H", [("depth", 7, 8), ("agenda", 7, 8), ("nobatch", 5, 8), ("depth", 300, 64)])
def test_concats_that_only_products_read_are_not_copied(mode, rows, H):
    """Section 3.3 (operands that already lie in memory are used where they are): a CONCAT batch whose only
    readers are matrix products is not written by the forward pass; the products read every row's pieces from
    the rows of their producers, and so do the weight-gradient tiles.  Values, gradients and parameter
    gradients against the oracle, bit-identical to the run that copies every CONCAT, which batches stay
    uncopied, and reading such a node's value (its row is filled in on demand)."""
    from paper_1705_07860_amd import binding as ob
    p, g, kinds = _concat_graph(rows, H)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    total = int(o.v_off[-1])
    m_ = {"depth": ob.OB_BYDEPTH, "agenda": ob.OB_BYAGENDA, "nobatch": ob.OB_NOBATCH}[mode]
    say(f"  concat graph: {g.n} nodes, mode {mode}, {rows} rows, H {H}")
    c, root = run_gpu(p, g, m_, arena=512 << 20)
    st = c.stats()
    uncopied = sum(len(kinds[k]) * w for k, w in (("c1", H), ("c2", 2 * H), ("c3", 3 * H), ("c4", 4 * H), ("cu", 2 * H)))
    if mode == "nobatch":
        uncopied += len(kinds["cd"]) * 3 * H      # one product per batch: no second piece structure in any batch
    assert st["uncopied_floats"] == uncopied, (st["uncopied_floats"], uncopied)
    bo, ids, _, _ = c.schedule_read()
    assert (st["n_uncopied_batches"], st["uncopied_floats"]) == expected_uncopied_concats(g, bo, ids)
    if mode == "depth":
        assert st["n_uncopied_batches"] == 5
    v = kinds["c3"][-1]
    assert rel_err(c.value_read(int(v), 3 * H), o.value(int(v))) <= TOL       # filled in when asked for
    check_against_oracle(c, p, g, o, root, what=f"concat in place/{mode}")
    vals, grads = c.all_read(0, total), c.all_read(1, total)
    pg = [c.param_grad_read(pid, m.shape) for pid, m in enumerate(p.mats)]
    c.close()
    # the same graph with every CONCAT copied: same bits everywhere
    c = ob.Context(arena_bytes=512 << 20, mode=m_)
    c.debug_set(ob.OB_DBG_SET_CONCAT_COPY, 1)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(g.root)
    assert c.stats()["n_uncopied_batches"] == 0
    c.backward(g.root)
    assert np.array_equal(c.all_read(0, total), vals)
    assert np.array_equal(c.all_read(1, total), grads)
    for pid, m in enumerate(p.mats):
        assert np.array_equal(c.param_grad_read(pid, m.shape), pg[pid]), p.names[pid]
    c.close()


@pytest.mark.parametrize("seed", range(6))
def test_random_dags_with_concats_read_in_place(seed):
    """Random graphs over every operation with rows of 8 elements: CONCAT nodes of views, leaves and results feed
    products, sums, slices and losses in every mix.  Which CONCAT batches stay uncopied must follow the rule, and
    values and gradients must match the oracle, in depth and in agenda mode."""
    from paper_1705_07860_amd import binding as ob
    p, g = wl.random_dag(1200 + seed, n_nodes=400, dim=8)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for mode in (ob.OB_BYDEPTH, ob.OB_BYAGENDA):
        c, root = run_gpu(p, g, mode, arena=256 << 20)
        st = c.stats()
        bo, ids, _, _ = c.schedule_read()
        want = expected_uncopied_concats(g, bo, ids)
        say(f"  dag {seed}, mode {mode}: {want[0]} CONCAT batches need no copy")
        assert (st["n_uncopied_batches"], st["uncopied_floats"]) == want
        check_against_oracle(c, p, g, o, root, what=f"concat dag {seed}/mode {mode}")
        c.close()


def test_uncopied_concat_rows_are_filled_in_for_a_later_evaluation_stage():
    """A CONCAT that only a product reads when it is evaluated is not copied; nodes added (or evaluated)
    afterwards that read it in any other way get its row filled in first (Section 3.1 and 3.3 together)."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(5)
    pb = wl.ParamBuilder(rng, std=0.3)
    H = 8
    W = pb.add("W", 12, 2 * H)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    cats, first = [], []
    for i in range(6):
        a, b = gb.tanh(gb.input(rng.standard_normal(H))), gb.input(rng.standard_normal(H))
        cats.append(gb.concat((a, b)))
        first.append(gb.sqnorm(gb.matvec(W, -1, cats[-1])))
    r1 = gb.add(first)
    later = [gb.sqnorm(gb.cmult(gb.tanh(cc), cc)) for cc in cats] + [gb.sqnorm(gb.matvec(W, -1, cats[0]))]
    root = gb.add(later + [r1])
    g = gb.finish(root, 6)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c = ob.Context(arena_bytes=64 << 20)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(r1)
    assert c.stats()["n_uncopied_batches"] == 1
    c.forward(g.root)
    assert c.stats()["n_stages"] == 2
    check_against_oracle(c, p, g, o, g.root, what="uncopied concat read by a later stage")
    assert c.stats()["n_stages"] == 2
    c.close()


def _graph_part(g, lo, hi):
    """Nodes lo .. hi-1 of a graph as the arrays of one bulk call (operand ids stay global)."""
    from paper_1705_07860_amd.workloads import Graph
    e0, e1 = int(g.in_off[lo]), int(g.in_off[hi])
    return Graph(op=g.op[lo:hi], out_dim=g.out_dim[lo:hi], in_off=g.in_off[lo:hi + 1] - e0, in_idx=g.in_idx[e0:e1],
                 param=g.param[lo:hi], bias=g.bias[lo:hi], aux0=g.aux0[lo:hi], aux1=g.aux1[lo:hi], payload=g.payload,
                 root=hi - 1)


def test_forward_in_stages_and_graph_extension(workload_cache):
    """Section 3.1: evaluation happens when a value is asked for, and the graph may grow afterwards.
    A forward of a longer prefix, and a forward after nodes were added to an evaluated graph,
    evaluate only the nodes that have no value yet; values, and after the backward pass gradients,
    are those of one forward of the finished graph."""
    from paper_1705_07860_amd import binding as ob
    from tests.helpers import stage_schedule
    p, g, o = workload_cache("rnn")
    total = int(o.v_off[-1])
    first_sq = int(np.nonzero(g.op == wl.OP_SQNORM)[0][0])
    # (a) the whole graph is known; forward of a prefix, then of everything
    c = ob.Context(arena_bytes=64 << 20)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    c.forward(first_sq)
    early = c.value_read(first_sq, 1)[0]
    assert abs(early - o.value(first_sq)[0]) <= TOL * abs(o.value(first_sq)[0])
    c.forward(g.root)
    st = c.stats()
    assert (st["n_stages"], st["n_nodes"]) == (2, g.n - first_sq - 1)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = stage_schedule(S.by_depth, g, first_sq + 1, g.n)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL    # gathered from both stages
    for v in (0, first_sq, first_sq + 1, g.root):
        assert rel_err(c.value_read(v, int(g.out_dim[v])), o.value(v)) <= TOL
    check_against_oracle(c, p, g, o, g.root, what="rnn/staged forward")
    assert c.stats()["n_stages"] == 2                # the backward pass ran over the two stages as they are
    for v in (0, first_sq, first_sq + 1, g.root):
        assert rel_err(c.grad_read(v, int(g.out_dim[v])), o.node_grad(v)) <= TOL
    c.close()
    # (b) the graph is built in two parts around an evaluation
    c = ob.Context(arena_bytes=64 << 20)
    c.params_create(p)
    c.param_grad_zero()
    k = first_sq + 1
    assert c.add_bulk(_graph_part(g, 0, k)) == 0
    c.forward(first_sq)
    assert c.value_read(first_sq, 1)[0] == early
    assert c.add_bulk(_graph_part(g, k, g.n)) == k
    c.forward(g.root)
    assert c.stats()["n_stages"] == 2
    check_against_oracle(c, p, g, o, g.root, what="rnn/extended graph")
    assert c.stats()["n_stages"] == 2
    # a second backward pass adds the same parameter gradients once more; after a reset the graph is one evaluation again
    c.backward(g.root)
    for pid, m in enumerate(p.mats):
        assert rel_err(c.param_grad_read(pid, m.shape), 2 * o.param_grad(pid)) <= TOL
    c.reset()
    c.param_grad_zero()
    c.forward(g.root)
    assert c.stats()["n_stages"] == 1
    check_against_oracle(c, p, g, o, g.root, what="rnn/extended graph, evaluated again in one piece")
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    c.close()


@pytest.mark.parametrize("name,mode", [("tagger", "depth"), ("tree", "depth"), ("parser", "agenda")])
def test_forward_in_many_stages_at_full_size(name, mode, workload_cache):
    """A full-size graph evaluated in five stages cut at arbitrary node ids (in the middle of
    instances and of LSTM cells): after every stage the new values match the oracle, earlier
    values are still there, and the stage's schedule is the reference schedule of the stage's
    graph; the backward pass then gives the gradients of the whole graph."""
    from paper_1705_07860_amd import binding as ob
    from tests.helpers import stage_schedule
    p, g, o = workload_cache(name)
    ref = S.by_depth if mode == "depth" else S.by_agenda
    rng = np.random.default_rng(77)
    cuts = sorted(int(x) for x in rng.choice(np.arange(1000, g.n - 1000), size=4, replace=False)) + [g.n]
    c = ob.Context(arena_bytes=3 << 30, mode=ob.OB_BYDEPTH if mode == "depth" else ob.OB_BYAGENDA)
    c.params_create(p)
    c.param_grad_zero()
    c.add_bulk(g)
    lo = 0
    for k, hi in enumerate(cuts):
        c.forward(hi - 1)
        st = c.stats()
        assert (st["n_stages"], st["n_nodes"]) == (k + 1, hi - lo)
        bo, ids, bd, _ = c.schedule_read()
        rbo, rids, rbd = ref(g, hi) if k == 0 else stage_schedule(ref, g, lo, hi)
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
        probe = np.unique(np.concatenate((rng.integers(lo, hi, size=150), rng.integers(0, hi, size=50), [lo, hi - 1])))
        worst = max(rel_err(c.value_read(int(v), int(g.out_dim[v])), o.value(int(v))) for v in probe)
        say(f"  {name} stage {k}: nodes [{lo}, {hi}) read {st['n_proxies']} earlier nodes, batches={st['n_batches']}, "
            f"sched {st['ms_schedule']:.3f} ms, fwd {st['ms_forward']:.3f} ms, worst rel err {worst:.2e}")
        assert worst <= TOL
        lo = hi
    st0 = c.stats()
    c.backward(g.root)
    st1 = c.stats()
    # nothing was evaluated again: still five stages, and the last stage's forward events are the ones from before
    assert st1["n_stages"] == len(cuts) and abs(st1["ms_forward"] - st0["ms_forward"]) < 1e-3
    total = int(o.v_off[-1])
    assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL
    assert segment_rel_err(c.all_read(1, total), o.grad[:total], o.v_off) <= TOL
    for pid, m in enumerate(p.mats):
        assert rel_err(c.param_grad_read(pid, m.shape), o.param_grad(pid)) <= TOL, p.names[pid]
    c.close()


@pytest.mark.parametrize("mode,launch,fuse", [("nobatch", 0, 2), ("agenda", 1, 2), ("depth", 0, 1), ("depth", 0, 0)])
def test_stages_in_every_mode_and_on_a_forked_context(mode, launch, fuse):
    """Staged forwards under the other batching modes, under hipGraph launches and the other fusion
    levels, on a context forked from the one that owns the parameters."""
    from paper_1705_07860_amd import binding as ob
    p, g = wl.make("rnn")
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    owner = ob.Context(arena_bytes=64 << 20, mode={"nobatch": ob.OB_NOBATCH, "agenda": ob.OB_BYAGENDA, "depth": ob.OB_BYDEPTH}[mode],
                       launch=launch)
    owner.set_fusion(fuse)
    owner.params_create(p)
    owner.param_grad_zero()
    c = owner.fork(arena_bytes=128 << 20)
    cuts = [40, 41, 150, g.n]
    lo = 0
    for k, hi in enumerate(cuts):
        assert c.add_bulk(_graph_part(g, lo, hi)) == lo
        c.forward(hi - 1)
        assert c.stats()["n_stages"] == k + 1
        for v in range(lo, hi, 7):
            assert rel_err(c.value_read(v, int(g.out_dim[v])), o.value(v)) <= TOL
        lo = hi
    check_against_oracle(c, p, g, o, g.root, what=f"stages {mode} launch {launch} fuse {fuse}")
    c.close()
    owner.close()


def test_growing_graph_demo_agrees_with_itself():
    """The runnable demo at a small size: growing the graph in stages, evaluating the prefix again
    every time and one forward of the finished graph give the same loss."""
    from paper_1705_07860_amd import grow_demo
    res = grow_demo.run_all(chains=5, steps=4, repeats=2, arena_bytes=256 << 20, report=say, hidden=32, emb=16, classes=7)
    losses = {kind: loss for kind, _, _, loss in res}
    assert set(losses) == {"oneshot", "stages", "again"}
    ref = losses["oneshot"]
    assert all(abs(v - ref) <= 1e-5 * abs(ref) for v in losses.values())


def test_graph_grown_node_by_node_and_a_full_arena():
    """The pattern of a model that looks at a value before it decides what to add (Section 3.1): a
    graph grown in many small steps, a forward after each.  With an arena too small to stack all
    stages the library evaluates everything again instead, with the same values."""
    from paper_1705_07860_amd import binding as ob
    p, g = wl.random_dag(941, n_nodes=150, dim=8)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for arena, expect_fallback in ((256 << 20, False), (6 << 20, True)):
        c = ob.Context(arena_bytes=arena)
        c.params_create(p)
        c.param_grad_zero()
        lo, stages_seen = 0, []
        while lo < g.n:
            hi = min(g.n, lo + 1 + (lo * 7) % 13)
            assert c.add_bulk(_graph_part(g, lo, hi)) == lo
            c.forward(hi - 1)
            stages_seen.append(c.stats()["n_stages"])
            for v in (lo, hi - 1, (lo * 5) % hi):
                assert rel_err(c.value_read(v, int(g.out_dim[v])), o.value(v)) <= TOL
            lo = hi
        say(f"  arena {arena >> 20} MB: stages after each forward {stages_seen}")
        assert (min(stages_seen[1:]) == 1) == expect_fallback
        if not expect_fallback:
            assert stages_seen == list(range(1, len(stages_seen) + 1))
        check_against_oracle(c, p, g, o, g.root, what=f"grown dag, arena {arena >> 20} MB")
        c.close()


def test_arena_too_small_is_an_error_not_a_crash():
    from paper_1705_07860_amd import binding as ob
    p, g = wl.make("rnn")
    c = ob.Context(arena_bytes=64 << 10)
    c.params_create(p)
    c.add_bulk(g)
    with pytest.raises(ob.ObError) as e:
        c.forward(g.root)
    assert e.value.code == -5
    c.close()


def test_odd_dimensions_duplicate_lookups_and_wide_sum():
    """Dimensions that are not multiples of 4 or 32, the same table row looked up many times, a
    node used twice by one consumer, and a sum over many operands."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(12)
    pb = wl.ParamBuilder(rng, std=0.4)
    E = pb.add("E", 5, 37)
    W = pb.add("W", 45, 37)
    b = pb.add("b", 45, 1)
    W2 = pb.add("W2", 3, 45)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for i in range(70):
        x = gb.lookup(E, i % 3)                      # rows 0..2 many times, rows 3,4 never
        h = gb.tanh(gb.matvec(W, b, x))
        hh = gb.cmult(h, h)                          # same operand twice
        s = gb.slice(hh, 3, 44)
        z = gb.concat((s, gb.slice(h, 0, 4)))        # 41 + 4 = 45
        q = gb.add((z, h, hh))
        sc = gb.matvec(W2, -1, gb.sigmoid(q))
        losses.append(gb.pick_nls(sc, i % 3))
        losses.append(gb.sqnorm(s))
    g = gb.finish(gb.add(losses), 70)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, root, what="odd")
    assert not np.any(c.param_grad_read(E, (5, 37))[3:])     # untouched rows stay zero
    c.close()


@pytest.mark.parametrize("dims", [(50, 70, 300), (64, 128, 523), (40, 132, 300), (96, 200, 400)])
def test_large_batches_of_matrix_products(dims):
    """Matrix-product batches with hundreds of rows (the wide forward tiles): ragged rows and
    columns, a contraction length that is not a multiple of 4 in the first case, operands that are
    gathered (every other lookup row) rather than evenly spaced."""
    from paper_1705_07860_amd import binding as ob
    k, m, nrow = dims
    rng = np.random.default_rng(1000 + k)
    pb = wl.ParamBuilder(rng, std=0.3)
    E = pb.add("E", 40, k)
    W = pb.add("W", m, k)
    b = pb.add("b", m, 1)
    U = pb.add("U", 3, m)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for i in range(nrow):
        x = gb.lookup(E, (7 * i) % 40)
        if i % 2:
            x = gb.tanh(x)                           # half of the rows come from another batch
        h = gb.tanh(gb.matvec(W, b, x))
        losses.append(gb.pick_nls(gb.matvec(U, -1, h), i % 3))
    g = gb.finish(gb.add(losses), nrow)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=256 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, root, what=f"wide{dims}")
    c.close()


def test_parameter_gradients_accumulate_until_zeroed(workload_cache):
    from paper_1705_07860_amd import binding as ob
    p, g, o = workload_cache("rnn")
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    c.backward(root)
    g1 = c.param_grad_read(0, p.mats[0].shape)
    c.backward(root)
    g2 = c.param_grad_read(0, p.mats[0].shape)
    assert rel_err(g2, 2 * g1.astype(np.float64)) < 1e-6
    c.param_grad_zero()
    c.backward(root)
    assert np.array_equal(c.param_grad_read(0, p.mats[0].shape), g1)
    c.close()


def _smallest_arena(p, g, fuse, most=64 << 20):
    """Bytes of the smallest arena, in steps of 256, that holds a forward and a backward pass."""
    from paper_1705_07860_amd import binding as ob

    def fits(units):
        c = ob.Context(arena_bytes=256 * units)
        try:
            c.set_fusion(fuse)
            c.params_create(p)
            c.param_grad_zero()
            c.add_bulk(g)
            c.forward(g.root)
            c.backward(g.root)
            return True
        except ob.ObError as e:
            assert e.code == -5
            return False
        finally:
            c.close()

    no, yes = 0, most // 256
    assert fits(yes)
    while yes - no > 1:
        mid = (no + yes) // 2
        if fits(mid):
            yes = mid
        else:
            no = mid
    return 256 * yes


@pytest.mark.parametrize("H,rows", [(2, 60), (2, 200), (64, 40)])
def test_gated_cells_need_no_larger_arena(H, rows):
    """The tables for gated cells are used where there is room for them: the smallest arena that holds a graph is that of a
    plan without fusion, which has none, and there the results have the bits that they have in a large one."""
    from paper_1705_07860_amd import binding as ob
    p, g = _cell_graph(H, 1, True, rows, "")
    need = {fuse: _smallest_arena(p, g, fuse) for fuse in (0, 1, 2)}
    say(f"  {g.n} nodes: smallest arenas {need}")
    assert need[1] <= need[0] and need[2] <= need[0]
    total = int(g.out_dim.sum())
    out = []
    for arena in (need[2], 128 << 20):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=arena)
        c.backward(root)
        kinds = c.debug_read(ob.OB_DBG_CHAINS).reshape(-1, 12)[:, 3]
        assert c.stats()["arena_used_bytes"] <= arena
        out.append([int(np.sum(kinds == 3))] + [c.grad_read(v, int(g.out_dim[v])).view(np.uint32) for v in range(0, g.n, 7)]
                   + [c.value_read(v, int(g.out_dim[v])).view(np.uint32) for v in range(0, g.n, 7)]
                   + [c.param_grad_read(k, m.shape).view(np.uint32) for k, m in enumerate(p.mats)])
        c.close()
    say(f"  chains of cells: {out[0][0]} in the smallest arena, {out[1][0]} in a large one")
    assert out[1][0] >= 2 and (H > 2 or out[0][0] == 0)
    for a, b in zip(out[0][1:], out[1][1:]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("streams", ["whole chip", "disjoint compute units"])
def test_forked_contexts_share_parameters_and_pipeline_scheduling(streams):
    """Two graphs in flight: a forked context schedules its graph on a second stream while the
    first one executes; both share one parameter set, and the accumulated parameter gradient is
    the sum of the two minibatches' gradients.  Second case: the streams come from
    ob_stream_create_on_cus, scheduling on compute units [0, 32), execution on the rest."""
    import torch
    from paper_1705_07860_amd import binding as ob
    p = wl.tagger_params()
    gs = [wl.tagger_minibatch(p, seed=41 + j, lengths=[4 + j, 9, 2, 6 + 2 * j]) for j in range(2)]
    os_ = []
    for g in gs:
        o = Oracle(g, p, "f64")
        o.forward()
        o.backward(g.root)
        os_.append(o)
    raw = []
    if streams == "whole chip":
        ex, sc = torch.cuda.Stream(), torch.cuda.Stream()
    else:
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        with pytest.raises(ob.ObError) as e:
            ob.stream_create_on_cus(n_cu - 8, 16)          # reaches beyond the device's units
        assert e.value.code == -8
        raw = [ob.stream_create_on_cus(32, n_cu - 32), ob.stream_create_on_cus(0, 32)]
        ex, sc = torch.cuda.ExternalStream(raw[0]), torch.cuda.ExternalStream(raw[1])
    a = ob.Context(arena_bytes=256 << 20, stream=ex, sched_stream=sc)
    a.params_create(p)
    a.param_grad_zero()
    b = a.fork(arena_bytes=256 << 20, stream=ex, sched_stream=sc)
    with pytest.raises(ob.ObError) as e:
        b.param_create(np.zeros((2, 2), np.float32))
    assert e.value.code == -6
    cs = [a, b]
    for c, g in zip(cs, gs):
        c.add_bulk(g)
        c.upload()
    cs[0].schedule(gs[0].root)
    for j in range(2):
        cs[j].forward(gs[j].root)
        cs[j].backward(gs[j].root)
        if j == 0:
            cs[1].schedule_async(gs[1].root)  # queued behind nothing: overlaps the execution of graph 0
    for c, g, o in zip(cs, gs, os_):
        total = int(o.v_off[-1])
        assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL
        assert segment_rel_err(c.all_read(1, total), o.grad[:total], o.v_off) <= TOL
        bo, ids, bd, _ = c.schedule_read()
        rbo, rids, rbd = S.by_depth(g)
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    for pid, m in enumerate(p.mats):
        ref = os_[0].param_grad(pid) + os_[1].param_grad(pid)
        assert rel_err(b.param_grad_read(pid, m.shape), ref) <= TOL, p.names[pid]
    # a second round on the same contexts after reset (the arenas are reused)
    a.param_grad_zero()
    for c, g in zip(cs, gs):
        c.reset()
        c.schedule(g.root)
        c.forward(g.root)
        c.backward(g.root)
    for pid, m in enumerate(p.mats):
        ref = os_[0].param_grad(pid) + os_[1].param_grad(pid)
        assert rel_err(a.param_grad_read(pid, m.shape), ref) <= TOL, p.names[pid]
    b.close()
    a.close()
    torch.cuda.synchronize()
    for h in raw:
        ob.stream_destroy(h)


def test_stacked_matrix_products():
    """MATVEC feeding MATVEC directly, with and without a non-linearity in between."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(3)
    pb = wl.ParamBuilder(rng, std=0.3)
    W = [pb.add(f"W{i}", 24, 24) for i in range(4)]
    b0 = pb.add("b0", 24, 1)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for i in range(9):
        h = gb.input(rng.standard_normal(24))
        h = gb.matvec(W[0], b0, h)
        h = gb.matvec(W[1], -1, h)
        h = gb.matvec(W[2], -1, gb.tanh(gb.matvec(W[3], -1, h)))
        losses.append(gb.sqnorm(h))
    g = gb.finish(gb.add(losses), 9)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, root, what="stacked")
    c.close()


@pytest.mark.parametrize("n_inst", [1500, 2000, 9000])
def test_more_parameter_uses_than_nodes_or_edges(n_inst):
    """Two products with biases behind a look-up, and a loss: five uses of parameters for four nodes and four edges an
    instance.  Above 8 192 pairs a sort goes back and forth between two pairs of buffers, which must hold all of the uses."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(n_inst)
    pb = wl.ParamBuilder(rng, std=0.5)
    E, W, b, U, d = pb.add("E", 40, 6), pb.add("W", 7, 6), pb.add("b", 7, 1), pb.add("U", 5, 7), pb.add("d", 5, 1)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = [gb.pick_nls(gb.matvec(U, d, gb.matvec(W, b, gb.lookup(E, int(r)))), int(r) % 5) for r in rng.integers(0, 40, n_inst)]
    g = gb.finish(gb.add(losses), n_inst)
    assert 5 * n_inst > max(g.n, g.n_edges) + 1
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for mode in (ob.OB_BYDEPTH, ob.OB_BYAGENDA):
        c, root = run_gpu(p, g, mode, arena=256 << 20)
        check_against_oracle(c, p, g, o, root, what=f"{n_inst} instances, mode {mode}")
        c.close()


def test_long_chain_uses_the_unfused_plan_and_the_long_slot_table():
    """More batches than a fused launch plan can hold (4096) and more launch slots than the
    read-back window (2048): a 4300-deep chain of alternating tanh / sigmoid nodes runs with one
    launch per depth level and still matches the oracle."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(77)
    pb = wl.ParamBuilder(rng, std=0.5)
    E = pb.add("E", 3, 8)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    x = gb.lookup(E, 1)
    y = gb.lookup(E, 2)
    for i in range(4300):
        x = gb.tanh(x) if i % 2 else gb.sigmoid(x)
        if i % 500 == 0:
            x = gb.add((x, y))
    g = gb.finish(gb.sqnorm(x), 1)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    st = c.stats()
    assert st["n_batches"] > 4096 and st["n_slots"] == st["n_steps"] > 2048
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids, rbd = S.by_depth(g)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
    check_against_oracle(c, p, g, o, root, what="long chain")
    c.close()


@pytest.mark.parametrize("arities,copies", [((13, 14, 15, 16, 17), 40), ((2, 14, 15, 300), 7), ((1,), 131_070), ((1,), 131_080)])
def test_agenda_counters_of_few_and_many_operands(arities, copies):
    """Agenda counters of four bits hold up to fourteen operands, longer lists are counted in memory, also where a node is an
    operand more than once; graphs of up to 262 144 nodes have them in LDS (the last two lie on either side)."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(copies)
    pb = wl.ParamBuilder(rng, std=0.3)
    p = pb.done() if len(arities) == 1 else None
    if p is None:
        pb.add("E", 3, 4)
        p = pb.done()
    g = wl.GraphBuilder(p)
    nodes = [g.input(rng.standard_normal(4)) for _ in range(copies if len(arities) == 1 else 60)]
    if len(arities) == 1:
        out = [g.sqnorm(v) for v in nodes]
    else:
        for k in range(copies):
            for a in arities:
                nodes.append(g.add([nodes[int(q)] for q in rng.integers(max(0, len(nodes) - 200), len(nodes), a)]))
                nodes.append(g.tanh(nodes[-1]))
        out = [g.sqnorm(v) for v in nodes[60:]]
    gr = g.finish(g.add(out), 1)
    c, root = run_gpu(p, gr, ob.OB_BYAGENDA, arena=1 << 30)
    bo, ids, _, _ = c.schedule_read()
    want = S.by_agenda(gr)
    assert np.array_equal(bo, want[0]) and np.array_equal(ids, want[1])
    c.close()


@pytest.mark.parametrize("rows,wide", [(3, 15), (70, 14), (70, 16), (600, 900)])
def test_agenda_entries_of_nodes_with_few_and_many_consumers(rows, wide):
    """An entry of an agenda list holds up to six consumers, more are looked up: 1 to 12 of them a node.  Sums of `wide` operands, the
    same node twice and more among them, are counted down by several lanes of a wave at once, some lanes of it for different sums."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(rows + wide)
    pb = wl.ParamBuilder(rng, std=0.3)
    pb.add("E", 3, 4)
    p = pb.done()
    g = wl.GraphBuilder(p)
    ends = []
    for r in range(rows):
        x = g.tanh(g.input(rng.standard_normal(4)))
        ends += [g.sigmoid(x) if (r + k) % 3 else g.tanh(g.tanh(x)) for k in range(1 + r % 12)]
    sums = []
    for k in range(7):
        sums.append(g.add([ends[int(q)] for q in rng.integers(0, len(ends), wide)]))
        sums.append(g.add([ends[k % len(ends)]] * wide + [ends[-1]]))
    gr = g.finish(g.add([g.sqnorm(v) for v in sums + ends]), 1)
    c, root = run_gpu(p, gr, ob.OB_BYAGENDA, arena=256 << 20)
    bo, ids, _, _ = c.schedule_read()
    want = S.by_agenda(gr)
    assert np.array_equal(bo, want[0]) and np.array_equal(ids, want[1])
    c.close()


def test_agenda_rejects_more_signatures_than_it_can_rank():
    """1100 slices with pairwise different ranges are 1100 signatures; agenda mode ranks at most
    1024 and must fail cleanly (depth-based batching takes the same graph)."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(78)
    pb = wl.ParamBuilder(rng, std=0.5)
    E = pb.add("E", 2, 1200)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    x = gb.lookup(E, 0)
    parts = [gb.sqnorm(gb.slice(x, i, i + 3)) for i in range(1100)]
    g = gb.finish(gb.add(parts), 1)
    c = ob.Context(arena_bytes=64 << 20, mode=ob.OB_BYAGENDA)
    c.params_create(p)
    c.add_bulk(g)
    with pytest.raises(ob.ObError) as e:
        c.forward(g.root)
    assert e.value.code == -6
    c.close()
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    check_against_oracle(c, p, g, o, root, what="many signatures")
    c.close()


def test_sgd_step_matches_the_oracle_and_lowers_the_loss():
    """Section 2's update: after backward, theta - lr * grad on the GPU equals the oracle's update
    of the same parameters; gradients are cleared; a second forward gives a smaller loss."""
    from paper_1705_07860_amd import binding as ob
    p = wl.tagger_params()
    g = wl.tagger_minibatch(p, seed=wl.SEED_BASE + 31, lengths=[5, 2, 8, 3])
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=512 << 20)
    loss0 = float(c.value_read(root, 1)[0])
    c.backward(root)
    lr = 0.05
    c.sgd_step(lr, zero_grad=True)
    ref = o.sgd_params(lr)
    for pid, m in enumerate(p.mats):
        got = c.param_read(pid, m.shape)
        assert rel_err(got, ref[pid]) <= TOL, p.names[pid]
        assert not np.any(c.param_grad_read(pid, m.shape))
    c.reset()
    c.forward(root)
    loss1 = float(c.value_read(root, 1)[0])
    say(f"  loss {loss0:.5f} -> {loss1:.5f}")
    assert loss1 < loss0
    c.close()


def test_update_walks_the_touched_rows_of_an_embedding_table():
    """Two minibatches (two contexts on one parameter set) add their gradients before one update:
    the table's touched rows are the union of both, every other row keeps its bits, the dense
    matrices are updated as before, and afterwards every gradient is zero again, so that a third
    backward pass gives that minibatch's gradient alone.  Then the same with the gradients only
    cleared (no update)."""
    from paper_1705_07860_amd import binding as ob
    p = wl.tagger_params()
    ga = wl.tagger_minibatch(p, seed=wl.SEED_BASE + 41, lengths=[4, 7, 2])
    gb_ = wl.tagger_minibatch(p, seed=wl.SEED_BASE + 42, lengths=[6, 3])
    oa, ob_ = Oracle(ga, p, "f64"), Oracle(gb_, p, "f64")
    for o, g in ((oa, ga), (ob_, gb_)):
        o.forward()
        o.backward(g.root)
    ca = ob.Context(arena_bytes=512 << 20)
    ca.params_create(p)
    ca.param_grad_zero()
    cb = ca.fork(arena_bytes=512 << 20, stream=ca._stream)
    for c, g in ((ca, ga), (cb, gb_)):
        c.add_bulk(g)
        c.forward(g.root)
        c.backward(g.root)
    emb = p.index("E") if "E" in p.names else max(range(len(p.mats)), key=lambda i: p.mats[i].shape[0])
    before = [m.copy() for m in p.mats]
    lr = 0.1
    ca.sgd_step(lr, zero_grad=True)
    rows_a = set(int(r) for r in ga.aux0[ga.op == wl.OP_LOOKUP])
    rows_b = set(int(r) for r in gb_.aux0[gb_.op == wl.OP_LOOKUP])
    touched = sorted(rows_a | rows_b)
    for pid, m in enumerate(p.mats):
        ref = m.astype(np.float64) - lr * (oa.param_grad(pid) + ob_.param_grad(pid))
        got = ca.param_read(pid, m.shape)
        assert rel_err(got, ref) <= TOL, p.names[pid]
        assert not np.any(ca.param_grad_read(pid, m.shape)), p.names[pid]
    got_e = ca.param_read(emb, p.mats[emb].shape)
    untouched = np.ones(p.mats[emb].shape[0], bool)
    untouched[touched] = False
    assert np.array_equal(got_e[untouched], before[emb][untouched])       # bit for bit
    assert np.all(np.any(got_e[touched] != before[emb][touched], axis=1))
    # a third backward pass: this minibatch's gradient alone (nothing left over in rows only the others touched)
    cb.reset()
    cb.forward(gb_.root)
    cb.backward(gb_.root)
    params_now = wl.Params([ca.param_read(pid, m.shape) for pid, m in enumerate(p.mats)], p.names)
    o3 = Oracle(gb_, params_now, "f64")
    o3.forward()
    o3.backward(gb_.root)
    for pid, m in enumerate(p.mats):
        assert rel_err(cb.param_grad_read(pid, m.shape), o3.param_grad(pid)) <= TOL, p.names[pid]
    only_a = sorted(rows_a - rows_b)
    assert not np.any(cb.param_grad_read(emb, p.mats[emb].shape)[only_a])
    # clearing alone walks the touched rows too
    ca.param_grad_zero()
    for pid, m in enumerate(p.mats):
        assert not np.any(ca.param_grad_read(pid, m.shape)), p.names[pid]
    ca.reset()
    ca.forward(ga.root)
    ca.backward(ga.root)
    o4 = Oracle(ga, params_now, "f64")
    o4.forward()
    o4.backward(ga.root)
    for pid, m in enumerate(p.mats):
        assert rel_err(ca.param_grad_read(pid, m.shape), o4.param_grad(pid)) <= TOL, p.names[pid]
    cb.close()
    ca.close()


def test_synthetic_equal_length_tagger_small():
    """The stacked two-layer BiLSTM labeler of Section 4.1 at a small size, both batching strategies."""
    from paper_1705_07860_amd import binding as ob
    p = wl.sync_tagger_params(vocab=50, emb=24, hidden=16, tags=7)
    g = wl.sync_tagger_minibatch(p, n_sent=5, length=6)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for mode, ref in ((ob.OB_BYDEPTH, S.by_depth), (ob.OB_BYAGENDA, S.by_agenda)):
        c, root = run_gpu(p, g, mode, arena=256 << 20)
        bo, ids, bd, _ = c.schedule_read()
        rbo, rids, rbd = ref(g)
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
        check_against_oracle(c, p, g, o, root, what=f"sync tagger mode {mode}")
        c.close()


def labels_of(batch_off, node_ids):
    """Per node, the index of the batch that holds it."""
    lab = np.empty(len(node_ids), np.int32)
    lab[np.asarray(node_ids, np.int64)] = np.repeat(np.arange(len(batch_off) - 1), np.diff(batch_off))
    return lab


def check_manual(p, g, o, lab, what, fuse=2, arena=2 << 30, n_nodes=None):
    from paper_1705_07860_amd import binding as ob
    from tests.helpers import manual_schedule
    c, root = run_gpu(p, g, ob.OB_MANUAL, arena=arena, fuse=fuse, labels=lab, n_nodes=n_nodes)
    bo, ids, bd, _ = c.schedule_read()
    rbo, rids = manual_schedule(lab, n_nodes)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids)
    assert np.array_equal(bd, np.arange(len(rbo) - 1))
    st = c.stats()
    say(f"manual {what}: batches={st['n_batches']} slots={st['n_slots']} sched {st['ms_schedule']:.3f} ms")
    if n_nodes is None:
        check_against_oracle(c, p, g, o, root, what=f"{what}/manual")
    return c


@pytest.mark.parametrize("name", ["rnn", "tagger", "tree"])
def test_manual_batching_given_the_reference_schedules(name, workload_cache):
    """Manual batching (Section 2) with the batches of the depth-based and of the agenda-based
    reference schedule handed in as labels (stretched, so that they are not dense): the library
    runs exactly those batches, and values and gradients match the oracle."""
    p, g, o = workload_cache(name)
    for ref in (S.by_depth, S.by_agenda):
        rbo, rids, _ = ref(g)
        lab = labels_of(rbo, rids) * 3 + 1
        c = check_manual(p, g, o, lab, f"{name} {ref.__name__}")
        bo, ids, _, _ = c.schedule_read()
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids)
        c.close()


@pytest.mark.parametrize("fuse", [0, 1, 2])
def test_manual_batching_by_statement_on_the_equal_length_tagger(fuse):
    """Section 4.1's labeler over equal-length sentences, batched the way a program written over
    a batch of sentences would run it: one batch per statement, every launch-fusion level."""
    p = wl.sync_tagger_params(vocab=50, emb=24, hidden=16, tags=7)
    g = wl.sync_tagger_minibatch(p, n_sent=5, length=6)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    check_manual(p, g, o, wl.sync_tagger_manual_labels(g), f"sync tagger fuse {fuse}", fuse=fuse, arena=256 << 20).close()


def test_manual_batching_full_width_and_prefix():
    """The labeler at the layer sizes Section 4.1 states (16 sentences of 40 words), then a
    prefix of the graph under the same labels, then another labelling on the same context."""
    from paper_1705_07860_amd import binding as ob
    from tests.helpers import manual_schedule
    p = wl.sync_tagger_params()
    g = wl.sync_tagger_minibatch(p, n_sent=16, length=40)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    lab = wl.sync_tagger_manual_labels(g)
    c = check_manual(p, g, o, lab, "sync tagger 16 x 40")
    # a prefix: forget the evaluation, evaluate the first sentences' nodes only
    c.reset()
    k = 3 * ((g.n - 1) // 16)
    c.forward(k - 1)
    bo, ids, _, _ = c.schedule_read()
    rbo, rids = manual_schedule(lab, k)
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids)
    assert rel_err(c.value_read(k - 1, int(g.out_dim[k - 1])), o.value(k - 1)) <= TOL
    # new labels on the same graph: the depth-based batches
    rbo, rids, _ = S.by_depth(g)
    c.set_manual_batches(labels_of(rbo, rids))
    c.param_grad_zero()
    c.forward(g.root)
    bo, ids, _, _ = c.schedule_read()
    assert np.array_equal(bo, rbo) and np.array_equal(ids, rids)
    check_against_oracle(c, p, g, o, g.root, what="relabelled")
    c.close()


@pytest.mark.parametrize("seed", [930, 931, 932, 933])
def test_manual_batching_on_random_dags(seed):
    p, g = wl.random_dag(seed, n_nodes=120, dim=8)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    rbo, rids, _ = S.by_depth(g)
    check_manual(p, g, o, labels_of(rbo, rids), f"dag {seed}", arena=64 << 20).close()
    # every node a batch of its own is a valid labelling too
    check_manual(p, g, o, np.arange(g.n, dtype=np.int32), f"dag {seed} singletons", arena=64 << 20).close()


def test_headline_loop_as_benchmarked(workload_cache):
    """The loop bench.py times by default, on the headline configuration (config 3, full size): a ring of
    contexts forked from one parameter set; every step hands a minibatch over anew (ob_graph_new,
    ob_add_bulk, upload and scheduling on the schedule stream, queued one step ahead of the execution),
    the schedule stream confined to compute units [0, 32) and the execution stream to the others.  The
    minibatches differ in size, so a context's graph store and tables are reused for graphs larger and
    smaller than the ones before.  After the loop every context's values and node gradients, and the
    parameter gradients of the last step, match the oracle and the schedule is the reference one."""
    import torch
    from paper_1705_07860_amd import binding as ob
    p, g0, o0 = workload_cache("tagger_char")
    cfg = wl.CONFIGS["tagger_char"]
    graphs = [g0] + [cfg["batch"](p, j) for j in (1, 2)]
    oracles = [o0]
    for g in graphs[1:]:
        o = Oracle(g, p, "f64")
        o.forward()
        o.backward(g.root)
        oracles.append(o)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    raw = [ob.stream_create_on_cus(32, n_cu - 32), ob.stream_create_on_cus(0, 32)]
    ex, sc = torch.cuda.ExternalStream(raw[0]), torch.cuda.ExternalStream(raw[1])
    pool, steps = 4, 9                      # step i runs graph i % 3 in context i % 4
    ctxs = []
    for j in range(pool):
        if j == 0:
            c = ob.Context(arena_bytes=1 << 30, stream=ex, sched_stream=sc)
            c.params_create(p)
            c.param_grad_zero()
        else:
            c = ctxs[0].fork(arena_bytes=1 << 30, stream=ex, sched_stream=sc)
        ctxs.append(c)

    def hand_over(i):
        c = ctxs[i % pool]
        c.graph_new()
        c.add_bulk(graphs[i % 3])
        c.schedule_async(graphs[i % 3].root)

    hand_over(0)
    for i in range(steps):
        if i + 1 < steps:
            hand_over(i + 1)
        c, g = ctxs[i % pool], graphs[i % 3]
        c.param_grad_zero()
        c.forward(g.root)
        c.backward(g.root)
    for i in range(steps - pool, steps):    # the last step of every context
        c, g, o = ctxs[i % pool], graphs[i % 3], oracles[i % 3]
        total = int(o.v_off[-1])
        assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL
        assert segment_rel_err(c.all_read(1, total), o.grad[:total], o.v_off) <= TOL
        bo, ids, bd, _ = c.schedule_read()
        rbo, rids, rbd = S.by_depth(g)
        assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
        assert c.stats()["n_depth_retries"] == 0
    last = oracles[(steps - 1) % 3]
    for pid, m in enumerate(p.mats):
        assert rel_err(ctxs[0].param_grad_read(pid, m.shape), last.param_grad(pid)) <= TOL, p.names[pid]
    for c in reversed(ctxs):
        c.close()
    torch.cuda.synchronize()
    for h in raw:
        ob.stream_destroy(h)


@pytest.mark.parametrize("mode,lookahead", [("depth", 1), ("agenda", 2)])
def test_full_size_pipelined_loop_as_benchmarked(workload_cache, mode, lookahead):
    """The loop bench.py times, at the tagger's full size: contexts forked from one parameter set,
    one execution stream, scheduling of steps i + 1 .. i + lookahead queued on schedule streams of
    their own before step i executes, minibatches cycling through the contexts.  After the loop
    every context's values and node gradients, and the parameter gradients of the last step, match
    the oracle, and every context holds the schedule of its strategy (Section 3.2)."""
    import torch
    from paper_1705_07860_amd import binding as ob
    p, g0, o0 = workload_cache("tagger")
    cfg = wl.CONFIGS["tagger"]
    graphs = [g0] + [cfg["batch"](p, j) for j in range(1, 2 + lookahead)]
    oracles = [o0]
    for g in graphs[1:]:
        o = Oracle(g, p, "f64")
        o.forward()
        o.backward(g.root)
        oracles.append(o)
    ex, scs = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(lookahead)]
    ctxs = []
    for j, g in enumerate(graphs):
        if j == 0:
            c = ob.Context(arena_bytes=1 << 30, stream=ex, sched_stream=scs[0],
                           mode=ob.OB_BYAGENDA if mode == "agenda" else ob.OB_BYDEPTH)
            c.params_create(p)
            c.param_grad_zero()
        else:
            c = ctxs[0].fork(arena_bytes=1 << 30, stream=ex, sched_stream=scs[j % lookahead])
        c.add_bulk(g)
        c.upload()
        ctxs.append(c)
    pool, steps = len(graphs), 7

    def sched(i):
        c = ctxs[i % pool]
        c.reset()
        c.schedule_async(graphs[i % pool].root)

    for i in range(lookahead):
        sched(i)
    for i in range(steps):
        if i + lookahead < steps:
            sched(i + lookahead)
        c, g = ctxs[i % pool], graphs[i % pool]
        c.param_grad_zero()
        c.forward(g.root)
        c.backward(g.root)
    last = (steps - 1) % pool
    for c, g, o in zip(ctxs, graphs, oracles):
        total = int(o.v_off[-1])
        assert segment_rel_err(c.all_read(0, total), o.val[:total], o.v_off) <= TOL
        assert segment_rel_err(c.all_read(1, total), o.grad[:total], o.v_off) <= TOL
        bo, ids, bd, _ = c.schedule_read()
        if mode == "depth":
            rbo, rids, rbd = S.by_depth(g)
            assert np.array_equal(bo, rbo) and np.array_equal(ids, rids) and np.array_equal(bd, rbd)
        else:
            rbo, rids, _ = S.by_agenda(g)
            assert np.array_equal(bo, rbo) and np.array_equal(ids, rids)
    for pid, m in enumerate(p.mats):
        assert rel_err(ctxs[0].param_grad_read(pid, m.shape), oracles[last].param_grad(pid)) <= TOL, p.names[pid]
    for c in reversed(ctxs):
        c.close()


@pytest.mark.parametrize("d", [1, 3, 255, 4095, 4096, 4097, 9001])
def test_reading_one_node_of_any_width(d):
    """ob_value_read / ob_grad_read leave up to 4096 elements of a row in pinned memory themselves and copy the rest:
    widths around both sides of that.  An input's value must come back bit for bit (so must the row of a CONCAT
    nobody reads, which the forward pass may leave unwritten); tanh rounds within 4 units of 2^-24, the gradient
    g = 2 t (1 - t^2) of sum t^2 is four such roundings."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(d)
    pb = wl.ParamBuilder(rng)
    pb.add("W", 4, 4)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    x0, y0 = rng.standard_normal(d).astype(np.float32), rng.standard_normal(4).astype(np.float32)
    x, y = gb.input(x0), gb.input(y0)
    cat = gb.concat((y, y))
    t = gb.tanh(x)
    g = gb.finish(gb.sqnorm(t), 1)
    c, root = run_gpu(p, g, ob.OB_BYDEPTH, arena=64 << 20)
    c.backward(root)
    th = np.tanh(x0.astype(np.float64))
    assert np.array_equal(c.value_read(x, d), x0)
    assert np.array_equal(c.value_read(cat, 8), np.concatenate([y0, y0]))
    assert np.abs(c.value_read(t, d) - th).max() <= 4 * 2.0 ** -24
    assert np.abs(c.grad_read(x, d) - 2 * th * (1 - th * th)).max() <= 32 * 2.0 ** -24
    assert rel_err(c.value_read(root, 1), np.asarray([np.sum(th * th)])) <= TOL
    c.close()


def _pull_rows_graph(d, R, k, odd_by):
    """40 rows t of width d, in order, with two consumers each; row k of every second tile of R rows, and of the last,
    is out of line with the others.  Returns the parameters, the graph, the ids of the rows t and which are odd."""
    rng = np.random.default_rng(d + k)
    pb = wl.ParamBuilder(rng, std=0.3)
    W = pb.add("W", d, 8)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    odd = [i % R == k and ((i // R) % 2 == 1 or i // R == 39 // R) for i in range(40)]
    ys = [gb.matvec(W, -1, gb.input(rng.standard_normal(8))) for _ in range(40)]
    ts, ss = [gb.tanh(y) for y in ys], [gb.sigmoid(y) for y in ys]
    losses, late = [], []
    for i in range(40):
        # "value": the factor beside t comes from elsewhere, so the value that t's gradient is read with is out of line
        losses.append(gb.sqnorm(gb.cmult(ts[i], ss[(i + 7) % 40] if odd_by == "value" and odd[i] else ss[i])))
        if odd_by == "offset" and odd[i]:
            late.append(i)         # "offset": same consumer, its gradient row behind those of all others
        else:
            losses.append(gb.sqnorm((gb.sigmoid if odd_by == "kind" and odd[i] else gb.tanh)(ts[i])))
        if odd_by == "count" and odd[i]:
            losses.append(gb.sqnorm(gb.sigmoid(ts[i])))
    losses += [gb.sqnorm(gb.tanh(ts[i])) for i in late]
    return p, gb.finish(gb.add(losses), 40), np.asarray(ts), np.asarray(odd)


@pytest.mark.parametrize("odd_by", ["count", "kind", "offset", "value"])
@pytest.mark.parametrize("d", [512, 341, 256, 204, 64, 60])
def test_pull_tiles_of_two_to_seventeen_rows(d, odd_by):
    """A pull tile holds as many rows as fit 1024 elements (2, 3, 5, 4, 16 and 17 here) and compares its rows' consumer
    edges four or sixteen rows at a time.  One row of every second tile, and of the last, is out of line (a consumer more, a consumer
    of another kind, a gradient or a value row at another distance), at each place of a tile in turn.  Tiles of like rows
    are read as such (up to sixteen rows), and none with a row of another count or kind is."""
    from paper_1705_07860_amd import binding as ob
    R = 1024 // d
    for k in range(R):
        p, g, ts, odd = _pull_rows_graph(d, R, k, odd_by)
        o = Oracle(g, p, "f64")
        o.forward()
        o.backward(g.root)
        for fuse in (2, 0):
            c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=fuse, arena=128 << 20)
            tiles = c.debug_read(ob.OB_DBG_TILES_PULL).reshape(-1, 48)
            order = c.debug_read(ob.OB_DBG_ORDER)
            seen = 0
            for t in tiles:        # words 0, 5, 6, 7, 40: first schedule position of the batch, row0, edges (all ones: rows differ), rows, stride
                rows = np.searchsorted(ts, order[t[0] + t[5] + np.arange(t[7]) * t[40]])
                if (rows >= 40).any() or not np.array_equal(ts[rows], order[t[0] + t[5] + np.arange(t[7]) * t[40]]):
                    continue
                seen += rows.size
                if not odd[rows].any():
                    assert (t[6] == 2) == (rows.size <= 16), (d, k, fuse, rows)
                elif odd_by in ("count", "kind") and rows.size > 1:
                    assert t[6] == 0xffffffff, (d, k, fuse, rows)
            assert seen == 40
            check_against_oracle(c, p, g, o, root, what=f"pull rows/{d}/{odd_by} at {k}/fuse {fuse}")
            c.close()


@pytest.mark.parametrize("rows,arity", [(1, 8), (1, 9), (3, 9), (300, 2), (300, 8), (300, 9), (2, 700)])
def test_batch_dependencies_of_rows_with_few_and_many_operands(rows, arity):
    """The dependencies between batches are collected row by row, up to eight operands by the row's own thread and more
    by its workgroup; the operands here come from many batches in another order for each row, and a workgroup's rows
    meet more distinct dependencies than its set in LDS places close together."""
    from paper_1705_07860_amd import binding as ob
    rng = np.random.default_rng(rows * 1000 + arity)
    pb = wl.ParamBuilder(rng, std=0.3)
    E = pb.add("E", 1, 4)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    level = [gb.input(rng.standard_normal(4)) for _ in range(40)]
    pool = list(level)
    for k in range(30):                       # chains of different depth: every level is a batch of its own
        level = [gb.tanh(v) if (i + k) % 3 else gb.sigmoid(v) for i, v in enumerate(level)]
        pool += level
    losses = [gb.sqnorm(gb.add([pool[i] for i in rng.choice(len(pool), size=arity, replace=False)])) for _ in range(rows)]
    g = gb.finish(gb.add(losses + [gb.sqnorm(gb.lookup(E, 0))]), rows)
    o = Oracle(g, p, "f64")
    o.forward()
    o.backward(g.root)
    for fuse in (2, 1):
        c, root = run_gpu(p, g, ob.OB_BYDEPTH, fuse=fuse, arena=256 << 20)
        check_against_oracle(c, p, g, o, root, what=f"dependencies/{rows}/{arity}/fuse {fuse}")
        c.close()


def _median_schedule_ms(graphs, rounds=7, wide=None):
    """Median scheduling time (GPU events) of each of the given (params, graph) pairs, taken in turn, the first
    round of each left out.  wide: for each, whether it is planned by the launches for large graphs whatever its size."""
    from paper_1705_07860_amd import binding as ob
    ctxs = []
    for k, (p, _) in enumerate(graphs):
        c = ob.Context(arena_bytes=512 << 20, mode=ob.OB_BYDEPTH)
        c.params_create(p)
        if wide:
            c.debug_set(ob.OB_DBG_SET_WIDE_PLAN, wide[k])
        ctxs.append(c)
    ms = [[] for _ in graphs]
    for i in range(rounds + 1):
        for k, (_, g) in enumerate(graphs):
            ctxs[k].graph_new()
            ctxs[k].add_bulk(g)
            ctxs[k].forward(g.root)
            if i:
                ms[k].append(ctxs[k].stats()["ms_schedule"])
    for c in ctxs:
        c.close()
    return [float(np.median(m)) for m in ms]


def test_a_fused_plan_on_few_compute_units_costs_little_more_than_an_unfused_one(workload_cache):
    """A schedule stream confined to 32 compute units plans 64 sentences with a character model (189 000 nodes), with launch
    fusion and without: 1.17 times the time.  With a workgroup that fills a unit for every 256 nodes, to look for gated cells
    in, it was 1.30 times."""
    import torch
    from paper_1705_07860_amd import binding as ob
    p, g, _ = workload_cache("tagger_char")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    raw = [ob.stream_create_on_cus(32, n_cu - 32), ob.stream_create_on_cus(0, 32)]
    ex, sc = torch.cuda.ExternalStream(raw[0]), torch.cuda.ExternalStream(raw[1])
    ms = {0: [], 2: []}
    ctxs = {}
    for fuse in ms:
        ctxs[fuse] = ob.Context(arena_bytes=1 << 30, stream=ex, sched_stream=sc)
        ctxs[fuse].set_fusion(fuse)
        ctxs[fuse].params_create(p)
    for i in range(12):
        for fuse, c in ctxs.items():
            c.graph_new()
            c.add_bulk(g)
            c.forward(g.root)
            if i:
                ms[fuse].append(c.stats()["ms_schedule"])
    for c in ctxs.values():
        c.close()
    torch.cuda.synchronize()
    for h in raw:
        ob.stream_destroy(h)
    unfused, fused = float(np.median(ms[0])), float(np.median(ms[2]))
    say(f"  unfused {unfused:.3f} ms, fused {fused:.3f} ms")
    assert fused <= 1.25 * unfused


def _sum_recurrences(n, steps, arity):
    """n recurrences; every step adds up `arity` rows: the product of the state before it and looked-up rows."""
    rng = np.random.default_rng(arity)
    pb = wl.ParamBuilder(rng, std=0.1)
    E, W = pb.add("E", 50, 16), pb.add("W", 16, 16)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    losses = []
    for _ in range(n):
        h = gb.lookup(E, 0)
        for _ in range(steps):
            h = gb.tanh(gb.add([gb.matvec(W, -1, h)] + [gb.lookup(E, int(r)) for r in rng.integers(0, 50, arity - 1)]))
        losses.append(gb.sqnorm(h))
    return p, gb.finish(gb.add(losses), n)


@pytest.mark.parametrize("arity", [5, 12])
def test_recurrences_over_wider_sums_schedule_about_as_fast(arity):
    """The depth pass keeps four operands of a node at hand.  Nodes with more must not be what a schedule's time goes
    to: the same recurrences with sums of 5 and 12 operands have 1.2 and 2.3 times the nodes and measure 1.2 times
    the time; walked one after the other by their waves they took 14 to 16 times as long."""
    four, more = _median_schedule_ms([_sum_recurrences(64, 60, 4), _sum_recurrences(64, 60, arity)])
    say(f"  4 operands {four:.3f} ms, {arity} operands {more:.3f} ms")
    assert more <= 4 * four


def _random_arity_graph(n, arities, reach, seed):
    """n nodes of one element.  The arity of a node is drawn from `arities` (less where there are not as many nodes
    before it), its operands from the `reach` nodes before it or, one time in four, from all of them."""
    rng = np.random.default_rng(seed)
    gb = wl.GraphBuilder(wl.Params([], []))
    for v in range(n):
        a = min(int(rng.choice(arities)), v)
        if a == 0:
            gb.input(rng.standard_normal(1))
            continue
        low = 0 if rng.integers(4) == 0 else max(0, v - reach)
        ops = [int(u) for u in rng.integers(low, v, size=a)]
        if rng.integers(2):
            ops[int(rng.integers(a))] = v - 1
        gb.tanh(ops[0]) if a == 1 else gb.add(ops)
    return gb.finish(n - 1, 1)


@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 2049, 6000])
@pytest.mark.parametrize("arities,reach", [([0, 1, 2, 3, 4, 5], 40), ([0, 0, 0, 1, 4, 5, 6, 12, 13], 600), ([0] * 30 + [1, 511, 512, 513, 800], 1500),
                                           ([5], 8), ([3, 9], 3000), ([0] * 200 + [1] * 20 + [2600], 5000)])
def test_depths_of_nodes_of_any_arity_across_id_ranges(n, arities, reach):
    """The depth pass goes by ranges of 1024 ids.  Up to four operands of a node are looked at together, more through a
    window of three, and the longest lists by a whole wave 512 entries at a time (which of the two depends on how many such
    nodes its wave has), with operands in the range itself and in lower ones: depths are exact and nothing is repeated.
    Signatures of such nodes are put together by one thread or by many: the batches are those of the reference."""
    from paper_1705_07860_amd import binding as ob
    g = _random_arity_graph(n, arities, reach, n + len(arities))
    c = ob.Context(arena_bytes=512 << 20, mode=ob.OB_BYDEPTH)
    c.add_bulk(g)
    c.forward(g.root)
    assert np.array_equal(c.debug_read(ob.OB_DBG_DEPTH).astype(np.int64), S.depths(g))
    assert c.stats()["n_depth_retries"] == 0
    for got, want in zip(c.schedule_read(), S.by_depth(g)):
        assert np.array_equal(got, want)
    c.close()


def _dag_of(n, seed, dim):
    """The first n - 1 nodes of a random graph over all operations, and the squared norm of the last of them as its root."""
    p, g = wl.random_dag(seed, n_nodes=n + 40, dim=dim)
    assert len(g.op) >= n
    g = _graph_part(g, 0, n - 1)
    last = {"op": wl.OP_SQNORM, "out_dim": 1, "in_off": int(g.in_off[-1]) + 1, "in_idx": n - 2, "param": -1, "bias": -1, "aux0": 0, "aux1": 0}
    for k, v in last.items():
        a = getattr(g, k)
        setattr(g, k, np.append(a, np.asarray(v, a.dtype)))
    g.root = n - 1
    return p, g


def _plan(p, g, wide, fuse, copy):
    """Everything that a schedule fixes, and what the forward and backward passes of it give."""
    from paper_1705_07860_amd import binding as ob
    c = ob.Context(arena_bytes=512 << 20, mode=ob.OB_BYDEPTH)
    c.set_fusion(fuse)
    c.params_create(p)
    c.param_grad_zero()
    c.debug_set(ob.OB_DBG_SET_WIDE_PLAN, wide)
    c.debug_set(ob.OB_DBG_SET_CONCAT_COPY, copy)
    c.add_bulk(g)
    root = len(g.op) - 1
    c.forward(root)
    out = {k: c.debug_read(getattr(ob, "OB_DBG_" + k)) for k in ("DEPTH", "SIG", "SUCC_OFF", "SUCC_EDGE", "ORDER", "VAL_OFF",
                                                               "CHAINS", "LORDER")}
    total = int(g.out_dim.sum())
    out["values"] = c.all_read(0, total).view(np.uint32)
    if g.out_dim[root] == 1:
        c.backward(root)
        out["gradients"] = c.all_read(1, total).view(np.uint32)
        for pid, m in enumerate(p.mats):
            out[f"parameter {pid}"] = c.param_grad_read(pid, m.shape).view(np.uint32)
    st = c.stats()
    out["counts"] = np.array([st[k] for k in sorted(st) if k.startswith("n_") and k != "n_launch_sched"])
    c.close()
    return out, st["n_launch_sched"]


def _same_plan(p, g, fuse=2, copy=0):
    small, few = _plan(p, g, 0, fuse, copy)
    wide, many = _plan(p, g, 1, fuse, copy)
    assert (few < many) == (len(g.op) <= 2048 and 0 < int(g.in_off[-1]) <= 4096)
    assert small.keys() == wide.keys()
    for k in small:
        assert np.array_equal(small[k], wide[k]), k


@pytest.mark.parametrize("n", [2, 3, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("dim,fuse,copy", [(6, 2, 0), (32, 1, 1), (33, 2, 0)])
def test_a_small_graph_is_scheduled_as_a_large_one_would_be(n, dim, fuse, copy):
    """Graphs of up to 2 048 nodes and 4 096 edges are scheduled by one workgroup in one launch: every table is that of the
    launches for larger graphs, around the sizes where a workgroup takes a second round and where the rule ends."""
    p, g = _dag_of(n, 40 + n + dim, dim)
    _same_plan(p, g, fuse, copy)


@pytest.mark.parametrize("n,arities,reach", [(2048, [0, 0, 0, 1, 2], 40), (1100, [2, 3], 700), (1025, [0] * 400 + [1] * 200 + [9] * 50 + [800] * 2, 1000),
                                             (700, [4, 5, 6, 9], 8), (2048, [0] * 40 + [33], 2000), (1366, [3], 5), (1368, [3], 5),
                                             (2048, [0] * 900 + [1, 5, 12, 13, 24, 25, 511, 512, 513], 2000), (1024, [0] * 250 + [1] * 20 + [13, 700], 900),
                                             (900, [4, 3, 2], 3)])
def test_a_small_graph_of_any_arity_is_scheduled_as_a_large_one_would_be(n, arities, reach):
    """The same with operand lists of every length and with edges on both sides of the 4 096 that the rule allows."""
    _same_plan(wl.Params([], []), _random_arity_graph(n, arities, reach, n + len(arities)))


def _one_sum(rows):
    gb = wl.GraphBuilder(wl.Params([], []))
    return wl.Params([], []), gb.finish(gb.add([gb.input(np.ones(1)) for _ in range(rows)]), 1)


@pytest.mark.parametrize("graph", [lambda: _one_sum(2046), lambda: _one_sum(1100), lambda: _sum_recurrences(1, 140, 12)], ids=["2046", "1100", "140 of 12"])
def test_wide_sums_of_a_small_graph_schedule_no_slower_than_in_a_large_one(graph):
    """The one launch that plans small graphs takes long operand lists by whole waves and shorter ones ahead of their last
    operand: 0.73, 0.75 and 0.78 of the time of the launches for large graphs.  Walked two by two in list order by a thread each,
    the sums took 2.1 and 1.5 times as long as those, the steps over sums of twelve 1.4 times."""
    pg = graph()
    one, many = _median_schedule_ms([pg, pg], rounds=15, wide=[0, 1])
    say(f"  one launch {one:.3f} ms, many {many:.3f} ms")
    assert one <= 1.1 * many


@pytest.mark.parametrize("H,nf,sums,rows", [(8, 1, True, 20), (64, 2, False, 12), (100, 0, True, 9)])
def test_a_small_graph_of_gated_cells_is_scheduled_as_a_large_one_would_be(H, nf, sums, rows):
    p, g = _cell_graph(H, nf, sums, rows, None)
    assert len(g.op) <= 2048
    _same_plan(p, g)


def test_depths_of_more_id_ranges_than_the_chip_holds_at_once():
    """1 026 ranges of 1 024 ids, operands drawn from all nodes before: a range waits for any lower one, also where not
    all of them can be on the chip together."""
    from paper_1705_07860_amd import binding as ob
    n = 1024 * 1025 + 3
    rng = np.random.default_rng(n)
    arity = rng.integers(2, 4, size=n)
    arity[rng.random(n) < 0.6] = 0
    arity[:3] = 0
    arity[-1] = 2
    in_off = np.concatenate([[0], np.cumsum(arity)])
    cons = np.repeat(np.arange(n), arity)
    leaf = arity == 0
    zero, none = np.zeros(n, np.int64), np.full(n, -1)
    g = wl.Graph(op=np.where(leaf, wl.OP_INPUT, wl.OP_ADD), out_dim=zero + 1, in_off=in_off,
                 in_idx=(rng.random(cons.size) * cons).astype(np.int64), param=none, bias=none,
                 aux0=np.where(leaf, np.cumsum(leaf) - 1, 0), aux1=zero, payload=rng.standard_normal(int(leaf.sum())), root=n - 1)
    c = ob.Context(arena_bytes=4 << 30, mode=ob.OB_BYDEPTH)
    c.add_bulk(g)
    c.forward(g.root)
    assert np.array_equal(c.debug_read(ob.OB_DBG_DEPTH).astype(np.int64), S.depths(g))
    assert c.stats()["n_depth_retries"] == 0
    c.close()


def test_a_long_path_through_many_id_ranges_is_no_reason_to_give_up():
    """The bound on a range's wait is on idle polls while nothing below it ends.  A chain of 100 000 nodes ends a wave of
    256 ids every 30 to 40 us, some 50 polls; its last ranges wait some 20 000 polls in all, over three times the bound set here
    (which must be above 1 024: ended waves are looked at once in as many polls)."""
    from paper_1705_07860_amd import binding as ob
    gb = wl.GraphBuilder(wl.Params([], []))
    h = gb.input(np.ones(4))
    for _ in range(100000):
        h = gb.tanh(h)
    g = gb.finish(gb.sqnorm(h), 1)
    c = ob.Context(arena_bytes=1 << 30, mode=ob.OB_BYDEPTH)
    c.debug_set(ob.OB_DBG_SET_DEPTH_SPIN, 6000)
    c.add_bulk(g)
    c.forward(g.root)
    assert np.array_equal(c.debug_read(ob.OB_DBG_DEPTH), np.arange(g.n))
    assert c.stats()["n_depth_retries"] == 0
    c.close()


def _sums_side_by_side(m, arity):
    """m sums with neighbouring ids, each of `arity` of the same 2048 rows."""
    rng = np.random.default_rng(arity)
    pb = wl.ParamBuilder(rng, std=0.1)
    E = pb.add("E", 50, 16)
    p = pb.done()
    gb = wl.GraphBuilder(p)
    xs = [gb.lookup(E, int(r)) for r in rng.integers(0, 50, 2048)]
    ys = [gb.add([xs[i] for i in rng.integers(0, 2048, arity)]) for _ in range(m)]
    return p, gb.finish(gb.add([gb.sqnorm(y) for y in ys]), m)


def test_sums_of_nine_operands_schedule_about_as_fast_as_of_eight():
    """Up to eight operands of a node are taken by one thread where nodes are set up and where the dependencies between
    batches are collected, more by its workgroup: neither may be what a schedule's time goes to.  Taken by the workgroup
    node after node in both, the sums of nine made scheduling 4.1 times as long as those of eight, in the second alone 1.5
    times; with the operands shared out over the threads it is 1.0."""
    eight, nine = _median_schedule_ms([_sums_side_by_side(4096, 8), _sums_side_by_side(4096, 9)])
    say(f"  8 operands {eight:.3f} ms, 9 operands {nine:.3f} ms")
    assert nine <= 1.25 * eight
