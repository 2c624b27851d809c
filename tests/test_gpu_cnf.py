"""GPU parity: the CNF transformation (tt_cnf_transform) against the
oracle's Algorithm 1, expression by expression (output, kind, clause range,
variables, table, support) and variable class by variable class."""
import json
import pathlib

import numpy as np
import pytest

import paper_2502_08673_amd as tt
from gpu_util import note
from oracle import transform as T
from workloads import tseitin_instances

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
GOLDEN = pathlib.Path(__file__).parent / "golden"


def run(instances):
    lits, coff, ioff, nv = tt.cnf_csr(instances)
    n_inst = len(instances)
    n_cl = int(ioff[-1])
    var_class = torch.full((int((nv + 1).sum()),), 0xEE, dtype=torch.uint8, device="cuda")
    expr = torch.zeros((max(n_cl, 1) * 640,), dtype=torch.uint8, device="cuda")
    n_expr = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    status = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    note(f"cnf_transform instances={n_inst} clauses={n_cl}")
    tt.cnf_transform(lits, coff, ioff, nv, var_class, expr, n_expr, status)
    torch.cuda.synchronize()
    recs = expr.cpu().numpy().view(tt.CNF_EXPR_DTYPE)
    return var_class.cpu().numpy(), recs, n_expr.cpu().numpy(), status.cpu().numpy(), ioff, nv


KIND = {"IV": tt.TT_CNF_IV, "PO": tt.TT_CNF_PO, "AUX": tt.TT_CNF_AUX}


def table_int(rec):
    n = int(rec["n_vars"])
    words = [int(w) for w in rec["table"]]
    t = sum(w << (64 * i) for i, w in enumerate(words))
    return t & ((1 << (1 << n)) - 1)


def check_instance(t, clauses, nv, var_class, recs, n_expr, status, ioff, voff, stop_at=None):
    PO, PI, IV, E = T.transform(clauses if stop_at is None else clauses[:stop_at])
    if stop_at is not None:  # the device stopped at clause stop_at: compare what was found before
        E = [e for e in E if e.last < stop_at - 1 or e.kind != "AUX"]
    assert n_expr[t] == len(E), t
    base = int(ioff[t])
    for q, e in enumerate(E):
        r = recs[base + q]
        assert int(r["out"]) == e.out and int(r["kind"]) == KIND[e.kind], (t, q)
        assert (int(r["first"]), int(r["last"])) == (e.first, e.last), (t, q)
        n = int(r["n_vars"])
        assert list(r["vars"][:n]) == e.vars, (t, q)
        assert table_int(r) == e.table, (t, q)
        sup = [e.vars[j] for j in range(n) if (int(r["support"]) >> j) & 1]
        assert sup == e.support, (t, q)
    if stop_at is None:
        cls = var_class[voff: voff + nv + 1]
        for x in range(1, nv + 1):
            assert bool(cls[x] & tt.TT_CNF_CLS_PI) == (x in PI), (t, x)
            assert bool(cls[x] & tt.TT_CNF_CLS_IV) == (x in IV), (t, x)
            assert bool(cls[x] & tt.TT_CNF_CLS_PO) == (x in PO), (t, x)


def test_fig1_and_worked_example():
    g = json.loads((GOLDEN / "fig1_cnf.json").read_text())
    inst = [(14, T.parse_dimacs(g["dimacs"])),
            (108, [[-4, -107, 5], [-4, 107, -5], [4, -108, 5], [4, 108, -5]])]
    var_class, recs, n_expr, status, ioff, nv = run(inst)
    assert list(status) == [0, 0]
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, var_class, recs, n_expr, status, ioff, voff)
        voff += n + 1


def test_random_tseitin_batch():
    """300 random circuits as CNF (gates of every kind, unit constraint on
    the last output), plus an empty instance and unit clauses."""
    inst = tseitin_instances(seed=123, n_inst=300)
    inst.insert(7, (3, []))
    inst.insert(50, (5, [[-5], [2, 3], [1]]))
    var_class, recs, n_expr, status, ioff, nv = run(inst)
    assert (status == 0).all()
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, var_class, recs, n_expr, status, ioff, voff)
        voff += n + 1


def test_wide_tables_and_limit():
    """An XOR of five inputs (SC of 6 variables, one-word tables), an 11-input
    AND (a 2^11-row table over 32 words, 12-variable auxiliary tables), and a
    chain of binary clauses whose SC outgrows 12 variables (status 1, the
    expressions found before it kept)."""
    xs = [1, 2, 3, 4, 5]
    xor5 = []
    import itertools
    for bits in itertools.product([0, 1], repeat=6):
        if sum(bits) % 2 == 1:
            xor5.append([-x if b else x for x, b in zip(xs + [6], bits)])
    and11 = [[12] + [-x for x in range(1, 12)]] + [[-12, x] for x in range(1, 12)]
    wide_aux = [[x, x + 1] for x in range(1, 12)] + [[-1, -12]]
    chain = [[-2, 1], [2, -1]] + [[x, x + 1] for x in range(3, 20)]
    inst = [(6, xor5), (12, and11), (12, wide_aux), (20, chain)]
    var_class, recs, n_expr, status, ioff, nv = run(inst)
    assert list(status[:3]) == [0, 0, 0] and status[3] == 1
    voff = 0
    for t, (n, cl) in enumerate(inst[:3]):
        check_instance(t, cl, n, var_class, recs, n_expr, status, ioff, voff)
        voff += n + 1
    # the chain: x2 = x1 found first; SC then gathers x3 .. x15 and stops
    # when the thirteenth variable arrives (clause index 2 + 12 - 1 = 13)
    check_instance(3, chain, 20, var_class, recs, n_expr, status, ioff, voff, stop_at=13)


def test_handle_runs_twice_with_identical_results():
    inst = tseitin_instances(seed=9, n_inst=64)
    lits, coff, ioff, nv = tt.cnf_csr(inst)
    n_cl = int(ioff[-1])
    outs = []
    with tt.Cnf(lits, coff, ioff, nv) as h:
        for _ in range(2):
            vc = torch.zeros((int((nv + 1).sum()),), dtype=torch.uint8, device="cuda")
            ex = torch.zeros((n_cl * 640,), dtype=torch.uint8, device="cuda")
            ne = torch.zeros((len(nv),), dtype=torch.int32, device="cuda")
            stt = torch.full((len(nv),), -1, dtype=torch.int32, device="cuda")
            note("cnf handle run")
            h.run(vc, ex, ne, stt)
            torch.cuda.synchronize()
            outs.append((vc.cpu().numpy(), ex.cpu().numpy(), ne.cpu().numpy(), stt.cpu().numpy()))
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    var_class, ex, ne, stt = outs[0]
    recs = ex.view(tt.CNF_EXPR_DTYPE)
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, var_class, recs, ne, stt, ioff, voff)
        voff += n + 1


def test_instance_too_large_for_lds_reads_global_memory():
    """A 2500-gate circuit (about 9000 clauses): its clauses do not fit a
    block's LDS, so the kernel form that reads them from global memory runs;
    same results as the oracle."""
    inst = tseitin_instances(seed=77, n_inst=2, n_gates=(2500, 2500))
    lits, coff, ioff, nv = tt.cnf_csr(inst)
    assert 4 * (2 * (ioff[1] - ioff[0]) + 1 + (coff[ioff[1]] - coff[ioff[0]])) > 64 * 1024
    var_class, recs, n_expr, status, ioff, nv = run(inst)
    assert (status == 0).all()
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, var_class, recs, n_expr, status, ioff, voff)
        voff += n + 1


def test_repeated_literals_count_once():
    """A clause is a set of literals: (x1 x1) is the unit clause (x1), and
    (-x2 -x2)(x1 x2) defines x1 from nothing once -x2 is a unit.  Both must
    match the oracle, which reads every clause as a set."""
    inst = [(1, [[1, 1]]), (2, [[-2, -2], [1, 2]]), (3, [[1, 2, 1], [-3, 2, 2], [3, -2]])]
    var_class, recs, n_expr, status, ioff, nv = run(inst)
    assert list(status) == [0, 0, 0]
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, var_class, recs, n_expr, status, ioff, voff)
        voff += n + 1


def _and(ins, f):
    return [[f] + [-x for x in ins]] + [[-f, x] for x in ins]


@pytest.mark.parametrize("n_inst,offset", [(1, 0), (9, 0), (70, 0), (9, 8)])
def test_variable_order_and_sc_sizes_around_the_eight_lane_form(n_inst, offset):
    """Instances whose SC reaches 2 to 8 variables (the eight-lane form holds
    five, its clauses five literals; the others go to a wave each, before or
    after they started in eight lanes), in shuffled variable names so that no
    order of first use is the sorted one, with partial groups of eight (1, 9,
    70 instances) and with records at an 8-byte offset."""
    rng = np.random.default_rng(n_inst + offset)
    inst = []
    for t in range(n_inst):
        nv, cl = tseitin_instances(seed=1000 + t, n_inst=1)[0]
        k = 2 + t % 7
        cl = cl + _and(list(range(nv + 1, nv + k)), nv + k)  # SC of k variables, clause of k literals
        m = nv + k
        k = 2 + (t // 2) % 7  # an auxiliary SC of k variables in binary clauses
        cl = cl + [[x, x + 1] for x in range(m + 1, m + k)] + [[-(m + 1), -(m + k)]]
        m += k
        name = rng.permutation(m) + 1
        inst.append((m, [[int(np.sign(L)) * int(name[abs(L) - 1]) for L in c] for c in cl]))
    lits, coff, ioff, nv = tt.cnf_csr(inst)
    n_cl = int(ioff[-1])
    var_class = torch.full((int((nv + 1).sum()),), 0xEE, dtype=torch.uint8, device="cuda")
    buf = torch.zeros((n_cl * 640 + 16,), dtype=torch.uint8, device="cuda")
    expr = buf[offset: offset + n_cl * 640]
    n_expr = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    status = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    note(f"cnf shuffled instances={n_inst} offset={offset}")
    tt.cnf_transform(lits, coff, ioff, nv, var_class, expr, n_expr, status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    recs = expr.cpu().numpy().view(tt.CNF_EXPR_DTYPE)
    vc, ne = var_class.cpu().numpy(), n_expr.cpu().numpy()
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, vc, recs, ne, status.cpu().numpy(), ioff, voff)
        voff += n + 1
    assert not buf[: offset].any() and not buf[offset + n_cl * 640:].any()


@pytest.mark.parametrize("n_inst", [1, 9, 70])
def test_an_instance_goes_on_after_an_sc_that_outgrew_the_eight_lanes(n_inst):
    """A circuit, SCs of six to eight variables in binary clauses, some of them
    the circuit's inputs and outputs (their classes decide what the SC can
    give), a gate of six inputs (a clause of seven literals), and a second
    circuit: the records before, of and after those SCs and the classes, also
    where an SC is the instance's first, and with several in a row (the
    instance then stays with the wave kernel)."""
    rng = np.random.default_rng(n_inst)
    inst = []
    for t in range(n_inst):
        nv, cl = tseitin_instances(seed=1100 + t, n_inst=1)[0] if t % 4 else (0, [])
        k = 6 + t % 3
        old = [int(x) for x in rng.permutation(nv)[: min(nv, t % 5)] + 1]
        xs = [int(x) for x in rng.permutation(old + list(range(nv + 1, nv + 1 + k - len(old))))]
        # the chain's variables occur nowhere later; the circuit before them is closed by its last output
        chain = [[xs[i], -xs[i + 1] if i % 2 else xs[i + 1]] for i in range(k - 1)] + [[-xs[0], -xs[-1]]]
        m = max([nv] + xs)
        for _ in range(t % 7 // 2):  # up to three more in a row
            chain += [[x, x + 1] for x in range(m + 1, m + k)] + [[-(m + 1), -(m + k)]]
            m += k
        if t % 2:
            chain += _and(list(range(m + 1, m + 7)), m + 7)
            m += 7
        nv2, cl2 = tseitin_instances(seed=1200 + t, n_inst=1)[0]
        cl = cl + chain + [[int(np.sign(L)) * (abs(L) + m) for L in c] for c in cl2]
        inst.append((m + nv2, cl))
    lits, coff, ioff, nv = tt.cnf_csr(inst)
    var_class = torch.full((int((nv + 1).sum()),), 0xEE, dtype=torch.uint8, device="cuda")
    expr = torch.zeros((int(ioff[-1]) * 640,), dtype=torch.uint8, device="cuda")
    n_expr = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    status = torch.full((n_inst,), -1, dtype=torch.int32, device="cuda")
    note(f"cnf goes on after a wide SC, instances={n_inst}")
    with tt.Cnf(lits, coff, ioff, nv) as h:
        for _ in range(2):
            h.run(var_class, expr, n_expr, status)
    torch.cuda.synchronize()
    st, recs = status.cpu().numpy(), expr.cpu().numpy().view(tt.CNF_EXPR_DTYPE)
    vc, ne = var_class.cpu().numpy(), n_expr.cpu().numpy()
    voff = 0
    for t, (n, cl) in enumerate(inst):
        check_instance(t, cl, n, vc, recs, ne, st, ioff, voff)
        voff += n + 1
