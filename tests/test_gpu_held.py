"""Plans of FILTER and unconstrained layers whose rows wait for their selection on the chip: the un-predicted projection
is one launch that makes the selection itself and writes every row once.  Every output against the oracle, at the edges of
what a workgroup holds (rows of one to ten chunks a lane, ragged rows, one row to 256 rows an item, layers of one item and
of more groups than the selection ranks from registers), and with no patience at all, so that rows are written before
their selection is known and finished by whoever comes second."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_14628_amd as pkg
import workloads as wk

pytestmark = pytest.mark.gpu

F, C, N = wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_NONE
# (c_out, c_in, khw, mode, k): row lengths 1 .. 10240 floats, on either side of four floats, a wave and the whole workgroup
EDGES = [(700, 1, 1, F, 300), (260, 2, 1, F, 7), (2600, 4, 1, F, 1300), (90, 5, 1, F, 90), (300, 7, 9, F, 100),
         (64, 64, 1, F, 1), (129, 65, 1, F, 64), (40, 255, 1, F, 39), (37, 256, 1, F, 12), (33, 2047, 1, F, 20),
         (18, 2048, 1, F, 5), (21, 2049, 1, F, 11), (1, 512, 9, F, 1), (19, 1024, 9, F, 9), (7, 9215, 1, F, 3),
         (9, 10240, 1, F, 4), (30, 100, 1, N, 30), (3, 2050, 1, N, 3), (300, 6144, 1, F, 120)]   # (size, for the 2600 groups)


# tiles of 64 rows by 256 columns (64 of a ragged row): one row, one strip, channels across strips, more channels than the
# selection ranks from registers, one and all channels kept
TILES = [(1, 4, 1, C, 2), (63, 8, 1, C, 1), (64, 64, 4, C, 30), (65, 65, 4, C, 64), (129, 28, 9, C, 28), (200, 60, 9, C, 25),
         (64, 86, 6, C, 40), (70, 2500, 1, C, 1200), (130, 512, 9, C, 200), (17, 23, 3, C, 5), (40, 100, 1, N, 40),
         (3, 2050, 1, N, 3), (256, 512, 9, C, 200)]              # (size, for the 2500 groups)


@pytest.fixture(params=["", "0"], ids=["patient", "impatient"])
def patience(request, monkeypatch):
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE"):
        monkeypatch.delenv(name, raising=False)
    if request.param:
        monkeypatch.setenv("HSADMM_HELD_PATIENCE", request.param)


def _launches(plan, call):
    pkg.hsadmm_kernel_timing_enable(plan, True)
    call()
    torch.cuda.synchronize()
    got = {k: v[1] for k, v in pkg.hsadmm_kernel_timing_read(plan).items() if v[1]}
    pkg.hsadmm_kernel_timing_enable(plan, False)
    return got


def _weighted_launches(wl, W, U, a, b):
    from tests.gpu_harness import GpuRun
    r = GpuRun(wl, W, U)
    pkg.hsadmm_plan_set_node_weights(r.plan, a, b)
    Zg, Vd = torch.zeros_like(r.dU), torch.zeros_like(r.dU)
    got = _launches(r.plan, lambda: pkg.hsadmm_project_weighted_compact(r.plan, r.dW, r.dU, Zg, Vd, r.dZ, None, r.dmask, None,
                                                                        r.dpacked, r.doff, r.dkept, r.ws))
    r.close()
    return got


def _tiles(wl):
    return sum(-(-l.c_out // 64) * -(-l.c_in * l.khw // (64 if l.c_in * l.khw % 4 else 256)) for l in wl.layers if l.mode == C)


def _early(ws):
    """Items that the last call wrote before their selection was known: their state words are its number (a negative NaN's
    pattern, a multiple of four) and 2 or 3."""
    words = ws.cpu().numpy()[:ws.numel() // 8 * 8].view(np.uint64)
    return int(np.count_nonzero(((words >> np.uint64(50)) == 0x3FFD) & ((words & np.uint64(3)) >= 2)))


@pytest.mark.parametrize("weighted", [False, True], ids=["step", "weighted"])
@pytest.mark.parametrize("mode", [F, C], ids=["filter", "channel"])
@pytest.mark.parametrize("keep", [0.3, 0.7])
def test_rows_written_early_are_finished_by_whoever_comes_second(mode, keep, weighted, monkeypatch):
    """Without patience rows are written before their selection is known, in either early form, and finished by their own
    workgroup or by the one that has selected.  The launch has one workgroup an item: none that waits on behalf of others,
    and could give up."""
    from tests.gpu_harness import GpuRun, check_against_oracle
    from tests.test_gpu_weighted import _phase4_chain
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE"):
        monkeypatch.delenv(name, raising=False)
    monkeypatch.setenv("HSADMM_HELD_PATIENCE", "0")
    wl = wk.custom_workload([(128, 64, 9, mode, int(keep * (128 if mode == F else 64)))], R=4, seed=12, sigma_replica=0.03)
    W, U = wk.generate(wl)
    t = wl.table()
    r = GpuRun(wl, W, U)
    pkg.hsadmm_kernel_timing_enable(r.plan, True)
    if weighted:
        rng = np.random.default_rng(5)
        _phase4_chain(wl, W, U, np.float32([0.6]), np.float32([0.3]), rng, fused_dual=True, one_call=True)
        dev = r.dev
        Zg, Vd = (torch.from_numpy(rng.standard_normal(wl.n_arena).astype(np.float32)).to(dev) for _ in range(2))
        pkg.hsadmm_project_weighted_compact(r.plan, r.dW, r.dU, Zg, Vd, r.dZ, None, r.dmask, None, r.dpacked, r.doff, r.dkept,
                                            r.ws)
    else:
        ref = oracle.project(t, W, U, want_wbar=True)
        r.step(fused=True)
        rep = check_against_oracle(wl, r.outputs(), ref, oracle.compact(t, ref["Z"], ref["mask"]))
        assert all(v == 0 for v in rep.values()), rep
    torch.cuda.synchronize()
    assert _early(r.ws) >= 1
    grid = pkg.hsadmm_kernel_grids(r.plan)["weighted_pass1" if weighted else "project_pass1"]
    # rows of 144 chunks share a wave: four at once, one slot's worth an item; tiles of 64 rows by 256 columns
    assert grid == (32 if mode == F else 6)
    r.close()


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 8])
def test_edges_of_what_a_workgroup_holds(R, patience):
    from tests.gpu_harness import GpuRun
    from tests.test_gpu_parity import _run
    wl = wk.custom_workload(EDGES, R=R, seed=40 + R, sigma_replica=0.03)
    _run(wl, pack_align=4 if R == 3 else 1)
    r = GpuRun(wl, *wk.generate(wl))
    assert _launches(r.plan, r.project_compact) == {"project_pass1": 1}
    r.close()


@pytest.mark.parametrize("R", [1, 2, 3, 4, 8])
def test_edges_with_the_full_candidate(R, patience):
    """The candidate of Eq. (9), with and without the shrinkage, then the expansion with the inter-node dual: against the
    oracle's chain."""
    from tests.test_gpu_weighted import _phase4_chain
    wl = wk.custom_workload(EDGES, R=R, seed=60 + R, sigma_replica=0.03)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(R)
    L = len(wl.layers)
    a, b = rng.uniform(0.3, 1.0, L).astype(np.float32), rng.uniform(0.0, 0.7, L).astype(np.float32)
    for one_call in (True, False):
        _phase4_chain(wl, W, U, a, b, rng, fused_dual=True, one_call=one_call)
    assert _weighted_launches(wl, W, U, a, b) == {"weighted_pass1": 1}


@pytest.mark.parametrize("R", [1, 2, 3, 4, 8])
def test_tiles_of_channel_groups(R, patience):
    from tests.gpu_harness import GpuRun
    from tests.test_gpu_parity import _run
    from tests.test_gpu_weighted import _phase4_chain
    wl = wk.custom_workload(TILES, R=R, seed=80 + R, sigma_replica=0.03)
    _run(wl, pack_align=4 if R == 3 else 1)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(R)
    L = len(wl.layers)
    a, b = rng.uniform(0.3, 1.0, L).astype(np.float32), rng.uniform(0.0, 0.7, L).astype(np.float32)
    for one_call in (True, False):
        _phase4_chain(wl, W, U, a, b, rng, fused_dual=True, one_call=one_call)
    r = GpuRun(wl, W, U)
    assert _launches(r.plan, r.project_compact) == {"project_pass1": 1}
    r.close()
    # (eight replicas: fewer than 80 tiles keep the other path)
    assert (_weighted_launches(wl, W, U, a, b) == {"weighted_pass1": 1}) == (R != 8 or _tiles(wl) >= 80)


@pytest.mark.parametrize("n_layers", [1, 40])
def test_small_and_full_items(n_layers, patience):
    """Layers alone (items of one chunk a lane) and enough of them to fill every place with ten."""
    from tests.test_gpu_parity import _run
    _run(wk.custom_workload([(128, 64, 9, F, 50), (96, 512, 1, F, 40)] * n_layers + [(64, 96, 1, N, 64)], R=2, seed=3,
                            sigma_replica=0.03), determinism=False)


@pytest.mark.parametrize("shapes", [
    [(384, 128, 9, F, 150), (512, 256, 1, F, 200), (100, 512, 1, N, 100), (300, 147, 1, F, 100)],
    [(384, 128, 9, C, 50), (512, 256, 1, C, 200), (100, 512, 1, N, 100), (300, 148, 1, C, 100)]], ids=["filter", "channel"])
def test_steps_on_one_workspace_with_every_option_and_replayed(shapes, patience):
    """Outer iterations with the selection record, the dual in place and in a second buffer, on one scratch that starts as
    garbage, then replayed from a captured graph (where a call's number is always the same)."""
    wl = wk.custom_workload(shapes, R=3, seed=8, sigma_replica=0.03)
    W, U = wk.generate(wl)
    t = wl.table()
    dev = torch.device("cuda:0")
    plan = pkg.Plan(t)
    dW = [torch.from_numpy(np.ascontiguousarray(W[r])).to(dev) for r in range(wl.R)]
    refs, u = [], U.copy()
    for _ in range(6):
        refs.append(oracle.project(t, W, u))
        u = refs[-1]["U"]

    def buffers():
        n = wl.n_arena
        return {"U": torch.from_numpy(U.copy()).to(dev), "U2": torch.zeros(n, device=dev), "Z": torch.zeros(n, device=dev),
                "mask": torch.zeros(plan.groups_total, dtype=torch.uint8, device=dev),
                "sel": torch.zeros(plan.groups_total, dtype=torch.int32, device=dev),
                "ws": torch.full((plan.workspace_bytes,), 0xF4, dtype=torch.uint8, device=dev),
                "packed": torch.zeros(plan.packed_capacity_elems, device=dev),
                "off": torch.zeros(plan.n_layers + 1, dtype=torch.int64, device=dev),
                "kept": torch.zeros(plan.groups_total, dtype=torch.int32, device=dev)}

    def step(b, out_of_place, stream=None):
        pkg.hsadmm_step(plan, dW, U=b["U"], U_out=b["U2"] if out_of_place else None, Z=b["Z"], mask=b["mask"], sel=b["sel"],
                        packed=b["packed"], layer_off=b["off"], kept_idx=b["kept"], workspace=b["ws"], stream=stream)

    def check(b, it, dual):
        torch.cuda.synchronize()
        ref = refs[it]
        assert np.array_equal(b["mask"].cpu().numpy(), ref["mask"]), it
        for name, want in (("Z", ref["Z"]), (dual, ref["U"])):
            g = b[name].cpu().numpy()
            for l in wl.layers:
                sl = slice(l.elem_off, l.elem_off + l.n)
                assert np.array_equal(g[sl].view(np.uint32), want[sl].view(np.uint32)), (it, name, l.name)
        refc = oracle.compact(t, ref["Z"], ref["mask"])
        assert np.array_equal(b["off"].cpu().numpy(), refc["layer_off"])
        assert np.array_equal(b["kept"].cpu().numpy()[:refc["kept_idx"].size], refc["kept_idx"])
        assert np.array_equal(b["packed"].cpu().numpy()[:refc["packed"].size].view(np.uint32), refc["packed"].view(np.uint32))
        ranks = np.concatenate([np.where(m, np.cumsum(m) - 1, -1) for m in
                                (ref["mask"][l.group_base:l.group_base + l.groups].astype(np.int64) for l in wl.layers)])
        assert np.array_equal(b["sel"].cpu().numpy(), ranks), it

    b = buffers()
    for it in range(6):
        step(b, it % 2 == 1)
        check(b, it, "U2" if it % 2 else "U")
        if it % 2:
            b["U"].copy_(b["U2"])

    g = buffers()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step(g, False, stream=side)
    torch.cuda.synchronize()
    scratch = torch.zeros(1 << 16, device=dev)
    for it in range(6):
        graph.replay()
        check(g, it, "U")
        scratch.add_(1.0)
    plan.close()


def test_equal_rows_go_to_the_lower_index(patience):
    from tests.gpu_harness import GpuRun, check_against_oracle
    wl = wk.custom_workload([(300, 128, 1, F, 150), (2500, 16, 1, F, 1100)], R=4, seed=3, sigma_replica=0.03)
    W, U = (np.array(x) for x in wk.generate(wl))
    for l, n in ((wl.layers[0], 128), (wl.layers[1], 16)):
        for r in range(1, l.c_out):
            at = l.elem_off + n * r
            W[:, at:at + n] = W[:, l.elem_off:l.elem_off + n]
            U[at:at + n] = U[l.elem_off:l.elem_off + n]
    t = wl.table()
    ref = oracle.project(t, W, U, want_wbar=True)
    r = GpuRun(wl, W, U)
    r.step(fused=True)
    rep = check_against_oracle(wl, r.outputs(), ref, oracle.compact(t, ref["Z"], ref["mask"]))
    assert all(v == 0 for v in rep.values()), rep
    r.close()


def test_two_streams_at_once(patience):
    """Two calls at the same time, each wanting every place on the chip."""
    wl = wk.custom_workload([(512, 512, 9, F, 200)] * 4 + [(2048, 512, 1, F, 900)] * 3, R=2, seed=5, sigma_replica=0.03)
    W, U = wk.generate(wl)
    ref = oracle.project(wl.table(), W, U)
    dev = torch.device("cuda:0")
    plan = pkg.Plan(wl.table())
    dW = [torch.from_numpy(np.ascontiguousarray(W[r])).to(dev) for r in range(wl.R)]
    dU = torch.from_numpy(U.copy()).to(dev)
    sets = []
    for _ in range(2):
        sets.append((torch.cuda.Stream(), torch.zeros_like(dU), torch.zeros_like(dU),
                     torch.zeros(plan.groups_total, dtype=torch.uint8, device=dev),
                     torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device=dev)))
    torch.cuda.synchronize()
    for _ in range(5):
        for st, U2, Z, mask, ws in sets:
            pkg.hsadmm_step(plan, dW, U=dU, U_out=U2, Z=Z, mask=mask, workspace=ws, stream=st)
    torch.cuda.synchronize()
    for _, U2, Z, mask, _ in sets:
        assert np.array_equal(mask.cpu().numpy(), ref["mask"])
        for got, want in ((Z, ref["Z"]), (U2, ref["U"])):
            g = got.cpu().numpy()
            for l in wl.layers:
                sl = slice(l.elem_off, l.elem_off + l.n)
                assert np.array_equal(g[sl].view(np.uint32), want[sl].view(np.uint32)), l.name
    plan.close()


@pytest.mark.parametrize("shape", [(1024, 1024, 9, C, 400), (768, 10240, 1, F, 300)], ids=["tiles", "rows"])
def test_the_largest_layers_find_their_places(shape, monkeypatch):
    """Layers of as many items as a plan may count on (three quarters of the places): alone on the device none of them waits
    in vain."""
    from tests.gpu_harness import GpuRun
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE", "HSADMM_HELD_PATIENCE"):
        monkeypatch.delenv(name, raising=False)
    wl = wk.custom_workload([shape], R=2, seed=4, sigma_replica=0.03)
    W, U = wk.generate(wl, threads=8)
    ref = oracle.project(wl.table(), W, U)
    r = GpuRun(wl, W, U, want_wbar=False)
    assert _launches(r.plan, r.project_compact) == {"project_pass1": 1}
    assert _early(r.ws) == 0
    assert np.array_equal(r.dmask.cpu().numpy(), ref["mask"])
    r.close()


@pytest.mark.parametrize("mode", [F, C], ids=["filter", "channel"])
@pytest.mark.parametrize("groups,size,one", [(2048, 0, True), (2304, 255, False), (2304, 256, True), (16384, 14336, True),
                                             (16388, 14340, False)])
def test_layers_of_many_groups_wait_only_where_their_selection_is_worth_it(mode, groups, size, one, monkeypatch):
    """A layer of more groups than the selecting workgroup ranks from registers, in plans of `size` times 4096 elements beside
    it, on either side of both lines of the rule."""
    from tests.gpu_harness import GpuRun, check_against_oracle
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE", "HSADMM_HELD_PATIENCE"):
        monkeypatch.delenv(name, raising=False)
    unit, few = (4 if mode == F else 64), 4096                   # floats a group; columns of the other layers
    own = groups * unit
    rest = max(0, size * 4096 - own)
    shapes = [(groups, unit, 1, mode, groups // 3) if mode == F else (unit, groups, 1, mode, groups // 3)]
    while rest > 0:                                              # ... other layers make up the size, the last one a part
        rows = min(512, -(-rest // few)) if rest >= few else 1
        cols = few if rest >= few else rest // 4 * 4
        rows = min(rows, rest // cols)
        shapes.append((rows, cols // 4, 4, mode, max(1, (rows if mode == F else cols // 4) // 2)))
        rest -= rows * cols
    wl = wk.custom_workload(shapes, R=1, seed=6, sigma_replica=0.03)
    assert sum(l.n for l in wl.layers) // 4096 == max(size, own // 4096)
    W, U = wk.generate(wl, threads=8)
    t = wl.table()
    ref = oracle.project(t, W, U, want_wbar=True)
    r = GpuRun(wl, W, U)
    got = _launches(r.plan, lambda: r.step(fused=True))
    assert (got.get("select_topk", 0) == 0) == one, got
    rep = check_against_oracle(wl, r.outputs(), ref, oracle.compact(t, ref["Z"], ref["mask"]))
    assert all(v == 0 for v in rep.values()), rep
    assert _early(r.ws) == 0
    r.close()


@pytest.mark.parametrize("weighted", [False, True], ids=["step", "weighted"])
@pytest.mark.parametrize("mode", [F, C], ids=["filter", "channel"])
def test_values_that_are_not_finite_fare_as_in_separate_launches(mode, weighted, monkeypatch):
    """Infinities, NaN, zeros of both signs, the smallest and largest magnitudes and layers of zeros (every key tied): the one
    launch against the launches it takes the place of, bit for bit where a value is not NaN."""
    monkeypatch.delenv("HSADMM_FORCE_ESTIMATE", raising=False)
    shapes = [(96, 64, 9, mode, 40), (130, 256, 1, mode, 60), (64, 48, 1, mode, 48 if mode == C else 64), (40, 100, 1, mode, 3)]
    wl = wk.custom_workload(shapes, R=3, seed=17, sigma_replica=0.03)
    W, U = (np.array(x) for x in wk.generate(wl))
    rng = np.random.default_rng(2)
    for l, values in ((wl.layers[0], [np.inf, -np.inf, 0.0, -0.0, 1e-45, 3e38]), (wl.layers[1], [np.nan, np.inf, -3e38, 1e-40])):
        at = l.elem_off + rng.choice(l.n, 4 * len(values), replace=False)
        W[:, at] = np.float32(values * 4)
        U[l.elem_off + rng.choice(l.n, len(values), replace=False)] = np.float32(values)
    last = wl.layers[-1]
    W[:, last.elem_off:last.elem_off + last.n] = 0.0
    U[last.elem_off:last.elem_off + last.n] = 0.0
    n, dev = wl.n_arena, torch.device("cuda:0")
    zv = rng.standard_normal((2, n)).astype(np.float32)

    def outputs(held):
        if held:
            monkeypatch.delenv("HSADMM_NO_ESTIMATE", raising=False)
        else:
            monkeypatch.setenv("HSADMM_NO_ESTIMATE", "1")
        plan = pkg.Plan(wl.table())
        dW = [torch.from_numpy(np.ascontiguousarray(w)).to(dev) for w in W]
        Zg, Vd = (torch.from_numpy(x.copy()).to(dev) for x in zv)
        out = {"U": torch.from_numpy(U.copy()).to(dev), "Z": torch.zeros(n, device=dev),
               "mask": torch.zeros(plan.groups_total, dtype=torch.uint8, device=dev),
               "packed": torch.zeros(plan.packed_capacity_elems, device=dev),
               "off": torch.zeros(plan.n_layers + 1, dtype=torch.int64, device=dev),
               "kept": torch.zeros(plan.groups_total, dtype=torch.int32, device=dev)}
        ws = torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device=dev)
        rest = (out["Z"], None, out["mask"], None, out["packed"], out["off"], out["kept"], ws)
        if weighted:
            pkg.hsadmm_plan_set_node_weights(plan, [0.6] * 4, [0.3] * 4)
            got = _launches(plan, lambda: pkg.hsadmm_project_weighted_compact(plan, dW, out["U"], Zg, Vd, *rest))
        else:
            got = _launches(plan, lambda: pkg.hsadmm_project_compact(plan, dW, out["U"], *rest))
        assert (sum(got.values()) == 1) == held, got
        plan.close()
        return {k: v.cpu().numpy() for k, v in out.items()}

    one, several = outputs(True), outputs(False)
    for name, got in one.items():
        want = several[name]
        if got.dtype == np.float32:
            assert np.array_equal(np.isnan(got), np.isnan(want)), name
            got, want = (np.where(np.isnan(x), np.float32(0), x).view(np.uint32) for x in (got, want))
        assert np.array_equal(got, want), name


@pytest.mark.parametrize("weighted", [False, True], ids=["step", "weighted"])
@pytest.mark.parametrize("shape", [(1024, 64, 1, F, 400), (64, 1024, 1, F, 30), (512, 64, 9, C, 30)], ids=["short", "long", "tiles"])
@pytest.mark.parametrize("whole", [0, 1, 3, 12, 60])
def test_tags_and_states_stay_in_their_part_of_the_scratch(shape, weighted, whole, monkeypatch):
    """Few and many unconstrained layers beside a held one: the words of this call lie within four words a row item."""
    from tests.gpu_harness import GpuRun
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE", "HSADMM_HELD_PATIENCE"):
        monkeypatch.delenv(name, raising=False)
    wl = wk.custom_workload([shape] + [(70, 64, 1, N, 70)] * whole, R=2, seed=9, sigma_replica=0.03)
    W, U = wk.generate(wl)
    r = GpuRun(wl, W, U)
    if weighted:
        pkg.hsadmm_plan_set_node_weights(r.plan, [1.0] * len(wl.layers), [0.0] * len(wl.layers))
        zeros = torch.zeros_like(r.dU)
        got = _launches(r.plan, lambda: pkg.hsadmm_project_weighted_compact(r.plan, r.dW, r.dU, zeros, zeros, r.dZ, None, r.dmask,
                                                                            None, r.dpacked, r.doff, r.dkept, r.ws))
    else:
        got = _launches(r.plan, r.project_compact)
    words = r.ws.cpu().numpy()[:r.ws.numel() // 8 * 8].view(np.uint64)
    at = np.flatnonzero((words >> np.uint64(50)) == 0x3FFD)
    if sum(got.values()) == 1:                                   # (else there was no room, and none was taken)
        held = pkg.hsadmm_kernel_grids(r.plan)["weighted_pass1" if weighted else "project_pass1"]
        assert _launches(r.plan, lambda: r.compact(cached=True)) == {"compact_gather": 1}     # a workgroup a row item
        assert at.size > 0 and at[-1] - at[0] < 4 * pkg.hsadmm_kernel_grids(r.plan)["compact_gather"], held
    else:
        assert at.size == 0
    assert np.array_equal(r.dmask.cpu().numpy(), oracle.project(wl.table(), W, U)["mask"])
    r.close()


@pytest.mark.parametrize("R,width,one", [(1, 45, True), (4, 61, False), (8, 61, True), (3, 139, False), (8, 139, False), (8, 187, True),
                                         (4, 64, True)])
def test_few_ragged_layers_keep_the_weighted_step_in_launches_of_its_own(R, width, one, monkeypatch):
    """On either side of the sizes between which they do."""
    from tests.test_gpu_weighted import _phase4_chain
    for name in ("HSADMM_NO_ESTIMATE", "HSADMM_FORCE_ESTIMATE", "HSADMM_HELD_PATIENCE"):
        monkeypatch.delenv(name, raising=False)
    w = width
    wl = wk.custom_workload([(w, 3, 9, F, w // 2), (2 * w, w, 9, F, w), (2 * w, 2 * w, 9, F, w), (4 * w, 2 * w, 9, F, 2 * w),
                             (10, 4 * w, 1, F, 5)], R=R, seed=21, sigma_replica=0.03)
    W, U = wk.generate(wl, threads=8)
    rng = np.random.default_rng(R)
    a, b = rng.uniform(0.3, 1.0, 5).astype(np.float32), rng.uniform(0.0, 0.7, 5).astype(np.float32)
    assert (_weighted_launches(wl, W, U, a, b) == {"weighted_pass1": 1}) == one
    _phase4_chain(wl, W, U, a, b, rng, fused_dual=True, one_call=True)
