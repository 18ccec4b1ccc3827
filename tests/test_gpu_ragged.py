"""Row lengths around the 128-bit word (four floats), the lanes of a wave and the wide-row threshold: rows that are not
whole words move as 128-bit accesses at any float's address with their last one to three floats on their own, and the
last lane of a column tile overlaps its neighbour.  Every output against the oracle, to the tolerances of the calls'
own tests (floats bit for bit, keys to 1e-12: fp64 sums of at most a few thousand squares in another order)."""
import numpy as np
import pytest

import workloads as wk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROW_LENGTHS = [1, 2, 3, 4, 5, 6, 7, 9, 13, 63, 255, 257, 258, 259, 511, 1023, 2047, 2049, 2050, 2051]


def _workload(mode, R, seed, rows=37):
    shapes = []
    for n in ROW_LENGTHS:
        ci, khw = (n // 3, 3) if n % 3 == 0 else (n, 1)
        G = ci if mode == wk.MODE_CHANNEL else rows
        shape = (rows, ci, khw, mode, max(1, (2 * G) // 5))
        shapes.append(shape + (max(1, ci // 2),) if mode == wk.MODE_BOTH else shape)
    return wk.custom_workload(shapes, R=R, seed=seed, sigma_replica=0.03)


@pytest.mark.parametrize("mode", [wk.MODE_NONE, wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_BOTH])
@pytest.mark.parametrize("R", [1, 4, 5])
def test_row_lengths_that_are_not_whole_words(mode, R):
    from tests.test_gpu_frozen import _check_frozen
    from tests.test_gpu_parity import _run
    from tests.test_gpu_weighted import _phase4_chain
    import oracle
    wl = _workload(mode, R, 10 * R + mode)
    _run(wl, want_wbar=True, want_sqnorm=True)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(77 + R)
    L = len(wl.layers)
    a, b = rng.uniform(0.3, 1.0, L).astype(np.float32), rng.uniform(0.0, 0.7, L).astype(np.float32)
    _phase4_chain(wl, W, U, a, b, rng, fused_dual=True, one_call=True)
    _check_frozen(wl, W, U, oracle.project(wl.table(), W, U)["mask"])


def test_row_lengths_that_are_not_whole_words_with_the_estimate(monkeypatch):
    from tests.test_gpu_parity import _run
    monkeypatch.setenv("HSADMM_FORCE_ESTIMATE", "1")
    _run(_workload(wk.MODE_FILTER, 4, 5), want_wbar=True, want_sqnorm=True)


@pytest.mark.parametrize("mode", [wk.MODE_NONE, wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_BOTH])
@pytest.mark.parametrize("R", [1, 2, 4, 5, 8])
def test_every_form_of_the_step_on_rows_that_are_not_whole_words(mode, R):
    """The weighted candidate with the dual out of place, un-predicted and under a right and a partly wrong prediction,
    with and without the residual norms: floats, masks and ranks are the oracle's, and neither the prediction nor the
    norms change a bit of the group keys, nor the prediction one of the norms (every form adds a row in one order)."""
    from tests.test_gpu_hinted import _Bufs, degrade, record_of
    import oracle
    import paper_2512_14628_amd as pkg
    wl = _workload(mode, R, 100 * R + mode)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(7 * R + mode)
    t, L = wl.table(), len(wl.layers)
    a, bb = oracle.node_coefficients(rng.uniform(1e-3, 2e-3, L), rng.uniform(1e-4, 3e-4, L), 1e-4, 16, R)
    Zg, Vd, Zp = (rng.standard_normal(wl.n_arena).astype(np.float32) * s for s in (0.05, 0.01, 0.05))
    ref = oracle.project_weighted(t, W, U, Zg, Vd, a, bb, want_wbar=True)
    refc = oracle.compact(t, oracle.add_arenas(t, ref["Z"], Vd), ref["mask"])
    sq = oracle.residuals(t, W, ref["Z"], Zp)
    b = _Bufs(wl, W, U, 1)
    dev = b.U.device
    dZg, dVd, dZp = (torch.from_numpy(x).to(dev) for x in (Zg, Vd, Zp))
    coef = torch.from_numpy(np.stack([a, bb], axis=1).astype(np.float32).reshape(-1).copy()).to(dev)
    right = record_of(wl, ref["mask"])
    keys = norms = None
    for name, rec in (("none", None), ("right", right), ("wrong", record_of(wl, degrade(wl, ref["mask"], 0.2, rng)))):
        for with_norms in (False, True):
            case = "%s, norms %s" % (name, with_norms)
            b.reset()
            b.out_of_place = True
            res = torch.full((4 * L,), -7.0, dtype=torch.float64, device=dev)
            pkg.hsadmm_step(b.plan, b.W, U=b.U, U_out=b.Uout, Zg=dZg, Vd=dVd, coef=coef, Z=b.Z, Wbar=b.Wbar, mask=b.mask,
                            sqnorm=b.key, sel=b.sel, sel_prev=None if rec is None else torch.from_numpy(rec).to(dev),
                            packed=b.packed, layer_off=b.off, kept_idx=b.kept, workspace=b.ws,
                            **(dict(residuals=res, Zi_prev=dZp) if with_norms else {}))
            got = b.outputs()
            assert np.array_equal(got["mask"], ref["mask"]) and np.array_equal(got["sel"], right), case
            for key in ("Z", "U", "Wbar"):
                for l in wl.layers:
                    sl = slice(l.elem_off, l.elem_off + l.n)
                    assert np.array_equal(got[key][sl].view(np.uint32), ref[key][sl].view(np.uint32)), (case, key, l.name)
            assert np.array_equal(got["layer_off"], refc["layer_off"]), case
            n = int(refc["layer_off"][-1])
            assert np.array_equal(got["packed"][:n].view(np.uint32), refc["packed"][:n].view(np.uint32)), case
            np.testing.assert_allclose(got["key"], ref["key"], rtol=1e-12, err_msg=case)
            if keys is None:
                keys = got["key"].view(np.uint64)
            assert np.array_equal(got["key"].view(np.uint64), keys), "keys differ in their last bits: " + case
            if with_norms:
                r = res.cpu().numpy().reshape(4, L)[:2]
                for li, l in enumerate(wl.layers):
                    np.testing.assert_allclose(r[:, li], sq[:2, li], rtol=max(1e-12, l.n * R * 2.0 ** -53), err_msg=case)
                if norms is None:
                    norms = r.view(np.uint64)
                assert np.array_equal(r.view(np.uint64), norms), "norms differ in their last bits: " + case
    b.plan.close()


@pytest.mark.parametrize("mode", [wk.MODE_NONE, wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_BOTH])
@pytest.mark.parametrize("R", [1, 2, 4, 5, 8])
def test_retraining_iteration_on_rows_that_are_not_whole_words(mode, R):
    """The passes of an iteration after the masks are frozen, with and without the residual norms, under a mask of half the
    groups: every output the oracle's, the norms to the bound of their own test."""
    from tests.test_gpu_weighted import _check_weighted_frozen
    wl = _workload(mode, R, 200 * R + mode)
    W, U = wk.generate(wl)
    rng = np.random.default_rng(9 * R + mode)
    L = len(wl.layers)
    a, b = rng.uniform(0.3, 1.0, L).astype(np.float32), rng.uniform(0.0, 0.7, L).astype(np.float32)
    Zg, Vd = ((rng.standard_normal(wl.n_arena) * s).astype(np.float32) for s in (0.05, 0.01))
    _check_weighted_frozen(wl, W, U, a, b, Zg, Vd, (rng.random(wl.groups_total) < 0.5).astype(np.uint8))


def test_wide_rows_that_are_not_whole_words_ask_for_no_more_scratch_than_the_static_array_holds():
    """240 000 rows of 2049 floats: 52 bytes of scratch a row and 36 an item of four rows fit the static array (16 MiB),
    which hsadmm_project_compact_static therefore takes; 36 bytes for every row would not."""
    import paper_2512_14628_amd as pkg
    rows = 240000
    plan = pkg.Plan(dict(elem_off=[0], c_out=[rows], c_in=[2049], khw=[1], mode=[wk.MODE_FILTER], k=[rows // 2], k_in=[0]))
    assert plan.workspace_bytes <= 16 << 20, plan.workspace_bytes
    plan.close()


@pytest.mark.parametrize("mode", [wk.MODE_FILTER, wk.MODE_CHANNEL, wk.MODE_BOTH])
def test_wide_rows_that_are_not_whole_words_in_a_plan_that_outgrows_the_static_array(mode):
    """350 000 groups beside them bring the plan's scratch over 16 MiB, where such rows come four to a work item."""
    from tests.test_gpu_parity import _run
    shapes = [(350000, 1, 1, wk.MODE_NONE, 350000)]
    for rows, n in ((37, 2050), (6, 3619), (1, 2049)):
        shapes.append((rows, n, 1, mode, max(1, (n if mode == wk.MODE_CHANNEL else rows) // 2)) +
                      ((n // 3,) if mode == wk.MODE_BOTH else ()))
    _run(wk.custom_workload(shapes, R=3, seed=40 + mode, sigma_replica=0.03), want_wbar=True, want_sqnorm=True)


@pytest.mark.parametrize("mode", [wk.MODE_CHANNEL, wk.MODE_BOTH])
@pytest.mark.parametrize("R", [1, 4, 5])
def test_column_tiles_of_ragged_rows_four_columns_to_a_lane(mode, R):
    """In a plan of 512 tiles and more the lanes of a tile of ragged CHANNEL rows own four columns each, the last one
    overlapping its neighbour; the plans above are smaller, and theirs own one.  A layer of 512 whole-word tiles brings this
    plan over the line.  (The column sums of BOTH layers are always taken so.)"""
    from tests.test_gpu_hinted import _Bufs, _hinted_step, record_of
    from tests.test_gpu_parity import _run
    import oracle
    shapes = [(8192, 1024, 1, wk.MODE_CHANNEL, 300)]
    for n in (4, 5, 6, 7, 63, 255, 257, 258, 259, 511, 1023, 2049, 2051):
        rows = 70 if n < 300 else 5
        shapes.append((rows, n, 1, mode, (n if mode == wk.MODE_CHANNEL else rows) // 2) +
                      ((n // 2,) if mode == wk.MODE_BOTH else ()))
    wl = wk.custom_workload(shapes, R=R, seed=60 + R + mode, sigma_replica=0.03)
    _run(wl, want_wbar=True, want_sqnorm=True)
    # ... and under a right prediction with the dual out of place, where tiles write and pack
    W, U = wk.generate(wl)
    t = wl.table()
    ref = oracle.project(t, W, U)
    refc = oracle.compact(t, ref["Z"], ref["mask"])
    b = _Bufs(wl, W, U, 1)
    b.reset()
    _hinted_step(b, torch.from_numpy(record_of(wl, ref["mask"])).to(b.U.device), out_of_place=True)
    got = b.outputs()
    assert np.array_equal(got["mask"], ref["mask"])
    n = int(refc["layer_off"][-1])
    assert np.array_equal(got["packed"][:n].view(np.uint32), refc["packed"][:n].view(np.uint32))
    for key in ("Z", "U"):
        for l in wl.layers:
            sl = slice(l.elem_off, l.elem_off + l.n)
            assert np.array_equal(got[key][sl].view(np.uint32), ref[key][sl].view(np.uint32)), (key, l.name)
    b.plan.close()
