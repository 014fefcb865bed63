"""Post-processing on pressure levels through the C ABI against the oracle:
zonal and time means, eddy fluxes, valid fractions, the mass
streamfunction and the first-layer grid-imprinting map [w*] over two
snapshots of a small gas giant, with pressure
levels reaching outside the columns' pressure range."""
import numpy as np
import pytest

import workloads
from oracle import dynamics as odyn
from oracle import postproc as opp
from tests.conftest import oracle_grid
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_zonal_means_match_the_oracle():
    from paper_1607_05535_amd import thor
    w = workloads.small_gas_giant(glevel=3, n_lev=12)
    w.noise_amp = 2.0
    nb = 9
    G = oracle_grid(w.glevel)
    _, lat = odyn.lon_lat(G.P)
    edges = -np.pi / 2 + np.arange(nb + 1) * np.pi / nb
    assert np.min(np.abs(lat[:, None] - edges[None, 1:-1])) > 1e-9   # no column on a band edge
    model, ost = odyn.model_from_workload(w, G)
    p0 = odyn.fields(model, ost)["p"]
    plev = np.linspace(0.5 * p0[:, -1].min(), 1.05 * p0[:, 0].max(), 14)
    say(f"[zonal] {w.name}: {nb} bands, {len(plev)} levels, 2 snapshots")
    grid = thor.Grid(w.glevel)
    st = thor.State(grid, *thor.structs_from_workload(w))
    z = thor.Zonal(st, grid, w.radius, w.gravity, nb, plev)
    snaps, wsnaps = [], []
    for _ in range(2):
        st.step(1, w.n_acoustic)
        z.accumulate()
        ost = odyn.run(model, ost, 1, w.n_acoustic)
        snaps.append(opp.snapshot(model, ost, plev, nb))
        wsnaps.append(opp.imprint_snapshot(model, ost, nb))
    got, n = z.result()
    imp, n_imp = z.imprint()
    imp_ref = opp.imprint_map(wsnaps)
    assert n_imp == 2
    wscale = np.abs(opp.first_layer_w(model, ost)).max()
    assert np.abs(imp_ref).max() > 1e-3 * wscale          # the map is not trivially zero
    imp_err = np.abs(imp - imp_ref).max() / wscale
    say(f"        [w*] error {imp_err:.2e} (scale {wscale:.3e} m/s)")
    assert imp_err < 1e-9
    ref, cnt = opp.time_mean(snaps)
    ref["psi"] = opp.streamfunction(ref["v"], plev, w.radius, w.gravity)
    assert n == 2
    assert np.array_equal(got["snapshots"], cnt)
    assert (cnt == 0).any() and (cnt == 2).any()          # levels outside every column exist
    assert np.abs(got["weight"] - ref["weight"]).max() < 1e-12
    speed = max(np.abs(ref["u"]).max(), np.abs(ref["v"]).max())
    errs = {}
    for k in ("u", "v"):
        errs[k] = np.abs(got[k] - ref[k]).max() / speed
    for k in ("T", "theta"):
        errs[k] = np.abs(got[k] / np.where(ref[k] == 0, 1, ref[k]) - np.where(ref[k] == 0, 0, 1)).max()
    for k in ("upvp", "vpTp", "psi"):
        errs[k] = np.abs(got[k] - ref[k]).max() / max(np.abs(ref[k]).max(), 1e-300)
    say(f"        errors {errs}")
    for k, e in errs.items():
        assert e < 1e-9, (k, e)
    z.reset()
    got, n = z.result()
    assert n == 0 and np.all(got["snapshots"] == 0) and np.all(got["u"] == 0)
    imp, n_imp = z.imprint()
    assert n_imp == 0 and np.all(imp == 0)


@pytest.mark.parametrize("n_lev,n_plev,n_bands", [(1, 2, 3), (2, 1, 1), (13, 33, 41), (33, 5, 7), (64, 17, 201)])
def test_zonal_means_at_the_edges_of_the_work_split(n_lev, n_plev, n_bands):
    """Level counts from one to 64, more bands than latitudes (empty bands; an
    odd number of bands, so that no column sits on a band edge)
    and a column count that is no multiple of a workgroup's columns."""
    from paper_1607_05535_amd import thor
    w = workloads.small_gas_giant(glevel=2, n_lev=n_lev)
    w.z_top *= min(1.0, n_lev / 12)   # layers thin enough for a hydrostatic column
    w.noise_amp = 2.0
    G = oracle_grid(w.glevel)
    model, ost = odyn.model_from_workload(w, G)
    ost = odyn.run(model, ost, 1, w.n_acoustic)
    p0 = odyn.fields(model, ost)["p"]
    plev = np.geomspace(0.5 * p0[:, -1].min(), 1.05 * p0[:, 0].max(), n_plev + 2)[1:-1]
    grid = thor.Grid(w.glevel)
    st = thor.State(grid, *thor.structs_from_workload(w))
    st.step(1, w.n_acoustic)
    z = thor.Zonal(st, grid, w.radius, w.gravity, n_bands, plev)
    z.accumulate()
    got, n = z.result()
    ref, cnt = opp.time_mean([opp.snapshot(model, ost, plev, n_bands)])
    assert n == 1 and np.array_equal(got["snapshots"], cnt)
    speed = max(np.abs(ref["u"]).max(), np.abs(ref["v"]).max(), 1e-300)
    for k, scale in (("u", speed), ("v", speed), ("T", 1300.0), ("theta", max(np.abs(ref["theta"]).max(), 1.0)),
                     ("upvp", speed ** 2), ("vpTp", speed * 10.0), ("weight", 1.0)):
        assert np.abs(got[k] - ref[k]).max() <= 1e-9 * scale, k
    imp, _ = z.imprint()
    imp_ref = opp.imprint_map([opp.imprint_snapshot(model, ost, n_bands)])
    assert np.abs(imp - imp_ref).max() <= 1e-9 * max(np.abs(opp.first_layer_w(model, ost)).max(), 1e-300)


def test_zonal_means_in_several_passes_over_the_levels():
    """More pressure levels than the interpolation takes at a time (64), the
    last pass with one."""
    test_zonal_means_at_the_edges_of_the_work_split(9, 129, 5)


def test_many_bands_on_a_small_grid():
    """More bands than columns: a record per column at most (88 bytes per
    pressure level, beside 64 of sums per band and level), and the same means."""
    import ctypes
    from paper_1607_05535_amd import thor
    w = workloads.small_gas_giant(glevel=2, n_lev=12)
    st = thor.State(thor.Grid(2), *thor.structs_from_workload(w))
    N, nb, plev = st.n_col, 4095, np.linspace(1e3, 1e7, 1024)
    n = ctypes.c_size_t()
    assert thor.lib().thor_zonal_bytes(st.handle, nb, plev.ctypes.data, plev.size, ctypes.byref(n)) == 0
    arrays = 8 * plev.size + N * (88 * plev.size + 8) + 4 * (nb + 1) + 64 * nb * plev.size + N * 8 + 4 * (nb + 1) + \
        4 * N + 16 * N
    assert n.value <= arrays + 10 * 256
    test_zonal_means_at_the_edges_of_the_work_split(9, 3, nb)
