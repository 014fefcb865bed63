"""The checkpoint and the scalars of an output interval against the diagnostic
fields.  The checkpoint holds the same words.  The scalars use the fields'
formulas, so each is within 8 units of FP64 rounding of the value NumPy
forms from the fields (the sum of three squares may be contracted)."""
import numpy as np
import pytest

from tests.gpu_util import lib_state, say, small_earth

pytestmark = pytest.mark.gpu
EPS = 8 * np.finfo(np.float64).eps


def check_scalars(st):
    u, v, w, T = (st.field(n)[0] for n in ("u", "v", "w", "T"))
    sc = st.scalars()[0]
    want = dict(max_speed=np.nanmax(np.sqrt(u * u + v * v + w * w)), max_w=np.nanmax(np.abs(w)), min_T=np.nanmin(T),
                max_T=np.nanmax(T))
    assert np.array_equal(sc["mass"], st.mass()[0], equal_nan=True)
    for k, x in want.items():
        assert abs(sc[k] - x) <= EPS * abs(x), (k, sc[k], x)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("glevel,n_lev", [(0, 1), (2, 7), (3, 33), (2, 64)])
def test_output_equals_the_fields(glevel, n_lev, precision):
    say(f"[output] g{glevel} L{n_lev} precision {precision}")
    st = lib_state(small_earth(glevel=glevel, n_lev=n_lev), precision)
    rng = np.random.default_rng(n_lev)
    blob = st.export()[0]
    blob[4:] *= 1.0 + 0.01 * rng.standard_normal(blob.size - 4)
    st.load(blob)
    out, rc = st.export()
    assert rc == 0
    NL = st.n_col * st.n_lev
    for i, name in enumerate(("rho", "Mx", "My", "Mz", "rhotheta", "W")):
        assert np.array_equal(out[4 + i * NL:4 + (i + 1) * NL], st.field(name)[0].ravel()), name
    check_scalars(st)


def test_scalars_pass_over_nan_and_say_so():
    from paper_1607_05535_amd import thor
    st = lib_state(small_earth(glevel=2, n_lev=8))
    blob = st.export()[0]
    blob[4:4 + 40] = np.nan          # the density of the first cells
    st.load(blob)
    check_scalars(st)
    assert st.scalars()[1] == thor.THOR_ENONFINITE
