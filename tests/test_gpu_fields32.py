"""The FP32 field extraction against the FP64 diagnostics of the same state,
at level counts that fill, leave over and undercut its groups of four
levels, into aligned and unaligned outputs."""
import numpy as np
import pytest

from tests.gpu_util import lib_state, small_earth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_lev,offset", [(1, 0), (3, 0), (4, 0), (4, 1), (13, 0), (32, 0), (32, 3), (37, 0), (64, 0)])
def test_fields32_equal_the_fp64_fields(n_lev, offset, precision):
    import torch
    from paper_1607_05535_amd import thor
    w = small_earth(glevel=2, n_lev=n_lev, n_large=1)
    st = lib_state(w, precision)
    st.step(1, w.n_acoustic)
    n = 5 * st.n_col * n_lev
    buf = torch.full((n + offset + 4,), -7.0, device="cuda:0")
    thor.thor_state_fields32(st, buf[offset:])
    got = buf.cpu().numpy()
    assert np.all(got[:offset] == -7.0) and np.all(got[offset + n:] == -7.0)   # nothing outside
    got = got[offset:offset + n].reshape(5, st.n_col, n_lev).astype(np.float64)
    ref = {k: st.field(k)[0] for k in ("T", "u", "v", "w", "p")}
    speed = max(np.abs(ref[k]).max() for k in ("u", "v", "w"))
    for i, k in enumerate(("T", "u", "v", "w", "p")):
        # one FP32 rounding, plus FP64 rounding of sums of components for the winds
        bar = 2.0 ** -24 * np.abs(ref[k]) + (1e-14 * speed if k in "uvw" else 2e-15 * np.abs(ref[k])) + 1e-44
        assert np.all(np.abs(got[i] - ref[k]) <= bar), (k, np.abs(got[i] - ref[k]).max())
