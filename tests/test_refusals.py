"""What create says where it refuses a near field: the options that it takes
there, transforms among them."""
import ctypes

import pytest

import paper_1503_08509_amd as fp


@pytest.mark.parametrize("q,opts", [(4, {}), (3, {"boundary": fp.BOUNDARY_GROUNDED, "solver": fp.SOLVER_FDM}),
                                    (3, {"boundary": fp.BOUNDARY_INSULATED, "solver": fp.SOLVER_FDM})])
def test_near_field_refusal_names_what_is_taken(q, opts):
    h, d, o = ctypes.c_void_p(), (ctypes.c_int32 * 3)(8, 8, 8), fp.default_options()
    o.near_field = fp.NEAR_FFT
    for k, v in opts.items():
        setattr(o, k, v)
    assert fp.lib().fep3m_create_ex(1.0, 100, d, q, ctypes.byref(o), ctypes.byref(h)) == fp.ERR_UNSUPPORTED
    msg = fp.lib().fep3m_last_error(None).decode()
    assert "near_field = AUTO or DIRECT" in msg and "the direct near field" not in msg
