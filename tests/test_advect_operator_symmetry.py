"""The two symmetries by which the advected operators are stored as one real
matrix per pair of modes (+-m_x, m_z), checked on the host construction: with
coefficient n scaled by 1 (even) or i (odd) the operator is real, and the one at
-k_x is the conjugate of the one at k_x with the w rows and columns negated.
The operators are refined to about one rounding, so both hold to a few units of
1e-16 of the largest entry (1e-14 asked)."""
import ctypes as C

import numpy as np
import pytest

from paper_1804_05087_amd import _lib


def _operator(N, kx, kz, re=400.0, inv_dt=0.01):
    lib = _lib.load()
    out = np.zeros(18 * (N - 1) * (N + 1))
    assert lib.sp_advected_mode_operator(N, C.c_double(kx), C.c_double(kz), C.c_double(re),
                                         C.c_double(inv_dt), C.c_void_p(out.ctypes.data)) == 0
    return out.view(np.complex128).reshape(3 * (N - 1), 3 * (N + 1)).T


@pytest.mark.parametrize("N", [8, 19, 32])
@pytest.mark.parametrize("kx,kz", [(1.3, 0.0), (1.3, 2.5), (0.0, 2.5), (4.1, 5.0)])
def test_real_after_scaling_and_paired(N, kx, kz):
    S = _operator(N, kx, kz)
    p = np.where(np.arange(N + 1) % 2 == 0, 1.0 + 0j, 1j)
    scaled = S * np.tile(p[:N - 1], 3)[None, :] / np.tile(p, 3)[:, None]
    top = np.abs(S).max()
    assert np.abs(scaled.imag).max() < 1e-14 * top
    w_row = np.repeat([1.0, 1.0, -1.0], N + 1)[:, None]
    w_col = np.repeat([1.0, 1.0, -1.0], N - 1)[None, :]
    assert np.abs(_operator(N, -kx, kz) - w_row * S.conj() * w_col).max() < 1e-14 * top
