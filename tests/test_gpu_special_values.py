"""Accepted values that make an operand of a quotient or root zero, infinite or too large to square:
silicon near absolute zero and far above any temperature, wavelengths at which the index of silicon
or the photon energy's square overflow.  Every photon has the oracle's fate."""
import numpy as np
import pytest

import oracle as O
from paper_1504_06570_amd.scene import configs as C
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def phx():
    from paper_1504_06570_amd import phx
    return phx


@pytest.mark.parametrize("temperature,wavelength", [
    (0.5, 600e-9), (0.5, 1000e-9),        # exp(E_p / kT) infinite
    (0.9449, 600e-9), (0.9449, 1050e-9),  # just finite, its reciprocal subnormal
    (1e19, 600e-9),                       # exp(E_p / kT) - 1 zero
    (1e200, 600e-9),                      # the gap's shift squared infinite
    (173.0, 4e-9),                        # the index of silicon infinite
    (173.0, 1e-160),                      # the square of the photon energy infinite
    (173.0, 1e-310),                      # the photon energy infinite
])
def test_fates_at_the_limits_of_the_silicon_formulas(phx, temperature, wavelength):
    s = C.telescope(scale=1e-3)
    s.prescription.silicon.temperature = temperature
    s.sources.lam_lo[:] = wavelength
    s.sources.lam_hi[:] = wavelength
    s.physics = C.PHYS_SILICON | C.PHYS_DIFFUSION
    tr = phx.Tracer(s)
    _, _, _, ev = tr.trace(event_stride=1)
    gev = phx.events_to_numpy(ev)
    tr.close()
    oev = O.Oracle(s).trace_sources()
    assert np.isin(oev["status"], (phx.DETECTED, phx.OFF_CHIP, phx.ESCAPED)).sum() > 9000
    rep = parity.compare(gev, oev)
    assert rep["worst_converted"] < 1e-12 and rep["worst_pos"] < 1e-11, rep
