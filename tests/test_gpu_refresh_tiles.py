"""The refresh with the stress invariant and the history divergence on every
tile they run on, with ragged last tiles and chunks, against the FP64 oracle:
power law, yield cap, stress history, with and without the background shear."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08716_amd import inputs

from test_gpu_parity import COEF, STATE, _compare, _pair
from test_gpu_tilings import GRIDS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", GRIDS)
@pytest.mark.parametrize("shear", [0.0, 0.3])
def test_refresh_matches_the_oracle_on_every_tile(shape, shear):
    nx, ny, nz = shape
    cfg = inputs.config_production(nx, ny, nz)
    cfg.phys = cfg.phys.replace(dpcap=True, coh=1.0, fric_deg=30.0, tau_y_min=1e-3, shear_bg=shear, dts_rule=False)
    g, o = _pair(cfg)
    # a history and a stress state: iterations of a first step
    g.begin_step(False)
    o.begin_step()
    g.iterate(16)
    o.iterate(16)
    o.end_step()
    g.begin_step(True)
    o.begin_step()
    for r_eta, r_mu in ((1.0, 1.0), (0.4, 0.7)):
        g.refresh(r_eta, r_mu)
        o.refresh(r_eta, r_mu)
        # the history divergence shows in the next sweeps
        g.iteration(True, False)
        o.iteration(True, False)
    _compare(g, o, STATE + COEF)
    assert np.abs(g.get("sxx")).max() > 0
