"""Tabulated embedding on frames of enough columns for the LDS window of the
first intervals (ten per CU), against the oracle's tabulated evaluation: rows
inside and past the window, a table shorter than the window whose end is
passed inside it, and the wider copper layout."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_22867_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("system,grid", [("water", I.COMPRESS_GRID_WATER), ("water", (4.0, 8.0, 0.1)),
                                         ("water", (1.0, 2.0, 0.1)), ("copper", I.COMPRESS_GRID_COPPER),
                                         ("copper", (0.9, 1.9, 0.1))])
def test_windowed_table_matches_oracle(system, grid):
    from paper_2410_22867_amd import dpse
    if system == "water":
        fr, desc, p = I.water_box(1000, 31.1, 21), I.WATER, I.init_params(I.WATER, 100, I.WATER_OUTPUT_SCALE)
    else:
        fr, desc, p = I.copper_fcc((9, 9, 10), 3.634, 0.1, 22), I.COPPER, I.init_params(I.COPPER, 101)
    print("windowed table", system, grid, fr.n, flush=True)
    dev = torch.device("cuda:0")
    model = dpse.Model(desc, p)
    model.compress(*grid)
    ctx = dpse.Context(model, fr.n)
    x, t = torch.tensor(fr.coords, device=dev), torch.tensor(fr.types, device=dev)
    nl, _ = ctx.build_nlist(x, t, fr.box)
    r = ctx.compute(x, t, fr.box, nl, mode="fp64_tab")
    torch.cuda.synchronize()
    o = oracle.compute(fr.coords, fr.types, fr.box, desc, p, table=(oracle.tabulate(desc, p, *grid), *grid))
    assert ctx.status() == (dpse.FLAG_TABLE_RANGE if o["clipped"] else 0)
    assert abs(r["E"].item() - o["E"]) <= 1e-10 * abs(o["E"])
    assert np.abs(r["F"].cpu().numpy() - o["F"]).max() <= 1e-9
    W = r["W"].cpu().numpy().reshape(3, 3)
    assert np.abs(W - o["W"]).max() <= 1e-9 * max(1.0, np.abs(o["W"]).max())
