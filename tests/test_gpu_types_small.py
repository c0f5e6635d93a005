"""Three and four atom types on frames of few atoms (the list's one-launch
binning and sort, the fitting layers one per launch, the first layer with the
sums of three and four T sections, the embedding nets' shares over nine and
sixteen nets) and on one just large enough for the 16-bit embedding forward's
full grid: list, energies, forces and virial against the FP64 oracle, the
mixed forms' atomic energies too, and the parameter gradients.

Bars: FP64 and the relative force errors as for full frames; the 16-bit forms'
E_i as for their fused first layer (5 and 1 meV); MIX-fp32's 0.01 meV, the FP16
bar scaled down by the operands' precision (2^-24 against 2^-11) and up by the
square root of the 1,600 FP32 roundings in a sum, rounded up."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2410_22867_amd import inputs as I

pytestmark = pytest.mark.gpu

REL_F = {"bf16": 2e-2, "fp16": 4e-3, "mix_fp32": 2e-5, "mix_fp16": 4e-3}
EI_MAX = {"bf16": 5e-3, "fp16": 1e-3, "mix_fp32": 1e-5, "mix_fp16": 1e-3}
GRAD = {"fp64": 1e-9, "bf16": 0.05, "mix_fp32": 1e-4}


def _case(ntypes, mols):
    """Water with every tenth oxygen of a third type and, of four, every ninth hydrogen of a fourth."""
    desc = dataclasses.replace(I.WATER, ntypes=ntypes, sel=(46, 92, 24, 32)[:ntypes],
                               masses=(I.MASS_O, I.MASS_H, 22.99, 39.1)[:ntypes])
    sites = int(np.ceil(round(mols ** (1 / 3), 9)))
    fr = I.water_box(mols, max(I.water_density_box(mols), 12.42, 2.95 * sites), 81)
    t = fr.types.copy()
    t[np.nonzero(t == 0)[0][::10]] = 2
    if ntypes == 4:
        t[np.nonzero(t == 1)[0][::9]] = 3
    return desc, I.Frame(fr.coords, t.astype(np.int32), fr.box), I.init_params(desc, 131, I.WATER_OUTPUT_SCALE)


@pytest.mark.parametrize("ntypes,mols", [(3, 64), (3, 214), (3, 340), (3, 500), (4, 64), (4, 214), (4, 340), (4, 500),
                                         (4, 1400)])
def test_small_frames_of_many_types(ntypes, mols):
    from paper_2410_22867_amd import dpse
    desc, fr, p = _case(ntypes, mols)
    dev = torch.device("cuda:0")
    ctx = dpse.Context(dpse.Model(desc, p), fr.n)
    x, t = torch.tensor(fr.coords, device=dev), torch.tensor(fr.types, device=dev)
    gE = torch.full((1,), -0.7, dtype=torch.float64, device=dev)
    o = oracle.compute(fr.coords, fr.types, fr.box, desc, p, grad_scale=-0.7)
    print("list of", ntypes, "types", fr.n, flush=True)
    nl, ov = ctx.build_nlist(x, t, fr.box)
    assert np.array_equal(nl.cpu().numpy(), o["nlist"]) and int(ov) == oracle.nlist(fr.coords, fr.types, fr.box, desc)[1]
    assert ctx.status() & ~dpse.FLAG_SEL_OVERFLOW == 0
    for mode in ("fp64", "bf16", "fp16", "mix_fp32", "mix_fp16"):
        print(ntypes, "types", fr.n, mode, flush=True)
        r = {k: v.cpu().numpy() for k, v in ctx.compute(x, t, fr.box, nl, mode=mode, want_atom_energy=True).items()}
        e_i = np.abs(r["Ei"] - o["Ei"]).max()
        if mode == "fp64":
            assert abs(r["E"][0] - o["E"]) <= 1e-10 * abs(o["E"])
            assert e_i <= 1e-10 * np.abs(o["Ei"]).max()
            assert np.abs(r["F"] - o["F"]).max() <= 1e-9
            assert np.abs(r["W"].reshape(3, 3) - o["W"]).max() <= 1e-9 * max(1.0, np.abs(o["W"]).max())
        else:
            assert e_i <= EI_MAX[mode]
            assert abs(r["E"][0] - r["Ei"].sum()) <= 1e-12 * np.abs(r["Ei"]).sum()
            assert np.sqrt(((r["F"] - o["F"]) ** 2).mean()) <= REL_F[mode] * np.sqrt((o["F"] ** 2).mean())
        if mode in GRAD:
            print("gradient", ntypes, "types", fr.n, mode, flush=True)
            g = ctx.backward_params(gE).cpu().numpy()
            assert np.abs(g - o["grad"]).max() <= GRAD[mode] * np.abs(o["grad"]).max()
    assert ctx.status() == 0


@pytest.mark.parametrize("mols,fits", [(64, (48, 64, 176, 192, 224)), (299, (64, 224)), (300, (64, 192)), (427, (192, 176))])
def test_fitting_routes_of_other_widths(mols, fits):
    """Both sides of the widths and atom counts at which narrower fitting
    layers change their kernels, two types: as above without the gradients."""
    from paper_2410_22867_amd import dpse
    _, fr, _ = _case(3, mols)
    fr = I.Frame(fr.coords, np.where(fr.types == 2, 0, fr.types).astype(np.int32), fr.box)
    dev = torch.device("cuda:0")
    x, t = torch.tensor(fr.coords, device=dev), torch.tensor(fr.types, device=dev)
    for fit in fits:
        desc = dataclasses.replace(I.WATER, fit=(fit,) * 3)
        p = I.init_params(desc, 132, I.WATER_OUTPUT_SCALE)
        o = oracle.compute(fr.coords, fr.types, fr.box, desc, p)
        ctx = dpse.Context(dpse.Model(desc, p), fr.n)
        nl, _ = ctx.build_nlist(x, t, fr.box)
        for mode in ("fp64", "bf16", "mix_fp32"):
            print("width", fit, fr.n, mode, flush=True)
            r = {k: v.cpu().numpy() for k, v in ctx.compute(x, t, fr.box, nl, mode=mode, want_atom_energy=True).items()}
            if mode == "fp64":
                assert np.abs(r["Ei"] - o["Ei"]).max() <= 1e-10 * np.abs(o["Ei"]).max()
                assert np.abs(r["F"] - o["F"]).max() <= 1e-9
            else:
                assert np.abs(r["Ei"] - o["Ei"]).max() <= EI_MAX[mode]
                assert np.sqrt(((r["F"] - o["F"]) ** 2).mean()) <= REL_F[mode] * np.sqrt((o["F"] ** 2).mean())


def test_widest_layer_pairs_on_a_large_frame():
    """256-wide fitting layers from 32,768 atoms on: the two-tile pair kernel
    holds 66 KB of activations in LDS.  Atomic energies and forces against the
    oracle on sampled atoms."""
    from paper_2410_22867_amd import dpse
    desc = dataclasses.replace(I.WATER, fit=(256,) * 3)
    p = I.init_params(desc, 100, I.WATER_OUTPUT_SCALE)
    fr = I.water_box(11000, max(I.water_density_box(11000), 2.95 * 23), 82)
    dev = torch.device("cuda:0")
    ctx = dpse.Context(dpse.Model(desc, p), fr.n)
    x, t = torch.tensor(fr.coords, device=dev), torch.tensor(fr.types, device=dev)
    nl, _ = ctx.build_nlist(x, t, fr.box)
    print("layer pairs", desc.fit, fr.n, flush=True)
    r = {k: v.cpu().numpy() for k, v in ctx.compute(x, t, fr.box, nl, want_atom_energy=True).items()}
    rows = np.random.default_rng(7).choice(fr.n, 64, replace=False)
    o = oracle.compute(fr.coords, fr.types, fr.box, desc, p, rows=rows)
    assert np.abs(r["Ei"][rows] - o["Ei"]).max() <= 1e-10 * np.abs(o["Ei"]).max()
    for k in rows[:4]:
        assert np.abs(r["F"][k] - oracle.force_on(fr.coords, fr.types, fr.box, desc, p, int(k))).max() <= 1e-9
    assert np.abs(r["F"].sum(0)).max() < 1e-8
    assert ctx.status() == 0
