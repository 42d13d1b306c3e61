"""The lane-per-atom form of the list build (dilute cells) at the sizes where it
can go wrong: the narrowest boxes (separations at the edge of the packed
coordinates), cell rows of more runs of 64 atoms than wavefronts launched for
them, rows so sparse that a run's cells do not fit one union, ranges of more than
one pass of candidates, with and without excluded pairs, against the oracle's
lists bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name: atoms, box, r_core, r_shell, atoms drawn into one cell row
SYSTEMS = {
    "three_cells": (100, 3.3, 1.05, 1.08, 0),       # n_c = 3, R = 1
    "seven_cells": (1190, 7.2, 1.0, 2.9, 0),        # n_c = 7 = 2 R + 1
    "sparse_rows": (3000, 70.0, 1.0, 2.5, 0),       # 0.6 atoms per row of 70 cells
    "one_full_row": (3000, 70.0, 1.0, 2.5, 700),    # 11 runs in a row, 10 atoms per cell
    "packed_row": (2000, 24.0, 1.0, 3.0, 1500),     # 60 atoms per cell: several passes and tiles
    "one_atom": (1, 9.0, 1.0, 2.0, 0),
}
MODES = {"split": dict(p_shell=4), "full": dict(p_shell=0), "core": dict(p_shell=4, shell_source="stencil"),
         "skin": dict(p_shell=4, skin=0.03)}


@pytest.mark.parametrize("per_mol", [1, 3])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("name", SYSTEMS)
def test_lane_lists_bit_exact(orc, name, mode, per_mol):
    from paper_2204_13595_amd import irbe
    n, box, r_core, r_shell, row = SYSTEMS[name]
    if name == "three_cells" and mode == "skin":
        r_core = 1.0
    rng = np.random.default_rng(n + row)
    pos_np = rng.uniform(0.0, box, (n, 3))
    if row:
        at = rng.permutation(n)[:row]
        pos_np[at, 1] = (2.0 + rng.uniform(0.05, 0.95, row)) * r_core
        pos_np[at, 2] = (3.0 + rng.uniform(0.05, 0.95, row)) * r_core
    mol = np.full(n, -1, np.int32) if per_mol == 1 else (np.arange(n) // per_mol).astype(np.int32)
    dev = torch.device("cuda", 0)
    h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_kspace=4, n_types=1, precision="fp64", device=dev,
                    **MODES[mode])
    pos = torch.tensor(pos_np, device=dev)
    h.set_system(torch.zeros(n, dtype=torch.int32, device=dev), torch.ones(n, dtype=torch.float64, device=dev),
                 torch.tensor(mol, device=dev), np.array([0.1]), np.array([0.1]))
    skin = MODES[mode].get("skin", 0.0)
    for _ in range(2):  # rows grown by the first build, then as kept
        h.build_lists(pos, 1)
    ref = orc.build_lists(orc.quantize(pos_np, box), mol, box, r_core, r_shell, full=mode == "full",
                          stencil=mode == "core", skin=skin)
    if mode != "full":
        assert np.array_equal(h.debug("core_off"), ref.core_off)
        assert np.array_equal(h.debug("core_idx"), ref.core_idx)
    if mode != "core":
        assert np.array_equal(h.debug("shell_off"), ref.shell_off)
        assert np.array_equal(h.debug("shell_idx"), ref.shell_idx)
    h.close()
