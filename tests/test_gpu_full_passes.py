"""Full-list forces where the passes over a list end: clusters whose every atom
lists all the others, of sizes around one, two and three passes of 64 entries
(the excluded partners follow the list in the same sequence), and a single pair,
against the FP64 oracle; with a skin, at moved positions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOX, R_CORE, R_SHELL = 3.0, 0.9, 1.4


@pytest.mark.parametrize("skin", [0.0, 0.05])
@pytest.mark.parametrize("per_mol", [1, 3])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 66, 67, 128, 129, 130, 193])
def test_full_list_pass_edges(orc, n, per_mol, skin):
    from paper_2204_13595_amd import irbe
    rng = np.random.default_rng(n)
    # sites of a lattice of spacing 0.12 nm (no close pairs) within a ball of 0.48 nm, jittered
    g = np.arange(-4, 5) * 0.12
    sites = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    sites = sites[(sites ** 2).sum(1) < 0.48 ** 2]
    pos_np = sites[rng.permutation(len(sites))[:n]] + rng.uniform(-0.02, 0.02, (n, 3)) + 1.1
    q = rng.choice([-0.7, 0.7], n)
    mol = np.full(n, -1, np.int32) if per_mol == 1 else (np.arange(n) // per_mol).astype(np.int32)
    t = np.zeros(n, np.int32)
    sig, eps = np.array([0.15]), np.array([0.4])
    dev = torch.device("cuda", 0)
    for precision, dt, tol in (("fp64", torch.float64, 1e-11), ("mixed", torch.float32, 1e-5)):
        h = irbe.Handle(n, BOX, r_core=R_CORE, r_shell=R_SHELL, p_shell=0, p_kspace=8, n_types=1, skin=skin,
                        precision=precision, device=dev)
        h.set_system(torch.tensor(t, device=dev), torch.tensor(q, dtype=dt, device=dev), torch.tensor(mol, device=dev),
                     sig, eps)
        pos = torch.tensor(pos_np, dtype=dt, device=dev)
        h.build_lists(pos, 1)
        lists = orc.build_lists(orc.quantize(pos.double().cpu().numpy(), BOX), mol, BOX, R_CORE, R_SHELL, full=True,
                                skin=skin)
        d = np.random.default_rng(3).uniform(-1.0, 1.0, (n, 3)) * skin / (2.0 * np.sqrt(3.0)) * 0.99
        pos = pos + torch.tensor(d, dtype=dt, device=dev)
        f = h.compute_forces(pos, 1).double().cpu().numpy()
        qd = torch.tensor(q, dtype=dt).double().numpy()
        p = orc.Params(box=BOX, r_core=R_CORE, r_shell=R_SHELL, p_shell=0, p_kspace=8, n_types=1, skin=skin)
        ref = orc.forward(None, qd, t, mol, sig, eps, p, step=1, mode="full",
                          s=orc.quantize(pos.double().cpu().numpy(), BOX), lists=lists)
        assert np.sqrt(((f - ref.force) ** 2).sum() / (ref.force ** 2).sum()) < tol
        h.close()
