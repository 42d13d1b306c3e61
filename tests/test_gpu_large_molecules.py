"""Lists of dense cells with molecules of so many atoms that the build excludes them by
their ids (more than 200 partners) and just below, with atoms of no molecule beside
them, against the oracle's lists bit for bit; and forces with 32-bit entries and masks
alike."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODES = {"split": dict(p_shell=40), "split32": dict(p_shell=40, shell_entries=32), "full": dict(p_shell=0),
         "core": dict(p_shell=40, shell_source="stencil"), "skin": dict(p_shell=40, skin=0.04)}
# name: atoms, box, r_core, r_shell
BOXES = {"wrapped": (1501, 2.6, 0.5, 1.2), "narrow": (2303, 5.1, 0.5, 1.2), "line": (1100, 5.1, 0.5, 0.9)}


def _system(name, per_mol):
    n, box, r_core, r_shell = BOXES[name]
    rng = np.random.default_rng(n + per_mol)
    pos = rng.uniform(0.0, box, (n, 3))
    if name == "line":
        pos[:, 1] = 2.0 + 0.2 * pos[:, 1] / box
    # molecules of neighbouring atoms, every seventh atom of none; ids in another order than the atoms
    order = np.lexsort((pos[:, 0], np.floor(pos[:, 1] / 0.9), np.floor(pos[:, 2] / 0.9)))
    mol = np.empty(n, np.int32)
    mol[order] = 1000 - np.arange(n, dtype=np.int32) // per_mol
    mol[::7] = -1
    return n, box, r_core, r_shell, pos, mol


@pytest.mark.parametrize("per_mol", [230, 238, 600, 1400])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("name", BOXES)
def test_lists_bit_exact(orc, name, mode, per_mol):
    from paper_2204_13595_amd import irbe
    n, box, r_core, r_shell, pos_np, mol = _system(name, per_mol)
    dev = torch.device("cuda", 0)
    h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_kspace=4, n_types=1, precision="fp64", device=dev,
                    **MODES[mode])
    h.set_system(torch.zeros(n, dtype=torch.int32, device=dev), torch.ones(n, dtype=torch.float64, device=dev),
                 torch.tensor(mol, device=dev), np.array([0.1]), np.array([0.1]))
    pos = torch.tensor(pos_np, device=dev)
    for _ in range(2):  # rows grown by the first build, then as kept
        h.build_lists(pos, 1)
    ref = orc.build_lists(orc.quantize(pos_np, box), mol, box, r_core, r_shell, full=mode == "full",
                          stencil=mode == "core", skin=MODES[mode].get("skin", 0.0))
    if mode != "full":
        assert np.array_equal(h.debug("core_off"), ref.core_off)
        assert np.array_equal(h.debug("core_idx"), ref.core_idx)
    if mode != "core":
        assert np.array_equal(h.debug("shell_off"), ref.shell_off)
        assert np.array_equal(h.debug("shell_idx"), ref.shell_idx)
    h.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_excluded_pairs_reach_the_forces(orc, precision):
    """The partners' sorted indices are those of this build: forces against the oracle."""
    from paper_2204_13595_amd import irbe
    n, box, r_core, r_shell, _, mol = _system("wrapped", 600)
    rng = np.random.default_rng(3)
    g = (np.arange(12) + 0.5) * (box / 12)
    pos_np = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)[:n] + rng.uniform(-0.03, 0.03, (n, 3))
    dev = torch.device("cuda", 0)
    dt = torch.float64 if precision == "fp64" else torch.float32
    q = rng.uniform(-0.5, 0.5, n)
    q -= q.mean()
    t = np.zeros(n, np.int32)
    sig, eps = np.array([[0.15]]), np.array([[0.4]])
    h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_shell=40, p_kspace=20, n_types=1, precision=precision,
                    device=dev)
    x, qd = torch.tensor(pos_np, dtype=dt, device=dev), torch.tensor(q, dtype=dt, device=dev)
    h.set_system(torch.tensor(t, device=dev), qd, torch.tensor(mol, device=dev), sig, eps)
    h.build_lists(x, 1)
    f = h.compute_forces(x, 1).double().cpu().numpy()
    ref = orc.forward(x.double().cpu().numpy(), qd.double().cpu().numpy(), t, mol, sig, eps,
                      orc.Params(box=box, p_shell=40, p_kspace=20, n_types=1), step=1, mode="rbl")
    err = np.sqrt(((f - ref.force) ** 2).sum() / (ref.force ** 2).sum())
    assert err < (1e-10 if precision == "fp64" else 1e-5)
    h.close()


@pytest.mark.parametrize("skin", [0.0, 0.04])
@pytest.mark.parametrize("per_mol", [513, 514, 900])
def test_full_list_forces(orc, per_mol, skin):
    """Full lists without energies: excluded partners in the list's passes (up to 512) and
    before them, atoms of either kind and of no molecule in one wavefront."""
    from paper_2204_13595_amd import irbe
    n, box, r_core, r_shell = 1700, 2.6, 0.5, 1.2
    rng = np.random.default_rng(per_mol)
    g = (np.arange(12) + 0.5) * (box / 12)
    sites = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    pos_np = sites[rng.permutation(len(sites))[:n]] + rng.uniform(-0.02, 0.02, (n, 3))
    order = np.lexsort((pos_np[:, 0], np.floor(pos_np[:, 1] / 0.7), np.floor(pos_np[:, 2] / 0.7)))
    mol = np.full(n, -1, np.int32)  # every eighth atom along the order of none
    member = order[np.arange(n) % 8 != 3]
    mol[member[:per_mol]] = 7
    rest = member[per_mol:]
    mol[rest] = 20 + np.arange(len(rest)) // 300
    q = rng.choice([-0.7, 0.7], n)
    t, sig, eps = np.zeros(n, np.int32), np.array([0.15]), np.array([0.4])
    dev = torch.device("cuda", 0)
    for precision, dt, tol in (("fp64", torch.float64, 1e-11), ("mixed", torch.float32, 1e-5)):
        h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_shell=0, p_kspace=8, n_types=1, skin=skin,
                        precision=precision, device=dev)
        h.set_system(torch.tensor(t, device=dev), torch.tensor(q, dtype=dt, device=dev), torch.tensor(mol, device=dev),
                     sig, eps)
        pos = torch.tensor(pos_np, dtype=dt, device=dev)
        h.build_lists(pos, 1)
        s = orc.quantize(pos.double().cpu().numpy(), box)
        lists = orc.build_lists(s, mol, box, r_core, r_shell, full=True, skin=skin)
        f = h.compute_forces(pos, 1).double().cpu().numpy()
        p = orc.Params(box=box, r_core=r_core, r_shell=r_shell, p_shell=0, p_kspace=8, n_types=1, skin=skin)
        ref = orc.forward(None, torch.tensor(q, dtype=dt).double().numpy(), t, mol, sig, eps, p, step=1, mode="full",
                          s=s, lists=lists)
        assert np.sqrt(((f - ref.force) ** 2).sum() / (ref.force ** 2).sum()) < tol
        h.close()
