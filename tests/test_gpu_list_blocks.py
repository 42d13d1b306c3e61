"""The block form of the list build (dense cells) and its shell lists as masks,
at the sizes where they can go wrong: blocks of one atom and of partly filled
cells, stencils that wrap the box and the narrowest that do not, blocks of more
than one tile of mask words and of more than a mask row holds, stencils of more
than 128 rows, molecules of more than eight atoms. Lists against the oracle's
bit for bit; forces and gradients with masks against those with 32-bit indices
bit for bit (both kernels read the same members in the same order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name: atoms, box, r_core, r_shell, atoms per molecule (1: none excluded)
SYSTEMS = {
    "wrap_few": (257, 2.5, 0.6, 1.2, 1),         # n_c = 4 < 2 R + 1: about 4 atoms per cell
    "wrap_dense": (4000, 2.5, 0.6, 1.2, 3),      # 62 atoms per cell: two blocks per cell, more than 128 words
    "narrowest": (1721, 3.5, 0.5, 1.2, 3),       # n_c = 2 R + 1: one cell per segment
    "molecules": (4099, 5.0, 0.5, 1.2, 12),      # 11 excluded partners per atom, a last molecule of 7
    "two_tiles": (8000, 4.0, 0.5, 1.2, 3),       # blocks of 128 to 256 mask words
    "beyond_masks": (16000, 4.0, 0.5, 1.2, 1),   # more than 256 words: 32-bit entries
    "many_rows": (23500, 4.0, 0.22, 1.2, 1),     # 169 stencil rows
}
MODES = {"split": dict(p_shell=20), "split32": dict(p_shell=20, shell_entries=32), "full": dict(p_shell=0),
         "core": dict(p_shell=20, shell_source="stencil"), "skin": dict(p_shell=20, skin=0.02)}


def _positions(n, box, seed=31):
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, box, size=(n, 3))
    pos[::5] += box  # images
    return pos


def _handle(name, precision="fp64", **kw):
    from paper_2204_13595_amd import irbe
    n, box, r_core, r_shell, per_mol = SYSTEMS[name]
    dev = torch.device("cuda", 0)
    dt = torch.float64 if precision == "fp64" else torch.float32
    h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_kspace=8, n_types=2, precision=precision, device=dev, **kw)
    mol = np.full(n, -1, np.int32) if per_mol == 1 else (np.arange(n) // per_mol).astype(np.int32)
    rng = np.random.default_rng(5)
    q = rng.choice([-0.5, 0.5], n)
    t = rng.integers(0, 2, n).astype(np.int32)
    h.set_system(torch.tensor(t, device=dev), torch.tensor(q, dtype=dt, device=dev), torch.tensor(mol, device=dev),
                 np.array([0.05, 0.04, 0.04, 0.0]), np.array([0.5, 0.4, 0.4, 0.0]))
    return h, torch.tensor(_positions(n, box), dtype=dt, device=dev), mol


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("name", SYSTEMS)
def test_block_lists_bit_exact(orc, name, mode):
    n, box, r_core, r_shell, _ = SYSTEMS[name]
    if mode == "core" and name == "many_rows":
        pytest.skip("stencil sampling supports at most 128 stencil rows")
    h, pos, mol = _handle(name, **MODES[mode])
    skin = MODES[mode].get("skin", 0.0)
    ref = orc.build_lists(orc.quantize(pos.cpu().numpy(), box), mol, box, r_core, r_shell, full=mode == "full",
                          stencil=mode == "core", skin=skin)
    for step in range(2):  # a waiting build, then a queued one
        h.build_lists(pos, step)
        h.sync()
        if mode != "full":
            assert np.array_equal(h.debug("core_off"), ref.core_off)
            assert np.array_equal(h.debug("core_idx"), ref.core_idx)
        if mode != "core":
            assert np.array_equal(h.debug("shell_off"), ref.shell_off)
            assert np.array_equal(h.debug("shell_idx"), ref.shell_idx)
    if mode == "split":
        bits = int(h.debug("shell_bits")[0])
        assert bits == (32 if name in ("beyond_masks", "many_rows") else 16)
        rows = np.array([0, n // 2, n - 1], dtype=np.int64)
        want = np.concatenate([ref.shell_idx[ref.shell_off[i]:ref.shell_off[i + 1]] for i in rows])
        assert np.array_equal(h.debug_rows("shell_idx", rows), want)
    h.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("p_shell", [5, 64, 131, 260])
@pytest.mark.parametrize("name", ["wrap_dense", "narrowest", "two_tiles"])
def test_masks_and_indices_agree(name, p_shell, precision):
    """Batches of part of one pass, one pass, the passes after the first two and
    more than some lists hold."""
    out = {}
    for entries in (0, 32):
        h, pos, _ = _handle(name, precision, p_shell=p_shell, shell_entries=entries)
        h.build_lists(pos, 2)
        assert int(h.debug("shell_bits")[0]) == (16 if entries == 0 else 32)
        G = torch.tensor(np.random.default_rng(6).standard_normal(tuple(pos.shape)), dtype=pos.dtype, device=pos.device)
        res = []
        for step in (2, 3):  # the first backward decodes the ranks, the second reads the forward's batch
            res.append(h.compute_forces(pos, step).clone())
            gp, gq, _ = h.compute_forces_backward(pos, step, G)
            atomics = int(h.debug("adj_atomics")[0])
            res += [gp, gq] if atomics == 0 else []
        res += list(h.compute_forces(pos, 4, energy=True))
        out[entries] = res
        h.close()
    assert len(out[0]) == len(out[32])
    for a, b in zip(out[0], out[32]):
        assert torch.equal(a, b)
