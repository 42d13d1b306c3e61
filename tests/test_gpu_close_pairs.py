"""Forces of overlapping atoms (start positions before a minimization) in mixed precision:
finite wherever the force itself is far from the largest float, in every form of the pair
kernels, and within the rounding of r^-14 (14 steps of 2^-23, and a few more) of the FP64
evaluation of the same fixed-point positions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, BOX = 512, 4.0


@pytest.mark.parametrize("p_shell,skin", [(0, 0.0), (0, 0.05), (40, 0.0), (40, 0.05)])
@pytest.mark.parametrize("r", [0.001, 0.002, 0.004, 0.03])
def test_overlapping_pair(p_shell, skin, r):
    from paper_2204_13595_amd import irbe
    rng = np.random.default_rng(6)
    g = (np.arange(8) + 0.5) * (BOX / 8)
    pos = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) + rng.uniform(-0.1, 0.1, (N, 3))
    d = rng.standard_normal(3)
    pos[100] = pos[200] + r * d / np.sqrt((d * d).sum())
    # (positions on the grid of the fixed-point coordinates that FP32 can hold)
    pos = np.round(pos * 2.0 ** 19) * 2.0 ** -19
    dev = torch.device("cuda", 0)
    out = {}
    for precision, dt in (("mixed", torch.float32), ("fp64", torch.float64)):
        h = irbe.Handle(N, BOX, r_core=0.5, r_shell=1.2, p_shell=p_shell, p_kspace=20, n_types=1, skin=skin,
                        precision=precision, device=dev)
        q = torch.tensor(np.where(np.arange(N) % 2 == 0, 0.4, -0.4), dtype=dt, device=dev)
        h.set_system(torch.zeros(N, dtype=torch.int32, device=dev), q, torch.full((N,), -1, dtype=torch.int32, device=dev),
                     np.array([[0.3]]), np.array([[0.5]]))
        x = torch.tensor(pos, dtype=dt, device=dev)
        h.build_lists(x, 2)
        out[precision] = h.compute_forces(x, 2).double().cpu()
        h.close()
    for i in (100, 200):
        a, b = out["mixed"][i], out["fp64"][i]
        assert torch.isfinite(a).all()
        assert float((a - b).norm()) <= 32 * 2.0 ** -23 * float(b.norm())
