"""Both forms of the batch draw, by half a wavefront per atom (small systems, up
to 128 draws) and by one thread per atom, against the oracle's batches rank for
rank: numbers of draws around a lane's four and the half wavefront's 128, lists a
little longer than the batch (most draws taken, chains of taken steps), lists of
every length around it, the largest system of the one form and the smallest of the
other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _compare(orc, n, box, r_core, r_shell, p_shell, steps):
    from paper_2204_13595_amd import irbe
    rng = np.random.default_rng(n + p_shell)
    pos_np = rng.uniform(0.0, box, (n, 3))
    mol = np.full(n, -1, np.int32)
    dev = torch.device("cuda", 0)
    h = irbe.Handle(n, box, r_core=r_core, r_shell=r_shell, p_shell=p_shell, p_kspace=2, n_types=1, precision="fp64",
                    device=dev)
    pos = torch.tensor(pos_np, device=dev)
    h.set_system(torch.zeros(n, dtype=torch.int32, device=dev), torch.ones(n, dtype=torch.float64, device=dev),
                 torch.tensor(mol, device=dev), np.array([0.05]), np.array([0.1]))
    h.build_lists(pos, 0)
    lists = orc.build_lists(orc.quantize(pos_np, box), mol, box, r_core, r_shell)
    for step in steps:
        h.compute_forces(pos, step)
        b_off, b_rank, _ = orc.shell_batches(h.cfg.seed, step, lists, p_shell)
        assert np.array_equal(h.debug("batch_off"), b_off)
        assert np.array_equal(h.debug("batch_rank"), b_rank)
    h.close()
    return np.diff(lists.shell_off)


@pytest.mark.parametrize("p_shell", [1, 3, 4, 5, 63, 127, 128, 129, 160])
def test_draws_bit_exact(orc, p_shell):
    ns = _compare(orc, 400, 2.6, 0.5, 1.25, p_shell, [0, 7, (1 << 33) + 5])
    if p_shell == 160:
        assert (ns <= p_shell).any() and (ns == p_shell + 1).any()  # every member, and all but one


@pytest.mark.parametrize("n", [32767, 32768])
def test_draws_at_the_change_of_form(orc, n):
    _compare(orc, n, 19.0, 0.8, 1.0, 5, [3])
