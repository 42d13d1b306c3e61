"""New LJ tables reach the kernels by either way of the upload (kernel arguments
up to four types, copies above), and a backward uses its own forward's tables and
charges after the handle has taken others, also from a stream that is not the
handle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, BOX = 600, 3.0


def _system(n_types, precision, seed):
    from paper_2204_13595_amd import irbe
    rng = np.random.default_rng(seed)
    g = (np.arange(9) + 0.5) * (BOX / 9)
    sites = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    pos = sites[rng.permutation(len(sites))[:N]] + rng.uniform(-0.05, 0.05, (N, 3))
    dev = torch.device("cuda", 0)
    dt = torch.float64 if precision == "fp64" else torch.float32
    t = torch.tensor(rng.integers(0, n_types, N).astype(np.int32), device=dev)
    mol = torch.full((N,), -1, dtype=torch.int32, device=dev)
    q = torch.tensor(rng.uniform(-0.5, 0.5, N), dtype=dt, device=dev)

    def tables(k):
        r = np.random.default_rng(100 + k)
        s, e = r.uniform(0.1, 0.3, (n_types, n_types)), r.uniform(0.2, 0.6, (n_types, n_types))
        return (s + s.T) / 2, (e + e.T) / 2

    def handle(k):
        h = irbe.Handle(N, BOX, p_shell=30, p_kspace=10, n_types=n_types, precision=precision, device=dev)
        h.set_system(t, q, mol, *tables(k))
        return h

    return torch.tensor(pos, dtype=dt, device=dev), q, tables, handle


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_types", [1, 4, 5, 16])
def test_tables_by_either_upload(n_types, precision):
    pos, q, tables, handle = _system(n_types, precision, n_types)
    a, b = handle(0), handle(1)
    a.build_lists(pos, 3)
    b.build_lists(pos, 3)
    a.compute_forces(pos, 3)
    a.update_parameters(lj_sigma=tables(1)[0], lj_eps=tables(1)[1])
    fa, ea = a.compute_forces(pos, 3, energy=True)
    fb, eb = b.compute_forces(pos, 3, energy=True)
    assert torch.equal(fa, fb) and torch.equal(ea, eb)
    a.close()
    b.close()


@pytest.mark.parametrize("other_stream", [False, True])
def test_backward_takes_its_forwards_tables(other_stream):
    from paper_2204_13595_amd.irbe import IRBEForce
    pos, q, tables, handle = _system(3, "fp64", 7)
    h = handle(0)
    h.build_lists(pos, 5)
    dev = pos.device
    grad = torch.randn(N, 3, dtype=torch.float64, device=dev, generator=torch.Generator(dev).manual_seed(1))

    def leaves(k):
        return [x.clone().requires_grad_(True) for x in
                (pos, q * (1.0 + 0.1 * k), *(torch.tensor(t, device=dev) for t in tables(k)))]

    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if other_stream else torch.cuda.current_stream()):
        alone = leaves(0)
        f = IRBEForce.apply(*alone, h, 5)
        torch.cuda.synchronize()
        want = torch.autograd.grad(f, alone, grad_outputs=grad)
        torch.cuda.synchronize()
        first, second = leaves(0), leaves(1)
        f1 = IRBEForce.apply(*first, h, 5)
        torch.cuda.synchronize()
        IRBEForce.apply(*second, h, 5)
        torch.cuda.synchronize()
        got = torch.autograd.grad(f1, first, grad_outputs=grad * 1.0)
        torch.cuda.synchronize()
    for x, y in zip(got, want):
        assert float((x - y).abs().max()) <= 1e-13 * float(y.abs().max())
    h.close()
