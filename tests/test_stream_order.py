"""IRBEForce called from another stream than its handle's (no GPU: streams that run
their queued work only when another one waits for them). The handle's stream waits for
the inputs, copies of non-contiguous ones included, and the calling stream waits for the
handle's before it reads the outputs."""
import pytest

torch = pytest.importorskip("torch")

N, NT2 = 5, 4


class Stream:
    """Work of the handle is queued and done when another stream waits for it."""

    device_index = 0

    def __init__(self, log):
        self.queue, self.log = [], log

    def wait_stream(self, other):
        self.log.append(("wait", self, other))
        for f in other.queue:
            f()
        other.queue.clear()


class FakeHandle:
    n_types = 2

    def __init__(self, stream, log):
        self.stream, self.device, self.log = stream, torch.device("cpu"), log
        self.raw_stream = id(stream)

    def update_parameters(self, charge=None, lj_sigma=None, lj_eps=None):
        self.log.append(("params", charge))

    def _later(self, out, value):
        self.stream.queue.append(lambda: out.fill_(value))
        return out

    def compute_forces(self, pos, step):
        self.log.append(("forces", pos))
        return self._later(torch.full((N, 3), -1.0), 1.0)

    def compute_forces_backward(self, pos, step, grad, want_charge, want_lj):
        self.log.append(("backward", grad))
        assert pos.is_contiguous() and grad.is_contiguous()
        return (self._later(torch.full((N, 3), -1.0), 2.0), self._later(torch.full((N,), -1.0), 3.0),
                self._later(torch.full((2 * NT2,), -1.0, dtype=torch.float64), 4.0))


@pytest.mark.parametrize("table_dtype", [torch.float32, torch.float64])
def test_order_across_streams(monkeypatch, table_dtype):
    from paper_2204_13595_amd.irbe import IRBEForce
    log, kept = [], []
    mine, current = Stream(log), Stream(log)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a, **k: current)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda i: id(current), raising=False)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: kept.append((t.data_ptr(), s)), raising=False)
    real = torch.Tensor.contiguous

    def contiguous(t, *a, **k):
        if not t.is_contiguous():
            log.append(("copy",))
        return real(t, *a, **k)

    monkeypatch.setattr(torch.Tensor, "contiguous", contiguous)
    h = FakeHandle(mine, log)
    pos = torch.zeros(3, N).t().requires_grad_(True)
    q = torch.zeros(2 * N)[::2].requires_grad_(True)
    tables = [torch.ones(2, 2, dtype=table_dtype, requires_grad=True) for _ in range(2)]

    def check(call, first):
        kinds = [e[0] for e in log]
        at = kinds.index(call)
        before = [i for i, e in enumerate(log) if e == ("wait", mine, current)]
        after = [i for i, e in enumerate(log) if e == ("wait", current, mine)]
        assert before and max(i for i, k in enumerate(kinds) if k == "copy") < max(before) < kinds.index("params")
        assert after and at < min(after)
        # what the handle's stream reads stays allocated until it has
        read = [e[1] for e in log if e[0] in ("params", call)]
        assert all((t.data_ptr(), mine) in kept for t in read)
        log.clear()

    f = IRBEForce.apply(pos, q, *tables, h, 1)
    check("forces", f)
    assert float(f.detach().min()) == 1.0
    grads = torch.autograd.grad(f, [pos, q, *tables], grad_outputs=torch.ones(3, N).t())
    check("backward", grads)
    for g, want, x in zip(grads, (2.0, 3.0, 4.0, 4.0), (pos, q, *tables)):
        assert g.dtype == x.dtype and g.shape == x.shape
        assert float(g.min()) == float(g.max()) == want


def test_no_waits_on_the_handles_stream(monkeypatch):
    from paper_2204_13595_amd.irbe import IRBEForce
    log = []
    mine = Stream(log)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda i: id(mine), raising=False)
    x = [torch.zeros(N, 3, requires_grad=True), torch.zeros(N, requires_grad=True),
         torch.ones(2, 2, requires_grad=True), torch.ones(2, 2, requires_grad=True)]
    f = IRBEForce.apply(*x, FakeHandle(mine, log), 1)
    torch.autograd.grad(f, x, grad_outputs=torch.ones(N, 3))
    assert not [e for e in log if e[0] == "wait"]


def test_host_values_are_the_forwards_own():
    """Tables of two types on the host: the values kept for the backward are no view of them."""
    from paper_2204_13595_amd.irbe import _tables_on_host
    s, e = torch.ones(2, 2, dtype=torch.float64), torch.ones(2, 2, dtype=torch.float32)
    a, b = _tables_on_host(s, e)
    s.fill_(7.0)
    e.fill_(7.0)
    assert a.max() == 1.0 and b.max() == 1.0
