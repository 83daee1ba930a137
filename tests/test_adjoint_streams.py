"""On which stream the gradient's passes work (CPU: a stand-in lattice that only
records; GPU: a lattice on a stream of its own against one on torch's)."""
from contextlib import contextmanager

import pytest
import torch
from torch.overrides import TorchFunctionMode

from paper_1202_6074_amd import adjoint


class _Stream:
    def __init__(self, name, log):
        self.name, self.log = name, log

    def wait_stream(self, other):
        self.log.append((self.name, "waits for", other.name))


class _Lattice:
    """What the passes use of a Lattice; every kernel call is recorded as work on its stream."""
    device, dtype, in_place, sgs_force, nx, ny, nz = torch.device("cpu"), torch.float64, False, False, 3, 2, 2

    def __init__(self, log):
        self.log, self.stream = log, _Stream("lattice", log)
        self.buf = torch.zeros((27, 2, 2, 3), dtype=self.dtype)

    def state_buffer(self):
        return self.buf

    def lam_buffer(self):
        return torch.zeros((2, 2, 27, 3), dtype=self.dtype)

    def reduce(self):
        self.log.append(("lattice", "reduce"))
        return {"ke": 1.0}

    def adjoint_steps(self, first, rest, lam, lam_tmp, gF):
        self.log.append(("lattice", "kernels"))
        return lam, lam_tmp

    def _kernels(self, *a):
        self.log.append(("lattice", "kernels"))

    set_force = steps_between = steps_record = energy_seed = _kernels

    def _after_use(self, *tensors):
        self.log.append(("lattice", "uses", len(tensors)))


class _Record(TorchFunctionMode):
    """Records torch's own work on tensors as work on the current stream."""
    def __init__(self, log, now):
        super().__init__()
        self.log, self.now = log, now

    def __torch_function__(self, func, types, args=(), kwargs=None):
        if getattr(func, "__name__", "") in ("copy_", "clone"):
            self.log.append((self.now[0].name, func.__name__))
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("nsteps,K", [(5, 2), (4, 4), (0, 3)])
def test_passes_work_on_the_lattices_stream(monkeypatch, nsteps, K):
    log = []
    lat, now = _Lattice(log), [_Stream("caller", log)]

    @contextmanager
    def on(stream):
        before, now[0] = now[0], stream
        yield
        now[0] = before

    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: now[0])
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: log.append(("kept for", s.name)))
    F = torch.ones((3, 2, 2, 3), dtype=lat.dtype, requires_grad=True)
    with _Record(log, now):
        E = adjoint.EnergyAdjoint.apply(F, lat, torch.zeros_like(lat.buf), nsteps, K)
        half = len(log)
        E.backward()
    for part in (log[:half], log[half:]):
        work = [k for k, e in enumerate(part) if e[0] in ("lattice", "caller") and e[1] not in ("waits for", "uses")]
        assert all(part[k][0] == "lattice" for k in work), part
        assert part.index(("lattice", "waits for", "caller")) < work[0]
        assert part.index(("caller", "waits for", "lattice")) > work[-1]
    assert ("lattice", "uses", 2) in log[:half] and ("kept for", "caller") in log[half:]


@pytest.mark.gpu
@pytest.mark.parametrize("nsteps,K", [(9, 4), (6, 6)])
def test_gradient_on_a_stream_of_its_own(nsteps, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1202_6074_amd.lattice import Lattice
    shape = (64, 48, 40)   # long enough kernels for work on another stream to come too early
    g = torch.Generator().manual_seed(5)
    u = (0.05 * torch.randn((3,) + shape[::-1], generator=g)).cuda()
    F = (1e-4 * torch.randn((3,) + shape[::-1], generator=g)).cuda()
    got = []
    for stream in (None, torch.cuda.Stream()):
        lat = Lattice(shape, storage="f32", stream=stream)
        lat.set_relaxation(1.7, cs_smag=0.12)
        torch.cuda.synchronize()
        lat.init_equilibrium(u)
        torch.cuda.synchronize()
        f0 = lat.state_buffer().clone()
        for _ in range(2):
            got.append(adjoint.energy_and_grad(lat, F, f0, nsteps, K))
    for E, grad in got[1:]:
        assert E == got[0][0] and torch.equal(grad, got[0][1])
