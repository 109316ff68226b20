"""Read-back of fields and populations to host arrays below, at and above the
size from which it runs in parallel blocks, and from several threads."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import ib_cases
import paper_2609_02298_amd as ib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    ib.load_library()


# 24 B per node in fields(), 72 in populations(): blocks of 2 MiB, from 4 MiB
@pytest.mark.parametrize("nx,ny", [(3, 3), (417, 418), (417, 420), (512, 512), (1023, 257), (1500, 811)])
def test_populations_come_back_as_set(nx, ny):
    print(f"read-back {nx}x{ny}", flush=True)
    pops = ib_cases.random_populations(nx, ny, nx + ny)
    sim = ib.Sim(dict(nx=nx, ny=ny, tau=0.8, bc=(ib.PERIODIC,) * 4, bodies=[]))
    sim.set_populations(pops)
    for _ in range(2):
        assert np.array_equal(sim.populations(), pops)
        rho, ux, uy = sim.fields()
        # sums of nine doubles in some order
        assert np.abs(rho - pops.sum(0)).max() < 9 * np.finfo(float).eps * 2
        ex = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1])[:, None, None]
        ey = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])[:, None, None]
        assert np.abs(ux - (pops * ex).sum(0) / rho).max() < 1e-15
        assert np.abs(uy - (pops * ey).sum(0) / rho).max() < 1e-15
    sim.close()


def test_read_back_from_several_threads():
    print("read-back from several threads", flush=True)
    pops = [ib_cases.random_populations(700, 500, k) for k in range(3)]
    sims = [ib.Sim(dict(nx=700, ny=500, tau=0.8, bc=(ib.PERIODIC,) * 4, bodies=[])) for _ in pops]
    for s, p in zip(sims, pops):
        s.set_populations(p)

    def read(k):
        return all(np.array_equal(sims[k].populations(), pops[k]) for _ in range(6))

    with ThreadPoolExecutor(3) as ex:
        assert all(ex.map(read, range(3)))
    for s in sims:
        s.close()


def test_populations_come_back_into_pinned_memory():
    import ctypes as C
    import torch
    print("read-back into pinned memory", flush=True)
    pops = ib_cases.random_populations(700, 500, 8)
    sim = ib.Sim(dict(nx=700, ny=500, tau=0.8, bc=(ib.PERIODIC,) * 4, bodies=[]))
    sim.set_populations(pops)
    for pinned in (True, False, True):
        out = torch.zeros(pops.shape, dtype=torch.float64, pin_memory=pinned)
        assert sim.L.ib_lbm_get_populations(sim.h, C.cast(out.data_ptr(), C.POINTER(C.c_double))) == 0
        assert np.array_equal(out.numpy(), pops)
    sim.close()
