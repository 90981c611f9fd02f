"""ecpic_set_state and ecpic_get_state with the memory that their header allows, through the
C ABI: host, device, and device addresses that are no multiple of 8 (copied, as host memory is).
The state comes back as it went in, bitwise: x inside the box, v and v^{n-1} are stored as
they are; the fields to the rounding of their transforms.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2606_15035_amd import ecpic as E
from paper_2606_15035_amd import workloads as W
from tests.test_gpu_parity import gpu, gpu_cfg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [None, 0, 4])
def test_state_through(offset, gpu):  # noqa: F811
    wl = W.random_plasma((8, 8, 4), (1.0, 1.0, 0.5), 3001, r=2, dt=0.2, vth=0.1, seed=5)
    F = W.random_fields(wl.n, 9, seed=6)
    g = E.Sim(gpu_cfg(wl), wl.np)
    given = [wl.x, wl.v, 0.5 * wl.v, F]

    def there(a):
        if offset is None:
            return a, C.c_void_p(a.ctypes.data)
        t = gpu.zeros(a.nbytes + 8, dtype=gpu.uint8, device="cuda")
        t[offset:offset + a.nbytes] = gpu.from_numpy(a.reshape(-1).view(np.uint8)).cuda()
        gpu.cuda.synchronize()
        return t, C.c_void_p(t.data_ptr() + offset)

    src = [there(np.ascontiguousarray(a)) for a in given]
    E._check(E.lib().ecpic_set_state(g._h, *[p for _, p in src], wl.q, wl.m))
    dst = [there(np.zeros_like(a)) for a in given]
    E._check(E.lib().ecpic_get_state(g._h, *[p for _, p in dst]))
    for (buf, _), a, exact in zip(dst, given, (True, True, True, False)):
        if offset is not None:
            b = buf[offset:offset + a.nbytes].cpu().numpy().copy().view(np.float64)
        else:
            b = buf
        b = b.reshape(a.shape)
        if exact:
            assert np.array_equal(a, b)
        else:
            assert np.abs(a - b).max() <= 1e-14 * np.abs(a).max()
