"""Host-array calls go through a staging buffer that the solve keeps: as one
copy up to 256 KiB of fields, kept up to 16 MiB, given back above.
The same values as the device-array calls, over these sizes and in a second
pass with other fields."""
import numpy as np
import pytest
import torch

from paper_1608_06345_amd import lbm
from paper_1608_06345_amd.inputs import shear_wave_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,shape", [
    (2, (200, 4, 1)),
    (2, (2048, 4, 1)),    # 256 KiB: the last size of one copy
    (2, (2731, 3, 1)),    # one cell more
    (3, (31, 33, 7)),     # moments in three copies, temperature in one
    (2, (2048, 256, 1)),  # 16 MiB: the last size kept
    (2, (2731, 192, 1)),  # above: freed, then made again
])
def test_host_calls_equal_device_calls(dim, shape):
    n = shape[0] * shape[1] * shape[2]
    with lbm.Solver(dim, 1.4, 0.7, 0.8, *shape) as s:
        for seed in (1, 2):
            f = shear_wave_fields(dim, *shape, seed=seed)
            s.init_fields(*f)
            s.step(2)
            host = (*s.moments(), s.temperature())
            d = [torch.from_numpy(np.ascontiguousarray(a).ravel()).cuda() for a in f]
            torch.cuda.synchronize()
            lbm.lbm_init_fields_dev(s.h, *d)
            s.step(2)
            out = [torch.empty(k * n, dtype=torch.float64, device="cuda")
                   for k in (1, dim, 1, 1)]
            torch.cuda.synchronize()
            lbm.lbm_moments_dev(s.h, *out[:3])
            lbm.lbm_temperature_dev(s.h, out[3])
            s.synchronize()
            for a, b in zip(host, out):
                assert np.array_equal(np.ravel(a), b.cpu().numpy())
