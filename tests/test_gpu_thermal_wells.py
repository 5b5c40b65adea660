"""The check of a well list by one workgroup and by several: the list's length
around the switch (16384 wells), and an entry out of order or off the grid at
the ends and at the workgroups' seams (1024 wells each)."""
import pytest
import torch

from paper_1812_03952_amd import rsolve as rs
from test_gpu_thermal import _assemble, _device, _tp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [16383, 16384, 16385, 20481])
def test_long_well_lists(nw):
    tp = _tp((41, 40, 13))
    q = rs.thermal_params()
    d, u, u0 = _device(tp, q)
    good = torch.arange(nw, dtype=torch.int32, device="cuda")
    d["wkind"] = torch.ones(nw, dtype=torch.int32, device="cuda")
    d["wval"] = torch.ones(nw, dtype=torch.float64, device="cuda")
    d["wcell"] = good
    vals, res = _assemble(tp, q, d, u, u0)
    assert torch.isfinite(vals).all() and torch.isfinite(res).all()
    n = 41 * 40 * 13
    for at, cell in ((0, -1), (1023, 1022), (1024, 1023), (nw - 1, nw - 2), (nw - 1, n)):
        d["wcell"] = good.clone()
        d["wcell"][at] = cell
        with pytest.raises(rs.RsError) as e:
            _assemble(tp, q, d, u, u0)
        assert e.value.status == -1, (at, cell)
