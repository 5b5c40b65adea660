"""The thermal assembly at the edges of its tiles (8 x 4 x 2 cells): one tile,
one cell past it in each direction, single cells along an axis."""
import pytest
import torch

from paper_1812_03952_amd import rsolve as rs
import test_gpu_thermal as tt
from test_gpu_thermal import _assemble, _device, _tp

pytestmark = pytest.mark.gpu

DIMS = [(8, 4, 2), (9, 5, 3), (17, 4, 1), (1, 9, 3), (16, 1, 4)]


@pytest.mark.parametrize("dims", DIMS)
def test_tile_edges_match_oracle(dims):
    tt.test_assembly_matches_oracle(dims)


@pytest.mark.parametrize("nw", [0, 1, 1025])
def test_well_lists(nw):
    """No wells, one, and more than the check's workgroup has threads (an entry
    out of order past them is refused, and nothing else is)."""
    tp = _tp((33, 17, 9))
    q = rs.thermal_params()
    d, u, u0 = _device(tp, q)
    d["wcell"] = torch.arange(nw, dtype=torch.int32, device="cuda") * 3
    d["wkind"] = torch.ones(nw, dtype=torch.int32, device="cuda")
    d["wval"] = torch.ones(nw, dtype=torch.float64, device="cuda")
    vals, res = _assemble(tp, q, d, u, u0)
    assert torch.isfinite(vals).all() and torch.isfinite(res).all()
    if nw > 1:
        d["wcell"][-1] = d["wcell"][-2]
        with pytest.raises(rs.RsError) as e:
            _assemble(tp, q, d, u, u0)
        assert e.value.status == -1
