"""The matrix handle keeps one error word for the calls that take or decouple
values: each reports its own values' error and leaves none to the next, on
whatever stream that comes."""
import pytest
import torch

import synth
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("same_stream", [True, False])
def test_an_error_is_reported_once(same_stream):
    dp = rs.DeviceProblem(synth.small(9, 7, 5, seed=61))
    A = dp.bsr()
    nan, singular = dp.vals.clone(), dp.vals.clone()
    nan[5] = float("nan")
    first = slice(0, 16)                                # cell 0's row starts with its diagonal block
    singular[first] = 0.0
    other = torch.cuda.current_stream() if same_stream else torch.cuda.Stream()
    torch.cuda.synchronize()
    calls = [(lambda v, s: rs.bsr_update(A, v, stream=s)),
             (lambda v, s: rs.bsr_update_decouple(A, v, rs.ABF, 64, stream=s)),
             (lambda v, s: rs.bsr_attach_decouple(A, v, rs.ABF, 32, stream=s))]
    for i, bad in enumerate(calls):
        for good in calls:
            with pytest.raises(rs.RsError) as e:
                bad(nan, None)
            assert e.value.status == -5
            good(dp.vals, other)
            if i:
                with pytest.raises(rs.RsError) as e:
                    bad(singular, other)
                assert e.value.status == -4
                good(dp.vals, None)
            rs.decouple(A, rs.QIMPES, 64)
