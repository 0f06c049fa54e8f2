"""Streaming ends of cached plans: from 128 MiB the first pass of an
out-of-place transform streams its loads, from 32 MiB the last pass of a
transposing plan streams its stores.  Access modes change no arithmetic, so
the results are the same bits as those of the plan with every pass cached."""
import re

import pytest
import torch

import paper_1501_07350_amd as offt

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128


def _cached(plan_string):
    """The plan with every pass's accesses cached."""
    return re.sub(r"\b([abc]=[^;|]+)", r"\1/c", plan_string)


# (shape, batch, dtype, layout): the first sizes on both sides of each line,
# with remainders in the last tile
CASES = [
    ((200, 200, 216), 1, C128, "natural"),        # 131.8 MiB
    ((200, 200, 200), 1, C128, "natural"),  # 122.1 MiB
    ((45, 60, 50), 125, C64, "natural"),              # 128.7 MiB of small grids
    ((256, 256, 256), 1, C128, "natural"),            # 256 MiB, the last cached size
    ((128, 128, 128), 1, C128, "cba"),                # 32 MiB
    ((125, 128, 128), 1, C128, "cba"),                # 31.25 MiB
    ((250, 270, 300), 1, C64, "cba"),                 # 154 MiB: both ends
]


@pytest.mark.parametrize("shape,batch,dtype,layout", CASES)
def test_streaming_ends_change_no_bits(shape, batch, dtype, layout):
    lead = (batch,) if batch > 1 else ()
    gen = torch.Generator(device="cuda").manual_seed(7)
    real = torch.float64 if dtype == C128 else torch.float32
    x = torch.view_as_complex(torch.rand(lead + shape + (2,), dtype=real, device="cuda", generator=gen) - 0.5)
    plan = offt.Plan(shape, batch=batch, dtype=dtype, layout=layout, normalize_inverse=True)
    cached = offt.Plan(shape, batch=batch, dtype=dtype, layout=layout, normalize_inverse=True,
                       tune="forced", forced_plan=_cached(plan.describe()))
    spec = lead + tuple(plan.spectral_shape)
    y = plan.forward(x, torch.empty(spec, dtype=dtype, device="cuda"))
    ref = cached.forward(x, torch.empty(spec, dtype=dtype, device="cuda"))
    assert torch.equal(torch.view_as_real(y), torch.view_as_real(ref))
    z = plan.backward(y, torch.empty_like(x))
    ref = cached.backward(y, torch.empty_like(x))
    assert torch.equal(torch.view_as_real(z), torch.view_as_real(ref))
    if layout == "natural":
        # in place the loads are cached
        assert torch.equal(torch.view_as_real(plan.forward(x, x)), torch.view_as_real(y))
    plan.close()
    cached.close()
