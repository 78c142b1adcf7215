"""BiCGStab(l) where it cannot go on: the status, what it counts, and the iterate it hands back."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu

DIMS, MASS = (6, 10, 4, 12), 0.1


def packed(hisq, sloppy):
    fat, lng = inputs.make_links(DIMS, "near_unit", device="cuda")
    return (hisq.pack_gauge(fat, lng, DIMS, hisq.GAUGE_F64),
            hisq.pack_gauge(fat, lng, DIMS, hisq.fmt(sloppy).gauge))


@pytest.mark.parametrize("where", ["b", "x0"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_input_is_a_breakdown(where, bad):
    hisq = need_gpu()
    g64, gs = packed(hisq, "single")
    b = inputs.gaussian_spinor(oracle.volume(DIMS), inputs.SOURCE_SEED, device="cuda")
    x0 = torch.zeros_like(b)
    (b if where == "b" else x0)[17, 1] = complex(0.25, bad)
    with pytest.raises(hisq.HisqError) as e:
        hisq.bicgstab_solve(b, g64, gs, MASS, sloppy="single", x0=x0)
    assert e.value.status == -5
