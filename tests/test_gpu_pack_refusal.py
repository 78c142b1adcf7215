"""A refused pack call leaves its destinations and its descriptor as they were."""
import pytest
import torch

from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu

STORES = [(g, r) for g in range(5) for r in (18, 12, 8) if r != 8 or g in (0, 3)]
DIMS = (6, 10, 12, 14)


@pytest.mark.parametrize("fault", ["nan fat", "inf long", "sign"])
@pytest.mark.parametrize("gf,recon", STORES)
def test_refused_links_are_not_packed(gf, recon, fault):
    hisq = need_gpu()
    if fault == "sign" and recon == 18:
        pytest.skip("full storage takes long links of any form")
    fat, lng = inputs.make_links(DIMS, "near_unit", device="cuda")
    good = hisq.pack_gauge(fat, lng, DIMS, gf, long_recon=recon)
    before = good.fat.clone(), good.lng.clone()
    if fault == "nan fat":
        fat[3, -1, 2, 2] = complex(float("nan"), 0.1)
    elif fault == "inf long":
        lng[0, 5, 0, 1] = complex(0.1, float("inf"))
    else:
        lng[2, 77] *= -1.0                   # one link of the other sign
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_gauge_pack_recon(good.fat, good.lng, torch.view_as_real(fat), torch.view_as_real(lng), DIMS, gf,
                                   recon)
    assert e.value.status == (-1 if fault == "sign" else -7)
    assert torch.equal(good.fat, before[0]) and torch.equal(good.lng, before[1])
