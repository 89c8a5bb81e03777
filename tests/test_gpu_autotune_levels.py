"""stitch_autotune measures the passes that stitch_frame launches: the settings of small levels, whose
passes share a launch, stay as they were, and a saved choice gives them back."""
import numpy as np
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def test_settings_of_shared_levels_stay(tmp_path):
    W, H, L = 1600, 1200, 5                      # levels 2 and 3 of a camera over all of it: 120 and 30 thousand samples
    frame = torch.randint(0, 256, (H, W, 3), dtype=torch.uint8, device=DEV)
    new = lambda: P.Plan([(W, H)], [np.eye(3)], [np.full((H, W), 255, np.uint8)], W, H, L)
    plan = new()
    ref = plan.frame([frame]).clone()
    plan.set_config([2] * (L - 1), [128] * (L - 1))
    cfg = plan.autotune([frame], cache_path=tmp_path / "tune.txt")
    assert cfg["tile_rows"][2:L - 1] == [128, 128] and cfg["wg_per_cu"][2:L - 1] == [2, 2], cfg
    assert torch.equal(plan.frame([frame]), ref)
    again = new()
    assert again.autotune([frame], cache_path=tmp_path / "tune.txt") == cfg
    assert torch.equal(again.frame([frame]), ref)
