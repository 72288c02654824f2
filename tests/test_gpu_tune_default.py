"""The autotuner compares with the built-in workgroup target: every entry of its cache
has the built-in target's time beside the chosen one's, the chosen one is no slower,
and the built-in target stays where nothing beat it."""
import json

import pytest
import torch

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")


@pytest.mark.parametrize("n_max,B_max", [(16384, 64), (5000, 16)])
def test_untuned_target_is_timed(tmp_path, n_max, B_max):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = P.lib()
    path = tmp_path / "tune.json"
    try:
        P.tune(P.Context(0), str(path), n_max=n_max, B_max=B_max)
        entries = json.loads(path.read_text())["entries"]
        assert len(entries) == 3 * (4 if B_max == 64 else 3)
        for e in entries:
            assert 0.0 < e["ms"] <= e["untuned_ms"] < 1e3, e
            if e["ms"] == e["untuned_ms"]:
                assert e["target_wgs"] == 1024, e
        P.tune_load(str(path))
    finally:
        lib.nfr_tune_clear()
