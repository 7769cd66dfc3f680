"""The autotuner's JSON cache: a shape stored by a build with other candidates is
timed again, one stored by this build is applied."""
import json

import pytest

from paper_2607_28265_amd import _lib, autotune


class _Theta:
    shape = (250, 13)


class _Ctx:
    n_freq, n_det, device, handle = 1000, 3, 0, None

    def __init__(self):
        self.applied = []

    def set_full_shape(self, a, b):
        self.applied.append((a, b))

    def set_het_shape(self, a, b, c):
        self.applied.append((a, b, c))


@pytest.mark.parametrize("like,kept", [(_lib.GW_FULL, False), (_lib.GW_HET, True)])
def test_stored_shapes(tmp_path, monkeypatch, like, kept):
    path = tmp_path / "shapes.json"
    monkeypatch.setenv("GW_AUTOTUNE_CACHE", str(path))
    monkeypatch.setattr(_lib, "gw_autotune", lambda *a: ((0, 0, 0), 0.5))
    import torch
    dev = torch.cuda.get_device_name(0) if torch.cuda.is_available() else "none"
    path.write_text(json.dumps({json.dumps([dev, like, 250, 1000, 3, 1, 1, None]): {"shape": [128, 64, 0], "ms": 1.0}}))
    ctx = _Ctx()
    shape, ms = autotune.tune(ctx, _Theta(), like, 1, 1)
    if kept:
        assert shape == (128, 64, 0) and ms is None and ctx.applied == [(128, 64, 0)]
    else:
        assert shape == (0, 0, 0) and ms == 0.5 and not ctx.applied
        shape, ms = autotune.tune(ctx, _Theta(), like, 1, 1)
        assert shape == (0, 0, 0) and ms is None and ctx.applied == [(0, 0)]
