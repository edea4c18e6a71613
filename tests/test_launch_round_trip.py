"""What kron_get_launch reports, kron_set_launch takes back: a saved and
restored entry, and an autotuner result applied again, keep the kernel."""
import json

import pytest
import torch

import paper_1304_7054_amd as kron
from paper_1304_7054_amd import tune

COLUMNS = [("f32", 7), ("f32", 10), ("f64", 4), ("f64", 16), ("bf16", 7)]  # 3-D, default: the column kernels


@pytest.mark.parametrize("mode,n", COLUMNS)
def test_every_reported_shape_can_be_set_again(mode, n):
    code = tune.MODES[mode]
    old = kron.kron_get_launch(code, 3, n)
    try:
        kron.kron_set_launch(code, 3, n, -1, 0)
        default = kron.kron_get_launch(code, 3, n)
        kron.kron_set_launch(code, 3, n, *default)
        assert kron.kron_get_launch(code, 3, n) == default
        for blocks in range(65):
            for variant in range(12):
                kron.kron_set_launch(code, 3, n, blocks, variant)
                assert kron.kron_get_launch(code, 3, n) == (blocks, variant)
    finally:
        kron.kron_set_launch(code, 3, n, *old)


def test_saved_default_loads_as_the_default(tmp_path, monkeypatch):
    """Also from a table that marks the default as "builtin"."""
    monkeypatch.setattr(tune, "device_key", lambda: "gfx950|hip-test")
    path = str(tmp_path / "t.json")
    old = kron.kron_get_launch(kron.MODE_F32, 3, 7)
    try:
        kron.kron_set_launch(kron.MODE_F32, 3, 7, -1, 0)
        default = kron.kron_get_launch(kron.MODE_F32, 3, 7)
        for entry in ({"blocks_per_cu": default[0], "variant": default[1]},
                      {"blocks_per_cu": 64, "variant": 8, "builtin": True}):
            tune.save({tune.entry_key("gfx950|hip-test", "f32", 3, 7): json.loads(json.dumps(entry))}, path)
            kron.kron_set_launch(kron.MODE_F32, 3, 7, 2, 5)
            assert tune.load(path) == 1
            assert kron.kron_get_launch(kron.MODE_F32, 3, 7) == default
    finally:
        kron.kron_set_launch(kron.MODE_F32, 3, 7, *old)


@pytest.mark.gpu
@pytest.mark.parametrize("mode,n", COLUMNS)
def test_restored_entry_keeps_the_kernel(mode, n):
    """Bits of the result: the columns contract the slow axis first, the
    variants the fast one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    code, dt = tune.MODES[mode], kron._binding._MODE_DTYPE[tune.MODES[mode]]
    g = torch.Generator(device="cuda").manual_seed(23)
    mats = [torch.randn(n * n, generator=g, device="cuda").to(dt) for _ in range(3)]
    X = torch.randn(300 * n ** 3, generator=g, device="cuda").to(dt)
    fn = getattr(kron, f"kron3d_batched_{mode}")

    def result():
        Y = torch.empty_like(X)
        fn(n, *mats, X, Y, 300)
        return Y

    old = kron.kron_get_launch(code, 3, n)
    try:
        kron.kron_set_launch(code, 3, n, -1, 0)
        want = result()
        kron.kron_set_launch(code, 3, n, 0, 0)
        assert not torch.equal(result(), want)
        kron.kron_set_launch(code, 3, n, -1, 0)
        saved = kron.kron_get_launch(code, 3, n)
        kron.kron_set_launch(code, 3, n, *saved)
        assert torch.equal(result(), want)
        tuned = tune.tune_case(mode, 3, n, target_bytes=1 << 20, reps=1)
        after = result()
        kron.kron_set_launch(code, 3, n, tuned["blocks_per_cu"], tuned["variant"])
        assert torch.equal(result(), after)
    finally:
        kron.kron_set_launch(code, 3, n, *old)
