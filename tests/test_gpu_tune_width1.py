"""GPU: the autotuner's workgroup size where the widths it chose make every size
the same launch."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
def test_size_is_not_noise(layout, tmp_path, monkeypatch):
    from paper_1601_04017_amd import lpht
    monkeypatch.setenv("XDG_CACHE_HOME", str(tmp_path))
    for _ in range(4):
        tuning, report = lpht.autotune(layout, 18, reps=1, cache=False)
        if tuning["g_find"][1] == 1 and tuning["g_modify"][1] == 1:
            assert tuning["block_threads"] == 256
            assert len(set(report["block_ms"])) == 1
