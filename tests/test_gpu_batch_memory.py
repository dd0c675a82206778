"""A batch whose state-parallel PBs would take more survivor memory with a wave
each than the budget or the device has takes fewer waves (persistent ones) and is
not refused; its frames equal the oracle's (no tolerance)."""
import pytest

from test_gpu_batch import check_batch, log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

K9 = dict(K=9, gens=(0o557, 0o663, 0o711), L=54, mapping=2)


def test_more_than_the_device_has(torch, pbvd, monkeypatch):  # noqa: F811
    log("batch memory: device")
    # 31,250 PBs of 350,000 stages: 350 GB with a wave each, 46 GB on 4096 waves
    monkeypatch.setenv("PBVD_WORKSPACE_MB", str(1 << 20))
    D, per = 350000, 250
    n = D * per
    frames = [(i * (n + 8) * 3, n, i * (n // 8), 0) for i in range(125)]
    with pbvd.Batch([dict(K9, D=D)]) as b:
        b.set_frames(frames, 125 * (n + 8) * 3, 125 * (n // 8))
        info = b.info()
        assert info["tiles"] == 125 * per and info["workspace_bytes"] < 100 << 30


def test_more_than_the_budget(torch, pbvd, monkeypatch):  # noqa: F811
    log("batch memory: budget")
    monkeypatch.setenv("PBVD_WORKSPACE_MB", "2")
    info = check_batch(torch, pbvd, [dict(K9, D=64), dict(K=7, gens=(0o171, 0o133), L=42, D=64, mapping=1)], 60, 100,
                       1500, seed=4)[4]
    assert info["workspace_bytes"] < 4 << 20
