"""The mapping a batch chooses for codes that leave it open: the wave mapping
for few PBs (one list launch for all K, or for one K, where a wave is there for
every PB, persistent waves otherwise), tiles of the register kernel for many.
Every frame against the CPU oracle (bits are equal: no tolerance)."""
import pytest

from test_gpu_batch import check_batch, log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

ALL_K = [dict(K=3, gens=(0o7, 0o5), D=24, L=18), dict(K=4, gens=(0o15, 0o17), D=64, L=24, terminated=False),
         dict(K=5, gens=(0o25, 0o27, 0o33, 0o37), D=40, L=30), dict(K=6, gens=(0o53, 0o75), D=64, L=36, input_kind=1),
         dict(K=7, gens=(0o171, 0o133), D=64, L=42), dict(K=7, gens=(0o133, 0o171, 0o165), D=32, L=42),
         dict(K=8, gens=(0o247, 0o371), D=64, L=48, terminated=False), dict(K=9, gens=(0o557, 0o663, 0o711), D=96, L=54)]


@pytest.mark.parametrize("frames,hi", [(1, 40), (9, 700), (120, 1500)])
@pytest.mark.parametrize("path", ["list", "persistent", "tiles"])
def test_batch_auto_mapping(torch, pbvd, monkeypatch, path, frames, hi):  # noqa: F811
    if path == "persistent":
        monkeypatch.setenv("PBVD_PERSISTENT_WAVES", "3")  # fewer waves than PBs: work counters
    if path == "tiles":
        monkeypatch.setenv("PBVD_WAVE_MAX_PBS", "0")
    # one K, two (the smallest and the largest) or all
    codes = {1: ALL_K[4:5], 9: [ALL_K[0], ALL_K[7]], 120: ALL_K}[frames]
    log("batch auto mapping: %s, %d frames up to %d bits" % (path, frames, hi))
    _, _, _, _, info = check_batch(torch, pbvd, codes, frames, 1, hi, seed=frames)
    if path != "tiles":
        assert info["tiles"] == info["blocks"]  # a work item per PB


def test_batch_auto_mapping_threshold(torch, pbvd, monkeypatch):  # noqa: F811
    """Shares of wave_max that reach exactly one stay on the wave mapping, one
    PB more does not."""
    monkeypatch.setenv("PBVD_WAVE_MAX_PBS", "128")
    codes = [dict(K=7, gens=(0o171, 0o133), D=8, L=42)]
    log("batch auto mapping: threshold")
    assert check_batch(torch, pbvd, codes, 1, 1024, 1024, seed=3)[4]["tiles"] == 128
    assert check_batch(torch, pbvd, codes, 1, 1025, 1025, seed=3)[4]["tiles"] < 128
