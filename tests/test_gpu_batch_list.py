"""Batches on the wave mapping with more PBs than the device holds waves: every
frame against the CPU oracle (bits are equal: no tolerance), and the mapping the
library chooses against tiles of the register kernel in time.  A launch of a wave
per PB takes less than the tiles at these counts (24 and 27 us, 105 and 86 before
the shares of a batch of several K were weighed); 1.25 leaves room for noise."""
import pytest

from test_gpu_batch import check_batch, log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

K3 = dict(K=3, gens=(0o7, 0o5), L=18)
K7 = dict(K=7, gens=(0o171, 0o133), L=42)
K9 = dict(K=9, gens=(0o557, 0o663, 0o711), L=54)


@pytest.mark.parametrize("code,D,frames,hi", [(K7, 16, 500, 512), (K9, 8, 250, 300)], ids=["K7", "K9"])
def test_more_blocks_than_waves(torch, pbvd, code, D, frames, hi):  # noqa: F811
    log("batch list: K=%d" % code["K"])
    info = check_batch(torch, pbvd, [dict(code, D=D)], frames, 100, hi, seed=D)[4]
    assert info["tiles"] == info["blocks"] > (8192 if code is K7 else 4096)


def _us(torch, pbvd, codes, frames):
    fr, so, oo = [], 0, 0
    for ci, n in frames:
        fr.append((so, n, oo, ci))
        so += (n + codes[ci]["K"] - 1) * len(codes[ci]["gens"])
        oo += (n + 7) // 8
    syms = torch.randint(-60, 61, (so,), dtype=torch.int8, device="cuda").view(torch.uint8)
    out = torch.zeros(oo, dtype=torch.uint8, device="cuda")
    with pbvd.Batch(codes) as b:
        b.set_frames(fr, so, oo)
        best = 1e9
        for _ in range(12):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            b.decode(syms, out)
            t0.record()
            for _ in range(10):
                b.decode(syms, out)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) * 100)
        return best


@pytest.mark.parametrize("codes,frames", [
    ([dict(K7, D=16)], [(0, 1000)] * 200),
    ([dict(K7, D=64)], [(0, 1000)] * 1000),
    ([dict(K3, D=16)], [(0, 1000)] * 255),
    ([dict(K7, D=512), dict(K3, D=512)], [(0, 4096)] * 3840 + [(1, 100)]),
    ([dict(K9, D=512), dict(K3, D=512)], [(0, 4096)] * 1920 + [(1, 100)]),
], ids=["K7 12600 short", "K7 16000", "K3 16065 short", "K7 30720 and K3 1", "K9 15360 and K3 1"])
def test_chosen_mapping_is_not_the_slower(torch, pbvd, monkeypatch, codes, frames):  # noqa: F811
    log("batch list: chosen mapping, %d frames" % len(frames))
    chosen = _us(torch, pbvd, codes, frames)
    monkeypatch.setenv("PBVD_WAVE_MAX_PBS", "0")
    tiles = _us(torch, pbvd, codes, frames)
    monkeypatch.delenv("PBVD_WAVE_MAX_PBS")
    chosen = min(chosen, _us(torch, pbvd, codes, frames))  # (the clock rises while the first one runs)
    print("%.1f us, tiles %.1f" % (chosen, tiles), flush=True)
    assert chosen <= 1.25 * tiles
