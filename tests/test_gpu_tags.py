"""The register kernel with survivor tags at the edges of its loops: forward
ranges around whole trips and groups of four stages, overlaps shorter than a
group, blocks that start from the known state and end before every state is
reached, blocks of different lengths in one wave, symbol buffers at every byte
alignment, and symbols drawn from the whole int8 range with runs of -128 (the
widest metrics and many ties).  Bits and final metrics equal the oracle's
exactly (integer arithmetic)."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# the registered codes of 32 states and more
CODES = [(7, (0o171, 0o133)), (7, (0o133, 0o171, 0o165)), (9, (0o557, 0o663, 0o711)), (6, (0o53, 0o75)),
         (7, (0o133, 0o171)), (8, (0o247, 0o371)), (9, (0o561, 0o753)), (6, (0o47, 0o53, 0o75)),
         (7, (0o117, 0o127, 0o155, 0o171)), (6, (0o46, 0o73))]


def extreme_symbols(rng, n):
    buf = rng.integers(0, 256, n, dtype=np.uint8)
    style = rng.integers(0, 4)
    if style == 1:
        buf = rng.choice(np.array([0x80, 0x7f], np.uint8), n)
    elif style == 2:
        buf[rng.random(n) < 0.8] = 0x80
    elif style == 3:
        buf[rng.random(n) < 0.9] = 0
    return buf


def decode(torch, pbvd, K, gens, D, L, terminated, kind, lanes, buf, at, n, want_pm=True):
    R = len(gens)
    T = n + (K - 1 if terminated else 0)
    d = torch.from_numpy(buf).cuda()[at:at + T * R]
    with pbvd.Plan(K, gens, D, L, terminated, kind, lanes_per_pb=lanes) as plan:
        nb = plan.num_blocks(n)
        out, pm = plan.decode_ex(d, n, 0, nb, want_pm=want_pm)
        torch.cuda.synchronize()
        return np.unpackbits(out.cpu().numpy(), bitorder="little")[:n], pm.cpu().numpy()[:nb] if want_pm else None


@pytest.mark.parametrize("code", CODES, ids=lambda c: "k%d_%o" % (c[0], c[1][0]))
def test_trip_and_group_edges(code, monkeypatch):
    import torch
    from paper_1608_00066_amd import pbvd
    K, gens = code
    V, R = K - 1, len(gens)
    U = V * 4 // math.gcd(V, 4)
    rng = np.random.default_rng(10 * K + R)
    monkeypatch.setenv("PBVD_FOLD_SIMDS", "1")
    lane_sets = [1] + ([2] if K >= 7 else []) + ([4] if K >= 8 else []) + ([8] if K == 9 else [])
    for T in (1, 2, V, V + 1, U - 1, U, U + 1, 2 * U, 3 * U + 5, 7 * U + 2, 40 * U + 3):
        for D, L in ((8192, 0), (8, 0), (16, 1), (13, 3), (32, 4), (24, 24), (U, U), (40, V + 2)):
            terminated = bool(rng.integers(0, 2)) and T > V
            n = T - (V if terminated else 0)
            if n > 2000 and D < 16:
                continue
            kind, at, lanes = int(rng.integers(0, 2)), int(rng.integers(0, 4)), int(rng.choice(lane_sets))
            buf = extreme_symbols(rng, T * R + 4)
            print("tags: K=%d R=%d T=%d D=%d L=%d term=%d kind=%d at=%d lanes=%d" % (K, R, T, D, L, terminated, kind, at,
                                                                                  lanes), flush=True)
            ref = oracle.decode(K, gens, D, L, buf[at:at + T * R], n, terminated=terminated, input_kind=kind, want_pm=True)
            bits, pm = decode(torch, pbvd, K, gens, D, L, terminated, kind, lanes, buf, at, n)
            assert np.array_equal(bits, ref["bits"])
            assert np.array_equal(pm, ref["final_pm"])
            bits, _ = decode(torch, pbvd, K, gens, D, L, terminated, kind, lanes, buf, at, n, want_pm=False)
            assert np.array_equal(bits, ref["bits"])


@pytest.mark.parametrize("code", CODES, ids=lambda c: "k%d_%o" % (c[0], c[1][0]))
def test_mixed_lengths_in_a_tile(code):
    """Frames from one bit to a few blocks in a batch: tiles of blocks of
    different lengths, known starts next to each other, unterminated ends."""
    import torch
    from paper_1608_00066_amd import pbvd
    K, gens = code
    R = len(gens)
    rng = np.random.default_rng(20 * K + R)
    for D, L, terminated in ((64, 6 * K, True), (24, 3, True), (16, 0, False), (40, 11, False)):
        codes = [dict(K=K, gens=gens, D=D, L=L, terminated=terminated, lanes_per_pb=int(1 if K < 7 else rng.integers(1, 3)))]
        frames, so, oo = [], int(rng.integers(0, 4)), 0
        for _ in range(90):
            n = int(rng.integers(1, 4 * D))
            frames.append((so, n, oo, 0))
            so += (n + (K - 1 if terminated else 0)) * R
            oo += (n + 7) // 8
        buf = extreme_symbols(rng, so)
        print("tags batch: K=%d R=%d D=%d L=%d term=%d lanes=%d" % (K, R, D, L, terminated, codes[0]["lanes_per_pb"]),
              flush=True)
        out = torch.zeros(oo, dtype=torch.uint8, device="cuda")
        with pbvd.Batch(codes) as b:
            b.set_frames(frames, so, oo)
            b.decode(torch.from_numpy(buf).cuda(), out)
            torch.cuda.synchronize()
        host = out.cpu().numpy()
        for s, n, o, _ in frames:
            T = n + (K - 1 if terminated else 0)
            ref = oracle.decode(K, gens, D, L, buf[s:s + T * R], n, terminated=terminated)["bits"]
            assert np.array_equal(np.unpackbits(host[o:o + (n + 7) // 8], bitorder="little")[:n], ref), "frame of %d bits" % n
