"""The state-parallel kernel at the edges of its loops: forward ranges one
stage around whole trips (W = V floor(32 / V) stages) and pairs of trips,
starts in the middle of a round of phases, known and unknown start states,
symbol buffers at every byte alignment, and symbols drawn from the whole int8
range (ties and the widest metrics).  Bits, final metrics and survivor
decisions equal the oracle's exactly (integer arithmetic)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CODES = {3: (0o7, 0o5), 4: (0o13, 0o15, 0o17), 5: (0o25, 0o27, 0o33, 0o37), 6: (0o47, 0o53, 0o75),
         7: (0o171, 0o133), 8: (0o225, 0o331, 0o367), 9: (0o557, 0o663, 0o711)}


@pytest.mark.parametrize("K", sorted(CODES))
def test_trip_edges(K):
    import torch
    from paper_1608_00066_amd import pbvd
    gens, V, R = CODES[K], K - 1, len(CODES[K])
    W = V * (32 // V)
    rng = np.random.default_rng(100 + K)
    for terminated in (True, False):
        for T in (V + 1, W - 1, W, W + 1, W + V + 1, 2 * W, 3 * W - 1, 3 * W, 4 * W + 1, 5 * W + 2, 62 * W, 125 * W + 3):
            n = T - (V if terminated else 0)
            if n < 1:
                continue
            # one block (known start) and several short ones
            for D, L in ((8192, 0), (16, V + 3)):
                at = int(rng.integers(0, 4))  # byte alignment of the first symbol
                kind = int(rng.integers(0, 2))
                buf = rng.integers(0, 256, T * R + 4, dtype=np.uint8)
                if rng.random() < 0.5:
                    buf[rng.random(buf.size) < 0.7] = 0x80  # mostly -128: ties
                syms = buf[at:at + T * R]
                d = torch.from_numpy(buf).cuda()[at:at + T * R]
                print("wave rounds: K=%d T=%d D=%d L=%d term=%d at=%d kind=%d" % (K, T, D, L, terminated, at, kind),
                      flush=True)
                with pbvd.Plan(K, gens, D, L, terminated, kind, mapping=pbvd.PBVD_MAP_WAVE) as plan:
                    nb = plan.num_blocks(n)
                    out, pm = plan.decode_ex(d, n, 0, nb, want_pm=True)
                    out2, dec = plan.debug_survivors(d, n, 0, nb) if D + L < 100 else (out, None)
                    torch.cuda.synchronize()
                ref = oracle.decode(K, gens, D, L, syms, n, terminated=terminated, input_kind=kind, want_pm=True,
                                    want_dec=dec is not None)
                for o in (out, out2):
                    assert np.array_equal(np.unpackbits(o.cpu().numpy(), bitorder="little")[:n], ref["bits"])
                assert np.array_equal(pm.cpu().numpy()[:nb], ref["final_pm"])
                if dec is not None:
                    assert np.array_equal(dec.cpu().numpy()[:nb], ref["dec"])
