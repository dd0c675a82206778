"""The register kernel's tag body at the end of the input: whether a wave's last
trips fetch whole windows of symbols depends on how far its blocks' ends lie from
the end of the buffer, here every distance from 0 to beyond two trips, for a wave
of whole blocks and the edge blocks after it, with blocks of less than one trip
and of a few (bits are equal to the oracle's: no tolerance)."""
import numpy as np
import pytest

import oracle
from test_gpu_batch import log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CODES = [(6, (0o53, 0o75)), (7, (0o171, 0o133)), (7, (0o133, 0o171, 0o165)), (7, (0o117, 0o127, 0o155, 0o171)),
         (8, (0o247, 0o371)), (9, (0o557, 0o663, 0o711))]


@pytest.mark.parametrize("K,gens", CODES, ids=["K%d_R%d" % (c[0], len(c[1])) for c in CODES])
@pytest.mark.parametrize("D,L", [(8, 1), (16, 9), (16, 40)])
def test_distance_of_the_last_window_from_the_input_end(torch, pbvd, K, gens, D, L):  # noqa: F811
    log("tag windows: K=%d R=%d D=%d L=%d" % (K, len(gens), D, L))
    rng = np.random.default_rng(K * D + L)
    with pbvd.Plan(K, gens, D, L, mapping=1, lanes_per_pb=1) as plan, \
            pbvd.Plan(K, gens, D, L, terminated=False, mapping=1, lanes_per_pb=1) as open_plan:
        for extra in range(0, 62):
            n = 66 * D + extra
            p = open_plan if extra % 3 == 1 else plan
            term = p is plan
            syms = rng.integers(-128, 128, (n + (K - 1 if term else 0)) * len(gens), dtype=np.int8)
            want = np.packbits(oracle.decode(K, gens, D, L, syms, n, terminated=term)["bits"], bitorder="little")
            got = p.decode(torch.from_numpy(syms).cuda(), n)
            assert np.array_equal(got.cpu().numpy()[:want.size], want), (extra, term)
