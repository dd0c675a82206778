"""A captured stream call whose blocks do not end on whole bytes, on a plan
whose earlier calls took another kernel: the capture allocates nothing that
those calls have not allocated, and every replay equals the oracle's bits
(no tolerance) with the plan's own eager calls in between."""
import numpy as np
import pytest

import oracle
from test_gpu_batch import log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,gens", [(3, (0o7, 0o5)), (5, (0o23, 0o35))], ids=["K3", "K5"])
def test_capture_after_calls_of_another_kernel(torch, pbvd, monkeypatch, K, gens):  # noqa: F811
    log("capture: K=%d" % K)
    monkeypatch.setenv("PBVD_WAVE_MAX_PBS", "8")
    D, L, n, count = 100, 6 * K, 2000, 5
    rng = np.random.default_rng(K)
    syms = rng.integers(-128, 128, (n + K - 1) * len(gens), dtype=np.int8)
    bits = oracle.decode(K, gens, D, L, syms, n, terminated=True)["bits"]
    whole, part = np.packbits(bits, bitorder="little"), np.packbits(bits[:count * D], bitorder="little")
    d_syms = torch.from_numpy(syms).cuda()
    out = torch.zeros(part.size, dtype=torch.uint8, device="cuda")
    all_out = torch.zeros(whole.size, dtype=torch.uint8, device="cuda")
    with pbvd.Plan(K, gens, D, L) as plan:
        assert plan.call_lanes(n) == 1 and plan.call_lanes(n, 0, count) == 64
        plan.decode(d_syms, n, out=all_out)  # the register kernel
        torch.cuda.synchronize()
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                plan.decode_ex(d_syms, n, 0, count, out=out)  # the state-parallel kernel
        torch.cuda.current_stream().wait_stream(s)
        for _ in range(3):
            out.fill_(0x5A)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), part)
            all_out.fill_(0x5A)
            plan.decode(d_syms, n, out=all_out)
            torch.cuda.synchronize()
            assert np.array_equal(all_out.cpu().numpy(), whole)
        del g
