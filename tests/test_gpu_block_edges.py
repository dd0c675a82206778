"""Output of stream calls whose blocks do not end on whole bytes: the blocks
exchange the bits of the byte at each boundary between them, so the decode
needs no zeroed staging.  Against the CPU oracle (bits are equal: no
tolerance); the bytes around the output stay untouched, and repeated calls
find the boundaries' words cleared."""
import numpy as np
import pytest

import oracle
from test_gpu_batch import log, pbvd, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

CODES = [(3, (0o7, 0o5)), (6, (0o53, 0o75)), (7, (0o171, 0o133)), (8, (0o247, 0o371)), (9, (0o557, 0o663, 0o711))]


def symbols(K, gens, n, terminated, seed):
    rng = np.random.default_rng(seed)
    return rng.integers(-128, 128, (n + (K - 1 if terminated else 0)) * len(gens), dtype=np.int8)


@pytest.mark.parametrize("K,gens", CODES, ids=["K%d" % c[0] for c in CODES])
@pytest.mark.parametrize("mapping,lanes", [(2, 0), (1, 1), (1, 2)], ids=["wave", "lanes1", "lanes2"])
def test_block_edges(torch, pbvd, K, gens, mapping, lanes):  # noqa: F811
    if lanes == 2 and K < 7:
        pytest.skip("one lane per block")
    log("block edges: K=%d mapping %d lanes %d" % (K, mapping, lanes))
    # blocks of fewer bits than a head and a tail, around whole words and the
    # trips of the kernels; 4, 12, 20, 200: whole bytes or less
    for D, n in ((9, 1), (9, 10), (9, 1000), (11, 737), (12, 600), (13, 14), (31, 1999), (33, 2113), (63, 3000),
                 (100, 6413), (257, 4000), (777, 1555), (2001, 4100), (4, 333), (20, 997), (200, 3333)):
        terminated = (D + n) % 3 != 0
        L = K + D % 30
        syms = symbols(K, gens, n, terminated, D * n)
        want = np.packbits(oracle.decode(K, gens, D, L, syms, n, terminated=terminated)["bits"], bitorder="little")
        d_syms = torch.from_numpy(syms).cuda()
        with pbvd.Plan(K, gens, D, L, terminated=terminated, mapping=mapping, lanes_per_pb=lanes) as plan:
            for shift in (0, 1, 3):  # alignment of the output
                buf = torch.full((want.size + 8,), 0xA5, dtype=torch.uint8, device="cuda")
                out = buf[shift:shift + want.size]
                for _ in range(2):
                    out.fill_(0x5A)
                    plan.decode(d_syms, n, out=out)
                torch.cuda.synchronize()
                host = buf.cpu().numpy()
                assert np.array_equal(host[shift:shift + want.size], want), (D, n, L, shift)
                assert np.all(host[:shift] == 0xA5) and np.all(host[shift + want.size:] == 0xA5), (D, n, shift)


@pytest.mark.parametrize("K,gens", CODES[2:3] + CODES[4:], ids=["K7", "K9"])
def test_block_edges_ranges_and_launches(torch, pbvd, monkeypatch, K, gens):  # noqa: F811
    """Ranges of blocks, and calls of several launches (a small survivor
    budget), end and start in the middle of a byte."""
    log("block edges: ranges, K=%d" % K)
    monkeypatch.setenv("PBVD_WORKSPACE_MB", "1")
    D, L, n = 101, 45, 40000
    syms = symbols(K, gens, n, True, 5)
    bits = oracle.decode(K, gens, D, L, syms, n, terminated=True)["bits"]
    d_syms = torch.from_numpy(syms).cuda()
    for mapping in (1, 2):
        with pbvd.Plan(K, gens, D, L, mapping=mapping) as plan:
            nb = plan.num_blocks(n)
            for first, count in ((0, nb), (0, 7), (5, 1), (3, nb - 3), (nb - 1, 1)):
                lo, hi = first * D, min(n, (first + count) * D)
                want = np.packbits(bits[lo:hi], bitorder="little")
                out = torch.full((want.size,), 0x5A, dtype=torch.uint8, device="cuda")
                plan.decode_ex(d_syms, n, first, count, out=out)
                torch.cuda.synchronize()
                assert np.array_equal(out.cpu().numpy(), want), (mapping, first, count)


def test_block_edges_graph_replays(torch, pbvd):  # noqa: F811
    log("block edges: graph replays")
    K, gens, D, L, n = 7, (0o171, 0o133), 100, 42, 50001
    syms = symbols(K, gens, n, True, 9)
    want = np.packbits(oracle.decode(K, gens, D, L, syms, n, terminated=True)["bits"], bitorder="little")
    d_syms = torch.from_numpy(syms).cuda()
    out = torch.zeros(want.size, dtype=torch.uint8, device="cuda")
    with pbvd.Plan(K, gens, D, L) as plan:
        plan.decode(d_syms, n, out=out)
        torch.cuda.synchronize()
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                plan.decode(d_syms, n, out=out)
        torch.cuda.current_stream().wait_stream(s)
        for _ in range(3):
            out.fill_(0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
            plan.decode(d_syms, n, out=out)  # eager work between the replays
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
        del g
