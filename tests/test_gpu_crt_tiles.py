"""RNS <-> integer conversion at the edges of the kernels' tiles, against the CPU oracle: chains whose
digit slices and column tiles are full, one short and one over (and the register-size steps between
kernels), coefficient counts off the workgroup's 256, primes too short for the wide shift, and the
integers next to 0 and Q, where the quotient estimate goes either way.  Exact, so no tolerance."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")


def host(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("L,bits,logN,P", [
    (1, 20, 1, 1), (4, 62, 5, 3), (5, 60, 8, 1), (7, 62, 6, 5), (8, 60, 7, 3), (15, 61, 8, 3), (16, 60, 9, 1),
    (17, 60, 6, 1), (31, 62, 7, 1), (32, 62, 7, 1), (47, 60, 6, 2), (48, 61, 7, 3), (64, 62, 8, 1), (6, 14, 3, 7),
    (9, 30, 6, 2), (9, 47, 6, 2),
])
def test_conversion_tile_edges(L, bits, logN, P):
    N = 1 << logN
    primes = synth.gen_primes(9600 + L + bits, N, bits, L)
    Q = 1
    for q in primes:
        Q *= q
    plan = ntt.ntt_plan_create(N, primes)
    try:
        W = ntt.ntt_crt_words(plan)
        words = np.stack([synth.uniform_wide(9700 + L, p, Q, N) for p in range(P)])
        edge = [0, Q - 1, 1, Q - 2, min(Q - 1, 1 << 12), Q - min(Q - 1, 1 << 12), Q // 2][:N]
        words[P - 1, :, :len(edge)] = synth.ints_to_words(edge, W)
        res = torch.empty((P, L, N), dtype=torch.int64, device="cuda")
        ntt.ntt_rns_decompose(plan, dev(words), W, res)
        assert np.array_equal(host(res), oracle.rns_decompose_words(words, primes)), "decompose"
        out = torch.empty((P, W, N), dtype=torch.int64, device="cuda")
        ntt.ntt_crt_reconstruct(plan, res, out)
        assert np.array_equal(host(out), words), "reconstruct"
        for Wx in {1, 4, 5, 64}:      # widths of their own, every byte set in one coefficient
            wide = np.stack([synth.uniform_wide(9800 + Wx, p, 1 << (64 * Wx), N) for p in range(P)])
            wide[0, :, N - 1] = np.uint64(0xFFFFFFFFFFFFFFFF)
            ntt.ntt_rns_decompose(plan, dev(wide), Wx, res)
            assert np.array_equal(host(res), oracle.rns_decompose_words(wide, primes)), f"decompose {Wx} words"
    finally:
        plan.destroy()


@pytest.mark.parametrize("L,bits", [(5, 60), (13, 60), (29, 61), (45, 60), (64, 62)])   # one per kernel
def test_conversion_wide_workgroups(L, bits):
    """Launches of 2^16 coefficients and more, whose workgroups have 512 lanes: 513 polynomials of 128
    coefficients end half way through one.  Against the oracle; exact."""
    N, P = 128, 513
    primes = synth.gen_primes(9900 + L, N, bits, L)
    Q = 1
    for q in primes:
        Q *= q
    plan = ntt.ntt_plan_create(N, primes)
    try:
        W = ntt.ntt_crt_words(plan)
        words = np.stack([synth.uniform_wide(9950 + L, p, Q, N) for p in range(P)])
        edge = [0, Q - 1, 1, Q - 2]
        words[P - 1, :, N - len(edge):] = synth.ints_to_words(edge, W)
        res = torch.empty((P, L, N), dtype=torch.int64, device="cuda")
        ntt.ntt_rns_decompose(plan, dev(words), W, res)
        assert np.array_equal(host(res), oracle.rns_decompose_words(words, primes)), "decompose"
        out = torch.full((P, W, N), -1, dtype=torch.int64, device="cuda")
        ntt.ntt_crt_reconstruct(plan, res, out)
        assert np.array_equal(host(out), words), "reconstruct"
    finally:
        plan.destroy()
