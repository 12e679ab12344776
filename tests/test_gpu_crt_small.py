"""Decomposition of short integers and of few coefficients, against the CPU oracle: the kernel for one
word at the ends of its blocks and prime widths, and launches whose matrix tiles are spread over
workgroups, evenly and with a shorter last part.  Exact, so no tolerance."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")


@pytest.mark.parametrize("L,bits,logN,P,words", [
    (1, 20, 1, 1, (1, 2)), (3, 14, 3, 7, (1, 2, 12, 13)), (60, 62, 7, 3, (1, 2, 12, 13)), (7, 61, 7, 2, (1, 64)),
    (61, 60, 10, 1, (1, 4, 57)),       # 16 tiles in as many parts, one prime in the last
    (60, 60, 13, 1, (1, 12, 13, 56)),  # 15 tiles: 15 parts, and 8 of which the last has one tile
    (45, 60, 14, 1, (2, 5, 42)),       # 12 tiles: 6 parts of 2, and 4 of 3
    (30, 61, 16, 1, (1, 8, 30)),       # 512 lanes: 4 parts and 2 over 8 tiles
])
def test_decompose_short_and_small(L, bits, logN, P, words):
    N = 1 << logN
    primes = synth.gen_primes(9500 + L + bits, N, bits, L)
    plan = ntt.ntt_plan_create(N, primes)
    try:
        for W in words:
            x = np.stack([synth.uniform_wide(9510 + W, p, 1 << (64 * W), N) for p in range(P)])
            x[0, :, 0], x[P - 1, :, N - 1] = 0, np.uint64(0xFFFFFFFFFFFFFFFF)
            x[P - 1, 0, N // 2] = np.uint64(primes[L - 1])
            res = torch.full((P, L, N), -1, dtype=torch.int64, device="cuda")
            ntt.ntt_rns_decompose(plan, torch.from_numpy(np.ascontiguousarray(x).view(np.int64)).to("cuda"), W, res)
            got = res.cpu().numpy().view(np.uint64)
            assert np.array_equal(got, oracle.rns_decompose_words(x, primes)), f"{W} words"
    finally:
        plan.destroy()
