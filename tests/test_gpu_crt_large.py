"""Conversions of more than 2^31 coefficients in one call: their kernels take two lanes per coefficient,
and a launch has fewer than 2^32 lanes.  One prime, so that 48 GB hold both sides; exact."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")


def test_conversions_above_2_31_coefficients():
    N, P, words = 1 << 17, (1 << 14) + 1, 2
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of free device memory")
    q = int(synth.gen_primes(9960, N, 60, 1)[0])
    plan = ntt.ntt_plan_create(N, [q])
    x = res = back = None
    try:
        high = 0x123456789ABCDEF
        x = torch.empty((P, words, N), dtype=torch.int64, device="cuda")
        gen = torch.Generator(device="cuda")
        gen.manual_seed(9961)
        x[:, 0].random_(0, 1 << 62, generator=gen)
        x[:, 1] = high
        res = torch.full((P, 1, N), -1, dtype=torch.int64, device="cuda")
        ntt.ntt_rns_decompose(plan, x, words, res)
        for p in range(0, P, 512):      # (x_0 mod q + x_1 2^64 mod q) mod q, both below 2^60
            want = (x[p:p + 512, 0] % q + (high << 64) % q) % q
            assert torch.equal(res[p:p + 512, 0], want), f"decompose, polynomials from {p}"
        x = None
        back = torch.full((P, 1, N), -1, dtype=torch.int64, device="cuda")
        ntt.ntt_crt_reconstruct(plan, res, back)     # one prime: the integer is the residue
        for p in range(0, P, 512):
            assert torch.equal(back[p:p + 512], res[p:p + 512]), f"reconstruct, polynomials from {p}"
    finally:
        plan.destroy()
        x = res = back = None
        torch.cuda.empty_cache()
