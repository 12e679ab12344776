"""32-bit words on both sides of the column-tile rule (32 columns up to 2^21 residues, 8192 / N1 above),
at every tile that differs: transforms and products against the CPU oracle.  Exact, so no tolerance."""
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")

THREADS = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("logN,log2_n1,L,P", [(13, 0, 64, 4), (13, 0, 86, 3), (13, 5, 257, 1), (14, 7, 43, 3),
                                              (16, 0, 11, 3), (17, 0, 8, 2), (17, 0, 17, 1), (17, 5, 17, 1)])
def test_column_tiles(logN, log2_n1, L, P):
    N = 1 << logN
    primes = synth.gen_primes(8100 + logN + L, N, 30, L)
    psis = oracle.roots(primes, N)
    a, b = synth.residue_batch(8101, primes, N, P), synth.residue_batch(8102, primes, N, P)
    a[0, :, 0] = np.array(primes, dtype=np.uint64) - np.uint64(1)
    dev = [torch.from_numpy(v.astype(np.int32)).to("cuda") for v in (a, b)]
    plan = ntt.ntt_plan_create(N, primes, word_bits=32, log2_n1=log2_n1)
    try:
        c = torch.empty_like(dev[0])
        ntt.ntt_polymul_negacyclic_u32(plan, dev[0], dev[1], c)
        assert np.array_equal(c.cpu().numpy(), oracle.polymul(a, b, primes, psis, THREADS).astype(np.int32)), "product"
        ntt.ntt_forward_u32(plan, dev[0])
        assert np.array_equal(dev[0].cpu().numpy(), oracle.forward(a, primes, psis, THREADS).astype(np.int32)), "forward"
        ntt.ntt_inverse_u32(plan, dev[0])
        assert np.array_equal(dev[0].cpu().numpy(), a.astype(np.int32)), "inverse"
    finally:
        plan.destroy()
