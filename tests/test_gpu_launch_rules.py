"""The launch rules of automatic plans on both sides of their lines, against the CPU oracle: row
tiles of 4 values and 64 lanes up to 2^21 residues, and one pass for N = 2^13 from 192 vectors on
(transforms, products and batches, whose lists count their own vectors).  Exact, so no tolerance."""
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")

THREADS = min(16, os.cpu_count() or 1)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")


def host(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("logN,L,P,bits,ots", [
    (13, 64, 2, 60, 0), (13, 64, 3, 60, 0), (13, 64, 3, 62, 0), (13, 96, 2, 60, 2), (13, 191, 1, 60, 1),
    (14, 64, 2, 60, 0), (14, 43, 3, 60, 1), (15, 64, 1, 61, 0), (15, 13, 5, 60, 0), (16, 32, 1, 60, 0),
    (16, 33, 1, 60, 2), (17, 16, 1, 60, 0), (17, 17, 1, 60, 0),
])
def test_both_sides_of_the_rules(logN, L, P, bits, ots):
    N = 1 << logN
    primes = synth.gen_primes(7900 + logN, N, bits, L)
    psis = oracle.roots(primes, N)
    a, b = synth.residue_batch(7901, primes, N, P), synth.residue_batch(7902, primes, N, P)
    plan = ntt.ntt_plan_create(N, primes, ot_stages=ots)
    try:
        want = oracle.forward(a, primes, psis, THREADS)
        d = dev(a)
        for p in range(ntt.ntt_plan_num_passes(plan)):        # pass by pass: always the plan's split
            ntt.ntt_forward_pass(plan, d, p)
        assert np.array_equal(host(d), want)
        d = dev(a)
        ntt.ntt_forward(plan, d)
        assert np.array_equal(host(d), want)
        ntt.ntt_inverse(plan, d)
        assert np.array_equal(host(d), a)
        c = torch.empty_like(d)
        product = oracle.polymul(a, b, primes, psis, THREADS)
        ntt.ntt_polymul_negacyclic(plan, d, dev(b), c)
        assert np.array_equal(host(c), product)
        if P > 1:      # a batch whose lists lie on either side: one forward job, one key job per polynomial
            keys = oracle.forward(b[:1], primes, psis, THREADS)
            x, y = dev(a[:1]), dev(a)
            batch = ntt.ntt_batch_create([(plan, x, 1, 0, ntt.OP_FORWARD),
                                          (plan, y, P, 0, ntt.OP_FORWARD | ntt.OP_MULKEY | ntt.OP_INVERSE, dev(keys)[0])])
            ntt.ntt_batch_run(batch, ntt.BATCH_GROUPED)
            assert np.array_equal(host(x), want[:1])
            assert np.array_equal(host(y), oracle.polymul(a, np.repeat(b[:1], P, axis=0), primes, psis, THREADS))
            batch.destroy()
    finally:
        plan.destroy()
