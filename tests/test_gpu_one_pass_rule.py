"""N = 2^13 on both sides of the one-pass rule beyond one vector per CU (a part-filled last round goes in
two passes), for both arithmetic policies: transforms, products and a batch's key rows, against the CPU
oracle.  Exact, so no tolerance."""
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")

N, THREADS = 1 << 13, min(16, os.cpu_count() or 1)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")


def host(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("L,P,bits,ots", [(67, 5, 60, 0), (48, 7, 60, 1), (57, 7, 62, 0), (50, 8, 62, 0), (74, 8, 60, 0)])
def test_part_filled_rounds(L, P, bits, ots):     # 335, 336, 399, 400 and 592 vectors
    primes = synth.gen_primes(7950 + L, N, bits, L)
    psis = oracle.roots(primes, N)
    a, b = synth.residue_batch(7951, primes, N, P), synth.residue_batch(7952, primes, N, P)
    plan = ntt.ntt_plan_create(N, primes, ot_stages=ots)
    try:
        d = dev(a)
        ntt.ntt_forward(plan, d)
        assert np.array_equal(host(d), oracle.forward(a, primes, psis, THREADS)), "forward"
        ntt.ntt_inverse(plan, d)
        assert np.array_equal(host(d), a), "inverse"
        c = torch.empty_like(d)
        ntt.ntt_polymul_negacyclic(plan, d, dev(b), c)
        assert np.array_equal(host(c), oracle.polymul(a, b, primes, psis, THREADS)), "product"
        keys = oracle.forward(b[:1], primes, psis, THREADS)
        batch = ntt.ntt_batch_create([(plan, d, P, 0, ntt.OP_FORWARD | ntt.OP_MULKEY | ntt.OP_INVERSE, dev(keys)[0])])
        ntt.ntt_batch_run(batch, ntt.BATCH_GROUPED)
        assert np.array_equal(host(d), oracle.polymul(a, np.repeat(b[:1], P, axis=0), primes, psis, THREADS)), "batch"
        batch.destroy()
    finally:
        plan.destroy()
