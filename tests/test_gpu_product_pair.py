"""The two-operand product rows (both operands' forward stages, the product and the inverse stages in
one launch) against the CPU oracle at the edges of their dispatch: the smallest and largest
single-pass sizes, rows whose exchange buffers fit LDS twice and once, vector counts that leave padding
rows, both arithmetic policies, on-the-fly twiddles, and c in place of a.  Exact, so no tolerance."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")


@pytest.mark.parametrize("logN,log2_n1,L,P,bits,ots,r1", [
    (1, -1, 3, 1, 30, 0, 0), (4, -1, 5, 3, 60, 1, 0), (12, 0, 1, 3, 60, 0, 0), (12, -1, 2, 1, 62, 2, 4),
    (13, -1, 2, 1, 60, 0, 0), (13, -1, 1, 1, 61, 0, 0), (13, 6, 1, 3, 54, 0, 4), (8, 4, 3, 1, 60, 0, 0),
    (17, 4, 1, 1, 60, 1, 0), (16, 4, 1, 2, 62, 0, 0), (15, 10, 2, 1, 60, 2, 0),
])
def test_product(logN, log2_n1, L, P, bits, ots, r1):
    N = 1 << logN
    primes = synth.gen_primes(7700 + logN + L, N, bits, L)
    opts = dict(log2_n1=log2_n1, r1=r1)
    if ots:
        opts.update(ot_stages=ots, ot_log2_base=min(10, logN - 1))
    plan = ntt.ntt_plan_create(N, primes, **opts)
    try:
        a, b = synth.residue_batch(7701, primes, N, P), synth.residue_batch(7702, primes, N, P)
        a[0, :, 0] = np.array(primes, dtype=np.uint64) - np.uint64(1)
        b[P - 1, :, N - 1] = 0
        want = oracle.polymul(a, b, primes, oracle.roots(primes, N))
        da, db = (torch.from_numpy(v.view(np.int64)).to("cuda") for v in (a, b))
        c = torch.empty_like(da)
        ntt.ntt_polymul_negacyclic(plan, da, db, c)
        assert np.array_equal(c.cpu().numpy().view(np.uint64), want)
        assert np.array_equal(db.cpu().numpy().view(np.uint64), b) and np.array_equal(da.cpu().numpy().view(np.uint64), a)
        ntt.ntt_polymul_negacyclic(plan, da, db, da)      # c may alias a
        assert np.array_equal(da.cpu().numpy().view(np.uint64), want)
    finally:
        plan.destroy()


@pytest.mark.parametrize("logN,log2_n1,L,P", [(1, 0, 3, 1), (5, 0, 5, 3), (12, 0, 1, 3), (10, 5, 3, 1), (13, 0, 1, 1),
                                              (17, 5, 1, 3), (17, 0, 1, 1), (16, 10, 2, 1)])
def test_product_word32(logN, log2_n1, L, P):
    """The same on 32-bit words, at the narrow and the wide column tiles and rows of 2 to 4096 points."""
    N = 1 << logN
    primes = synth.gen_primes(7800 + logN + L, N, 30, L)
    plan = ntt.ntt_plan_create(N, primes, word_bits=32, log2_n1=log2_n1)
    try:
        a, b = synth.residue_batch(7801, primes, N, P), synth.residue_batch(7802, primes, N, P)
        a[0, :, 0] = np.array(primes, dtype=np.uint64) - np.uint64(1)
        want = oracle.polymul(a, b, primes, oracle.roots(primes, N)).astype(np.int32)
        da, db = (torch.from_numpy(v.astype(np.int32)).to("cuda") for v in (a, b))
        c = torch.empty_like(da)
        ntt.ntt_polymul_negacyclic_u32(plan, da, db, c)
        assert np.array_equal(c.cpu().numpy(), want)
        assert np.array_equal(db.cpu().numpy(), b.astype(np.int32)) and np.array_equal(da.cpu().numpy(), a.astype(np.int32))
        ntt.ntt_polymul_negacyclic_u32(plan, da, db, da)      # c may alias a
        assert np.array_equal(da.cpu().numpy(), want)
    finally:
        plan.destroy()
