"""Row kernels that the sweeps over plans reach no longer by themselves, against the CPU oracle.

* Rows with an NTT-domain key (a batch's forward + key product + inverse jobs): the dense product takes
  both operands through the rows, so the sweeps over products no longer run these.  Every split, OT
  depth and tile shape, for both arithmetic policies.
* The default tile (8 values, 128 lanes) of automatic plans with primes above 2^60: launches above 2^21
  residues, below which they take 4 values and 64 lanes.

Exact, so no tolerance."""
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")
from paper_2012_01968_amd import autotune  # noqa: E402

THREADS = min(16, os.cpu_count() or 1)
FULL = ntt.OP_FORWARD | ntt.OP_MULKEY | ntt.OP_INVERSE


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")


def host(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("bits", [60, 62])
@pytest.mark.parametrize("logN", list(range(1, 18)))
def test_key_rows(logN, bits):
    N, L, P = 1 << logN, 3, 2
    seed = 8200 + 20 * bits + logN
    primes = synth.gen_primes(seed, N, bits, L)
    psis = oracle.roots(primes, N)
    a, b = synth.residue_batch(seed, primes, N, P), synth.residue_batch(seed + 1, primes, N, 1)
    b[0, 0, :] = np.uint64(primes[0] - 1)
    da, key = dev(a), dev(oracle.forward(b, primes, psis, THREADS))[0]
    want = oracle.polymul(a, np.repeat(b, P, axis=0), primes, psis, THREADS)
    checked = 0
    for base in autotune.candidates(N):
        if base["kernel_path"] != ntt.PATH_SPLIT or base.get("ot_log2_base", min(10, logN - 1)) != min(10, logN - 1):
            continue
        # shapes that differ in the columns only run the same row kernel
        for opts in (o for o in autotune.tile_candidates(N, base) if "col_width" not in o):
            plan = ntt.ntt_plan_create(N, primes, **opts)
            try:
                d = da.clone()
                batch = ntt.ntt_batch_create([(plan, d, P, 0, FULL, key)])
                ntt.ntt_batch_run(batch, ntt.BATCH_GROUPED)
                torch.cuda.synchronize()
                assert np.array_equal(host(d), want), f"N=2^{logN} q<2^{bits} {opts}"
                batch.destroy()
                checked += 1
            finally:
                plan.destroy()
    assert checked > 0


@pytest.mark.parametrize("logN,L,P,bits,ots", [(13, 257, 1, 61, 0), (13, 37, 7, 62, 1), (14, 43, 3, 62, 0), (14, 65, 2, 61, 2),
                                               (15, 65, 1, 61, 0), (15, 13, 5, 62, 1), (16, 33, 1, 62, 0), (16, 11, 3, 61, 2),
                                               (17, 17, 1, 62, 0), (17, 6, 3, 61, 1)])
def test_wide_primes_above_the_small_launches(logN, L, P, bits, ots):
    N = 1 << logN
    assert N * L * P > 1 << 21
    primes = synth.gen_primes(8300 + logN + L, N, bits, L)
    psis = oracle.roots(primes, N)
    a, b = synth.residue_batch(8301, primes, N, P), synth.residue_batch(8302, primes, N, P)
    plan = ntt.ntt_plan_create(N, primes, ot_stages=ots)
    try:
        d, c = dev(a), torch.empty((P, L, N), dtype=torch.int64, device="cuda")
        ntt.ntt_polymul_negacyclic(plan, d, dev(b), c)
        assert np.array_equal(host(c), oracle.polymul(a, b, primes, psis, THREADS)), "product"
        ntt.ntt_forward(plan, d)
        assert np.array_equal(host(d), oracle.forward(a, primes, psis, THREADS)), "forward"
        ntt.ntt_inverse(plan, d)
        assert np.array_equal(host(d), a), "inverse"
        key = dev(oracle.forward(b[:1], primes, psis, THREADS))[0]
        batch = ntt.ntt_batch_create([(plan, d, P, 0, FULL, key)])
        ntt.ntt_batch_run(batch, ntt.BATCH_GROUPED)
        assert np.array_equal(host(d), oracle.polymul(a, np.repeat(b[:1], P, axis=0), primes, psis, THREADS)), "key rows"
        batch.destroy()
    finally:
        plan.destroy()
