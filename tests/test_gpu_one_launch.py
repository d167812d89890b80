"""Amplitude calls of small tensors, which run as one launch: every tensor size
up to the kernel's largest and the one above it, odd depths (the top slot is
removed and doubled), no and many open legs, more qubits than one chunk of
phases covers, dense rank-2 gates, against the oracle and against the
complex128 sweep (another path altogether) where no state vector fits."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def run(c, bits, k, options=None):
    from paper_2608_13110_amd import Plan
    print(f"  [gpu] n={c.n} d={c.d} k={k} batches={len(bits)}", flush=True)
    plan = Plan.from_circuit(c, options)
    d = torch.from_numpy(bits).cuda()
    got = plan.amplitudes(d, k)
    torch.cuda.synchronize()
    return plan, d, got.cpu().numpy()


@pytest.mark.parametrize("d", list(range(2, 28)))
@pytest.mark.parametrize("first_parity,nb", [(0, 1), (1, 5)])
def test_widths(d, first_parity, nb):
    n = 10
    c = H.mixed_circuit(n, d, 7 * d + first_parity, first_parity=first_parity, dense=0.3)
    bits = W.random_bitstrings(n, nb, W.rng_for(431, d, nb))
    psi = oracle.statevector(c)
    for k in sorted({0, 1, min(3, d // 2), min(6, d // 2), min(9, d // 2)}):
        _, _, got = run(c, bits, k)
        per, l2 = H.amp_errors(got, oracle.amplitudes(c, bits, k, psi), n)
        assert per < H.TOL_C64, (d, k, per, l2)


@pytest.mark.parametrize("n,d,k", [(3, 2, 0), (2, 24, 1), (40, 24, 6), (40, 21, 0), (70, 20, 5), (33, 23, 7)])
def test_against_complex128(n, d, k):
    c = H.mixed_circuit(n, d, 13 * n + d, dense=0.2)
    bits = W.random_bitstrings(n, 3, W.rng_for(433, n, d))
    plan, dev, got = run(c, bits, k)
    ref = plan.debug_amplitudes_c128(dev, k)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got, ref.cpu().numpy(), n)
    assert per < H.TOL_C64, (per, l2)


def test_many_batches_and_options():
    c = H.mixed_circuit(9, 14, 3, dense=0.3)
    bits = W.random_bitstrings(9, 3000, W.rng_for(439))
    ref = oracle.amplitudes(c, bits, 3)
    whole = None
    # any tile options without fused phases give the same updates, bit for bit
    for options in (None, dict(max_tile_bits=6, low_bits=2, reg_bits=3), dict(late_fold=2)):
        _, _, got = run(c, bits, 3, options)
        per, l2 = H.amp_errors(got, ref, 9)
        assert per < H.TOL_C64, (options, per, l2)
        whole = got if whole is None else whole
        assert np.abs(got - whole).max() <= 1e-13 * np.abs(whole).max()


@pytest.mark.parametrize("d", list(range(2, 25)))
def test_same_updates_as_the_own_passes(d):
    # the host emulation of the plan's own passes does the same FP32 updates in
    # the same order, so only the FP64 join and late program differ (up to 2^12
    # products: 2^12 x 2^-53, and amplitudes some 2^5 below the sum of the
    # products' sizes: 1e-11).  One update rounded in another order moves an
    # amplitude by some 2^-24 / 2^6.
    n = 9
    for k in sorted({0, min(3, d // 2)}):
        c = H.mixed_circuit(n, d, 37 * d + k, dense=0.3)
        bits = W.random_bitstrings(n, 3, W.rng_for(503, d, k))
        plan, _, got = run(c, bits, k)
        ref = plan.debug_emulate_device(bits, k)
        assert np.abs(got - ref).max() <= 1e-11 * max(np.abs(ref).max(), 2.0 ** (-n / 2)), (d, k)
