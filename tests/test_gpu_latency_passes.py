"""Passes over tensors too small to fill the chip (2^13 to 2^20 entries, no tile
options): every tensor size of the range and its neighbours, odd depths, several
batches up to where the other pass kernel takes over, against the oracle, and
where no state vector fits against the complex128 sweep."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d", list(range(24, 44)))
@pytest.mark.parametrize("first_parity,nb", [(0, 1), (1, 3)])
def test_widths(d, first_parity, nb):
    from paper_2608_13110_amd import Plan
    n = 9
    c = H.mixed_circuit(n, d, 5 * d + first_parity, first_parity=first_parity, dense=0.3)
    bits = W.random_bitstrings(n, nb, W.rng_for(443, d, nb))
    psi = oracle.statevector(c)
    plan = Plan.from_circuit(c)
    dev = torch.from_numpy(bits).cuda()
    for k in (0, 4):
        print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
        got = plan.amplitudes(dev, k)
        torch.cuda.synchronize()
        per, l2 = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits, k, psi), n)
        assert per < H.TOL_C64, (d, k, per, l2)


@pytest.mark.parametrize("n,d,k,nb", [(40, 26, 3, 1), (41, 33, 5, 2), (38, 40, 2, 1)])
def test_against_complex128(n, d, k, nb):
    from paper_2608_13110_amd import Plan
    c = H.mixed_circuit(n, d, 17 * n + d, dense=0.2)
    bits = W.random_bitstrings(n, nb, W.rng_for(449, n, d))
    plan = Plan.from_circuit(c)
    dev = torch.from_numpy(bits).cuda()
    print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
    got = plan.amplitudes(dev, k)
    ref = plan.debug_amplitudes_c128(dev, k)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got.cpu().numpy(), ref.cpu().numpy(), n)
    assert per < H.TOL_C64, (per, l2)


@pytest.mark.parametrize("d", [28, 33])
def test_same_updates_as_other_tiles(d):
    # as many batches as stay here and more, in one group and split over
    # several: the same updates whichever passes carry them, so the same bits
    # up to the FP64 late phase
    from paper_2608_13110_amd import Plan
    n, k = 10, 2
    c = H.mixed_circuit(n, d, 19 * d, dense=0.3)
    h = (d + 1) // 2
    nb = (1 << (20 - h)) + 3
    bits = torch.from_numpy(W.random_bitstrings(n, nb, W.rng_for(457, d))).cuda()
    print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
    plan, other = Plan.from_circuit(c), Plan.from_circuit(c, dict(max_tile_bits=9, low_bits=3, reg_bits=3))
    ws = torch.empty(plan.workspace_bytes(k, 5), dtype=torch.uint8, device="cuda")
    ref = other.amplitudes(bits, k)
    for got in (plan.amplitudes(bits, k), plan.amplitudes(bits[:-3].contiguous(), k), plan.amplitudes(bits, k, workspace=ws)):
        torch.cuda.synchronize()
        assert (got - ref[: len(got)]).abs().max().item() <= 1e-13 * ref.abs().max().item()


@pytest.mark.parametrize("d,nb", [(25, 130), (26, 130), (28, 70), (31, 40), (34, 10), (36, 5), (37, 3), (40, 2), (41, 1),
                                  (43, 1), (46, 1), (47, 1), (50, 1), (52, 1), (53, 1), (55, 1)])
def test_tiles_by_size(d, nb):
    # the tiles that calls without tile options take, at each change of the
    # rule, against the plan's own tiles asked for by name: the same bits up to
    # the FP64 late phase
    from paper_2608_13110_amd import Plan
    n, k = 7, 1
    c = H.mixed_circuit(n, d, 23 * d, dense=0.3)
    bits = torch.from_numpy(W.random_bitstrings(n, nb, W.rng_for(461, d))).cuda()
    print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
    got = Plan.from_circuit(c).amplitudes(bits, k)
    ref = Plan.from_circuit(c, dict(max_tile_bits=13, low_bits=4, reg_bits=5)).amplitudes(bits, k)
    torch.cuda.synchronize()
    assert (got - ref).abs().max().item() <= 1e-13 * ref.abs().max().item()
    per, _ = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits.cpu().numpy(), k), n)
    assert per < H.TOL_C64, per


@pytest.mark.parametrize("d,nb", [(48, 16), (50, 8), (52, 4), (52, 5), (54, 2), (56, 1)])
def test_streaming_tiles(d, nb):
    # tensors of 2 GiB in all, whose lines the passes mark as not to be kept, in
    # tiles of 256 threads (2^24 to 2^26 entries) and of 512, against 32 entries
    # per thread, where no pass does: the same bits up to the FP64 late phase
    from paper_2608_13110_amd import Plan
    n, k = 7, 1
    c = H.mixed_circuit(n, d, 41 * d, dense=0.3)
    bits = torch.from_numpy(W.random_bitstrings(n, nb, W.rng_for(509, d))).cuda()
    print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
    got = Plan.from_circuit(c).amplitudes(bits, k)
    ref = Plan.from_circuit(c, dict(max_tile_bits=13, low_bits=4, reg_bits=5)).amplitudes(bits, k)
    torch.cuda.synchronize()
    assert (got - ref).abs().max().item() <= 1e-13 * ref.abs().max().item()
