"""GPU tests of the ring geometry (Sec. 6.3) by slicing its wrap-pair CZ
bonds: the sum over 2^m open-chain slices (run in grouped launches of up to
1024 slices), through the C ABI, against the FP64 oracle's state vector of
the ring itself."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2608_13110_amd import lib
    lib()
    yield


@pytest.mark.parametrize("n,d,k,opts", [(6, 6, 0, None), (8, 8, 2, None), (10, 9, 2, None),
                                        (12, 12, 3, dict(max_tile_bits=6, low_bits=2, reg_bits=3)),
                                        (16, 16, 4, None), (20, 20, 4, dict(max_tile_bits=8)),
                                        # 4096 slices: four groups of 1024
                                        (24, 24, 2, None)])
def test_ring_matches_oracle(n, d, k, opts):
    from paper_2608_13110_amd import RingPlan
    c = W.ring_circuit(n, d, n, W.rng_for(140, n, d))
    bits = W.random_bitstrings(n, 3, W.rng_for(141, n, d))
    rp = RingPlan.from_circuit(c, opts)
    info = rp.info(k, len(bits))
    print(f"  [gpu] ring n={n} d={d} k={k}: {info['slices']} slices of width {info['width']}", flush=True)
    got = rp.amplitudes(torch.from_numpy(bits).cuda(), k)
    torch.cuda.synchronize()
    ref = oracle.amplitudes(c, bits, k)
    per, l2 = H.amp_errors(got.cpu().numpy(), ref, n)
    assert per < H.TOL_C64 and l2 < H.TOL_C64, (per, l2)
    rp.close()


def test_ring_equals_host_emulation_of_its_slices():
    from paper_2608_13110_amd import RingPlan
    c = W.with_gate_values(W.ring_circuit(10, 10, 0, W.rng_for(142, 1)), W.rng_for(142, 2))
    bits = W.random_bitstrings(10, 2, W.rng_for(142, 3))
    rp = RingPlan.from_circuit(c, dict(max_tile_bits=6, low_bits=2, reg_bits=3))
    got = rp.amplitudes(torch.from_numpy(bits).cuda(), 2).cpu().numpy()
    emu = rp.debug_emulate_device(bits, 2)
    per, l2 = H.amp_errors(got, emu, 10)
    assert per < 1e-6


@pytest.mark.parametrize("d,k,nb,opts", [
    (44, 2, 64, None),                              # 2^22 entries: the passes over the lowest slots stream
    (52, 3, 4, None),                               # 2^26: every pass, 256 threads a tile
    (56, 1, 1, None),                               # 2^28: 512 threads
    (52, 2, 4, dict(reg_bits=4, math=2)),           # fused phases
    (30, 2, 1 << 13, dict(max_tile_bits=13, reg_bits=4))])
def test_ring_of_slices_of_two_gib(d, k, nb, opts):
    # slices of 2 GiB run one by one, with the passes whose lines are not kept
    import dataclasses
    from paper_2608_13110_amd import RingPlan
    n = 10
    c = H.mixed_circuit(n, d, d, dense=0.3)
    wrap = [(layer, n - 1, W.GATE_CZ, None) for layer in range(1, d + 1) if W.brickwork_pairs(n, layer, 1)[:1] == [1]]
    c = dataclasses.replace(c, gates=sorted(list(c.gates) + wrap[3:5], key=lambda g: (g[0], g[1])))
    bits = W.random_bitstrings(n, nb, W.rng_for(143, d))
    rp = RingPlan.from_circuit(c, opts)
    info = rp.info(k, nb)
    print(f"  [gpu] ring n={n} d={d} k={k} batches={nb}: {info}", flush=True)
    assert info["slices"] == 4 and info["workspace_bytes"] >= 2 << 30
    got = rp.amplitudes(torch.from_numpy(bits).cuda(), k)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < H.TOL_C64 and l2 < H.TOL_C64, (per, l2)
    rp.close()


@pytest.mark.parametrize("wraps,k,nb", [(1, 0, 1), (1, 3, 3), (2, 0, 33), (2, 3, 100), (3, 2, 67), (4, 0, 5), (5, 3, 31), (6, 1, 9)])
def test_sum_of_few_slices(wraps, k, nb):
    # 2 to 64 slices, with fewer outputs than a block takes, as many, and more
    import dataclasses
    from paper_2608_13110_amd import RingPlan
    n, d = 10, 14
    c = H.mixed_circuit(n, d, wraps, dense=0.3)
    wrap = [(layer, n - 1, W.GATE_CZ, None) for layer in range(1, d + 1) if W.brickwork_pairs(n, layer, 1)[:1] == [1]]
    c = dataclasses.replace(c, gates=sorted(list(c.gates) + wrap[:wraps], key=lambda g: (g[0], g[1])))
    bits = W.random_bitstrings(n, nb, W.rng_for(144, wraps))
    rp = RingPlan.from_circuit(c)
    assert rp.info(k, nb)["slices"] == 1 << wraps
    print(f"  [gpu] ring n={n} d={d} k={k} batches={nb} slices={1 << wraps}", flush=True)
    got = rp.amplitudes(torch.from_numpy(bits).cuda(), k)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < H.TOL_C64 and l2 < H.TOL_C64, (per, l2)
    rp.close()
