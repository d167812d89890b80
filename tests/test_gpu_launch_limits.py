"""Calls whose threads, one launch for all of them, would reach the 2^32 that a
launch has to stay below."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_more_batches_than_one_launch_takes():
    # 2^23 + 5 batches of 2^12 entries: a block of 512 threads each
    from paper_2608_13110_amd import Plan
    n, d, nb = 3, 24, (1 << 23) + 5
    c = H.mixed_circuit(n, d, 5, dense=0.3)
    plan = Plan.from_circuit(c)
    assert plan.info(0)["boundary_bits"] == 12
    index = torch.from_numpy(W.rng_for(487).integers(0, 1 << n, size=nb, dtype=np.uint8)).cuda()
    bits = torch.stack([(index >> (n - 1 - j)) & 1 for j in range(n)], dim=1).contiguous()
    ws = torch.empty(plan.workspace_bytes(0, 64), dtype=torch.uint8, device="cuda")
    print(f"  [gpu] n={n} d={d} batches={nb}", flush=True)
    got = plan.amplitudes(bits, 0, workspace=ws)
    torch.cuda.synchronize()
    every = np.array([[(i >> (n - 1 - j)) & 1 for j in range(n)] for i in range(1 << n)], dtype=np.uint8)
    ref = torch.from_numpy(oracle.amplitudes(c, every, 0)).cuda()[index.long()]
    err = (got - ref).abs() / ref.abs().clamp_min(2.0 ** (-n / 2))
    assert err.max().item() < H.TOL_C64


def test_join_of_2_to_the_32_outputs():
    # 2^32 entries, three open legs and no removal folded: a thread per output
    # of the join is 2^32 of them
    from paper_2608_13110_amd import Plan
    n, d, k = 9, 64, 3
    c = H.mixed_circuit(n, d, 7, dense=0.3)
    plan = Plan.from_circuit(c, dict(late_fold=-1))
    assert plan.info(k)["boundary_bits"] == 32
    size = plan.workspace_bytes(k, 1)
    if torch.cuda.mem_get_info()[0] < size + (1 << 30):
        pytest.skip("needs %d GiB of free device memory" % (size >> 30))
    bits = W.random_bitstrings(n, 1, W.rng_for(491))
    print(f"  [gpu] n={n} d={d} k={k} workspace {size >> 30} GiB", flush=True)
    got = plan.amplitudes(torch.from_numpy(bits).cuda(), k)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < H.TOL_C64 and l2 < H.TOL_C64, (per, l2)
