"""The first late launch (the join with the early region, and the late
removals folded into it) at the edges of its kernels' ranges, against the
oracle: products of M rows, K terms and N = 2^k columns per batch, with K below,
at and above the 64, 128 and 256 terms where lanes and waves start to share a
row, fewer and more rows than a wave takes, and each column tile of the matrix
cores.  Tolerances: those of the complex64 and FP16 paths, the late phase
being FP64."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # n, d, k, late_fold, batches
    (9, 2, 0, 0, 3),      # K = 2
    (9, 10, 0, 0, 5),     # one row of K = 32
    (9, 12, 0, 0, 5),     # one row of K = 64
    (9, 14, 0, 0, 2),     # 128
    (9, 16, 0, 0, 2),     # 256
    (9, 24, 0, 0, 2),     # 4096
    (9, 26, 0, 0, 2),     # two rows of 4096, N = 2
    (9, 31, 0, 0, 2),     # odd depth, 8 or 16 rows
    (9, 16, 1, 4, 2),     # k = 1: K = 32
    (9, 16, 1, 5, 2),     # 64, M = 4 below the 32 rows of a block
    (9, 26, 1, 6, 2),     # 128, M = 64
    (9, 26, 2, 3, 2),     # N = 4, K = 32
    (9, 26, 2, 4, 2),     # 64
    (9, 26, 2, 6, 2),     # 256
    (9, 26, 3, -1, 2),    # N = 8, K = 8
    (9, 26, 3, 3, 2),     # 64
    (9, 26, 3, 7, 2),     # 1024, 8 rows
    (9, 18, 4, -1, 2),    # N = 16: 32 rows, a thread per output
    (9, 18, 4, 2, 2),     # K = 64, 8 rows: two column groups of eight
    (9, 20, 4, -1, 2),    # 64 rows: the 16-column tile, half its 128 rows
    (9, 24, 4, 1, 2),     # 128 rows
    (9, 22, 5, -1, 2),    # the 32-column tile
    (9, 26, 5, 2, 2),
    (9, 24, 6, -1, 2),    # the 64-column tile
    (9, 20, 5, 1, 2),     # N = 32, 16 rows: K = 64
    (9, 26, 1, 7, 2),     # N = 2, K = 256 and 32 rows
    (9, 25, 1, 5, 2),     # N = 2, K = 64: 64 rows or more on the matrix cores
]


@pytest.mark.parametrize("storage", ["c64", "f16"])
@pytest.mark.parametrize("n,d,k,fold,nb", CASES)
def test_first_late_launch(n, d, k, fold, nb, storage):
    from paper_2608_13110_amd import STORE_C64, STORE_F16_BLOCKSCALE, Plan
    c = H.mixed_circuit(n, d, 31 * d + k, dense=0.3)
    bits = W.random_bitstrings(n, nb, W.rng_for(409, d, k))
    print(f"  [gpu] n={n} d={d} k={k} fold={fold} storage={storage}", flush=True)
    plan = Plan.from_circuit(c, dict(late_fold=fold) if fold else None)
    mode = STORE_C64 if storage == "c64" else STORE_F16_BLOCKSCALE
    got = plan.amplitudes(torch.from_numpy(bits).cuda(), k, storage=mode)
    torch.cuda.synchronize()
    per, l2 = H.amp_errors(got.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < (H.TOL_C64 if storage == "c64" else 4e-2), (per, l2)


@pytest.mark.parametrize("d,k,nb", [(34, 3, 130), (40, 6, 17), (44, 8, 5), (36, 8, 65), (30, 7, 513), (32, 7, 257), (46, 1, 2), (48, 5, 1), (50, 4, 1), (52, 2, 1)])
def test_folded_join(d, k, nb):
    # calls of 2^24 entries or more fold three removals into the join matrix on
    # the device, from 2^26 entries on (and 2^25 with the option) so does the
    # plan's own join: against the late phase without a fold (FP64 both: 1e-12)
    # and the oracle
    from paper_2608_13110_amd import Plan
    n = 9
    c = H.mixed_circuit(n, d, 29 * d + k, dense=0.3)
    bits = W.random_bitstrings(n, nb, W.rng_for(463, d, k))
    dev = torch.from_numpy(bits).cuda()
    print(f"  [gpu] n={n} d={d} k={k} batches={nb}", flush=True)
    ref = Plan.from_circuit(c, dict(late_fold=-1)).amplitudes(dev, k)
    for options in (None, dict(late_fold=2)):
        got = Plan.from_circuit(c, options).amplitudes(dev, k)
        torch.cuda.synchronize()
        assert (got - ref).abs().max().item() <= 1e-12 * ref.abs().max().item(), options
    per, _ = H.amp_errors(ref.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < H.TOL_C64, per


@pytest.mark.parametrize("d,fold,nb", [(26, -1, 63), (26, -1, 64), (26, -1, 65), (26, -1, 300), (28, 2, 130), (33, 3, 65)])
def test_groups_of_32_columns(d, fold, nb):
    # 32 columns: few rows take other tiles than many, with the same bits, so a
    # call does not depend on the groups its workspace splits it into
    from paper_2608_13110_amd import Plan
    n, k = 9, 5
    c = H.mixed_circuit(n, d, 43 * d, dense=0.3)
    bits = W.random_bitstrings(n, nb, W.rng_for(521, d, nb))
    dev = torch.from_numpy(bits).cuda()
    print(f"  [gpu] n={n} d={d} k={k} fold={fold} batches={nb}", flush=True)
    plan = Plan.from_circuit(c, dict(late_fold=fold))
    whole = plan.amplitudes(dev, k)
    ws = torch.empty(plan.workspace_bytes(k, 7), dtype=torch.uint8, device="cuda")
    groups = plan.amplitudes(dev, k, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(whole, groups)
    per, l2 = H.amp_errors(whole.cpu().numpy(), oracle.amplitudes(c, bits, k), n)
    assert per < H.TOL_C64 and l2 < H.TOL_C64, (per, l2)
