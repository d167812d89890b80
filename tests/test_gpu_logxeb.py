"""log-XEB over one block's share of components and over many blocks', against
the oracle.  FP64 on both sides: the sums of up to 2^20 logarithms of size 50
agree to 2^20 x 2^-53 relative at worst, so 1e-9 on F and SE."""
import math

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def amps_of(nb, k, seed):
    rng = W.rng_for(419, nb, k, seed)
    shape = (nb, 1 << k)
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 2.0 ** -30


# 1024 components end the small block, 8192 the single one; 128 blocks of 1024 end the grid's growth
@pytest.mark.parametrize("nb,k,select", [(1, 0, False), (1024, 0, False), (1025, 0, False), (2048, 2, False), (2049, 2, False), (513, 3, False),
                                         (2051, 8, False), (2051, 8, True), (5000, 2, True), (1024, 10, False)])
def test_logxeb_sizes(nb, k, select):
    from paper_2608_13110_amd import logxeb
    z = amps_of(nb, k, 1)
    sel = W.rng_for(421, nb, k).integers(0, 1 << k, size=nb).astype(np.int32)
    d = torch.from_numpy(z).cuda()
    s = torch.from_numpy(sel).cuda() if select else None
    first = logxeb(d, k, 59, select=s).cpu().numpy()
    again = logxeb(d, k, 59, select=s).cpu().numpy()
    assert np.array_equal(first, again)
    p = np.abs(z) ** 2
    p = p[np.arange(nb), sel] if select else p.reshape(-1)
    f, se, lo, hi = oracle.logxeb(p, 59)
    assert first[4] == p.size
    assert abs(first[0] - f) < 1e-9 * max(1.0, abs(f))
    if p.size > 1:
        assert abs(first[1] - se) < 1e-9
        assert abs(first[2] - lo) < 1e-9 and abs(first[3] - hi) < 1e-9


@pytest.mark.parametrize("value,want", [(0.0, -math.inf), (math.inf, math.inf), (math.nan, math.nan)])
@pytest.mark.parametrize("nb", [100, 9000, 20000])
def test_logxeb_special_values(nb, value, want):
    # one zero, infinite or undefined probability decides the estimate
    from paper_2608_13110_amd import logxeb
    z = amps_of(nb, 0, 2)
    z[nb // 2] = value
    got = logxeb(torch.from_numpy(z).cuda(), 0, 59).cpu().numpy()
    assert got[0] == want or (math.isnan(want) and math.isnan(got[0]))
    assert got[1] == 0.0 and got[4] == nb


@pytest.mark.parametrize("nb,k,select", [(20480, 0, False), (20480, 2, True), (20481, 0, False), (20481, 3, True), (5121, 2, False)])
def test_logxeb_where_blocks_take_over(nb, k, select):
    # 20480 components end the single block
    test_logxeb_sizes(nb, k, select)


@pytest.mark.parametrize("value,want", [(0.0, -math.inf), (math.inf, math.inf), (math.nan, math.nan)])
@pytest.mark.parametrize("nb", [20481, 60000])
def test_logxeb_special_values_over_blocks(nb, value, want):
    test_logxeb_special_values(nb, value, want)
