"""The tables of every route that complex64 calls take in place of the plan's own
passes and late phase (one launch, latency passes, tiles by size, late removals
folded into the join), run on the host: the same FP32 updates in the same order,
so the same amplitudes bit for bit, and with the fold up to the FP64 rounding of
the late phase."""
import numpy as np
import pytest

import workloads as W
from paper_2608_13110_amd import (ROUTE_FOLDED, ROUTE_LATENCY, ROUTE_ONE, ROUTE_OWN, ROUTE_SIZED, TNC_E_DOMAIN, Plan,
                                  TncError)
from tests import helpers as H


def case(n, d, k, parity, nb=2, options=None):
    c = H.mixed_circuit(n, d, 11 * d + parity, first_parity=parity, dense=0.3)
    return Plan.from_circuit(c, options), W.random_bitstrings(n, nb, W.rng_for(499, d, parity))


def takes(plan, bits, k, route):
    try:
        return plan.debug_emulate_route(bits, k, route)
    except TncError as e:
        assert e.code == TNC_E_DOMAIN
        return None


@pytest.mark.parametrize("parity", [0, 1])
@pytest.mark.parametrize("d", list(range(2, 41)))
def test_routes_equal_the_own_passes(d, parity):
    n, nb = (7, 2) if d <= 26 else (4, 1)
    for k in sorted({0, min(1 + parity, d // 4)}):
        plan, bits = case(n, d, k, parity, nb)
        h = plan.info(k)["boundary_bits"]
        own = plan.debug_emulate_route(bits, k, ROUTE_OWN)
        assert np.array_equal(own, plan.debug_emulate_device(bits, k))
        got = {r: takes(plan, bits, k, r) for r in (ROUTE_SIZED, ROUTE_LATENCY, ROUTE_ONE)}
        # which sizes take which
        assert (got[ROUTE_ONE] is not None) == (h <= 12)
        assert (got[ROUTE_SIZED] is not None) == (h > 12)
        if h <= 12 or h > 20:
            assert got[ROUTE_LATENCY] is None
        for r, z in got.items():
            assert z is None or np.array_equal(z, own), (h, k, r)


def test_every_latency_size_is_taken():
    sizes = set()
    for d in range(25, 41):
        plan, bits = case(3, d, 0, 1, nb=1)
        if takes(plan, bits, 0, ROUTE_LATENCY) is not None:
            sizes.add(plan.info(0)["boundary_bits"])
    assert sizes == set(range(13, 21))


@pytest.mark.parametrize("n,d,k,options", [(9, 20, 4, dict(max_tile_bits=6, low_bits=2, reg_bits=3)),
                                           (9, 24, 0, dict(max_tile_bits=8)), (9, 18, 2, dict(reg_bits=1, max_tile_bits=9))])
def test_one_launch_equals_named_tiles(n, d, k, options):
    plan, bits = case(n, d, k, 1, options=options)
    assert np.array_equal(plan.debug_emulate_route(bits, k, ROUTE_ONE), plan.debug_emulate_route(bits, k, ROUTE_OWN))


@pytest.mark.parametrize("options", [dict(math=2, reg_bits=4), dict(max_tile_bits=12, low_bits=3)])
def test_plans_with_tile_options_keep_their_passes(options):
    plan, bits = case(7, 30, 2, 1, nb=1, options=options)
    for r in (ROUTE_SIZED, ROUTE_LATENCY, ROUTE_ONE):
        assert takes(plan, bits, 2, r) is None


@pytest.mark.parametrize("d,k", [(28, 1), (30, 3), (34, 5), (36, 8), (33, 4)])
def test_folded_join(d, k):
    # FP64 on both sides, 2^k state entries through at most d layers: 1e-13
    plan, bits = case(9, d, k, 1, nb=1)
    own = plan.debug_emulate_route(bits, k, ROUTE_OWN)
    got = plan.debug_emulate_route(bits, k, ROUTE_FOLDED)
    assert np.abs(got - own).max() <= 1e-13 * np.abs(own).max()


def test_unknown_routes_are_refused():
    plan, bits = case(7, 12, 1, 1)
    for r in (-1, 5):
        assert takes(plan, bits, 1, r) is None
