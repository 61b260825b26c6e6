"""The sizes at which a backward call changes its route (embc_route.h)."""
import pytest

from route import route


def cfg(T, dim, batch=1024, **kw):
    return {"rows": [1000] * T, "dim": dim, "batch": batch, **kw}


@pytest.mark.parametrize("T,dim,lookups,want", [
    (1, 16, 1, "small"), (1, 256, 8192, "small"), (1, 16, 8193, "mid"), (513, 16, 8192, "general"),
    (513, 16, 1 << 20, "general"),
    # below 2M lookups, whatever the width
    (1, 256, (1 << 21) - 1, "mid"), (1, 16, 1 << 21, "general"),
    # past 2M: at most 2^18 lookups per table, and few columns in all or per table
    (8, 16, 1 << 21, "mid"), (8, 16, (1 << 21) + 1, "general"), (512, 16, (1 << 23) - 1, "mid"), (512, 16, 1 << 23, "general"),
    (24, 64, 6_291_456, "mid"), (24, 64, 6_291_457, "general"), (60, 64, 60 << 17, "mid"), (60, 64, (60 << 17) + 1, "general"),
    (100, 128, 100 << 16, "mid"), (100, 128, (100 << 16) + 1, "general"), (128, 256, 128 << 15, "mid"),
    (128, 256, (128 << 15) + 1, "general"), (32, 256, 3_200_000, "general"), (10, 128, 2_600_000, "mid"),
])
def test_route_by_size(T, dim, lookups, want):
    assert route(cfg(T, dim), lookups) == want


@pytest.mark.parametrize("T,batch,lookups,want", [
    # past 8192 lookups a table may hold more than its workgroup's LDS
    (2, 50, 16_384, "small"), (2, 50, 16_385, "mid"), (8, 100, 21_440, "small"), (8, 100, 21_441, "mid"),
    (100, 50, 32_480, "small"), (100, 50, 32_481, "mid"), (512, 50, 65_536, "small"), (512, 50, 65_537, "mid"),
    # but not where all bags have one length
    (26, 2048, 26 * 2048, "small"), (26, 2048, 26 * 2048 + 1, "mid"), (26, 2048, 26 * 2048 - 1, "mid"),
    (16, 100, 16 * 100 * 20, "small"), (8, 128, 65_536, "small"), (8, 8, 64_000, "small"), (9, 7, 63_000, "mid"),
    (26, 2521, 26 * 2521, "mid"),
    (1, 8192, 8192, "small"), (8, 70_000, 100, "mid"),
])
def test_small_calls(T, batch, lookups, want):
    assert route(cfg(T, 16, batch), lookups) == want


@pytest.mark.parametrize("frac,rows,lookups,want", [
    # one set (16 ways)
    (1e-6, 1024, 12_000, "small"), (1e-6, 1025, 12_000, "mid"), (1e-6, 10**6, 8192, "small"), (1e-6, 10**6, 8193, "mid"),
    (1e-6, 10**6, 8610, "small"),
    # seven sets, eight, many, none
    (0.0157, 7168, 12_000, "small"), (0.0157, 7175, 12_000, "mid"), (0.0157, 8200, 12_000, "small"),
    (0.001, 10**7, 20_000, "small"), (0.0, 10**7, 12_000, "small"),
])
def test_small_calls_by_rows_per_set(frac, rows, lookups, want):
    """Three tables of 410 bags: 8610 lookups are 7 per bag."""
    assert route({"rows": [500, rows, 40], "dim": 16, "batch": 410, "cache_fraction": frac, "assoc": 16}, lookups) == want


def test_calls_without_bags_or_lookups():
    assert route(cfg(3, 16), 0) == "small" and route(cfg(3, 16), 0, batch=0) == "small"
    assert route(cfg(3, 16), 100_000, batch=0) == "general" and route(cfg(600, 16), 0) == "general"
