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
    (2, 64, 12_416, "small"), (2, 64, 12_417, "mid"), (8, 100, 12_800, "small"), (8, 100, 12_801, "mid"),
    (100, 50, 18_688, "small"), (100, 50, 18_689, "mid"), (512, 50, 45_056, "small"), (512, 50, 45_057, "mid"),
    # but not where all bags have one length
    (26, 2048, 26 * 2048, "small"), (26, 2048, 26 * 2048 + 1, "mid"), (26, 2048, 26 * 2048 - 1, "mid"),
    (16, 100, 16 * 100 * 20, "small"), (8, 128, 65_536, "small"), (8, 127, 8 * 127 * 64, "mid"), (26, 2521, 26 * 2521, "mid"),
    (1, 8192, 8192, "small"), (8, 70_000, 100, "mid"),
])
def test_small_calls(T, batch, lookups, want):
    assert route(cfg(T, 16, batch), lookups) == want


@pytest.mark.parametrize("frac,assoc,rows,lookups,want", [
    (1e-6, 16, 1024, 12_000, "small"), (1e-6, 16, 1025, 12_000, "mid"), (1e-6, 16, 10**6, 8192, "small"),
    (0.02, 16, 10**7, 12_000, "small"), (0.01, 16, 10**7, 12_000, "mid"), (0.0, 16, 10**7, 12_000, "small"),
    (0.001, 16, 10**7, 12_000, "mid"), (0.001, 16, 10**7, 12_300, "small"), (1e-6, 16, 10**6, 8400, "small"),
])
def test_small_calls_by_rows_per_set(frac, assoc, rows, lookups, want):
    assert route({"rows": [500, rows, 40], "dim": 16, "batch": 350 if lookups % 1050 == 0 else 410, "cache_fraction": frac, "assoc": assoc}, lookups) == want


def test_calls_without_bags_or_lookups():
    assert route(cfg(3, 16), 0) == "small" and route(cfg(3, 16), 0, batch=0) == "small"
    assert route(cfg(3, 16), 100_000, batch=0) == "general" and route(cfg(600, 16), 0) == "general"
