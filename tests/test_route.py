"""The sizes at which a backward call changes its route (embc_route.h)."""
import pytest

from route import route


def cfg(T, dim, batch=1024):
    return {"rows": [1000] * T, "dim": dim, "batch": batch}


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


def test_calls_without_bags_or_lookups():
    assert route(cfg(3, 16), 0) == "small" and route(cfg(3, 16), 0, batch=0) == "small"
    assert route(cfg(3, 16), 100_000, batch=0) == "general" and route(cfg(600, 16), 0) == "general"
