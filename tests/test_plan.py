"""Host checks of the rules that pick the kernels of a call and size its workspace (csrc/plan.h)."""
import random

import pytest

from paper_2011_09208_amd import buildlib
from tests import plan_rules


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return plan_rules.load(str(tmp_path_factory.mktemp("plan")))


@pytest.fixture(scope="module")
def ws():
    if buildlib.is_stale():
        buildlib.build()
    from paper_2011_09208_amd import binding
    return binding


def drawn(n, seed, max_b=70000, max_d=4096, max_c=150000):
    """Sizes spread over their logarithms, every other batch and width at or beside the edge of a tile."""
    rng = random.Random(seed)
    for _ in range(n):
        B, C = (int(m ** rng.random()) for m in (max_b, max_c))
        D = 64 * int((max_d // 64) ** rng.random())
        if rng.random() < 0.5:
            B = max(1, (B + 32) // 64 * 64 + rng.choice((-1, 0, 1)))
        if rng.random() < 0.5:
            C = max(1, (C + 32) // 64 * 64 + rng.choice((-1, 0, 1)))
        yield B, D, C


def test_the_rules_tested_here_are_the_librarys(rules, ws):
    for B, D, C in drawn(2000, seed=1):
        assert rules.fwd_bytes_(B, D, C) == ws.fwd_workspace_bytes(B, D, C), (B, D, C)
        assert rules.bwd_bytes_(B, D, C) == ws.bwd_workspace_bytes(B, D, C), (B, D, C)
