"""Host-side: the framed list build reads whole rounds of a tile's plan, also
past the segments it holds; the memory of the plans covers them for the last
tile whatever lies behind it in the workspace."""
import ctypes as C

import pytest

HEAD = 80 + 16 * 64  # header and row positions of a plan, 16 bytes a segment after them


@pytest.fixture(scope="module")
def plan_bytes():
    from paper_1412_3387_amd import binding, build
    if build.needs_build():
        build.build()
    f = binding.lib()._ZN2md16build_plan_bytesElib  # md::build_plan_bytes(int64, int, bool)
    f.argtypes, f.restype = [C.c_int64, C.c_int, C.c_bool], C.c_size_t
    return f


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("seg_cap", [256, 300, 450, 600, 1050, 2040])
def test_plans_cover_the_read_ahead(plan_bytes, threads, seg_cap):
    """A round is one segment per eight lanes; a tile of nseg segments reads
    five rounds from every round that holds one of them."""
    per_round = threads // 8
    last = 0
    for nseg in range(seg_cap + 1):
        rounds = -(-nseg // per_round)
        last = max(last, (max(rounds, 1) - 1 + 5) * per_round - 1)
    for tiles in (1, 7):
        assert plan_bytes(tiles, seg_cap, False) >= (tiles - 1) * (HEAD + 16 * seg_cap) + HEAD + 16 * (last + 1)
