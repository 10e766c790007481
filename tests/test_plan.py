"""The attention planner's routes at the lines of its rule, asked of the built
library (no GPU): which kernel a bf16 D = 128 call takes."""
import pytest

from tests.plan import attn_kernel, attn_plan


@pytest.mark.parametrize("args,kernel", [
    # n_seq, Hq, Hkv, D, max_q, max_pages, page_size
    ((64, 32, 4, 128, 8, 513, 16), "stream-k"),      # verification windows, contexts to 8192
    ((64, 32, 4, 128, 8, 64, 16), "tiles"),          # contexts to 1000
    ((8, 32, 4, 128, 1024, 64, 16), "tiles"),        # prompts
    ((1, 16, 8, 128, 1, 94, 16), "stream-k"),        # one row
    ((300, 32, 4, 128, 1, 2048, 16), "register"),    # more sequences than the stream-K tables hold
    ((32, 16, 8, 128, 5, 65, 64), "stream-k"),       # 64-slot pages
    # larger pages: too few partials fit for every item or compute unit to get a workgroup
    ((24, 16, 8, 128, 3, 30, 32), "register"),
    ((20, 64, 8, 128, 3, 28, 32), "register"),
    ((4, 16, 8, 128, 1, 81, 32), "register"),        # few rows, 158 workgroups
    ((4, 16, 8, 128, 1, 137, 32), "stream-k"),       # 254
    ((32, 32, 4, 128, 5, 24, 64), "stream-k"),       # 254 workgroups for 128 items
])
def test_routes(args, kernel):
    assert attn_kernel(attn_plan(*args)) == kernel


@pytest.mark.parametrize("args", [
    (16, 32, 4, 128, 512, 2048, 16),      # a prompt chunk among one-row windows to 32K tokens
    (4, 32, 4, 128, 1024, 320, 16),       # a generous max_q
    (2, 32, 4, 128, 2048, 1024, 16),
])
def test_long_walks_are_cut(args):
    p = attn_plan(*args)
    assert attn_kernel(p) == "tiles" and p.tile_split and p.tile_walk <= 48
    blocks = -(-args[5] * args[6] // 32)
    tiles = -(-args[4] * args[1] // args[2] // 128)
    assert p.tile_units >= max(tiles, blocks // 16)
