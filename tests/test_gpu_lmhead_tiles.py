"""GPU parity of the LM head for every row tile that the planner can choose
(192 and 320 rows, one and several of them), against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_36546_amd import ops
from tests import parity
from tests.workload import to_np

pytestmark = pytest.mark.gpu

FULL = 257 * 256          # vocabulary tiles for one whole round of 256, and one more


def _case(M, V, Hd, seed, dup=False):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    h = torch.randn(M, Hd, generator=gen, device="cuda")
    h = (h / h.pow(2).mean(1, keepdim=True).sqrt()).to(torch.bfloat16)
    W = (torch.randn(V, Hd, generator=gen, device="cuda") * 0.1).to(torch.bfloat16)
    if dup:
        # equal logits on both sides of the middle of record groups (entries 63 | 64)
        for g in range(0, V // 128, 3):
            W[128 * g + 64] = W[128 * g + 63]
    prop = np.random.default_rng(seed).integers(0, V, size=M)
    return h, W, prop


@pytest.mark.parametrize("M", [129, 192, 250, 257, 320, 321, 384, 500, 600])
@pytest.mark.parametrize("last", [208, 64, 130])
def test_row_tiles(M, last):
    """192 rows (M = 129, 192: four waves; 321, 384 at Hd = 1024: eight waves,
    two tiles), 256 (250; 500: two tiles), 320 (257, 320; 600: two tiles), each with a last
    vocabulary tile that ends inside a half group, at its end, or two entries
    into a group."""
    V, K = FULL + last, 16
    h, W, prop = _case(M, V, 1024 if M in (321, 384) else 128, M + last, dup=True)
    print(f"[lmhead tiles] M={M} V={V}", flush=True)
    g = ops.lmhead_logsoftmax_verify(h, W, torch.from_numpy(prop.astype(np.int32)).cuda(), K)
    rows = np.unique(np.r_[0, 31, 32, 63, 64, 127, 128, M // 2, M - 2, M - 1, np.arange(0, M, 29)])
    rows = rows[rows < M]
    logits = oracle.logits_fp64(to_np(h)[rows], to_np(W))
    ref = oracle.lmhead_logsoftmax(None, None, prop[rows], K, logits=logits)
    parity.check_lmhead(g, ref, logits, K, rows=rows)
    # equal logits rank by index: a duplicate follows its original directly
    gi = to_np(g["topk_idx"]).astype(np.int64)[rows]
    for r in gi:
        for i in np.nonzero((r % 128 == 64) & (r // 128 % 3 == 0) & (r < V - 128))[0]:
            assert i > 0 and r[i - 1] == r[i] - 1, r
    packed = ops.lmhead_pack_w(W)
    t = ops.lmhead_logsoftmax_verify(h, packed, torch.from_numpy(prop.astype(np.int32)).cuda(), K)
    for key in ("lse", "logp_prop", "argmax", "topk_idx", "topk_logp", "entropy"):
        assert torch.equal(g[key], t[key]), key


@pytest.mark.parametrize("M", [128, 192, 256])
def test_turned_sums(M):
    """Hd = 2048: every vocabulary tile starts its sum at another channel, the
    same one for both layouts of W."""
    V, K = FULL + 130, 16
    h, W, prop = _case(M, V, 2048, M)
    p = torch.from_numpy(prop.astype(np.int32)).cuda()
    g = ops.lmhead_logsoftmax_verify(h, W, p, K)
    rows = np.arange(0, M, 13)
    logits = oracle.logits_fp64(to_np(h)[rows], to_np(W))
    parity.check_lmhead(g, oracle.lmhead_logsoftmax(None, None, prop[rows], K, logits=logits), logits, K, rows=rows)
    t = ops.lmhead_logsoftmax_verify(h, ops.lmhead_pack_w(W), p, K)
    for key in ("lse", "logp_prop", "argmax", "topk_idx", "topk_logp", "entropy"):
        assert torch.equal(g[key], t[key]), key


@pytest.mark.parametrize("M", [300, 384])
def test_uniform_logits_join_halves(M):
    """W = 0: every logit ties, within and across the joined half groups."""
    V, K = FULL + 3, 32
    h = torch.ones(M, 64, device="cuda", dtype=torch.bfloat16)
    W = torch.zeros(V, 64, device="cuda", dtype=torch.bfloat16)
    prop = torch.zeros(M, dtype=torch.int32, device="cuda")
    g = ops.lmhead_logsoftmax_verify(h, W, prop, K)
    np.testing.assert_array_equal(to_np(g["topk_idx"]), np.tile(np.arange(K), (M, 1)))
    np.testing.assert_allclose(to_np(g["lse"]), np.log(V), atol=1e-4)
    np.testing.assert_allclose(to_np(g["entropy"]), np.log(V), atol=1e-3)


def test_draws_from_joined_records():
    """The draw reads the quarter sums of the joined halves: each token's
    interval in the fp64 CDF holds u within the draw's stated 1e-5."""
    M, V = 320, FULL + 100
    h, W, prop = _case(M, V, 64, 5)
    h = h * 4
    ws = torch.empty(ops.lmhead_workspace_size(M, 64, V, 8), dtype=torch.uint8, device="cuda")
    ops.lmhead_logsoftmax_verify(h, W, torch.from_numpy(prop.astype(np.int32)).cuda(), 8, workspace=ws)
    u = torch.linspace(0, 0.9999, M, device="cuda")
    tok = to_np(ops.lmhead_sample(h, W, 8, ws, u)).astype(np.int64)
    p = torch.softmax(h.double() @ W.double().t(), 1)
    c = torch.cumsum(p, 1).cpu().numpy()
    for m in range(M):
        lo = c[m, tok[m] - 1] if tok[m] > 0 else 0.0
        assert lo - 1e-5 <= float(u[m]) <= c[m, tok[m]] + 1e-5, m


@pytest.mark.parametrize("M,V,Hd", [
    (1, 130, 64),             # one stage; the second group has two entries
    (8, 66000, 2048),         # one group per workgroup, its sum turned by the group
    (9, 66000, 2048),         # two groups per workgroup
    (33, 65792 + 128, 128),   # two groups per workgroup, the last workgroup with one
    (64, 65792 + 129, 192),   # and with one group and an entry
    (64, 5003, 4096),
    (64, 90000, 1024),        # several rounds: row-major streamed, tiled in 64-row tiles
    (7, 90000, 512),          # several rounds of short rows: 64-row tiles
    (5, 8192, 2048),          # few groups: 64-row tiles, sums turned
    (20, 8193, 2048),         # row-major streamed, tiled in 64-row tiles: the same turn
    (65, 32003, 128),         # two row tiles
    (128, 2048, 2048),
])
def test_few_rows(M, V, Hd):
    h, W, prop = _case(M, V, Hd, M + V, dup=True)
    print(f"[lmhead tiles] M={M} V={V} Hd={Hd}", flush=True)
    K = min(16, V)
    p = torch.from_numpy(prop.astype(np.int32)).cuda()
    g = ops.lmhead_logsoftmax_verify(h, W, p, K)
    logits = oracle.logits_fp64(to_np(h), to_np(W))
    parity.check_lmhead(g, oracle.lmhead_logsoftmax(None, None, prop, K, logits=logits), logits, K)
    t = ops.lmhead_logsoftmax_verify(h, ops.lmhead_pack_w(W), p, K)
    # hidden rows off a 16-byte boundary take the copy and the 64-row tiles: the
    # same order of the sums, so the same bits
    off = torch.empty(h.numel() + 4, dtype=h.dtype, device="cuda")[4:].view(h.shape)
    off.copy_(h)
    o = ops.lmhead_logsoftmax_verify(off, W, p, K)
    for key in ("lse", "logp_prop", "argmax", "topk_idx", "topk_logp", "entropy"):
        assert torch.equal(g[key], t[key]) and torch.equal(g[key], o[key]), key
    parity.check_lmhead(o, oracle.lmhead_logsoftmax(None, None, prop, K, logits=logits), logits, K)


@pytest.mark.parametrize("M,V,Hd", [(1, 130, 64), (33, 4000, 192), (70, 20000, 64)])
def test_fp32_split_and_staged(M, V, Hd):
    """fp32: few tiles split the channels over the waves; V = 20000 with two
    row tiles stages them."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    h = torch.randn(M, Hd, generator=gen, device="cuda")
    W = torch.randn(V, Hd, generator=gen, device="cuda") * 0.1
    prop = np.random.default_rng(V).integers(0, V, size=M)
    g = ops.lmhead_logsoftmax_verify(h, W, torch.from_numpy(prop.astype(np.int32)).cuda(), 16)
    logits = oracle.logits_fp64(to_np(h), to_np(W))
    parity.check_lmhead(g, oracle.lmhead_logsoftmax(None, None, prop, 16, logits=logits), logits, 16)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Hd", [64, 320, 4096])
def test_recomputed_groups(Hd, dtype):
    """Seven of the top 16 in each of two groups: their 128 logits are
    recomputed, at hidden sizes below, between and at multiples of a pass."""
    V, K = 3000, 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(Hd)
    h = torch.randn(3, Hd, generator=gen, device="cuda")
    W = torch.randn(V, Hd, generator=gen, device="cuda") / Hd ** 0.5
    top = [*range(200, 207), *range(2950, 2957)]
    for r, v in enumerate(top):
        W[v] += h.mean(0) * (8 + 0.25 * r) / Hd
    h, W = h.to(dtype), W.to(dtype)
    prop = np.array([0, 203, 2999])
    g = ops.lmhead_logsoftmax_verify(h, W, torch.from_numpy(prop.astype(np.int32)).cuda(), K)
    logits = oracle.logits_fp64(to_np(h), to_np(W))
    per_group = [max(np.bincount(np.argsort(-l)[:K] // 128)) for l in logits]
    assert min(per_group) >= 4, per_group
    parity.check_lmhead(g, oracle.lmhead_logsoftmax(None, None, prop, K, logits=logits), logits, K)
