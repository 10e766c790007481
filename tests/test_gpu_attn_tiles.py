"""GPU parity of verify_attn_paged on its tiles (long windows and short
contexts) and of the window append, against the fp64 oracle, and of the
stream-K split on batches of the same lengths when the page table is wide."""
import numpy as np
import pytest
import torch

from paper_2609_36546_amd import inputs, ops
from tests import parity, plan
from tests.workload import to_np

pytestmark = pytest.mark.gpu


def _batch(Hq, Hkv, ks, lo, hi, ps, seed, B=4, D=128, dtype="bf16"):
    shape = inputs.ModelShape("heads", Hq=Hq, Hkv=Hkv, D=D, hidden=64, vocab=512)
    cfg = inputs.scaled(inputs.WORKLOADS["teacher-bf16"], B=B, ctx_lo=lo, ctx_hi=hi, k_choices=ks,
                        page_size=ps, models=(shape,), dtype=dtype)
    print(f"[tiles] heads {Hq}/{Hkv} D={D} B={B} ctx=[{lo},{hi}] k={ks} ps={ps} seed={seed}", flush=True)
    return inputs.make_batch(cfg, seed=seed, device="cuda")


def _check(b, **kw):
    mdl = b.models[0]
    out, kc, vc = parity.run_gpu_attention(mdl, b, seq_ids=mdl.seq_ids, **kw)
    ref, rkc, rvc = parity.oracle_attention(mdl, b, to_np(mdl.seq_ids).astype(np.int64), mdl.shape.D)
    parity.check_attention_rows(out, ref, to_np(mdl.rows).astype(np.int64), mdl.q.dtype)
    np.testing.assert_array_equal(to_np(kc), rkc.astype(np.float32))
    np.testing.assert_array_equal(to_np(vc), rvc.astype(np.float32))


def _wide(mdl, pages):
    """The page table with more columns than any sequence needs (poison pages)."""
    pt = mdl.page_table
    pad = torch.full((pt.shape[0], pages), mdl.poison_page, dtype=pt.dtype, device=pt.device)
    return torch.cat([pt, pad], 1).contiguous()


@pytest.mark.parametrize("ps", [16, 32, 64])
@pytest.mark.parametrize("Hq,Hkv,ks,lo,hi", [
    (32, 4, (1, 37, 130), 0, 0),        # prompts: up to nine 128-row tiles, the last partly filled
    (16, 8, (1, 5, 31, 0), 0, 90),      # one 64-row tile, empty windows among them
    (16, 8, (33, 64), 17, 200),         # two query heads per KV head: exactly one 128-row tile, and one row over 64
    (4, 4, (1, 16, 65), 30, 33),        # one query head per KV head, contexts around one key block
])
def test_tiles(Hq, Hkv, ks, lo, hi, ps):
    b = _batch(Hq, Hkv, ks, lo, hi, ps, seed=50 + ps)
    assert plan.attn_kernel(plan.plan_of(b, b.models[0])) == "tiles"
    _check(b)


@pytest.mark.parametrize("ps", [16, 64])
@pytest.mark.parametrize("Hq,Hkv,ks,lo,hi,B,max_q,keys", [
    (32, 4, (1, 70, 0, 130), 1500, 2600, 4, 1500, 0),    # pieces of 16 blocks, of 80 and of 144 beside each other
    (32, 4, (1, 5, 9), 1400, 3300, 16, 512, 32768),      # one-tile windows in longer pieces, past the stream-K tables
    (16, 8, (1, 33, 64), 1530, 1600, 3, 900, 0),         # around the blocks that a tile walks whole
    (8, 8, (65, 128, 129), 1500, 2100, 5, 1200, 0),      # one query head: half-filled tiles and groups
])
def test_tiles_cut_by_keys(Hq, Hkv, ks, lo, hi, B, max_q, keys, ps):
    """Windows with long contexts under bounds that make the planner take the
    tiles: their keys are cut into pieces and merged."""
    b = _batch(Hq, Hkv, ks, lo, hi, ps, seed=65, B=B)
    pt = _wide(b.models[0], keys // ps) if keys else None
    p = plan.plan_of(b, b.models[0], max_q, pt)
    assert plan.attn_kernel(p) == "tiles" and p.tile_split
    _check(b, max_q=max_q, **({"page_table": pt} if keys else {}))


def test_tiles_over_two_batches_of_page_ids():
    """A prompt chunk whose tiles walk more than 256 key blocks: the page ids
    are read in two batches."""
    b = _batch(8, 4, (1, 1100), 7650, 7750, 16, seed=61, B=2)
    assert plan.attn_kernel(plan.plan_of(b, b.models[0], 8000)) == "tiles"
    _check(b, max_q=8000)


def test_generous_bounds_cost_little():
    """Sixteen one-row windows with contexts to 32K tokens: a max_q of 512
    takes the tiles, whose walks of such contexts are cut; uncut they took five
    times the call with the tight bound (now 1.25)."""
    b = _batch(32, 4, (1,), 16000, 32700, 16, seed=66, B=16)
    mdl, dev = b.models[0], b.models[0].q.device
    ctx, cu = torch.from_numpy(b.ctx_lens).to(dev), torch.from_numpy(b.cu_q).to(dev)
    assert plan.attn_kernel(plan.plan_of(b, mdl, 512)) == "tiles"
    us = {}
    for max_q in (1, 512):
        ws = torch.empty(ops.attn_workspace_size(16, 32, 4, 128, max_q, mdl.page_table.shape[1], 16),
                         dtype=torch.uint8, device=dev)
        times = []
        for _ in range(12):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            ops.verify_attn_paged(mdl.q, mdl.k_new, mdl.v_new, mdl.k_pool, mdl.v_pool, mdl.page_table, ctx, cu,
                                  max_q=max_q, workspace=ws)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1) * 1e3)
        us[max_q] = sorted(times)[len(times) // 2]
    print(f"[tiles] max_q 1: {us[1]:.0f} us, 512: {us[512]:.0f} us", flush=True)
    assert us[512] < 2 * us[1]


@pytest.mark.parametrize("D,dtype,ps", [(64, "bf16", 16), (64, "bf16", 64), (64, "f32", 32)])
def test_append_of_few_rows(D, dtype, ps):
    """Windows of up to four rows go straight to the pages, over page ends
    too; five rows go through LDS."""
    _check(_batch(4, 2, (1, 3, 4, 5, 0), 5, 150, ps, seed=67, B=40, D=D, dtype=dtype))


@pytest.mark.parametrize("D,dtype,ps", [(64, "bf16", 32), (64, "f32", 16)])
def test_append_of_long_windows(D, dtype, ps):
    """Windows over several 64-position chunks of the append, starting and
    ending inside a run of slots."""
    _check(_batch(4, 2, (3, 64, 131), 5, 150, ps, seed=62, D=D, dtype=dtype))


def test_append_of_arrays_off_a_16_byte_boundary():
    """Caches that start 8 bytes off a 16-byte boundary take the register
    kernel and the append's element-wise path."""
    b = _batch(8, 4, (1, 7, 40), 5, 150, 32, seed=63)
    mdl = b.models[0]

    def moved(x):
        buf = torch.empty(x.numel() + 4, dtype=x.dtype, device=x.device)
        y = buf[4:].view(x.shape)
        y.copy_(x)
        assert y.data_ptr() % 16 == 8
        return y

    kc, vc = moved(mdl.k_pool), moved(mdl.v_pool)
    dev = mdl.q.device
    out = ops.verify_attn_paged(mdl.q, mdl.k_new, mdl.v_new, kc, vc, mdl.page_table,
                                torch.from_numpy(b.ctx_lens).to(dev), torch.from_numpy(b.cu_q).to(dev), max_q=40)
    ref, rkc, rvc = parity.oracle_attention(mdl, b, to_np(mdl.seq_ids).astype(np.int64), 128)
    parity.check_attention_rows(out, ref, to_np(mdl.rows).astype(np.int64), mdl.q.dtype)
    np.testing.assert_array_equal(to_np(kc), rkc.astype(np.float32))
    np.testing.assert_array_equal(to_np(vc), rvc.astype(np.float32))


@pytest.mark.parametrize("ps", [16, 32, 64])
@pytest.mark.parametrize("Hq,Hkv,ks,lo,hi,B,keys", [
    (32, 4, (0, 1, 8, 16), 0, 300, 12, 32768),   # items without rows between others
    (32, 4, (0, 4, 16), 0, 40, 60, 32768),       # fewer key blocks than workgroups
    (32, 2, (16, 5, 0), 0, 700, 5, 32768),       # two 128-row items over the same keys
    (16, 8, (1, 8), 480, 540, 64, 32768),        # the whole grid, about sixteen blocks to a share
    (16, 8, (1,), 0, 60, 1, 32768),              # a single short sequence
    (16, 8, (1, 5), 900, 2500, 4, 2100),         # larger pages: about half the grid's partials fit the workspace
])
def test_stream_k_with_a_wide_page_table(Hq, Hkv, ks, lo, hi, B, keys, ps):
    """Short contexts under a page table sized for long ones: the planner goes
    by the table's width, so these batches take the stream-K split."""
    b = _batch(Hq, Hkv, ks, lo, hi, ps, seed=64, B=B)
    pt = _wide(b.models[0], keys // ps)
    assert plan.attn_kernel(plan.plan_of(b, b.models[0], None, pt)) == "stream-k"
    _check(b, page_table=pt)


def _block_rounded(q, K, V, limits, scale):
    """Attention rows in 64 bits but for the probabilities, rounded to bf16
    against the maximum of their 32-key block, and the outputs, to bf16; and
    the rows unrounded.  q [R, D], K / V [N, D], limits [R] visible keys."""
    s = (q @ K.t()) * scale / np.log(2.0)
    s = s.masked_fill(torch.arange(K.shape[0])[None, :] >= limits[:, None], -torch.inf)
    exact = torch.softmax(s * np.log(2.0), 1) @ V
    pad = -s.shape[1] % 32
    b = torch.nn.functional.pad(s, (0, pad), value=-torch.inf).view(len(q), -1, 32)
    m = b.amax(2, keepdim=True)
    p = torch.where(torch.isinf(b), torch.zeros_like(b), torch.exp2(b - m))
    w = torch.exp2(m - m.amax(1, keepdim=True))
    low = (p.to(torch.bfloat16).double() * w).flatten(1)[:, : s.shape[1]]
    return (low @ V / (p * w).sum((1, 2))[:, None]).to(torch.bfloat16).double(), exact


@pytest.mark.parametrize("Hq,Hkv,ks,lo,hi,ps,B,kernel", [
    (16, 8, (1,), 1500, 1500, 16, 1, "stream-k"),      # fewer workgroups than the grid: four blocks each
    (32, 4, (8,), 700, 2900, 16, 2, "stream-k"),       # the same, three to five blocks each
    (32, 4, (5,), 1500, 2500, 64, 12, "stream-k"),     # 64-slot pages
    (32, 4, (8,), 700, 900, 16, 3, "stream-k"),
    (32, 4, (8,), 150, 300, 16, 3, "tiles"),           # few windows, short contexts
    (16, 8, (200,), 0, 0, 16, 1, "tiles"),             # a short prompt
])
def test_rounding_of_probabilities(Hq, Hkv, ks, lo, hi, ps, B, kernel):
    """Calls of few key blocks round each block's probabilities against the
    block's own maximum: the error against 64 bits is that of a model of this
    rounding (2% apart at most: the hardware's exp2 and fp32 scores turn a few
    roundings over), where one maximum for a whole piece or row gives 5 to 15%
    more."""
    b = _batch(Hq, Hkv, ks, lo, hi, ps, seed=70 + B, B=B)
    mdl = b.models[0]
    assert plan.attn_kernel(plan.plan_of(b, mdl)) == kernel
    out, kc, vc = parity.run_gpu_attention(mdl, b, seq_ids=mdl.seq_ids)
    G, D = Hq // Hkv, 128
    table = mdl.page_table.cpu().long()
    kc, vc, q, out = kc.cpu(), vc.cpu(), mdl.q.cpu(), out.cpu().double()
    got = want = 0.0
    for i in range(B):
        L, r0, r1 = int(b.ctx_lens[i]), int(b.cu_q[i]), int(b.cu_q[i + 1])
        pos = torch.arange(L + r1 - r0)
        K = kc[table[i, pos // ps], :, :, pos % ps].reshape(len(pos), Hkv, D).double()
        V = vc[table[i, pos // ps], :, :, pos % ps].double()
        limits = L + 1 + torch.arange(r1 - r0)
        for h in range(Hq):
            low, exact = _block_rounded(q[r0:r1, h].double(), K[:, h // G], V[:, h // G], limits, D ** -0.5)
            got += float(((out[r0:r1, h] - exact) ** 2).sum())
            want += float(((low - exact) ** 2).sum())
    print(f"[rounding] error against the model's: {(got / want) ** 0.5:.4f}", flush=True)
    assert (got / want) ** 0.5 < 1.02


@pytest.mark.parametrize("Hq,Hkv,k", [(32, 4, 8), (32, 4, 16), (16, 8, 1)])   # 64- and 128-row items
@pytest.mark.parametrize("blocks", [1, 7, 8, 19, 20, 39, 40, 63, 64, 149, 150, 152, 153])
def test_stream_k_shares_of_few_blocks(blocks, Hq, Hkv, k):
    """One sequence of the given key blocks per item: on both sides of every
    change of the blocks per workgroup, and shares of exactly eight blocks,
    which keep equal spans below the full grid."""
    L = max(0, 32 * blocks - k)
    b = _batch(Hq, Hkv, (k,), L, L, 16, seed=68, B=1)
    pt = _wide(b.models[0], 1024)
    assert plan.attn_kernel(plan.plan_of(b, b.models[0], None, pt)) == "stream-k"
    _check(b, page_table=pt)
