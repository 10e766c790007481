"""The attention planner's choice (kernels.h: AttnPlan), asked of the library."""
import ctypes

from paper_2609_36546_amd import ops


class AttnPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in (
        "n_qg", "qt", "sub", "chunk", "max_chunks", "tile", "tile_units", "tile_split", "tile_walk", "max_mask",
        "sk", "sk_grid", "sk_qt", "sk_n_qg")] + [(n, ctypes.c_size_t) for n in (
            "part_o_bytes", "part_lse_bytes", "workspace_bytes", "sk_o_bytes", "sk_lse_bytes")]


def attn_plan(n_seq, Hq, Hkv, D, max_q, max_pages, page_size):
    f = getattr(ops.lib(), "_ZN4ipdv9attn_planEiiiiiii")   # ipdv::attn_plan(int x 7)
    f.argtypes, f.restype = [ctypes.c_int] * 7, AttnPlan
    p = f(n_seq, Hq, Hkv, D, max_q, max_pages, page_size)
    assert p.workspace_bytes == ops.attn_workspace_size(n_seq, Hq, Hkv, D, max_q, max_pages, page_size)
    return p


def attn_kernel(p):
    """The kernel that a bf16 call with D = 128 and 16-byte aligned arrays takes."""
    return "tiles" if p.tile else "stream-k" if p.sk else "register"


def plan_of(batch, mdl, max_q=None, page_table=None):
    s, pt = mdl.shape, mdl.page_table if page_table is None else page_table
    k = int((batch.cu_q[1:] - batch.cu_q[:-1]).max()) if max_q is None else max_q
    return attn_plan(mdl.seq_ids.shape[0], s.Hq, s.Hkv, s.D, max(k, 1), pt.shape[1], batch.cfg.page_size)
