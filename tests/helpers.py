"""Test-side helpers: widen workloads to fp64 and flatten a request's cache (independent of oracle and HIP path)."""
import numpy as np

from paper_2508_08192_amd import workloads as W


def widen(a):
    """float64 view of a workload array (float32 values or bf16 bit patterns)."""
    if a.dtype == np.uint16:
        return W.bf16_bits_to_f32(a).astype(np.float64)
    return a.astype(np.float64)


def logical_kv(w, b, n=None):
    """K and V of request b at logical positions 0..n-1 as fp64 arrays [Hkv, n, D]."""
    n = int(w.seq_lens[b]) + w.T if n is None else n
    ps = w.page_size
    K = np.empty((w.Hkv, n, w.D))
    V = np.empty((w.Hkv, n, w.D))
    for pos in range(n):
        if w.page_table is None:
            page, slot = b, pos
        else:
            page, slot = int(w.page_table[b, pos // ps]), pos % ps
        K[:, pos, :] = widen(w.k_cache[page, :, slot, :])
        V[:, pos, :] = widen(w.v_cache[page, :, slot, :])
    return K, V


def ancestors_inclusive(parent, i):
    out = []
    cur = int(i)
    while cur >= 0:
        out.append(cur)
        cur = int(parent[cur])
    return out[::-1]


def run_oracle(w, **kw):
    import oracle
    if w.kv_start is not None:
        kw.setdefault("kv_start", w.kv_start)
    return oracle.tree_attn_oracle(w.q, w.k_cache, w.v_cache, w.page_table, w.seq_lens, w.tree_parent,
                                   scale=w.scale, **kw)


# ----------------------------------------------------------------------------- GPU side

def to_device(w, device="cuda:0"):
    """Upload a workload: returns a dict of torch tensors holding exactly the workload's bits."""
    import torch

    def up(a):
        if a is None:
            return None
        if a.dtype == np.uint16:
            return torch.from_numpy(a.view(np.int16)).to(device).view(torch.bfloat16)
        return torch.from_numpy(a).to(device)

    d = dict(q=up(w.q), k_cache=up(w.k_cache), v_cache=up(w.v_cache), page_table=up(w.page_table),
             seq_lens=up(w.seq_lens), tree_parent=up(w.tree_parent))
    d["out"] = torch.empty_like(d["q"])
    d["lse"] = torch.empty((w.B, w.Hq, w.T), dtype=torch.float32, device=device)
    return d


def run_hip(w, dev=None, **opts):
    """One call through the C-ABI; returns (out, lse) as fp64 numpy arrays."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    d = to_device(w) if dev is None else dev
    d["out"].fill_(float("nan"))
    d["lse"].fill_(float("nan"))
    args = (d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"])
    if w.kv_start is not None and "kv_start" not in opts:
        opts = dict(opts, kv_start=torch.from_numpy(w.kv_start).cuda())
    if opts or w.scale != float(1.0 / np.sqrt(w.D)):
        ta.tree_attn_fwd_ex(*args, scale=w.scale, **opts)
    else:
        ta.tree_attn_fwd(*args)
    torch.cuda.synchronize()
    return d["out"].float().cpu().numpy().astype(np.float64), d["lse"].cpu().numpy().astype(np.float64)


# Tolerances of the parity bar.  bf16 inputs with fp32 accumulation: max-abs <= 1e-2 and mean-abs <= 1e-3;
# fp32: <= 1e-5.  Outputs shrink like 1/sqrt(L) for long prefixes, so a relative gate rides along:
# max-abs error <= 2e-2 of the largest oracle magnitude (bf16) / 1e-4 (fp32).
def assert_parity(got, got_lse, ref, ref_lse, dtype, what=""):
    err = np.abs(got - ref)
    assert np.isfinite(got).all(), what + ": non-finite output"
    scale = np.abs(ref).max()
    if dtype == "f32":
        assert err.max() <= 1e-5, "%s: max-abs %.3g" % (what, err.max())
        assert err.max() <= 1e-4 * scale + 1e-30, "%s: relative %.3g" % (what, err.max() / scale)
        assert np.abs(got_lse - ref_lse).max() <= 1e-5, "%s: lse %.3g" % (what, np.abs(got_lse - ref_lse).max())
    else:
        assert err.max() <= 1e-2, "%s: max-abs %.3g" % (what, err.max())
        assert err.mean() <= 1e-3, "%s: mean-abs %.3g" % (what, err.mean())
        assert err.max() <= 2e-2 * scale + 1e-30, "%s: relative %.3g" % (what, err.max() / scale)
        assert np.abs(got_lse - ref_lse).max() <= 1e-3, "%s: lse %.3g" % (what, np.abs(got_lse - ref_lse).max())


def with_decoy_pages(dev):
    """The caches as views of larger allocations of NaN: page ids just past them lie in memory this process owns."""
    import torch
    for key in ("k_cache", "v_cache"):
        t = dev[key]
        full = torch.full((t.shape[0] + 4,) + tuple(t.shape[1:]), float("nan"), dtype=t.dtype, device="cuda")
        full[:t.shape[0]] = t
        dev[key] = full[:t.shape[0]]
    return dev


def check_requests_with_mistakes(dtype, D, folded, kernel=0, lens=(300, 90, 61, 40, 128, 33), copies=1, alone=None):
    """A page id outside the cache in a prefix and under the tree tokens (also where their rows come from k_new and the page
    only receives them), a bad length, a cyclic tree given as parents and as masks: NaN rows, the status bit, nothing written
    for the tokens whose page does not exist, and every other request as it was.  The mistakes are in the first six requests of
    `copies` times six; `alone`: whether the lists of the plain call are walked alone (None: not asked)."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    B, T, Hq, Hkv, ps = 6 * copies, 19, 4, 2, 16
    lens = list(lens) * copies
    assert lens[0] > 112 and lens[1] % ps != 0 and (lens[2] + T - 1) // ps > lens[2] // ps and lens[4] % ps == 0
    trees = np.stack([W.bfs_tree(T, [3], 5)] * B)
    w = W.make_workload("mistakes", B=B, T=T, Hq=Hq, Hkv=Hkv, D=D, seq_lens=lens, trees=trees, page_size=ps, seed=91, dtype=dtype)
    n_pages = w.k_cache.shape[0]
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    tol, lse_tol = (1e-5, 1e-5) if dtype == "f32" else (1e-2, 1e-3)        # as assert_parity: the schedule may differ
    k_new, v_new = (torch.randn(B, T, Hkv, D, generator=torch.Generator().manual_seed(s)).to(dt).cuda() for s in (1, 2))

    def call(table, seq, tree, **kw):
        d = with_decoy_pages(to_device(w))
        d["page_table"], d["seq_lens"], d["tree_parent"] = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (table, seq, tree))
        if folded:
            kw = dict(kw, k_new=k_new, v_new=v_new)
        out, lse = torch.zeros_like(d["q"]), torch.zeros_like(d["lse"])
        own = torch.zeros(1, dtype=torch.int32, device="cuda")
        ta.tree_attn_last_status()
        ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], out, lse,
                            status=own, kernel=kernel, **kw)
        bits = ta.tree_attn_last_status()
        assert bits == int(own.item())
        return out, lse, d["k_cache"], d["v_cache"], bits

    if alone is not None:
        d = to_device(w)
        plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                                 d["lse"], kernel=kernel)
        assert (plan["merge_workgroups"] == 0) == alone, plan
    good = call(w.page_table, w.seq_lens, trees)
    assert good[4] == 0 and torch.isfinite(good[0]).all()
    tree_page = w.page_table.copy()
    tree_page[1, lens[1] // ps] = n_pages                       # holds the last prefix tokens and the first of the tree
    tree_page[2, (lens[2] + T - 1) // ps] = n_pages + 3         # holds the last tokens of the tree alone
    tree_page[4, lens[4] // ps] = -1                            # the prefix ends on a page: the tree's alone
    prefix = w.page_table.copy()
    prefix[0, 7] = n_pages
    bad_len = w.seq_lens.copy()
    bad_len[3] = -1
    bad_len[5] = w.page_table.shape[1] * ps
    cyc = trees.copy()
    cyc[2, 1], cyc[2, 2] = 2, 1
    masks = torch.zeros((B, T), dtype=torch.int64, device="cuda")
    ta.tree_attn_encode(torch.from_numpy(cyc).cuda(), masks)
    for what, table, seq, tree, kw, hit, bit in (
            ("page of the tree", tree_page, w.seq_lens, trees, {}, [1, 2, 4], ta.TA_STATUS_BAD_PAGE),
            ("page of the prefix", prefix, w.seq_lens, trees, {}, [0], ta.TA_STATUS_BAD_PAGE),
            ("length", w.page_table, bad_len, trees, {}, [3, 5], ta.TA_STATUS_BAD_SEQLEN),
            ("parents", w.page_table, w.seq_lens, cyc, {}, [2], ta.TA_STATUS_BAD_PARENT),
            ("masks", w.page_table, w.seq_lens, trees, {"tree_masks": masks}, [2], ta.TA_STATUS_BAD_PARENT)):
        for splits in (0, 1):
            print("mistakes %s D=%d folded=%s kernel=%d splits=%d: %s" % (dtype, D, folded, kernel, splits, what), flush=True)
            out, lse, k, v, bits = call(table, seq, tree, num_splits=splits, **kw)
            assert bits == bit, (what, bits)
            for b in hit:
                assert torch.isnan(out[b]).all() and torch.isnan(lse[b]).all(), (what, b)
            rest = [b for b in range(B) if b not in hit]
            assert (out[rest].float() - good[0][rest].float()).abs().max() <= tol, what
            assert (lse[rest] - good[1][rest]).abs().max() <= lse_tol, what
            if what == "page of the tree" and folded:
                rows = (k != to_device(w)["k_cache"]).any(dim=3).any(dim=1).sum().item()
                # (6 of request 1's tokens lie on its bad page, 16 of request 2's, 16 of request 4's)
                lost = sum(int(table[b, (lens[b] + i) // ps] not in range(n_pages)) for b in range(B) for i in range(T))
                assert lost > 0 and rows == B * T - lost
