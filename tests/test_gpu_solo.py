"""Lists of a few tiles, which one workgroup walks alone and whose outputs it writes (no merge pass): around the sizes where
that begins and ends, runs, row blocks and window starts at their edges, the write-back folded in, requests with mistakes,
more workgroups than the device has compute units; against the fp64 oracle and the cut lists."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, check_requests_with_mistakes, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu


def _solo(w, d, **kw):
    from paper_2508_08192_amd import treeattn as ta
    plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                             d["lse"], **kw)
    return plan["merge_workgroups"] == 0


def _check(w, what, solo=True, **kw):
    d = to_device(w)
    assert _solo(w, d) == solo, what
    print(what, flush=True)
    got, lse = run_hip(w, d, **kw)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, w.dtype, what)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("T,Hq,Hkv", [(1, 1, 1), (8, 4, 2), (17, 1, 1), (33, 1, 1), (13, 5, 1), (64, 4, 2)])
@pytest.mark.parametrize("ps", [0, 1, 16, 64])
def test_runs_row_blocks_and_windows(dtype, D, T, Hq, Hkv, ps):
    lens = [0, 1, 15, 16, 31, 33, 63, 64, 65, 127, 128 - T % 64]
    if dtype == "f32" and D == 128:            # up to three tiles
        lens = [min(x, 65) for x in lens]
    rng = np.random.default_rng(D + T)
    trees = np.stack([W.random_tree(T, min(T, 7), rng) for _ in lens])
    w = W.make_workload("solo", B=len(lens), T=T, Hq=Hq, Hkv=Hkv, D=D, seq_lens=lens, trees=trees, page_size=ps, seed=17 + T,
                        paged=ps > 0, dtype=dtype)
    what = "solo %s D=%d T=%d %d/%d ps=%d" % (dtype, D, T, Hq, Hkv, ps)
    _check(w, what)
    w.kv_start = np.int32([0, 1, 14, 3, 31, 32, 62, 0, 64, 65, 5])
    _check(w, what + " windows")


@pytest.mark.parametrize("dtype,D,Hq,T,tiles", [("bf16", 128, 4, 8, 9), ("bf16", 64, 4, 8, 13), ("f32", 64, 4, 4, 5), ("f32", 128, 4, 4, 3)])
def test_where_it_ends(dtype, D, Hq, T, tiles):
    """One list: the longest one that is not cut, and one of a tile more."""
    for n, solo in ((tiles, True), (tiles + 1, False)):
        L = (n - 1) * 64
        w = W.make_workload("end", B=1, T=T, Hq=Hq, Hkv=1, D=D, seq_lens=[L], trees=W.chain_tree(T), page_size=0, seed=n, paged=False,
                            dtype=dtype)
        _check(w, "solo %s D=%d %d tiles" % (dtype, D, n), solo)


@pytest.mark.parametrize("dtype,D,B,Hkv,T,G", [("bf16", 128, 256, 1, 8, 4), ("bf16", 128, 65, 4, 8, 4), ("bf16", 64, 128, 2, 16, 4),
                                               ("bf16", 64, 150, 2, 8, 4), ("f32", 64, 129, 2, 4, 2), ("f32", 128, 520, 2, 4, 4),
                                               ("bf16", 128, 300, 1, 5, 1), ("bf16", 128, 100, 4, 11, 3), ("bf16", 64, 70, 8, 3, 4),
                                               ("bf16", 128, 60, 2, 27, 4), ("bf16", 128, 60, 1, 64, 4), ("bf16", 64, 200, 2, 16, 4)])
def test_as_many_lists_as_compute_units_and_more(dtype, D, B, Hkv, T, G):
    rng = np.random.default_rng(B)
    w = W.make_workload("many", B=B, T=T, Hq=G * Hkv, Hkv=Hkv, D=D, seq_lens=rng.integers(0, 300, size=B), trees=W.chain_tree(T),
                        page_size=32, seed=B, dtype=dtype)
    w.kv_start = (w.seq_lens // 3).astype(np.int32)
    _check(w, "solo %s D=%d B=%d" % (dtype, D, B))


def test_write_back_of_more_lists_than_compute_units():
    """The four-wave kernel's part of the write-back, for one and for two blocks of rows."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    for T in (5, 12):
        w = W.make_workload("pairs", B=100, T=T, Hq=12, Hkv=3, D=128, seq_lens=np.arange(100), trees=W.chain_tree(T), page_size=16, seed=T)
        new = [torch.randn(100, T, 3, 128, generator=torch.Generator().manual_seed(s)).bfloat16().cuda() for s in (1, 2)]
        res = []
        for folded in (False, True):
            d = to_device(w)
            assert _solo(w, d)
            args = (d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"])
            if folded:
                ta.tree_attn_fwd_ex(*args, k_new=new[0], v_new=new[1])
            else:
                ta.tree_attn_append(new[0], new[1], *args[1:5])
                ta.tree_attn_fwd(*args)
            torch.cuda.synchronize()
            res.append([d[x] for x in ("out", "lse", "k_cache", "v_cache")])
        for x, y in zip(*res):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,D,T,skew", [(dtype, D, T, skew) for dtype in ("bf16", "f32") for D in (64, 128)
                                            for T, skew in ((7, 0), (33, 0), (7, 1)) if dtype == "f32" or not skew])
def test_write_back_folded_in(dtype, D, T, skew):
    """The same outputs and caches as write-back and call in turn, bit for bit; fp32 rows of k_new that begin anywhere too
    (such rows of bf16 take the scalar kernel)."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    lens = [0, 5, 64, 100]
    w = W.make_workload("fold", B=4, T=T, Hq=6, Hkv=2, D=D, seq_lens=lens, trees=W.chain_tree(T), page_size=16, seed=T, dtype=dtype)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    new = []
    for s in (1, 2):
        flat = torch.randn(4 * T * 2 * D + 1, generator=torch.Generator().manual_seed(s)).to(dt).cuda()
        new.append(flat[skew:skew + 4 * T * 2 * D].view(4, T, 2, D))
    res = []
    for folded in (False, True):
        d = to_device(w)
        assert _solo(w, d)
        args = (d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"])
        if folded:
            ta.tree_attn_fwd_ex(*args, k_new=new[0], v_new=new[1])
        else:
            ta.tree_attn_append(new[0], new[1], *args[1:5])
            ta.tree_attn_fwd(*args)
        torch.cuda.synchronize()
        res.append([d[x] for x in ("out", "lse", "k_cache", "v_cache")])
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("copies", [1, 22])
def test_requests_with_mistakes(dtype, D, folded, copies):
    """Up to three tiles a list; 22 times six requests: more workgroups than the device has compute units (bf16: the four-wave
    kernel; fp32, whose 38 rows are three blocks, cuts those)."""
    check_requests_with_mistakes(dtype, D, folded, 0, lens=(125, 90, 61, 40, 112, 33), copies=copies,
                                 alone=copies == 1 or dtype == "bf16")


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
def test_values_that_are_not_finite(dtype, D):
    """An infinite score, all scores at -inf, a NaN and an infinity among the values: the rows that the cut lists spoil, and no
    other, hold no number."""
    import torch
    w = W.make_workload("inf", B=4, T=4, Hq=4, Hkv=1, D=D, seq_lens=[70, 70, 70, 70], trees=W.chain_tree(4), page_size=0, paged=False,
                        seed=3, dtype=dtype)
    d = to_device(w)
    d["q"][:, :, 0] = 1.0
    d["k_cache"][0, 0, 20] = float("inf")
    d["k_cache"][1, 0, :] = float("-inf")
    d["v_cache"][2, 0, 3, 7] = float("nan")
    d["v_cache"][3, 0, 69, 7] = float("inf")
    assert _solo(w, d)
    a, b = run_hip(w, d), run_hip(w, d, num_splits=1)
    for x, y in zip(a, b):
        assert np.array_equal(np.isfinite(x), np.isfinite(y))


@pytest.mark.parametrize("seed", range(48))
def test_forms_against_the_scalar_kernel(seed):
    """Orders and strides of every tensor, page sizes, windows, masks, a subset of the nodes asking, the write-back folded in, no
    log-sum-exp: random combinations on lists walked alone, by either number of waves.  Both kernels take the same inputs in
    fp32 sums; bf16 probabilities and outputs are 2^-9 each off, 1e-2 of the largest as elsewhere, fp32 1e-5."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    rng = np.random.default_rng(seed)
    bf16, D = bool(seed % 2), 64 if seed % 4 < 2 else 128
    dt = torch.bfloat16 if bf16 else torch.float32
    Hkv, G, T = int(rng.choice([1, 2, 3, 8])), int(rng.choice([1, 2, 4, 5])), int(rng.choice([1, 3, 8, 17, 33, 64]))
    Hq = Hkv * G
    B = int(rng.choice([1, 2, 5])) if seed % 3 else -(-280 // Hkv)     # every third: more lists than compute units, small trees
    T = T if seed % 3 else min(T, 8 if bf16 else 3)
    ps = int(rng.choice([0, 1, 8, 32, 128]))
    most = 64 if D == 128 and not bf16 else 128
    lens = rng.integers(0, most + 1, size=B)
    gen = torch.Generator().manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen).to(dt)

    def laid_out(t, order, pad):
        """The same values with the dimensions in memory in this order and `pad` more elements per row."""
        inv = [order.index(i) for i in range(t.dim())]
        full = torch.zeros([t.shape[i] for i in order[:-1]] + [t.shape[-1] + pad], dtype=t.dtype)
        full[..., :t.shape[-1]] = t.permute(order)
        return full.cuda()[..., :t.shape[-1]].permute(inv)

    if ps:
        width = int((lens.max() + T - 1) // ps + 1)
        ids = rng.permutation(B * width).astype(np.int32).reshape(B, width)
        table = torch.from_numpy(np.concatenate([ids, ids[:, :1]], axis=1)).cuda()[:, :width]
        shape = (B * width, Hkv, ps, D)
    else:
        table, shape = None, (B, Hkv, int(lens.max()) + T, D)
    tok, node = rng.choice([0, 16], size=2)
    kv = [laid_out(normal(*shape), [0, 1, 2, 3] if rng.random() < 0.5 else [0, 2, 1, 3], int(tok)) for _ in range(2)]
    Tq = int(rng.integers(1, T + 1))
    q = laid_out(normal(B, Tq, Hq, D), [0, 1, 2, 3] if rng.random() < 0.5 else [0, 2, 1, 3], int(node))
    seq = torch.zeros(2 * B, dtype=torch.int32, device="cuda")
    seq[::2] = torch.from_numpy(lens.astype(np.int32)).cuda()
    trees = np.stack([W.random_tree(T, min(T, 6), rng) for _ in range(B)]) if rng.random() < 0.5 else W.random_tree(T, min(T, 6), rng)
    parent = torch.from_numpy(np.ascontiguousarray(trees)).cuda()
    opts = {"q_node_offset": T - Tq}
    if rng.random() < 0.5:
        opts["kv_start"] = torch.from_numpy((lens * rng.random(B)).astype(np.int32)).cuda()
    if rng.random() < 0.5:
        opts["tree_masks"] = torch.empty(tuple(parent.shape), dtype=torch.int64, device="cuda")
        ta.tree_attn_encode(parent, opts["tree_masks"])
    if rng.random() < 0.5:
        opts["k_new"], opts["v_new"] = (laid_out(normal(B, T, Hkv, D), [0, 2, 1, 3] if rng.random() < 0.5 else [0, 1, 2, 3], 8)
                                        for _ in range(2))
    out_order = [0, 1, 2, 3] if rng.random() < 0.5 else [0, 2, 1, 3]
    with_lse = rng.random() < 0.8
    res = []
    for kernel in (0, 1):
        k, v = (x.clone(memory_format=torch.preserve_format) for x in kv)
        out = laid_out(torch.zeros(B, Tq, Hq, D, dtype=dt), out_order, 8)
        lse = torch.zeros(B, Tq, Hq, device="cuda").permute(0, 2, 1) if with_lse else None
        if kernel == 0:
            plan = ta.tree_attn_plan(q, k, v, table, seq[::2], parent, out, lse)
            assert plan["merge_workgroups"] == 0, plan
        print("solo forms seed=%d kernel=%d %s D=%d B=%d %d/%d T=%d/%d ps=%d %s" %
              (seed, kernel, dt, D, B, Hq, Hkv, Tq, T, ps, sorted(opts)), flush=True)
        ta.tree_attn_last_status()
        ta.tree_attn_fwd_ex(q, k, v, table, seq[::2], parent, out, lse, kernel=kernel, **opts)
        assert ta.tree_attn_last_status() == 0
        res.append((out.float(), lse, k, v))
    (o0, l0, k0, v0), (o1, l1, k1, v1) = res
    assert torch.isfinite(o0).all()
    tol = 1e-2 if bf16 else 1e-5
    assert (o0 - o1).abs().max() <= tol * o1.abs().max()
    if with_lse:
        assert (l0 - l1).abs().max() <= (1e-3 if bf16 else 1e-5 * max(1.0, float(l1.abs().max())))
    assert torch.equal(k0, k1) and torch.equal(v0, v1)
