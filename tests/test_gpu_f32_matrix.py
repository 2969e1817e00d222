"""fp32 attention on the matrix cores (head_dim 64 and 128): sizes at the edges of its runs of 16 tokens, of the rounds of
its four waves and of its groups of 32 rows, every way the tree tokens and the schedule reach it, values at which a
probability of zero is not enough, and requests with mistakes, against the fp64 oracle and the scalar kernel."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, check_requests_with_mistakes, run_hip, run_oracle, to_device, with_decoy_pages

pytestmark = pytest.mark.gpu
GENERIC = 1


def _check(w, what, **kw):
    print("f32 matrix " + what, flush=True)
    got, lse = run_hip(w, **kw)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, "f32", what)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,Hq,Hkv", [(1, 1, 1), (8, 4, 1), (33, 1, 1), (11, 6, 2), (13, 5, 1), (64, 4, 2)])
@pytest.mark.parametrize("ps", [0, 4, 64])
def test_runs_row_groups_and_tree_ends(D, T, Hq, Hkv, ps):
    """Prefixes at and around a run, a tile and a round of the waves; 1 to 128 rows in one to four groups, even and uneven;
    trees of one and two runs."""
    lens = [0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 700]
    rng = np.random.default_rng(D + T)
    trees = np.stack([W.random_tree(T, min(T, 7), rng) for _ in lens])
    for splits in (0, 2):
        w = W.make_workload("runs", B=len(lens), T=T, Hq=Hq, Hkv=Hkv, D=D, seq_lens=lens, trees=trees, page_size=ps or 64,
                            seed=41 + T, paged=ps > 0, dtype="f32")
        _check(w, "D=%d T=%d ps=%d splits=%d" % (D, T, ps, splits), num_splits=splits)


@pytest.mark.parametrize("B", [64, 65, 257])
def test_schedule_in_registers_and_in_lds_with_windows(B):
    rng = np.random.default_rng(B)
    w = W.make_workload("sched", B=B, T=4, Hq=4, Hkv=2, D=64, seq_lens=rng.integers(0, 200, size=B), trees=W.chain_tree(4),
                        page_size=32, seed=B, dtype="f32")
    w.kv_start = (w.seq_lens // 3).astype(np.int32)
    _check(w, "B=%d" % B)


@pytest.mark.parametrize("B,D,Hq,T", [(64, 64, 4, 4), (65, 64, 4, 4), (65, 128, 4, 9), (257, 64, 4, 4), (257, 128, 8, 12)])
@pytest.mark.parametrize("cost", [1, 2])
def test_schedule_of_cut_lists_in_registers_and_in_lds(B, D, Hq, T, cost):
    """The same batches with a list cost named, which keeps lists of a few tiles on the cut path; blocks of 16 and of 32 rows."""
    from paper_2508_08192_amd import treeattn as ta
    rng = np.random.default_rng(B)
    w = W.make_workload("sched", B=B, T=T, Hq=Hq, Hkv=2, D=D, seq_lens=rng.integers(0, 200, size=B), trees=W.chain_tree(T),
                        page_size=32, seed=B, dtype="f32")
    w.kv_start = (w.seq_lens // 3).astype(np.int32)
    d = to_device(w)
    plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"],
                             item_cost=cost)
    assert plan["table_row"] == -1 and plan["merge_workgroups"] > 0, plan
    _check(w, "cut B=%d D=%d T=%d cost=%d" % (B, D, T, cost), item_cost=cost)


@pytest.mark.parametrize("D", [64, 128])
def test_options_agree_with_the_scalar_kernel(D):
    """Masks encoded before the call, a subset of the nodes asking, the write-back folded in, rows whose start is no multiple
    of 16 bytes (which the scalar kernel keeps): both kernels give the same results up to the order of fp32 sums (2^-24 of
    a value per step of sums over up to 300 terms that partly cancel: 1e-5 of the largest)."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    lens = [5, 300, 64]
    T, Hq, Hkv, off = 12, 4, 2, 7
    w = W.make_workload("opts", B=3, T=T, Hq=Hq, Hkv=Hkv, D=D, seq_lens=lens, trees=W.bfs_tree(T, [3], 4), page_size=16,
                        seed=77, dtype="f32")
    d = to_device(w)
    g = torch.Generator(device="cuda").manual_seed(3)
    k_new = torch.randn(3, T, Hkv, D, generator=g, device="cuda")
    v_new = torch.randn(3, T, Hkv, D, generator=g, device="cuda")
    masks = torch.empty((T,), dtype=torch.int64, device="cuda")
    ta.tree_attn_encode(d["tree_parent"], masks)
    wide = torch.randn(3, T, Hq, D + 1, generator=g, device="cuda")
    qs = {"whole": wide[..., :D].contiguous(), "some": wide[:, off:, :, :D].contiguous(), "unaligned": wide[..., 1:]}
    for name, q in qs.items():
        for kw in ({}, {"tree_masks": masks}, {"k_new": k_new, "v_new": v_new}):
            if name == "some":
                kw = dict(kw, q_node_offset=off)
            res = []
            for kernel in (0, GENERIC):
                k, v = d["k_cache"].clone(), d["v_cache"].clone()
                out = torch.full((3, q.shape[1], Hq, D), float("nan"), device="cuda")
                lse = torch.full((3, Hq, q.shape[1]), float("nan"), device="cuda")
                print("f32 options D=%d %s %s kernel=%d" % (D, name, sorted(kw), kernel), flush=True)
                ta.tree_attn_fwd_ex(q, k, v, d["page_table"], d["seq_lens"], d["tree_parent"], out, lse, kernel=kernel, **kw)
                torch.cuda.synchronize()
                res.append((out, lse, k, v))
            (o0, l0, k0, v0), (o1, l1, k1, v1) = res
            assert torch.isfinite(o0).all() and (o0 - o1).abs().max() <= 1e-5 * o1.abs().max()
            assert (l0 - l1).abs().max() <= 1e-5 * l1.abs().max()
            assert torch.equal(k0, k1) and torch.equal(v0, v1)


def test_infinities_and_nans_come_out_as_from_the_scalar_kernel():
    """An infinite value in the last attended token of a ragged prefix (whose places after it repeat that token with
    probability zero), an infinite score, a NaN key, keys whose scores are all -inf, a NaN in a row beyond the prefix."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    L = [37, 37, 37, 40, 33, 70]
    w = W.make_workload("inf", B=6, T=3, Hq=2, Hkv=1, D=64, seq_lens=L, trees=W.chain_tree(3), page_size=128, seed=9,
                        dtype="f32", paged=False)
    d = to_device(w)
    inf = float("inf")
    d["q"].abs_()
    d["v_cache"][0, 0, 36, 5] = inf
    d["k_cache"][1, 0, 20, 3] = inf
    d["k_cache"][2, 0, 36, 3] = float("nan")
    d["k_cache"][3, 0, :3, 1] = -inf
    d["k_cache"][4, 0, :36, 1] = -inf
    d["v_cache"][5, 0, 73:] = float("nan")
    d["k_cache"][5, 0, 73:] = float("nan")
    res = []
    for kernel in (0, GENERIC):
        print("f32 infinities kernel=%d" % kernel, flush=True)
        out, lse = torch.zeros_like(d["q"]), torch.zeros((6, 2, 3), device="cuda")
        ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], None, d["seq_lens"], d["tree_parent"], out, lse, kernel=kernel)
        torch.cuda.synchronize()
        res.append((out, lse))
    (o0, l0), (o1, l1) = res
    torch.testing.assert_close(o0, o1, rtol=1e-5, atol=1e-5, equal_nan=True)
    torch.testing.assert_close(l0, l1, rtol=1e-5, atol=1e-5, equal_nan=True)
    assert torch.isinf(o0[0, :, :, 5]).all() and torch.isfinite(o0[3]).all() and torch.isfinite(o0[5]).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("below", [120, 130, 140, 200])
@pytest.mark.parametrize("splits", [0, 1])
def test_an_infinite_value_counts_however_small_its_probability(D, below, splits):
    """A run of 16 tokens whose scores lie 2^below under the others' (a wave of its own walks it), one value of it infinite:
    that column is no number, the others are, and the log-sum-exp is that of the other tokens."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    w = W.make_workload("far", B=1, T=1, Hq=2, Hkv=1, D=D, seq_lens=[64], trees=W.chain_tree(1), page_size=128, seed=5,
                        dtype="f32", paged=False)
    d = to_device(w)
    d["q"].zero_()
    d["q"][..., 0] = 1.0
    d["k_cache"][..., 0] = 0.0
    d["k_cache"][0, 0, 16:32, 0] = -below * float(np.log(2) * np.sqrt(D))
    d["v_cache"][0, 0, 20, 5] = float("inf")
    print("f32 far below D=%d below=%d splits=%d" % (D, below, splits), flush=True)
    out, lse = torch.zeros_like(d["q"]), torch.zeros((1, 2, 1), device="cuda")
    ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], None, d["seq_lens"], d["tree_parent"], out, lse, num_splits=splits)
    torch.cuda.synchronize()
    finite = torch.isfinite(out)
    assert not finite[..., 5].any()
    finite[..., 5] = True
    assert finite.all() and (lse - float(np.log(49))).abs().max() <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("folded", [False, True])
def test_requests_with_mistakes_are_spoiled_and_reported(D, folded):
    check_requests_with_mistakes("f32", D, folded)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("offset,row", [(1, 0), (0, 1), (3, 2)])
def test_folded_write_back_of_unaligned_rows_gives_the_bits_of_append_and_the_plain_call(D, offset, row):
    """k_new and v_new whose rows start anywhere: the same kernel runs as for the plain call, so out, lse and the caches are
    bit for bit those of tree_attn_append followed by it."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    B, T, Hkv = 3, 18, 2
    w = W.make_workload("f32fold", B=B, T=T, Hq=4, Hkv=Hkv, D=D, seq_lens=[5, 300, 64], trees=W.bfs_tree(T, [3], 5),
                        page_size=16, seed=7, dtype="f32")
    d = to_device(w)
    g = torch.Generator(device="cuda").manual_seed(5)

    def dense():
        flat = torch.randn(offset + B * T * Hkv * (D + row), generator=g, device="cuda")
        return flat[offset:].view(B, T, Hkv, D + row)[..., :D]
    k_new, v_new = dense(), dense()
    args = (d["page_table"], d["seq_lens"], d["tree_parent"])
    k1, v1 = d["k_cache"].clone(), d["v_cache"].clone()
    o1, l1 = torch.zeros_like(d["q"]), torch.zeros_like(d["lse"])
    o2, l2 = torch.zeros_like(o1), torch.zeros_like(l1)
    print("f32 unaligned k_new D=%d offset=%d row=%d" % (D, offset, row), flush=True)
    ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], *args, o1, l1, k_new=k_new, v_new=v_new)
    ta.tree_attn_append(k_new, v_new, k1, v1, d["page_table"], d["seq_lens"])
    ta.tree_attn_fwd(d["q"], k1, v1, *args, o2, l2)
    torch.cuda.synchronize()
    assert torch.equal(k1, d["k_cache"]) and torch.equal(v1, d["v_cache"])
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


@pytest.mark.parametrize("D,ps", [(64, 4), (64, 64), (128, 16)])
def test_pages_before_the_window_are_never_read(D, ps):
    import torch
    from paper_2508_08192_amd import treeattn as ta
    lens, starts = [700, 333, 90, 130], np.int32([333, 200, 90, 7])
    w = W.make_workload("f32released", B=4, T=8, Hq=8, Hkv=2, D=D, seq_lens=lens, trees=W.chain_tree(8), page_size=ps,
                        seed=15, dtype="f32")
    w.kv_start = starts
    d = with_decoy_pages(to_device(w))
    pt = w.page_table.copy()
    for b in range(4):
        pt[b, :int(starts[b]) // ps] = w.k_cache.shape[0] + 1
    d["page_table"] = torch.from_numpy(pt).cuda()
    ref, ref_lse = run_oracle(w)
    ta.tree_attn_last_status()
    for splits in (0, 3):
        print("f32 released pages D=%d ps=%d splits=%d" % (D, ps, splits), flush=True)
        got, lse = run_hip(w, d, num_splits=splits)
        assert ta.tree_attn_last_status() == 0
        assert_parity(got, lse, ref, ref_lse, "f32", "released pages")


@pytest.mark.parametrize("T", [16, 17, 48, 49])
def test_edges_of_the_runs_of_sixteen_tokens(T):
    lens = [15, 16, 17, 47, 48, 49, 79, 80, 81]
    rng = np.random.default_rng(T)
    trees = np.stack([W.random_tree(T, 7, rng) for _ in lens])
    for D in (64, 128):
        for splits in (0, 2):
            w = W.make_workload("runs16", B=len(lens), T=T, Hq=2, Hkv=1, D=D, seq_lens=lens, trees=trees, page_size=8, seed=T,
                                dtype="f32")
            _check(w, "runs of 16: D=%d T=%d splits=%d" % (D, T, splits), num_splits=splits)
