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
