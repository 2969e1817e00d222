"""Calls that choose their kernel by themselves: one to sixteen blocks of 32 query rows on the key-split kernel, in row
groups of 32 and in groups of 256 whose parts lie in several workgroups, with every option, against the fp64 oracle and the
pipelined kernel; and the sizes at which the choice falls."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu
MFMA = 2


def _plan(w, d, kernel=0):
    from paper_2508_08192_amd import treeattn as ta
    return ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                             d["lse"], kernel=kernel)


@pytest.mark.parametrize("T,Hq,Hkv", [(1, 3, 1), (32, 1, 1), (33, 1, 1), (32, 5, 1), (64, 4, 1), (43, 6, 1), (64, 16, 2), (63, 8, 1)])
@pytest.mark.parametrize("ps,scale_up", [(16, 1), (0, 7)])
def test_row_blocks_of_the_key_split_kernel(T, Hq, Hkv, ps, scale_up):
    lens = [0, 65, 300, 128 * scale_up]
    rng = np.random.default_rng(T)
    trees = np.stack([W.random_tree(T, min(T, 7), rng) for _ in lens])
    w = W.make_workload("blocks", B=len(lens), T=T, Hq=Hq, Hkv=Hkv, D=128, seq_lens=lens, trees=trees, page_size=ps or 64,
                        seed=T, paged=ps > 0)
    w.kv_start = np.int32([0, 64, 33, 0])
    d = to_device(w)
    rows = T * Hq // Hkv
    plan = _plan(w, d)
    blocks = -(-rows // 32)
    if blocks == 1 or blocks > 4:
        assert plan["key_split"] == 1 and plan["rows_per_group"] == (32 if blocks == 1 else 256), plan
    assert _plan(w, d, MFMA)["key_split"] == 0
    ref, ref_lse = run_oracle(w)
    for kernel in (0, MFMA):
        print("kernel choice T=%d %d/%d ps=%d kernel=%d" % (T, Hq, Hkv, ps, kernel), flush=True)
        got, lse = run_hip(w, d, kernel=kernel)
        assert_parity(got, lse, ref, ref_lse, "bf16", "rows %d kernel %d" % (rows, kernel))


def test_parts_of_a_row_group_with_every_option():
    """320 query rows in two groups of 256 whose ten parts lie in ten workgroups: a subset of the nodes, given masks, the
    write-back folded in, a bad page and a bad length each spoiling its own request only."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    T, Hq, lens = 64, 6, [200, 70, 129, 40]
    w = W.make_workload("parts", B=4, T=T, Hq=Hq, Hkv=1, D=128, seq_lens=lens, trees=W.bfs_tree(T, [4, 2], 8), page_size=32,
                        seed=3)
    d = to_device(w)
    masks = torch.empty((T,), dtype=torch.int64, device="cuda")
    ta.tree_attn_encode(d["tree_parent"], masks)
    g = torch.Generator(device="cuda").manual_seed(1)
    k_new = torch.randn(4, T, 1, 128, generator=g, device="cuda").bfloat16()
    v_new = torch.randn(4, T, 1, 128, generator=g, device="cuda").bfloat16()
    q = d["q"][:, 10:].contiguous()
    d["page_table"][1, 1] = 1 << 30
    d["seq_lens"][3] = -5
    res = []
    for kernel in (0, MFMA):
        k, v = d["k_cache"].clone(), d["v_cache"].clone()
        out, lse = torch.zeros_like(q), torch.zeros((4, Hq, T - 10), device="cuda")
        ta.tree_attn_last_status()
        print("kernel choice: every option, kernel=%d" % kernel, flush=True)
        ta.tree_attn_fwd_ex(q, k, v, d["page_table"], d["seq_lens"], d["tree_parent"], out, lse, kernel=kernel,
                            tree_masks=masks, q_node_offset=10, k_new=k_new, v_new=v_new)
        torch.cuda.synchronize()
        assert ta.tree_attn_last_status() == ta.TA_STATUS_BAD_PAGE | ta.TA_STATUS_BAD_SEQLEN
        res.append((out.float(), lse, k, v))
    (o0, l0, k0, v0), (o1, l1, k1, v1) = res
    for b in (1, 3):
        assert torch.isnan(o0[b]).all() and torch.isnan(l0[b]).all()
    for b in (0, 2):
        # both kernels take the probabilities as bf16 (2^-9 each) and round the result to bf16 (2^-9): 1e-2 as elsewhere
        assert (o0[b] - o1[b]).abs().max() <= 1e-2 * o1[b].abs().max() and (l0[b] - l1[b]).abs().max() <= 1e-3
    assert torch.equal(k0, k1) and torch.equal(v0, v1)


@pytest.mark.parametrize("T,Hq,Hkv,ps", [(8, 12, 3, 16), (23, 4, 4, 0), (50, 4, 4, 32)])
@pytest.mark.parametrize("cost", [0, 9])
def test_many_lists_are_finished_without_a_merge(T, Hq, Hkv, ps, cost):
    """At least two lists per workgroup: the ones that lie whole in a share are written by the KV pass, the others merged,
    with the write-back folded in, a strided output, bad requests among them and no log-sum-exp asked for.  A list cost that
    is named keeps them cut; without one the shorter of these batches are walked alone."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    B = 200
    rng = np.random.default_rng(T)
    w = W.make_workload("many", B=B, T=T, Hq=Hq, Hkv=Hkv, D=128, seq_lens=rng.integers(0, 200, size=B),
                        trees=W.random_tree(T, 5, rng), page_size=ps or 64, seed=T, paged=ps > 0)
    w.seq_lens[5] = 900 if ps == 0 else w.seq_lens[5]
    w = W.make_workload("many", B=B, T=T, Hq=Hq, Hkv=Hkv, D=128, seq_lens=w.seq_lens, trees=w.tree_parent, page_size=ps or 64,
                        seed=T, paged=ps > 0)
    d = to_device(w)
    ref, ref_lse = run_oracle(w)
    d["out"] = torch.zeros((B, T, Hq, 132), dtype=d["q"].dtype, device="cuda")[..., 4:132] if T == 8 else d["out"]
    print("kernel choice: many lists T=%d" % T, flush=True)
    if cost:
        plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                                 d["lse"], item_cost=cost)
        assert plan["merge_workgroups"] > 0 and plan["key_split"] == (T < 50) and B * Hkv >= 2 * plan["kv_workgroups"], plan
    got, lse = run_hip(w, d, item_cost=cost)
    assert_parity(got, lse, ref, ref_lse, "bf16", "many lists T=%d" % T)
    for _ in range(3):                                  # repeated calls leave the same
        again, lse2 = run_hip(w, d, item_cost=cost)
        assert np.array_equal(again, got) and np.array_equal(lse2, lse)
    ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], None,
                        item_cost=cost)
    torch.cuda.synchronize()
    assert np.array_equal(d["out"].float().cpu().numpy().astype(np.float64), got)
    d["seq_lens"][7] = -1
    ta.tree_attn_last_status()
    bad, bad_lse = run_hip(w, d, item_cost=cost)
    assert ta.tree_attn_last_status() == ta.TA_STATUS_BAD_SEQLEN
    assert np.isnan(bad[7]).all() and np.isnan(bad_lse[7]).all()
    keep = [b for b in range(B) if b != 7]
    assert_parity(bad[keep], bad_lse[keep], ref[keep], ref_lse[keep], "bf16", "beside a bad request")
    d["seq_lens"][7] = int(w.seq_lens[7])
    k_new = torch.randn(B, T, Hkv, 128, device="cuda").bfloat16()
    v_new = torch.randn(B, T, Hkv, 128, device="cuda").bfloat16()
    args = (d["page_table"], d["seq_lens"], d["tree_parent"])
    k1, v1 = d["k_cache"].clone(), d["v_cache"].clone()
    o1, l1 = torch.zeros_like(d["q"]), torch.zeros_like(d["lse"])
    ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], *args, o1, l1, k_new=k_new, v_new=v_new, item_cost=cost)
    ta.tree_attn_append(k_new, v_new, k1, v1, d["page_table"], d["seq_lens"])
    o2, l2 = torch.zeros_like(o1), torch.zeros_like(l1)
    ta.tree_attn_fwd_ex(d["q"], k1, v1, *args, o2, l2, item_cost=cost)
    torch.cuda.synchronize()
    assert torch.equal(k1, d["k_cache"]) and torch.equal(v1, d["v_cache"]) and torch.equal(o1, o2) and torch.equal(l1, l2)


@pytest.mark.parametrize("T,Hq,L", [(33, 1, 500), (64, 2, 4000), (50, 5, 130), (64, 8, 20000)])
def test_head_dim_64_with_32_and_64_rows_a_workgroup(T, Hq, L):
    """Small batches of head_dim 64 keep 32 rows per workgroup whatever their number, larger ones 64."""
    lens = [L, L // 7]
    w = W.make_workload("d64", B=2, T=T, Hq=Hq, Hkv=1, D=64, seq_lens=lens, trees=W.chain_tree(T), page_size=64, seed=T)
    d = to_device(w)
    blocks = -(-T * Hq // 32)
    small = 2 * (-(-L // 64) + 1) * blocks <= 16 * 256
    assert _plan(w, d)["rows_per_group"] == (32 if small else 64)
    print("kernel choice: head_dim 64, T=%d Hq=%d L=%d" % (T, Hq, L), flush=True)
    got, lse = run_hip(w, d)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, "bf16", "T=%d Hq=%d L=%d" % (T, Hq, L))


def test_values_that_are_not_finite_come_out_alike_with_and_without_a_merge():
    """Lists that the KV pass finishes by itself follow the same rules as merged ones: an infinity or a NaN among the attended
    values spoils the whole row and leaves the log-sum-exp; scores that are all minus infinity leave neither."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    B, T, Hq, Hkv = 160, 8, 16, 4
    w = W.make_workload("nonfinite", B=B, T=T, Hq=Hq, Hkv=Hkv, D=128, seq_lens=[40 + 3 * b for b in range(B)],
                        trees=W.chain_tree(T), page_size=1024, seed=12, paged=False)
    d = to_device(w)
    d["q"].abs_()
    inf = float("inf")
    for b in range(0, B, 8):                        # in every eighth request, so that some of each lie whole in a share
        d["v_cache"][b, 1, 20, 5] = inf
        d["v_cache"][b + 1, 2, 7, 9] = float("nan")
        d["k_cache"][b + 2, 3, :, 1] = -inf
        d["v_cache"][b + 3, 0, 30, :] = -inf
    hurt = {0: 1, 1: 2, 2: 3, 3: 0}
    res = []
    for kw in ({}, {"num_splits": 256}):            # 640 lists: at 256 shares most are finished by the KV pass
        out, lse = torch.zeros_like(d["q"]), torch.zeros_like(d["lse"])
        for kernel in (0, MFMA):
            print("kernel choice: not finite, kernel=%d %s" % (kernel, kw), flush=True)
            ta.tree_attn_fwd_ex(d["q"], d["k_cache"], d["v_cache"], None, d["seq_lens"], d["tree_parent"], out, lse,
                                kernel=kernel, **kw)
            torch.cuda.synchronize()
            res.append((out.float().clone(), lse.clone()))
    G = Hq // Hkv
    for out, lse in res:
        for b in range(B):
            for g in range(Hkv):
                rows, l = out[b, :, g * G:(g + 1) * G], lse[b, g * G:(g + 1) * G]
                if hurt.get(b % 8) == g:
                    assert torch.isnan(rows).all(), (b, g)
                    assert (torch.isnan(l) if b % 8 == 2 else torch.isfinite(l)).all(), (b, g)
                else:
                    assert torch.isfinite(rows).all() and torch.isfinite(l).all(), (b, g)
