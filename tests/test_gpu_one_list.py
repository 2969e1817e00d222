"""One list on the key-split kernel: lengths around those where the number of its shares changes (64 or 128 partial results, shares of
two, three, four, six and eight tiles, the end of the rule), in tables that hold no more and twice as much, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu


EDGES = (59, 60, 122, 123, 187, 251, 252, 314, 506, 507)


@pytest.mark.parametrize("D,T,Hq,tiles", [(128, T, Hq, t) for T, Hq in ((8, 8), (7, 5)) for t in EDGES] +
                         [(128, 4, 5, t) for t in (314, 506, 507)] +           # (one block of rows: from 257 tiles on)
                         [(64, 4, 8, t) for t in EDGES + (1018, 1019)])
def test_shares_of_one_list(D, T, Hq, tiles):
    from paper_2508_08192_amd import treeattn as ta
    for wide in (False, True):
        L = 64 * (tiles - 1) - 7
        w = W.make_workload("one", B=1, T=T, Hq=Hq, Hkv=1, D=D, seq_lens=[L], trees=W.chain_tree(T), page_size=64, seed=tiles)
        if wide:
            w.page_table = np.ascontiguousarray(np.concatenate([w.page_table, w.page_table], axis=1))
        d = to_device(w)
        plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"])
        assert plan["key_split"] == 1 and plan["merge_kernel"] == ta.TA_MERGE_D128_WIDE and plan["merge_workgroups"] > 0, plan
        print("one list D=%d T=%d tiles=%d wide=%s" % (D, T, tiles, wide), flush=True)
        got, lse = run_hip(w, d)
        ref, ref_lse = run_oracle(w)
        assert_parity(got, lse, ref, ref_lse, "bf16", "D=%d T=%d tiles=%d wide=%s" % (D, T, tiles, wide))


@pytest.mark.parametrize("D,T,Hq,tiles", [
    (128, 64, 8, 61), (128, 64, 8, 66), (128, 64, 8, 130),          # sixteen workgroups: none are left out
    (128, 32, 8, 120), (64, 16, 8, 251), (64, 8, 8, 530), (64, 16, 8, 300),
    (128, 16, 8, 251), (128, 16, 8, 300), (128, 8, 8, 60), (128, 8, 8, 251), (128, 8, 8, 400), (128, 8, 8, 505), (128, 8, 8, 506),
    (128, 4, 8, 270), (64, 4, 8, 505), (64, 4, 8, 530), (64, 4, 8, 1018)])
def test_number_of_partial_results(D, T, Hq, tiles):
    """The owners that the KV pass leaves in the workspace are the first and the last of as many workgroups as the rule gives."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    from tests.test_schedule_model import _cuts, one_list_parts
    w = W.make_workload("one", B=1, T=T, Hq=Hq, Hkv=1, D=D, seq_lens=[64 * (tiles - 1) - 7], trees=W.chain_tree(T), page_size=64, seed=1)
    d = to_device(w)
    args = (d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"], d["lse"])
    plan = ta.tree_attn_plan(*args)
    assert plan["key_split"] == 1 and plan["merge_kernel"] == ta.TA_MERGE_D128_WIDE and plan["merge_workgroups"] > 0, plan
    ws = torch.zeros(plan["workspace_bytes"], dtype=torch.uint8, device="cuda")
    print("one list, partial results D=%d T=%d tiles=%d" % (D, T, tiles), flush=True)
    ta.tree_attn_fwd_ex(*args, workspace=ws)
    torch.cuda.synchronize()
    owners = ws[plan["workspace_bytes"] - 256:].view(torch.int32)[:2].tolist()          # behind the partial results
    total, n_wg = tiles + plan["item_cost"] - 1, plan["kv_workgroups"]
    cuts, _ = _cuts(total, n_wg, plan["min_share"], one_list_parts(D, n_wg))
    last = max(k for k in range(n_wg) if cuts[k] < min(tiles, cuts[k + 1]))             # (padding stands behind the tiles)
    assert owners == [0, last], (owners, last)
