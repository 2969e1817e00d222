"""The merge of head_dim 64 (16 lanes per output row): one, a few, exactly 16, more than 16 partial results per list, a
workgroup per row, a last wave with idle parts, and outputs that are not aligned for it, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,Hq,Hkv,L,splits", [
    (1, 1, 1, 40, 1), (5, 3, 1, 200, 3), (7, 4, 2, 1000, 32), (9, 1, 1, 1200, 15), (9, 1, 1, 1200, 17), (33, 33, 1, 1300, 20),
    (64, 16, 2, 1100, 40), (3, 2, 1, 4000, 0)])
@pytest.mark.parametrize("aligned", [True, False])
def test_merge_of_head_dim_64(dtype, T, Hq, Hkv, L, splits, aligned):
    import torch
    w = W.make_workload("merge64", B=2, T=T, Hq=Hq, Hkv=Hkv, D=64, seq_lens=[L, L // 3], trees=W.chain_tree(T), page_size=32,
                        seed=T + splits, dtype=dtype)
    d = to_device(w)
    if not aligned:
        d["out"] = torch.zeros((2, T, Hq, 66), dtype=d["q"].dtype, device="cuda")[..., 1:65]
    print("merge64 %s T=%d %d/%d L=%d splits=%d aligned=%s" % (dtype, T, Hq, Hkv, L, splits, aligned), flush=True)
    got, lse = run_hip(w, d, num_splits=splits)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, dtype, "T=%d L=%d splits=%d" % (T, L, splits))
    assert np.isfinite(lse).all()
