"""One list on the key-split kernel: lengths around those where the number of its shares changes (64 or 128 partial results, shares of
two, three, four, six and eight tiles, the end of the rule), in tables that hold no more and twice as much, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,T,Hq", [(128, 8, 8), (128, 4, 5), (64, 4, 8)])
@pytest.mark.parametrize("tiles", [59, 60, 122, 123, 187, 251, 252, 314, 506, 507, 1018, 1019])
def test_shares_of_one_list(D, T, Hq, tiles):
    if tiles > 600 and D == 128:
        return                                 # (beyond the rule there)
    for wide in (False, True):
        L = 64 * (tiles - 1) - 7
        w = W.make_workload("one", B=1, T=T, Hq=Hq, Hkv=1, D=D, seq_lens=[L], trees=W.chain_tree(T), page_size=64, seed=tiles)
        if wide:
            w.page_table = np.ascontiguousarray(np.concatenate([w.page_table, w.page_table], axis=1))
        print("one list D=%d T=%d tiles=%d wide=%s" % (D, T, tiles, wide), flush=True)
        got, lse = run_hip(w, to_device(w))
        ref, ref_lse = run_oracle(w)
        assert_parity(got, lse, ref, ref_lse, "bf16", "D=%d T=%d tiles=%d wide=%s" % (D, T, tiles, wide))
