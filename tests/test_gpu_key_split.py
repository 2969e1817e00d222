"""Key-split matrix-core kernel (head_dim 64, or on request): sizes at the edges of its runs of 32 tokens, its row blocks,
the page ids a wave keeps and the ways it holds the schedule, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, check_requests_with_mistakes, run_hip, run_oracle

pytestmark = pytest.mark.gpu
MFMA_BASIC = 3


def _check(w, what, **kw):
    got, lse = run_hip(w, kernel=MFMA_BASIC, **kw)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, "bf16", what)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,Hq,Hkv", [(1, 1, 1), (8, 4, 1), (33, 1, 1), (32, 2, 1), (13, 5, 1), (64, 4, 2)])
@pytest.mark.parametrize("ps", [0, 16, 64])
def test_runs_row_blocks_and_tree_ends(D, T, Hq, Hkv, ps):
    """Prefixes that end at and around a run of 32 tokens, a tile of 64 and a round of all waves; 1 to 128 rows; trees of
    one and two runs."""
    lens = [0, 1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 700]
    rng = np.random.default_rng(D + T)
    trees = np.stack([W.random_tree(T, min(T, 7), rng) for _ in lens])
    for splits in (0, 2):
        w = W.make_workload("runs", B=len(lens), T=T, Hq=Hq, Hkv=Hkv, D=D, seq_lens=lens, trees=trees, page_size=ps,
                            seed=31 + T, paged=ps > 0)
        _check(w, "D=%d T=%d ps=%d splits=%d" % (D, T, ps, splits), num_splits=splits)


@pytest.mark.parametrize("D,ps,L", [(64, 64, 16384 + 95), (64, 16, 2 * 8192 + 33), (64, 8, 4500), (128, 16, 8192 + 40),
                                    (64, 4, 300), (64, 1, 150)])
def test_more_runs_than_a_wave_keeps_page_ids_for(D, ps, L):
    """One share longer than the 64 page ids a wave holds at a time (64, 32 or 16 runs of its own), and pages of fewer
    than eight tokens, which are looked up row by row."""
    w = W.make_workload("ids", B=1, T=9, Hq=4, Hkv=1, D=D, seq_lens=[L], trees=W.bfs_tree(9, [3], 4), page_size=ps, seed=5)
    _check(w, "D=%d ps=%d" % (D, ps), num_splits=1)


@pytest.mark.parametrize("B", [64, 65, 256, 257])
def test_schedule_in_registers_and_in_lds(B):
    rng = np.random.default_rng(B)
    w = W.make_workload("sched", B=B, T=4, Hq=4, Hkv=2, D=64, seq_lens=rng.integers(0, 200, size=B), trees=W.chain_tree(4),
                        page_size=32, seed=B)
    w.kv_start = (w.seq_lens // 3).astype(np.int32)
    _check(w, "B=%d" % B)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("folded", [False, True])
def test_requests_with_mistakes_are_spoiled_and_reported(D, folded):
    check_requests_with_mistakes("bf16", D, folded, MFMA_BASIC)
