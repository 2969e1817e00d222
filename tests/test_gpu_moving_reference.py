"""The lines of the running softmax that run where a reference moves: keys that outdo all before them, each for one query row, in
every quarter of a lane's sixteen tokens, in even and odd tiles and runs, in mid-walk.  All blocks of the pipelined kernel and the
key-split kernel, against the fp64 oracle.  (Values that are normal move a reference in the first tile or two and hardly ever after.)"""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu
MFMA, MFMA_BASIC = 2, 3
PACED, NARROW, WIDE = 0, 1, 2


def _climbing(T, Hq, D, L, n, seed, table=0):
    """n keys spread over the prefix, tile parity and place in the sixteen tokens all changing, each along the query of a
    row of its own; what a row meets a second time is longer."""
    w = W.make_workload("climb", B=1, T=T, Hq=Hq, Hkv=1, D=D, seq_lens=[L], trees=W.random_tree(T, min(T, 5), np.random.default_rng(seed)),
                        page_size=64, seed=seed, kv_std=0.5)
    q = W.bf16_bits_to_f32(w.q[0]).reshape(T * Hq, D).astype(np.float64)
    rows = T * Hq
    for j in range(n):
        r = (j * 11) % rows
        # a score of this many powers of two above zero; those of the other keys stay below 4
        up = 8.0 + 10.0 * (j // rows + j * 4 // n)
        key = q[r] / np.linalg.norm(q[r]) ** 2 * np.sqrt(D) * np.log(2.0) * up
        pos = (L * (j + 1)) // (n + 2) // 16 * 16 + 4 * (j % 4) + (j // 4) % 4
        w.k_cache[int(w.page_table[0, pos // 64]), 0, pos % 64] = W.to_bf16_bits(key.astype(np.float32))
    if table:
        w.page_table = np.pad(w.page_table, ((0, 0), (0, max(0, table - w.page_table.shape[1]))))
    return w


def _moves(w, tile):
    """Rows whose running maximum (powers of two, tile by tile) rises by more than 4 after the first two tiles."""
    L, T = int(w.seq_lens[0]), w.T
    K = np.concatenate([W.bf16_bits_to_f32(w.k_cache[int(p), 0]) for p in w.page_table[0, :-(-L // 64)]])[:L].astype(np.float64)
    q = W.bf16_bits_to_f32(w.q[0]).reshape(T * w.Hq, w.D).astype(np.float64)
    s = q @ K.T / np.sqrt(w.D) / np.log(2.0)
    m = np.maximum.accumulate(np.stack([s[:, i:i + tile].max(1) for i in range(0, L, tile)]), 0)
    return int(((m[2:] - m[1:-1]) > 4).sum())


def _run(w, what, kernel, splits):
    d = to_device(w)
    print(what, flush=True)
    got, lse = run_hip(w, d, kernel=kernel, num_splits=splits)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, "bf16", what)
    return d


@pytest.mark.parametrize("T,Hq,table,blocks", [
    (8, 4, 0, PACED), (16, 4, 0, PACED), (12, 8, 0, PACED), (16, 8, 0, PACED), (16, 8, 400, WIDE), (63, 2, 400, WIDE),
    (20, 8, 0, NARROW), (28, 8, 0, NARROW), (32, 8, 0, NARROW), (32, 8, 400, WIDE), (15, 15, 400, WIDE)])
@pytest.mark.parametrize("n", [16, 61])
def test_pipelined_kernel(T, Hq, table, blocks, n):
    from paper_2508_08192_amd import treeattn as ta
    w = _climbing(T, Hq, 128, 64 * 70 + 9, n, T + n, table)
    assert _moves(w, 64) >= n // 2
    splits = 1 if table else 2
    d = _run(w, "climbing keys T=%d Hq=%d blocks=%d n=%d" % (T, Hq, blocks, n), MFMA, splits)
    plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                             d["lse"], kernel=MFMA, num_splits=splits)
    assert plan["blocks"] == blocks and plan["key_split"] == 0, plan


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,Hq,n", [(8, 4, 16), (16, 4, 61), (5, 3, 61), (64, 4, 61)])
@pytest.mark.parametrize("splits", [1, 3])
def test_key_split_kernel(D, T, Hq, n, splits):
    """Eight waves take every eighth run of 32 tokens, so a list long enough for each to meet several of the keys."""
    w = _climbing(T, Hq, D, 64 * 90 + 37, n, T + n)
    assert _moves(w, 32) >= n // 2
    _run(w, "climbing keys, key-split, D=%d T=%d Hq=%d n=%d splits=%d" % (D, T, Hq, n, splits), MFMA_BASIC, splits)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,Hq", [(8, 4), (3, 5)])
def test_lists_walked_alone(D, T, Hq):
    """Waves that walk a whole list move their reference whenever they can."""
    from paper_2508_08192_amd import treeattn as ta
    w = _climbing(T, Hq, D, 64 * 7 + 21, 13, T)
    assert _moves(w, 32) >= 4
    d = _run(w, "climbing keys, walked alone, D=%d T=%d" % (D, T), 0, 0)
    plan = ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                             d["lse"])
    assert plan["merge_workgroups"] == 0, plan
