"""The pipelined kernel's wide blocks (16x16x32 products; long shares of row groups of which all waves have rows): shares of
every number of tiles around those that the steady-state loop takes, rows at the edges of the two sixteens a lane holds,
trees of every length and pages of several sizes, a softmax reference that moves in mid-walk, values that are no numbers;
against the fp64 oracle.  The same shapes with other blocks where some waves have none.  (tests/test_pipelined_blocks.py holds the
rule itself.)"""
import numpy as np
import pytest

from paper_2508_08192_amd import workloads as W
from tests.helpers import assert_parity, run_hip, run_oracle, to_device

pytestmark = pytest.mark.gpu
MFMA = 2
PACED, NARROW, WIDE = 0, 1, 2
LONG = 200 * 64                                # tokens a table has to hold for the wide blocks to be chosen


def _workload(T, Hq, Hkv, lens, ps, seed, long=True):
    rng = np.random.default_rng(seed)
    trees = np.stack([W.random_tree(T, min(T, 7), rng) for _ in lens])
    # values of half the size: a node that sees two tokens has outputs as large as they are, and bf16 rounds one of 4 and more by
    # up to 1.6e-2, which alone is more than the parity bar of 1e-2 (of less than 4: 7.8e-3)
    w = W.make_workload("wide", B=len(lens), T=T, Hq=Hq, Hkv=Hkv, D=128, seq_lens=lens, trees=trees, page_size=ps, seed=seed,
                        paged=ps > 0, kv_std=0.5)
    if long and ps:
        w.page_table = np.pad(w.page_table, ((0, 0), (0, max(0, LONG // ps - w.page_table.shape[1]))))
    elif long:
        room = ((0, 0), (0, 0), (0, max(0, LONG - w.k_cache.shape[2])), (0, 0))
        w.k_cache, w.v_cache = np.pad(w.k_cache, room), np.pad(w.v_cache, room)
    return w


def _blocks(T, Hq, Hkv):
    rows = T * Hq // Hkv
    return WIDE if rows > 64 and (rows - 1) % (128 if rows <= 128 else 256) >= (96 if rows <= 128 else 224) else \
        PACED if rows <= 128 else NARROW


def _plan(d, splits, kernel=MFMA):
    from paper_2508_08192_amd import treeattn as ta
    return ta.tree_attn_plan(d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"], d["out"],
                             d["lse"], kernel=kernel, num_splits=splits)


def _check(w, what, splits, blocks):
    d = to_device(w)
    assert _plan(d, splits)["blocks"] == blocks, what
    print(what, flush=True)
    got, lse = run_hip(w, d, kernel=MFMA, num_splits=splits)
    ref, ref_lse = run_oracle(w)
    assert_parity(got, lse, ref, ref_lse, "bf16", what)


@pytest.mark.parametrize("T,Hq,Hkv", [(64, 2, 1), (1, 97, 1), (49, 2, 1), (45, 5, 1), (37, 13, 1), (32, 8, 1), (51, 5, 1),
                                      (64, 16, 2), (13, 5, 1), (17, 4, 1), (33, 5, 1)])
@pytest.mark.parametrize("ps", [0, 4, 16, 64])
def test_tiles_rows_and_tree_ends(T, Hq, Hkv, ps):
    lens = [0, 1, 15, 16, 17, 47, 48, 63, 64, 65, 128, 129, 192, 255, 256, 257, 320, 383, 384, 449, 512, 577, 640, 700]
    w = _workload(T, Hq, Hkv, lens, ps, 7 + T)
    for splits in (1, 2):
        _check(w, "wide T=%d %d/%d ps=%d splits=%d" % (T, Hq, Hkv, ps, splits), splits, _blocks(T, Hq, Hkv))


@pytest.mark.parametrize("T,Hq", [(16, 8), (32, 8)])
def test_reference_moves_in_mid_walk(T, Hq):
    """Keys that grow along the list, in single tiles and single rows: the reference moves again and again, within the
    steady-state loop and in the tiles around it."""
    L = 64 * 70 + 9
    w = _workload(T, Hq, 1, [L], 64, 3)
    k = w.k_cache.copy()
    rng = np.random.default_rng(5)
    for pos in (200, 640, 1000, 1801, 2300, 3111, L - 70, L - 3):
        page = int(w.page_table[0, pos // 64])
        row = (k[page, 0, pos % 64].astype(np.uint32) << 16).view(np.float32) * np.float32(2.0 + 8.0 * rng.random())
        k[page, 0, pos % 64] = (row.view(np.uint32) >> 16).astype(np.uint16)
    w.k_cache = k
    _check(w, "moving reference T=%d" % T, 1, WIDE)


@pytest.mark.parametrize("T,Hq", [(16, 8), (32, 8)])
def test_a_value_that_is_no_number_spoils_its_rows(T, Hq):
    w = _workload(T, Hq, 1, [64 * 66, 64 * 30 + 5], 64, 11)
    v = w.v_cache.copy()
    v[int(w.page_table[0, 20]), 0, 13, 77] = 0x7fc0
    w.v_cache = v
    d = to_device(w)
    assert _plan(d, 1)["blocks"] == WIDE
    got, lse = run_hip(w, d, kernel=MFMA, num_splits=1)
    ref, ref_lse = run_oracle(w)
    assert np.isnan(got[0]).all() and np.isfinite(lse[0]).all()
    assert_parity(got[1:], lse[1:], ref[1:], ref_lse[1:], "bf16", "no number T=%d" % T)


@pytest.mark.parametrize("T,Hq,Hkv,offset", [(40, 8, 2, 8), (64, 4, 1, 4), (64, 8, 1, 0), (28, 8, 2, 0)])
@pytest.mark.parametrize("splits", [1, 2])
def test_every_option_on_wide_blocks(T, Hq, Hkv, offset, splits):
    """64 to 512 query rows a KV head: a subset of the nodes, given masks, the write-back folded in (its own instance of the
    kernel), a bad page and a bad length each spoiling its own request only; against append and the scalar kernel."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    w = _workload(T, Hq, Hkv, [700, 70, 385, 40], 32, 3 + T)
    B, Tq = 4, T - offset
    d = to_device(w)
    masks = torch.empty((B, T), dtype=torch.int64, device="cuda")
    ta.tree_attn_encode(d["tree_parent"], masks)
    k_new, v_new = (torch.randn(B, T, Hkv, 128, generator=torch.Generator().manual_seed(s)).mul_(0.5).bfloat16().cuda() for s in (1, 2))
    d["q"] = d["q"][:, offset:].contiguous()
    d["page_table"][1, 1] = 1 << 30
    d["seq_lens"][3] = -5
    rest = (d["page_table"], d["seq_lens"], d["tree_parent"])

    def call(kernel, folded, **kw):
        k, v = d["k_cache"].clone(), d["v_cache"].clone()
        out, lse = torch.zeros_like(d["q"]), torch.zeros((B, Hq, Tq), device="cuda")
        if folded:
            kw = dict(kw, k_new=k_new, v_new=v_new)
        else:
            ta.tree_attn_append(k_new, v_new, k, v, d["page_table"], d["seq_lens"])
        ta.tree_attn_last_status()
        print("wide, every option, T=%d rows=%d kernel=%d folded=%s" % (T, Tq * Hq // Hkv, kernel, folded), flush=True)
        ta.tree_attn_fwd_ex(d["q"], k, v, *rest, out, lse, kernel=kernel, q_node_offset=offset, **kw)
        assert ta.tree_attn_last_status() == ta.TA_STATUS_BAD_PAGE | ta.TA_STATUS_BAD_SEQLEN
        for b in (1, 3):
            assert torch.isnan(out[b]).all() and torch.isnan(lse[b]).all()
        return out[[0, 2]].float(), lse[[0, 2]], k, v

    d["out"], d["lse"] = torch.empty_like(d["q"]), torch.empty((B, Hq, Tq), device="cuda")
    assert _plan(d, splits)["blocks"] == WIDE
    ref = call(1, False)
    plain = call(MFMA, False, num_splits=splits)
    for given in ({}, {"tree_masks": masks}):
        got = call(MFMA, True, num_splits=splits, **given)
        assert all(torch.equal(x, y) for x, y in zip(got, plain))         # append followed by the plain call, bit for bit
    # probabilities as bf16 (2^-9 each) and the result rounded to bf16 (2^-9): 1e-2 as elsewhere
    assert (plain[0] - ref[0]).abs().max() <= 1e-2 * ref[0].abs().max() and (plain[1] - ref[1]).abs().max() <= 1e-3


@pytest.mark.parametrize("T,Hq", [(16, 8), (32, 8)])
def test_a_captured_call_replays(T, Hq):
    """A captured call on wide blocks leaves what an eager one does, replay after replay, also for lengths set in between."""
    import torch
    from paper_2508_08192_amd import treeattn as ta
    w = _workload(T, Hq, 1, [64 * 66 + 3, 1500], 64, 5)
    d = to_device(w)
    args = (d["q"], d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"], d["tree_parent"])
    assert _plan(d, 1)["blocks"] == WIDE
    call = lambda out, lse: ta.tree_attn_fwd_ex(*args, out, lse, kernel=MFMA, num_splits=1)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call(d["out"], d["lse"])
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            call(d["out"], d["lse"])
    for lens in ([64 * 66 + 3, 1500], [640, 64 * 20], [4000, 0]):
        d["seq_lens"].copy_(torch.tensor(lens, dtype=torch.int32))
        out, lse = torch.zeros_like(d["out"]), torch.zeros_like(d["lse"])
        call(out, lse)
        d["out"].zero_()
        d["lse"].zero_()
        torch.cuda.synchronize()
        print("wide, replay T=%d %s" % (T, lens), flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, d["out"]) and torch.equal(lse, d["lse"])
