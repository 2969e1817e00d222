"""tree_attn_compact and tree_attn_append bit for bit where a row is moved in 16-byte pieces and where it cannot be, and
where the moved rows fill one phase of the workgroup's registers exactly, by one column too many, or several times."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pool(shape, dtype, shift, seed):
    """A cache whose rows start `shift` elements past an aligned address."""
    import torch
    bits = torch.int16 if dtype == "bf16" else torch.int32
    g = torch.Generator().manual_seed(seed)
    n = int(np.prod(shape))
    flat = torch.randint(-30000, 30000, (n + shift,), generator=g, dtype=bits).cuda()
    return flat.view(torch.bfloat16 if dtype == "bf16" else torch.float32)[shift:].view(shape), bits


# 4096 pieces are held at once: T 16, Hkv 8, D 128 in bf16 is 16 * 256 = 4096 of them, T 17 leaves columns for a second
# phase, T 64 in fp32 with D 256 has 64 * 1024 in sixteen phases
@pytest.mark.parametrize("dtype,D,Hkv,T,ps,shift", [
    ("bf16", 128, 8, 16, 16, 0), ("bf16", 128, 8, 17, 32, 0), ("f32", 256, 8, 64, 64, 0), ("bf16", 8, 1, 1, 0, 0),
    ("bf16", 128, 2, 16, 16, 1), ("bf16", 20, 3, 33, 5, 0), ("f32", 6, 2, 12, 0, 0), ("f32", 64, 2, 8, 16, 2)])
def test_rows_move_whole_whatever_their_alignment(dtype, D, Hkv, T, ps, shift):
    import torch
    from oracle import kv_compact_oracle as KC
    from paper_2508_08192_amd import treeattn as ta
    rng = np.random.default_rng(7)
    B, lens = 3, np.int32([3, 0, 41])
    per = ps or 128
    pages = [-(-(int(L) + T) // per) for L in lens]
    table, n_pages = None, B
    if ps:
        ids = rng.permutation(sum(pages) + 2)
        n_pages, table, at = len(ids), np.zeros((B, max(pages)), np.int32), 0
        for b, k in enumerate(pages):
            table[b, :k] = ids[at:at + k]
            at += k
    kc, bits = _pool((n_pages, Hkv, per, D), dtype, shift, 1)
    vc, _ = _pool((n_pages, Hkv, per, D), dtype, shift, 2)
    k_new, _ = _pool((B, T, Hkv, D), dtype, shift, 3)
    v_new, _ = _pool((B, T, Hkv, D), dtype, shift, 4)
    raw = np.int16 if dtype == "bf16" else np.int32

    def host(t):
        return t.view(bits).cpu().numpy().copy()
    k0, v0, kn, vn = host(kc), host(vc), host(k_new), host(v_new)
    for b in range(B):
        for i in range(T):
            pos = int(lens[b]) + i
            page, slot = (int(table[b, pos // per]), pos % per) if ps else (b, pos)
            k0[page, :, slot] = kn[b, i]
            v0[page, :, slot] = vn[b, i]
    sl = torch.from_numpy(lens).cuda()
    pt = None if table is None else torch.from_numpy(table).cuda()
    print("pieces %s D=%d Hkv=%d T=%d ps=%d shift=%d" % (dtype, D, Hkv, T, ps, shift), flush=True)
    ta.tree_attn_append(k_new, v_new, kc, vc, pt, sl)
    torch.cuda.synchronize()
    assert np.array_equal(host(kc), k0) and np.array_equal(host(vc), v0)

    acc = np.zeros((B, T), np.int32)
    n = np.int32([T, max(1, T // 2), T])
    for b in range(B):
        acc[b] = rng.permutation(T)                     # sources are also destinations
    k_ref, v_ref, lens_ref, skipped = KC.kv_compact_oracle(k0, v0, table, lens, acc, n, T)
    assert not skipped
    out = torch.empty_like(sl)
    ta.tree_attn_compact(kc, vc, pt, sl, torch.from_numpy(acc).cuda(), torch.from_numpy(n).cuda(), T, seq_lens_out=out)
    torch.cuda.synchronize()
    assert np.array_equal(host(kc), k_ref.view(raw)) and np.array_equal(host(vc), v_ref.view(raw))
    assert np.array_equal(out.cpu().numpy(), lens_ref)
    assert ta.tree_attn_last_status() == 0


@pytest.mark.parametrize("dtype,ps", [("bf16", 16), ("f32", 8), ("bf16", 0)])
def test_a_path_longer_than_the_tree(dtype, ps):
    """Nodes may repeat, so a path can be longer than the tree: its rows go to positions behind the tree's, through pages of
    their own; where those do not exist, or the table ends before them, the request is left alone.  The entries behind a
    path's end name no nodes at all."""
    import torch
    from oracle import kv_compact_oracle as KC
    from paper_2508_08192_amd import treeattn as ta
    B, T, A, Hkv, D = 5, 4, 40, 2, 64
    lens = np.int32([3, 0, 41, 30, 50])
    per = ps or 128
    rng = np.random.default_rng(3)
    table, n_pages = None, B
    if ps:
        n_pages = B * (96 // ps)
        table = rng.permutation(n_pages).astype(np.int32).reshape(B, -1)
        table[3, 48 // ps] = n_pages + 1                # request 3's positions from 48 on; its tree ends at 34
    kc, bits = _pool((n_pages, Hkv, per, D), dtype, 0, 1)
    vc, _ = _pool((n_pages, Hkv, per, D), dtype, 0, 2)
    raw = np.int16 if dtype == "bf16" else np.int32

    def host(t):
        return t.view(bits).cpu().numpy().copy()
    n = np.int32([40, 1, 6, 19, 40])
    capacity = 96 if ps else per
    lens[4] = capacity - T                              # room for the tree, none for the path
    acc = rng.integers(0, T, size=(B, A)).astype(np.int32)
    for b in range(B):
        acc[b, n[b]:] = 1 << 30
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    healthy = [0, 1, 2] if ps else [0, 1, 2, 3]
    k_ref, v_ref, lens_ref, skipped = KC.kv_compact_oracle(host(kc), host(vc), None if table is None else table, lens, acc,
                                                           np.where(np.isin(np.arange(B), healthy), n, 0).astype(np.int32), T)
    assert not skipped
    ta.tree_attn_last_status()
    print("path longer than the tree %s ps=%d" % (dtype, ps), flush=True)
    ta.tree_attn_compact(kc, vc, None if table is None else torch.from_numpy(table).cuda(), torch.from_numpy(lens).cuda(),
                         torch.from_numpy(acc).cuda(), torch.from_numpy(n).cuda(), T, seq_lens_out=out)
    status = ta.tree_attn_last_status()
    assert status == ta.TA_STATUS_BAD_SEQLEN | (ta.TA_STATUS_BAD_PAGE if ps else 0)
    assert np.array_equal(host(kc), k_ref.view(raw)) and np.array_equal(host(vc), v_ref.view(raw))
    assert np.array_equal(out.cpu().numpy(), lens_ref)
