"""Which blocks the pipelined kernel is built on (no GPU needed): the plan says so, and the generator writes what the plan means."""
import ctypes
import importlib.util
import os
import re

import pytest

from paper_2508_08192_amd import treeattn as ta
from paper_2508_08192_amd.treeattn import Desc

PACED, NARROW, WIDE = 0, 1, 2
MFMA = 2


def _call(rows, lists, tiles):
    """A call of `lists` requests with one KV head and `rows` query rows, in a table of `tiles` tiles and the tree's."""
    T = next(t for t in range(min(rows, 64), 0, -1) if rows % t == 0)
    G, table = rows // T, tiles - 1 + -(-T // 64)
    return (Desc((lists, T, G, 128), ta.TA_BF16), Desc((lists * table, 1, 64, 128), ta.TA_BF16),
            Desc((lists * table, 1, 64, 128), ta.TA_BF16), Desc((lists, table), ta.TA_I32), Desc((lists,), ta.TA_I32),
            Desc((T,), ta.TA_I32), Desc((lists, T, G, 128), ta.TA_BF16), Desc((lists, G, T), ta.TA_F32))


def _plan(rows, lists, tiles, kernel=MFMA, **kw):
    return ta.tree_attn_plan(*_call(rows, lists, tiles), kernel=kernel, **kw)


@pytest.mark.parametrize("rows", [1, 32, 33, 64, 65, 72, 96, 128, 129, 136, 160, 192, 224, 256, 320, 512])
@pytest.mark.parametrize("lists,tiles", [(32, 20), (400, 5)])
def test_only_row_groups_of_up_to_128_rows_are_paced(rows, lists, tiles):
    """The wait in a paced tile costs calls of 129 rows and more 1 to 2 %."""
    p = _plan(rows, lists, tiles)
    assert p["key_split"] == 0 and p["merge_workgroups"] > 0
    assert p["blocks"] == (PACED if rows <= 128 else NARROW), p


@pytest.mark.parametrize("rows", [65, 72, 96, 97, 128, 129, 136, 160, 192, 224, 225, 256, 320, 480, 512])
def test_wide_blocks_only_where_all_waves_have_rows(rows):
    """Otherwise they take up to 1.08 times as long, whatever the length."""
    full = 96 < rows <= 128 or 224 < rows <= 256 or rows == 512
    for lists, tiles in ((16, 4000), (100, 1500), (600, 900)):
        assert _plan(rows, lists, tiles)["blocks"] == (WIDE if full else PACED if rows <= 128 else NARROW), (lists, tiles)


@pytest.mark.parametrize("rows,line,form", [(256, 96, NARROW), (512, 96, NARROW), (128, 96, PACED)])
def test_wide_blocks_only_for_long_shares_of_long_lists(rows, line, form):
    """Tiles per workgroup and per list, both: many short lists in a share leave no steady state."""
    wgs = 256 // -(-rows // 256)
    for lists in (1, 8, 64, 256, 400):
        runs = max(lists, wgs)
        for tiles, want in (((line * runs - 1) // lists, form), (-(-line * runs // lists), WIDE)):
            p = _plan(rows, lists, tiles)
            assert p["kv_workgroups"] == wgs and p["blocks"] == want, (lists, tiles, p)
    assert _plan(rows, 400, line // 2)["blocks"] == form           # (line tiles and more a workgroup)
    assert _plan(rows, 1, 2 * line, num_splits=2)["blocks"] == WIDE and _plan(rows, 1, line, num_splits=2)["blocks"] == form


def test_the_key_split_kernel_has_no_blocks():
    assert _plan(32, 32, 20, kernel=3)["key_split"] == 1 and _plan(32, 32, 20, kernel=3)["blocks"] == 0


def test_key_split_is_zero_or_one_whatever_the_blocks():
    """plan[14] as a caller of the C function reads it: `if (plan[14])`."""
    for rows, lists, tiles, kernel, blocks in ((64, 32, 20, MFMA, PACED), (256, 32, 20, MFMA, NARROW), (256, 16, 4000, MFMA, WIDE),
                                               (32, 32, 20, 3, 0), (256, 16, 4000, 1, 0)):
        descs = [ta._desc(x) for x in _call(rows, lists, tiles)]
        plan, opts = (ctypes.c_int64 * 16)(), ta._opts(None, 0, kernel, None, None, 0)
        args = [ctypes.byref(d) for d in descs] + [ctypes.byref(opts), 256]
        assert ta.load_library().tree_attn_plan(*args, plan) == ta.TA_OK
        assert plan[14] == (1 if kernel == 3 else 0), list(plan)
        assert ta.load_library().tree_attn_plan_blocks(*args) == blocks
    args[-2] = ctypes.byref(ta._opts(None, 0, 9, None, None, 0))
    assert ta.load_library().tree_attn_plan_blocks(*args) == ta.TA_ERR_OPTS


def _steady_loop(text, struct):
    """The lines of a struct's steady-state loop, without the ones behind its branch back."""
    body = text[re.search(r"^struct %s\b" % struct, text, re.M).start():]
    lines = re.findall(r'"([^"\\]*)\\n\\t"', body[body.index(" fast_loop("):body.index("}", body.index(" fast_loop("))])
    return lines[:lines.index("s_cbranch_scc1 1b") + 1]


def test_only_paced_blocks_wait_in_the_steady_state():
    path = os.path.join(os.path.dirname(ta.__file__), "csrc", "gen_sp_block.py")
    spec = importlib.util.spec_from_file_location("gen_sp_block", path)
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    text = gen.generate()
    paced, narrow, wide = (_steady_loop(text, s) for s in ("SpPaced", "SpNarrow", "SpWide"))
    assert "s_nop 7" not in narrow and "s_nop 7" not in wide
    assert paced.count("s_nop 7") == 8 and len(narrow) > 400              # two tiles; else they are the same work:
    assert sorted(x for x in paced if x[0] == "v" or x[:2] == "ds") == sorted(x for x in narrow if x[0] == "v" or x[:2] == "ds")
