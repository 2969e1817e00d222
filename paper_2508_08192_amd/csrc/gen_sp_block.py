#!/usr/bin/env python3
"""Writes ta_sp_block.inc: the per-tile blocks of the 256-row KV-pass kernel as single inline-asm statements.

    python gen_sp_block.py > ta_sp_block.inc

One block of tile i holds up to three streams, merged into one in-order instruction sequence so that a wave keeps
the matrix pipe and the vector ALU busy at the same time:

  PV   O^T += V^T(i-1) . P^T(i-1)        16 A fragments, by transposing LDS reads from the row-major V tile (two
                                         ds_read_b64_tr_b16 each)
  S    S^T(i+1) = K(i+1) . Q^T           16 A fragments from the swizzled K tile
  SM   running softmax of S^T(i) -> P(i) about 155 vector instructions

The blocks exist in two forms.  Narrow: v_mfma_f32_32x32x16_bf16, one per fragment (Paced: the same with a wait in every
steady-state tile).  Wide: v_mfma_f32_16x16x32_bf16, two per fragment.  Their 32-deep products move 8 accumulator values per lane
in and out of the register file where the narrow one moves 16, and draw less power for it: in a loop of nothing but products of normal
values this card sustains 1.99 PFLOP/s with them and 1.75 with the narrow ones, 1.77 and 1.57 with the fragments' LDS reads beside them.  But a wave issues 32 instructions more per tile:
4 lists x 8 KV heads of 131072 tokens, 256 rows, busy cycles of a compute unit per tile 3513 narrow and 3740 wide, of a launch
back to back 0.90 M at 1.55 GHz and 0.96 M at 1.67 GHz.  So they are for calls whose clock is what the power allows (the rule
stands in ta_host.cpp): those lists 591 -> 574 us a call, 64 lists of 2048 to 32768 tokens 174.0 -> 169.6, either as a single
call 535 -> 522 and 177.5 -> 178.0.  Narrow and Wide below say how rows, tokens and head-dim columns lie in the lanes.

The large operands live in fixed physical VGPRs that the compiler never sees: the kernel is compiled with
amdgpu_num_vgpr(16), which confines the register allocator to v0..v31 (the attribute counts in units of two on
this target), and everything from v32 up belongs to these blocks from the first to the last of a walk.  (The
softmax addresses single registers of the score and probability tuples, which asm operands cannot express.)

  v[48:111] O (4 x 16)   v[112:143] score buffer A   v[144:175] score buffer B   v[176:191] P   v[192:223] Q
  v[224:247] ring of 6 LDS fragments   v[248:255] softmax temporaries
  v[38:41] v44 v45 v36 v253 V fragment addresses of the current block (one per head-dim block, narrow: four); the last two are
  K fragment addresses once the V fragments are requested   v[46:47] page-lookup temporaries
  v34 v35 v37 v42 further softmax temporaries   v43 alpha   v250 bf16 (1, 1)   v[251:252] references of the lane's rows
  v[32:33] lane constants: LDS offsets of the lane's V fragments and K fragments

V fragments.  The V tile lies in LDS as it lies in the cache, one 256-byte row per token, with the 32-byte blocks of
a row XOR-placed by (token & 7).  ds_read_b64_tr_b16 works on groups of 16 lanes: lane j names 8 bytes (four
elements E_j[0..3]) and lane i receives E_{4k + i/4}[i % 4] for k = 0..3.  With lanes 4k..4k+3 of a group on the four
8-byte pieces of one 32-byte block of token k, lane i receives head-dim column (16 * block + i) of four tokens: the
A operand of the second product (rows = head-dim columns, contraction = tokens) without any re-layout.  The token
sets (narrow: 16kb + 4hf + {0..3}, then + 8, for the lane's half hf of the wave; wide: 32kb + 4g + {0..3}, then + 16, for its
group g) follow the contraction slots the probabilities occupy after the first product.  Four groups on one block of sixteen
token rows (wide) meet no bank conflict; two on two neighbouring blocks of eight (narrow) lose a third of the LDS cycles to them
(LDS busy 28 % of the cycles instead of 44 %).

Small helpers move values between the two worlds: zero_o, load_q, set_bases, scale_o, row_totals, mask_A/B, put_q15.

S^T(i) and S^T(i+1) alternate between buffers A and B, so every block exists in an "A current" and a "B current"
flavour.  P has one buffer: the PV MFMAs, which read P(i-1), come first in program order and the conversion that
overwrites a part of P is emitted only after the last MFMA reading that part (MFMA reads its A/B operands
when it issues).  A fragment is requested DIST fragments before its MFMAs.

Running softmax in base 2 with a lazily moved reference M (scaled units): M changes only when the tile maximum
exceeds M + 4, so P <= 16 and the rescaling of O is rare.  So is the exchange of maxima between the lanes of a row, which
only happens in a tile where some lane holds a score above M + 4, in lines that stand behind the block (with the exchange in every
tile the narrow blocks take 0.5 to 1.4 % longer where the vector ALU counts, 256 rows and 8 or 4 tiles per workgroup 37.2 -> 36.9 and
31.9 -> 31.5 us a call).  Two row sums are
kept: l of the fp32 probabilities (for the log-sum-exp) and l2 of their bf16 roundings, which are the weights the PV
product actually applies -- normalising O by l2 makes the output an exact weighted mean of V rows.  (With l alone
the output of a row that sees two or three keys is off by the rounding of their weights, up to 0.4 % of a value.)
"""
O, SA, SB, P, Q, FR, TMP = 48, 112, 144, 176, 192, 224, 248
NF = 6
DIST = NF - 1
TM_A, TM_B, ONES, M1, M0, T_TK, PS0, PS1 = (TMP + i for i in range(8))   # M0, M1: references of the lane's two rows

X0, X1, X2, X3 = 34, 35, 37, 42   # more softmax temporaries: a dependent vector instruction issues 9 clocks after
                           # its producer, an independent one after 5, so maxima and sums run as four chains
PT0, PT1 = 46, 47          # page lookup of the fast blocks: LDS address of the page id, the id itself
VA_BASE, KA_BASE, KADDR = 32, 33, 36   # lane constants and the K fragment address of the current block
RL = (38, 39, 40, 41, 44, 45, KADDR, T_TK)   # V fragment addresses of the current block, head-dim blocks 0..7
AL = 43                    # alpha of the lane's own row, where a reference has moved
S_CMP = 90                 # s[90:91]: lane mask of "the reference moves" (a select on an SGPR mask is a plain
                           # vector instruction; the same select on VCC costs four times as much on this chip)


def v(n):
    return "v%d" % n


def vr(n, k):
    return "v[%d:%d]" % (n, n + k - 1)


def frag(r):
    return FR + 4 * (r % NF)


class Narrow:
    """v_mfma_f32_32x32x16_bf16: a lane holds one query row, lane & 31, with 4 * (lane >> 5) + {0..3} of every eight tokens
    or head-dim columns."""
    name, rows, pace = "SpNarrow", 1, 0                   # rows of a lane, waits in its steady-state tiles
    # four scores of one row at a time: (row, score registers, P registers, last PV fragment multiplied with these)
    quads = [(0, [4 * g + k for k in range(4)], [2 * g, 2 * g + 1], 4 * (g // 2) + 3) for g in range(8)]
    # the row of O's register quads (head-dim columns in ascending order per row), and where one goes in the staging block:
    # (xor, offset) on the address of the first
    out_row = [0] * 16
    out_at = [(c << 4, 0) for c in range(16)]
    q_loads = [(0, 4 * k, 32 * k) for k in range(8)]      # (row, register, byte offset)
    # of a score register: row, high half of the tile's mask?, bit
    mask_bits = [(0, t >> 4, 8 * (t % 16 // 4) + t % 4) for t in range(32)]

    @staticmethod
    def across_row(a, b, op):
        """Register a: op over the lanes of the row."""
        return ["v_mov_b32 %s, %s" % (v(b), v(a)), "s_nop 1", "v_permlane32_swap_b32 %s, %s" % (v(a), v(b)), "s_nop 1",
                "%s %s, %s, %s" % (op, v(a), v(a), v(b))]

    @staticmethod
    def for_rows(a, b):
        """A value of the lane's own row in register a: for each of its rows (a, b)."""
        return []

    @staticmethod
    def steps(has_pv, has_s, sn, sva, ska):
        out = []
        mfma = "v_mfma_f32_32x32x16_bf16 %s, %s, %s, %s"
        for r in range(16 if has_pv else 0):
            kb, db = r >> 2, r & 3
            f = frag(len(out))
            rd = []
            if kb == 0:
                rd.append(("v_add_u32 %s, %s, %s" % (v(RL[0]), sva, v(VA_BASE)) if db == 0 else
                           "v_xor_b32 %s, %d, %s" % (v(RL[db]), 64 * db, v(RL[0])), False))     # see V tile layout
            rd += [("ds_read_b64_tr_b16 %s, %s offset:%d" % (vr(f, 2), v(RL[db]), kb * 4096), True),
                   ("ds_read_b64_tr_b16 %s, %s offset:%d" % (vr(f + 2, 2), v(RL[db]), kb * 4096 + 2048), True)]
            dst = vr(O + 16 * db, 16)
            out.append((rd, [mfma % (dst, vr(f, 4), vr(P + 4 * kb, 4), dst)]))
        for r in range(16 if has_s else 0):
            kk, tb = r >> 1, r & 1
            f = frag(len(out))
            rd = []
            if r == 0:
                rd.append(("v_add_u32 %s, %s, %s" % (v(KADDR), ska, v(KA_BASE)), False))
            elif tb == 0:
                rd.append(("v_xor_b32 %s, %d, %s" % (v(T_TK), kk * 32, v(KADDR)), False))
            rd.append(("ds_read_b128 %s, %s offset:%d" % (vr(f, 4), v(KADDR) if kk == 0 else v(T_TK), tb * 8192), True))
            dst = vr(sn + 16 * tb, 16)
            out.append((rd, [mfma % (dst, vr(f, 4), vr(Q + 4 * kk, 4), "0" if kk == 0 else dst)]))
        return out


class Paced(Narrow):
    """The narrow blocks with a wait of four s_nop 7 early in every steady-state tile, for row groups of up to 128 rows, where at
    least half of the waves only move tiles.  128 rows without it: 0.97 to 1.0 of the time back to back, and single calls after
    a copy, which run at a higher clock, 0.97 to 1.01 on four cards, but 1.07 to 1.28 on a fifth (16 lists of 49152 tokens 88.5 us
    with it, 105.1 without).  32 and 64 rows: both within 1 %.  With more rows the waves wait for the products and it only costs:
    time with it over that without, back to back and single, 136 to 192 rows 1.0 to 1.02 and 1.0 to 1.04, 224 to 512 rows 1.0 to
    1.01 and 1.0 to 1.02."""
    name, pace = "SpPaced", 4


class Wide:
    """v_mfma_f32_16x16x32_bf16: a lane holds two query rows, (lane & 15) + 16 rb, with 4 * (lane >> 4) + {0..3} of every
    sixteen tokens or head-dim columns.  What there is one of per row (the reference while it moves, alpha, scales) sits in
    the lane's own row, (lane & 15) + 16 * (lane >> 5): a permlane32 swap of the two rows' registers is at once the exchange
    between the wave's halves and the move to that place, and the same swap of a register and its copy brings both rows'
    values back."""
    name, rows, pace = "SpWide", 2, 0

    quads = [(rb, [8 * tb + 4 * rb + k for k in range(4)], [8 * (tb // 2) + 4 * rb + 2 * (tb & 1) + h for h in range(2)],
              8 * (tb // 2) + 7) for tb in range(4) for rb in range(2)]
    out_row = [c & 1 for c in range(16)]
    out_at = [((c >> 1) << 5, 4096 * (c & 1)) for c in range(16)]
    q_loads = [(rb, 16 * rb + 4 * k, 64 * k) for rb in range(2) for k in range(4)]
    mask_bits = [(t >> 2 & 1, t >> 4, 16 * (t >> 3 & 1) + t % 4) for t in range(32)]

    @staticmethod
    def across_row(a, b, op):
        """Registers a and b, values of the lane's two rows: a = op over the lanes of its own row."""
        return ["s_nop 1", "v_permlane32_swap_b32 %s, %s" % (v(a), v(b)), "s_nop 1", "%s %s, %s, %s" % (op, v(a), v(a), v(b)),
                "v_mov_b32 %s, %s" % (v(b), v(a)), "s_nop 1", "v_permlane16_swap_b32 %s, %s" % (v(a), v(b)), "s_nop 1",
                "%s %s, %s, %s" % (op, v(a), v(a), v(b))]

    @staticmethod
    def for_rows(a, b):
        return ["v_mov_b32 %s, %s" % (v(b), v(a)), "s_nop 1", "v_permlane32_swap_b32 %s, %s" % (v(a), v(b)), "s_nop 1"]

    @staticmethod
    def steps(has_pv, has_s, sn, sva, ska):
        out = []
        mfma = "v_mfma_f32_16x16x32_bf16 %s, %s, %s, %s"
        for r in range(16 if has_pv else 0):
            kb, db = r >> 3, r & 7
            f = frag(len(out))
            rd = []
            if kb == 0:
                rd.append(("v_add_u32 %s, %s, %s" % (v(RL[0]), sva, v(VA_BASE)) if db == 0 else
                           "v_xor_b32 %s, %d, %s" % (v(RL[db]), 32 * db, v(RL[0])), False))
            rd += [("ds_read_b64_tr_b16 %s, %s offset:%d" % (vr(f, 2), v(RL[db]), kb * 8192), True),
                   ("ds_read_b64_tr_b16 %s, %s offset:%d" % (vr(f + 2, 2), v(RL[db]), kb * 8192 + 4096), True)]
            dst = [vr(O + 8 * db + 4 * rb, 4) for rb in range(2)]
            out.append((rd, [mfma % (dst[rb], vr(f, 4), vr(P + 8 * kb + 4 * rb, 4), dst[rb]) for rb in range(2)]))
        for r in range(16 if has_s else 0):
            kk, tb = r >> 2, r & 3
            f = frag(len(out))
            rd = []
            if r == 0:
                rd.append(("v_add_u32 %s, %s, %s" % (v(KADDR), ska, v(KA_BASE)), False))
            elif tb == 0:
                rd.append(("v_xor_b32 %s, %d, %s" % (v(T_TK), kk * 64, v(KADDR)), False))
            rd.append(("ds_read_b128 %s, %s offset:%d" % (vr(f, 4), v(KADDR) if kk == 0 else v(T_TK), tb * 4096), True))
            dst = [vr(sn + 8 * tb + 4 * rb, 4) for rb in range(2)]
            out.append((rd, [mfma % (dst[rb], vr(f, 4), vr(Q + 16 * rb + 4 * kk, 4), "0" if kk == 0 else dst[rb])
                             for rb in range(2)]))
        return out


def move_references(sh, moved):
    """The lines that run when some score of the tile exceeds its row's reference by more than 4: rows whose maximum does
    so move on to it, their sums are rescaled, and O will be (`moved` says so, AL holds alpha).  The registers of the
    row sums are free here.  They stand behind the block (see out_of_line): a branch that is taken in every tile costs
    more than the instructions that it skips."""
    a, b, t, x = (v(r) for r in (TM_A, TM_B, PS0, PS1))
    lines = ["s_mov_b32 %s, 1" % moved] + sh.across_row(TM_A, TM_B, "v_max_f32")
    if sh.rows == 2:                                         # the reference of the lane's own row
        lines += ["v_mov_b32 %s, %s" % (t, v(M0)), "v_mov_b32 %s, %s" % (x, v(M1)), "s_nop 1",
                  "v_permlane32_swap_b32 %s, %s" % (t, x), "s_nop 1"]
    else:
        lines += ["v_mov_b32 %s, %s" % (t, v(M0))]
    lines += ["v_mul_f32 %s, %%[c], %s" % (a, a),                     # tile maximum in scaled units
              "v_add_f32 %s, 4.0, %s" % (b, t),
              "v_cmp_gt_f32 s[%d:%d], %s, %s" % (S_CMP, S_CMP + 1, a, b),
              "s_nop 1",                                              # a lane mask written by a vector compare needs two
                                                                      # wait states before a vector instruction reads it
              "v_cndmask_b32 %s, %s, %s, s[%d:%d]" % (v(M0), t, a, S_CMP, S_CMP + 1),   # new reference
              "v_sub_f32 %s, %s, %s" % (v(AL), t, v(M0)),
              "v_exp_f32 %s, %s" % (v(AL), v(AL))]                    # alpha = 2^(M_old - M_new); 1 when unchanged
    lines += sh.for_rows(M0, M1) + ["s_nop 0", "v_mov_b32 %s, %s" % (v(X2), v(AL))] + sh.for_rows(X2, X3)
    for rb in range(sh.rows):
        lines += ["v_mul_f32 %%[%s%d], %%[%s%d], %s" % (w, rb, w, rb, v((X2, X3)[rb])) for w in "lw"]
    return lines


def out_of_line(condition, lines, label):
    """An item that runs `lines` if the condition holds; they stand behind the block's last line (see with_tails)."""
    return dict(t=["s_cbranch_%s %df" % (condition, label), "%d:" % (label + 10)],
                tail=["%d:" % label] + lines + ["s_branch %db" % (label + 10)])


def with_tails(lines, seq):
    tails = [x for it in seq for x in it.get("tail", [])]
    return lines + ["s_branch 1f"] + tails + ["1:"] if tails else lines


def softmax_ops(sh, sc, moved, label):
    """(instruction or list of instructions that stay together, the last of which may be an item of out_of_line; index of
    the PV fragment whose MFMAs must already be issued or -1) in program order.  Scores are taken in pairs of quads, with two
    chains of maxima and sums for either (a dependent vector instruction issues late): the lane's two rows, or two pieces of
    its one."""
    s = lambda n: v(sc + n)
    ops = []
    add = lambda ins, need=-1: ops.append((ins, need))
    pairs = [sh.quads[2 * j:2 * j + 2] for j in range(4)]
    mx = ((TM_A, X0), (TM_B, X1))
    for j in range(4):
        for h in range(2):
            for e in range(2):
                r, sco = v(mx[e][j & 1]), pairs[j][e][1]
                x = (s(sco[2 * h]), s(sco[2 * h + 1]))
                if j < 2 and h == 0:
                    add("v_max_f32 %s, %s, %s" % ((r,) + x))
                else:
                    add("v_max3_f32 %s, %s, %s, %s" % ((r, r) + x))
    mr = (M0, M1) if sh.rows == 2 else (M0, M0)
    # Does a score of this lane exceed its row's reference by more than 4?  Only then the lanes of a row ask each other
    # for the tile's maximum (in every tile: up to 13 instructions more and a chain of 150 clocks).
    if sh.rows == 2:
        add("v_max_f32 %s, %s, %s" % (v(TM_A), v(TM_A), v(X0)))
        add("v_max_f32 %s, %s, %s" % (v(TM_B), v(TM_B), v(X1)))
        add("v_fma_f32 %s, %s, %%[c], -%s" % (v(X0), v(TM_A), v(M0)))
        add("v_fma_f32 %s, %s, %%[c], -%s" % (v(X1), v(TM_B), v(M1)))
        add("v_cmp_lt_f32 s[%d:%d], 4.0, %s" % (S_CMP, S_CMP + 1, v(X0)))
        add(["v_cmp_lt_f32 vcc, 4.0, %s" % v(X1), "s_or_b64 vcc, vcc, s[%d:%d]" % (S_CMP, S_CMP + 1)] +
            [out_of_line("vccnz", move_references(sh, moved), label)])
    else:
        add("v_max_f32 %s, %s, %s" % (v(TM_A), v(TM_A), v(TM_B)))
        add("v_max3_f32 %s, %s, %s, %s" % (v(TM_A), v(TM_A), v(X0), v(X1)))
        add("v_fma_f32 %s, %s, %%[c], -%s" % (v(X0), v(TM_A), v(M0)))
        add(["v_cmp_lt_f32 vcc, 4.0, %s" % v(X0), out_of_line("vccnz", move_references(sh, moved), label)])

    def stage_a(j):                                          # x = 2^(s*c - M) for eight scores, in place
        xs = [(s(q[1][k]), mr[q[0]]) for k in range(4) for q in pairs[j]]
        for x, m in xs:
            add("v_fma_f32 %s, %s, %%[c], -%s" % (x, x, v(m)))
        for x, m in xs:
            add("v_exp_f32 %s, %s" % (x, x))

    ps = ((PS0, X2), (PS1, X3))                              # the row sums
    d2 = ((TM_A, X0), (TM_B, X1))                            # the sums of the rounded values

    def stage_b(j):                                          # row sums and the four packed P registers
        if j == 0:
            for h in range(2):
                for e in range(2):
                    sco = pairs[j][e][1]
                    add("v_add_f32 %s, %s, %s" % (v(ps[e][h]), s(sco[2 * h]), s(sco[2 * h + 1])))
        else:
            for k in range(4):
                for e in range(2):
                    r = v(ps[e][k & 1])
                    add("v_add_f32 %s, %s, %s" % (r, r, s(pairs[j][e][1][k])))
        for h in range(2):
            for e in range(2):
                rb, sco, pr, need = pairs[j][e]
                add("v_cvt_pk_bf16_f32 %s, %s, %s" % (v(P + pr[h]), s(sco[2 * h]), s(sco[2 * h + 1])), need)
        # second row sum, of the rounded values: what the PV product really weighs V with
        for h in range(2):
            for e in range(2):
                r, (rb, sco, pr, need) = v(d2[e][h]), pairs[j][e]
                add("v_dot2_f32_bf16 %s, %s, %s, %s" % (r, v(P + pr[h]), v(ONES), "0" if j == 0 else r), need)

    stage_a(0)
    for j in range(1, 4):
        stage_a(j)
        stage_b(j - 1)
    stage_b(3)
    tot = [(PS0, X2), (PS1, X3), (TM_A, X0), (TM_B, X1)]       # (the dot results: 3 wait states before another reader)
    for a, b in tot:
        add("v_add_f32 %s, %s, %s" % (v(a), v(a), v(b)))
    if sh.rows == 1:
        add("v_add_f32 %s, %s, %s" % (v(PS0), v(PS0), v(PS1)))
        add("v_add_f32 %s, %s, %s" % (v(TM_A), v(TM_A), v(TM_B)))
    for a, t in ((PS0, "l0"), (PS1, "l1"), (TM_A, "w0"), (TM_B, "w1")):
        if int(t[1]) < sh.rows:
            add("v_add_f32 %%[%s], %%[%s], %s" % (t, t, v(a)))
    return ops


def weave(steps, aux, pre):
    """One in-order sequence: the fragment fetches run DIST fragments ahead, `pre` items of `aux` hide the latency of the
    first fetches, the rest of `aux` is spread evenly between the MFMAs.  An aux item with mf = k may not come before
    the MFMAs of fragment k (it overwrites what they read).  Items are dicts: t (text), lds (tag of an LDS operation it
    starts), needs (tags whose data it uses)."""
    n = len(steps)
    seq = []

    def put_reads(r):
        for text, is_lds in steps[r][0]:
            seq.append(dict(t=text, lds=("f", r, len(seq)) if is_lds else None))

    def tags(r):
        return [x["lds"] for x in seq if x.get("lds") and x["lds"][:2] == ("f", r)]

    for r in range(min(DIST, n)):
        put_reads(r)
    vi = 0
    pre = min(pre, len(aux))
    while vi < pre and aux[vi].get("mf", -1) < 0:
        seq.append(aux[vi])
        vi += 1
    pre = vi
    for r in range(n):
        if r + DIST < n:
            put_reads(r + DIST)
        nm = len(steps[r][1])
        for h in range(nm):
            seq.append(dict(t=steps[r][1][h], needs=tags(r) if h == 0 else None))
            target = pre + (len(aux) - pre) * (nm * r + h + 1) // (nm * n)
            while vi < len(aux) and vi < target:
                need = aux[vi].get("mf", -1)
                if need > r or need == r and h < nm - 1:
                    break                             # this part of P is still being read
                seq.append(aux[vi])
                vi += 1
    seq += aux[vi:]
    return seq


def with_waits(seq):
    """Instruction lines of a sequence, with an exact `s_waitcnt lgkmcnt` in front of every item that uses the data of
    an LDS operation (LDS operations return in order: waiting until k younger ones are outstanding is enough)."""
    lines, issued, done = [], [], -1
    for it in seq:
        needs = it.get("needs")
        if needs:
            pos = max(issued.index(x) for x in needs)
            if pos > done:
                lines.append("s_waitcnt lgkmcnt(%d)" % (len(issued) - 1 - pos))
                done = pos
        lines += it["t"] if isinstance(it["t"], list) else [it["t"]]
        if it.get("lds"):
            issued.append(it["lds"])
            assert len(issued) - 1 - done <= 15, "more LDS operations in flight than the counter can hold"
        if it.get("flush"):
            issued, done = [], -1
    return lines


def sm_item(t, need, c="%[c]"):
    put = lambda lines: [x.replace("%[c]", c) for x in lines]
    if isinstance(t, str):
        return dict(t=put([t]), mf=need)
    if isinstance(t[-1], dict):
        return dict(t=put(t[:-1]) + t[-1]["t"], tail=put(t[-1]["tail"]), mf=need)
    return dict(t=put(t), mf=need)


# sums of the probabilities (l) and of their roundings (w) of the lane's two rows, over the lane's own tokens
SUMS_SIG = ["float &l0", "float &l1", "float &w0", "float &w1"]


def sums_out(sh):
    return ['[%s] "+v"(%s)' % (x, x) for x in ("l0", "w0", "l1", "w1")[:2 * sh.rows]]


def block(sh, name, cur, has_pv, has_s, has_sm):
    sc, sn = (SA, SB) if cur == "A" else (SB, SA)
    steps = sh.steps(has_pv, has_s, sn, "%[sva]", "%[ska]")
    ops = softmax_ops(sh, sc, "%[mv]", 2) if has_sm else []
    aux = [sm_item(t, need) for t, need in ops]
    seq = [dict(t="s_nop 7")] + ([dict(t="s_mov_b32 %[mv], 0")] if has_sm else [])
    seq += weave(steps, aux, 10 if steps else len(aux))
    lines = with_waits(seq)
    if has_pv and not has_s:
        lines += ["s_nop 15", "s_nop 7"]              # O is read by ordinary code next
    lines = with_tails(lines, seq)
    outs, ins, sig = [], [], []
    if has_pv:
        ins += ['[sva] "s"(sva)']
        sig += ["uint32_t sva"]
    if has_sm:
        outs += sums_out(sh) + ['[mv] "=&s"(moved)']
        sig += SUMS_SIG + ["uint32_t &moved"]
        ins += ['[c] "s"(c)']
        sig += ["float c"]
    if has_s:
        ins += ['[ska] "s"(ska)']
        sig += ["uint32_t ska"]
    clob = ['"memory"', '"vcc"'] + (['"scc"', '"s%d"' % S_CMP, '"s%d"' % (S_CMP + 1)] if has_sm else [])
    return emit(name, sig, lines, outs, ins, clob)


# Scalar registers of the fast loop (clobbers): constants copied from the operands once, and temporaries.
S_KG, S_VG = 60, 62                     # s[60:61], s[62:63]: cache base of this KV head (K, V)
S_KSP, S_VSP, S_KSS, S_VSS = 64, 65, 66, 67      # page and slot strides in bytes
S_PSHIFT, S_PMASK, S_PCADJ, S_C = 68, 69, 70, 71  # page shift/mask, LDS address of the page-id cache, softmax scale
S_KDST, S_VDST = 72, 73                 # LDS targets of this wave's loads
S_MOVED = 92                            # 1: a reference has moved in this tile
ST = 80                                 # s80..s85 temporaries, s[86:87] K tile base, s[88:89] V tile base


def sg(n):
    return "s%d" % n


def scale_o(sh):
    """O times alpha, which a lane holds for its own row."""
    lines = ["v_mov_b32 %s, %s" % (v(TM_A), v(AL))] + sh.for_rows(TM_A, TM_B)
    lines += ["v_mul_f32 %s, %s, %s" % (v(O + k), v((TM_A, TM_B)[sh.out_row[k // 4]]), v(O + k)) for k in range(64)]
    return lines + ["s_nop 3"]


def fast_step_items(sh, cur, label, helper=False):
    """One tile of the steady state as a list of items (no waits yet): the full block (PV, S, softmax) plus
    everything else the tile needs -- page lookup and addresses of tile i+3, its four cache loads, ring bookkeeping,
    the (rare) rescaling of O, and the closing barrier.
    helper=True leaves the block itself out: a wave without query rows still moves its share of the tiles."""
    sc, sn = (SA, SB) if cur == "A" else (SB, SA)
    steps = [] if helper else sh.steps(True, True, sn, "%[vp]", "%[kn]")
    sm = [] if helper else [sm_item(t, need, sg(S_C)) for t, need in softmax_ops(sh, sc, sg(S_MOVED), label + 2)]
    page_a = [  # page id of the tile to load: LDS read now, used a few MFMAs later; slot part of the addresses
        dict(t="s_lshr_b32 %s, %%[pos], %s" % (sg(ST), sg(S_PSHIFT))),
        dict(t="s_lshl_b32 %s, %s, 2" % (sg(ST), sg(ST))),
        dict(t="s_add_u32 %s, %s, %s" % (sg(ST), sg(ST), sg(S_PCADJ))),
        dict(t="v_mov_b32 %s, %s" % (v(PT0), sg(ST))),
        dict(t="ds_read_b32 %s, %s" % (v(PT1), v(PT0)), lds=("p", 0)),
        dict(t="s_and_b32 %s, %%[pos], %s" % (sg(ST + 1), sg(S_PMASK))),
        dict(t="s_mul_i32 %s, %s, %s" % (sg(ST + 2), sg(ST + 1), sg(S_KSS))),
        dict(t="s_mul_hi_u32 %s, %s, %s" % (sg(ST + 3), sg(ST + 1), sg(S_KSS))),
        dict(t="s_mul_i32 %s, %s, %s" % (sg(ST + 4), sg(ST + 1), sg(S_VSS))),
        dict(t="s_mul_hi_u32 %s, %s, %s" % (sg(ST + 5), sg(ST + 1), sg(S_VSS))),
    ]
    page_b = [
        dict(t="v_readfirstlane_b32 %s, %s" % (sg(ST), v(PT1)), needs=[("p", 0)]),
        dict(t="s_nop 3"),
    ] + [dict(t=x) for x in [
        "s_mul_i32 s86, %s, %s" % (sg(ST), sg(S_KSP)), "s_mul_hi_u32 s87, %s, %s" % (sg(ST), sg(S_KSP)),
        "s_add_u32 s86, s86, %s" % sg(ST + 2), "s_addc_u32 s87, s87, %s" % sg(ST + 3),
        "s_add_u32 s86, s86, %s" % sg(S_KG), "s_addc_u32 s87, s87, %s" % sg(S_KG + 1),
        "s_mul_i32 s88, %s, %s" % (sg(ST), sg(S_VSP)), "s_mul_hi_u32 s89, %s, %s" % (sg(ST), sg(S_VSP)),
        "s_add_u32 s88, s88, %s" % sg(ST + 4), "s_addc_u32 s89, s89, %s" % sg(ST + 5),
        "s_add_u32 s88, s88, %s" % sg(S_VG), "s_addc_u32 s89, s89, %s" % sg(S_VG + 1),
    ]]
    dma = [["s_add_u32 m0, %s, %%[ik]" % sg(S_KDST), "s_nop 0", "global_load_lds_dwordx4 %[koff0], s[86:87] nt"],
           ["s_add_u32 m0, m0, 0x400", "s_nop 0", "global_load_lds_dwordx4 %[koff1], s[86:87] nt"],
           ["s_add_u32 m0, %s, %%[iv]" % sg(S_VDST), "s_nop 0", "global_load_lds_dwordx4 %[voff0], s[88:89] nt"],
           ["s_add_u32 m0, m0, 0x400", "s_nop 0", "global_load_lds_dwordx4 %[voff1], s[88:89] nt"]]

    def ring(reg, wrap):
        return ["s_add_u32 %s, %s, 0x4000" % (reg, reg), "s_cmp_eq_u32 %s, 0x%x" % (reg, wrap),
                "s_cselect_b32 %s, 0, %s" % (reg, reg)]
    # (three K slots: the one after the next tile's is the next to load into; five V slots: the one before the current tile's)
    rings = ["s_mov_b32 %[ik], %[kn]"] + ring("%[kn]", 0xc000) + ["s_mov_b32 %[iv], %[vp]"] + ring("%[vp]", 0x14000) + \
        ["s_add_u32 %[pos], %[pos], 64"]

    aux = list(page_a)
    aux += sm[:12] + [dict(t="s_nop 7")] * (0 if helper else sh.pace)
    aux += page_b
    rest = sm[12:]
    # Loads of tile i+3: one every 10 softmax instructions from the 92nd on (80 behind the first 12); they are not needed
    # before the end of the next block.  Time of a call with them from the 16th, 52nd or 102nd on over that: 64 rows and fewer
    # 0.998 to 1.003; 256 rows (wide), 64 lists of 2048 to 32768 tokens and 4 x 8 of 131072, 0.992, 0.993 to 0.996, 0.995;
    # 448 rows (not paced), 30 lists x 4 heads of 16191 tokens 0.986, 0.990, 0.994.
    di, dma_end = 0, 0
    if helper:
        for x in dma:
            aux += [dict(t=y) for y in x]
        di = 4
    for j, item in enumerate(rest):
        aux.append(item)
        if j >= 80 and (j - 80) % 10 == 0 and di < 4:
            aux += [dict(t=x) for x in dma[di]]
            di += 1
            dma_end = len(aux)                     # the loads read the ring positions ik and iv
    assert di == 4
    if helper:
        aux += [dict(t=x) for x in rings]
    else:
        # ring bookkeeping: behind the last load, one scalar instruction after every fourth other one (a compare and
        # the select that reads its SCC stay neighbours: other scalar work writes SCC too)
        k, i = dma_end, 0
        while i < len(rings):
            grp = rings[i:i + 2] if rings[i].startswith("s_cmp") else rings[i:i + 1]
            at = min(k, len(aux))
            for x in reversed(grp):
                aux.insert(at, dict(t=x))
            i += len(grp)
            k += 4 + len(grp)

    seq = [] if helper else [dict(t="s_nop 3"), dict(t="s_mov_b32 %s, 0" % sg(S_MOVED))]
    seq += weave(steps, aux, 16)
    if not helper:
        # O still holds sums relative to the old reference when it moved (rare): rescale, then close the tile
        item = out_of_line("scc1", ["s_nop 15", "s_nop 7"] + scale_o(sh), label)
        seq += [dict(item, t=["s_cmp_lg_u32 %s, 0" % sg(S_MOVED)] + item["t"])]
    seq += [dict(t="s_waitcnt vmcnt(4)"), dict(t="s_waitcnt lgkmcnt(0)", flush=True), dict(t="s_barrier")]
    return seq


def fast_loop(sh, name, helper=False):
    """`cnt` pairs of steady-state tiles (buffer A current, then buffer B) as one asm statement with its own loop,
    so that the scalar bookkeeping of a tile is issued in the shadow of its matrix and vector work.
    Ring positions (byte offsets): ik, iv = slots the next loads go to; kn = K slot of tile i+1; vp = V slot of
    tile i-1."""
    head = ["s_mov_b64 s[%d:%d], %%[kg]" % (S_KG, S_KG + 1), "s_mov_b64 s[%d:%d], %%[vg]" % (S_VG, S_VG + 1),
            "s_mov_b64 s[%d:%d], %%[sp]" % (S_KSP, S_VSP), "s_mov_b64 s[%d:%d], %%[ss]" % (S_KSS, S_VSS),
            "s_mov_b64 s[%d:%d], %%[pp]" % (S_PSHIFT, S_PMASK), "s_mov_b64 s[%d:%d], %%[pc]" % (S_PCADJ, S_C),
            "s_mov_b64 s[%d:%d], %%[dst]" % (S_KDST, S_VDST), "1:"]
    seq = [dict(t=t) for t in head] + fast_step_items(sh, "A", 2, helper) + fast_step_items(sh, "B", 3, helper)
    seq += [dict(t="s_sub_u32 %[cnt], %[cnt], 1"), dict(t="s_cmp_lg_u32 %[cnt], 0"), dict(t="s_cbranch_scc1 1b")]
    lines = with_tails(with_waits(seq), seq)
    sig = ([] if helper else SUMS_SIG) + ["uint32_t &ik", "uint32_t &iv", "uint32_t &kn", "uint32_t &vp",
           "uint32_t &pos", "uint32_t &cnt", "uint64_t kg", "uint64_t vg", "uint64_t sp", "uint64_t ss", "uint64_t pp",
           "uint64_t pc", "uint64_t dst", "uint32_t koff0", "uint32_t koff1", "uint32_t voff0", "uint32_t voff1"]
    outs = ([] if helper else sums_out(sh)) + \
           ['[%s] "+s"(%s)' % (x, x) for x in ("ik", "iv", "kn", "vp", "pos", "cnt")]
    ins = ['[%s] "s"(%s)' % (x, x) for x in ("kg", "vg", "sp", "ss", "pp", "pc", "dst")] + \
          ['[%s] "v"(%s)' % (x, x) for x in ("koff0", "koff1", "voff0", "voff1")]
    clob = ['"memory"', '"vcc"', '"scc"'] + ['"s%d"' % i for i in list(range(60, 74)) + list(range(80, 93))]
    return emit(name, sig, lines, outs, ins, clob)


def emit(name, sig, lines, outs, ins, clob):
    code = ["static __device__ __forceinline__ void %s(%s)" % (name, ", ".join(sig)), "{", "    asm volatile("]
    for ln in lines:
        code.append('        "%s\\n\\t"' % ln)
    code.append("        : " + ", ".join(outs))
    code.append("        : " + ", ".join(ins))
    code.append("        : " + ", ".join(clob) + ");")
    code.append("}")
    return "\n".join(code)


def helpers(sh):
    out = []
    # O = 0, references at -inf, the constant of the row sums.  Naming v255 as clobbered makes the
    # compiler size the kernel's register file for all 256 VGPRs.
    out.append(emit("zero_o", [], ["v_mov_b32 %s, 0" % v(O + k) for k in range(64)] +
                    ["v_mov_b32 %s, 0xff800000" % v(r) for r in (M0, M1)] +
                    ["v_mov_b32 %s, 0x3f803f80" % v(ONES)], [], [], ['"memory"', '"v255"']))      # bf16 (1, 1)
    # Q of the lane's rows straight from global memory into its registers, in 16-byte pieces.
    # Nothing waits here; the caller's next wait on the vector-memory counter covers these loads.
    lines = ["global_load_dwordx4 %s, %%[q%d], off offset:%d" % (vr(Q + r, 4), rb, at) for rb, r, at in sh.q_loads]
    out.append(emit("load_q", ["const void *q0", "const void *q1"], lines, [],
                    ['[q%d] "v"(q%d)' % (rb, rb) for rb in range(sh.rows)], ['"memory"']))
    out.append(emit("set_bases", ["uint32_t va", "uint32_t ka"],
                    ["v_mov_b32 %s, %%%d" % (v(r), k) for k, r in enumerate((VA_BASE, KA_BASE))], [],
                    ['"v"(va)', '"v"(ka)'], ['"memory"']))
    out.append(emit("scale_o", [], ["s_nop 15", "s_nop 7"] + scale_o(sh), [], [], ['"memory"']))
    # Row sums (l0, w0) and reference of the lane's own row, from the lane's sums over its own tokens.
    if sh.rows == 2:
        lines = ["v_mov_b32 %%[m], %s" % v(M0), "v_mov_b32 %s, %s" % (v(TM_A), v(M1)), "s_nop 1",
                 "v_permlane32_swap_b32 %[l0], %[l1]", "v_permlane32_swap_b32 %[w0], %[w1]",
                 "v_permlane32_swap_b32 %%[m], %s" % v(TM_A), "s_nop 1",
                 "v_add_f32 %[l0], %[l0], %[l1]", "v_add_f32 %[w0], %[w0], %[w1]"]
    else:
        lines = ["v_mov_b32 %%[m], %s" % v(M0)]
    swap = "v_permlane%d_swap_b32" % (16 * (3 - sh.rows))
    lines += ["v_mov_b32 %s, %%[l0]" % v(TM_A), "v_mov_b32 %s, %%[w0]" % v(TM_B), "s_nop 1",
              "%s %%[l0], %s" % (swap, v(TM_A)), "%s %%[w0], %s" % (swap, v(TM_B)), "s_nop 1",
              "v_add_f32 %%[l0], %%[l0], %s" % v(TM_A), "v_add_f32 %%[w0], %%[w0], %s" % v(TM_B)]
    out.append(emit("row_totals", SUMS_SIG + ["float &m"], lines, sums_out(sh) + ['[m] "=&v"(m)'], [], ['"memory"']))
    # Scores whose bit is clear become -inf: lo, hi = the bits of tokens 0..31 and 32..63 for the lane's row 0 or 1,
    # shifted down by the lane's first token.
    for cur, base in (("A", SA), ("B", SB)):
        lines = ["s_nop 15", "s_nop 7", "v_mov_b32 %s, 0xff800000" % v(TMP)]
        for t, (rb, hi, bit) in enumerate(sh.mask_bits):
            x = v(base + t)
            lines.append("v_and_b32 %s, 0x%x, %%[%s%d]" % (v(TMP + 1), 1 << bit, ("lo", "hi")[hi], rb))
            lines.append("v_cmp_eq_u32 vcc, 0, %s" % v(TMP + 1))
            lines.append("v_cndmask_b32 %s, %s, %s, vcc" % (x, x, v(TMP)))
        words = ["lo0", "hi0", "lo1", "hi1"]
        out.append(emit("mask_" + cur, ["uint32_t " + x for x in words], lines, [],
                        ['[%s] "v"(%s)' % (x, x) for x in words[:2 * sh.rows]], ['"memory"', '"vcc"']))
    # Epilogue: the lane's 64 values of O (its part of its rows) become 16-bit fixed point with one scale per
    # row -- value = scale * int16, scale = inv * (largest magnitude of the row) / 32767 -- and go to the row-major
    # staging block in LDS, 256 bytes per row, four values (8 bytes) at a time: out_at on the byte address a0 of the
    # first (the caller folds row, the lane's columns and chunk swizzle into it).  The rounding to int16 is the
    # "add 1.5 * 2^23" trick: the low 16 bits of the sum are the rounded value in two's complement.
    # inv and sc are values of the lane's own row; sc comes back NaN when that row holds a NaN (the sum of its values is
    # one then).
    T0, T1, T2, T3, AM, SU, XS, AM1 = (TMP + i for i in range(8))
    # two chains of maxima and two of sums: the lane's two rows, or the halves of its one
    am, su = (AM, AM1), (SU, XS)
    val = [[], []]
    for c in range(16):
        val[sh.out_row[c] if sh.rows == 2 else c & 1] += [v(O + 4 * c + k) for k in range(4)]
    lines = ["s_nop 15", "s_nop 7"]
    for e in range(2):
        lines += ["v_max3_f32 %s, |%s|, |%s|, |%s|" % ((v(am[e]),) + tuple(val[e][:3])),
                  "v_add_f32 %s, %s, %s" % ((v(su[e]),) + tuple(val[e][:2]))]
    for k in range(2, 32):
        for e in range(2):
            if k == 31:
                lines.append("v_max_f32 %s, %s, |%s|" % (v(am[e]), v(am[e]), val[e][k]))
            elif k % 2 == 1:
                lines.append("v_max3_f32 %s, %s, |%s|, |%s|" % (v(am[e]), v(am[e]), val[e][k], val[e][k + 1]))
            lines.append("v_add_f32 %s, %s, %s" % (v(su[e]), v(su[e]), val[e][k]))
    if sh.rows == 1:
        lines += ["v_max_f32 %s, %s, %s" % (v(AM), v(AM), v(AM1)), "v_add_f32 %s, %s, %s" % (v(SU), v(SU), v(XS))]
    lines += sh.across_row(AM, AM1, "v_max_f32") + sh.across_row(SU, XS, "v_add_f32")
    lines += ["v_mul_f32 %s, %%[inv], %s" % (v(T0), v(AM)),
              "v_mul_f32 %%[sc], 0x38000100, %s" % v(T0),                   # * 1/32767
              "v_cmp_u_f32 vcc, %s, %s" % (v(SU), v(SU)),
              "v_mov_b32 %s, 0x7fc00000" % v(T1),
              "v_cndmask_b32 %%[sc], %%[sc], %s, vcc" % v(T1),
              "v_rcp_f32 %s, %s" % (v(T2), v(AM)),
              "v_cmp_gt_f32 vcc, %s, 0" % v(AM),
              "s_nop 0",
              "v_mul_f32 %s, 0x46fffe00, %s" % (v(T2), v(T2)),              # 32767 / max
              "v_cndmask_b32 %s, 0, %s, vcc" % (v(AM), v(T2)),               # an all-zero row: every value stays 0
              "v_mov_b32 %s, 0x4b400000" % v(SU),                            # 1.5 * 2^23
              "v_mov_b32 %s, 0x05040100" % v(XS)]                            # byte selector: low halves of two registers
    lines += sh.for_rows(AM, AM1)
    for c in range(16):
        for j in range(4):
            lines.append("v_fma_f32 %s, %s, %s, %s" % (v(T0 + j), v(O + 4 * c + j), v(am[sh.out_row[c]]), v(SU)))
        lines.append("v_perm_b32 %s, %s, %s, %s" % (v(O + 2 * c), v(T1), v(T0), v(XS)))
        lines.append("v_perm_b32 %s, %s, %s, %s" % (v(O + 2 * c + 1), v(T3), v(T2), v(XS)))
        lines.append("v_xor_b32 %s, 0x%x, %%[a0]" % (v(T0), sh.out_at[c][0]))
        lines.append("ds_write_b64 %s, v[%d:%d] offset:%d" % (v(T0), O + 2 * c, O + 2 * c + 1, sh.out_at[c][1]))
    lines.append("s_waitcnt lgkmcnt(0)")
    out.append(emit("put_q15", ["float inv", "uint32_t a0", "float &sc"], lines, ['[sc] "=&v"(sc)'],
                    ['[inv] "v"(inv)', '[a0] "v"(a0)'], ['"memory"', '"vcc"']))
    return out


def generate():
    """The whole text of ta_sp_block.inc."""
    out = ["// Generated by gen_sp_block.py -- do not edit."]
    for sh in (Narrow, Wide):
        body = [block(sh, "s_first", "B", False, True, False)]           # S^T(0) into buffer A ("current" B is unused)
        for cur in "AB":
            body.append(block(sh, "full_" + cur, cur, True, True, True))
            body.append(block(sh, "last_" + cur, cur, True, False, True))    # no tile after this one
        body.append(block(sh, "head_A", "A", False, True, True))             # tile 0 when a tile 1 follows
        body.append(block(sh, "only_A", "A", False, False, True))            # tile 0 of a one-tile walk
        body.append(block(sh, "pv", "A", True, False, False))                # drain: the last tile's P . V
        body.append(fast_loop(sh, "fast_loop"))
        body += helpers(sh)
        out.append("struct %s {\n%s\n};" % (sh.name, "\n\n".join(body)))
    out.append("struct %s : %s {\n%s\n};" % (Paced.name, Narrow.name, fast_loop(Paced, "fast_loop")))
    out.append(fast_loop(Narrow, "sp_fast_loop_helper", helper=True))
    return "\n\n".join(out) + "\n"


if __name__ == "__main__":
    import sys
    sys.stdout.write(generate())
