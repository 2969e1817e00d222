// Host logic of libtreeattn: descriptor validation, launch planning and the dispatch table.  Plain C++ with no
// device runtime behind it, so this file also builds with g++ under -fsanitize=address,undefined
// (see build.py: build_host_checked) and every rule in it can be exercised on a machine without a GPU.
// See include/treeattn.h for the contract of every entry point.
#include <initializer_list>
#include <limits.h>
#include <math.h>
#include <string.h>

#include "ta_params.h"

size_t ta_host_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A workspace of at least `bytes` from alloc (null: no room); its size, or 0.  In steps of 32 MB: fewer buffers on the way, and
// large pages whatever the calls before needed (B 32, 32/8 heads, T 16, L 512..8192 after calls of all sizes: 110.3 to 110.8
// us with steps of 1 and 2 MB, 109.2 to 110.0 with this one).  Where that does not fit, what is needed may.
size_t ta_host_grow(size_t bytes, void *(*alloc)(size_t), void **buf)
{
    for (size_t step : {(size_t)32 << 20, (size_t)1 << 20}) {
        const size_t n = ta_host_align_up(bytes, step);
        *buf = alloc(n);
        if (*buf)
            return n;
    }
    return 0;
}

namespace {

bool strides_ok(const ta_tensor *t)
{
    for (int i = 0; i < t->ndim; ++i)
        if (t->stride[i] < 0)
            return false;
    return t->stride[t->ndim - 1] == 1 || t->shape[t->ndim - 1] <= 1;
}

// rows of a dense K/V tensor as the matrix-core kernels load them: 16-byte aligned, strides within 32 bits
bool new_rows_aligned(const ta_tensor *n)
{
    return ((uintptr_t)n->data % 16) == 0 && n->stride[0] % 8 == 0 && n->stride[1] % 8 == 0 && n->stride[2] % 8 == 0 &&
           n->stride[0] < INT32_MAX && n->stride[1] < INT32_MAX;
}

// Do all rows (D elements, the last dimension) start on 16 bytes and end there?
// A dimension of extent 1 has no stride that counts.
bool rows_of_16_bytes(const ta_tensor *t, int64_t D)
{
    const int64_t per16 = t->dtype == TA_BF16 ? 8 : 4;
    if ((uintptr_t)t->data % 16 != 0 || D % per16 != 0)
        return false;
    for (int i = 0; i < t->ndim - 1; ++i)
        if (t->shape[i] > 1 && t->stride[i] % per16 != 0)
            return false;
    return true;
}

int mfma_rows_group(int rows)
{
    // 32 rows per wave; workgroups of 1, 2, 4 or 8 such waves, at most TA_ROW_GROUP rows.
    int grp = 32;
    while (grp < rows && grp < TA_ROW_GROUP)
        grp *= 2;
    return grp;
}

// Section 3.4, "Attention kernel": the split is chosen per batch size and tree size.  First matching row wins.
//   family, rows <=, lists <=, workgroups per CU x4, smallest share, item cost, wide merge from parts, wide max rows
// The pipelined matrix-core kernel runs one workgroup per compute unit (its tile rings fill the LDS).  A partial
// result costs rows * D * 4 bytes written and read again against TA_TILE * D * 4 bytes per tile of keys and values,
// hence the longer smallest shares of the larger row groups; the fixed work of entering a list is worth about eight
// tiles' time there, and seven to eight in the key-split kernel (head_dim 64, L 730..12152 with 40 lists: 21.8 us with a
// cost of 3, 19.8 with 8; one list of 14265 tokens 14.6 and 12.3); nothing for the scalar one.  With few lists cut over the
// whole chip (batch size one) the merge becomes a latency problem and one workgroup per output row is faster from
// 13 partials per list on, while the batch has at most 1024 output rows.
// A single list counts less fixed work: what it adds mostly keeps workgroups idle (8000 tokens, 32 rows: 17.9 us a call
// without any, which leaves shares of one tile, 16.3 with three to fifteen units).
const TADispatchRow kTable[] = {
    {TA_KERNEL_MFMA, 32, 1, 4, 1, 6, 13, 1024},
    {TA_KERNEL_MFMA, 32, INT32_MAX, 4, 1, 9, 13, 1024},
    {TA_KERNEL_MFMA, 64, INT32_MAX, 4, 1, 9, 13, 1024},
    {TA_KERNEL_MFMA, 128, INT32_MAX, 4, 2, 9, 13, 1024},
    {TA_KERNEL_MFMA, 256, INT32_MAX, 4, 4, 9, 13, 1024},
    {TA_KERNEL_MFMA_BASIC, 256, INT32_MAX, 4, 1, 8, 13, 1024},
    {TA_KERNEL_GENERIC, 256, INT32_MAX, 16, 1, 1, 13, 1024},
};
// fp32 on the matrix cores (ta_f32.hip) stands outside the table (a plan names row -1): one workgroup per compute unit and
// row group -- two fit, but what fp32 calls hold is at most a few tiles per unit, and twice as many shares only cost more
// partial results (36 MB: 22.5 us a call against 24.6) -- and a list's fixed work counts one tile (36 MB in 16 lists: 22.5
// against 25.6 us with none and 22.1 with two; 128 lists of up to three tiles 12.7, two: 13.8); a single list counts none
// (three tiles: 11.8 against 13.3 us).
const TADispatchRow kF32Rows[2] = {{TA_KERNEL_GENERIC, TA_F32_ROWS, 1, 4, 1, 1, 13, 1024},
                                   {TA_KERNEL_GENERIC, TA_F32_ROWS, INT32_MAX, 4, 1, 2, 13, 1024}};
constexpr int kTableRows = (int)(sizeof(kTable) / sizeof(kTable[0]));

// Workgroups of the key-split kernel along a share's length when `slices` of them, with 32 or 64 rows each, serve it side by
// side.  These follow each other one grid row apart, and a row of a whole number of XCDs puts them on the same one, where
// the share comes out of the L2 for all but the first (4 lists of 24000 tokens, 160 rows: 50.6 us a call with 51 workgroups
// a row, 31.5 with 48).
int64_t key_split_workgroups(int64_t want, int slices)
{
    if (slices == 1)
        return want;
    const int64_t n = want / slices;
    return n > 8 ? n - n % 8 : n;
}

// Do lists of up to `tiles` tiles go to one workgroup each?  0: no; TA_SOLO_WIDE: eight waves, a workgroup per compute unit;
// TA_SOLO_PAIR: four waves, two workgroups.  What it saves is the merge pass, its launch and the partial results, 4 to 8 us;
// what it costs is that a list is not cut, and the host does not see how long each is.  So the lines lie where the cut is
// no faster whatever the lengths: all equal, evenly spread, one or an eighth of them long and the rest a sixteenth (or one
// token), the long ones anywhere or last.  Below: time over that of the cut, the worst of those, by graph replay; over random
// shapes with T 1 to 64 and 1 to 8 heads per KV head at the line or one or two tiles below it, 516 calls by ten distributions,
// the worst was 1.02 (head_dim 64, a tile above the line, 1.06).
//
// Up to a workgroup per compute unit, the more of them there are the fewer the cut would give each list:
//   bf16, head_dim 128: 1 to 16 workgroups 0.88 to 0.91 at 9 tiles, 32 0.89 at 10 and 1.03 at 12, 64 0.87 at 10 and 1.0 at 12; 128 0.80 at
//     10 and 0.88 at 14 (eight blocks 1.01 at 12), 1.06 at 16; 192 0.84 at 14, 0.95 at 18, 1.12 at 20; 256 0.89 at 20, 0.97 at 29 (four blocks 1.08);
//   head_dim 64: 1 to 16 0.84 to 0.91 at 13, 64 0.87 to 0.95 at 16 and 1.01 at 18, 115 1.06 at 16 with five blocks, 128 0.95 at 18 and 1.04 at 20 (two blocks 1.16 at 23), 192 0.95 at
//     20, 1.01 at 25 and 1.14 at 28, 256 0.92 at 22 and 1.03 at 26 with eight blocks, 0.91 at 33 with one; in blocks of 64 rows 0.76 to 0.96 at 14 and up to
//     1.11 at 16 with 132 workgroups, 0.82 at 16 with 256;
//   fp32, blocks of 16 rows, head_dim 64: one and two workgroups 1.0 at 4 and 1.03 at 5 (a launch less: 10.5 -> 8.8 us where the
//     host sets the pace), 8 to 64 0.96 to 0.99 at 5, 1.12 at 6; 128 0.94 at 5, 1.0 at 6 and 1.07 at 7, 192 0.87 at 6 and 1.11 at 8, 256 0.89 at 8,
//     1.0 at 10, 1.21 at 14;
//   head_dim 128: 1.0 at 3 with one workgroup, 0.83 to 0.85 with more, 64 1.14 at 4; 128 0.95 at 4, 1.04 at 5; 192 0.95 at 5, 1.05 at 6; 256
//     0.89 at 6, 0.99 at 7, 1.04 at 8.
// More workgroups than compute units are dealt out as others end, so one's start should fall into another's stream: four waves
// and half of the LDS each.  One block of rows, head_dim 128: 264 lists 0.90 at 12 tiles, 0.98 at 14, 1.02 at 16; 384 0.97 at 16, 1.04 at 18; 512
// 0.88 at 19, 1.0 at 26 and 1.21 at 33; 1024 0.85 at 19 and 0.99 at 33, but 1080, whose last ones run with most of the chip idle, 1.07 at 22;
// head_dim 64 0.65 to 0.93 there.  Two to eight blocks, which read the keys from the L2 again: up to 512 workgroups 0.64 to 0.80 at
// 5, 0.76 to 0.99 at 10; two blocks and 1024 0.72 at 3, 0.83 at 6.  fp32, eight waves, head_dim 64: 272 lists 0.92 at 7, 384 1.03 at 8; 512 0.91 at 8, 1.07 at 10, 1.77
// at 32; 1024 0.85 at 14 and 1.02 at 20; head_dim 128: 272 0.99 at 3 and 1.09 at 4, 384 0.97 at 5 and 1.06 at 6, 512 0.98 at 5 and 1.10 at 6, 1024 0.93 at
// 7, 1.03 at 8 and 1.18 at 12.
// Not taken: eight waves for longer lists, four and more per compute unit.  0.96 to 1.01 at 40 to 80 tiles with 512 to 2048 lists of
// equal or evenly spread lengths, but 1.04 to 1.68 where one list or an eighth of them is much longer than the rest (1024 lists, 66 tiles:
// 61.2 -> 79.4 us).
int solo_kind(bool f32, int D, int block_rows, int blocks, int64_t lists, int64_t cus, int64_t tiles)
{
    const int64_t wgs = lists * blocks;
    auto line = [&](int64_t least, int64_t base, int64_t rise) {
        const int64_t l = base + rise * wgs / cus;
        return l > least ? l : least;
    };
    if (wgs <= cus) {
        const int64_t limit = f32 ? (D == 64 ? line(5, 1, 7) : line(3, 2, 4))
                              : D == 128 ? line(9, 1, 18) : block_rows > 32 ? 14 : line(13, 12, 8);
        return tiles <= limit ? TA_SOLO_WIDE : 0;
    }
    if (f32) {
        const int64_t limit = D == 64 ? (wgs < 2 * cus ? 7 : wgs < 4 * cus ? 8 : 14) : 2 * wgs < 3 * cus ? 3 : wgs < 4 * cus ? 5 : 7;
        return blocks == 1 && tiles <= limit ? TA_SOLO_WIDE : 0;
    }
    if (block_rows > 32)
        return 0;
    const int64_t one = 2 * wgs < 3 * cus ? 14 : wgs < 2 * cus ? 16 : 18;
    const int64_t more = wgs <= 2 * cus && blocks <= 8 ? 10 : wgs <= 4 * cus && blocks == 2 ? 6 : 0;
    return tiles <= (blocks == 1 ? one : more) ? TA_SOLO_PAIR : 0;
}

int find_row(int family, int rows_grp, int64_t lists)
{
    for (int i = 0; i < kTableRows; ++i)
        if (kTable[i].family == family && rows_grp <= kTable[i].rows_grp_max && lists <= kTable[i].lists_max)
            return i;
    return -1;
}

}  // namespace

const TADispatchRow *ta_host_dispatch_table(int *n_rows)
{
    *n_rows = kTableRows;
    return kTable;
}

int ta_host_merge_rows(const TAParams &p)
{
    return p.merge_kind == TA_MERGE_WIDE ? 1 : p.merge_kind == TA_MERGE_ROW ? 1024 / p.D : TA_MERGE_ROWS;
}

// Everything that can be decided from the descriptors alone.
int ta_host_build_problem(const ta_tensor *q, const ta_tensor *k, const ta_tensor *v, const ta_tensor *pt,
                          const ta_tensor *sl, const ta_tensor *par, const ta_tensor *out, const ta_tensor *lse,
                          const ta_opts *opts, int num_cus, TAProblem *pr)
{
    if (!q || !k || !v || !sl || !par || !out)
        return TA_ERR_NULL;
    if (q->dtype != TA_BF16 && q->dtype != TA_F32)
        return TA_ERR_DTYPE;
    if (k->dtype != q->dtype || v->dtype != q->dtype || out->dtype != q->dtype)
        return TA_ERR_DTYPE;
    if (sl->dtype != TA_I32 || par->dtype != TA_I32 || (pt && pt->dtype != TA_I32) || (lse && lse->dtype != TA_F32))
        return TA_ERR_DTYPE;
    if (q->ndim != 4 || k->ndim != 4 || v->ndim != 4 || out->ndim != 4 || sl->ndim != 1 ||
        (par->ndim != 1 && par->ndim != 2) || (pt && pt->ndim != 2) || (lse && lse->ndim != 3))
        return TA_ERR_RANK;
    // T: nodes of the tree, all of them keys; Tq: the nodes that ask, q_off .. q_off+Tq-1 (all of them by default)
    const int64_t B = q->shape[0], Tq = q->shape[1], Hq = q->shape[2], D = q->shape[3];
    const int64_t T = par->shape[par->ndim - 1], q_off = opts ? opts->q_node_offset : 0;
    const int64_t n_pages = k->shape[0], Hkv = k->shape[1], ps = k->shape[2];
    if (B < 0 || B > TA_MAX_BATCH)
        return TA_ERR_BATCH;
    if (T < 1 || T > TA_MAX_TREE || Tq < 1 || Tq > TA_MAX_TREE)
        return TA_ERR_TREE_SIZE;
    if (Tq > T)
        return TA_ERR_SHAPE;                     // more query nodes than the tree has
    if (q_off < 0 || q_off + Tq > T)
        return TA_ERR_OPTS;
    if (D < 1 || D > TA_MAX_HEAD_DIM)
        return TA_ERR_HEAD_DIM;
    if (Hq < 1 || Hkv < 1 || Hq % Hkv != 0)
        return TA_ERR_HEADS;
    if (Hq > 65535 || ps < 1 || ps > (1 << 30) || n_pages < 0 || n_pages > INT32_MAX)
        return TA_ERR_SHAPE;
    if (k->shape[3] != D)
        return TA_ERR_SHAPE;
    for (int i = 0; i < 4; ++i)
        if (v->shape[i] != k->shape[i] || out->shape[i] != q->shape[i])
            return TA_ERR_SHAPE;
    if (sl->shape[0] != B)
        return TA_ERR_SHAPE;
    if (par->ndim == 2 && par->shape[0] != B)
        return TA_ERR_SHAPE;
    if (lse && (lse->shape[0] != B || lse->shape[1] != Hq || lse->shape[2] != Tq))
        return TA_ERR_SHAPE;
    if (pt && pt->shape[0] != B)
        return TA_ERR_SHAPE;
    if (!pt && n_pages < B)
        return TA_ERR_SHAPE;
    if (!strides_ok(q) || !strides_ok(k) || !strides_ok(v) || !strides_ok(out) || !strides_ok(par) ||
        (pt && !strides_ok(pt)))
        return TA_ERR_STRIDE;
    if (lse)
        for (int i = 0; i < 3; ++i)
            if (lse->stride[i] < 0)
                return TA_ERR_STRIDE;
    if (sl->stride[0] < 0)
        return TA_ERR_STRIDE;
    const int64_t capacity = pt ? pt->shape[1] * ps : ps;
    if (capacity < T)
        return TA_ERR_PAGE_TABLE;
    if (capacity > INT32_MAX)
        return TA_ERR_SHAPE;
    if (B > 0) {
        if (!q->data || !k->data || !v->data || !sl->data || !par->data || !out->data ||
            (pt && !pt->data) || (lse && !lse->data))
            return TA_ERR_NULL;
    }
    int kernel = TA_KERNEL_AUTO, num_splits = 0, item_cost = 0;
    const ta_tensor *kn = nullptr, *vn = nullptr;
    float scale = 0.f;
    void *user_ws = nullptr;
    size_t user_ws_bytes = 0;
    if (opts) {
        if (opts->item_cost < 0 || opts->item_cost > 4096 || opts->reserved != 0 || opts->num_splits < 0 ||
            opts->kernel < TA_KERNEL_AUTO ||
            opts->kernel > TA_KERNEL_MFMA_BASIC)
            return TA_ERR_OPTS;
        kernel = opts->kernel;
        num_splits = opts->num_splits;
        item_cost = opts->item_cost;
        if (opts->tree_masks && (((uintptr_t)opts->tree_masks % 8) != 0 || opts->tree_masks_stride < 0))
            return TA_ERR_OPTS;
        if (opts->kv_start && ((uintptr_t)opts->kv_start % 4) != 0)
            return TA_ERR_OPTS;
        if (opts->status && ((uintptr_t)opts->status % 4) != 0)
            return TA_ERR_OPTS;
        if ((opts->k_new != nullptr) != (opts->v_new != nullptr))
            return TA_ERR_OPTS;
        if (opts->k_new) {
            // the tree tokens' K/V of this step, dense: [B, T, Hkv, D] in the cache's dtype, rows contiguous
            for (const ta_tensor *n : {opts->k_new, opts->v_new}) {
                if (n->dtype != k->dtype)
                    return TA_ERR_DTYPE;
                if (n->ndim != 4)
                    return TA_ERR_RANK;
                if (n->shape[0] != B || n->shape[1] != T || n->shape[2] != Hkv || n->shape[3] != D)
                    return TA_ERR_SHAPE;
                if (!strides_ok(n) || n->stride[3] != 1)
                    return TA_ERR_STRIDE;
                if (B > 0 && !n->data)
                    return TA_ERR_NULL;
            }
            kn = opts->k_new;
            vn = opts->v_new;
        }
        scale = opts->scale;
        user_ws = opts->workspace;
        user_ws_bytes = opts->workspace_bytes;
        if (user_ws && ((uintptr_t)user_ws % 256) != 0)
            return TA_ERR_WORKSPACE;
    }
    if (!(scale > 0.f) || !isfinite(scale))
        scale = 1.0f / sqrtf((float)D);

    int ps_shift = -1;
    for (int s = 0; s <= 30; ++s)
        if (((int64_t)1 << s) == ps)
            ps_shift = s;
    const bool mfma_ok = q->dtype == TA_BF16 && (D == 128 || D == 64) && (!pt || ps_shift >= 0) &&
                         q->stride[2] % 8 == 0 && q->stride[1] % 8 == 0 && q->stride[0] % 8 == 0 &&
                         k->stride[0] % 8 == 0 && k->stride[1] % 8 == 0 && k->stride[2] % 8 == 0 &&
                         v->stride[0] % 8 == 0 && v->stride[1] % 8 == 0 && v->stride[2] % 8 == 0 &&
                         ((uintptr_t)q->data % 16) == 0 && ((uintptr_t)k->data % 16) == 0 &&
                         ((uintptr_t)v->data % 16) == 0 && k->stride[0] < INT32_MAX && k->stride[2] < INT32_MAX &&
                         v->stride[0] < INT32_MAX && v->stride[2] < INT32_MAX && Hq / Hkv <= 256 &&
                         (!kn || (new_rows_aligned(kn) && new_rows_aligned(vn)));
    int basic = kernel == TA_KERNEL_MFMA_BASIC ? 1 : 0;
    if (basic)
        kernel = TA_KERNEL_MFMA;
    // fp32 goes to the matrix cores where rows can be loaded in 16-byte pieces (a call that names the scalar kernel gets it).
    // Rows of k_new and v_new may start anywhere: a call with the write-back folded in runs the kernel of the plain call.
    auto rows16 = [](const ta_tensor *n) {
        return (uintptr_t)n->data % 16 == 0 && n->stride[0] % 4 == 0 && n->stride[1] % 4 == 0 && n->stride[2] % 4 == 0 &&
               n->stride[3] == 1;
    };
    const bool f32_mfma = kernel == TA_KERNEL_AUTO && q->dtype == TA_F32 && (D == 128 || D == 64) && Hq / Hkv <= 256 &&
                          (!pt || ps_shift >= 0) && rows16(q) && rows16(k) && rows16(v);
    if (kernel == TA_KERNEL_MFMA && !mfma_ok)
        return TA_ERR_OPTS;
    const bool auto_kernel = kernel == TA_KERNEL_AUTO;
    if (auto_kernel)
        kernel = mfma_ok ? TA_KERNEL_MFMA : TA_KERNEL_GENERIC;
    if (kernel == TA_KERNEL_MFMA && (D != 128 || B > TA_SP_MAX_BATCH))
        basic = 1;                               // what the pipelined kernel does not take: head_dim 64, very large batches

    TAParams &p = pr->p;
    memset(&p, 0, sizeof p);
    p.rows = (int)(Tq * (Hq / Hkv));
    const int64_t lists = B * Hkv;
    const int64_t tiles_cap = lists * ((capacity - T + TA_TILE - 1) / TA_TILE + 1);
    if (tiles_cap > INT32_MAX)                              // schedule units are counted in 32 bits
        return TA_ERR_SHAPE;
    // Which matrix-core kernel (head_dim 128; a call that names TA_KERNEL_MFMA gets the pipelined one).  The key-split
    // kernel has eight waves computing from the first tile on, the pipelined one as many as there are blocks of 32 rows, but
    // the former keeps 32 rows: it walks the keys again for every further 32.  The line is drawn by `units`, blocks times
    // tiles per compute unit.  The host does not see the lengths, so tiles are counted from what the page table can hold: a
    // table much wider than its requests may give a small batch to the kernel of a larger one.  Beside each line the time
    // of the key-split kernel over the pipelined one's, by units:
    //   one block: 0.85 to 0.98 from two units on, 0.91 to 1.04 below with two lists and more, one list 1.01 to 1.03 up to
    //     one unit and 0.94 at two (in a table of 32768 tokens, contexts of 100 to 1000 and few lists 1.08 to 1.10);
    //   one list of more: 0.95 to 1.0 up to two units, 0.82 to 0.98 from three to seventeen;
    //   two blocks: 0.95 to 1.05 up to three units; above, with a whole number of workgroups per list, lists of equal
    //     length 0.80 to 0.98 (1.05 up to five units), uneven ones 0.94 to 1.03, with sixteen per list and more 0.83 to 1.04;
    //     otherwise 0.91 to 1.10 (28, 48 and 56 lists);
    //   three and four: whole numbers of workgroups and equal lengths 0.83 to 1.02 from seven units on, 0.92 to 1.13 at four
    //     to six; uneven lists 0.99 to 1.03 up to five units, 1.05 to 1.20 from seven to sixteen, with sixteen workgroups per
    //     list and more 0.93 to 1.03 up to ten;
    //   five and more, whose tiles cost the pipelined kernel's eight waves more: 0.73 to 0.98 up to ten units for all lists,
    //     one list 0.80 to 0.97 up to 31, whole numbers and equal lengths 0.80 to 1.0 up to 26, uneven 1.0 to 1.2 from 20 on.
    // One workgroup per list and fewer than two is for none of them: uneven lists then take 1.2 to 1.35 times as long.
    const int slices = (p.rows + 31) / 32;
    const int64_t ks_wg = key_split_workgroups(num_cus, slices);
    const int64_t units = tiles_cap * slices;
    const bool whole = lists > 0 && ks_wg % lists == 0, many = ks_wg >= 16 * lists;
    const bool equal = B == 1 && whole;                     // (the lists of one request are of one length)
    auto within = [&](int64_t from_x2, int64_t to) { return 2 * units > from_x2 * num_cus && units <= to * num_cus; };
    const bool ks_fits = slices == 1 ? lists > 1 || units > num_cus
                         : ks_wg < 2 * lists ? false
                         : lists == 1 ? within(0, 32)
                         : slices > 4 ? within(0, equal ? 28 : 12)
                         : slices == 2 ? (whole || many) && within(7, 16)
                         : equal ? within(13, 16) : many && within(7, 10);
    const bool ks = kernel == TA_KERNEL_MFMA && (basic || (auto_kernel && ks_fits));
    p.basic = ks;
    p.f32_mfma = f32_mfma;
    p.q = q->data; p.k = k->data; p.v = v->data; p.out = out->data;
    p.lse = lse ? (float *)lse->data : nullptr;
    p.page_table = pt ? (const int32_t *)pt->data : nullptr;
    p.seq_lens = (const int32_t *)sl->data;
    p.parent = (const int32_t *)par->data;
    p.q_sb = q->stride[0]; p.q_st = q->stride[1]; p.q_sh = q->stride[2];
    p.o_sb = out->stride[0]; p.o_st = out->stride[1]; p.o_sh = out->stride[2];
    p.k_sp = k->stride[0]; p.k_sh = k->stride[1]; p.k_ss = k->stride[2];
    p.v_sp = v->stride[0]; p.v_sh = v->stride[1]; p.v_ss = v->stride[2];
    if (lse) { p.lse_sb = lse->stride[0]; p.lse_sh = lse->stride[1]; p.lse_st = lse->stride[2]; }
    p.pt_sb = pt ? pt->stride[0] : 0;
    p.par_sb = par->ndim == 2 ? par->stride[0] : 0;
    p.sl_s = sl->stride[0];
    p.B = (int)B; p.T = (int)T; p.Hq = (int)Hq; p.Hkv = (int)Hkv; p.G = (int)(Hq / Hkv); p.D = (int)D;
    p.ps = (int)ps; p.ps_shift = ps_shift; p.capacity = (int)capacity; p.n_pages = (int)n_pages;
    p.q_off = (int)q_off;
    p.g_magic = (1u << 24) / (uint32_t)p.G + 1u;
    p.masks_in = opts ? (const unsigned long long *)opts->tree_masks : nullptr;
    p.masks_sb = opts ? opts->tree_masks_stride : 0;
    p.kv_start = opts ? (const int32_t *)opts->kv_start : nullptr;
    p.status2 = opts ? opts->status : nullptr;
    p.is_bf16 = q->dtype == TA_BF16;
    if (kn) {
        p.kn = kn->data; p.vn = vn->data;
        p.kn_sb = kn->stride[0]; p.kn_st = kn->stride[1]; p.kn_sh = kn->stride[2];
        p.vn_sb = vn->stride[0]; p.vn_st = vn->stride[1]; p.vn_sh = vn->stride[2];
        const int es = p.is_bf16 ? 2 : 4;
        const int per16 = 16 / es;
        auto vec_ok = [&](const void *ptr, int64_t a, int64_t b2, int64_t c) {
            return ((uintptr_t)ptr % 16) == 0 && a % per16 == 0 && b2 % per16 == 0 && c % per16 == 0;
        };
        p.kn_vec = D % per16 == 0 && vec_ok(kn->data, kn->stride[0], kn->stride[1], kn->stride[2]) &&
                   vec_ok(vn->data, vn->stride[0], vn->stride[1], vn->stride[2]) &&
                   vec_ok(k->data, k->stride[0], k->stride[1], k->stride[2]) &&
                   vec_ok(v->data, v->stride[0], v->stride[1], v->stride[2]);
    }
    p.scale_log2e = scale * 1.4426950408889634f;

    // ---- the launch plan: one row of the dispatch table, unless the options fix a value
    TAPlan &pl = pr->plan;
    pl.kernel = kernel;
    const int family = kernel == TA_KERNEL_MFMA ? (basic ? TA_KERNEL_MFMA_BASIC : TA_KERNEL_MFMA) : TA_KERNEL_GENERIC;
    if (kernel == TA_KERNEL_MFMA) {
        // head_dim 64 can keep 64 rows; 32 are faster where the same few tiles fall on a compute unit (time with 32 rows over
        // that with 64: up to four units 0.83 to 1.04, at eight 0.76 to 1.05, at twelve 0.74 to 1.08, one list 0.79 to 0.93,
        // at sixteen 0.74 to 1.18, mostly 1.0 to 1.08), but not with one workgroup per list (equal lists 0.84 to 1.08, uneven
        // ones 1.13 to 1.37) and fewer (1.2 to 1.5)
        p.ks_rows = pl.ks_rows = D == 64 && slices > 1 && !(units <= (int64_t)16 * num_cus && ks_wg >= 2 * lists) ? 64 : 32;
        pl.rows_grp = ks && (basic || slices <= 4) ? p.ks_rows : mfma_rows_group(p.rows);
        pl.threads = 512;
    } else if (f32_mfma) {
        // as few groups of up to 32 rows as hold them, of equal size, so that the scratch holds no more rows than needed
        const int groups = (p.rows + TA_F32_ROWS - 1) / TA_F32_ROWS;
        pl.rows_grp = (p.rows + groups - 1) / groups;
        pl.threads = 256;
    } else {
        pl.rows_grp = p.rows < TA_ROW_GROUP ? p.rows : TA_ROW_GROUP;
        pl.threads = 256;
    }
    pl.n_rg = (p.rows + pl.rows_grp - 1) / pl.rows_grp;
    const int row = f32_mfma ? -1 : find_row(family, pl.rows_grp, lists);
    if (row < 0 && !f32_mfma)
        return TA_ERR_OPTS;                                 // cannot happen: every family ends in a catch-all row
    const TADispatchRow &dr = f32_mfma ? kF32Rows[lists > kF32Rows[0].lists_max] : kTable[row];
    pl.table_row = row;
    pl.item_cost = item_cost > 0 ? item_cost : dr.item_cost;
    p.pad = pl.item_cost - 1;
    if (tiles_cap + lists * p.pad > INT32_MAX)
        return TA_ERR_SHAPE;
    int64_t want = (int64_t)num_cus * dr.wg_per_cu_x4 / 4;
    if (ks)
        want = key_split_workgroups(want, (p.rows + p.ks_rows - 1) / p.ks_rows);
    else if (kernel == TA_KERNEL_MFMA || f32_mfma)
        want /= pl.n_rg;                                    // the row groups of a list run side by side
    if (want < 1)
        want = 1;
    pl.n_wg = (int)(num_splits > 0 ? num_splits : want);
    pl.min_q = num_splits > 0 ? 1 : dr.min_share;
    if (pl.n_wg > tiles_cap)
        pl.n_wg = (int)(tiles_cap > 0 ? tiles_cap : 1);
    pl.n_slots = pl.n_wg + (int)lists;
    p.rows_grp = pl.rows_grp; p.n_rg = pl.n_rg; p.n_wg = pl.n_wg; p.min_q = pl.min_q;
    // The pipelined kernel's wide blocks (16x16x32 products) draw less power and take more instructions.  They are for calls whose
    // clock is what the power allows: all waves of every row group that computes have rows (four of groups of 128, eight of 256),
    // and stay in their steady-state loops, which a run of one list's tiles in one share is for.  Time over that of the narrow blocks,
    // over 4 to 400 lists of equal and evenly spread lengths, by tiles per share or list, whichever are fewer: back to back; with
    // matrix products of a layer's size before each call; single calls after a copy, which run at a higher clock.
    //   256, 240 and 512 rows: 12 tiles 1.0 to 1.05, 0.98 to 1.05, 1.0 to 1.04; 24 0.97 to 1.01, 0.91 to 1.04, 1.0 to 1.05; 48
    //     0.97 to 0.99, 0.92 to 1.01, 0.98 to 1.01; 100 and more 0.96 to 0.99, 0.96 to 1.0, 0.96 to 1.0;
    //   128 and 100 rows: 24 0.98 to 1.02, 0.99 to 1.04, 0.99 to 1.03; 32 0.97 to 0.99, 1.0 to 1.02, 0.99 to 1.0; 48 0.96 to 0.99,
    //     0.95 to 1.02, 0.98 to 1.01; 100 and more 0.95 to 0.98, 0.91 to 1.0, 0.98 to 1.01;
    //   some waves without rows: 136 to 192 rows 0.98 to 1.07 and single 1.01 to 1.08 at any length, 224 single up to 1.06, 320
    //     single 1.0 to 1.05, 96 0.97 to 1.03 and single 0.99 to 1.04; 64 rows 1.02 to 1.03.
    // So 48 tiles are the line.  Tiles are counted from what the page table can hold: twice that many, for lengths spread evenly
    // or a table twice as wide as its requests.  What a window leaves of the tiles the host does not know.
    const bool waves_full = (p.rows - 1) % pl.rows_grp >= pl.rows_grp - 32;
    const bool wide = !p.kv_start && pl.rows_grp > 64 && waves_full &&
                      tiles_cap >= 96 * (lists > pl.n_wg ? lists : (int64_t)pl.n_wg);
    // Otherwise the narrow ones, in row groups of up to 128 rows with a wait in every tile (figures beside Paced in gen_sp_block.py).
    if (kernel == TA_KERNEL_MFMA && !ks)
        p.blocks = wide ? TA_BLOCKS_WIDE : pl.rows_grp > 128 ? TA_BLOCKS_NARROW : TA_BLOCKS_PACED;

    // merge kernel: partials per list the schedule produces on average = the KV pass's workgroups spread over the
    // lists, plus the one boundary each list shares with its neighbour
    const bool out_aligned = ((uintptr_t)out->data % 16) == 0 && p.o_sb % 4 == 0 && p.o_st % 4 == 0 && p.o_sh % 4 == 0;
    p.merge_kind = TA_MERGE_GENERAL;
    if ((D == 128 || D == 64) && out_aligned) {
        const int64_t l1 = lists > 0 ? lists : 1;
        const int64_t parts = (pl.n_wg + l1 - 1) / l1 + 1;
        const bool wide = dr.wide_from_parts > 0 && parts >= dr.wide_from_parts && lists * p.rows <= dr.wide_max_rows;
        p.merge_kind = wide ? TA_MERGE_WIDE : TA_MERGE_ROW;
    }
    // Partial format of the matrix-core kernels: 16-bit fixed point with a scale per row, which halves what the KV pass
    // writes (C3 128.6 -> 125.0 us, p4 215.1 -> 210.2, C2 26.5 -> 24.1; batch-one shapes 1 to 2 us of 35).  The kernels
    // whose inputs may be fp32 keep fp32 partials.
    p.part_q15 = kernel == TA_KERNEL_MFMA ? 1 : 0;
    // With at least two lists per workgroup most lie whole in a share, and their partial results need not be written,
    // merged and read again (its stores need the alignment that the row merge needs): B 128, 32/8 heads, T 8, L 256..4096
    // 206.6 -> 202.5 us a call.  With 16 rows and fewer there is nothing to gain (59.6 and 60.0).
    p.direct = ks && D == 128 && p.rows > 16 && p.merge_kind == TA_MERGE_ROW && lists >= 2 * (int64_t)pl.n_wg;
    if (ks && lists == 1 && num_splits == 0 && p.merge_kind == TA_MERGE_WIDE) {
        const int parts = 8192 / (int)D;                    // (fewer workgroups: see ta_share)
        p.one_parts = pl.n_wg > parts || (D == 128 && pl.n_wg == parts) ? parts : 0;
    }
    // Lists of a few tiles go to one workgroup each (per block of rows), which writes the outputs itself: no schedule, no
    // partial results, no merge pass.  (Its 16- and 8-byte stores need the alignment that the row merge needs.)
    int solo_rows = f32_mfma ? 16 : 32;
    if (!f32_mfma && D == 64 && p.rows > 32 && lists * ((p.rows + 31) / 32) > num_cus && lists * ((p.rows + 63) / 64) <= num_cus)
        solo_rows = 64;
    const int solo_groups = (p.rows + solo_rows - 1) / solo_rows;
    if (auto_kernel && (f32_mfma || kernel == TA_KERNEL_MFMA) && num_splits == 0 && item_cost == 0 && lists > 0 &&
        p.merge_kind != TA_MERGE_GENERAL)
        p.solo = solo_kind(f32_mfma, (int)D, solo_rows, solo_groups, lists, num_cus, tiles_cap / lists);
    pl.merge_kind = p.merge_kind;
    const int mrows = ta_host_merge_rows(p);
    pl.merge_wgs = (int)lists * ((p.rows + mrows - 1) / mrows);

    const size_t rows_total = (size_t)pl.n_slots * pl.n_rg * pl.rows_grp;
    pr->ws_o_bytes = ta_host_align_up(rows_total * D * sizeof(float), 256);
    pr->ws_lse_bytes = ta_host_align_up(rows_total * sizeof(float), 256);
    // (with 16-bit partials: rows_total * 8 bytes of {log-sum-exp, scale} fit into the unused half of the ws_o area)
    pr->ws_ls_off = p.part_q15 ? ta_host_align_up(rows_total * D * 2, 256) : pr->ws_o_bytes;
    p.ls = p.part_q15 ? 2 : 1;
    if (p.solo) {                                           // (a plan keeps the figures of the cut, but for the merge pass)
        p.direct = 0;
        p.ks_rows = solo_rows;
        if (f32_mfma) {
            p.n_rg = solo_groups;
            p.rows_grp = (p.rows + solo_groups - 1) / solo_groups;
        }
        pl.merge_wgs = 0;
    }
    pr->ws_bytes = pr->ws_o_bytes + pr->ws_lse_bytes + ta_host_align_up((size_t)lists * 2 * sizeof(int32_t), 256);
    if (user_ws) {
        if (user_ws_bytes < pr->ws_bytes)
            return TA_ERR_WORKSPACE;
        p.ws_o = (float *)user_ws;
        p.ws_lse = (float *)((char *)user_ws + pr->ws_ls_off);
        p.ws_parts = (int32_t *)((char *)user_ws + pr->ws_o_bytes + pr->ws_lse_bytes);
    }
    return TA_OK;
}

void ta_host_fill_plan(const TAProblem &pr, int64_t plan[16])
{
    for (int i = 0; i < 16; ++i)
        plan[i] = 0;
    plan[0] = pr.plan.kernel;
    plan[1] = pr.plan.n_wg;
    plan[2] = pr.plan.threads;
    plan[3] = TA_TILE;
    plan[4] = pr.plan.n_rg;
    plan[5] = pr.plan.rows_grp;
    plan[6] = pr.plan.n_slots;
    plan[7] = pr.plan.merge_wgs;
    plan[8] = pr.plan.min_q;
    plan[9] = pr.plan.item_cost;
    plan[10] = pr.plan.merge_kind;
    plan[11] = pr.plan.table_row;
    plan[12] = (int64_t)pr.ws_bytes;
    plan[13] = pr.p.part_q15;
    const bool ks = pr.plan.kernel == TA_KERNEL_MFMA && pr.p.basic;
    plan[14] = ks;
    plan[15] = ks ? pr.plan.ks_rows : pr.plan.rows_grp;
}

size_t ta_host_workspace_bytes(int32_t B, int32_t T, int32_t Hq, int32_t Hkv, int32_t D, int32_t dtype, int32_t num_cus)
{
    if (B < 0 || B > TA_MAX_BATCH || T < 1 || T > TA_MAX_TREE || Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || D < 1 ||
        D > TA_MAX_HEAD_DIM || (dtype != TA_BF16 && dtype != TA_F32) || num_cus <= 0)
        return 0;
    // Worst case over the dispatch table: most workgroups per CU of any row, rows padded to the MFMA row group.
    int per_cu_x4 = 4;
    for (int i = 0; i < kTableRows; ++i)
        per_cu_x4 = kTable[i].wg_per_cu_x4 > per_cu_x4 ? kTable[i].wg_per_cu_x4 : per_cu_x4;
    const int rows = T * (Hq / Hkv);
    const int rows_grp = mfma_rows_group(rows);
    const size_t n_rg = (rows + rows_grp - 1) / rows_grp;
    const size_t slots = (size_t)num_cus * per_cu_x4 / 4 + (size_t)B * Hkv;
    const size_t rows_total = slots * n_rg * rows_grp;
    return ta_host_align_up(rows_total * D * sizeof(float), 256) + ta_host_align_up(rows_total * sizeof(float), 256) +
           ta_host_align_up((size_t)B * Hkv * 2 * sizeof(int32_t), 256);
}

int ta_host_check_encode(const ta_tensor *tree_parent, const ta_tensor *masks, int *B_out, int *T_out, int64_t *par_sb)
{
    if (!tree_parent || !masks)
        return TA_ERR_NULL;
    if (tree_parent->dtype != TA_I32 || masks->dtype != TA_U64)
        return TA_ERR_DTYPE;
    if ((tree_parent->ndim != 1 && tree_parent->ndim != 2) || masks->ndim != tree_parent->ndim)
        return TA_ERR_RANK;
    const int nd = tree_parent->ndim;
    const int64_t B = nd == 2 ? tree_parent->shape[0] : 1, T = tree_parent->shape[nd - 1];
    if (T < 1 || T > TA_MAX_TREE)
        return TA_ERR_TREE_SIZE;
    if (B < 0 || B > TA_MAX_BATCH)
        return TA_ERR_BATCH;
    for (int i = 0; i < nd; ++i)
        if (masks->shape[i] != tree_parent->shape[i])
            return TA_ERR_SHAPE;
    if (!strides_ok(tree_parent) || !strides_ok(masks) || (nd == 2 && masks->stride[0] != T && B > 1))
        return TA_ERR_STRIDE;
    if (B > 0 && (!tree_parent->data || !masks->data))
        return TA_ERR_NULL;
    *B_out = (int)B;
    *T_out = (int)T;
    *par_sb = nd == 2 ? tree_parent->stride[0] : 0;
    return TA_OK;
}

int ta_host_check_append(const ta_tensor *kn, const ta_tensor *vn, const ta_tensor *k, const ta_tensor *v,
                         const ta_tensor *pt, const ta_tensor *sl, TAAppend *out)
{
    if (!kn || !vn || !k || !v || !sl)
        return TA_ERR_NULL;
    if ((kn->dtype != TA_BF16 && kn->dtype != TA_F32) || vn->dtype != kn->dtype || k->dtype != kn->dtype ||
        v->dtype != kn->dtype || sl->dtype != TA_I32 || (pt && pt->dtype != TA_I32))
        return TA_ERR_DTYPE;
    if (kn->ndim != 4 || vn->ndim != 4 || k->ndim != 4 || v->ndim != 4 || sl->ndim != 1 || (pt && pt->ndim != 2))
        return TA_ERR_RANK;
    const int64_t B = kn->shape[0], T = kn->shape[1], Hkv = kn->shape[2], D = kn->shape[3], ps = k->shape[2];
    if (B < 0 || B > TA_MAX_BATCH)
        return TA_ERR_BATCH;
    if (T < 1 || T > TA_MAX_TREE)
        return TA_ERR_TREE_SIZE;
    if (D < 1 || D > TA_MAX_HEAD_DIM)
        return TA_ERR_HEAD_DIM;
    for (int i = 0; i < 4; ++i)
        if (vn->shape[i] != kn->shape[i] || v->shape[i] != k->shape[i])
            return TA_ERR_SHAPE;
    if (Hkv < 1 || k->shape[1] != Hkv || k->shape[3] != D || ps < 1 || sl->shape[0] != B || k->shape[0] < 0 ||
        k->shape[0] > INT32_MAX)
        return TA_ERR_SHAPE;
    if (pt ? (pt->shape[0] != B || pt->shape[1] < 1) : k->shape[0] < B)
        return TA_ERR_PAGE_TABLE;
    if (!strides_ok(kn) || !strides_ok(vn) || !strides_ok(k) || !strides_ok(v) || !strides_ok(sl) ||
        (pt && !strides_ok(pt)) || kn->stride[3] != 1 || vn->stride[3] != 1 || k->stride[3] != 1 || v->stride[3] != 1 ||
        (pt && pt->stride[1] != 1))
        return TA_ERR_STRIDE;
    const int64_t capacity = pt ? pt->shape[1] * ps : ps;
    if (capacity < T)
        return TA_ERR_PAGE_TABLE;
    if (capacity > INT32_MAX)
        return TA_ERR_SHAPE;
    if (B > 0 && (!kn->data || !vn->data || !k->data || !v->data || !sl->data || (pt && !pt->data)))
        return TA_ERR_NULL;
    TAAppend &a = *out;
    memset(&a, 0, sizeof a);
    a.k_new = kn->data; a.v_new = vn->data; a.k = k->data; a.v = v->data;
    a.page_table = pt ? (const int32_t *)pt->data : nullptr;
    a.seq_lens = (const int32_t *)sl->data;
    a.kn_sb = kn->stride[0]; a.kn_st = kn->stride[1]; a.kn_sh = kn->stride[2];
    a.vn_sb = vn->stride[0]; a.vn_st = vn->stride[1]; a.vn_sh = vn->stride[2];
    a.k_sp = k->stride[0]; a.k_sh = k->stride[1]; a.k_ss = k->stride[2];
    a.v_sp = v->stride[0]; a.v_sh = v->stride[1]; a.v_ss = v->stride[2];
    a.pt_sb = pt ? pt->stride[0] : 0;
    a.sl_s = sl->stride[0];
    a.B = (int)B; a.T = (int)T; a.Hkv = (int)Hkv; a.D = (int)D; a.ps = (int)ps; a.capacity = (int)capacity;
    a.n_pages = (int)k->shape[0];
    a.elem_bytes = kn->dtype == TA_BF16 ? 2 : 4;
    a.vec = rows_of_16_bytes(kn, D) && rows_of_16_bytes(vn, D) && rows_of_16_bytes(k, D) && rows_of_16_bytes(v, D);
    return TA_OK;
}

int ta_host_check_compact(const ta_tensor *k, const ta_tensor *v, const ta_tensor *pt, const ta_tensor *sl,
                          const ta_tensor *ac, const ta_tensor *na, int32_t tree_size, const ta_tensor *so,
                          TACompact *out)
{
    if (!k || !v || !sl || !ac || !na)
        return TA_ERR_NULL;
    if ((k->dtype != TA_BF16 && k->dtype != TA_F32) || v->dtype != k->dtype || sl->dtype != TA_I32 ||
        ac->dtype != TA_I32 || na->dtype != TA_I32 || (pt && pt->dtype != TA_I32) || (so && so->dtype != TA_I32))
        return TA_ERR_DTYPE;
    if (k->ndim != 4 || v->ndim != 4 || sl->ndim != 1 || ac->ndim != 2 || na->ndim != 1 || (pt && pt->ndim != 2) ||
        (so && so->ndim != 1))
        return TA_ERR_RANK;
    const int64_t B = ac->shape[0], A = ac->shape[1], Hkv = k->shape[1], D = k->shape[3], ps = k->shape[2];
    const int64_t T = tree_size;
    if (B < 0 || B > TA_MAX_BATCH)
        return TA_ERR_BATCH;
    if (T < 1 || T > TA_MAX_TREE || A < 1 || A > TA_MAX_TREE)
        return TA_ERR_TREE_SIZE;
    if (D < 1 || D > TA_MAX_HEAD_DIM)
        return TA_ERR_HEAD_DIM;
    for (int i = 0; i < 4; ++i)
        if (v->shape[i] != k->shape[i])
            return TA_ERR_SHAPE;
    if (Hkv < 1 || ps < 1 || sl->shape[0] != B || na->shape[0] != B || (so && so->shape[0] != B) || k->shape[0] < 0 ||
        k->shape[0] > INT32_MAX)
        return TA_ERR_SHAPE;
    if (pt ? (pt->shape[0] != B || pt->shape[1] < 1) : k->shape[0] < B)
        return TA_ERR_PAGE_TABLE;
    if (!strides_ok(k) || !strides_ok(v) || !strides_ok(ac) || (pt && !strides_ok(pt)) || k->stride[3] != 1 ||
        v->stride[3] != 1 || (pt && pt->stride[1] != 1) || sl->stride[0] < 0 || na->stride[0] < 0 ||
        (so && so->stride[0] < 0))
        return TA_ERR_STRIDE;
    const int64_t capacity = pt ? pt->shape[1] * ps : ps;
    if (capacity < T)
        return TA_ERR_PAGE_TABLE;
    if (capacity > INT32_MAX)
        return TA_ERR_SHAPE;
    if (B > 0 && (!k->data || !v->data || !sl->data || !ac->data || !na->data || (pt && !pt->data) || (so && !so->data)))
        return TA_ERR_NULL;
    if (so && B > 1) {
        // the lengths may be updated in place; any other overlap of the two arrays would let one request's new length
        // be read as another's old one
        const bool same = so->data == sl->data && so->stride[0] == sl->stride[0];
        const uintptr_t a0 = (uintptr_t)sl->data, a1 = a0 + (uintptr_t)((B - 1) * sl->stride[0] + 1) * 4;
        const uintptr_t b0 = (uintptr_t)so->data, b1 = b0 + (uintptr_t)((B - 1) * so->stride[0] + 1) * 4;
        if (!same && a0 < b1 && b0 < a1)
            return TA_ERR_STRIDE;
    }
    TACompact &c = *out;
    memset(&c, 0, sizeof c);
    c.k = k->data; c.v = v->data;
    c.page_table = pt ? (const int32_t *)pt->data : nullptr;
    c.seq_lens = (const int32_t *)sl->data;
    c.accepted = (const int32_t *)ac->data;
    c.n_accepted = (const int32_t *)na->data;
    c.seq_lens_out = so ? (int32_t *)so->data : nullptr;
    c.k_sp = k->stride[0]; c.k_sh = k->stride[1]; c.k_ss = k->stride[2];
    c.v_sp = v->stride[0]; c.v_sh = v->stride[1]; c.v_ss = v->stride[2];
    c.pt_sb = pt ? pt->stride[0] : 0;
    c.sl_s = sl->stride[0]; c.acc_sb = ac->stride[0]; c.na_s = na->stride[0]; c.slo_s = so ? so->stride[0] : 0;
    c.B = (int)B; c.T = (int)T; c.A = (int)A; c.Hkv = (int)Hkv; c.D = (int)D; c.ps = (int)ps; c.capacity = (int)capacity;
    c.n_pages = (int)k->shape[0];
    c.elem_bytes = k->dtype == TA_BF16 ? 2 : 4;
    c.vec = rows_of_16_bytes(k, D) && rows_of_16_bytes(v, D);
    return TA_OK;
}

// ---- entry points that need no device at all
extern "C" {

int tree_attn_version(void) { return TREEATTN_VERSION; }

const char *tree_attn_strerror(int status)
{
    switch (status) {
    case TA_OK: return "ok";
    case TA_ERR_NULL: return "a required descriptor or data pointer is NULL";
    case TA_ERR_DTYPE: return "unsupported or mismatching element type";
    case TA_ERR_RANK: return "wrong number of dimensions";
    case TA_ERR_SHAPE: return "shapes disagree";
    case TA_ERR_STRIDE: return "innermost stride must be 1 and strides must be non-negative";
    case TA_ERR_HEADS: return "query heads must be a multiple of KV heads";
    case TA_ERR_HEAD_DIM: return "head_dim out of range";
    case TA_ERR_TREE_SIZE: return "tree size must be in [1, 64]";
    case TA_ERR_PAGE_TABLE: return "page table cannot hold the tree tokens";
    case TA_ERR_WORKSPACE: return "workspace too small or misaligned, or it would have to grow under stream capture";
    case TA_ERR_HIP: return "HIP runtime call failed";
    case TA_ERR_BATCH: return "batch size out of range";
    case TA_ERR_OPTS: return "invalid option";
    default: return "unknown status";
    }
}

static int plan_problem(const ta_tensor *q, const ta_tensor *k_cache, const ta_tensor *v_cache, const ta_tensor *page_table,
                        const ta_tensor *seq_lens, const ta_tensor *tree_parent, const ta_tensor *out, const ta_tensor *lse,
                        const ta_opts *opts, int32_t num_cus, TAProblem *pr)
{
    ta_opts o;
    if (opts) {
        o = *opts;
        o.workspace = nullptr;      // planning never needs the scratch itself
        o.workspace_bytes = 0;
    }
    return ta_host_build_problem(q, k_cache, v_cache, page_table, seq_lens, tree_parent, out, lse, opts ? &o : nullptr,
                                 num_cus > 0 ? num_cus : 256, pr);
}

int tree_attn_plan(const ta_tensor *q, const ta_tensor *k_cache, const ta_tensor *v_cache,
                   const ta_tensor *page_table, const ta_tensor *seq_lens, const ta_tensor *tree_parent,
                   const ta_tensor *out, const ta_tensor *lse, const ta_opts *opts, int32_t num_cus,
                   int64_t plan[16])
{
    if (!plan)
        return TA_ERR_NULL;
    TAProblem pr;
    int rc = plan_problem(q, k_cache, v_cache, page_table, seq_lens, tree_parent, out, lse, opts, num_cus, &pr);
    if (rc != TA_OK)
        return rc;
    ta_host_fill_plan(pr, plan);
    return TA_OK;
}

int tree_attn_plan_blocks(const ta_tensor *q, const ta_tensor *k_cache, const ta_tensor *v_cache,
                          const ta_tensor *page_table, const ta_tensor *seq_lens, const ta_tensor *tree_parent,
                          const ta_tensor *out, const ta_tensor *lse, const ta_opts *opts, int32_t num_cus)
{
    TAProblem pr;
    int rc = plan_problem(q, k_cache, v_cache, page_table, seq_lens, tree_parent, out, lse, opts, num_cus, &pr);
    return rc != TA_OK ? rc : pr.p.blocks;
}

int tree_attn_dispatch_row(int32_t index, int64_t row[8])
{
    if (!row)
        return TA_ERR_NULL;
    if (index < 0 || index >= kTableRows)
        return TA_ERR_OPTS;
    const TADispatchRow &r = kTable[index];
    row[0] = r.family; row[1] = r.rows_grp_max; row[2] = r.lists_max; row[3] = r.wg_per_cu_x4;
    row[4] = r.min_share; row[5] = r.item_cost; row[6] = r.wide_from_parts; row[7] = r.wide_max_rows;
    return TA_OK;
}

}  // extern "C"
