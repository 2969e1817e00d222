// Matrix-core KV pass of libtreeattn for gfx950, fp32 inputs: head_dim 64 or 128, fp32 products and sums throughout
// (v_mfma_f32_16x16x4_f32, a chain of fp32 multiply-adds per element, rounded as the vector ALU rounds them).
//
// A workgroup keeps up to 32 query rows of one (request, KV head); its four waves (eight where it walks a whole list alone,
// with up to 16 rows) split the KEYS of its share, each takes every fourth (eighth) run of 16 tokens with its own running
// softmax, and their results meet in LDS when the item ends, like in
// ta_mfma_ks.hip.  Per run (transposed products, a lane owns one query row of each block of 16 throughout):
//     S^T[token, row] = K . Q^T        A = K (registers), B = Q (LDS)
//     O^T[d, row]    += V^T . P^T      A = V^T (registers), B = P (registers)
// The contraction index of each product may run in any order as long as both operands agree, and that order is chosen so
// that neither K nor V passes through LDS: lane (r, q) -- r the lane modulo 16, q its quarter of the wave -- loads of token
// r's row of K the 16-byte pieces q, q + 4, ..., and each of the four values of a piece is one step of the first product
// (a step contracts over the four quarters); the accumulator of S^T leaves in lane (r, q) the tokens 4 q + i of query row
// r, so step i of the second product contracts over these four tokens, of whose rows of V a lane loads the 16-byte pieces
// r and (head_dim 128) r + 16: whole rows, coalesced.
//
// What bounds it: up to some 30 MB, which is what fp32 calls hold, the chain of dependent steps -- lengths, page ids, the
// rows, the products of a run (4096 clocks at head_dim 128 and 32 rows, 3.0 us with everything around them in a wave that
// has its SIMD for itself), the waves' meeting -- so runs are short and a tile of 64 tokens occupies all four waves at once
// (runs of 32 tokens: 25.1 us for the call below).  Far above, the memory: at 32 rows a compute unit's products consume
// 64 KB in 1.7 us (four runs of 16 tokens at 1 KB), and its share of 6.8 TB/s in that time is 45 KB.
// KV pass by kernel trace: B 8, 8/2 heads, head_dim 128, T 8, L 200..4000 (36 MB) 17.9 us, where the vector-ALU kernel took
// 122; one list of 128 tokens, head_dim 64, 28 rows 7.2, 27.5 there.  Error against 64 bits over sizes of all these ranges:
// 2.9e-7 of the result (2-norm) where that kernel had 4.0e-7, the first product being summed in two chains.
#include <type_traits>

#include "ta_common.h"

typedef float f32_x4 __attribute__((ext_vector_type(4)));

#define F32_SUB 16                               // tokens a wave takes at a time
#define F32_ROWS TA_F32_ROWS                     // query rows of a workgroup

__device__ __forceinline__ void f32_lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Waves of a workgroup.  Two on a SIMD share its matrix pipe: eight waves gain only where a workgroup walks a whole list
// (36 MB in 16 lists, 190 of 256 workgroups busy with up to three tiles: 21.1 us a call with four, 22.0 with eight).
constexpr int f32_waves(bool solo) { return solo ? 8 : 4; }

// RB: blocks of 16 query rows (SOLO: one); NEW: the tree tokens of this step lie in tensors of their own (ta_opts.k_new);
// SOLO: workgroup x walks list x from end to end and writes its outputs (see p.solo)
template <int DH, int RB, bool NEW, bool SOLO>
__global__ __launch_bounds__(64 * f32_waves(SOLO), 2) void ta_f32_kv_kernel(TA_SCHED_PARAMS, TAParams p)
{
    const TASched sc = TA_SCHED;
    constexpr int F32_NW = f32_waves(SOLO);
    constexpr int NJ = DH / 16;                  // 16-byte pieces of a K row a lane loads
    constexpr int NH = DH / 64;                  // 16-byte pieces of a V row a lane loads
    constexpr int CH = DH / 4;                   // 16-byte chunks of a row
    constexpr int ROWS = 16 * RB;
    // (global memory by type: an address put together from integers would be loaded as a flat one, and its wait is for all)
    typedef const __attribute__((address_space(1))) float *gfloat;
    // (rows of k_new and v_new start at any element, those of the caches on 16 bytes: both are loaded 16 bytes at a time)
    typedef f32_x4 f32_piece __attribute__((aligned(4)));
    typedef const __attribute__((address_space(1))) f32_piece *gpiece;
    // Q rows while an item is walked, then the waves' results; row r's chunk c lies at chunk c ^ (r & 15)
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float (*lds)[ROWS * DH] = (float (*)[ROWS * DH])smem;
    float (*stat)[2][ROWS] = (float (*)[2][ROWS])(lds + F32_NW);  // reference and sum of a wave's rows
    int *wbad = (int *)(stat + F32_NW);                                   // TA_STATUS_* bits a wave has met
    // more than 64 requests: [B + 1] schedule, [B] lengths, [B] window starts
    int *cum = wbad + F32_NW, *lens = cum + p.B + 1, *starts = lens + p.B;

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = blockIdx.x, rg = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, qt = lane >> 4;
    // Schedule (see ta_build_schedule); up to 64 requests every wave keeps it in registers, lane b for request b
    const bool in_regs = sc.B <= TA_WAVE;
    int s_len = 0, s_start = 0, s_units = 0, s_cum = 0, total;
    int t, t_end;
    if constexpr (SOLO) {
        s_len = sc.seq_lens[(int64_t)(w / sc.Hkv) * sc.sl_s];
        s_start = ta_kv_start(sc, w / sc.Hkv);
        ta_touch_args<TAParams>(s_len);
        t = 0;
        t_end = 1;
    } else {
        if (in_regs) {
            if (lane < sc.B) {
                s_len = sc.seq_lens[(int64_t)lane * sc.sl_s];
                s_start = ta_kv_start(sc, lane);
                s_units = ta_list_tiles(sc, s_len, s_start) + sc.pad;
            }
            s_cum = ta_wave_scan(s_units);
            total = sc.Hkv * __builtin_amdgcn_readlane(s_cum, 63);
        } else {
            total = sc.Hkv * ta_build_schedule(sc, cum, lens, starts);
        }
        ta_wg_range(sc, total, w, t, t_end);
        t = __builtin_amdgcn_readfirstlane(t);
        t_end = __builtin_amdgcn_readfirstlane(t_end);
    }
    const int rows_here = min(p.rows_grp, p.rows - rg * p.rows_grp);
    const float c = p.scale_log2e;
    // what depends on the lane is derived where it is used: hoisted out of the loops, it would be spilled
    auto fresh = [](int x) {
        asm volatile("" : "+v"(x));
        return x;
    };

    while (t < t_end) {
        // ---- the next item: a list (b, g), its tiles [j0, j1), i.e. the prefix tokens [max(lo, S), hi), walked in runs of
        // 16 from lo, and the T tree tokens; run u belongs to wave u % F32_NW
        int b, g, L, S, n_b, j0, j1, slot = 0;
        if constexpr (SOLO) {
            t = t_end;
            b = w / sc.Hkv;
            g = w - b * sc.Hkv;
            L = s_len;
            S = s_start;
            n_b = ta_list_tiles(sc, L, S);
            j0 = 0;
            j1 = n_b;
        } else {
            int cum_b, cum_e;
            if (in_regs) {
                b = __popcll(__ballot(p.Hkv * s_cum <= t));
                cum_e = __builtin_amdgcn_readlane(s_cum, b);
                cum_b = cum_e - __builtin_amdgcn_readlane(s_units, b);
                L = __builtin_amdgcn_readlane(s_len, b);
                S = __builtin_amdgcn_readlane(s_start, b);
            } else {
                b = __builtin_amdgcn_readfirstlane(ta_find_request(p, cum, t));
                cum_b = __builtin_amdgcn_readfirstlane(cum[b]);
                cum_e = __builtin_amdgcn_readfirstlane(cum[b + 1]);
                L = __builtin_amdgcn_readfirstlane(lens[b]);
                S = __builtin_amdgcn_readfirstlane(starts[b]);
            }
            const int n_u = cum_e - cum_b;                             // schedule units of one list
            g = (t - p.Hkv * cum_b) / n_u;
            const int seg_start = p.Hkv * cum_b + g * n_u;
            n_b = n_u - p.pad;
            j0 = t - seg_start;
            j1 = min(n_b, t_end - seg_start);
            if (j1 <= j0) {
                t = seg_start + n_u;                                   // t lies in the list's trailing padding
                continue;
            }
            t = seg_start + (j1 == n_b ? n_u : j1);
            slot = w + b * p.Hkv + g;
            ta_note_owner(p, b, g, w, j0, j1, n_b);
        }
        int bad = ta_request_ok(p, L, S) ? 0 : TA_STATUS_BAD_SEQLEN;
        const int tile0 = bad ? 0 : S / TA_TILE;
        const bool has_tree = j1 == n_b;
        const int lo = max((tile0 + j0) * TA_TILE, S) & ~(F32_SUB - 1);
        const int hi = min((tile0 + (has_tree ? n_b - 1 : j1)) * TA_TILE, L);
        const int n_pre = !bad && hi > lo ? (hi - lo + F32_SUB - 1) / F32_SUB : 0;
        const int n_sub = bad ? 0 : n_pre + (has_tree ? (p.T + F32_SUB - 1) / F32_SUB : 0);
        auto sub_pos = [&](int u) { return u < n_pre ? lo + u * F32_SUB : L + (u - n_pre) * F32_SUB; };
        auto sub_end = [&](int u) {
            return u < n_pre ? min(hi, lo + (u + 1) * F32_SUB) : L + min(p.T, (u - n_pre + 1) * F32_SUB);
        };
        // Token r16 of run u, or, where the run has none there (past its end, before the window), its first attended one:
        // its page id, requested here, and the address of its rows once that id is there.
        auto token_at = [&](int u) {
            const int first = max(sub_pos(u), S), pos = sub_pos(u) + r16;
            return pos >= first && pos < sub_end(u) ? pos : first;
        };
        auto request_page = [&](int u) {
            const int pos = token_at(u);
            return p.page_table ? p.page_table[(int64_t)b * p.pt_sb + (pos >> p.ps_shift)] : b;
        };
        gfloat ka, va;
        auto locate = [&](int u, int page) {
            const int pos = token_at(u);
            int at = pos;
            if (p.page_table) {
                if (!ta_page_ok(p, page)) {        // must never become an address
                    bad |= TA_STATUS_BAD_PAGE;
                    page = 0;
                }
                at = pos & (p.ps - 1);
            }
            if constexpr (NEW)
                // (their pages have been checked like any: the merge pass, which writes the rows there, leaves out without a
                // word those whose page does not exist)
                if (u >= n_pre) {
                    ka = (gfloat)p.kn + (int64_t)b * p.kn_sb + (int64_t)(pos - L) * p.kn_st + (int64_t)g * p.kn_sh;
                    va = (gfloat)p.vn + (int64_t)b * p.vn_sb + (int64_t)(pos - L) * p.vn_st + (int64_t)g * p.vn_sh;
                    return;
                }
            ka = (gfloat)p.k + (int64_t)page * p.k_sp + (int64_t)g * p.k_sh + (int64_t)at * p.k_ss;
            va = (gfloat)p.v + (int64_t)page * p.v_sp + (int64_t)g * p.v_sh + (int64_t)at * p.v_ss;
        };
        f32_x4 k[NJ], v[4][NH];
        auto load_k = [&]() {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                k[j] = *(gpiece)(ka + 4 * (4 * j + qt));
        };
        auto load_v = [&]() {                      // (one path for all: a branch here, and the wait for K would be for V too)
            const uint32_t a_lo = (uint32_t)(uintptr_t)va, a_hi = (uint32_t)((uintptr_t)va >> 32);
            const int ln = fresh(lane), from = (ln >> 4) * 16, col = 4 * (ln & 15);       // (lane 4 q, in bytes)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t lo_ = __builtin_amdgcn_ds_bpermute(from + 4 * i, (int)a_lo);
                const uint32_t hi_ = __builtin_amdgcn_ds_bpermute(from + 4 * i, (int)a_hi);
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    v[i][h] = *(gpiece)((gfloat)((uint64_t)hi_ << 32 | lo_) + 64 * h + col);
            }
        };

        // ---- Q rows to LDS (rows past the group's end repeat its first row, their results are never stored), page ids
        // and parents
        int u = wave, page = 0, parent = -1;
        const int u_end = n_sub - 1 - ((n_sub - 1 - wave) & (F32_NW - 1));     // this wave's last run
        unsigned long long gmask = 0;
        if (u < n_sub)
            page = request_page(u);
        const int tree_u = has_tree ? n_pre + ((wave - n_pre) & (F32_NW - 1)) : n_sub;    // first tree run of this wave
        if (tree_u < n_sub && lane < p.T) {
            if (p.masks_in)
                gmask = ta_given_mask(p, b, lane);
            else
                parent = p.parent[(int64_t)b * p.par_sb + lane];
        }
        {
            constexpr int NT = 64 * F32_NW, PER = (ROWS * CH + NT - 1) / NT;     // chunks per thread (16 x 64, eight waves: every other)
            f32_x4 q[PER];
            const int tid_q = fresh(tid);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int x = tid_q + i * NT, row = x / CH, ch = x % CH;
                const int R = rg * p.rows_grp + (row < rows_here ? row : 0);
                const int node = (int)__umulhi((uint32_t)R << 8, p.g_magic);          // R / G
                q[i] = *(const f32_x4 *)((const float *)p.q + (int64_t)b * p.q_sb + (int64_t)node * p.q_st +
                                         (int64_t)(g * p.G + R - node * p.G) * p.q_sh + 4 * ch);
            }
            if (u < n_sub) {                       // (these go out before Q is waited for)
                locate(u, page);
                load_k();
                load_v();
                page = request_page(min(u + F32_NW, u_end));
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int x = tid_q + i * NT, row = x / CH, ch = x % CH;
                if (ROWS * CH >= NT || row < ROWS)
                    *(f32_x4 *)(lds[0] + row * DH + 4 * (ch ^ (row & 15))) = q[i];
            }
        }
        // the ancestor masks, in a wave that has tree tokens: lane i walks up from node i
        unsigned long long tmask[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            tmask[rb] = ~0ull;
        if (tree_u < n_sub) {
            unsigned long long m = 0;
            bool wrong = false;
            if (p.masks_in) {
                m = gmask;
                wrong = lane < p.T && !ta_given_mask_ok(m, lane);
            } else {
                int cur = lane < p.T ? lane : -1;
                for (int steps = 0; __any(cur >= 0); ++steps) {
                    wrong |= cur >= 0 && (cur >= p.T || steps >= p.T);
                    if (cur >= 0)
                        m |= 1ull << (cur & 63);
                    const int up = __shfl(parent, cur & 63, TA_WAVE);
                    cur = cur >= 0 && !wrong ? up : -1;
                }
            }
            if (wrong)
                bad |= TA_STATUS_BAD_PARENT;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int row = rb * 16 + r16;
                const int node = p.q_off + (int)__umulhi((uint32_t)(rg * p.rows_grp + row) << 8, p.g_magic);
                const uint32_t m_lo = __shfl((uint32_t)m, node & 63, TA_WAVE), m_hi = __shfl((uint32_t)(m >> 32), node & 63, TA_WAVE);
                if (row < rows_here)
                    tmask[rb] = ((unsigned long long)m_hi << 32) | m_lo;
            }
        }
        f32_x4 o[RB][4 * NH];                      // block 4 h + e, row m of the matrix: column 64 h + 4 m + e
        float m_run[RB], l_run[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            m_run[rb] = -INFINITY;
            l_run[rb] = 0.f;
#pragma unroll
            for (int db = 0; db < 4 * NH; ++db)
                o[rb][db] = f32_x4{0.f, 0.f, 0.f, 0.f};
        }
        f32_lds_barrier();

        // S^T = K . Q^T of the run whose K is in registers
        auto scores = [&](f32_x4 (&s)[RB]) {
            f32_x4 s2[RB];                         // (two shorter chains: a smaller rounding error, no time)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                s[rb] = s2[rb] = f32_x4{0.f, 0.f, 0.f, 0.f};
            uint32_t qa = (uint32_t)(r16 * DH * 4 + ((qt ^ r16) << 4));        // chunk 4 j + q of row r: ^ 64 j
            asm volatile("" : "+v"(qa));           // (made here: the addresses kept over the loop would be spilled)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                f32_x4 q[RB];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    q[rb] = *(const f32_x4 *)(smem + (qa ^ (64u * j)) + rb * 16 * DH * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        (j & 1 ? s2[rb] : s[rb]) =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][e], q[rb][e], j & 1 ? s2[rb] : s[rb], 0, 0, 0);
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                s[rb] += s2[rb];
            __builtin_amdgcn_sched_barrier(0);     // K's registers are free from here on
        };
        // running softmax (base 2) and O^T += V^T . P^T of run u
        auto accumulate = [&](int u, f32_x4 (&s)[RB]) {
            // which tokens count: bit i for token 4 q + i
            const int pos0 = sub_pos(u), cnt = sub_end(u) - pos0;
            uint32_t vm = cnt < F32_SUB ? (1u << cnt) - 1u : (1u << F32_SUB) - 1u;          // tokens the run has
            if (u < n_pre && pos0 < S)
                vm &= ~((1u << (S - pos0)) - 1u);
            const bool full = vm == (1u << F32_SUB) - 1u;
            if (!full || u >= n_pre) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const uint32_t on = (u >= n_pre ? vm & (uint32_t)(tmask[rb] >> ((u - n_pre) * F32_SUB)) : vm) >> (4 * qt);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (!((on >> i) & 1u))
                            s[rb][i] = -INFINITY;
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                s[rb] *= c;
                float mx = fmaxf(fmaxf(s[rb][0], s[rb][1]), fmaxf(s[rb][2], s[rb][3]));
                mx = fmaxf(mx, __shfl_xor(mx, 16, TA_WAVE));
                const float m_new = fmaxf(m_run[rb], fmaxf(mx, __shfl_xor(mx, 32, TA_WAVE)));
                if (__any(m_new != m_run[rb])) {
                    const float alpha = m_new == m_run[rb] ? 1.f : exp2f(m_run[rb] - m_new);
                    m_run[rb] = m_new;
                    l_run[rb] *= alpha;
#pragma unroll
                    for (int db = 0; db < 4 * NH; ++db)
                        o[rb][db] *= alpha;
                }
                // (a row that has not seen a token yet keeps -inf: its probabilities are exp2(-inf) = 0)
                const float ref = m_run[rb] == -INFINITY ? 0.f : m_run[rb];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    s[rb][i] = __builtin_amdgcn_exp2f(s[rb][i] - ref);
                l_run[rb] += (s[rb][0] + s[rb][1]) + (s[rb][2] + s[rb][3]);
            }
            // A run that is not full repeats a token's row in the places it has no token for; the probability there is
            // zero, and the row is made zero as well, lest an infinity in it count.
            if (!full) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!((vm >> (4 * qt + i)) & 1u))
#pragma unroll
                        for (int h = 0; h < NH; ++h)
                            v[i][h] = f32_x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int db = 0; db < 4 * NH; ++db)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        o[rb][db] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][db / 4][db % 4], s[rb][i], o[rb][db], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);     // V's registers are free from here on
        };
        if (u < n_sub) {
            f32_x4 s[RB];
            // (the last run stands after the loop, so that every pass of the loop issues the same loads: their number is
            // what lets the wait for K leave V's in flight)
#pragma unroll 1
            for (; u + F32_NW < n_sub; u += F32_NW) {
                scores(s);
                locate(u + F32_NW, page);
                load_k();
                page = request_page(min(u + 2 * F32_NW, u_end));
                accumulate(u, s);
                load_v();
            }
            scores(s);
            accumulate(u, s);
        }

        // ---- the waves' results meet
        f32_lds_barrier();                         // nobody reads Q any more
        const int tid_e = fresh(tid), r_e = tid_e & 15, q_e = (tid_e >> 4) & 3;
        {
            int wb = 0;
            for (int bit = TA_STATUS_BAD_PARENT; bit <= TA_STATUS_BAD_PAGE; bit <<= 1)
                wb |= __any(bad & bit) ? bit : 0;
            if ((tid_e & 63) == 0)
                wbad[wave] = wb;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float l_tot = l_run[rb] + __shfl_xor(l_run[rb], 16, TA_WAVE);
                l_tot += __shfl_xor(l_tot, 32, TA_WAVE);
                const int row = rb * 16 + r_e;
                if (q_e == 0) {
                    stat[wave][0][row] = m_run[rb];
                    stat[wave][1][row] = l_tot;
                }
                if (wave < n_sub)                  // (what a wave without runs would put there is not read)
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f32_x4 x;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            x[e] = o[rb][4 * h + e][i];
                        *(f32_x4 *)(lds[wave] + row * DH + 4 * ((16 * h + 4 * q_e + i) ^ r_e)) = x;
                    }
            }
        }
        f32_lds_barrier();
        {
            constexpr int TPR = 64 * F32_NW / ROWS < CH ? 64 * F32_NW / ROWS : CH;      // threads per row
            const int row = min(tid_e / TPR, ROWS - 1);
            const bool mine = tid_e / TPR < rows_here;                     // (16 x 64, eight waves: half have no row)
            int any_bad = 0;
            float mw[F32_NW], big = -INFINITY, l_tot = 0.f;
#pragma unroll
            for (int x = 0; x < F32_NW; ++x) {
                any_bad |= wbad[x];
                mw[x] = stat[x][0][row];
                big = fmaxf(big, mw[x]);
            }
            // the waves that met a score above -inf; only they are added up, also where the weight of one vanishes: a zero times an
            // infinity among its values is the NaN that column is due
            uint32_t met = 0;
#pragma unroll
            for (int x = 0; x < F32_NW; ++x) {
                met |= (mw[x] != -INFINITY ? 1u : 0u) << x;
                mw[x] = mw[x] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[x] - big);     // weight of the wave's result
                l_tot = fmaf(mw[x], stat[x][1][row], l_tot);
            }
            const float inv = 1.f / l_tot;
            if (SOLO && mine) {
                // no merge: the outputs as the merge pass makes them of one partial result
                const float lse2 = big + log2f(l_tot);
                const bool nan = any_bad || l_tot == 0.f || lse2 != lse2 || lse2 == INFINITY;
                const int R = rg * p.rows_grp + row, node = (int)__umulhi((uint32_t)R << 8, p.g_magic), h = g * p.G + R - node * p.G;
                float *dst = (float *)p.out + (int64_t)b * p.o_sb + (int64_t)node * p.o_st + (int64_t)h * p.o_sh;
#pragma unroll
                for (int i = 0; i < CH / TPR; ++i) {
                    const int ch = tid_e % TPR + i * TPR;
                    f32_x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int x = 0; x < F32_NW; ++x)
                        if ((met >> x) & 1u)
                            acc += mw[x] * *(const f32_x4 *)(lds[x] + row * DH + 4 * (ch ^ (row & 15)));
                    acc *= inv;
                    const float q_nan = __uint_as_float(0x7fc00000u);
                    *(f32_x4 *)(dst + 4 * ch) = nan ? f32_x4{q_nan, q_nan, q_nan, q_nan} : acc;
                }
                if (p.lse && tid_e % TPR == 0)
                    p.lse[(int64_t)b * p.lse_sb + (int64_t)h * p.lse_sh + (int64_t)node * p.lse_st] =
                        nan ? __uint_as_float(0x7fc00000u) : lse2 * 0.6931471805599453f;
            }
            if (!SOLO && mine) {
                const int64_t wrow = ta_ws_row(p, slot, rg, row);
#pragma unroll
                for (int i = 0; i < CH / TPR; ++i) {
                    const int ch = tid_e % TPR + i * TPR;
                    f32_x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int x = 0; x < F32_NW; ++x)
                        if ((met >> x) & 1u)
                            acc += mw[x] * *(const f32_x4 *)(lds[x] + row * DH + 4 * (ch ^ (row & 15)));
                    *(f32_x4 *)(p.ws_o + wrow * DH + 4 * ch) = any_bad ? f32_x4{0.f, 0.f, 0.f, 0.f} : acc * inv;
                }
                // (a NaN log-sum-exp poisons the row in the merge; a sum of zero: no score above -inf among the tokens)
                if (tid_e % TPR == 0)
                    p.ws_lse[wrow] = any_bad || l_tot == 0.f ? __uint_as_float(0x7fc00000u) : big + log2f(l_tot);
            }
            if (any_bad && tid_e == 0)
                ta_raise(p, any_bad);
        }
        if constexpr (!SOLO)
            f32_lds_barrier();                     // the next item's Q may overwrite the results
        if constexpr (SOLO && NEW) {               // the merge pass's part of the write-back
            TAScatter wb;
            ta_scatter_load(p, b, g, rg, gridDim.y, wb);
            ta_scatter_locate(p, b, g, wb);
            ta_scatter_store(p, b, g, rg, gridDim.y, wb);
        }
    }
}

template <int DH, int RB, bool NEW, bool SOLO>
static hipError_t launch_f32(const TAParams &p, hipStream_t stream, int dev)
{
    constexpr int NW = f32_waves(SOLO);
    constexpr size_t fixed = NW * (16 * RB * DH + 2 * 16 * RB + 1) * sizeof(float);
    static_assert(fixed + (SOLO ? 0 : sizeof(int) * (3 * TA_MAX_BATCH + 1)) <= 160 * 1024, "LDS of the largest batch");
    const size_t smem = fixed + (SOLO || p.B <= TA_WAVE ? 0 : sizeof(int) * (3 * (size_t)p.B + 1));
    static bool attr_set[64] = {};      // per device and instance; setting it twice is harmless
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void *)ta_f32_kv_kernel<DH, RB, NEW, SOLO>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess)
            return e;
        attr_set[dev] = true;
    }
    const dim3 grid(SOLO ? p.B * p.Hkv : p.n_wg, p.n_rg);
    hipLaunchKernelGGL((ta_f32_kv_kernel<DH, RB, NEW, SOLO>), grid, dim3(64 * NW), smem, stream, TA_SCHED_ARGS(p), p);
    return hipGetLastError();
}

hipError_t ta_launch_f32(const TAParams &p, hipStream_t stream, int dev)
{
    if (dev < 0 || dev >= 64)
        return hipErrorInvalidDevice;
    if (p.rows_grp > F32_ROWS || p.part_q15 || p.ls != 1 || (p.D != 64 && p.D != 128))
        return hipErrorInvalidValue;
    auto launch = [&](auto d, auto fold, auto alone) {
        constexpr int DH = decltype(d)::value;
        constexpr bool NEW = decltype(fold)::value, SOLO = decltype(alone)::value;
        if (p.rows_grp <= 16)
            return launch_f32<DH, 1, NEW, SOLO>(p, stream, dev);
        if constexpr (SOLO)
            return hipErrorInvalidValue;                     // (a list walked alone is in blocks of up to 16 rows)
        else
            return launch_f32<DH, 2, NEW, false>(p, stream, dev);
    };
    auto fold = [&](auto d, auto alone) { return p.kn ? launch(d, std::true_type{}, alone) : launch(d, std::false_type{}, alone); };
    auto with = [&](auto d) { return p.solo ? fold(d, std::true_type{}) : fold(d, std::false_type{}); };
    return p.D == 64 ? with(std::integral_constant<int, 64>{}) : with(std::integral_constant<int, 128>{});
}
