// Key-split matrix-core KV pass of libtreeattn for gfx950: bf16, head_dim 64 or 128, fp32 accumulation.
//
// A workgroup keeps up to 32 (head_dim 64: 64) query rows of one (request, KV head) and its waves split the KEYS of its share: wave w takes
// every NW-th run of 32 tokens, with its own running softmax over all the rows, and the waves' results meet in LDS when
// the item ends.  Nothing is exchanged inside the loop: each wave moves its own K and V rows HBM -> LDS into a ring only
// it reads (global_load_lds_dwordx4), waits with its own vmcnt and never meets a barrier.  Every wave computes, whatever
// the number of rows, and a share of a few tiles is walked by all waves at once.
//
// Per 32 tokens (both products transposed, so that a lane owns one query row per 32-row block; see ta_mfma.hip):
//     S^T[token, row] = K . Q^T        A = K fragment (LDS), B = Q fragment (registers)
//     O^T[d, row]    += V^T . P^T      A = V^T fragment (transposing LDS reads), B = P (registers)
// each K and V fragment feeding RB row blocks.
//
// More rows are served by workgroups side by side, which share the stream through the L2 (see key_split_workgroups).
// Head_dim 128 takes it where it is the faster of the two (the measured line stands in ta_host.cpp): calls of B 1, 32/8
// heads, T 64, L 4096 (256 rows) 27.5 -> 19.8 us, B 128, T 8, L 256..4096 208.4 -> 199 against the pipelined kernel.
//
// Q is loaded once per workgroup, whole rows at a time, and handed to the waves through LDS; with each wave loading its own
// fragments, 32 rows by 32 scattered bytes at a time, and all eight waves' blocks added up whether or not a wave had a
// run, the calls of one request took 0.8 us longer (one KV head, 8192 tokens, folded: 16.3 -> 15.5 us; T 64, L 4096
// 20.5 -> 20.2; head_dim 64, B 16 41.2 -> 39.6).
//
// What bounds it: the HBM stream.  In its loop a compute unit of head_dim 64 and 64 rows streams at the memory's rate
// (16 lists x 16384 tokens x 8 heads, 538 MB: 93 us, 5.8 TB/s); beside it stand 4.5 us at the start without a byte on
// its way (lengths, then page ids and Q, then the first tokens: three round trips and the instructions between them) and
// the end of an item, where the waves wait for the slowest (a run of 32 tokens takes a wave 3 us when all stream).
// Head_dim 64, B 16, 32/8 heads, T 16, L 2048..8192: KV pass 37.6 us; the kernel it replaced, which staged 64-token tiles
// through registers for all waves between barriers and computed with two waves of eight, took 115 us.
// Why eight waves: 64 KB in flight per compute unit are too few (four waves: 130 us on the 538 MB).  Two workgroups of
// four waves per unit share its bandwidth unevenly, the older one takes more (ends at 156 and 185 us of one launch),
// and cut the work into twice as many partial results.  They run where lists are short, uncut and more than the compute
// units (TA_SOLO_PAIR, the lines stand in ta_host.cpp): no partial results there, and one's start falls into the other's
// stream (1024 lists of 19 tiles 0.85 of the cut's time).
#include <initializer_list>

#include "ta_common.h"

typedef __bf16 ks_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 ks_bf16x2 __attribute__((ext_vector_type(2)));
typedef float ks_f32x2 __attribute__((ext_vector_type(2)));
typedef float ks_f32x16 __attribute__((ext_vector_type(16)));
typedef short ks_s4 __attribute__((ext_vector_type(4)));

#define KS_SUB 32                                // tokens a wave takes at a time
#define KS_LENS 256                              // batches of up to this many requests keep their lengths in LDS

__device__ __forceinline__ uint32_t ks_pack(float lo, float hi)
{
    ks_f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, ks_bf16x2));
}

__device__ __forceinline__ float ks_dot_ones(uint32_t pair, float acc)      // acc + both bf16 values of the pair
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(ks_bf16x2, pair), __builtin_bit_cast(ks_bf16x2, 0x3f803f80u), acc, false);
}

__device__ __forceinline__ float ks_swap_max(float x)      // over the two lanes that share a query row
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Largest x of the LPR (4, 8 or 16) neighbouring lanes that share an output row, in each of them.
template <int LPR>
__device__ __forceinline__ uint32_t ks_row_max(uint32_t x)
{
    static_assert(LPR == 4 || LPR == 8 || LPR == 16, "lanes of a row");
    auto up = [&](uint32_t y) { x = y > x ? y : x; };
    up(__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false));     // lanes 1 0 3 2 of every four
    up(__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false));     // 2 3 0 1
    if (LPR >= 8)
        up(__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, false));    // mirrored within eight
    if (LPR == 16)
        up(__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));    // rotated by eight within sixteen
    return x;
}

__device__ __forceinline__ void ks_lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void ks_vm_wait()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Every lane moves 16 bytes from its global address (64-bit, or a scalar base plus a lane offset) to LDS
// lds_wave_base + 16 * lane.  M0 is not used by anything else in this kernel.
__device__ __forceinline__ void ks_dma(const void *gptr, uint32_t lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gptr), "s"(lds_wave_base)
                 : "memory");
}

__device__ __forceinline__ void ks_dma_s(const void *base, uint32_t off, uint32_t lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base),
                 "s"(lds_wave_base)
                 : "memory");
}

// Four such loads in a row, 1 KB apart in memory and in LDS (the instruction's offset counts on both sides).
__device__ __forceinline__ void ks_dma_4k(const void *base, uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3,
                                          uint32_t lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %4 nt\n\tglobal_load_lds_dwordx4 %1, %4 offset:1024 nt\n\t"
                 "global_load_lds_dwordx4 %2, %4 offset:2048 nt\n\tglobal_load_lds_dwordx4 %3, %4 offset:3072 nt"
                 ::"v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(base), "s"(lds_wave_base)
                 : "memory");
}

// Sizes of one instance.  RB: 32-row blocks a wave keeps; NW: waves of a workgroup; OCC: workgroups per compute unit,
// which share its LDS.  A wave's ring holds NS runs of 32 tokens of K and as many of V, and is at least as large as its
// RB * 32 x DH block of fp32 results, which it stages there at the end.
template <int DH, int RB, int NW, int OCC>
struct KsShape {
    static constexpr int ROW = DH * 2;                     // bytes of a token row
    static constexpr int SUBB = KS_SUB * ROW;              // bytes of 32 K (or V) rows
    static constexpr int REGION = 128 * 1024 / OCC / NW < 4 * SUBB ? 128 * 1024 / OCC / NW : 4 * SUBB;   // LDS of a wave
    static constexpr int RING = NW * REGION;
    static constexpr int NS = REGION / (2 * SUBB);         // runs in flight
    static constexpr int LD = SUBB / 1024;                 // 1 KB loads per run of K (or V)
    static constexpr int RPL = KS_SUB / LD;                // token rows per load
    static constexpr int ROWS = 32 * RB;
    static constexpr int NT = 64 * NW;
    static constexpr int QB = ROWS * ROW;                  // bytes of the Q rows
    static constexpr int QP = (QB / 16 + NT - 1) / NT;     // 16-byte pieces of them a thread loads
    static_assert(NS >= 1 && NS <= 2 && REGION >= ROWS * DH * 4, "ring and staging area");
    static_assert(NW >= 4 && NW % 4 == 0, "at most one of a list's last three runs per wave; results are added up in fours");
};

// What a workgroup's lists are.  KS_CUT: a share of the line of all lists.  KS_DIRECT: the same, and the outputs of a list that
// lies in one share are written here (an instance of its own: calls without many lists are 1 % slower with that code in
// the kernel).  KS_SOLO: workgroup x walks list x from end to end (see p.solo).
enum { KS_CUT, KS_DIRECT, KS_SOLO };

// LDS of a workgroup.  (A workgroup that walks one list alone keeps no schedule.)
template <int DH, int RB, int NW, int OCC, int MODE>
static constexpr size_t ks_smem(int B)
{
    using C = KsShape<DH, RB, NW, OCC>;
    return C::RING + C::QB + sizeof(float) * 3 * NW * C::ROWS + sizeof(int) * NW +
           (MODE == KS_SOLO || B <= TA_WAVE ? 0 : sizeof(int) * (B + 2 + (B <= KS_LENS ? 2 * B : 0)));
}

template <int DH, int RB, int NW, int OCC, int MODE>
__global__ __launch_bounds__(64 * NW, OCC * NW / 4) void ta_mfma_ks_kernel(TA_SCHED_PARAMS, TAParams p)
{
    const TASched sc = TA_SCHED;
    using C = KsShape<DH, RB, NW, OCC>;
    constexpr bool SOLO = MODE == KS_SOLO;
    constexpr int NKK = DH / 16, NDB = DH / 32, SLOTS = DH / 8;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char *const qrows = smem + C::RING;                                 // Q rows of the item, placed like a run's K rows
    float *stat = (float *)(qrows + C::QB);                              // [NW][3][ROWS]: reference, sum, sum of rounded
    int *wbad = (int *)(stat + 3 * NW * C::ROWS);                        // [NW]: TA_STATUS_* bits a wave has met
    int *cum = wbad + NW;                                                 // more than 64 requests: [B + 1] schedule
    int *lens = cum + sc.B + 1, *starts = lens + sc.B;                      // and, up to KS_LENS, lengths and window starts
    const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char *)smem);

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = blockIdx.x, row0 = blockIdx.y * C::ROWS;               // first of the workgroup's query rows
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, hf = lane >> 5;
    // Schedule (see ta_build_schedule).  Up to 64 requests every wave keeps it in registers, lane b for request b: no
    // exchange between the waves, which start on their own.
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
            }
            ta_touch_args<TAParams>();
            if (lane < sc.B)
                s_units = ta_list_tiles(sc, s_len, s_start) + sc.pad;
            s_cum = ta_wave_scan(s_units);
            total = sc.Hkv * __builtin_amdgcn_readlane(s_cum, 63);
        } else {
            total = sc.Hkv * ta_build_schedule(sc, cum, sc.B <= KS_LENS ? lens : nullptr, sc.B <= KS_LENS ? starts : nullptr);
        }
        ta_wg_range(sc, total, w, t, t_end);
        t = __builtin_amdgcn_readfirstlane(t);
        t_end = __builtin_amdgcn_readfirstlane(t_end);
    }
    const int rows_here = min(C::ROWS, p.rows - row0);
    const float c = p.scale_log2e;
    const bool paged = p.page_table != nullptr;
    const uint32_t ksp = (uint32_t)p.k_sp, kss = (uint32_t)p.k_ss, vsp = (uint32_t)p.v_sp, vss = (uint32_t)p.v_ss;
    // 16-byte slots of a row in LDS: K slot s of row r holds chunk s ^ kx(r), V slot s chunk s ^ 2 vx(r); both spread
    // the sixteen (K) or eight (V) rows a fragment read touches at once over all banks
    auto kx = [](int r) { return DH == 64 ? (r >> 1) & 7 : r & 15; };
    auto vx = [](int r) { return DH == 64 ? 2 * ((r >> 1) & 1) + ((r >> 2) & 1) : 2 * (r & 3) + ((r >> 2) & 1); };
    const uint32_t region = lds0 + wave * C::REGION;
    char *const kring = smem + wave * C::REGION, *const vring = kring + C::NS * C::SUBB;
    // fragment offsets of this lane inside a run
    const int kf_row = r32 * C::ROW, kf_x = kx(r32);
    const int vtk = 4 * hf + ((lane >> 2) & 3), vh16 = (lane >> 4) & 1;
    const int vf_row = vtk * C::ROW + (lane & 3) * 8, vf_x = vx(vtk);
    // load role of this lane: row lrow of the RPL rows of a load, slot dslot
    const int lrow = lane / SLOTS, dslot = lane % SLOTS;
    constexpr int OFFS = DH == 64 ? 2 : 4, VOFFS = DH == 64 ? 1 : 2;       // the placement repeats after that many loads
    uint32_t koff[OFFS], voff[VOFFS];                                      // lane offset from the load's first row
#pragma unroll
    for (int k = 0; k < OFFS; ++k)
        koff[k] = (lrow * kss + (dslot ^ kx(k * C::RPL + lrow)) * 8) * 2;
#pragma unroll
    for (int k = 0; k < VOFFS; ++k)
        voff[k] = (lrow * vss + (dslot ^ (2 * vx(k * C::RPL + lrow))) * 8) * 2;
    const bool fast_geom = (!paged || p.ps_shift >= 3) && kss < (1u << 22) && vss < (1u << 22);
    // whole runs: 32 rows one after the other in memory
    const bool dense = (!paged || p.ps_shift >= 5) && kss == DH && vss == DH;
    // page ids a wave keeps: lane l holds the page of part l % ppr of its run pg_base + l / ppr
    const int ppr_shift = !paged || p.ps_shift >= 5 ? 0 : 5 - min(5, p.ps_shift);   // log2 of pages per run (fast_geom: <= 2)
    // what an item's start and end derive from the thread id is derived there: hoisted, it would be spilled in the loop
    auto fresh_lane = [&]() {
        int x = lane;
        asm volatile("" : "+v"(x));
        return x;
    };

    // ---- the current item: a list (b, g), its tiles [j0, j1), i.e. the prefix tokens [max(lo, S), hi), walked in runs of
    // 32 from lo, and the T tree tokens; run u belongs to wave u % NW
    int b = -1, g = 0, slot = 0, L = 0, S = 0, lo = 0, hi = 0, n_pre = 0, n_sub = 0, n_full = 0, bad = 0;
    bool has_tree = false, whole = false;                  // whole: a list that lies in this share alone
    uint4 q_piece[C::QP] = {};                             // this thread's pieces of the item's Q rows
    int pg = 0, pg_first = 0, pg_last = 0, parent = 0;     // pages of full runs, of the first and of the last run; tree
    unsigned long long gmask = 0;
    const uint16_t *kgp = nullptr, *vgp = nullptr;
    auto sub_pos = [&](int u) { return u < n_pre ? lo + u * KS_SUB : L + (u - n_pre) * KS_SUB; };
    auto sub_end = [&](int u) { return u < n_pre ? min(hi, lo + (u + 1) * KS_SUB) : L + min(sc.T, (u - n_pre + 1) * KS_SUB); };
    // this wave's run among those that are not full: the ragged end of the prefix and the tree's (n_sub: none)
    auto last_own = [&]() {
        const int u = n_full + ((wave - n_full) & (NW - 1));
        return u < n_sub ? u : n_sub;
    };
    auto page_of = [&](int pos) { return p.page_table[(int64_t)b * p.pt_sb + (pos >> p.ps_shift)]; };
    auto load_pages = [&](int i0) {                        // pages of this wave's full runs i0, i0 + 1, ...
        const int l = fresh_lane();
        const int pos = lo + (wave + NW * (i0 + (l >> ppr_shift))) * KS_SUB + (l & ((1 << ppr_shift) - 1)) * (KS_SUB >> ppr_shift);
        return pos >= S && pos < lo + n_full * KS_SUB ? page_of(pos) : 0;
    };
    // Moves on to the next item of [t, t_end) and requests what its start needs: Q, page ids, parents.  False at the end.
    auto next_item = [&]() {
        while (t < t_end) {
            int n_b, j0, j1;
            if constexpr (SOLO) {
                t = t_end;
                b = w / sc.Hkv;
                g = w - b * sc.Hkv;
                L = s_len;
                S = s_start;
                n_b = ta_list_tiles(sc, L, S);
                j0 = 0;
                j1 = n_b;
                whole = true;
            } else {
                int cum_b, cum_e;
                if (in_regs) {
                    b = __popcll(__ballot(sc.Hkv * s_cum <= t));
                    cum_e = __builtin_amdgcn_readlane(s_cum, b);
                    cum_b = cum_e - __builtin_amdgcn_readlane(s_units, b);
                } else {
                    if (b < 0)
                        b = ta_find_request(sc, cum, t);
                    else if ((int64_t)sc.Hkv * cum[b + 1] <= t)
                        ++b;
                    b = __builtin_amdgcn_readfirstlane(b);
                    cum_b = __builtin_amdgcn_readfirstlane(cum[b]);
                    cum_e = __builtin_amdgcn_readfirstlane(cum[b + 1]);
                }
                const int n_u = cum_e - cum_b;                          // schedule units of one list
                g = (t - sc.Hkv * cum_b) / n_u;
                const int seg_start = sc.Hkv * cum_b + g * n_u;
                n_b = n_u - sc.pad;
                j0 = t - seg_start;
                j1 = min(n_b, t_end - seg_start);
                if (j1 <= j0) {
                    t = seg_start + n_u;                               // t lies in the list's trailing padding
                    continue;
                }
                t = seg_start + (j1 == n_b ? n_u : j1);
                slot = w + b * sc.Hkv + g;
                whole = MODE == KS_DIRECT && j0 == 0 && j1 == n_b;
                ta_note_owner(p, b, g, w, j0, j1, n_b, whole);
                if (in_regs) {
                    L = __builtin_amdgcn_readlane(s_len, b);
                    S = __builtin_amdgcn_readlane(s_start, b);
                } else {
                    L = __builtin_amdgcn_readfirstlane(sc.B <= KS_LENS ? lens[b] : sc.seq_lens[(int64_t)b * sc.sl_s]);
                    S = __builtin_amdgcn_readfirstlane(sc.B <= KS_LENS ? starts[b] : ta_kv_start(sc, b));
                }
            }
            bad = ta_request_ok(sc, L, S) ? 0 : TA_STATUS_BAD_SEQLEN;
            const int tile0 = bad ? 0 : S / TA_TILE;
            has_tree = j1 == n_b;
            const int jp = has_tree ? n_b - 1 : j1;
            lo = max((tile0 + j0) * TA_TILE, S) & ~(KS_SUB - 1);
            hi = min((tile0 + jp) * TA_TILE, L);
            n_pre = !bad && hi > lo ? (hi - lo + KS_SUB - 1) / KS_SUB : 0;
            n_full = !bad && hi > lo ? (hi - lo) / KS_SUB : 0;
            n_sub = bad ? 0 : n_pre + (has_tree ? (sc.T + KS_SUB - 1) / KS_SUB : 0);
            kgp = (const uint16_t *)p.k + (int64_t)g * p.k_sh;
            vgp = (const uint16_t *)p.v + (int64_t)g * p.v_sh;
            const int l = fresh_lane();
#pragma unroll
            for (int i = 0; i < C::QP; ++i) {
                // rows past the group's end repeat its first row (their results are never stored)
                const int x = i * C::NT + wave * 64 + l, row = x / SLOTS;
                if (C::QB / 16 >= C::NT || row < C::ROWS) {
                    const int R = row0 + (row < rows_here ? row : 0);
                    const int node = (int)__umulhi((uint32_t)R << 8, p.g_magic);      // R / G
                    q_piece[i] = *(const uint4 *)((const uint16_t *)p.q + (int64_t)b * p.q_sb + (int64_t)node * p.q_st +
                                               (int64_t)(g * p.G + R - node * p.G) * p.q_sh + 8 * (x % SLOTS));
                }
            }
            if (wave >= n_sub)
                return true;                                       // nothing to walk for this wave
            const int ul = last_own();
            if (paged) {
                pg = load_pages(0);
                // runs that are not full: lane r holds the page of row r
                if (wave == 0)
                    pg_first = page_of(max(lo, S) + min(l & 31, sub_end(0) - 1 - max(lo, S)));
                if (ul < n_sub)
                    pg_last = page_of(max(S, min(sub_pos(ul) + (l & 31), sub_end(ul) - 1)));
            }
            if (ul < n_sub && ul >= n_pre && l < sc.T) {
                if (p.masks_in)
                    gmask = ta_given_mask(p, b, l);
                else
                    parent = p.parent[(int64_t)b * p.par_sb + l];
            }
            return true;
        }
        return false;
    };
    auto checked = [&](int id) {                           // a page id as an address: one outside the cache is reported
        if (!ta_page_ok(p, id)) {
            bad |= TA_STATUS_BAD_PAGE;
            id = 0;
        }
        return id;
    };

    bool more = next_item();
    while (more) {
        ks_f32x16 o[RB][NDB];
        float m_run[RB], l_run[RB], l2_run[RB];
        unsigned long long tmask[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            m_run[rb] = -INFINITY;
            l_run[rb] = 0.f;
            l2_run[rb] = 0.f;
            tmask[rb] = ~0ull;
        }
        const int u_last = last_own();
        int u = wave, pg_base = 0;
        // everything requested is here: no wait of the compiler for it may fall behind the loads into LDS, which it does
        // not know of
#pragma unroll
        for (int i = 0; i < C::QP; ++i)
            asm volatile("" : "+v"(q_piece[i].x), "+v"(q_piece[i].y), "+v"(q_piece[i].z), "+v"(q_piece[i].w));
        if (u < n_sub) {
            asm volatile("" : "+v"(pg), "+v"(pg_first), "+v"(pg_last), "+v"(parent), "+v"(gmask));
            if (paged) {
                pg = checked(pg);
                pg_first = checked(pg_first);
                pg_last = checked(pg_last);
            }
        }

        // Q rows to LDS.  (Each wave loading its own fragments, 32 rows by 32 scattered bytes at a time, kept the load units
        // busy for most of a microsecond.)
        {
            const int l = fresh_lane();
#pragma unroll
            for (int i = 0; i < C::QP; ++i) {
                const int x = i * C::NT + wave * 64 + l, row = x / SLOTS;
                if (C::QB / 16 >= C::NT || row < C::ROWS)
                    *(uint4 *)(qrows + row * C::ROW + (((x % SLOTS) ^ kx(row)) << 4)) = q_piece[i];
            }
        }

        // Loads of run u, K or V part, into ring slot sl: LD loads of 1 KB.
        auto issue = [&](int u, int sl, bool is_v) {
            const uint32_t dst = region + (is_v ? C::NS * C::SUBB : 0) + sl * C::SUBB;
            const uint32_t sp = is_v ? vsp : ksp, ss = is_v ? vss : kss;
            const uint16_t *gp = is_v ? vgp : kgp;
            const int pos0 = sub_pos(u);
            const bool full = u < n_full && pos0 >= S;
            if (full && fast_geom) {
                const int pl = ((u - wave) / NW - pg_base) << ppr_shift;           // lane that holds the run's first page
                uint32_t off[OFFS];
#pragma unroll
                for (int k = 0; k < OFFS; ++k)
                    off[k] = is_v ? voff[k % VOFFS] : koff[k];
                if (dense) {
                    const uint32_t page = paged ? (uint32_t)__builtin_amdgcn_readlane(pg, pl) : (uint32_t)b;
                    const uint32_t sr = paged ? (uint32_t)(pos0 & (p.ps - 1)) : (uint32_t)pos0;
                    const char *base = (const char *)(gp + (uint64_t)page * sp + (uint64_t)sr * DH);
#pragma unroll
                    for (int k = 0; k < C::LD; k += 4)
                        ks_dma_4k(base + k * 1024, off[0], off[1], off[2 % OFFS], off[3 % OFFS], dst + k * 1024);
                } else {
#pragma unroll
                    for (int k = 0; k < C::LD; ++k) {
                        const int r0 = k * C::RPL;
                        uint32_t page = (uint32_t)b, sr = (uint32_t)(pos0 + r0);
                        if (paged) {
                            page = (uint32_t)__builtin_amdgcn_readlane(pg, pl + (r0 >> (5 - ppr_shift)));
                            sr = (uint32_t)((pos0 + r0) & (p.ps - 1));
                        }
                        ks_dma_s(gp + (uint64_t)page * sp + (uint64_t)sr * ss, off[k % OFFS], dst + k * 1024);
                    }
                }
            } else {
                // rows past the run's end and rows before the window start read an attended token of the run (their
                // probabilities are exactly zero); the tree tokens of this step may lie in tensors of their own, dense:
                // request stride for the page, token stride for the slot
                const bool from_new = p.kn && u >= n_pre;
                const uint16_t *gb = gp;
                uint64_t spx = sp, ssx = ss;
                if (from_new) {
                    gb = is_v ? (const uint16_t *)p.vn + (int64_t)g * p.vn_sh : (const uint16_t *)p.kn + (int64_t)g * p.kn_sh;
                    spx = (uint64_t)(is_v ? p.vn_sb : p.kn_sb);
                    ssx = (uint64_t)(is_v ? p.vn_st : p.kn_st);
                }
                const int first = max(pos0, S), end = sub_end(u);
                const int pgr = u == u_last ? pg_last : pg_first;
                const bool own_pages = paged && u != u_last && u != 0;             // pages of fewer than eight tokens
#pragma unroll 4
                for (int k = 0; k < C::LD; ++k) {
                    const int row = k * C::RPL + lrow;
                    int pos = pos0 + row;
                    pos = pos < end && pos >= first ? pos : first;
                    uint32_t page = (uint32_t)b, sr = (uint32_t)pos;
                    if (from_new) {
                        sr -= (uint32_t)L;
                    } else if (paged) {
                        // (the first run's pages are kept from its first attended row on)
                        page = own_pages ? (uint32_t)checked(page_of(pos))
                                         : (uint32_t)__shfl(pgr, pos - (u == u_last ? pos0 : first), TA_WAVE);
                        sr = (uint32_t)(pos & (p.ps - 1));
                    }
                    const int chunk = dslot ^ (is_v ? 2 * vx(row) : kx(row));
                    ks_dma(gb + (uint64_t)page * spx + (uint64_t)sr * ssx + chunk * 8, dst + k * 1024);
                }
            }
        };
        // vmcnt: everything but the loads of the youngest n parts (a part = the K or the V rows of one run) is done
        auto wait_parts = [&](int n) {
            if (n >= 3)
                ks_vm_wait<3 * C::LD>();
            else if (n == 2)
                ks_vm_wait<2 * C::LD>();
            else if (n == 1)
                ks_vm_wait<C::LD>();
            else
                ks_vm_wait<0>();
        };
        // The waves meet once for Q.  A wave whose first runs are whole requests them before it does; one that makes its
        // addresses row by row, which takes longer, requests them behind, lest all wait for it (head_dim 128: 62 lists of four to
        // seventeen tiles 18.7 us a call with the meeting behind all loads, 17.3 before all and so; one list of 64 rows and
        // 64000 tokens 21.1 before all, 19.9 so).  Before all loads where that is the faster: head_dim 64, whose runs are half
        // as long (one list of 25600 tokens 13.4 us, 13.8 with early loads), and short lists walked alone (two tiles 9.4 and 9.9).
        const int u_2nd = u + (C::NS - 1) * NW;
        // (a scalar: each wave meets the others exactly once, by a branch)
        const int early = __builtin_amdgcn_readfirstlane(DH == 128 && !SOLO && fast_geom && u < n_full && lo + u * KS_SUB >= S &&
                                                         (u_2nd < n_full || u_2nd >= n_sub));
        if (!early)
            ks_lds_barrier();
#pragma unroll 1
        for (int k = 0; k < 2 * C::NS; ++k)                    // K and V of the wave's first run, and of its second
            if (u + (k >> 1) * NW < n_sub)
                issue(u + (k >> 1) * NW, k >> 1, k & 1);
        if (early)
            ks_lds_barrier();
        // while the first runs are on their way: Q fragments into every wave's registers, O = 0 and, in a wave that has tree
        // tokens, the ancestor masks
        uint4 qf[RB][NKK];
        if (u < n_sub) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int kk = 0; kk < NKK; ++kk)
                    qf[rb][kk] = *(const uint4 *)(qrows + rb * 32 * C::ROW + kf_row + (((2 * kk + hf) ^ kf_x) << 4));
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o[rb][db][i] = 0.f;
        if (u_last < n_sub && u_last >= n_pre) {
            // lane i walks up from node i
            const int l = fresh_lane();
            unsigned long long m = 0;
            bool wrong = false;
            if (p.masks_in) {
                m = gmask;
                wrong = l < sc.T && !ta_given_mask_ok(m, l);
            } else {
                int cur = l < sc.T ? l : -1;
                for (int steps = 0; __any(cur >= 0); ++steps) {
                    wrong |= cur >= 0 && (cur >= sc.T || steps >= sc.T);
                    if (cur >= 0)
                        m |= 1ull << (cur & 63);
                    const int up = __shfl(parent, cur & 63, TA_WAVE);
                    cur = cur >= 0 && !wrong ? up : -1;
                }
            }
            if (__any(wrong))
                bad |= TA_STATUS_BAD_PARENT;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int row = rb * 32 + (l & 31);
                const int node = p.q_off + (int)__umulhi((uint32_t)(row0 + row) << 8, p.g_magic);
                const uint32_t m_lo = __shfl((uint32_t)m, node & 63, TA_WAVE), m_hi = __shfl((uint32_t)(m >> 32), node & 63, TA_WAVE);
                if (row < rows_here)
                    tmask[rb] = ((unsigned long long)m_hi << 32) | m_lo;
            }
        }

        int sl = 0;
#pragma unroll 1
        for (; u < n_sub; u += NW) {
            // parts younger than this run's K: its V, and K and V of the next run when two fit the ring
            const int un = u + C::NS * NW;
            const bool next = u + NW < n_sub, ahead = un < n_sub;
            wait_parts(C::NS > 1 && next ? 3 : 1);
            // ---- S^T = K . Q^T
            ks_f32x16 s[RB];
            const char *kt = kring + sl * C::SUBB + kf_row;
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) {
                const uint4 kf = *(const uint4 *)(kt + (((2 * kk + hf) ^ kf_x) << 4));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const ks_f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(ks_bf16x8, kf),
                                                                    __builtin_bit_cast(ks_bf16x8, qf[rb][kk]),
                                                                    kk == 0 ? z : s[rb], 0, 0, 0);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the K rows are in registers: their slot is free
            if (ahead) {
                const int i = (un - wave) / NW - pg_base;
                if (paged && fast_geom && (i << ppr_shift) >= TA_WAVE) {
                    pg_base += i;                                          // the next 64 page ids (waits for all loads)
                    pg = checked(load_pages(pg_base));
                }
                issue(un, sl, false);
            }
            // ---- scores of tokens that do not exist, or that are no ancestors, become -inf
            const int pos0 = sub_pos(u), cnt = sub_end(u) - pos0;
            const bool tree = u >= n_pre;
            if (tree || cnt < KS_SUB || pos0 < S) {
                uint32_t vm = cnt < KS_SUB ? (1u << cnt) - 1u : ~0u;
                if (!tree && pos0 < S)
                    vm &= ~((1u << (S - pos0)) - 1u);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    uint32_t mm = vm;
                    if (tree)
                        mm &= (uint32_t)(tmask[rb] >> ((u - n_pre) * KS_SUB));
                    mm >>= 4 * hf;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (!((mm >> (8 * (i / 4) + (i % 4))) & 1u))
                            s[rb][i] = -INFINITY;
                }
            }
            // ---- running softmax
            uint4 pb[RB][2];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float t0 = s[rb][0], t1 = s[rb][1], t2 = s[rb][2], t3 = s[rb][3];
#pragma unroll
                for (int i = 4; i < 16; i += 4) {
                    t0 = fmaxf(t0, s[rb][i]);
                    t1 = fmaxf(t1, s[rb][i + 1]);
                    t2 = fmaxf(t2, s[rb][i + 2]);
                    t3 = fmaxf(t3, s[rb][i + 3]);
                }
                const float top = fmaxf(fmaxf(t0, t1), fmaxf(t2, t3)) * c;           // of this lane's sixteen scores
                // the reference moves only when a score exceeds it by more than 2^4 (base-2 units), so that O is
                // rarely rescaled; c > 0.  A wave that walks a whole list moves it whenever it can: the probability of the
                // largest score is then one, which bf16 holds exactly.  Relative error against 64 bits over forty calls: 2.05e-3 so,
                // 2.08e-3 with the lazy reference, 2.06e-3 with the lists cut, where more waves have such a score.
                // (the two lanes of a row exchange their maxima only then: with that in every run, and with the rounded values
                // added up one by one, head_dim 64, B 16, 32/8 heads, T 16 took 39.6 us a call instead of 39.05, one list of 64
                // rows and 8192 tokens 14.73 instead of 14.63)
                if (__any(top > m_run[rb] + (SOLO ? 0.f : 4.f))) {
                    const float m_new = fmaxf(m_run[rb], ks_swap_max(top));
                    const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[rb] - m_new);
                    m_run[rb] = m_new;
                    l_run[rb] *= alpha;
                    l2_run[rb] *= alpha;
#pragma unroll
                    for (int db = 0; db < NDB; ++db)
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            o[rb][db][i] *= alpha;
                }
            }
            // ---- V fragments.  Parts younger than this run's V: with two runs in the ring K and V of the next one
            // and the K just requested, with one the K just requested
            if (C::NS > 1)
                wait_parts(ahead ? 3 : next ? 2 : 0);
            else
                wait_parts(ahead ? 1 : 0);
            const char *vt = vring + sl * C::SUBB + vf_row;
            // All of them are requested here and arrive under the exponentials: left to the compiler, each was requested when
            // the one before had been used (head_dim 64, B 16 39.05 us a call, now 38.75; one list of 8192 tokens 14.63, now
            // 14.54).
            typedef __attribute__((address_space(3))) ks_s4 *lds_s4;
            typedef short s8 __attribute__((ext_vector_type(8)));
            s8 vf[2][NDB];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int db = 0; db < NDB; ++db) {
                    const char *a = vt + kb * 16 * C::ROW + (((2 * db + vh16) ^ vf_x) << 5);
                    const ks_s4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)a);
                    const ks_s4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(a + 8 * C::ROW));
                    vf[kb][db] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                // (a row that has not seen a token yet keeps -inf: its probabilities are exp2(-inf) = 0)
                const float neg_m = m_run[rb] == -INFINITY ? 0.f : -m_run[rb];
                float e[16], sum[2] = {0.f, 0.f}, sum2[2] = {0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    e[i] = __builtin_amdgcn_exp2f(fmaf(s[rb][i], c, neg_m));
                uint32_t pk[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    pk[i] = ks_pack(e[2 * i], e[2 * i + 1]);
                    sum[i & 1] += e[2 * i] + e[2 * i + 1];
                    sum2[i & 1] = ks_dot_ones(pk[i], sum2[i & 1]);
                }
                l_run[rb] += sum[0] + sum[1];
                l2_run[rb] += sum2[0] + sum2[1];
                pb[rb][0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                pb[rb][1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
            }
            // ---- O^T += V^T . P^T
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(ks_bf16x8, vf[kb][db]),
                                                                            __builtin_bit_cast(ks_bf16x8, pb[rb][kb]),
                                                                            o[rb][db], 0, 0, 0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the V rows are in registers
            if (ahead)
                issue(un, sl, true);
            sl = C::NS > 1 ? sl ^ 1 : 0;
        }

        // ---- the waves' results meet: each stages its RB * 32 x DH block (16-byte chunk ch of row r at chunk
        // ch ^ (r & 15)) in its own part of the ring, then every thread adds up its columns of one row over the waves
        const int n_live = min(NW, (n_sub + 3) & ~3);          // waves that had runs, in fours
        const int l_e = fresh_lane(), r32_e = l_e & 31, hf_e = l_e >> 5;
        {
            float *stage = (float *)(smem + wave * C::REGION);
            int wb = 0;
            if (__any(bad)) {
                for (int bit : {TA_STATUS_BAD_PARENT, TA_STATUS_BAD_SEQLEN, TA_STATUS_BAD_PAGE})
                    wb |= __any(bad & bit) ? bit : 0;
            }
            if (l_e == 0)
                wbad[wave] = wb;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int row = rb * 32 + r32_e;
                const float l_tot = l_run[rb] + __shfl_xor(l_run[rb], 32, TA_WAVE);
                const float l2_tot = l2_run[rb] + __shfl_xor(l2_run[rb], 32, TA_WAVE);
                if (hf_e == 0) {
                    stat[(wave * 3 + 0) * C::ROWS + row] = m_run[rb];
                    stat[(wave * 3 + 1) * C::ROWS + row] = l_tot;
                    stat[(wave * 3 + 2) * C::ROWS + row] = l2_tot;
                }
                if (wave < n_live)                             // (nobody reads what the others would put there)
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const int ch = db * 8 + 2 * i4 + hf_e;
                        *(float4 *)(stage + row * DH + ((ch ^ (row & 15)) << 2)) =
                            make_float4(o[rb][db][4 * i4], o[rb][db][4 * i4 + 1], o[rb][db][4 * i4 + 2], o[rb][db][4 * i4 + 3]);
                    }
            }
        }
        const int slot_e = slot, b_e = b, g_e = g;
        const bool whole_e = whole;
        more = next_item();                                    // its requests are on their way during the rest
        ks_lds_barrier();
        int any_bad = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k)
            any_bad |= wbad[k];
        {
            const int x_e = wave * 64 + l_e;
            constexpr int TPR = C::NT / C::ROWS, CPT = DH / TPR;         // threads per row, columns per thread
            const int row = x_e / TPR, c0 = (x_e % TPR) * (CPT / 4);
            float mw[NW], big = -INFINITY;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                mw[k] = stat[(k * 3 + 0) * C::ROWS + row];
                big = fmaxf(big, mw[k]);
            }
            float l_tot = 0.f, l2_tot = 0.f, acc[CPT];
#pragma unroll
            for (int i = 0; i < CPT; ++i)
                acc[i] = 0.f;
#pragma unroll
            for (int k0 = 0; k0 < NW; k0 += 4)
                if (k0 < n_live) {
#pragma unroll
                    for (int k = k0; k < k0 + 4; ++k) {
                        const float wgt = mw[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[k] - big);
                        l_tot = fmaf(wgt, stat[(k * 3 + 1) * C::ROWS + row], l_tot);
                        l2_tot = fmaf(wgt, stat[(k * 3 + 2) * C::ROWS + row], l2_tot);
#pragma unroll
                        for (int q = 0; q < CPT / 4; ++q) {
                            const float4 x = *(const float4 *)(smem + k * C::REGION + (row * DH + (((c0 + q) ^ (row & 15)) << 2)) * 4);
                            acc[4 * q + 0] = fmaf(wgt, x.x, acc[4 * q + 0]);
                            acc[4 * q + 1] = fmaf(wgt, x.y, acc[4 * q + 1]);
                            acc[4 * q + 2] = fmaf(wgt, x.z, acc[4 * q + 2]);
                            acc[4 * q + 3] = fmaf(wgt, x.w, acc[4 * q + 3]);
                        }
                    }
                }
            const float inv = any_bad ? 0.f : 1.f / l2_tot;
            // largest magnitude of the row, as bits: those of a NaN are above all others
            uint32_t top = 0;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                acc[i] *= inv;
                const uint32_t mag = __float_as_uint(acc[i]) & 0x7fffffffu;
                top = mag > top ? mag : top;
            }
            top = ks_row_max<TPR>(top);
            const bool nan_seen = top > 0x7f800000u;
            const float amax = nan_seen ? 0.f : __uint_as_float(top);
            float scale, to_q;
            ta_q15_scale(amax, nan_seen, scale, to_q);
            const float lse2 = any_bad ? __uint_as_float(0x7fc00000u) : big + log2f(l_tot);
            if (MODE != KS_CUT && whole_e) {
                // no merge: the rows go out as they are, by its rules: a NaN or an infinity spoils its row (the 16-bit format
                // holds neither), and no score above -inf leaves no log-sum-exp either
                if (row < rows_here) {
                    const int R = row0 + row, node = (int)__umulhi((uint32_t)R << 8, p.g_magic), h = g_e * p.G + R - node * p.G;
                    const bool nan = any_bad || nan_seen || amax == INFINITY || lse2 != lse2;
                    uint32_t *dst = (uint32_t *)((uint16_t *)p.out + (int64_t)b_e * p.o_sb + (int64_t)node * p.o_st +
                                                 (int64_t)h * p.o_sh + 4 * c0);
#pragma unroll
                    for (int q = 0; q < CPT / 4; ++q)
                        *(uint2 *)(dst + 2 * q) = nan ? make_uint2(0x7fc07fc0u, 0x7fc07fc0u)
                                                      : make_uint2(ks_pack(acc[4 * q], acc[4 * q + 1]), ks_pack(acc[4 * q + 2], acc[4 * q + 3]));
                    if (p.lse && x_e % TPR == 0)
                        p.lse[(int64_t)b_e * p.lse_sb + (int64_t)h * p.lse_sh + (int64_t)node * p.lse_st] =
                            lse2 == -INFINITY ? __uint_as_float(0x7fc00000u) : lse2 * 0.6931471805599453f;
                }
            } else if (row < rows_here) {
                const int64_t wrow = ta_ws_row(p, slot_e, 0, row0 + row);
                uint32_t *dst = (uint32_t *)(ta_part_row(p, wrow) + 8 * c0);
#pragma unroll
                for (int q = 0; q < CPT / 4; ++q)
                    *(uint2 *)(dst + 2 * q) = make_uint2(ta_q15_pack(acc[4 * q], acc[4 * q + 1], to_q),
                                                         ta_q15_pack(acc[4 * q + 2], acc[4 * q + 3], to_q));
                // (a NaN log-sum-exp poisons the row in the merge)
                if (x_e % TPR == 0)
                    *(float2 *)&p.ws_lse[2 * wrow] =
                        make_float2(lse2, scale);
            }
            if (any_bad && x_e == 0)
                ta_raise(p, any_bad);
        }
        ks_lds_barrier();                                      // the rings are free for the next item
    }
    if constexpr (SOLO) {
        if (p.kn) {                                            // the merge pass's part of the write-back
            TAScatter wb;
            ta_scatter_load(p, b, g, blockIdx.y, gridDim.y, wb);
            ta_scatter_locate(p, b, g, wb);
            ta_scatter_store(p, b, g, blockIdx.y, gridDim.y, wb);
        }
    }
}

template <int DH, int RB, int NW, int OCC, int MODE>
static hipError_t launch_ks(const TAParams &p, hipStream_t stream, int dev)
{
    const size_t smem = ks_smem<DH, RB, NW, OCC, MODE>(p.B);
    static_assert(OCC * ks_smem<DH, RB, NW, OCC, MODE>(TA_MAX_BATCH) <= 160 * 1024, "OCC workgroups per compute unit, whatever the batch");
    if (smem > 160 * 1024)
        return hipErrorInvalidValue;
    static bool attr_set[64] = {};      // per device and instance; setting it twice is harmless
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void *)ta_mfma_ks_kernel<DH, RB, NW, OCC, MODE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess)
            return e;
        attr_set[dev] = true;
    }
    hipLaunchKernelGGL((ta_mfma_ks_kernel<DH, RB, NW, OCC, MODE>), dim3(MODE == KS_SOLO ? p.B * p.Hkv : p.n_wg, (p.rows + 32 * RB - 1) / (32 * RB)), dim3(64 * NW), smem,
                       stream, TA_SCHED_ARGS(p), p);
    return hipGetLastError();
}

hipError_t ta_launch_mfma_ks(const TAParams &p, hipStream_t stream, int dev)
{
    if (dev < 0 || dev >= 64)
        return hipErrorInvalidDevice;
    if ((p.ks_rows != 32 && p.ks_rows != 64) || (!p.solo && p.rows_grp % p.ks_rows != 0) || !p.part_q15 || p.ls != 2)
        return hipErrorInvalidValue;
    if (p.solo == TA_SOLO_PAIR && p.ks_rows == 32)
        return p.D == 128 ? launch_ks<128, 1, 4, 2, KS_SOLO>(p, stream, dev) : launch_ks<64, 1, 4, 2, KS_SOLO>(p, stream, dev);
    if (p.solo && p.D == 128 && p.ks_rows == 32)
        return launch_ks<128, 1, 8, 1, KS_SOLO>(p, stream, dev);
    if (p.solo && p.D == 64)
        return p.ks_rows == 32 ? launch_ks<64, 1, 8, 1, KS_SOLO>(p, stream, dev) : launch_ks<64, 2, 8, 1, KS_SOLO>(p, stream, dev);
    if (p.D == 128 && p.ks_rows == 32 && !p.solo)
        return p.direct ? launch_ks<128, 1, 8, 1, KS_DIRECT>(p, stream, dev) : launch_ks<128, 1, 8, 1, KS_CUT>(p, stream, dev);
    if (p.D != 64 || p.direct || p.solo)
        return hipErrorInvalidValue;
    return p.ks_rows == 32 ? launch_ks<64, 1, 8, 1, KS_CUT>(p, stream, dev) : launch_ks<64, 2, 8, 1, KS_CUT>(p, stream, dev);
}
