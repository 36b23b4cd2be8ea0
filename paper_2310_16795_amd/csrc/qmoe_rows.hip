// Fused decode + product with the rows of a matrix shared by several lanes each: the form for
// calls whose items are too few, or whose rows are too long, to give every lane rows of its own
// (qmoe_product.h), and for single matrices.
#include "qmoe_dev.h"

namespace qmoe {
namespace {

// ---------------------------------------------------------------- a row per L lanes
//
// L lanes (1 .. 64, a power of two) share a matrix row.  Each takes a whole 16-byte piece of the row's codewords
// (eight) at a time, looks the eight entries up, adds their run lengths, and finds the column where its piece
// starts from a prefix sum over the row's lanes (data-parallel-primitive adds) -- one scan for eight codewords.  Then
// it applies its entries as the lane-per-row-range kernel does, without that kernel's bookkeeping for rows that end
// inside a piece, and the lanes' sums are added at the end of the row.
//
// The work of a launch -- every row of every item, weighted by what a row of a tile of that many tokens
// costs -- is cut into one contiguous share per workgroup, on the device, where the number of items is known: no
// hand-out, no last round that is nearly empty, and one or two tiles of activations to stage per workgroup.  L is
// chosen there too: as few lanes as keep the sixteen wavefronts of a workgroup at work.
constexpr int kRowsThreads = 1024;
constexpr int kRowsPadCols = 8 * 28 + 4;  // zeros behind the activations: a piece that starts past the row's end (corrupt
                                          // stream) reads at most this far


// Workgroup barrier for LDS traffic only: loads from global memory stay in flight across it (__syncthreads waits for them).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef u32x4 u32x4_any __attribute__((aligned(2)));
using gp_u32x4_any = const __attribute__((address_space(1))) u32x4_any *;

// How the rows of a launch are cut into shares: made by the host.
struct RowsSplit {
    int rows, x_slots;   // rows of a matrix; token tiles whose activations fit the LDS at once (1 or 2)
    double inv_item[4];  // 1 / (cost of a whole item of class k)
    double inv_grid;
    uint32_t round_cost[7];  // of a round of the wavefronts with 2^l lanes per row: twice the pieces of a row over its lanes, and two or three more
    // lane-interleaved layout: 1 / lanes, and the even split of the rows over the lanes (`lane_extra` lanes own a row more)
    float inv_lanes;
    int lanes, lane_rows, lane_extra;
};

struct RowsTile {
    int ntok, slot0;
    const __attribute__((address_space(3))) int *tok_ids;
    const __attribute__((address_space(3))) float *gate_s;
};

// What a lane needs to begin a group of 64 / L rows: three dependent trips to memory (descriptor, offsets, first piece), asked
// for before the activations are staged for a wavefront's first group, and during the group before for the others.
struct GroupHead {
    uint32_t K0, K1, raw;  // the row's first codeword, the next row's, scale (or grid pair) as stored
    uint32_t Ka, wave, at; // lane-interleaved layout: first codeword of the row's lane, first piece of its group of lanes, place there
    u32x4 v;               // the lane's first piece
};

// Rows are numbered in the order in which they are worked on.  Back to back: as they are.  Lane-interleaved: the first rows of
// all lanes of the layout, then their second rows and so on, so that neighbours, whose pieces the lanes of a wavefront read
// together, are neighbours in memory.  Row number n -> the matrix's row, and the first row of its lane.
// (Against rows back to back, us: one token 21.1 and 22.1, 64 tokens 83 and 85, 512 tokens 374 and 375 on 256 experts of
// 2080 x 6144; 512 tokens on 128 experts of 768 x 3072 88 and 96.  Not loading `Ka` where every lane has one row: slower, the
// branch waits for the loads before it.)
template <int LANES>
__device__ __forceinline__ int numbered_row(const RowsSplit &sp, int n, int &lane_of, int &lane_row)
{
    if constexpr (!LANES) {
        return n;
    } else {
        const int i = (int)(((float)n + 0.5f) * sp.inv_lanes);  // n / lanes (exact: rows and lanes are below 2^16)
        lane_of = n - i * sp.lanes;
        lane_row = lane_of * sp.lane_rows + min(lane_of, sp.lane_extra);
        return lane_row + i;
    }
}

template <int ASYM, int LANES>
__device__ __forceinline__ void head_offsets(const RowsSplit &sp, const qmoe_matrix &M, int r1, int number, GroupHead &h)
{
    int lane_of = 0, lane_row = 0;
    const int rr = numbered_row<LANES>(sp, min(number, r1 - 1), lane_of, lane_row);
    gp_u32 row_off = (gp_u32)M.row_off;
    h.K0 = row_off[rr];
    h.K1 = row_off[rr + 1];
    if constexpr (LANES) {
        h.Ka = row_off[lane_row];
        h.wave = ((gp_u32)M.wave_off)[lane_of >> 6];
        h.at = (uint32_t)(lane_of & 63);
    }
    if constexpr (ASYM) h.raw = M.minmax_bf16 ? ((gp_u32)M.minmax_bf16)[rr] : 0u;  // no pair array: decodes to zeros
    else h.raw = ((gp_u16)M.scale_f16)[rr];
}

// The 16-byte pieces of a row of n codewords.  `end` bounds the codewords' places in the row's pieces: piece q holds places
// 8 q .. 8 q + 7, and slots [from, to) of it are codewords of the row.
//
// Back to back: places count from the row's first codeword.  Rows begin anywhere in the stream, so a piece's address is a
// multiple of 2 only; a piece that would reach past the stream's last 16-byte boundary is read that much earlier and its
// first slots are somebody else's.
template <int LANES>
struct RowPieces {
    uint32_t K0, k_last;
    int n, end;
    uintptr_t codes;
    __device__ __forceinline__ RowPieces(const qmoe_matrix &M, const GroupHead &h, bool live)
    {
        const uint32_t cap = min(M.n_codes, kMaxCodes), K1 = min(h.K1, cap);
        K0 = min(h.K0, K1);
        end = n = live ? (int)(K1 - K0) : 0;
        k_last = max((cap + 7u) & ~7u, 8u) - 8u;
        codes = reinterpret_cast<uintptr_t>(M.codes);
    }
    __device__ __forceinline__ uint32_t slot0(int q) const { return K0 + 8u * (uint32_t)min(q, max((n - 1) >> 3, 0)); }
    __device__ __forceinline__ u32x4 load(int q) const { return *(gp_u32x4_any)(codes + 2u * (uintptr_t)min(slot0(q), k_last)); }
    __device__ __forceinline__ void slots(int q, int &from, int &to) const
    {
        const uint32_t at = slot0(q);
        from = (int)(at - min(at, k_last));
        to = from + n - 8 * q;
    }
};

// Lane-interleaved: a row is a part of its lane's stream, whose pieces lie 64 apart; places count from the start of the
// piece that holds the row's first codeword.
template <>
struct RowPieces<1> {
    uint32_t piece, last;
    int lead, n, end;
    uintptr_t codes;
    __device__ __forceinline__ RowPieces(const qmoe_matrix &M, const GroupHead &h, bool live)
    {
        const uint32_t cap = min(M.n_codes, kMaxCodes), K1 = min(h.K1, cap), K0 = min(h.K0, K1), before = K0 - min(h.Ka, K0);
        n = live ? (int)(K1 - K0) : 0;
        lead = (int)(before & 7u);
        end = n ? lead + n : 0;
        piece = h.wave + h.at + 64u * (before >> 3);
        last = max(cap >> 3, 1u) - 1u;  // (the buffer's last piece: offsets that are no offsets stay inside it)
        codes = reinterpret_cast<uintptr_t>(M.codes);
    }
    __device__ __forceinline__ u32x4 load(int q) const
    {
        return *(gp_u32x4)(codes + 16u * (uintptr_t)min(piece + 64u * (uint32_t)min(q, max((end - 1) >> 3, 0)), last));
    }
    __device__ __forceinline__ void slots(int q, int &from, int &to) const
    {
        from = q == 0 ? lead : 0;
        to = end - 8 * q;
    }
};

// Rows number r0 .. r1 of M for a tile whose activations are staged at LDS address xs_addr: the groups of 64 / L rows numbered
// `group`, `group` + wavefronts of the workgroup, ...  `head`: of group `group`, if `have`.
template <int TBI, int EPI, int ASYM, int LANES>
__device__ __forceinline__ void rows_block(const ProductArgs &a, const RowsSplit &sp, const qmoe_matrix &M, int r0, int r1, int group, int log2L,
                                           uint32_t xs_addr, const RowsTile &tile, lp_u32 table, GroupHead head, bool have)
{
    constexpr int NA = TBI * (1 + ASYM);
    const int lane = threadIdx.x & 63, waves = (int)blockDim.x >> 6, L = 1 << log2L;
    const int sub = lane & (L - 1), mine = lane >> log2L, R = 64 >> log2L;
    const uint32_t n_groups3 = 3u * (uint32_t)a.n_groups, last = (uint32_t)a.n_order - 1u, cols8 = 8u * (uint32_t)a.cols;
    for (int rg = r0 + group * R; rg < r1; rg += waves * R) {
        const int number = rg + mine;
        const bool live = number < r1;
        if (!have) {
            head_offsets<ASYM, LANES>(sp, M, r1, number, head);
            head.v = RowPieces<LANES>(M, head, live).load(sub);
        }
        const RowPieces<LANES> rp(M, head, live);
        const int end = rp.end;
        const uint32_t raw = head.raw;
        u32x4 v = head.v;
        head_offsets<ASYM, LANES>(sp, M, r1, number + waves * R, head);
        have = true;
        float acc[NA];
#pragma unroll
        for (int t = 0; t < NA; t++) acc[t] = 0.0f;
        uint32_t base8 = 0u;  // 8 * column where the row's pieces of this step begin
        for (int q = sub; __any(8 * q < end); q += L) {
            const u32x4 v_next = rp.load(q + L);
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 4; j++) order_entry2(table, v[j], n_groups3, last, e[2 * j], e[2 * j + 1]);
            // slots that are not the row's codewords become empty entries
            int from, to;
            rp.slots(q, from, to);
            if (!__all(from == 0 && to >= 8)) {
                const uint32_t keep = (0xFFu << from) & (to <= 0 ? 0u : (1u << min(to, 8)) - 1u);
#pragma unroll
                for (int j = 0; j < 8; j++) e[j] &= (uint32_t)__builtin_amdgcn_sbfe((int)keep, j, 1);
            }
            uint32_t len8 = 0u;
#pragma unroll
            for (int j = 0; j < 8; j++) len8 += e[j] & 0xFFu;
            const uint32_t incl = lanes_scan(len8, L, sub);
            uint32_t pos = (TBI == 1 ? xs_addr : 0u) + min(base8 + incl - len8, cols8);
            base8 += (uint32_t)__shfl((int)incl, lane | (L - 1), 64);
            if constexpr (TBI == 1) {
                uint32_t x[24];
#pragma unroll
                for (int j = 0; j < 8; j++) {
#pragma unroll
                    for (int z = 0; z < 3; z++) x[3 * j + z] = (uint32_t)(*(lp_u16)(uintptr_t)(pos + ((e[j] >> (8 + 8 * z)) & 0xFFu)));
                    pos += e[j] & 0xFFu;
                }
#pragma unroll
                for (int j = 0; j < 8; j++) add_one_token<ASYM>(x + 3 * j, e[j], acc);
            } else {
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    accumulate_tile<TBI, ASYM>(e[j], xs_addr, pos, acc);  // sums doubled
                    pos += e[j] & 0xFFu;
                }
            }
            v = v_next;
        }
        head.v = RowPieces<LANES>(M, head, number + waves * R < r1).load(sub);
#pragma unroll
        for (int t = 0; t < NA; t++) acc[t] = lanes_scan(acc[t], L, sub);
        if (live && sub == L - 1) {
            float scale, mid = 0.0f;  // y = scale * (signed sum) + mid * (sum under |weight|)
            if constexpr (ASYM) {
                const float w_min = __uint_as_float(raw << 16), w_max = __uint_as_float(raw & 0xFFFF0000u);
                scale = 0.5f * (w_max - w_min);
                mid = 0.5f * (w_max + w_min);
            } else {
                scale = half_bits_to_float((uint16_t)raw);
            }
            if constexpr (TBI != 1) {
                scale *= 0.5f;
                mid *= 0.5f;
            }
            int lane_of, lane_row;
            const int row = numbered_row<LANES>(sp, number, lane_of, lane_row);
#pragma unroll
            for (int t = 0; t < TBI; t++) {
                if (t < tile.ntok) {
                    float y = acc[t] * scale;
                    if constexpr (ASYM) y = fmaf(acc[NA - TBI + t], mid, y);
                    if constexpr (EPI == 0)
                        ((__attribute__((address_space(1))) float *)a.out)[(size_t)tile.tok_ids[t] * a.ld_out + row] = tile.gate_s[t] * y;
                    else
                        ((__attribute__((address_space(1))) uint16_t *)a.out)[(size_t)(tile.slot0 + t) * a.ld_out + row] =
                            float_to_bf16_bits(y > 0.0f ? y : 0.0f);
                }
            }
        }
    }
}

// What a row of a tile costs by the tile's class (none, as tiles have at most four tokens; three or four, two, one): nanoseconds
// per row of 1024 columns and workgroup, measured 17.3, 12.5 and 9.8.
constexpr int kRowCost[4] = {0, 31, 22, 17};

// A workgroup's share of a launch: from row r0 of item i0 to row r1 of item i1 (none of it: i1 < i0).  r0 is a row of item i0.
struct RowsShare {
    int i0, r0, i1, r1;
};

// (reciprocals to the last bit but one: every workgroup has the same ones, and whole quotients are rounded up first)
__host__ __device__ __forceinline__ float near_rcp(float v)
{
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(v);
#else
    return 1.0f / v;
#endif
}

// The largest number from `most` down to 1 that fits, 0 if none does: a lane tries each.
template <class Fits>
__host__ __device__ __forceinline__ int largest_that(int most, Fits &&fits)
{
#ifdef __HIP_DEVICE_COMPILE__
    for (int from = most; from >= 1; from -= 64) {
        const int mine = from - (int)(threadIdx.x & 63u);
        const unsigned long long yes = __ballot(mine >= 1 && fits(mine));
        if (yes) return from - __builtin_ctzll(yes);
    }
#else
    for (int g = most; g >= 1; g--)
        if (fits(g)) return g;
#endif
    return 0;
}

// Share `b` of `n` of all rows of the items, cls[k] of them of class k; by a whole wavefront (on the host: for qmoe_hook_rows_shares).
// (Double precision in place of 64-bit integer divisions, each of which is a hundred instructions: a place is the same function of its
// cost for the share that ends there and the one that begins there, so rounding moves a boundary by a few rows at most and loses none.)
__host__ __device__ __forceinline__ RowsShare rows_share(const int (&cls)[4], const RowsSplit &sp, int n, int b)
{
    const int n_items = cls[1] + cls[2] + cls[3], rows = sp.rows, eights = (rows + 7) >> 3;
    RowsShare s{0, 0, -1, 0};
    if (n_items < 1) return s;
    double total = 0.0;  // in costs of eight rows
#pragma unroll
    for (int k = 1; k < 4; k++) total += (double)cls[k] * (double)(kRowCost[k] * eights);
    // With fewer items than workgroups every workgroup can have a part of one item: a tile of class k is cut into
    // ceil(cost[k] / t) parts, t the smallest cost of a part for which the parts of all items fit the grid.
    int g = 0, parts[4] = {0, 0, 0, 0}, used = 0, top_cost = 1;
    if (n_items <= n) {
        int top = 1;  // how many there are of the costliest class present
#pragma unroll
        for (int k = 3; k >= 1; k--) {
            top_cost = cls[k] ? kRowCost[k] : top_cost;
            top = cls[k] ? cls[k] : top;
        }
        const float inv_cost = near_rcp((float)top_cost);
        auto parts_of = [&](int k, int g_) { return (int)ceilf((float)(kRowCost[k] * g_) * inv_cost - 1e-3f); };
        // (an even split of the cost would give it this many; rounding up needs fewer, rarely by more than a few)
        const int most = min((int)((float)n * near_rcp((float)top) + 1e-3f),
                             (int)((float)(top_cost * eights) * (float)n * near_rcp((float)total)) + 1);
        g = largest_that(most, [&](int g_) {
            int need = 0;
#pragma unroll
            for (int k = 1; k < 4; k++) need += parts_of(k, g_) * cls[k];
            return need <= n;
        });
#pragma unroll
        for (int k = 1; k < 4; k++) {
            parts[k] = parts_of(k, g);
            used += parts[k] * cls[k];
        }
    }
    // That is uneven when there are nearly as many items as workgroups; equal shares of the whole list begin and
    // end inside items, so most workgroups have two items to stage and work on -- side by side if the activations of
    // both fit the LDS (then a few per cent are worth it), one after the other otherwise, each with too few rows for
    // all wavefronts.
    if (g >= 1 && (float)(top_cost * eights) * (float)n <= (sp.x_slots > 1 ? 1.08f : 1.25f) * (float)total * (float)g) {
        if (b >= used) return s;
        int item = 0, p = 1, at = -1, left = b;
#pragma unroll
        for (int k = 1; k < 4; k++) {
            const int here = cls[k] * parts[k];
            if (at < 0) {
                if (left < here) {
                    p = parts[k];
                    const int whole = (int)(((float)left + 0.5f) * near_rcp((float)p));
                    item += whole;
                    at = left - whole * p;
                } else {
                    left -= here;
                    item += cls[k];
                }
            }
        }
        const float step = (float)eights * near_rcp((float)p);
        s.i0 = s.i1 = item;
        s.r0 = 8 * (int)((float)at * step);
        s.r1 = at + 1 == p ? rows : 8 * (int)((float)(at + 1) * step);
    } else {
        // the place in the list where the first b_ shares end; rows in eights
        auto place = [&](int b_, int &item, int &row) {
            double c = floor(total * sp.inv_grid * (double)b_);
            item = row = 0;
            bool found = false;
#pragma unroll
            for (int k = 1; k < 4; k++) {
                const double per = (double)(kRowCost[k] * eights), here = (double)cls[k] * per;
                if (!found) {
                    if (c < here) {
                        const int i = min((int)(c * sp.inv_item[k]), cls[k] - 1);
                        const double in_item = c - (double)i * per;
                        item += i;
                        row = 8 * max(0, min((int)((float)in_item * (1.0f / (float)kRowCost[k])), eights));
                        found = true;
                    } else {
                        c -= here;
                        item += cls[k];
                    }
                }
            }
        };
#ifdef __HIP_DEVICE_COMPILE__
        int item, row;  // even lanes where the share begins, odd ones where it ends
        place(b + (int)(threadIdx.x & 1u), item, row);
        s.i0 = __builtin_amdgcn_readlane(item, 0);
        s.r0 = __builtin_amdgcn_readlane(row, 0);
        s.i1 = __builtin_amdgcn_readlane(item, 1);
        s.r1 = __builtin_amdgcn_readlane(row, 1);
#else
        place(b, s.i0, s.r0);
        place(b + 1, s.i1, s.r1);
#endif
        s.r1 = min(s.r1, rows);
        // (A whole item's cost times its reciprocal may fall short of one: the place is then behind that item's last row.)
        if (s.r0 >= rows) {
            s.i0++;
            s.r0 = 0;
        }
        if (b + 1 == n) {
            s.i1 = n_items - 1;
            s.r1 = rows;
        }
        if (s.i0 >= n_items) s.i1 = -1;
    }
    return s;
}

// The items of a share, in LDS: what a wavefront needs to know of each is read where it is needed (kept in registers for
// several items, it is more than the scalar registers hold).
constexpr int kKeptSegments = 6;  // items of a share looked at together
struct RowsSegment {
    int expert, slot0, ntok, ra, rb;  // rows ra .. rb of the item
    int tok[kMaxTokenTile];           // its tokens
};
using lp_segment = const __attribute__((address_space(3))) RowsSegment *;

// A record of a workgroup's share for the second product, written by the same workgroup of the first: the share, and
// {expert, slot0 | tokens << 16} of the items it begins with.
static_assert(kRowsShareBytes == 4 * (4 + 2 * kKeptSegments), "record size");
constexpr int kShareInts = 4 + 2 * kKeptSegments;

// ---- grouping the tokens by expert inside the first product
//
// In a small call (rows_can_dispatch) the grouping is a few thousand operations, less than the launch of a kernel for it and
// the trips to memory for its results: every workgroup does it for itself, in LDS, and leaves its part of the lists that
// k_dispatch would write in the workspace.
constexpr int kInlineTokens = 512;
constexpr size_t kInlineMaskBytes = 64 * 1024;

struct InlineLists {
    int cls[4], kept, experts;  // items by class, tokens with an expert, experts with tokens
    lp_u32 items;               // [n] {expert, slot0 | ntok << 16}
    const __attribute__((address_space(3))) int *perm;  // [kept]
    const __attribute__((address_space(3))) int *off;   // [E] first slot of every expert, or (few tokens) ...
    lp_u32 sorted;                                      // ... nullptr, and [kept] the slots' experts
};

__device__ __forceinline__ size_t inline_mask_words(int E, int T) { return (size_t)E * ((T + 31) >> 5); }

// Up to 64 tokens: all of it in the registers of wavefront 0, a lane a token.  A ballot per bit of the experts tells a lane
// which tokens have the same expert and which a smaller one.  `e` the lane's expert (-1: none).
__device__ __forceinline__ void group_few(const DispatchArgs &d, int e, int *perm, uint32_t *items, uint32_t *sorted, int *totals)
{
    const int E = d.n_experts, lane = (int)threadIdx.x;
    const bool valid = e >= 0;
    const int key = valid ? e : E;  // (behind all experts)
    uint32_t eq[2] = {~0u, ~0u}, less[2] = {0u, 0u};
    for (int b = 31 - __builtin_clz(E); b >= 0; b--) {
        const uint32_t one = (uint32_t)__builtin_amdgcn_sbfe(key, (uint32_t)b, 1u);  // 0 or all ones
        const unsigned long long ones = __ballot(one != 0u);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const uint32_t o = (uint32_t)(ones >> (32 * h));
            less[h] |= eq[h] & ~o & one;
            eq[h] &= ~(o ^ one);
        }
    }
    const int rank = (int)__builtin_amdgcn_mbcnt_hi(eq[1], __builtin_amdgcn_mbcnt_lo(eq[0], 0u));
    const int slot = __popc(less[0]) + __popc(less[1]) + rank, left = __popc(eq[0]) + __popc(eq[1]) - rank;
    const int kept = __popcll(__ballot(valid));
    // into the slots' order: experts in order, an expert's tokens in theirs; a tile begins at every d.tb_wi-th (a power of two)
    if (valid) {
        const bool head = (rank & (d.tb_wi - 1)) == 0;
        perm[slot] = lane;
        items[slot] = (uint32_t)e | (head ? (uint32_t)min(left, d.tb_wi) << 16 : 0u) | (rank == 0 ? 1u << 24 : 0u);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t v = lane < kept ? items[lane] : 0u;
    const int expert = (int)(v & 0xFFFFu), m = (int)((v >> 16) & 0xFFu);
    if (lane < kept) sorted[lane] = (uint32_t)expert;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int base = 0, to = 0;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        const bool here = m > 0 && tile_class(m) == c;
        const unsigned long long all = __ballot(here);
        if (here) to = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
        base += __popcll(all);
        if (lane == c) totals[c] = __popcll(all);
    }
    if (m > 0) {
        items[2 * to] = (uint32_t)expert;
        items[2 * to + 1] = (uint32_t)lane | (uint32_t)m << 16;
    }
    const int experts = __popcll(__ballot((v >> 24) != 0u));
    if (lane == 0) {
        totals[4] = kept;
        totals[5] = experts;
    }
}

// More tokens: a bit per token and expert gives a token's rank among its expert's tokens and the expert's count; experts in
// order give slots and items (longest class first).  `e` the expert of token threadIdx.x.  Barriers wait for LDS only.
__device__ __forceinline__ void group_many(const DispatchArgs &d, int e, uint32_t *mask, int *off, int *perm, uint32_t *items, int *tmp,
                                           int *totals)
{
    const int T = d.n_tokens, E = d.n_experts, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mw = (T + 31) >> 5;
    for (int i = tid; i < E * mw; i += kRowsThreads) mask[i] = 0u;
    lds_barrier();
    if (e >= 0) atomicOr(&mask[e * mw + (tid >> 5)], 1u << (tid & 31));
    lds_barrier();
    const int chunk = (E + kRowsThreads - 1) / kRowsThreads, e0 = min(E, tid * chunk), e1 = min(E, e0 + chunk);
    // bits of words [0, to) of an expert's mask: four reads in flight
    auto bits = [&](int x, int to) {
        int n = 0;
        for (int w = 0; w < to; w += 4) {
            uint32_t v[4];
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = mask[x * mw + min(w + k, mw - 1)];
#pragma unroll
            for (int k = 0; k < 4; k++) n += w + k < to ? __popc(v[k]) : 0;
        }
        return n;
    };
    auto count = [&](int x) { return bits(x, mw); };
    const int kw = tile_class(d.tb_wi), log2_tb = __builtin_ctz(d.tb_wi);
    int sums[3] = {0, 0, 0};  // two 16-bit counts each: tokens | class 0, class 1 | class 2, class 3 | experts with tokens
    int n_first = 0;
    for (int x = e0; x < e1; x++) {
        const int n = count(x);
        if (x == e0) n_first = n;
        if (n) {
            const int whole = n >> log2_tb, rest = n & (d.tb_wi - 1), kr = rest ? tile_class(rest) : -1;
            auto of = [&](int k) { return (k == kw ? whole : 0) + (k == kr ? 1 : 0); };
            sums[0] += n | of(0) << 16;
            sums[1] += of(1) | of(2) << 16;
            sums[2] += of(3) | 1 << 16;
        }
    }
    // prefix sums: within the wavefronts, then every wavefront adds up the totals of those before it
    constexpr int waves = kRowsThreads / 64;
    int before[3], all[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        before[k] = wave_inclusive_scan(sums[k]);
        if (lane == 63) tmp[k * waves + wave] = before[k];
        before[k] -= sums[k];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int run = row_scan16(lane < waves ? tmp[k * waves + lane] : 0);
        all[k] = __builtin_amdgcn_readlane(run, waves - 1);
        before[k] += wave ? __builtin_amdgcn_readlane(run, __builtin_amdgcn_readfirstlane(wave) - 1) : 0;
    }
    const int cls[4] = {all[0] >> 16, all[1] & 0xFFFF, all[1] >> 16, all[2] & 0xFFFF};
    int slot = before[0] & 0xFFFF;
    int at[4] = {before[0] >> 16, cls[0] + (before[1] & 0xFFFF), cls[0] + cls[1] + (before[1] >> 16),
                 cls[0] + cls[1] + cls[2] + (before[2] & 0xFFFF)};
    for (int x = e0; x < e1; x++) {
        const int n = x == e0 ? n_first : count(x);
        off[x] = slot;
        const int whole = n >> log2_tb, rest = n & (d.tb_wi - 1), kr = tile_class(rest);
        int first = 0, last = 0;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            if (c == kw) {
                first = at[c];
                at[c] += whole;
            }
            if (c == kr && rest) last = at[c]++;
        }
        for (int i = 0; i < whole; i++) {
            items[2 * (first + i)] = (uint32_t)x;
            items[2 * (first + i) + 1] = (uint32_t)(slot + (i << log2_tb)) | (uint32_t)d.tb_wi << 16;
        }
        if (rest) {
            items[2 * last] = (uint32_t)x;
            items[2 * last + 1] = (uint32_t)(slot + (whole << log2_tb)) | (uint32_t)rest << 16;
        }
        slot += n;
    }
    if (tid < 4) totals[tid] = tid == 0 ? cls[0] : (tid == 1 ? cls[1] : (tid == 2 ? cls[2] : cls[3]));
    if (tid == 4) totals[4] = all[0] & 0xFFFF;
    if (tid == 5) totals[5] = all[2] >> 16;
    lds_barrier();
    if (e >= 0) {
        int rank = bits(e, tid >> 5);
        rank += __popc(mask[e * mw + (tid >> 5)] & ((1u << (tid & 31)) - 1u));
        perm[off[e] + rank] = tid;
    }
}

// `scratch`: LDS of inline_lds_bytes(E, T); `e` the expert of token threadIdx.x (-1: none).
__device__ __forceinline__ InlineLists group_tokens(const DispatchArgs &d, int e, unsigned char *scratch)
{
    const int T = d.n_tokens, E = d.n_experts;
    const bool few = T <= 64;
    int *totals = reinterpret_cast<int *>(scratch);                      // [8]
    uint32_t *mask = reinterpret_cast<uint32_t *>(totals + 8);           // (few tokens: none)
    int *off = reinterpret_cast<int *>(mask + (few ? 0 : inline_mask_words(E, T)));  // [E] first slot; few tokens: [T] experts by slot
    int *perm = off + (few ? T : E);                                     // [T]
    uint32_t *items = reinterpret_cast<uint32_t *>(perm + T);            // [2 T]
    int *tmp = reinterpret_cast<int *>(items + 2 * T);                   // [3 * 16] scan scratch
    if (few) {
        if (threadIdx.x < 64) group_few(d, e, perm, items, reinterpret_cast<uint32_t *>(off), totals);
    } else {
        group_many(d, e, mask, off, perm, items, tmp, totals);
    }
    lds_barrier();
    InlineLists r;
#pragma unroll
    for (int k = 0; k < 4; k++) r.cls[k] = __builtin_amdgcn_readfirstlane(totals[k]);
    r.kept = __builtin_amdgcn_readfirstlane(totals[4]);
    r.experts = __builtin_amdgcn_readfirstlane(totals[5]);
    r.items = (lp_u32)items;
    r.perm = (const __attribute__((address_space(3))) int *)perm;
    r.off = few ? nullptr : (const __attribute__((address_space(3))) int *)off;
    r.sorted = (lp_u32)(uint32_t *)off;
    return r;
}

// The lists as k_dispatch leaves them in the workspace, a part by every workgroup (one that wrote them all would be the last
// to begin its rows).
__device__ __forceinline__ void record_lists(const DispatchArgs &d, const InlineLists &r)
{
    const int i0 = (int)(threadIdx.x * gridDim.x + blockIdx.x), step = kRowsThreads * (int)gridDim.x;
    const int n = r.cls[0] + r.cls[1] + r.cls[2] + r.cls[3], E = d.n_experts;
    for (int i = i0; i <= E; i += step) {
        int slot = r.kept;  // slots below expert i
        if (i < E) {
            if (r.off) {
                slot = r.off[i];
            } else {
                int lo = 0;
                for (int half = 64; half >= 1; half >>= 1)
                    if (lo + half <= r.kept && (int)r.sorted[lo + half - 1] < i) lo += half;
                slot = lo;
            }
        }
        d.tok_off[i] = slot;
    }
    if (i0 < n) {
        const uint32_t v = r.items[2 * i0 + 1];
        d.items_wi[i0] = d.items_wo[i0] = Item{(int)r.items[2 * i0], (int)(v & 0xFFFFu), (int)(v >> 16), 0};
    }
    if (i0 < r.kept) d.perm[i0] = r.perm[i0];
    if (blockIdx.x == 0 && threadIdx.x < kLayerCounters) {
        const int k = (int)threadIdx.x;
        int v = 0;
        v = k == 0 ? r.kept : v;
        v = k == 1 ? d.n_tokens - r.kept : v;
        v = k == 2 ? r.experts : v;
        v = k == 3 || k == 4 ? n : v;
        v = k == 10 ? r.cls[0] : (k == 11 ? r.cls[1] : (k == 12 ? r.cls[2] : (k == 13 ? r.cls[3] : v)));
        d.counters[k] = v;
    }
}

// Activations of a tile on their way to LDS: column pairs threadIdx.x, + 1024, ... of up to four tokens.  All loads are
// issued before the first store (a loop that loads and stores a piece at a time waits for every load in turn: 4 us for
// four tokens of 3072 columns).
template <int PIECES = 4>  // 8192 columns
struct XPairs {
    static constexpr int kPieces = PIECES;
    uint32_t v[kPieces][4];
};
typedef uint32_t u32_any __attribute__((aligned(2)));
using gp_u32_any = const __attribute__((address_space(1))) u32_any *;

template <int PIECES>
__device__ __forceinline__ void x_load(XPairs<PIECES> &p, const uint16_t *x, const int (&row)[4], int ntok, int ldx, int cols, int base)
{
    uintptr_t src[4];
#pragma unroll
    for (int t = 0; t < 4; t++) src[t] = reinterpret_cast<uintptr_t>(x) + 2u * ((uintptr_t)(uint32_t)row[t] * (uint32_t)ldx);
#pragma unroll
    for (int k = 0; k < PIECES; k++) {
        const int c = 2 * (base + k * kRowsThreads + (int)threadIdx.x);
        const uintptr_t at = 2 * (uintptr_t)(uint32_t)min(c, cols - 2);
        if (2 * (base + k * kRowsThreads) < cols) {  // (uniform)
            p.v[k][0] = *(gp_u32_any)(src[0] + at);
            if (ntok > 1) p.v[k][1] = *(gp_u32_any)(src[1] + at);
            if (ntok > 2) {
                p.v[k][2] = *(gp_u32_any)(src[2] + at);
                p.v[k][3] = *(gp_u32_any)(src[3] + at);
            }
        }
    }
}

// One token: records {0, +x, 0, -x}; more: four tokens a column (a tile of two is read as two).  Behind the last token of three
// stand zeros: a field's dot product takes the neighbour in with a weight of zero, and an infinity would make that a NaN.
template <int PIECES>
__device__ __forceinline__ void x_store(const XPairs<PIECES> &p, unsigned char *xs, int ntok, int cols, int base)
{
#pragma unroll
    for (int k = 0; k < PIECES; k++) {
        if (2 * (base + k * kRowsThreads) >= cols) break;  // (uniform)
        const int c = 2 * (base + k * kRowsThreads + (int)threadIdx.x);
        u32x4 o;
        if (ntok <= 1) {
            const uint32_t v = p.v[k][0];
            o.x = v << 16;
            o.y = o.x ^ 0x80000000u;
            o.z = v & 0xFFFF0000u;
            o.w = o.z ^ 0x80000000u;
        } else {
            o.x = __builtin_amdgcn_perm(p.v[k][1], p.v[k][0], 0x05040100u);
            o.y = __builtin_amdgcn_perm(p.v[k][3], p.v[k][2], 0x05040100u);
            o.z = __builtin_amdgcn_perm(p.v[k][1], p.v[k][0], 0x07060302u);
            o.w = __builtin_amdgcn_perm(p.v[k][3], p.v[k][2], 0x07060302u);
            if (ntok == 3) {
                o.y &= 0xFFFFu;
                o.w &= 0xFFFFu;
            }
        }
        if (c < cols) *reinterpret_cast<u32x4 *>(xs + 8 * (size_t)c) = o;
    }
}

// zeros behind a tile's last column
__device__ __forceinline__ void x_pad(unsigned char *xs, int cols)
{
    static_assert(kRowsPadCols % 2 == 0 && kRowsPadCols / 2 <= kRowsThreads, "a pair a thread");
    if ((int)threadIdx.x < kRowsPadCols / 2) *reinterpret_cast<u32x4 *>(xs + 8 * (size_t)(cols + 2 * (int)threadIdx.x)) = u32x4{0u, 0u, 0u, 0u};
}

// LDS of the shares, segments and gates
constexpr int kRowsSmallBytes = (4 * 8 + (int)sizeof(RowsSegment) * kKeptSegments + 4 * 2 * kMaxTokenTile + 15) / 16 * 16;

// The table on its way to LDS: asked for first of all, stored when the loads that the rows wait for are on their way.  (Pieces of
// 16 bytes, the last one perhaps reaching into the space behind the table's last entry: the blob reserves kMaxOrderTable entries.)
struct TablePieces {
    static constexpr int kPieces = (kMaxOrderTable / 4 + kRowsThreads - 1) / kRowsThreads;
    u32x4 v[kPieces];
};

__device__ __forceinline__ void table_load(TablePieces &p, const uint32_t *table, int n)
{
    const int n4 = (n + 3) >> 2;
#pragma unroll
    for (int k = 0; k < TablePieces::kPieces; k++) p.v[k] = ((gp_u32x4)table)[min(k * kRowsThreads + (int)threadIdx.x, n4 - 1)];
}

__device__ __forceinline__ void table_store(const TablePieces &p, uint32_t *table_lds, int n)
{
    const int n4 = (n + 3) >> 2;
#pragma unroll
    for (int k = 0; k < TablePieces::kPieces; k++) {
        const int i = k * kRowsThreads + (int)threadIdx.x;
        if (i < n4) reinterpret_cast<u32x4 *>(table_lds)[i] = p.v[k];
    }
}

// The items of a batch (one or two, worked on side by side), the same in every lane.
struct RowsBatchItem {
    int expert, slot0, ntok, ra, rb;
};

// GROUP: the launch groups the tokens itself (first product of a small call); split2: of the second product, for whose
// shares it leaves records.
//
// Small calls are bound by the way to the first codeword: share -> descriptor -> row offsets -> codewords, each a trip to
// memory, with the table, the activations and the grouping beside them.  So the table is asked for first and stored last, a
// second product's record is read by every wavefront itself, what wavefront 0 works out goes round with one barrier, and no
// barrier waits for a load or a store of global memory (__syncthreads does).  One token on 2048 experts of 2080 x 6144: 21.5 -> 17.3 us;
// 128 on 128 of 768 x 3072: 45.6 -> 41.7; 512 on 128 of 1024 x 4096: 119.5 -> 114.8.
// (Tried and slower: eight wavefronts, 45.3 us for the second; the table straight into LDS with one copy of the staging code, for which
// registers spill, 47.9; what follows the grouping in one copy more of the code: the two kernels of a call do not fit the 64 KB of
// the instruction cache together then.)
template <int EPI, int ASYM, bool GROUP, int LANES>
__global__ __launch_bounds__(kRowsThreads) void k_rows(const ProductArgs a, const DispatchArgs d, const RowsSplit split, const RowsSplit split2)
{
    extern __shared__ __align__(16) unsigned char smem[];
    // LDS: table | shares and segments | gates of the tiles in work | activations of one or two tiles (before that, the lists
    // of the grouping)
    uint32_t *table_w = reinterpret_cast<uint32_t *>(smem);
    const size_t table_bytes = ((size_t)a.n_order * 4 + 15) & ~(size_t)15;
    int *share_s = reinterpret_cast<int *>(smem + table_bytes);                       // [8]
    RowsSegment *seg_s = reinterpret_cast<RowsSegment *>(share_s + 8);                // [kKeptSegments]
    float *gate_s = reinterpret_cast<float *>(seg_s + kKeptSegments);                 // [2][kMaxTokenTile]
    unsigned char *xs0 = smem + table_bytes + kRowsSmallBytes;
    const size_t xs_bytes = (size_t)(a.cols + kRowsPadCols) * max(a.tb_max, 4) * sizeof(uint16_t);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    constexpr int waves = kRowsThreads / 64;

    // A large call whose experts all have many tokens: nothing to do, and the matrix-core kernel waits for the compute units.  Seen
    // before the table is staged (3156 tokens on 28 experts of 392 x 3136 179.5 -> 178.4 us, 2943 on 10 of 1784 x 1360
    // 166.1 -> 165.5; not so 3532 on 132 of 640 x 1152, where the delay had the two chains' kernels meet better, 174.5 -> 178.7).
    if constexpr (!GROUP) {
        if (a.items && !a.shares && (a.class_counts[0] | a.class_counts[1] | a.class_counts[2] | a.class_counts[3]) == 0) return;
    }
    const bool recorded = !GROUP && a.shares && a.x_by_slot;  // the share is in a record of the first product's

    // ---- the first loads, in the order in which they are wanted
    int e = -1, record = 0;
    if constexpr (GROUP) {
        if ((int)threadIdx.x < d.n_tokens) e = d.expert_idx[threadIdx.x];
    } else if (recorded) {
        record = a.shares[blockIdx.x * kShareInts + (lane & (kShareInts - 1))];
    }
    TablePieces tp;
    table_load(tp, a.order_table, a.n_order);

    // ---- this workgroup's share of the rows
    InlineLists lists;
    if constexpr (GROUP) {
        if (e < 0 || e >= d.n_experts) e = -1;
        // The output rows of tokens without an expert are cleared by all workgroups, a row at a time and in whole lines: a rank
        // that holds a part of the experts has mostly such tokens (512 tokens, 448 of them without an expert, on experts of
        // 768 x 3072: 230 us when a thread of workgroup 0 cleared a row, 38 us now; 2080 x 6144: 559 and 89 us).  Here,
        // among the first loads: behind the grouping it cost calls on the asymmetric grid 0.7 us.
        for (int t = (int)blockIdx.x; t < d.n_tokens; t += (int)gridDim.x) {
            const int et = d.expert_idx[t];
            if (et < 0 || et >= d.n_experts)
                for (int c = (int)threadIdx.x; c < d.d_model; c += kRowsThreads)
                    ((__attribute__((address_space(1))) float *)d.y)[(size_t)t * d.d_model + c] = 0.0f;
        }
        lists = group_tokens(d, e, xs0);
    }
    // The items a share has at `i_base` and behind it, into LDS: by wavefront 0, eight lanes for each item, a token apiece.
    struct SegmentPart {
        int expert, slot0, ntok, tok;
        bool ok;
    };
    const int seg_k = lane / kMaxTokenTile, seg_t = lane % kMaxTokenTile;
    auto load_segments = [&](const RowsShare &sh, int i_base) -> SegmentPart {
        const int i = i_base + seg_k;
        SegmentPart p{-1, 0, 0, 0, false};
        const int rec_expert = GROUP ? 0 : __shfl(record, 4 + 2 * seg_k, 64), rec_at = GROUP ? 0 : __shfl(record, 5 + 2 * seg_k, 64);
        if (i <= sh.i1 && seg_k < kKeptSegments) {
            if constexpr (GROUP) {
                p.expert = (int)lists.items[2 * i];
                p.slot0 = (int)(lists.items[2 * i + 1] & 0xFFFFu);
                p.ntok = (int)(lists.items[2 * i + 1] >> 16);
            } else if (recorded) {  // (such a share is looked at in one go)
                p.expert = rec_expert;
                p.slot0 = rec_at & 0xFFFF;
                p.ntok = rec_at >> 16;
            } else if (a.items) {
                const Item it = a.items[i];
                p.expert = it.expert;
                p.slot0 = it.slot0;
                p.ntok = it.ntok;
            } else {
                p.expert = 0;
                p.slot0 = i * a.tb_max;
                p.ntok = a.batch - p.slot0;
            }
        }
        p.ntok = min(p.ntok, a.tb_max);
        p.ok = p.expert >= 0 && p.expert < a.n_experts && p.ntok > 0;
        if (p.ok) {
            const int at = p.slot0 + min(seg_t, p.ntok - 1);
            if constexpr (GROUP) p.tok = lists.perm[at];
            else p.tok = a.perm ? a.perm[at] : at;
        }
        return p;
    };
    auto store_segments = [&](const SegmentPart &p, const RowsShare &sh, int i_base) {
        const int i = i_base + seg_k;
        if (seg_k >= kKeptSegments) return;
        RowsSegment &g = seg_s[seg_k];
        if (seg_t == 0) {
            g.expert = p.ok ? p.expert : 0;
            g.slot0 = p.slot0;
            g.ntok = p.ntok;
            g.ra = i == sh.i0 ? sh.r0 : 0;
            g.rb = !p.ok ? g.ra : (i == sh.i1 ? sh.r1 : a.rows);
        }
        g.tok[seg_t] = p.tok;
    };
    SegmentPart seg_own{};  // (recorded: stored with the table)
    RowsShare sh;
    if (recorded) {
        sh = RowsShare{__builtin_amdgcn_readlane(record, 0), __builtin_amdgcn_readlane(record, 1), __builtin_amdgcn_readlane(record, 2),
                       __builtin_amdgcn_readlane(record, 3)};
        if (wave == 0) seg_own = load_segments(sh, sh.i0);
    } else {
        if (wave == 0) {
            if constexpr (GROUP) {
                sh = rows_share(lists.cls, split, (int)gridDim.x, (int)blockIdx.x);
            } else {
                int cls[4];
                if (a.items) {
#pragma unroll
                    for (int k = 0; k < 4; k++) cls[k] = a.class_counts[k];
                } else {
                    const int n = (a.batch + a.tb_max - 1) / a.tb_max;
                    cls[0] = 0;
                    cls[1] = a.tb_max > 2 ? n : 0;
                    cls[2] = a.tb_max == 2 ? n : 0;
                    cls[3] = a.tb_max == 1 ? n : 0;
                }
                sh = rows_share(cls, split, (int)gridDim.x, (int)blockIdx.x);
            }
            if (lane == 0) {
                share_s[0] = sh.i0;
                share_s[1] = sh.r0;
                share_s[2] = sh.i1;
                share_s[3] = sh.r1;
            }
            store_segments(load_segments(sh, sh.i0), sh, sh.i0);
        }
        if constexpr (GROUP) {
            if (wave == 1 && a.shares) {  // the second product's share
                const RowsShare s2 = rows_share(lists.cls, split2, (int)gridDim.x, (int)blockIdx.x);
                const int n = lists.cls[0] + lists.cls[1] + lists.cls[2] + lists.cls[3], i = min(s2.i0 + ((lane - 4) >> 1), n - 1);
                const int place = lane == 0 ? s2.i0 : (lane == 1 ? s2.r0 : (lane == 2 ? s2.i1 : s2.r1));
                if (lane < kShareInts)
                    a.shares[blockIdx.x * kShareInts + lane] = lane < 4 ? place : (n ? (int)lists.items[2 * i + (lane & 1)] : 0);
            }
            record_lists(d, lists);
        }
        lds_barrier();
        sh = RowsShare{__builtin_amdgcn_readfirstlane(share_s[0]), __builtin_amdgcn_readfirstlane(share_s[1]),
                       __builtin_amdgcn_readfirstlane(share_s[2]), __builtin_amdgcn_readfirstlane(share_s[3])};
    }
    if (sh.i0 > sh.i1 || (sh.i0 == sh.i1 && sh.r0 >= sh.r1)) return;

    // lanes per row for so many rows: the fewest for which the rounds of the workgroup's wavefronts, each as long as a
    // row's pieces over its lanes plus the round's own start and end (one or one and a half more), are shortest
    auto lanes_log2 = [&](uint32_t rows_here) -> int {
        uint32_t best = 0xFFFFFFFFu;
        int log2L = 0;
#pragma unroll
        for (int l = 0; l <= 6; l++) {
            const uint32_t cost = (((rows_here << l) + (uint32_t)kRowsThreads - 1u) / (uint32_t)kRowsThreads) * split.round_cost[l];
            log2L = cost < best ? l : log2L;
            best = min(best, cost);
        }
        return log2L;
    };
    RowsBatchItem b[2];
    int log2L = 0, groups0 = 0, head_k = 0;
    bool have = false;  // the wavefront has rows in the batch: its first group (of item head_k), begun in `head`
    GroupHead head{};
    // ---- a batch of one or two items: activations and the wavefront's first rows asked for, in this order; `meanwhile` runs
    // ahead of what has to wait for the row offsets (and says which token a lane of wavefront 0 holds, -1: ask the segments)
    auto stage = [&](lp_segment g0, lp_segment g1, auto meanwhile) {
        // the input rows of the tiles (of tokens past a tile's last: the last's again)
        int xrow[2][4];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (b[k].ra >= b[k].rb) continue;
            if (a.x_by_slot) {
#pragma unroll
                for (int t = 0; t < 4; t++) xrow[k][t] = b[k].slot0 + min(t, b[k].ntok - 1);
            } else {
                lp_segment g = k ? g1 : g0;
                int tok[4];
#pragma unroll
                for (int t = 0; t < 4; t++) tok[t] = g->tok[t];
#pragma unroll
                for (int t = 0; t < 4; t++) xrow[k][t] = __builtin_amdgcn_readfirstlane(tok[t]);
            }
        }
        log2L = lanes_log2((uint32_t)((b[0].rb - b[0].ra) + (b[1].rb - b[1].ra)));
        const int R = 64 >> log2L;
        groups0 = (b[0].rb - b[0].ra + R - 1) >> (6 - log2L);
        head_k = wave < groups0 ? 0 : 1;
        const int head_rb = head_k ? b[1].rb : b[0].rb, head_r = head_k ? b[1].ra + (wave - groups0) * R : b[0].ra + wave * R;
        have = head_r < head_rb;
        XPairs<> px[2];
#pragma unroll
        for (int k = 0; k < 2; k++)
            if (b[k].ra < b[k].rb) x_load(px[k], a.x, xrow[k], b[k].ntok, a.ldx, a.cols, 0);
        const int expert = head_k ? b[1].expert : b[0].expert;
        if (have) {
            const qmoe_matrix M = matrix_of(a, expert);
            head_offsets<ASYM, LANES>(split, M, head_rb, head_r + (lane >> log2L), head);
        }
        // (wavefront 0: the gates of the tiles' tokens)
        const bool gates = EPI == 0 && wave == 0 && lane < 2 * kMaxTokenTile;
        const int own = meanwhile();
        float gate = 1.0f;
        if (gates && a.gate) gate = a.gate[own >= 0 ? own : (lane < kMaxTokenTile ? g0 : g1)->tok[lane % kMaxTokenTile]];
        if (have) {
            const qmoe_matrix M = matrix_of(a, expert);
            head.v = RowPieces<LANES>(M, head, head_r + (lane >> log2L) < head_rb).load(lane & ((1 << log2L) - 1));
        }
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (b[k].ra >= b[k].rb) continue;
            unsigned char *xs = xs0 + (k ? xs_bytes : 0);
            x_store(px[k], xs, b[k].ntok, a.cols, 0);
            x_pad(xs, a.cols);
            for (int base = XPairs<>::kPieces * kRowsThreads; 2 * base < a.cols; base += kRowsThreads) {  // wide tiles
                XPairs<1> more;
                x_load(more, a.x, xrow[k], b[k].ntok, a.ldx, a.cols, base);
                x_store(more, xs, b[k].ntok, a.cols, base);
            }
        }
        if (gates) gate_s[lane] = gate;
    };
    // (Another fill of the segments than the first only in large calls: small ones have few items a share.)
    int i = sh.i0, i_base = sh.i0;
    auto segment = [&](int k) { return (lp_segment)(seg_s + min(i - i_base + k, kKeptSegments - 1)); };
    auto batch_of = [&]() {
#pragma unroll
        for (int k = 0; k < 2; k++) {
            lp_segment g = segment(k);
            b[k].expert = __builtin_amdgcn_readfirstlane(g->expert);
            b[k].slot0 = __builtin_amdgcn_readfirstlane(g->slot0);
            b[k].ntok = __builtin_amdgcn_readfirstlane(g->ntok);
            b[k].ra = __builtin_amdgcn_readfirstlane(g->ra);
            b[k].rb = __builtin_amdgcn_readfirstlane(g->rb);
        }
    };
    auto one_or_two = [&]() {
        if (split.x_slots < 2 || i + 1 > sh.i1) b[1].rb = b[1].ra;
    };
    if (recorded) {
        // (not from LDS: wavefront 0 puts it there below)
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int expert = __builtin_amdgcn_readlane(record, 4 + 2 * k), at = __builtin_amdgcn_readlane(record, 5 + 2 * k);
            const int ntok = min(at >> 16, a.tb_max);
            const bool ok = expert >= 0 && expert < a.n_experts && ntok > 0;
            b[k].expert = ok ? expert : 0;
            b[k].slot0 = at & 0xFFFF;
            b[k].ntok = ntok;
            b[k].ra = k ? 0 : sh.r0;
            b[k].rb = !ok ? b[k].ra : (sh.i0 + k == sh.i1 ? sh.r1 : a.rows);
        }
    } else {
        batch_of();
    }
    one_or_two();
    stage(segment(0), segment(1), [&]() {
        table_store(tp, table_w, a.n_order);
        if (recorded && wave == 0) store_segments(seg_own, sh, sh.i0);
        return recorded ? seg_own.tok : -1;
    });
    for (;;) {
        lds_barrier();
        int group = wave;  // the wavefront's first group of rows of the item
        for (int k = 0; k < 2; k++) {
            const RowsBatchItem &it = k ? b[1] : b[0];
            if (it.ra >= it.rb) continue;
            lp_segment g = segment(k);
            const qmoe_matrix M = matrix_of(a, it.expert);
            const bool first = have && k == head_k;
            RowsTile tile;
            tile.ntok = it.ntok;
            tile.slot0 = it.slot0;
            tile.tok_ids = g->tok;
            tile.gate_s = (const __attribute__((address_space(3))) float *)(gate_s + k * kMaxTokenTile);
            const uint32_t xs_addr = (uint32_t)(uintptr_t)(lp_u16)(uint16_t *)(xs0 + (k ? xs_bytes : 0));
            if (tile.ntok <= 1) rows_block<1, EPI, ASYM, LANES>(a, split, M, it.ra, it.rb, group, log2L, xs_addr, tile, (lp_u32)table_w, head, first);
            else if (tile.ntok <= 2) rows_block<2, EPI, ASYM, LANES>(a, split, M, it.ra, it.rb, group, log2L, xs_addr, tile, (lp_u32)table_w, head, first);
            else rows_block<4, EPI, ASYM, LANES>(a, split, M, it.ra, it.rb, group, log2L, xs_addr, tile, (lp_u32)table_w, head, first);
            group = (group - groups0) & (waves - 1);  // the second item's groups go on where the first one's end
        }
        i += split.x_slots;
        if (i > sh.i1) break;
        lds_barrier();  // the tiles (and the segments) before are done with
        if constexpr (!GROUP) {
            if (i - i_base >= kKeptSegments) {
                i_base += kKeptSegments;
                if (wave == 0) store_segments(load_segments(sh, i_base), sh, i_base);
                lds_barrier();
            }
        }
        batch_of();
        one_or_two();
        stage(segment(0), segment(1), []() { return -1; });
    }
}

size_t rows_fixed_bytes(int n_order) { return (((size_t)n_order * 4 + 15) & ~(size_t)15) + kRowsSmallBytes; }
size_t rows_tile_bytes(int cols, int tb) { return (size_t)(cols + kRowsPadCols) * 2 * (size_t)std::max(tb, 4); }
size_t inline_lds_bytes(int E, int T)
{
    return 4 * std::max((size_t)E * ((T + 31) / 32) + (size_t)E + 3 * (size_t)T + 64, 4 * (size_t)T + 8);
}

}  // namespace

int rows_tile_slots(int cols, int tb, int n_order, int max_lds)
{
    const size_t fixed = rows_fixed_bytes(n_order), tile = rows_tile_bytes(cols, tb);
    return fixed + 2 * tile <= (size_t)max_lds ? 2 : (fixed + tile <= (size_t)max_lds ? 1 : 0);
}

bool rows_can_dispatch(int n_experts, int n_tokens, int grid, int n_order, int max_lds)
{
    // (a share then spans at most n_tokens / grid + 2 items: all items cost at least what one token's does)
    if (n_tokens > kInlineTokens || n_tokens > (kKeptSegments - 2) * grid) return false;
    // The table is in LDS already when the lists are made: with the paper's they fit up to about 12000 experts and 32 tokens.
    return 4 * (size_t)n_experts * ((n_tokens + 31) / 32) <= kInlineMaskBytes &&
           rows_fixed_bytes(n_order) + inline_lds_bytes(n_experts, n_tokens) <= (size_t)max_lds;
}

RowsSplit rows_split(int rows, int cols, int lanes, int x_slots, int grid)
{
    RowsSplit sp;
    sp.rows = rows;
    sp.x_slots = x_slots;
    sp.inv_item[0] = 0.0;
    for (int k = 1; k < 4; k++) sp.inv_item[k] = 1.0 / (double)(kRowCost[k] * ((rows + 7) / 8));
    sp.inv_grid = 1.0 / grid;
    for (int l = 0; l <= 6; l++) sp.round_cost[l] = (uint32_t)(2 * ((cols / 176 + (1 << l)) >> l) + 2 + (l > 0));
    sp.lanes = lanes;
    sp.inv_lanes = lanes ? 1.0f / (float)lanes : 0.0f;
    sp.lane_rows = lanes ? rows / lanes : 0;
    sp.lane_extra = lanes ? rows % lanes : 0;
    return sp;
}

void rows_shares(int rows, const int (&cls)[4], int x_slots, int grid, int *out)
{
    const RowsSplit sp = rows_split(rows, 0, 0, x_slots, grid);
    for (int b = 0; b < grid; b++) {
        const RowsShare s = rows_share(cls, sp, grid, b);
        const int v[4] = {s.i0, s.r0, s.i1, s.r1};
        std::copy(v, v + 4, out + 4 * b);
    }
}

qmoe_status launch_rows(const ProductArgs &a, int x_slots, const DispatchArgs *da, int rows2, int x_slots2, int grid, int max_lds,
                        hipStream_t s)
{
    if (a.tb_max > kRowsTokenTile) return QMOE_E_LIMIT;
    size_t tiles = rows_tile_bytes(a.cols, a.tb_max) * (size_t)x_slots;
    if (da) tiles = std::max(tiles, inline_lds_bytes(da->n_experts, da->n_tokens));
    const size_t smem = rows_fixed_bytes(a.n_order) + tiles;
    if (smem > (size_t)max_lds) return QMOE_E_LIMIT;
    DispatchArgs d{};
    RowsSplit split2{};
    if (da) {
        d = *da;
        split2 = rows_split(rows2, 0, 0, x_slots2, grid);  // (its shares only)
    }
    const RowsSplit split = rows_split(a.rows, a.cols, a.lanes, x_slots, grid);
    auto launch = [&](auto kernel) -> qmoe_status {
        const qmoe_status st = allow_lds(kernel, smem);
        if (st != QMOE_OK) return st;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kRowsThreads), smem, s, a, d, split, split2);
        return QMOE_OK;
    };
    auto choose = [&](auto lanes) -> qmoe_status {
        constexpr int LANES = decltype(lanes)::value;
        if (da) return a.minmax ? launch(k_rows<1, 1, true, LANES>) : launch(k_rows<1, 0, true, LANES>);
        if (a.minmax) return a.epilogue ? launch(k_rows<1, 1, false, LANES>) : launch(k_rows<0, 1, false, LANES>);
        return a.epilogue ? launch(k_rows<1, 0, false, LANES>) : launch(k_rows<0, 0, false, LANES>);
    };
    const qmoe_status st = a.lanes ? choose(std::integral_constant<int, 1>{}) : choose(std::integral_constant<int, 0>{});
    if (st != QMOE_OK) return st;
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

}  // namespace qmoe
