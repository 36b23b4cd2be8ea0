// Step one of a layer call: tokens grouped by expert (stable), experts without tokens
// skipped (Section 5.1 of the paper), work lists for the product kernels.
#include "qmoe_dev.h"

namespace qmoe {
namespace {

// ---------------------------------------------------------------- dispatch
//
// One workgroup of up to 1024 threads groups the tokens by expert (stable) and writes the work lists of both products; the
// others of the launch clear the output rows of tokens without an expert.
//
// The tokens are cut into `parts` contiguous parts of whole 64s, and every part has a row of counts of its own in LDS, one
// per expert.  An expert's counts, added up over the parts before, are where each part's tokens of that expert begin, so in
// the end every part is scattered by a wavefront of its own, 64 tokens at a time, without a word to the others.
//
// Bound: a chain of trips to memory and barriers in one workgroup.  4001 tokens on 128 experts 28.5 us with one wavefront
// that walked all tokens' chunks and a rank by 64 broadcasts, now 8.3; 4224 on 256 34.4, now 9.0; 2048 on 2048 19.6, now 11.4;
// 100000 on 2048 596 us, now 106.
constexpr int kClearGrid = 64;  // workgroups that clear rows, at most

// The lanes whose token has the same expert: experts are told apart by their bits, one ballot each (experts below 2^bits).
__device__ __forceinline__ unsigned long long same_expert(int e, int bits)
{
    uint32_t lo = ~0u, hi = ~0u;
    for (int b = 0; b < bits; b++) {
        const uint32_t one = (uint32_t)__builtin_amdgcn_sbfe(e, (uint32_t)b, 1u);  // 0 or all ones
        const unsigned long long ones = __ballot(one != 0u);
        lo &= ~((uint32_t)ones ^ one);
        hi &= ~((uint32_t)(ones >> 32) ^ one);
    }
    return (unsigned long long)hi << 32 | lo;
}

// An expert's n tokens as tiles of `tb` and a rest, in the lists of their classes.  (The whole tiles first, without a choice of
// class in the loop: a crowded expert's tiles are one thread's work; 600 tokens on 128 experts, Zipf routing, 10.6 us with it, 7.3
// without.)
__device__ __forceinline__ void put_tiles(Item *items, int (&at)[4], int e, int slot, int n, int tb)
{
    const int whole = n / tb, rest = n - whole * tb;
    const int kw = tile_class(tb), kr = tile_class(rest);
    int first = 0, last = 0;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if (c == kw) {
            first = at[c];
            at[c] += whole;
        }
        if (c == kr && rest) last = at[c]++;
    }
    for (int i = 0; i < whole; i++) items[first + i] = Item{e, slot + i * tb, tb, 0};
    if (rest) items[last] = Item{e, slot + whole * tb, rest, 0};
}

// Place of an expert in a row of counts: a word is left free after every 32, so that threads with 2, 4, ... 16 consecutive experts
// each do not meet on a few banks (16384 experts, 4100 tokens 57 us without, 51 with).
__host__ __device__ __forceinline__ int spread(int e) { return e + (e >> 5); }
__host__ __device__ __forceinline__ int count_stride(int n_experts) { return spread(n_experts) + 1; }

// A call that may give all its experts to the matrix-core kernel: does it?  The host knows neither the routing nor how many tokens have an expert, and its
// rules (plan_mm) hold for calls in which nearly all have.  A pass of the few-token kernels, four tokens of an expert as a rule, decodes a matrix once, as a tile of 64
// does: where ten tiles are no more than mm_passes passes, all experts go to those kernels, which start sooner.  Us, matrix cores / few-token kernels / both,
// side by side on two streams: 716 experts of 696 x 680, 2422 tokens, uniform, asymmetric grid (12.7 passes for ten tiles) 163 / 134 / 157; 128 of 768 x 3072, 109
// of 1088 tokens left 86 / 57 / 60; 231 of 896 x 320, 1198 (16.7) 51 / 62 / 81.  Small layers lose from 14 on, large ones from 19 on (mm_passes 13 and 17).
// mm_split, large layers on the asymmetric grid: where tokens are missing and the experts below mm_else outnumber the other ones' tiles, both kernels one
// after the other are at worst 8 % slower than side by side, the matrix cores alone 15 % (122 of 1568 x 3464, 732 of 3457 tokens left, Zipf, 92 % zeros: 203 side by
// side, 210, 233).
// 2575 calls of 230 layers (1024 to 4100 tokens, 0 to 99 % of them without an expert, 0.15 to 10 * 10^8 weights a projection, both grids and routings, 80 to 92 % zeros):
// 0.79 of the time side by side, 1.08 at worst, six above 1.05; with only the host's lines, one kernel after the other below them, 0.88, 1.18 and 94.
// What it costs a call: 0.5 to 1 us (1024 threads that add to the same words of LDS one by one took 5 to 10).
template <int PARTS>
__device__ int choose_mm_min(const DispatchArgs &a, const int *cnt, int S, int e0, int e1, int kept, int *sums)
{
    int passes = 0, tiles = 0, few = 0, crowded = 0;
    for (int e = e0; e < e1; e++) {
        int n = 0;
#pragma unroll
        for (int p = 0; p < PARTS; p++) n += cnt[p * S + spread(e)];
        const int t = (n + kMmTokens - 1) / kMmTokens;
        passes += (n + kRowsTokenTile - 1) / kRowsTokenTile;
        tiles += t;
        if (n >= a.mm_else) crowded += t;
        else few += t;
    }
    const int v[4] = {passes, tiles, few, crowded};
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int wave_sum = wave_inclusive_scan(v[k]);  // (in lane 63)
        if ((threadIdx.x & 63) == 63 && wave_sum) atomicAdd(&sums[k], wave_sum);
    }
    __syncthreads();
    if (10LL * sums[0] <= (long long)a.mm_passes * sums[1]) return 0x7FFFFFFF;
    return a.mm_split && kept < a.mm_from && sums[2] > sums[3] ? a.mm_else : a.mm_min;
}

template <int PARTS>
__global__ __launch_bounds__(1024) void k_dispatch(const DispatchArgs a)
{
    extern __shared__ int sm[];
    const int E = a.n_experts, T = a.n_tokens;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x) {
        // a wavefront per token: its row is cleared in whole lines
        const int step = ((int)gridDim.x - 1) * (nthr >> 6);
        for (int t = ((int)blockIdx.x - 1) * (nthr >> 6) + wave; t < T; t += step) {
            const int e = a.expert_idx[t];
            if (e < 0 || e >= E)
                for (int c = lane; c < a.d_model; c += 64) a.y[(size_t)t * a.d_model + c] = 0.0f;
        }
        return;
    }
    const int per = ((T + PARTS - 1) / PARTS + 63) & ~63;  // tokens of a part
    const int S = count_stride(E);
    int *cnt = sm;               // [PARTS][S] tokens of the part, later the slot of its next one; expert e at spread(e)
    int *tmp = sm + PARTS * S;   // [17 * 12] scan scratch
    int *lost = tmp + 17 * 12;   // [1 + 4] tokens without an expert; sums of choose_mm_min
    for (int i = tid; i < PARTS * S; i += nthr) cnt[i] = 0;
    if (tid < 5) lost[tid] = 0;
    __syncthreads();
    int dropped = 0;
    for (int t0 = tid; t0 < T; t0 += 4 * nthr) {
        int e[4];
#pragma unroll
        for (int k = 0; k < 4; k++) e[k] = a.expert_idx[min(t0 + k * nthr, T - 1)];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int t = t0 + k * nthr;
            if (t >= T) continue;
            if (e[k] >= 0 && e[k] < E) atomicAdd(&cnt[(t / per) * S + spread(e[k])], 1);
            else dropped++;
        }
    }
    if (dropped) atomicAdd(lost, dropped);
    __syncthreads();
    // each thread owns a contiguous chunk of experts
    const int chunk = (E + nthr - 1) / nthr;
    const int e0 = min(E, tid * chunk), e1 = min(E, e0 + chunk);
    const int kept = T - *lost;
    int mm_min = kept >= a.mm_from ? a.mm_min : a.mm_else;
    if (kept < a.mm_below) mm_min = choose_mm_min<PARTS>(a, cnt, S, e0, e1, kept, lost + 1);

    // Work items of the scalar products are listed longest first (by tile_class): handed out in that
    // order, the last workgroups to finish are busy with short items.
    int s_tok = 0, s_act = 0, s_mm = 0;
    int s_wi[4] = {0, 0, 0, 0}, s_wo[4] = {0, 0, 0, 0};
    for (int e = e0; e < e1; e++) {
        int n = 0;
#pragma unroll
        for (int p = 0; p < PARTS; p++) n += cnt[p * S + spread(e)];
        s_tok += n;
        s_act += n > 0;
        if (n >= mm_min) {
            s_mm += (n + kMmTokens - 1) / kMmTokens;
        } else if (n > 0) {
            s_wi[tile_class(a.tb_wi)] += n / a.tb_wi;
            if (n % a.tb_wi) s_wi[tile_class(n % a.tb_wi)]++;
            s_wo[tile_class(a.tb_wo)] += n / a.tb_wo;
            if (n % a.tb_wo) s_wo[tile_class(n % a.tb_wo)]++;
        }
    }
    // all twelve sums in one scan
    const int sums[12] = {s_tok, s_act, s_mm, dropped, s_wi[0], s_wi[1], s_wi[2], s_wi[3],
                          s_wo[0], s_wo[1], s_wo[2], s_wo[3]};
    int before[12], all[12];
    block_exclusive_scan_n<12>(sums, tmp, before, all);
    int p_tok = before[0], p_mm = before[2];
    const int tot_tok = all[0], tot_act = all[1], tot_mm = all[2], tot_drop = all[3];
    int p_wi[4], p_wo[4], tot_wi = 0, tot_wo = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        p_wi[k] = tot_wi + before[4 + k];
        p_wo[k] = tot_wo + before[8 + k];
        tot_wi += all[4 + k];
        tot_wo += all[8 + k];
    }
    for (int e = e0; e < e1; e++) {
        int here[PARTS], n = 0;
#pragma unroll
        for (int p = 0; p < PARTS; p++) here[p] = cnt[p * S + spread(e)];
#pragma unroll
        for (int p = 0; p < PARTS; p++) {  // counts become the parts' cursors
            cnt[p * S + spread(e)] = p_tok + n;
            n += here[p];
        }
        a.tok_off[e] = p_tok;
        if (n >= mm_min) {
            for (int i = 0; i * kMmTokens < n; i++)
                a.items_mm[p_mm++] = Item{e, p_tok + i * kMmTokens, min(kMmTokens, n - i * kMmTokens), 0};
        } else {
            put_tiles(a.items_wi, p_wi, e, p_tok, n, a.tb_wi);
            put_tiles(a.items_wo, p_wo, e, p_tok, n, a.tb_wo);
        }
        p_tok += n;
    }
    if (tid == 0) {
        a.tok_off[E] = tot_tok;
        a.counters[0] = tot_tok;
        a.counters[1] = tot_drop;
        a.counters[2] = tot_act;
        a.counters[3] = tot_wi;
        a.counters[4] = tot_wo;
        a.counters[5] = 0; a.counters[6] = 0;  // work hand-out of the two scalar products
        a.counters[7] = tot_mm;
        a.counters[8] = 0; a.counters[9] = 0;  // work hand-out of the two matrix-core products
        for (int k = 0; k < 4; k++) a.counters[10 + k] = all[4 + k];  // items_wi by class
        a.counters[14] = 0; a.counters[15] = 0;
    }
    __syncthreads();

    // Stable scatter: part p by wavefront p, in token order.
    if (wave >= PARTS) return;
    const int bits = 32 - __builtin_clz(E);  // (E itself stands for "none")
    int *cursor = cnt + wave * S;
    const int t_end = min(T, (wave + 1) * per);
    auto expert_of = [&](int t) {
        const int e = a.expert_idx[min(t, T - 1)];
        return t < t_end && e >= 0 && e < E ? e : E;
    };
    constexpr int kAhead = 4;  // steps of 64 tokens whose experts are asked for together
    int next[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; k++) next[k] = expert_of(wave * per + 64 * k + lane);
    for (int base = wave * per; base < t_end; base += 64 * kAhead) {
        int now[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; k++) {
            now[k] = next[k];
            next[k] = expert_of(base + 64 * (kAhead + k) + lane);
        }
#pragma unroll
        for (int k = 0; k < kAhead; k++) {
            const int e = now[k];
            if (base + 64 * k >= t_end) break;
            const unsigned long long same = same_expert(e, bits);
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            int cur = 0;
            if (e < E) cur = cursor[spread(e)];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();  // every lane has read its cursor
            if (e < E) {
                a.perm[cur + rank] = base + 64 * k + lane;
                if (rank == 0) cursor[spread(e)] = cur + __popcll(same);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();  // the cursors are moved before the next 64 tokens read them
        }
    }
}

// The activations of the listed tiles in blocks of 16 tokens (see ProductArgs): a block stands in `out` where its slots' plain rows would.
// A wavefront takes 128 columns of a block; eight lanes read 128 bytes of a token in a run and write 128 bytes of a column group with eight others.
// What bounds it is its launch and four trips to memory, each after the one before (how many items, the item, its slots' tokens, their rows): 5.5 to 7.8 us in the
// layer call, by the trace, 4001 x 768 activations.
constexpr int kTileCols = 128;
__global__ __launch_bounds__(256) void k_tile_x(const ProductArgs a, uint16_t *out)
{
    const int lane = threadIdx.x & 63, piece = lane & 7;
    const int chunks = (a.cols + kTileCols - 1) / kTileCols, per_item = (kMmTokens / 16) * chunks;
    const int n_items = min(*a.n_items_dev, a.max_items);
    const long long total = (long long)n_items * per_item;
    for (long long u = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); u < total; u += 4LL * gridDim.x) {
        const int idx = (int)(u / per_item), in_item = (int)(u - (long long)idx * per_item), block = in_item / chunks;
        const Item it = a.items[idx];
        const int tb = min(16, min(it.ntok, kMmTokens) - 16 * block), slot0 = it.slot0 + 16 * block;
        if (tb < 1) continue;
        const int col = (in_item - block * chunks) * kTileCols + 8 * piece;
        u32x4 v[2][2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int j = min(8 * h + (lane >> 3), tb - 1);
            const uint16_t *row = a.x + (size_t)a.perm[slot0 + j] * a.ldx;
#pragma unroll
            for (int c = 0; c < 2; c++) v[h][c] = *(gp_u32x4)(row + min(col + 64 * c, a.cols - 8));
        }
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int j = 8 * h + (lane >> 3);
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int k = col + 64 * c;
                if (j < tb && k < a.cols)
                    *(__attribute__((address_space(1))) u32x4 *)(out + (size_t)slot0 * a.ldx + ((size_t)(k >> 3) * tb + j) * 8) = v[h][c];
            }
        }
    }
}

}  // namespace

template <int PARTS>
static qmoe_status launch_parts(const DispatchArgs &da, int threads, int max_lds, hipStream_t s)
{
    // parts: a wavefront each, as many as the tokens fill and the LDS has counts for (two at 16384 experts)
    const size_t smem = sizeof(int) * ((size_t)PARTS * (size_t)count_stride(da.n_experts) + 17 * 12 + 5);
    if constexpr (PARTS > 1) {
        if (PARTS > threads / 64 || 32 * PARTS >= da.n_tokens || smem > (size_t)max_lds)
            return launch_parts<PARTS / 2>(da, threads, max_lds, s);
    }
    const qmoe_status st = allow_lds(k_dispatch<PARTS>, smem);
    if (st != QMOE_OK) return st;
    const int waves = threads / 64, clear = da.y ? std::min(kClearGrid, (da.n_tokens + waves - 1) / waves) : 0;
    hipLaunchKernelGGL(k_dispatch<PARTS>, dim3(1 + clear), dim3(threads), smem, s, da);
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

qmoe_status launch_tile_x(const ProductArgs &a, uint16_t *out, int cus, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile_x, dim3(4 * cus), dim3(256), 0, s, a, out);
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

qmoe_status launch_dispatch_kernel(const DispatchArgs &da, int max_lds, hipStream_t s)
{
    // small layers: fewer wavefronts meet at the kernel's barriers and the scan has fewer partial sums
    const int need = da.n_tokens > da.n_experts ? da.n_tokens : da.n_experts;
    return launch_parts<16>(da, need <= 256 ? 256 : (need <= 512 ? 512 : 1024), max_lds, s);
}

}  // namespace qmoe
