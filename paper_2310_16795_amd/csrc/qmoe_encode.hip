// The encoder on the device (Section 4.3.3 "Encoding"): longest-prefix coding of ternary rows, codeword
// for codeword the stream of qmoe_encode_host.  With the run coder a row is parsed once: the wavefronts tell each other how
// many codewords come before theirs.  By the trie: count codewords per row, turn the counts into row offsets (one
// workgroup), write the codewords.
#include "qmoe_encode.h"

namespace qmoe {
namespace {

// exclusive prefix sum of one int per thread over the workgroup; `tmp` holds >= 32 ints
__device__ __forceinline__ int block_exclusive_scan(int v, int *tmp, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = (blockDim.x + 63) >> 6;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        int w = lane < nwaves ? tmp[lane] : 0;
        int wi = w;
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            const int up = __shfl_up(wi, d, 64);
            if (lane >= d) wi += up;
        }
        if (lane < nwaves) tmp[lane] = wi - w;  // exclusive per wave
        if (lane == nwaves - 1) tmp[16] = wi;   // grand total
    }
    __syncthreads();
    const int base = tmp[wave];
    total = tmp[16];
    __syncthreads();
    return base + incl - v;
}

__global__ void k_encode_clear(int *status)
{
    if (threadIdx.x < 2) status[threadIdx.x] = 0;
}

// ---------------------------------------------------------------- any dictionary: a row per lane, by the trie
//
// Walk pairs from the root while a child exists, emit the codeword of the deepest node that ends
// an entry, continue after that entry.  Every pair is a dependent read of a table in L2, so this is the form
// for dictionaries without a run coder only.

// Walks one row; returns 0 or the error, *count the codewords (each handed to `emit`).
template <class Emit>
__device__ __forceinline__ int walk_row(const EncodeArgs &a, int r, uint32_t *count, Emit &&emit)
{
    const int8_t *row = a.tern + (size_t)r * a.cols;
    const int np = a.cols / 2;
    uint32_t n = 0;
    int bad = 0;
    int i = 0;
    while (i < np) {
        int node = 0, best = -1, best_len = 0, depth = 0;
        while (i + depth < np) {
            const int va = row[2 * (i + depth)], vb = row[2 * (i + depth) + 1];
            if (va < -1 || va > 1 || vb < -1 || vb > 1) { bad = QMOE_E_BAD_SYMBOL; break; }
            // value -> symbol: 0 -> 0, -1 -> 1, +1 -> 2; pair index = 3 * first + second
            const int sa = va == 0 ? 0 : (va < 0 ? 1 : 2), sb = vb == 0 ? 0 : (vb < 0 ? 1 : 2);
            const int nx = a.child[(size_t)node * 9 + 3 * sa + sb];
            if (nx < 0) break;
            node = nx;
            depth++;
            const int c = a.code[node];
            if (c >= 0) { best = c; best_len = depth; }
        }
        if (bad) break;
        if (best < 0) { bad = QMOE_E_UNENCODABLE; break; }
        emit(n, best);
        n++;
        i += best_len;
    }
    *count = n;
    return bad;
}

__device__ __forceinline__ void report(const EncodeArgs &a, int error, int row)
{
    if (atomicCAS(&a.status[0], 0, error) == 0) a.status[1] = row;
}

template <bool WRITE>
__global__ __launch_bounds__(256) void k_encode(const EncodeArgs a)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.rows) return;
    if (WRITE && a.status[0] != 0) return;
    const size_t out = WRITE ? (size_t)a.row_off[r] : 0;
    uint32_t n = 0;
    const int bad = walk_row(a, r, &n, [&](uint32_t at, int code) {
        if (WRITE) a.codes[out + at] = (uint16_t)code;
    });
    if (bad) {
        report(a, bad, r);
        n = 0;
    }
    if (!WRITE) a.row_off[r + 1] = n;
}

// ---------------------------------------------------------------- the run coder: many lanes per row
//
// A row becomes two bit strings in LDS (non-zero, negative), and the longest entry at a position comes
// from the places of its next three non-zeros (qmoe_internal.h): one LDS read of the bits, two of the depth
// tables, about sixty vector instructions, no matter how many pairs the entry has.  The parse of a row is
// sequential -- an entry's end is the next one's start -- but a parse that starts in the wrong place falls into
// step with the right one after a few entries, so every lane parses a segment of the row from the
// segment's first pair and marks where entries begin; then it starts again from where the lane before it
// ended and goes on until it meets a mark of its first parse.  The last few lanes of a wavefront that have met none after
// that many steps are helped by all the others (91 us to the end of the slowest wavefront's parse without, 76 with).  Wavefronts share
// the depth tables; no barrier after those are staged.
//
// Where a row's codewords go depends on all rows before it.  A wavefront's rows are a group; when it has parsed them it
// publishes their number of codewords, looks at the groups before it -- 64 at a time, back to one that knows all before
// itself -- and publishes the sum.  The words for that are the row offsets that end the groups, which a last kernel turns into
// plain offsets.  A wavefront waits for lower groups only, and groups are given out by a ticket that a workgroup draws when
// it runs, so whatever is waited for is in work on some compute unit and waits for nobody above it.
//
// Bound: the chain of an entry (about 900 cycles) times the entries a wavefront goes through, with the two or
// three wavefronts per SIMD that the row strings leave room for.  16640 x 6144 values, 90 % zeros: 207 us
// with every row parsed twice, to count and to write, 112 now (23 packed, 13 and 17 the two parses, up to 45 in the last
// wavefront, 20 looked up, 9 copied out), 2680 us a pass by the trie (a row per lane, a dependent read of L2 per pair).

constexpr int kRcAlone = 16;  // entries of the second parse that the lanes take on their own, at least
constexpr int kRcHelp = 12;   // lanes of a wavefront that are helped, at most

struct Bits {
    uint32_t nz, neg;  // 28 values from a pair on
};

__device__ __forceinline__ Bits row_window(uint32_t bits_lds, int pair)
{
    typedef const __attribute__((address_space(3))) unsigned long long *p64;
    const uint32_t b = 2u * (uint32_t)pair;
    p64 p = (p64)(uintptr_t)(bits_lds + 8u * (b >> 5));
    const unsigned long long w0 = p[0], w1 = p[1];  // (nz, neg) words
    Bits r;
    r.nz = __builtin_amdgcn_alignbit((uint32_t)w1, (uint32_t)w0, b & 31u) & 0x0FFFFFFFu;
    r.neg = __builtin_amdgcn_alignbit((uint32_t)(w1 >> 32), (uint32_t)(w0 >> 32), b & 31u) & 0x0FFFFFFFu;
    return r;
}

// C(p2,2) + p1 and C(p3,3) + that (p (p - 1) (p - 2) / 6 is exact so for p up to 31); 24-bit products, which run
// at full rate
__device__ __forceinline__ uint32_t rank2(uint32_t p1, uint32_t p2) { return (__umul24(p2, p2 - 1u) >> 1) + p1; }
__device__ __forceinline__ uint32_t rank3(uint32_t c2, uint32_t p3)
{
    return (__umul24(__umul24(__umul24(p3, p3 - 1u), p3 - 2u), 10923u) >> 16) + c2;
}

// Pairs of the longest entry (at most `left`, 1..); 0: none fits.
__device__ __forceinline__ int longest_run(uint32_t depth_lds, int depth0, const Bits &v, int left)
{
    typedef const __attribute__((address_space(3))) unsigned char *p8;
    uint32_t w = v.nz | 0xF0000000u;  // positions 28..31 stand in for non-zeros that are not there
    const uint32_t p1 = (uint32_t)__builtin_ctz(w);
    w &= w - 1u;
    const uint32_t p2 = (uint32_t)__builtin_ctz(w);
    w &= w - 1u;
    const uint32_t p3 = (uint32_t)__builtin_ctz(w);
    w &= w - 1u;
    const int h1 = (int)(p1 >> 1), h2 = (int)(p2 >> 1), h3 = (int)(p3 >> 1), h4 = __builtin_ctz(w) >> 1;
    // signs (0 for a non-zero that is not there)
    const uint32_t s1 = __builtin_amdgcn_ubfe(v.neg, p1, 1u), s2 = __builtin_amdgcn_ubfe(v.neg, p2, 1u),
                   s3 = __builtin_amdgcn_ubfe(v.neg, p3, 1u);
    const uint32_t c2 = rank2(p1, p2), c3 = rank3(c2, p3), s23 = s2 + 2u * s3;
    // byte of two patterns of three that differ in the first sign
    const uint32_t d3 = *(p8)(uintptr_t)(depth_lds + min(4u * c3 + s23, (uint32_t)(kRcTwo / 2)));
    const int d12 = *(p8)(uintptr_t)(depth_lds + (uint32_t)kRcDepth3Bytes + 4u * c2 + (s1 + 2u * s2));
    const int limit = min(14, left);
    const int l3 = min(min((int)__builtin_amdgcn_ubfe(d3, 4u * s1, 4u), limit), h4), l2 = min(min(d12 & 15, limit), h3);
    const int l1 = min(min(d12 >> 4, limit), h2), l0 = min(min(depth0, limit), h1);
    return max(max(l3 > h3 ? l3 : 0, l2 > h2 ? l2 : 0), max(l1 > h1 ? l1 : 0, l0));
}

// The pattern of an entry of `pairs` pairs.
__device__ __forceinline__ int pattern_of(const Bits &v, int pairs)
{
    const uint32_t w = v.nz & ((1u << (2 * pairs)) - 1u);  // pairs <= 14
    const int k = __popc(w);
    const uint32_t top = 0x80000000u, w2 = w & (w - 1u), w3 = w2 & (w2 - 1u);
    const uint32_t p1 = (uint32_t)__builtin_ctz(w | top), p2 = (uint32_t)__builtin_ctz(w2 | top), p3 = (uint32_t)__builtin_ctz(w3 | top);
    const int s12 = (int)(((v.neg >> p1) & 1u) | (((v.neg >> p2) & 1u) << 1)), s3 = (int)((v.neg >> p3) & 1u);
    const uint32_t c2 = rank2(p1, p2);
    int i = kRcZero;
    i = k == 1 ? kRcOne + 2 * (int)p1 + (s12 & 1) : i;
    i = k == 2 ? kRcTwo + 4 * (int)c2 + s12 : i;
    i = k == 3 ? kRcThree + 8 * (int)rank3(c2, p3) + (s12 | s3 << 2) : i;
    return i;
}

// sixteen values -> sixteen bits each of non-zero and negative; `bad` collects bits of values that are not -1, 0, +1
__device__ __forceinline__ void pack16(const u32x4 &v, uint32_t &nz, uint32_t &neg, uint32_t &bad)
{
    nz = 0u;
    neg = 0u;
#pragma unroll
    for (int k = 3; k >= 0; k--) {
        const uint32_t one = v[k] & 0x01010101u, minus = (v[k] >> 7) & 0x01010101u;
        bad |= v[k] ^ (one | ((minus << 8) - minus));
        if (k == 1) {
            nz <<= 8;
            neg <<= 8;
        }
        const uint32_t weights = (k & 1) ? 0x80402010u : 0x08040201u;
        nz = __builtin_amdgcn_udot4(one, weights, nz, false);
        neg = __builtin_amdgcn_udot4(minus, weights, neg, false);
    }
}

// The number of codewords that a group's state says, and what it is the number of: all codewords up to the group's end, or
// the group's own (0: not known yet).
constexpr uint32_t kEncAll = 0x40000000u, kEncOwn = 0x80000000u, kEncCount = kEncAll - 1u;

__device__ __forceinline__ uint32_t *group_state(const RunCoderArgs &a, int group)
{
    return a.e.row_off + min(a.row0 + (long long)(group + 1) * (64 >> a.lanes_log2), (long long)a.row_end);
}

__device__ __forceinline__ void publish(uint32_t *state, uint32_t v)
{
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(state, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Codewords of the groups below `group` (by a whole wavefront): lane i looks at group - 1 - i.
__device__ __forceinline__ uint32_t codewords_before(const RunCoderArgs &a, int group)
{
    const int lane = threadIdx.x & 63;
    uint32_t sum = 0u;
    for (int at = group - 1; at >= 0;) {
        uint32_t v = kEncAll;
        if (at - lane >= 0) v = __hip_atomic_load(group_state(a, at - lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long all = __ballot((v & kEncAll) != 0u), unknown = __ballot(v == 0u);
        const int last = all ? __builtin_ctzll(all) : 63;
        if (unknown & (~0ull >> (63 - last))) {
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        sum += (uint32_t)__builtin_amdgcn_readlane(wave_inclusive_scan(lane <= last ? (int)(v & kEncCount) : 0), 63);
        if (all) break;
        at -= 64;
    }
    return sum;
}

// status[0] the first error, status[1] (while the encoder runs) the tickets drawn, row_off[0] (until its end) the error's row + 1
__device__ __forceinline__ void report_row(const EncodeArgs &e, int error, int row)
{
    if (atomicCAS(&e.row_off[0], 0u, (uint32_t)row + 1u) == 0u) e.status[0] = error;
}

// Clears what the chunk's groups publish in, the tickets and, ahead of the first chunk, the errors.
__global__ void k_encode_begin(const RunCoderArgs a)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < a.groups) *group_state(a, g) = 0u;
    if (g == 0) {
        a.e.status[1] = 0;
        if (a.row0 == 0) {
            a.e.status[0] = 0;
            a.e.row_off[0] = 0u;
        }
    }
}

// The groups' last offsets as plain offsets; behind the last chunk the error's row in its place.
__global__ __launch_bounds__(1024) void k_encode_end(const RunCoderArgs a)
{
    const unsigned long long base = a.row0 ? a.e.row_off[a.row0] : 0u;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.groups) return;
    uint32_t *state = group_state(a, g);
    const unsigned long long at = base + (*state & kEncCount);
    *state = (uint32_t)at;
    if (g != a.groups - 1) return;
    // (a chunk whose offsets do not fit ends with an error that stays, so what comes behind it does not matter)
    if (a.e.status[0] == 0 && (at > a.e.codes_cap || at > 0xFFFFFFFFull)) a.e.status[0] = QMOE_E_BUFFER_TOO_SMALL;
    if (a.row_end == a.e.rows) {
        const uint32_t row = a.e.row_off[0];
        a.e.status[1] = row ? (int)(row - 1u) : 0;
        a.e.row_off[0] = 0u;
    }
}

__global__ __launch_bounds__(1024) void k_encode_runs(const RunCoderArgs a)
{
    typedef __attribute__((address_space(3))) uint32_t *lw_u32;
    typedef __attribute__((address_space(3))) uint16_t *lw_u16;
    typedef u32x4 u32x4_any __attribute__((aligned(1)));
    typedef const __attribute__((address_space(1))) u32x4_any *gp_u32x4_any;
    extern __shared__ __align__(16) unsigned char smem[];
    const EncodeArgs &e = a.e;
    int *ticket_s = reinterpret_cast<int *>(smem + kRcDepthBytes);
    if (threadIdx.x == 0) *ticket_s = atomicAdd(&e.status[1], 1);
    const unsigned long long codes_base = a.row0 ? e.row_off[a.row0] : 0u;
    stage_words(reinterpret_cast<uint32_t *>(smem), a.depth, kRcDepthBytes / 4);
    __syncthreads();
    const uint32_t depth_lds = (uint32_t)(uintptr_t)(lw_u16)(uint16_t *)smem;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int L = 1 << a.lanes_log2, R = 64 >> a.lanes_log2;  // lanes per row, rows per wavefront
    const int sub = lane & (L - 1), mine = lane >> a.lanes_log2;
    const uint32_t rows_lds = depth_lds + (uint32_t)(kRcDepthBytes + kRcTicketBytes) + (uint32_t)(wave * R * a.row_lds);
    const int np = e.cols / 2;
    const int seg0 = sub * a.seg_pairs, seg1 = min(seg0 + a.seg_pairs, np);

    // a workgroup's groups follow each other
    const int ticket = __builtin_amdgcn_readfirstlane(*ticket_s), first_group = ticket * a.groups_per_wg + min(ticket, a.groups_extra);
    const int end_group = first_group + a.groups_per_wg + (ticket < a.groups_extra ? 1 : 0);
    for (int group = first_group + wave; group < end_group; group += waves) {
        const int row0 = a.row0 + group * R, row = row0 + mine;
        uint32_t tail_wrong = 0u;
        auto put = [&](int r, int c, uint32_t nz, uint32_t neg) {
            lw_u16 w = (lw_u16)(uintptr_t)(rows_lds + (uint32_t)(r * a.row_lds) + 8u * (uint32_t)(c >> 5) + (uint32_t)((c >> 3) & 2));
            w[0] = (uint16_t)nz;
            w[2] = (uint16_t)neg;
        };
        // ---- the wavefront's rows as bit strings (zeros behind the last value), boundary marks cleared
        // (a row is cut into pieces of 1024 values; eight pieces are asked for at a time, also across rows)
        uint32_t bad = 0u;
        const int pieces = (32 * a.bit_words + 1023) >> 10, n_rows = min(R, a.row_end - row0);
        for (int i0 = 0; i0 < n_rows * pieces; i0 += 8) {
            u32x4 v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int r = (i0 + k) / pieces, c = 1024 * (i0 + k - r * pieces) + 16 * lane;
                v[k] = u32x4{0u, 0u, 0u, 0u};
                if (r < n_rows && c + 16 <= e.cols)
                    v[k] = *(gp_u32x4_any)(reinterpret_cast<uintptr_t>(e.tern) + (size_t)(row0 + r) * e.cols + c);
            }
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int r = (i0 + k) / pieces, c = 1024 * (i0 + k - r * pieces) + 16 * lane;
                uint32_t nz, neg, wrong = 0u;
                pack16(v[k], nz, neg, wrong);
                if (r < n_rows && c < 32 * a.bit_words) put(r, c, nz, neg);
                if (__any(wrong != 0u) && mine == r) bad = 1u;
            }
        }
        if ((e.cols & 15) && lane < n_rows) {  // the values after a row's last whole sixteen
            u32x4 v{0u, 0u, 0u, 0u};
            const int c = e.cols & ~15;
            const uintptr_t src = reinterpret_cast<uintptr_t>(e.tern) + (size_t)(row0 + lane) * e.cols + c;
            for (int j = 0; c + j < e.cols; j++)
                v[j >> 2] |= (uint32_t)*(const __attribute__((address_space(1))) uint8_t *)(src + j) << (8 * (j & 3));
            uint32_t nz, neg, wrong = 0u;
            pack16(v, nz, neg, wrong);
            put(lane, c, nz, neg);
            tail_wrong = wrong;
        }
        if (__ballot(tail_wrong != 0u) >> mine & 1ull) bad = 1u;
        for (int i = lane; i < n_rows * a.mask_words; i += 64) {
            const int r = i / a.mask_words;
            *(lw_u32)(uintptr_t)(rows_lds + (uint32_t)(r * a.row_lds) + 8u * (uint32_t)a.bit_words + 4u * (uint32_t)(i - r * a.mask_words)) = 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        const bool live = row < a.row_end && seg0 < np;
        const uint32_t bits = rows_lds + (uint32_t)(mine * a.row_lds);
        lw_u32 marks = (lw_u32)(uintptr_t)(bits + 8u * (uint32_t)a.bit_words);
        bool odd = false;  // a position where no entry fits was met (perhaps only by a parse from the wrong place)

        // ---- every lane its segment, from the segment's first pair
        int end = seg0;
        if (live) {
            int word = seg0 >> 5;
            uint32_t set = 0u;
            while (end < seg1) {
                int len = longest_run(depth_lds, a.depth0, row_window(bits, end), np - end);
                odd |= len < 1;
                len = max(len, 1);
                if ((end >> 5) != word) {
                    marks[word] = set;
                    set = 0u;
                    word = end >> 5;
                }
                set |= 1u << (end & 31);
                end += len;
            }
            marks[word] = set;
        }
        // ---- again from where the lane before ended, until the two parses meet
        const int before_end = __shfl_up(end, 1, 64), from = sub == 0 ? 0 : before_end;
        const bool again = live && from != seg0;
        bool met = false;
        int t = from;
        auto step = [&]() {  // an entry of the second parse: its mark in the place of the first parse's up to its end
            const int w = t >> 5, b = t & 31;
            const uint32_t m = marks[w];
            if ((m >> b) & 1u) {
                met = true;
                return;
            }
            int len = longest_run(depth_lds, a.depth0, row_window(bits, t), np - t);
            odd |= len < 1;
            len = max(len, 1);
            const unsigned long long span = ((1ull << len) - 1ull) << b;
            marks[w] = (m & ~(uint32_t)span) | (1u << b);
            if ((uint32_t)(span >> 32) && 32 * (w + 1) < seg1) marks[w + 1] &= ~(uint32_t)(span >> 32);
            t += len;
        };
        // (an entry reaches at most 13 pairs into the segment)
        if (again) marks[seg0 >> 5] &= ~((1u << (from - seg0)) - 1u);
        for (int k = 0;; k++) {
            const bool on = again && !met && t < seg1, moved = again && !met && t >= seg1 && t != end;
            const int n_on = __popcll(__ballot(on));
            if (n_on == 0) break;
            // Most lanes meet their first parse after a few entries, one of 64 after fifty: the last ones are better off with the
            // whole wavefront's help.  (Sixteen steps at least: whoever is left is past the pairs that the lane before may
            // reach into the segment.)
            if (k >= kRcAlone && n_on <= 4 && __popcll(__ballot(on || moved)) <= kRcHelp) break;
            if (on) step();
        }
        bool pending = again && !met && t != end;
        if (__popcll(__ballot(pending)) > kRcHelp) {
            // rows whose parses hardly ever meet (long runs of zeros): every lane whose start has moved goes again, until none has;
            // after j rounds lane j is right
            int start = seg0;
            if (again) {
                start = from;
                if (!met) end = t;
            }
            bool moved;
            do {
                const int ahead = __shfl_up(end, 1, 64), now = sub == 0 ? 0 : ahead;
                moved = false;
                if (live && now != start) {
                    marks[seg0 >> 5] &= ~((1u << (now - seg0)) - 1u);
                    t = now;
                    met = false;
                    while (t < seg1 && !met) step();
                    if (!met) {
                        moved = t != end;
                        end = t;
                    }
                    start = now;
                }
            } while (__any(moved));
        } else if (__any(pending)) {
            // A window of 64 pairs at a time: every lane finds the entry that would begin at its pair, and the wavefront goes through
            // those that do, on into the next segments where it has to.  What is left to a lane begins at a mark.
            if (pending && t >= seg1) atomicAnd((uint32_t *)(marks + (seg1 >> 5)), ~((1u << (t - seg1)) - 1u));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            pending = pending && t < np && !((marks[min(t, np - 1) >> 5] >> (t & 31)) & 1u);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (pending) atomicOr((uint32_t *)(marks + (t >> 5)), 1u << (t & 31));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            unsigned long long todo = __ballot(pending);
            while (todo) {
                const int l = __builtin_ctzll(todo), its_row = l >> a.lanes_log2;
                const uint32_t its_bits = rows_lds + (uint32_t)(its_row * a.row_lds);
                lw_u32 its_marks = (lw_u32)(uintptr_t)(its_bits + 8u * (uint32_t)a.bit_words);
                int pos = __builtin_amdgcn_readlane(t, l), ended = np;
                for (bool first = true; pos < np; first = false) {
                    const int at = min(pos + lane, np - 1), width = min(64, np - pos);
                    const int run = longest_run(depth_lds, a.depth0, row_window(its_bits, at), np - at);
                    unsigned long long old = __ballot(lane < width && ((its_marks[at >> 5] >> (at & 31)) & 1u));
                    if (first) old &= ~1ull;
                    unsigned long long begun = 0ull;
                    int off = 0;
                    while (off < width && !((old >> off) & 1ull)) {
                        begun |= 1ull << off;
                        off += max(__builtin_amdgcn_readlane(run, off), 1);
                    }
                    if (__ballot(run < 1) & begun) odd |= mine == its_row;
                    const int stop = min(off, width);  // pairs of the window that are settled
                    const unsigned long long settled = stop == 64 ? ~0ull : (1ull << stop) - 1ull;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const int rel = 32 * ((pos >> 5) + lane) - pos;  // of a word's first pair in the window
                    if (lane < 3 && rel < 64) {
                        const uint32_t mask = rel >= 0 ? (uint32_t)(settled >> rel) : (uint32_t)(settled << -rel);
                        const uint32_t set = rel >= 0 ? (uint32_t)(begun >> rel) : (uint32_t)(begun << -rel);
                        if (mask) its_marks[(pos >> 5) + lane] = (its_marks[(pos >> 5) + lane] & ~mask) | (set & mask);
                    }
                    const int next = pos + off;
                    const bool joined = off < width;
                    // (the last entry may reach past the window)
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const int behind = pos + 64 + lane;
                    if (!joined && behind < min(next, np)) atomicAnd((uint32_t *)(its_marks + (behind >> 5)), ~(1u << (behind & 31)));
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    pos = next;
                    if (joined) {
                        ended = next;
                        break;
                    }
                }
                // (lanes that this parse went past have nothing left to do)
                todo &= todo - 1ull;
                todo &= ~__ballot(pending && lane > l && mine == its_row && t < ended);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- codewords of the segment, and of the row's segments before it
        int count = 0;
        if (live)
            for (int w = seg0 >> 5; 32 * w < seg1; w++) count += __popc(marks[w]);
        // Rows with something odd in them are walked by the trie: it says whether that is an error, and
        // which comes first in the row.  (Such a row has no codewords.)
        if (__any(odd || bad != 0u)) {
            const unsigned long long odd_lanes = __ballot(odd || bad != 0u);
            const unsigned long long row_lanes = L == 64 ? ~0ull : ((1ull << L) - 1ull) << (mine * L);
            int error = 0;
            if (sub == L - 1 && row < a.row_end && (odd_lanes & row_lanes)) {
                uint32_t n = 0;
                error = walk_row(e, row, &n, [](uint32_t, int) {});
                if (error) report_row(e, error, row);
            }
            if (__ballot(error != 0) & row_lanes) count = 0;
        }
        const int incl = wave_inclusive_scan(count), rel = incl - count;
        const uint32_t own = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
        uint32_t *state = group_state(a, group);
        if (group > 0) publish(state, kEncOwn | own);

        // ---- the segment's codewords, kAtOnce at a time (their trips to the two code tables overlap): put(n, c) takes entries n
        // .. n + kAtOnce - 1, those of the segment among them
        constexpr int kAtOnce = 8;
        auto codewords = [&](auto &&put) {
            // the segment's last entry ends where the next segment's first one begins, or with the row
            int last_end = np;
            if (seg1 < np) {
                const uint32_t ahead = marks[seg1 >> 5] & 0x3FFFu;
                last_end = ahead ? seg1 + __builtin_ctz(ahead) : np;
            }
            int w = seg0 >> 5;
            uint32_t set = marks[w];
            auto next = [&]() -> int {  // the next mark of the segment, or its end
                while (set == 0u && 32 * (w + 1) < seg1) set = marks[++w];
                if (set == 0u) return last_end;
                const int t = 32 * w + __builtin_ctz(set);
                set &= set - 1u;
                return t;
            };
            int at = next();
            for (int n = 0; n < count; n += kAtOnce) {
                uint32_t i[kAtOnce];
#pragma unroll
                for (int k = 0; k < kAtOnce; k++) {
                    const int to = n + k < count ? next() : at;
                    const int len = max(to - at, 1);
                    const Bits v = row_window(bits, min(at, np - 1));
                    i[k] = ((gp_u32)a.first)[pattern_of(v, min(len, 14))] + (uint32_t)len;
                    at = to;
                }
                uint16_t c[kAtOnce];
#pragma unroll
                for (int k = 0; k < kAtOnce; k++) c[k] = ((gp_u16)a.codes)[min(i[k], (uint32_t)kTableEntries - 1u)];
                put(n, c);
            }
        };
        // Before the groups before are all there, the codewords can be put into LDS, over the segment's bits that have been read:
        // from 8 bytes on (the lane before reads that far into the segment), 16 pairs of bits in 8 bytes.  They must never reach
        // what is still to be read, so entry n = 8, 16, ... has to begin in a word of 32 pairs, w of the segment, with
        // 8 + 2 n <= 16 w: always so where entries are longer than four pairs or so.
        bool early = 8 + 2 * ((count + kAtOnce - 1) / kAtOnce * kAtOnce) <= 8 * ((seg1 - seg0) >> 4) || count == 0;
        if (live) {
            int n = 0;
            for (int w = 0; 32 * w < seg1 - seg0; w++) {
                n += __popc(marks[(seg0 >> 5) + w]);
                const int eighth = (n - 1) & ~(kAtOnce - 1);  // the last n = 8, 16, ... in this word or before it
                early &= eighth < kAtOnce || 8 + 2 * eighth <= 16 * w;
            }
        }
        const bool in_lds = __all(early || !live);
        const uint32_t codes_lds = bits + 8u * (uint32_t)(seg0 >> 4) + 8u;
        if (in_lds && live) {
            codewords([&](int n, const uint16_t (&c)[kAtOnce]) {
                typedef __attribute__((address_space(3))) unsigned long long *lw_u64;
                lw_u64 to = (lw_u64)(uintptr_t)(codes_lds + 2u * (uint32_t)n);
#pragma unroll
                for (int h = 0; h < 2; h++)
                    to[h] = (unsigned long long)((uint32_t)c[4 * h] | (uint32_t)c[4 * h + 1] << 16) |
                            (unsigned long long)((uint32_t)c[4 * h + 2] | (uint32_t)c[4 * h + 3] << 16) << 32;
            });
        }
        // ---- codewords of the groups before
        const uint32_t before = group > 0 ? codewords_before(a, group) : 0u;
        publish(state, kEncAll | (before + own));
        if (sub == L - 1 && mine + 1 < n_rows) e.row_off[row + 1] = (uint32_t)(codes_base + before + (uint32_t)incl);
        const unsigned long long place = codes_base + before;  // of the group
        const int fit = (int)min((unsigned long long)own, e.codes_cap - min(place, e.codes_cap));
        typedef __attribute__((address_space(1))) uint16_t *gw_u16;
        gw_u16 out = (gw_u16)(e.codes + place);
        if (in_lds) {
            // a segment at a time, in whole lines
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int l0 = 0; l0 < 64; l0 += 4) {
                uint16_t c[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)codes_lds, l0 + k);
                    const int n = __builtin_amdgcn_readlane(count, l0 + k);
                    c[k] = lane < n ? *(const __attribute__((address_space(3))) uint16_t *)(uintptr_t)(from + 2u * (uint32_t)lane) : (uint16_t)0;
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int n = __builtin_amdgcn_readlane(count, l0 + k), at = __builtin_amdgcn_readlane(rel, l0 + k);
                    const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)codes_lds, l0 + k);
                    if (lane < n && at + lane < fit) out[at + lane] = c[k];
                    for (int j = 64 + lane; j < n; j += 64)  // (dense rows)
                        if (at + j < fit) out[at + j] = *(const __attribute__((address_space(3))) uint16_t *)(uintptr_t)(from + 2u * (uint32_t)j);
                }
            }
        } else if (live) {
            codewords([&](int n, const uint16_t (&c)[kAtOnce]) {
#pragma unroll
                for (int k = 0; k < kAtOnce; k++)
                    if (n + k < count && rel + n + k < fit) out[rel + n + k] = c[k];
            });
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// counts in row_off[1..rows] -> offsets; one workgroup, kPerThread consecutive rows a thread (a round's sum
// has to fit 32 bits: the launch takes one row a thread where the rows are that long)
template <int kPerThread>
__global__ __launch_bounds__(1024) void k_encode_offsets(const EncodeArgs a)
{
    __shared__ int tmp[32];
    unsigned long long base = 0;
    if (threadIdx.x == 0) a.row_off[0] = 0;
    for (int r0 = 0; r0 < a.rows; r0 += kPerThread * (int)blockDim.x) {
        const int r = r0 + kPerThread * (int)threadIdx.x;
        uint32_t c[kPerThread];
        unsigned long long sum = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; k++) c[k] = a.row_off[min(r + k, a.rows - 1) + 1];
#pragma unroll
        for (int k = 0; k < kPerThread; k++) {
            c[k] = r + k < a.rows ? c[k] : 0u;
            sum += c[k];
        }
        __syncthreads();  // every count of this round is read before an offset is written
        int total;
        const int excl = block_exclusive_scan((int)sum, tmp, total);
        unsigned long long at = base + (unsigned long long)(uint32_t)excl;
#pragma unroll
        for (int k = 0; k < kPerThread; k++) {
            at += c[k];
            if (r + k < a.rows) a.row_off[r + k + 1] = (uint32_t)at;
        }
        base += (unsigned long long)(uint32_t)total;
    }
    if (threadIdx.x == 0 && (base > a.codes_cap || base > 0xFFFFFFFFull)) atomicCAS(&a.status[0], 0, QMOE_E_BUFFER_TOO_SMALL);
}

}  // namespace

qmoe_status launch_encode(const RunCoderArgs &args, hipStream_t s)
{
    RunCoderArgs a = args;
    const EncodeArgs &e = a.e;
    const int np = e.cols / 2;
    a.bit_words = (e.cols + 31) / 32 + 1;
    a.mask_words = (np + 31) / 32 + 1;
    a.row_lds = (8 * a.bit_words + 4 * a.mask_words + 15) / 16 * 16;
    // Lanes per row.  A wavefront's time is its entries one after the other: those of a segment (about 11.5
    // pairs each), and those of the second parse until its lanes have fallen into step -- about
    // 45 (simulated at 80-92 % zeros: half the lanes need 2-9, one in a hundred 30-64; with the wavefront's help for the last
    // ones somewhat fewer, and never many more).  An entry takes about 900 cycles
    // from end to end and 340 of its SIMD's issue.  A wavefront's row strings have to fit the LDS next to the
    // depth tables.  (16640 x 6144 values, a pass of an earlier form: 89 us
    // with 8 lanes per row, as chosen; 156 us with 32, 170 us with 4.)
    int best_waves = 0, best_log2 = 0;
    double best = 0.0;
    for (int l = 0; l <= 6; l++) {
        const int R = 64 >> l;
        const int fit = std::min(16, (a.max_lds - kRcDepthBytes - kRcTicketBytes) / (R * a.row_lds));
        if (fit < 1 || !a.depth) continue;
        const int seg = (((np + (1 << l) - 1) >> l) + 31) / 32 * 32;
        const long long groups = (e.rows + R - 1) / R, rounds = (groups + (long long)a.cus * fit - 1) / ((long long)a.cus * fit);
        const int waves = (int)std::max(1LL, std::min<long long>(fit, (groups + a.cus * rounds - 1) / (a.cus * rounds)));
        const double steps = seg / 11.5 * (seg < 520 ? 2 : 1) + (l ? 45.0 : 0.0);
        const double cost = (double)rounds * steps * std::max(900.0, 340.0 * ((waves + 3) / 4));
        if (!best_waves || cost < best) {
            best = cost;
            best_log2 = l;
            best_waves = waves;
        }
    }
    a.lanes_log2 = best_log2;
    a.seg_pairs = (((np + (1 << best_log2) - 1) >> best_log2) + 31) / 32 * 32;
    if (best_waves) {
        const size_t smem = (size_t)kRcDepthBytes + kRcTicketBytes + (size_t)best_waves * (64 >> best_log2) * a.row_lds;
        const qmoe_status st = allow_lds(k_encode_runs, smem);
        if (st != QMOE_OK) return st;
        // Rows in chunks whose codewords (at most one a pair) a state can count: one, but for matrices of 2^31 values and more.
        const int R = 64 >> best_log2;
        long long chunk = std::max<long long>(R, (long long)(kEncCount / (uint32_t)np) / R * R);
        if (tuning().encode_rows > 0) chunk = std::min<long long>(chunk, std::max(R, tuning().encode_rows / R * R));
        for (long long r0 = 0; r0 < e.rows; r0 += chunk) {
            a.row0 = (int)r0;
            a.row_end = (int)std::min<long long>(e.rows, r0 + chunk);
            a.groups = (a.row_end - a.row0 + R - 1) / R;
            const int grid = std::min(a.cus, a.groups);  // (not as few workgroups as have a group for every wavefront: 117.9 us, 112)
            a.groups_per_wg = a.groups / grid;
            a.groups_extra = a.groups % grid;
            const int small = (a.groups + 255) / 256;
            hipLaunchKernelGGL(k_encode_begin, dim3(small), dim3(256), 0, s, a);
            hipLaunchKernelGGL(k_encode_runs, dim3(grid), dim3(64 * best_waves), smem, s, a);
            hipLaunchKernelGGL(k_encode_end, dim3(small), dim3(256), 0, s, a);
        }
        QMOE_HIP_TRY(hipGetLastError());
        return QMOE_OK;
    }
    // the status words are cleared by a kernel, not a memset node, so the call can be captured into a HIP graph
    hipLaunchKernelGGL(k_encode_clear, dim3(1), dim3(64), 0, s, e.status);
    const int grid = (e.rows + 255) / 256;
    hipLaunchKernelGGL(k_encode<false>, dim3(grid), dim3(256), 0, s, e);
    if (np < 100000)
        hipLaunchKernelGGL(k_encode_offsets<20>, dim3(1), dim3(1024), 0, s, e);
    else
        hipLaunchKernelGGL(k_encode_offsets<1>, dim3(1), dim3(1024), 0, s, e);
    hipLaunchKernelGGL(k_encode<true>, dim3(grid), dim3(256), 0, s, e);
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

}  // namespace qmoe
