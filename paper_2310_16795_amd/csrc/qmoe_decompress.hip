// Decompression of whole matrices (Section 4.3.3 of the paper mentions it as a variant): dense ternary (int8) or
// scaled bf16 copies, for consumers that want a plain matrix (a library GEMM, a check).
#include "qmoe_dev.h"

namespace qmoe {
namespace {

// A wavefront takes two rows, 32 lanes each (narrow matrices: eight rows of eight lanes each).  In a step every lane decodes
// a quarter of a 16-byte piece of its row (two codewords; the column where they start by a prefix sum over the row's
// lanes) and stores the weights, one byte a column, into the row's ring in LDS.  Whole groups of columns, eight a lane, then
// leave the ring: the lanes of a row write its 256 columns, 512 bytes in a run (int8: 256), and clear them.  A row's groups
// begin early by as many columns as it takes for their ends to fall on multiples of that run in the row's destination.
//
// Bound: the stores.  Per 64 codewords a compute unit has about 330 cycles of HBM write time (bf16) and the wavefront
// about 150 of vector issue, so what counts is that every compute unit has rows to write all the time, to the end (small
// units, the number of wavefronts chosen so that they divide evenly), and how the stores reach memory: runs of 128
// bytes 3.4 TB/s, marked non-temporal (the lines are whole) 4.0, runs of 512 bytes 4.3.
// (Also where the results would fit the caches: stored plainly into other buffers from call to call, one matrix of 2080 x 6144
// takes 15.4 us instead of 12.4, eight 58 instead of 49, although a product that reads them at once gains more than that --
// call and product with 64 tokens 30.4 instead of 35.1, and 195 instead of 211 -- as long as all results together stay below
// the last-level cache's 256 MB; twelve, or two calls of six before the products, lose there too.)
// 12 experts of 2080 x 6144, both projections, to bf16 (613 MB; a fill takes 95 us): 331 us with the kernel before, which
// gave a lane a row and a workgroup 512 rows (60 workgroups for the one projection, 144 for the other), now 134.
constexpr int kDcMaxWaves = 16;
constexpr int kDcWide = 32, kDcNarrow = 8;        // lanes per row
template <int LANES>
struct DcShape {
    static constexpr int kRows = 64 / LANES;      // rows of a wavefront
    static constexpr int kGroup = 8 * LANES;      // columns the lanes of a row write at once
    // columns a row's ring holds: what is left of a group (kGroup - 1) and two codewords a lane (56 columns)
    static constexpr int kRing = 64 * LANES;
    static constexpr int kRowBytes = kRing + 16;
};

using lw_u8 = __attribute__((address_space(3))) unsigned char *;
using lw_u64 = __attribute__((address_space(3))) unsigned long long *;
using gw_u64 = __attribute__((address_space(1))) unsigned long long *;
using gw_u32x4 = __attribute__((address_space(1))) u32x4 *;

// OUT 0: int8 in {-1, 0, +1}; 1: bf16(scale of the row) with the weight's sign, or 0;
// 2: the row's bf16 grid point w_max or w_min, or 0 (asymmetric grid)
template <int OUT, int kDcLanes>
__global__ __launch_bounds__(64 * kDcMaxWaves) void k_decompress(const DecompressArgs a)
{
    constexpr int kDcRows = DcShape<kDcLanes>::kRows, kDcGroup = DcShape<kDcLanes>::kGroup, kDcRing = DcShape<kDcLanes>::kRing,
                  kDcRowBytes = DcShape<kDcLanes>::kRowBytes;
    extern __shared__ __align__(16) unsigned char smem[];
    const size_t table_bytes = ((size_t)a.n_order * 4 + 15) & ~(size_t)15;
    uint32_t *table_w = reinterpret_cast<uint32_t *>(smem);
    stage_words(table_w, a.order_table, a.n_order);
    lp_u32 table = (lp_u32)table_w;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
    const int sub = lane & (kDcLanes - 1), mine = lane / kDcLanes;
    const uint32_t rings = (uint32_t)(uintptr_t)(lw_u8)(smem + table_bytes);
    const uint32_t ring = rings + (uint32_t)((wave * kDcRows + mine) * kDcRowBytes);  // this lane's row
    for (uint32_t i = 8u * (uint32_t)tid; i < (uint32_t)(waves * kDcRows * kDcRowBytes); i += 8u * blockDim.x)
        *(lw_u64)(uintptr_t)(rings + i) = 0ull;
    const uint32_t n_groups3 = 3u * (uint32_t)a.n_groups, last = (uint32_t)a.n_order - 1u, cols8 = 8u * (uint32_t)a.cols;
    // (a table too small for the index of every codeword: an unknown one may read other bytes as an entry, whose weights
    // need not lie inside its run)
    const bool any_entry = last < 0xFFFFu >> 2;

    // Which matrices have a destination: one bit each, so that the units of those that are asked for are dealt out.
    using lw_mask = __attribute__((address_space(3))) unsigned long long *;
    lw_mask mask = (lw_mask)(uintptr_t)(rings + (uint32_t)(waves * kDcRows * kDcRowBytes));  // [(n_mats + 63) / 64]
    const int mask_words = (a.n_mats + 63) / 64;
    for (int w = wave; w < mask_words; w += waves) {
        const int m = 64 * w + lane;
        const unsigned long long bits = __ballot(m < a.n_mats && a.out[m] != nullptr);
        if (lane == 0) mask[w] = bits;
    }
    __syncthreads();
    // Units of a matrix: kDcRows consecutive rows, or, in the lane-interleaved layout, the i-th rows of as many consecutive
    // lanes' row ranges (their pieces lie next to each other).  A wavefront takes every a.slots-th unit of a matrix: one, but
    // for the lane-interleaved layout of a matrix with rows that its lanes do not divide.
    constexpr int kBpe = OUT == 0 ? 1 : 2, kRunBytes = kDcGroup * kBpe;

    // The units of all wanted matrices are dealt out round robin.  A wavefront's next unit is as many units on as there are
    // wavefronts: so many matrices and so many slots, known to the host, and the matrix is found from the place of the last one
    // (with thousands of small matrices, a walk from the mask's first word and a division for every unit are most of a unit's time).
    const int first = (int)blockIdx.x * waves + wave;  // (below 2^16)
    int nth = __builtin_amdgcn_readfirstlane((int)(((float)first + 0.5f) * a.inv_slots)), slot = first - nth * a.slots;
    int word = 0, skip = nth;                 // the matrix is the skip-th of the bits left in this word and the words after it
    auto word_bits = [&](int w) -> unsigned long long {  // the same in every lane
        const unsigned long long b = mask[w];
        return (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b) |
               (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32;
    };
    unsigned long long bits = word_bits(0);
    int n_wanted = __popcll(bits);
    if (mask_words > 1) {
        n_wanted = 0;
        for (int w = 0; w < mask_words; w += 64) n_wanted += w + lane < mask_words ? __popcll(mask[w + lane]) : 0;
        n_wanted = __builtin_amdgcn_readlane(wave_inclusive_scan(n_wanted), 63);
    }
    while (nth < n_wanted) {
        for (;;) {
            const int n = __popcll(bits);
            if (skip < n) break;
            skip -= n;
            bits = word_bits(++word);
        }
        int m = 64 * word;
        {
            int at = 0;
            unsigned long long rest = bits;
#pragma unroll
            for (int half = 32; half >= 1; half >>= 1) {
                const int n = __popcll(rest & ((1ull << half) - 1ull));
                const bool up = skip >= n;
                skip -= up ? n : 0;
                at += up ? half : 0;
                rest >>= up ? half : 0;
            }
            bits &= ~0ull << at;              // this matrix and those after it
            m = __builtin_amdgcn_readfirstlane(m + at);  // (the same in every lane; said so, its descriptor is read into scalar registers)
        }
        const uintptr_t out = reinterpret_cast<uintptr_t>(a.out[m]);
        const qmoe_matrix M = a.mats[m];
        const int lanes = (int)M.lanes, base = lanes ? a.rows / lanes : 0, extra = a.rows - base * lanes;
        const int blocks = lanes / kDcRows, units = lanes ? blocks * (base + (extra ? 1 : 0)) : a.slots;
        for (int unit = slot; unit < units; unit += a.slots) {
            int row;
            bool live;
            if (lanes) {
                const int i = unit / blocks, l = (unit - i * blocks) * kDcRows + mine;
                row = l * base + min(l, extra) + i;
                live = i < base + (l < extra ? 1 : 0);
            } else {
                row = unit * kDcRows + mine;
                live = row < a.rows;
            }
            const RowStream rs = row_stream(M, live ? row : 0, live);
            uint32_t s2 = 0u;  // bf16 scale in both halves (OUT 2: the (w_min, w_max) pair as stored)
            if constexpr (OUT == 2) {
                if (M.minmax_bf16) s2 = ((gp_u32)M.minmax_bf16)[live ? row : 0];
            }
            if constexpr (OUT == 1) {
                const uint32_t b = float_to_bf16_bits(half_bits_to_float(((gp_u16)M.scale_f16)[live ? row : 0]));
                s2 = b | (b << 16);
            }
            const uintptr_t dst = out + (uintptr_t)kBpe * (uintptr_t)(live ? row : 0) * (uintptr_t)a.cols;
            // (destinations are 16-byte aligned and cols is a multiple of 8, so this is a multiple of 8 columns)
            int done = live ? -(int)((dst % kRunBytes) / kBpe) : 0;  // columns written out so far
            const int n = (int)rs.left, lead = (int)rs.sub;
            uint32_t pos8 = 0u;  // 8 * column the row has reached
            // quarter-piece h of the row: codewords 2 h - lead and 2 h - lead + 1
            int quarters = n ? (lead + n + 1) >> 1 : 0;
            if (lanes) quarters = min(quarters, 4 * (int)((rs.last - rs.pp) >> 10) + 4);  // (none behind `last`)
            auto load = [&](int h) -> uint32_t {
                const int at = max(min(h, quarters - 1), 0);
                return *(gp_u32)(rs.pp + rs.pstride * (uintptr_t)(at >> 2) + 4u * (uintptr_t)(at & 3));
            };
            uint32_t v = load(sub);
            bool more = true;
            for (int h0 = 0; more; h0 += kDcLanes) {
                const int h = h0 + sub;
                const uint32_t v_next = load(h + kDcLanes);
                uint32_t e[2];
                order_entry2(table, v, n_groups3, last, e[0], e[1]);
                uint32_t len8 = 0u;
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    if ((uint32_t)(2 * h - lead + j) >= (uint32_t)n) e[j] = 0u;  // not the row's codeword
                    len8 += e[j] & 0xFFu;
                }
                const uint32_t incl = lanes_scan(len8, kDcLanes, sub);
                uint32_t p = pos8 + incl - len8;
                pos8 += (uint32_t)__shfl((int)incl, lane | (kDcLanes - 1), 64);
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    // (an entry's unused fields come first and store a zero at the run's first column, ahead of its weights)
                    if (e[j]) {
#pragma unroll
                        for (int z = 0; z < kRunMaxNonzeros; z++) {
                            const uint32_t t = p + ((e[j] >> (8 + 8 * z)) & 0xFFu);  // 8 * column + the field's low three bits
                            // value bits of the field (2: +1, 6: -1): as they are (asymmetric grid: byte selectors), or at the top
                            // of the byte (0x40 / 0xC0)
                            *(lw_u8)(uintptr_t)(ring + ((t >> 3) & (uint32_t)(kDcRing - 1))) = (unsigned char)(OUT == 2 ? (t & 6u) : (t << 5));
                        }
                    }
                    p += e[j] & 0xFFu;
                }
                v = v_next;
                more = __any(2 * (h0 + kDcLanes) < lead + n);
                // ---- whole groups leave the ring; with the row's last codeword everything up to its end
                const int reached = 2 * (h0 + kDcLanes) < lead + n ? (int)(pos8 >> 3) : (live ? a.cols + kDcGroup - 1 : 0);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                while (__any(done + kDcGroup <= reached)) {
                    if (done + kDcGroup <= reached) {
                        const int k = done + 8 * sub;
                        done += kDcGroup;
                        if (k >= 0 && k + 8 <= a.cols) {
                            lw_u64 at = (lw_u64)(uintptr_t)(ring + ((uint32_t)k & (uint32_t)(kDcRing - 1)));
                            const unsigned long long d = *at;
                            *at = 0ull;
                            const uint32_t w0 = (uint32_t)d, w1 = (uint32_t)(d >> 32);
                            if constexpr (OUT == 0) {
                                // ring byte 0x40 -> 0x01, 0xC0 -> 0xFF, 0 -> 0
                                const uint32_t n0 = (w0 >> 7) & 0x01010101u, n1 = (w1 >> 7) & 0x01010101u;
                                const uint32_t o0 = ((w0 >> 6) & 0x01010101u) | ((n0 << 8) - n0), o1 = ((w1 >> 6) & 0x01010101u) | ((n1 << 8) - n1);
                                __builtin_nontemporal_store((unsigned long long)o0 | ((unsigned long long)o1 << 32), (gw_u64)(dst + (uintptr_t)k));
                            } else if constexpr (OUT == 2) {
                                __builtin_nontemporal_store(select_minmax(w0, w1, s2 << 16, s2 & 0xFFFF0000u), (gw_u32x4)(dst + 2 * (uintptr_t)k));
                            } else {
                                u32x4 o;
#pragma unroll
                                for (int i = 0; i < 4; i++) {
                                    // two ring bytes -> the high bytes of two 16-bit halves: 0x4000 / 0xC000 / 0
                                    const uint32_t b = __builtin_amdgcn_perm(0u, i < 2 ? w0 : w1, (i & 1) ? 0x030c020cu : 0x010c000cu);
                                    const uint32_t ones = (b >> 14) & 0x00010001u;
                                    o[i] = ((b & 0x80008000u) | s2) & ((ones << 16) - ones);
                                }
                                __builtin_nontemporal_store(o, (gw_u32x4)(dst + 2 * (uintptr_t)k));
                            }
                        }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            // A (corrupt) stream that ran past the row's width -- or has more codewords than columns, so many that the column may
            // have wrapped -- left weights in the ring behind its last column, which would be weights of the ring's next row.
            if (any_entry || __any(pos8 > cols8 || n > a.cols)) {
                for (int i = 8 * sub; i < kDcRing; i += 8 * kDcLanes) *(lw_u64)(uintptr_t)(ring + (uint32_t)i) = 0ull;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        slot += a.next_slot;
        skip = a.next_nth;
        if (slot >= a.slots) {
            slot -= a.slots;
            skip++;
        }
        nth += skip;
    }
}

}  // namespace

template <int LANES>
static size_t dc_lds_bytes(int n_order, int n_mats)
{
    return (((size_t)n_order * 4 + 15) & ~(size_t)15) + (size_t)kDcMaxWaves * DcShape<LANES>::kRows * DcShape<LANES>::kRowBytes +
           8 * (((size_t)n_mats + 63) / 64);
}

size_t decompress_lds_bytes(int n_order, int n_mats) { return dc_lds_bytes<kDcWide>(n_order, n_mats); }

template <int LANES>
static qmoe_status launch_dc(DecompressArgs a, int out_kind, bool minmax, int cus, hipStream_t s)
{
    constexpr int kRows = DcShape<LANES>::kRows;
    const size_t smem = dc_lds_bytes<LANES>(a.n_order, a.n_mats);
    a.slots = (a.rows + kRows - 1) / kRows;
    // as few wavefronts as take the units in the same number of rounds
    const long long total = (long long)a.n_mats * a.slots, most = (long long)cus * kDcMaxWaves, rounds = (total + most - 1) / most;
    const int waves = (int)std::max(1LL, std::min<long long>(kDcMaxWaves, (total + cus * rounds - 1) / (cus * rounds)));
    const int grid = (int)std::min<long long>((total + waves - 1) / waves, (long long)cus);
    a.next_nth = grid * waves / a.slots;
    a.next_slot = grid * waves % a.slots;
    a.inv_slots = 1.0f / (float)a.slots;
    auto launch = [&](auto kernel) -> qmoe_status {
        const qmoe_status st = allow_lds(kernel, smem);
        if (st != QMOE_OK) return st;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * waves), smem, s, a);
        return QMOE_OK;
    };
    const qmoe_status st =
        out_kind == 0 ? launch(k_decompress<0, LANES>) : (minmax ? launch(k_decompress<2, LANES>) : launch(k_decompress<1, LANES>));
    if (st != QMOE_OK) return st;
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

qmoe_status launch_decompress(const DecompressArgs &a, int out_kind, bool minmax, int cus, int max_lds, hipStream_t s)
{
    // A row of some hundred columns is one step of 32 lanes, most of them without a codeword, and a unit's trips to memory are
    // most of its time: eight rows a wavefront, eight lanes each, make them a quarter as many.  To int8, 256 rows a matrix,
    // wide and narrow: 2048 of 256 columns 131 and 60 us, 1024 of 512 columns 75 and 42, 682 of 768 columns 57 and 48, 512
    // of 1024 columns 47 and 46; in a single round a row's length counts, and the lines cross at 384 to 512 columns (42
    // matrices of 384: 7.7 and 7.2 us, 32 of 512: 6.8 and 7.8).
    const bool rounds = (long long)a.n_mats * ((a.rows + 1) / 2) >= 4LL * cus * kDcMaxWaves;
    if (a.cols <= (rounds ? 768 : 384) && dc_lds_bytes<kDcNarrow>(a.n_order, a.n_mats) <= (size_t)max_lds)
        return launch_dc<kDcNarrow>(a, out_kind, minmax, cus, s);
    return launch_dc<kDcWide>(a, out_kind, minmax, cus, s);
}

}  // namespace qmoe
