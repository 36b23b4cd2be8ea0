// The matrix-core product for crowded experts (Section 5.3 of the paper proposes decoding once for
// several tokens).
#include "qmoe_dev.h"

namespace qmoe {
namespace {

// ---------------------------------------------------------------- matrix-core product for crowded experts
//
// An expert with many tokens is a dense contraction once its ternary weights are
// in hand: y[token][row] = sum_k x[token][k] * W[row][k].  The scalar kernel
// would decode the matrix again for every few tokens; this one decodes it once per
// tile of up to 64 tokens.  A wavefront owns 64 rows (one lane per row) and walks
// the columns 64 at a time.  Every lane keeps a ring of 256 columns of its
// row in LDS, four bits a column, and decodes its codewords into it, as far ahead as the
// ring allows (so the lanes of a wavefront, whose codewords end at different
// columns, seldom wait for each other); then the wavefront multiplies the 64
// columns that are complete, for the 64 rows its lanes decoded, with the tokens'
// activations on the matrix cores, fp32 accumulators in registers.  The
// ring holds the weights as fp4 numbers (+-2.0), which one instruction widens to bf16, two at a time; the factor 2
// is taken out again, exactly, when a row is written.
// Only device-order streams (whole table in LDS) take this path.
//
// What bounds it: the length of a step on a wavefront, of which the LDS holds two per SIMD (rings, windows and table); they do
// not hide each other's waits altogether.  256 experts of 2080 x 6144 with 16 tokens each, first / second product, 394 / 348 us
// when this was measured: without the rounds 318 / 242, without the multiply 355 / 291, without rounds, multiply and stream loads
// 209 / 113, one step a unit 121 / 67; all rows of a wavefront the same (one line a load) and without the rounds 266 / 216.
// Vector units issue on 58 % of the cycles (142 instructions a step), the LDS works 45 %.
//
// (Four codewords a round and four bits a column: with one codeword a round and a byte a column, three byte stores a codeword and the
// ring cleared by stores, the same layer took 449 / 420 us with the units handed out by tickets, 430 / 361 this way; rows of mixed sparsity
// 498 / 475 and 493 / 435.  As it stands: 370 / 337, on the asymmetric grid 447 / 436.  Slower or no different, measured: the trips to memory of the
// next unit during the present one, 905 -> 930 us for 256 experts with 1 to 32 tokens; the activations of 64-token tiles a step ahead, 765 -> 785.)

constexpr int kMmKc = 64;                      // columns per step
constexpr int kMmRing = 256;                   // columns a lane's ring holds
constexpr int kMmGroup = 4;                    // codewords a lane decodes in a round
constexpr int kMmAhead = kMmRing - 28 * kMmGroup;  // a round may start this far past the step's first column (its runs then end
                                                   // below the first column that shares a place in the ring with the step)
constexpr int kMmRowBytes = kMmRing / 2;       // four bits a column
constexpr int kMmWindow = 16;                  // codewords of a lane's window: two pieces of eight

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// eight columns of four bits (0x4: +2, 0xC: -2 as an fp4 number) -> eight bf16
__device__ __forceinline__ bf16x8 mm_expand(uint32_t d)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 o[4];
    o[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(d, 1.0f, 0);
    o[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(d, 1.0f, 1);
    o[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(d, 1.0f, 2);
    o[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(d, 1.0f, 3);
    bf16x8 r;
    __builtin_memcpy(&r, o, 16);
    return r;
}

// The same on the asymmetric grid: byte selectors (0: zero, 2: w_max, 6: w_min) of the even and of the odd columns pick the
// row's own bf16 grid points out of lo = w_max << 16, hi = w_min << 16 (see select_minmax).
__device__ __forceinline__ bf16x8 mm_expand_minmax(uint32_t d, uint32_t hi, uint32_t lo)
{
    const uint32_t even = (d >> 1) & 0x06060606u, odd = (d >> 5) & 0x06060606u;
    u32x4 o;
    o.x = __builtin_amdgcn_perm(hi, lo, __builtin_amdgcn_perm(odd, even, 0x04040000u) + 0x01000100u);
    o.y = __builtin_amdgcn_perm(hi, lo, __builtin_amdgcn_perm(odd, even, 0x05050101u) + 0x01000100u);
    o.z = __builtin_amdgcn_perm(hi, lo, __builtin_amdgcn_perm(odd, even, 0x06060202u) + 0x01000100u);
    o.w = __builtin_amdgcn_perm(hi, lo, __builtin_amdgcn_perm(odd, even, 0x07070303u) + 0x01000100u);
    bf16x8 r;
    __builtin_memcpy(&r, &o, 16);
    return r;
}

using lw_u8 = __attribute__((address_space(3))) unsigned char *;
using lw_u32 = __attribute__((address_space(3))) uint32_t *;
using lw_u64 = __attribute__((address_space(3))) unsigned long long *;
using lw_u32x4 = __attribute__((address_space(3))) u32x4 *;
using lp_u64 = const __attribute__((address_space(3))) unsigned long long *;

// ---- the ring decoder ----
//
// One lane = one row.  A lane's codewords pass through a window of two 16-byte pieces (four groups of four codewords) in LDS.
// A round takes one group: four table entries are looked up side by side and their
// fields put into the lane's ring by ORs (a field without a weight ORs zero), which cost the LDS what stores of a byte do.  A step's operand read
// takes the weights out by exchanges with zero, so that nothing is cleared.
//
// The LDS begins with the table (at address 0; launch_product_mm sees to that), then the rings, then the windows.  A ring is 32 words
// of eight columns; the rings of eight rows lie word by word, [8 rows][32 words][row of the eight], so that a place -- four times a column, plus
// a constant -- has the word's address in its upper bits as it stands and the shift inside the word in its lower five.
__host__ __device__ inline size_t mm_table_bytes(int n_order) { return ((size_t)n_order * 4 + 2047) & ~(size_t)2047; }
constexpr size_t kMmWindowBytes = 2 * kMmWindow;  // a lane's
constexpr uint32_t kMmWord = 0x3E0;               // bits of a place that are the word's address
static_assert(kMmRing == 256 && kMmRowBytes == 128, "32 words of eight columns, 32 bytes from one to the next");

// The rings of rows 8 .. 15 of 16 begin four words on: the 16 rows x 4 words of an operand read fall on 64 banks.
__device__ __forceinline__ uint32_t ring_begin(uint32_t row) { return 128u * ((row >> 3) & 1u); }

// The table in LDS has its entries' bytes in another order than the one in memory, each halved: field 1, field 0, field 2,
// length.  A byte is 4 * position | weight as two signed bits; what the two low bits of a code flip, the signs of fields 1 and
// 2, is then bits 1 and 17, and one product of the code's low byte puts both there (its other bits are left to the mask).
__device__ __forceinline__ uint32_t ring_entry_bytes(uint32_t e)
{
    return (__builtin_amdgcn_perm(e, e, 0x00030102u) >> 1) & 0x7F7F7F7Fu;
}
constexpr uint32_t kMmFlipMul = 0x00010002u, kMmFlips = 0x00020002u, kMmPlaces = 0x7C7C7C7Cu, kMmWeights = 0x03030303u;

struct RingDecoder {
    // (codewords counted from the first of the row's first piece)
    uint32_t ci;               // the next group's first codeword
    uint32_t n;                // one past the row's last group.  What follows the row's last codeword in that group is somebody else's: its
                               // runs lie behind the row's last column, where the activations are zeros
    uint32_t have, asked;      // one past the last codeword in the window, and past the last one asked for
    uint32_t pos;              // place of the column where the next run starts
    uintptr_t first;           // the row's first piece
    uint32_t step_log2;        // codeword -> bytes from the first piece: 1, or 7 where a lane's pieces lie 1024 bytes apart
    uint32_t wrow, slot;       // LDS byte addresses of the lane's ring and window
};

// A piece on its way to the window.
struct RingPiece {
    u32x4 v;
    uint32_t at;  // its first codeword (kMmNoPiece: the lane asked for none)
};
constexpr uint32_t kMmNoPiece = ~0u;

// Asks for a lane's next piece where the window has room for it, or will have when the lane has used one more group, which it
// nearly always has by the time that the piece arrives.  (Asked for only when there is room, a piece is late for rows with a codeword
// for every 20 values or fewer: one step in eight of such a wavefront waited for it, and so for all that was in flight; one
// in a hundred now.)  All lanes load, those that ask for nothing the matrix's first
// piece: what is in flight at any point of the program is then known to the compiler, whose waits for the activations would
// otherwise be waits for the stream too.
__device__ __forceinline__ void ring_ask(RingDecoder &d, const void *codes, RingPiece &p)
{
    const bool ask = (int)(d.asked - d.ci) <= kMmWindow / 2 + kMmGroup && d.asked < d.n;  // (at first ci may be ahead, in the middle of the first piece)
    p.v = *(gp_u32x4)(ask ? d.first + ((uintptr_t)(d.asked << d.step_log2)) : reinterpret_cast<uintptr_t>(codes));
    p.at = ask ? d.asked : kMmNoPiece;
    d.asked += ask ? 8u : 0u;
}

// The window is kept by groups, [group][lane]: a wavefront's reads do not meet in a bank.  A piece that comes too early is
// dropped, and so is the one behind it, and asked for again.
__device__ __forceinline__ void ring_arrive(RingDecoder &d, RingPiece &p)
{
    asm volatile("" ::"v"(p.v));  // (the wait belongs here, whether a lane asked or not)
    const bool next = p.at == d.have, room = (int)(d.have - d.ci) <= kMmWindow / 2;
    d.asked = next && !room ? d.have : d.asked;
    if (next && room) {
        lw_u64 w = (lw_u64)(uintptr_t)(((d.have << 7) & 1024u) | d.slot);
        w[0] = (unsigned long long)p.v.x | ((unsigned long long)p.v.y << 32);
        w[64] = (unsigned long long)p.v.z | ((unsigned long long)p.v.w << 32);
        d.have += 8u;
    }
    p.at = kMmNoPiece;
}

__device__ __forceinline__ uint32_t byte_of(uint32_t v, int k) { return (v >> (8 * k)) & 0xFFu; }

struct RingTable {
    uint32_t groups3, last;  // 3 * groups and the last entry's index, twice each, side by side
};

__device__ __forceinline__ unsigned long long ring_codes_at(const RingDecoder &d, uint32_t at)
{
    return *(lp_u64)(uintptr_t)(((at << 7) & 0x600u) | d.slot);
}

// LDS byte offsets of two codewords' table entries: the index that order_entry2 takes, times four.
__device__ __forceinline__ void ring_entries_at(const RingTable &tab, uint32_t w, uint32_t &at0, uint32_t &at1)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    u16x2 c, g, l;
    __builtin_memcpy(&c, &w, 4);
    __builtin_memcpy(&g, &tab.groups3, 4);
    __builtin_memcpy(&l, &tab.last, 4);
    const u16x2 two = {2, 2};
    const u16x2 i = __builtin_elementwise_min(__builtin_elementwise_max(c >> two, __builtin_elementwise_sub_sat(c, g)), l);
    uint32_t both;
    __builtin_memcpy(&both, &i, 4);
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(at0) : "s"(2), "v"(both));
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(at1) : "s"(2), "v"(both));
}

// A group: its codewords and their entries as read.
struct RingGroup {
    uint32_t w[2], e[kMmGroup];
};

__device__ __forceinline__ RingGroup ring_look_up(const RingTable &tab, unsigned long long four)
{
    RingGroup g;
    uint32_t at[kMmGroup];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        g.w[h] = (uint32_t)(four >> (32 * h));
        ring_entries_at(tab, g.w[h], at[2 * h], at[2 * h + 1]);
    }
#pragma unroll
    for (int j = 0; j < kMmGroup; j++) g.e[j] = *(lp_u32)(uintptr_t)at[j];
    return g;
}

// A row's first group: of its codewords only those from `from` on are the row's.
__device__ __forceinline__ void ring_apply_part(RingDecoder &d, const RingGroup &g, uint32_t from)
{
#pragma unroll
    for (int j = 0; j < kMmGroup; j++) {
        const uint32_t k = d.ci + (uint32_t)j, flips = ((g.w[j >> 1] >> (16 * (j & 1))) & 0xFFu) * kMmFlipMul;
        const bool own = k >= from;
        const uint32_t places = own ? g.e[j] & kMmPlaces : 0u, weights = own ? (g.e[j] & kMmWeights) ^ (flips & kMmFlips) : 0u;
#pragma unroll
        for (int z = 0; z < 3; z++) {
            const uint32_t t = d.pos + byte_of(places, z);
            __hip_atomic_fetch_or((lw_u32)(uintptr_t)((t & kMmWord) | d.wrow), byte_of(weights, z) << (t & 31u), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        d.pos += places >> 24;
    }
    d.ci += kMmGroup;
}

// Rounds of one whole group per lane, until no lane of the wavefront that may go on (ci < stop) is before `end`.  A lane
// that sits out -- no group left in the window, or too far ahead (pos > lim) -- does so for the rest of the call.  `g`: the
// lanes' first groups.
//
// A group's codewords are read before the group ahead of it is applied, and looked up only if there is another round.  In assembly
// because lanes leave by the execution mask, which only shrinks: the compiler keeps old and new state of every lane apart
// and moves it back and forth (a round is 20 vector instructions a codeword here).
__device__ __forceinline__ void ring_rounds(RingDecoder &d, const RingTable &tab, RingGroup g, uint32_t stop, uint32_t lim, uint32_t end)
{
    uint32_t f, wt, pl, t0, t1, t2, a0, a1, a2;
    uint32_t n0, n1;
    unsigned long long all;
    asm volatile(
                 "s_mov_b64 %[all], exec\n\t"
                 "v_cmpx_lt_u32_e32 vcc, %[ci], %[stop]\n\t"
                 "v_cmpx_ge_u32_e32 vcc, %[lim], %[pos]\n\t"
                 "v_cmp_lt_u32_e32 vcc, %[pos], %[end]\n\t"
                 "s_cbranch_vccz 1f\n\t"
                 "0:\n\t"
                 "v_add_u32_e32 %[ci], 4, %[ci]\n\t"
                 "v_lshlrev_b32_e32 %[t0], 7, %[ci]\n\t"
                 "v_and_or_b32 %[t0], %[t0], %[groups], %[slot]\n\t"
                 "ds_read_b32 %[n0], %[t0]\n\t"
                 "ds_read_b32 %[n1], %[t0] offset:4\n\t"
                 "v_mul_u32_u24_sdwa %[f], %[w0], %[mul] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_and_b32_e32 %[wt], %[weights], %[e0]\n\t"
                 "v_and_b32_e32 %[pl], %[places], %[e0]\n\t"
                 "v_bitop3_b32 %[wt], %[f], %[wt], %[flips] bitop3:0x6c\n\t"
                 "v_add_u32_sdwa %[t0], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t1], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t2], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[pos], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t"
                 "v_and_or_b32 %[a0], %[t0], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a1], %[t1], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a2], %[t2], %[word], %[ring]\n\t"
                 "v_lshlrev_b32_sdwa %[t0], %[t0], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0\n\t"
                 "v_lshlrev_b32_sdwa %[t1], %[t1], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[t2], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2\n\t"
                 "ds_or_b32 %[a0], %[t0]\n\t"
                 "ds_or_b32 %[a1], %[t1]\n\t"
                 "ds_or_b32 %[a2], %[t2]\n\t"
                 "v_mul_u32_u24_sdwa %[f], %[w0], %[mul] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_and_b32_e32 %[wt], %[weights], %[e1]\n\t"
                 "v_and_b32_e32 %[pl], %[places], %[e1]\n\t"
                 "v_bitop3_b32 %[wt], %[f], %[wt], %[flips] bitop3:0x6c\n\t"
                 "v_add_u32_sdwa %[t0], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t1], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t2], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[pos], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t"
                 "v_and_or_b32 %[a0], %[t0], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a1], %[t1], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a2], %[t2], %[word], %[ring]\n\t"
                 "v_lshlrev_b32_sdwa %[t0], %[t0], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0\n\t"
                 "v_lshlrev_b32_sdwa %[t1], %[t1], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[t2], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2\n\t"
                 "ds_or_b32 %[a0], %[t0]\n\t"
                 "ds_or_b32 %[a1], %[t1]\n\t"
                 "ds_or_b32 %[a2], %[t2]\n\t"
                 "v_mul_u32_u24_sdwa %[f], %[w1], %[mul] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_and_b32_e32 %[wt], %[weights], %[e2]\n\t"
                 "v_and_b32_e32 %[pl], %[places], %[e2]\n\t"
                 "v_bitop3_b32 %[wt], %[f], %[wt], %[flips] bitop3:0x6c\n\t"
                 "v_add_u32_sdwa %[t0], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t1], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t2], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[pos], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t"
                 "v_and_or_b32 %[a0], %[t0], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a1], %[t1], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a2], %[t2], %[word], %[ring]\n\t"
                 "v_lshlrev_b32_sdwa %[t0], %[t0], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0\n\t"
                 "v_lshlrev_b32_sdwa %[t1], %[t1], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[t2], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2\n\t"
                 "ds_or_b32 %[a0], %[t0]\n\t"
                 "ds_or_b32 %[a1], %[t1]\n\t"
                 "ds_or_b32 %[a2], %[t2]\n\t"
                 "v_mul_u32_u24_sdwa %[f], %[w1], %[mul] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_and_b32_e32 %[wt], %[weights], %[e3]\n\t"
                 "v_and_b32_e32 %[pl], %[places], %[e3]\n\t"
                 "v_bitop3_b32 %[wt], %[f], %[wt], %[flips] bitop3:0x6c\n\t"
                 "v_add_u32_sdwa %[t0], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t1], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[t2], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t"
                 "v_add_u32_sdwa %[pos], %[pl], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t"
                 "v_and_or_b32 %[a0], %[t0], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a1], %[t1], %[word], %[ring]\n\t"
                 "v_and_or_b32 %[a2], %[t2], %[word], %[ring]\n\t"
                 "v_lshlrev_b32_sdwa %[t0], %[t0], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0\n\t"
                 "v_lshlrev_b32_sdwa %[t1], %[t1], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[t2], %[wt] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2\n\t"
                 "ds_or_b32 %[a0], %[t0]\n\t"
                 "ds_or_b32 %[a1], %[t1]\n\t"
                 "ds_or_b32 %[a2], %[t2]\n\t"
                 "v_cmpx_lt_u32_e32 vcc, %[ci], %[stop]\n\t"
                 "v_cmpx_ge_u32_e32 vcc, %[lim], %[pos]\n\t"
                 "v_cmp_lt_u32_e32 vcc, %[pos], %[end]\n\t"
                 "s_waitcnt lgkmcnt(12)\n\t"
                 "s_cbranch_vccz 1f\n\t"
                 "v_mov_b32_e32 %[w0], %[n0]\n\t"
                 "v_mov_b32_e32 %[w1], %[n1]\n\t"
                 "v_pk_lshrrev_b16 %[t0], 2, %[n0] op_sel_hi:[0,1]\n\t"
                 "v_pk_sub_u16 %[t1], %[n0], %[g3] clamp\n\t"
                 "v_pk_max_u16 %[t0], %[t0], %[t1]\n\t"
                 "v_pk_min_u16 %[t0], %[t0], %[last]\n\t"
                 "v_lshlrev_b32_sdwa %[a0], %[two], %[t0] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[two], %[t0] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
                 "ds_read_b32 %[e0], %[a0]\n\t"
                 "ds_read_b32 %[e1], %[t2]\n\t"
                 "v_pk_lshrrev_b16 %[t0], 2, %[n1] op_sel_hi:[0,1]\n\t"
                 "v_pk_sub_u16 %[t1], %[n1], %[g3] clamp\n\t"
                 "v_pk_max_u16 %[t0], %[t0], %[t1]\n\t"
                 "v_pk_min_u16 %[t0], %[t0], %[last]\n\t"
                 "v_lshlrev_b32_sdwa %[a1], %[two], %[t0] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
                 "v_lshlrev_b32_sdwa %[t2], %[two], %[t0] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
                 "ds_read_b32 %[e2], %[a1]\n\t"
                 "ds_read_b32 %[e3], %[t2]\n\t"
                 "s_waitcnt lgkmcnt(0)\n\t"
                 "s_branch 0b\n\t"
                 "1:\n\t"
                 "s_mov_b64 exec, %[all]\n\t"
                 : [ci] "+v"(d.ci), [pos] "+v"(d.pos), [w0] "+v"(g.w[0]), [w1] "+v"(g.w[1]), [e0] "+v"(g.e[0]), [e1] "+v"(g.e[1]),
                   [e2] "+v"(g.e[2]), [e3] "+v"(g.e[3]), [f] "=&v"(f), [wt] "=&v"(wt), [pl] "=&v"(pl), [t0] "=&v"(t0), [t1] "=&v"(t1),
                   [t2] "=&v"(t2), [a0] "=&v"(a0), [a1] "=&v"(a1), [a2] "=&v"(a2), [n0] "=&v"(n0), [n1] "=&v"(n1), [all] "=&s"(all)
                 : [stop] "v"(stop), [lim] "v"(lim), [end] "v"(end), [slot] "v"(d.slot), [ring] "v"(d.wrow), [groups] "s"(0x600u),
                   [mul] "s"(kMmFlipMul), [flips] "s"(kMmFlips), [weights] "s"(kMmWeights), [places] "s"(kMmPlaces), [word] "s"(kMmWord),
                   [g3] "s"(tab.groups3), [last] "s"(tab.last), [two] "s"(2)
                 : "vcc", "memory");
}

// The lane's row (none: an empty stream), its window filled, its ring cleared, its first group decoded.  `meanwhile` runs when the
// window's pieces have been asked for: what it asks for is on its way together with them.
template <class Meanwhile>
__device__ __forceinline__ void ring_setup(RingDecoder &d, const RingTable &tab, const qmoe_matrix &M, int row, bool row_live, uint32_t lane,
                                           uint32_t rings, uint32_t slot, Meanwhile &&meanwhile)
{
    const RowStream rst = row_stream(M, row, row_live);
    // (the row's pieces end with rst.last, which offsets that are none do not move behind the stream)
    const uint32_t pieces = (uint32_t)((rst.last - rst.pp) >> (M.lanes ? 10 : 4)) + 1u;
    // (2^24: no row has as many, and a place in the stream counts its bytes in 32 bits)
    const uint32_t n = rst.left ? min(min(rst.sub + rst.left, 8u * pieces), 1u << 24) : 0u;
    d.n = (n + kMmGroup - 1) & ~(uint32_t)(kMmGroup - 1);
    d.ci = rst.sub & ~(uint32_t)(kMmGroup - 1);
    d.first = rst.pp;
    d.step_log2 = M.lanes ? 7u : 1u;
    d.wrow = rings + 1024u * (lane >> 3) + 4u * (lane & 7u);
    d.slot = slot;
    d.have = d.asked = 0u;
    RingPiece p0, p1;
    ring_ask(d, M.codes, p0);
    ring_ask(d, M.codes, p1);
    meanwhile();
    d.pos = ring_begin(lane) + 2u;
#pragma unroll
    for (int i = 0; i < kMmRowBytes / 16; i++) ((lw_u32x4)(uintptr_t)rings)[64 * i + (int)lane] = u32x4{0u, 0u, 0u, 0u};
    ring_arrive(d, p0);
    ring_arrive(d, p1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (__any(rst.sub & 3u)) {
        if (d.ci < d.n) ring_apply_part(d, ring_look_up(tab, ring_codes_at(d, d.ci)), rst.sub);
    }
}

// Decode until every lane of the wavefront has passed column kc + 64 (or its row's end).  A lane that is there
// already keeps going as long as its next group's runs end before the first column that shares a
// place in the ring with the step, so the lanes of a wavefront, whose codewords end at different columns, seldom wait for each
// other.  `g`: the lanes' first groups, looked up during the multiply of the step before.  A piece arrives at the end of the step after the one it
// was asked for in: `older` has arrived and is asked for anew, `newer` is in flight.
__device__ __forceinline__ void ring_decode_step(RingDecoder &d, const RingTable &tab, uint32_t first, const void *codes, RingPiece &older, RingPiece &newer,
                                                 const RingGroup &g)
{
    const uint32_t lim = first + 4u * kMmAhead, end = first + 4u * kMmKc;
    ring_ask(d, codes, older);
    ring_rounds(d, tab, g, min(d.n, d.have), lim, end);
    if (__any(d.ci < d.n && d.pos < end)) {  // a lane's window is empty: everything that was asked for, and more
        ring_arrive(d, newer);
        ring_arrive(d, older);
        do {
            RingPiece now;
            ring_ask(d, codes, now);
            ring_arrive(d, now);
            ring_rounds(d, tab, ring_look_up(tab, ring_codes_at(d, d.ci)), min(d.n, d.have), lim, end);
        } while (__any(d.ci < d.n && d.pos < end));
    }
}

// ---- the matrix-core product ----
//
// Every wavefront works on its own: its 64 lanes decode 64 consecutive rows into their rings,
// and when all of them have passed the next 64 columns the wavefront multiplies those 64 x 64
// weights with the tile's activations, which every lane fetches straight from global memory
// in the layout the matrix cores want (a token's 8 consecutive columns = one 16-byte load;
// the eight wavefronts of a workgroup read the same lines, which the caches serve).  No
// workgroup barrier inside an item.
//
// MB: blocks of 16 tokens in the tile (1, 2 or 4).  D[row][token] += W[row][k] * X^T[k][token]
// with v_mfma_f32_16x16x32_bf16: operand lane l holds 8 consecutive k (group l / 16) of row
// or token l % 16; accumulator v of lane l is row 4 * (l / 16) + v, token l % 16 of the block.  This way round a lane has
// four consecutive rows of one token and writes them at once.  (Tokens and rows the other way round, sixteen stores of one value a lane
// for every 16 tokens: 743 -> 728 us for 256 experts of 2080 x 6144 with 16 tokens each; row scales asked for at the set-up instead of
// behind the last step, 728 -> 717.)
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Returns the tile's tokens (a bit each) whose results want mm_again.
template <int MB, int EPI, int ASYM>
__device__ __forceinline__ unsigned long long mm_item(const ProductArgs &a, const qmoe_matrix &M, int rblk, int slot0, int ntok,
                                                      uint32_t wt, uint32_t win)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lg = lane >> 4;

    // Lane t asks for token t now, and in the second product, which writes to the tokens' own rows of the output, scaled
    // by their gates, for its gate, among the other trips to memory of the set-up (two registers for the
    // length of the item); the lanes swap them when the activations are asked for and when the results are written.
    const int at_own = slot0 + min(lane, ntok - 1);
    const int tok_own = a.perm ? ((const __attribute__((address_space(1))) int *)a.perm)[at_own] : at_own;
    float gate_own = 1.0f;
    uint32_t scale_own = 0u;  // scale (or grid pair) of the lane's row as stored; the lanes swap these, too

    // ---- this lane's row (the wavefront's 64 rows are block `rblk` of the matrix) and its codewords
    const int r0 = rblk * 64;
    const int row = r0 + lane;
    const bool row_live = row < a.rows;
    RingDecoder dec;
    const RingTable tab{(uint32_t)(3 * a.n_groups) * 0x10001u, (uint32_t)(a.n_order - 1) * 0x10001u};
    const uint32_t rings = wt + (uint32_t)(wave * 64 * kMmRowBytes);
    // ---- this lane's part of the activations: token 16 * mb + l16, columns 8 * lg .. 8 * lg + 7 of every 32
    uintptr_t xsrc[MB];
    uint32_t xmul2[MB];  // bytes from one column's value to the next column's: 2, or (tiled) 2 * the block's tokens
    const bool x_col = 8 * lg + 8 <= a.cols;
    const int x_last = x_col ? a.cols - 8 * lg - 8 : 0;  // last column offset this lane may read at
    uint32_t x_end[MB];  // x_last in bytes
    auto address_x = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; mb++) {
        const int t = 16 * mb + l16;
        xmul2[mb] = 2u;
        // (a lane whose columns do not exist -- fewer than 8 * lg + 8 columns -- reads column 0 and drops it;
        // a lane without a token reads the block's first token, or the tile's last)
        const size_t col0 = x_col ? 8 * (size_t)lg : (size_t)0;
        if (a.x_tiled) {
            const int tb = min(16, ntok - 16 * mb);  // tokens in this block (<= 0: no such block)
            const size_t block0 = tb > 0 ? (size_t)(slot0 + 16 * mb) : (size_t)slot0;
            const size_t j = t < ntok ? (size_t)l16 : (size_t)0;
            xmul2[mb] = 2u * (uint32_t)__builtin_amdgcn_readfirstlane(max(tb, 1));
            xsrc[mb] = reinterpret_cast<uintptr_t>(a.x) + 2 * (block0 * (size_t)a.ldx + 8 * j) + col0 * (size_t)xmul2[mb];
        } else {
            const int tok = __shfl(tok_own, t, 64);  // (where the tile has no such token, its last one)
            const size_t xrow = a.x_by_slot ? (size_t)(slot0 + min(t, ntok - 1)) : (size_t)tok;
            xsrc[mb] = reinterpret_cast<uintptr_t>(a.x) + 2 * (xrow * (size_t)a.ldx + col0);
        }
        x_end[mb] = (uint32_t)x_last * xmul2[mb];
    }
    };
    // A step's activations are asked for before its weights are decoded and arrive meanwhile.  What a lane without a token brings is some other row's and multiplies into a result nobody writes.
    // Only a last step of fewer than 64 columns looks at its columns: a lane past the last one reads column 8 * lg and
    // drops it.
    constexpr int kAhead = MB == 4 ? 0 : 1;  // steps the activations are asked for ahead
    u32x4 xa[kAhead + 1][MB][2];
    auto fetch_x = [&](u32x4 (&to)[MB][2], int k) {
        if (k + kMmKc <= a.cols) {
#pragma unroll
            for (int mb = 0; mb < MB; mb++) {
                const uintptr_t at = xsrc[mb] + (uintptr_t)((uint32_t)k * xmul2[mb]);
                to[mb][0] = *(gp_u32x4)at;
                to[mb][1] = *(gp_u32x4)(at + 32u * xmul2[mb]);
            }
        } else {
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int ks = 0; ks < 2; ks++)
                    to[mb][ks] = *(gp_u32x4)(xsrc[mb] + (uintptr_t)min((uint32_t)(k + 32 * ks) * xmul2[mb], x_end[mb]));
        }
    };
    ring_setup(dec, tab, M, row, row_live, (uint32_t)lane, rings, win + (uint32_t)(wave * 64 * (int)kMmWindowBytes + lane * 8), [&]() {
        address_x();
        if constexpr (kAhead) fetch_x(xa[0], 0);
        if constexpr (EPI == 0) gate_own = a.gate ? a.gate[tok_own] : 1.0f;
        const int own = min(row, a.rows - 1);
        if constexpr (ASYM) scale_own = M.minmax_bf16 ? ((gp_u32)M.minmax_bf16)[own] : 0u;  // (no pair array: zeros)
        else scale_own = ((gp_u16)M.scale_f16)[own];
    });

    f32x4 acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; mb++)
#pragma unroll
        for (int nb = 0; nb < 4; nb++) acc[mb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // asymmetric grid, tiles of up to 32 tokens: a sum for each sign, the grid points are applied when a row is written; larger ones (no registers for
    // that): the grid points of the four rows whose weights this lane feeds to the matrix cores
    constexpr bool kTwoSums = ASYM && MB <= 2;
    f32x4 acc_neg[kTwoSums ? MB : 1][4];
    if constexpr (kTwoSums) {
#pragma unroll
        for (int mb = 0; mb < MB; mb++)
#pragma unroll
            for (int nb = 0; nb < 4; nb++) acc_neg[mb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    uint32_t g_hi[4] = {0u, 0u, 0u, 0u}, g_lo[4] = {0u, 0u, 0u, 0u};
    if constexpr (ASYM && !kTwoSums) {
#pragma unroll
        for (int nb = 0; nb < 4; nb++) {
            const uint32_t pair = (uint32_t)__shfl((int)scale_own, 16 * nb + l16, 64);
            g_hi[nb] = pair << 16;
            g_lo[nb] = pair & 0xFFFF0000u;
        }
    }
    // operand reads: row l16 of a block of 16, word lg (+ 4 for the upper half) of the step's eight
    const uint32_t wfrag = rings + 1024u * (uint32_t)(l16 >> 3) + 4u * (uint32_t)(l16 & 7);
    uint32_t word = 32u * (uint32_t)lg + ring_begin((uint32_t)l16), first = ring_begin((uint32_t)lane) + 2u;
    const int nsteps = (a.cols + kMmKc - 1) / kMmKc;

    RingPiece piece[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
        piece[k].v = u32x4{0u, 0u, 0u, 0u};
        piece[k].at = kMmNoPiece;
    }
    RingGroup group = ring_look_up(tab, ring_codes_at(dec, dec.ci));
    auto step = [&](auto parity, int c) {
        constexpr int P = decltype(parity)::value, X = P & kAhead;
        const int kc = c * kMmKc;
        // ---- decode until every lane has passed column kc + 64
        fetch_x(xa[kAhead ? 1 - P : 0], kc + kAhead * kMmKc);
        ring_decode_step(dec, tab, first, M.codes, piece[P], piece[1 - P], group);
        first += 4u * kMmKc;
        // the rows this wavefront multiplies are the ones its own lanes wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // The step's weights are taken out of the rings, which leaves zeros for the columns that come there next.
        uint32_t wd[2][4];
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            const uint32_t at = ((word + 128u * (uint32_t)ks) & kMmWord) | wfrag;
#pragma unroll
            for (int nb = 0; nb < 4; nb++)
                wd[ks][nb] = __hip_atomic_exchange((lw_u32)(uintptr_t)(at + (uint32_t)(nb * 16 * kMmRowBytes)), 0u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        word += 4u * kMmKc;
        // the next step's first groups, under this step's multiply
        ring_arrive(dec, piece[1 - P]);
        const unsigned long long four = ring_codes_at(dec, dec.ci);
        __builtin_amdgcn_sched_barrier(0);

        if (kc + kMmKc > a.cols) {
            asm volatile("");  // (a branch, not selects in every step)
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int ks = 0; ks < 2; ks++) xa[X][mb][ks] = x_col && kc + 32 * ks <= x_last ? xa[X][mb][ks] : u32x4{0u, 0u, 0u, 0u};
            if constexpr (ASYM && !kTwoSums) {  // (a grid point may be infinite)
#pragma unroll
                for (int ks = 0; ks < 2; ks++)
#pragma unroll
                    for (int nb = 0; nb < 4; nb++) wd[ks][nb] = x_col && kc + 32 * ks <= x_last ? wd[ks][nb] : 0u;
            }
        }

        // ---- multiply step c
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            bf16x8 bw[4], ax[MB];
#pragma unroll
            for (int nb = 0; nb < 4; nb++) {
                if constexpr (ASYM && !kTwoSums)
                    bw[nb] = mm_expand_minmax(wd[ks][nb], g_hi[nb], g_lo[nb]);
                else
                    bw[nb] = mm_expand(kTwoSums ? wd[ks][nb] & ~(wd[ks][nb] >> 1) & 0x44444444u : wd[ks][nb]);
            }
#pragma unroll
            for (int mb = 0; mb < MB; mb++) __builtin_memcpy(&ax[mb], &xa[X][mb][ks], 16);
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int nb = 0; nb < 4; nb++)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[nb], ax[mb], acc[mb][nb], 0, 0, 0);
            if constexpr (kTwoSums) {
#pragma unroll
                for (int nb = 0; nb < 4; nb++) bw[nb] = mm_expand(wd[ks][nb] & (wd[ks][nb] >> 1) & 0x44444444u);
#pragma unroll
                for (int mb = 0; mb < MB; mb++)
#pragma unroll
                    for (int nb = 0; nb < 4; nb++)
                        acc_neg[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[nb], ax[mb], acc_neg[mb][nb], 0, 0, 0);
            }
            if (ks == 0) {
                group = ring_look_up(tab, four);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // (two steps a turn, so that what is in flight keeps its registers; an odd number of steps ends with one that has no columns)
    int c = 0;
    do {
        step(std::integral_constant<int, 0>{}, c);
        step(std::integral_constant<int, 1>{}, c + 1);
        c += 2;
    } while (c < nsteps);

    // accumulator v of lane l: row 16 * nb + 4 * (l / 16) + v of the wavefront's 64, token 16 * mb + l % 16
    typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
    typedef u32x4 u32x4_word __attribute__((aligned(4)));
    typedef __attribute__((address_space(1))) float *gw_f32;
    typedef __attribute__((address_space(1))) uint16_t *gw_u16;
    float scale[4][4], scale_neg[kTwoSums ? 4 : 1][4];
#pragma unroll
    for (int nb = 0; nb < 4; nb++) {
#pragma unroll
        for (int v = 0; v < 4; v++) {
            // the weights were +-2, or the grid points themselves
            uint32_t raw = 0u;
            if constexpr (kTwoSums || !ASYM) raw = (uint32_t)__shfl((int)scale_own, 16 * nb + 4 * lg + v, 64);
            if constexpr (kTwoSums) {
                scale[nb][v] = 0.5f * __uint_as_float(raw & 0xFFFF0000u);  // w_max
                scale_neg[nb][v] = 0.5f * __uint_as_float(raw << 16);      // w_min
            } else if constexpr (!ASYM) {
                scale[nb][v] = 0.5f * half_bits_to_float((uint16_t)raw);
            } else {
                scale[nb][v] = 1.0f;
            }
        }
    }
#pragma unroll
    for (int mb = 0; mb < MB; mb++) {
        const int t = 16 * mb + l16;
        // where the lane's row r0 + 4 * lg goes (second product: in the output row of the lane's token, scaled by its gate), and how far
        // on the rows of the next 16 go
        uintptr_t to;
        uint32_t next = EPI == 0 ? 64u : 32u;
        float gate = 1.0f;
        if constexpr (EPI == 0) {
            const int tok = __shfl(tok_own, t, 64);
            gate = __shfl(gate_own, t, 64);
            to = reinterpret_cast<uintptr_t>(a.out) + 4 * ((size_t)tok * a.ld_out + (size_t)(r0 + 4 * lg));
        } else if (a.out_tiled) {
            const int tb = min(16, ntok - 16 * mb);
            to = reinterpret_cast<uintptr_t>(a.out) +
                 2 * ((size_t)(slot0 + 16 * mb) * a.ld_out + (size_t)(((r0 >> 3) + (lg >> 1)) * tb + l16) * 8 + (size_t)(4 * (lg & 1)));
            next = 32u * (uint32_t)tb;
        } else {
            to = reinterpret_cast<uintptr_t>(a.out) + 2 * ((size_t)(slot0 + t) * a.ld_out + (size_t)(r0 + 4 * lg));
        }
        if (t < ntok) {
#pragma unroll
            for (int nb = 0; nb < 4; nb++) {
                const int r = r0 + 16 * nb + 4 * lg;
                float val[4];
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    if constexpr (kTwoSums) {
                        // A grid point meets the sum of its own sign only, whose rounding it scales, and none at all where that is
                        // zero: one that the row does not use may be large or infinite.  The two often nearly cancel: the rounding of the
                        // first product is added back.
                        // (A signed sum and one under |weight|, their sum and difference taken here, save 24 instructions a step:
                        // 884 us instead of 964 for 256 experts of 2080 x 6144 with 16 tokens each, 962 / 1010 with 1-32, 217 / 217 for 4001
                        // tokens on 128 of 768 x 3072.  But each grid point then scales the rounding of both signs' sum: rows with two
                        // weights of one sign whose grid point is 100 / 2^14 times the other's were off by up to 9e-6 / 1.5e-3 of
                        // sum |w x|, 1.8e-7 this way.  A grid point picked per weight, as in larger tiles: 975, 998, 217 us, 6e-7.)
                        const float pos = acc[mb][nb][v], neg = acc_neg[mb][nb][v], s_pos = pos != 0.0f ? scale[nb][v] : 0.0f;
                        const float of_pos = pos * s_pos, rest = fmaf(pos, s_pos, -of_pos);
                        const float sum = neg != 0.0f ? fmaf(neg, scale_neg[nb][v], of_pos) : of_pos;
                        val[v] = fabsf(sum) < INFINITY ? sum + rest : sum;
                    } else {
                        val[v] = acc[mb][nb][v] * scale[nb][v];
                    }
                    if constexpr (EPI == 0) val[v] *= gate;
                    else val[v] = val[v] > 0.0f ? val[v] : 0.0f;
                }
                const uintptr_t at = to + (uintptr_t)((uint32_t)nb * next);
                if constexpr (EPI == 0) {
                    if (r + 4 <= a.rows) {
                        *(__attribute__((address_space(1))) u32x4_word *)at =
                            u32x4{__float_as_uint(val[0]), __float_as_uint(val[1]), __float_as_uint(val[2]), __float_as_uint(val[3])};
                    } else {
#pragma unroll
                        for (int v = 0; v < 3; v++)
                            if (r + v < a.rows) ((gw_f32)at)[v] = val[v];
                    }
                } else {
                    uint32_t h[4];
#pragma unroll
                    for (int v = 0; v < 4; v++) h[v] = float_to_bf16_bits(val[v]);
                    if (r + 4 <= a.rows) {
                        *(__attribute__((address_space(1))) u32x2_any *)at = u32x2_any{h[0] | h[1] << 16, h[2] | h[3] << 16};
                    } else {
#pragma unroll
                        for (int v = 0; v < 3; v++)
                            if (r + v < a.rows) ((gw_u16)at)[v] = (uint16_t)h[v];
                    }
                }
            }
        }
    }
    // (An activation that is not finite makes every row's sum so, one without weights too: one row's tells.  Behind the stores: ahead of them,
    // and the stores left out for such tokens, the compiler's order of the rows' ends cost the second product 346 -> 365 us.)
    unsigned long long again = 0;
#pragma unroll
    for (int mb = 0; mb < MB; mb++) again |= (__ballot(acc[mb][0][0] * 0.0f != 0.0f) & 0xFFFFull) << (16 * mb);
    again &= ~0ull >> (64 - ntok);
    return again;
}

// The given tokens of a unit without the matrix cores, which multiply weights of zero too: an activation that is infinite or no number would
// make NaN of its token's results in every row, and of the hidden vector zeros (the ReLU), where only rows with a weight there have a
// part in it.  One lane = one row, four tokens at a time, straight from the stream; four trips to memory a codeword bound it.  256 experts
// of 2080 x 6144 with 1-32 tokens each, a first call, us: 958 with finite activations, 1625 with one that is not, 14900 with none that is.
template <int EPI, int ASYM>
__device__ __forceinline__ void mm_again(const ProductArgs &a, const qmoe_matrix &M, int rblk, int slot0, int ntok, unsigned long long tokens)
{
    const int row = rblk * 64 + ((int)threadIdx.x & 63);
    const bool row_live = row < a.rows;
    const RowStream rst = row_stream(M, row, row_live);
    const uint32_t left = min(rst.left, (uint32_t)a.cols);  // (no codeword stands for fewer than two columns)
    float scale = 0.0f, w_neg = -1.0f, w_pos = 1.0f;
    if (row_live) {
        if constexpr (ASYM) {
            const uint32_t pair = M.minmax_bf16 ? ((gp_u32)M.minmax_bf16)[row] : 0u;
            w_neg = __uint_as_float(pair << 16);
            w_pos = __uint_as_float(pair & 0xFFFF0000u);
            scale = 1.0f;
        } else {
            scale = half_bits_to_float(((gp_u16)M.scale_f16)[row]);
        }
    }
    while (tokens) {
        constexpr int kAtOnce = 4;
        int slot[kAtOnce], tok[kAtOnce], n = 0;
        uintptr_t x[kAtOnce];
        uint32_t next8[kAtOnce];  // bytes from one column to the one eight columns on
        float sum[kAtOnce];
#pragma unroll
        for (int k = 0; k < kAtOnce; k++) {
            const int t = __builtin_ctzll(tokens ? tokens : 1ull << (slot[0] - slot0));  // (none left: the first again)
            n += tokens != 0;
            tokens &= tokens - (tokens != 0);
            slot[k] = slot0 + t;
            tok[k] = a.perm ? a.perm[slot[k]] : slot[k];
            if (a.x_tiled) {  // (see mm_item)
                const int b = t & ~15;
                x[k] = reinterpret_cast<uintptr_t>(a.x) + 2 * ((size_t)(slot0 + b) * a.ldx + (size_t)(8 * (t & 15)));
                next8[k] = 16u * (uint32_t)min(16, ntok - b);
            } else {
                x[k] = reinterpret_cast<uintptr_t>(a.x) + 2 * ((size_t)(a.x_by_slot ? slot[k] : tok[k]) * a.ldx);
                next8[k] = 16u;
            }
            sum[k] = 0.0f;
        }
        uint32_t col = 0;
        for (uint32_t i = 0; i < left && col < (uint32_t)a.cols; i++) {
            const uint32_t at = rst.sub + i, code = ((gp_u16)min(rst.pp + rst.pstride * (uintptr_t)(at >> 3), rst.last))[at & 7u];
            const uint32_t groups3 = 3u * (uint32_t)a.n_groups, single = code > groups3 ? code - groups3 : 0u;
            const uint32_t e = *(lp_u32)(uintptr_t)(4u * min(max(code >> 2, single), (uint32_t)(a.n_order - 1)));
            const uint32_t weights = (e & kMmWeights) ^ (((code & 0xFFu) * kMmFlipMul) & kMmFlips), places = e & kMmPlaces;
#pragma unroll
            for (int z = 0; z < 3; z++) {
                const uint32_t w = byte_of(weights, z), c = col + (byte_of(places, z) >> 2);
                if ((w & 1u) && c < (uint32_t)a.cols) {
                    const float g = w & 2u ? w_neg : w_pos;
#pragma unroll
                    for (int k = 0; k < kAtOnce; k++)
                        sum[k] = fmaf(g, __uint_as_float((uint32_t)*(gp_u16)(x[k] + (uintptr_t)((c >> 3) * next8[k] + 2u * (c & 7u))) << 16), sum[k]);
                }
            }
            col += places >> 26;
        }
        if (!row_live) continue;
#pragma unroll
        for (int k = 0; k < kAtOnce; k++) {
            if (k >= n) break;
            float val = sum[k] * scale;
            if constexpr (EPI == 0) {
                if (a.gate) val *= a.gate[tok[k]];
                reinterpret_cast<float *>(a.out)[(size_t)tok[k] * a.ld_out + row] = val;
            } else {
                size_t to = (size_t)slot[k] * a.ld_out + row;
                if (a.out_tiled) {
                    const int b = (slot[k] - slot0) & ~15, j = (slot[k] - slot0) & 15;
                    to = (size_t)(slot0 + b) * a.ld_out + ((size_t)(row >> 3) * min(16, ntok - b) + j) * 8 + (row & 7);
                }
                reinterpret_cast<uint16_t *>(a.out)[to] = float_to_bf16_bits(val > 0.0f ? val : 0.0f);
            }
        }
    }
}

// A ticket of the device counter for a wavefront, out of the `some` that its workgroup has drawn last.  pool: lock, next ticket, end of the
// drawn ones (in LDS, zeros at first).  Nobody draws again when the counter has given all `n` tickets.
__device__ __forceinline__ int pool_draw(int *pool, int *counter, int some, int n)
{
    int got = 0;
    if ((threadIdx.x & 63) == 0) {
        while (__hip_atomic_exchange(pool, 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) __builtin_amdgcn_s_sleep(1);
        got = pool[1];
        if (got >= pool[2] && got < n) {
            got = atomicAdd(counter, some);
            pool[2] = got + some;
        }
        pool[1] = got + 1;
        __hip_atomic_store(pool, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return min(__builtin_amdgcn_readfirstlane(got), n);
}

template <int EPI, int ASYM>
__global__ __launch_bounds__(kMmThreads) void k_product_mm(const ProductArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const size_t table_bytes = mm_table_bytes(a.n_order);
    uint32_t *table_w = reinterpret_cast<uint32_t *>(smem);
    unsigned char *wt = smem + table_bytes;                           // [512][kMmRowBytes] rings
    unsigned char *win = wt + (size_t)kMmThreads * kMmRowBytes;       // codeword windows: [wavefront][group][lane][4]

    // A unit of work is 64 rows of one (expert, token tile) item, and a wavefront takes it alone: once
    // the table is staged the wavefronts of a workgroup share the table and how they come by their units, and meet at no barrier (but
    // in step), so one wavefront's set-up (a chain of trips to memory) runs under the others' arithmetic, a matrix
    // whose rows are no multiple of 512 leaves no wavefront idle, and the units are small enough to
    // pack well.  A layer call brings a list of items, some or all of whose units are dealt out in advance, and a device counter for the rest, which a
    // workgroup's wavefronts draw from through a lock and a small stock in LDS (pool_draw), or, in step, eight at a time; where two rounds are dealt
    // out, they count in LDS what is taken of their workgroup's share.  All of that is below.  The single-matrix call
    // has neither list nor counter: its items are the tiles of 64 consecutive tokens of `single`, its units dealt out round robin.
    const bool listed = a.items != nullptr;
    if constexpr (EPI == 0) {  // (ahead of the return: all workgroups)
        if (a.clear_idx && *a.clear_count > 0) {
            for (int t = ((int)blockIdx.x * kMmThreads + (int)threadIdx.x) >> 6; t < a.n_tokens; t += (int)gridDim.x * (kMmThreads / 64)) {
                const int e = a.clear_idx[t];
                if (e >= 0 && e < a.n_experts) continue;
                for (int c = (int)threadIdx.x & 63; c < a.rows; c += 64) ((float *)a.out)[(size_t)t * a.ld_out + c] = 0.0f;
            }
        }
    }
    const int n_items = listed ? min(*a.n_items_dev, a.max_items) : (a.batch + kMmTokens - 1) / kMmTokens;
    const int total = (int)min((long long)n_items * a.mm_row_blocks, 0x7FFFFFFFLL);
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, waves = kMmThreads / 64;
    const int all_waves = (int)gridDim.x * waves;
    // No more workgroups than fill all their wavefronts stay (a workgroup holds its compute unit's LDS whole,
    // so one that runs half empty keeps the other kernels of a layer call off that compute unit); the
    // single-matrix call, which is after latency, spreads its units over as many compute units as it can, and so does a layer call
    // whose few-token kernels run before or after these or need little (kMmSpread): 64 experts of 768 x 3072 with 16 tokens each, second
    // product, 768 units on 96 compute units 51, on all of them 34 us.
    // `late`: the few-token chain beside this one holds whole compute units (k_product's workgroups stay for the launch) and has items.  Workgroups of
    // this kernel start late there, and those that run have to be able to take any unit: tickets for all but the whole rounds among the first seven
    // eighths, no more workgroups than needed, wavefronts in step also where one round does.  Units dealt out and spread / this, us: 427 experts of
    // 1688 x 4664, 1803 tokens, Zipf, asymmetric grid 626 / 583; 336 of 1320 x 3400, 1573, the same 366 / 329; 200 of 256 x 1000, 4000, Zipf 147 / 128; without few-token
    // items, 17 of 160 x 1456, 2864 tokens, uniform, asymmetric 77 / 98.  The kernel with several lanes per row is beside it for less of the time: 285 of 768 x 4576,
    // 1923 tokens, Zipf 233 / 253.
    const int few = a.mm_spread & kMmBeside ? a.n_items_dev[kCounterFew - kCounterMm] : 0;  // items of that chain
    const bool late = (a.mm_spread & kMmBesideHolds) && few > 0;
    const bool spread = listed && (a.mm_spread & kMmSpread) && !late && total < all_waves;
    const int wgs = listed && !spread ? (total + waves - 1) / waves : min(total, (int)gridDim.x);
    if ((int)blockIdx.x >= wgs) return;
    int *next_base = reinterpret_cast<int *>(win + (size_t)kMmThreads * kMmWindowBytes);  // [1], in-step hand-out only
    int *tok_sums = next_base + 1;                                                      // [2]
    int *pool = next_base + 3;                                                          // [3], see pool_draw
    int *taken = pool + 3;                                                              // [1] units of the workgroup's share that are taken
    if (threadIdx.x < 6) tok_sums[threadIdx.x] = 0;
    stage_words(table_w, a.order_table, a.n_order, ring_entry_bytes);
    __syncthreads();
    // In step or each wavefront for itself (see the loop)?  In step when most of the tokens sit in tiles of
    // more than 32: those read 4-8 KB of activations per wavefront and step.
    bool in_step = false;
    if (listed && a.mm_in_step && (late || total > all_waves)) {
        int big = 0, all = 0;
        for (int i = threadIdx.x; i < n_items; i += kMmThreads) {
            const int n = max(0, min(a.items[i].ntok, kMmTokens));
            all += n;
            big += n > 32 ? n : 0;
        }
        if (all) {
            atomicAdd(&tok_sums[0], all);
            atomicAdd(&tok_sums[1], big);
        }
        __syncthreads();
        in_step = 2 * tok_sums[1] > tok_sums[0];
    }

    const uint32_t wt_addr = (uint32_t)(uintptr_t)(lw_u8)wt, win_addr = (uint32_t)(uintptr_t)(lw_u8)win;
    // Which units: in a layer call of more than two rounds the first one of every wavefront and seven eighths of all are dealt out, consecutive ones (of the
    // same tile, as a rule) to a workgroup; the others are drawn from the device counter, `some` at a time for the whole workgroup.
    // The counter gives a ticket in 13 ns, whoever asks, those that find nothing left too: 2048 wavefronts whose units take 12 to 16 steps
    // wait for it, and a call of one round took 27 us for its tickets and as much again for the empty ones.  Tickets for all units but the whole
    // rounds among the first seven eighths / this, first and second product, us: 170 experts of 768 x 3072 with 16 tokens each 88.7 and
    // 76.9 / 66.4 and 44.4, 128 of 1024 x 4096 with 8 97.6 and 84.0 / 76.0 and 52.9, 63 of 2080 x 6144 with 1-32 100 and 116 / 95.7
    // and 96.9, 252 of them with 16 378 and 361 / 380 and 362.  Long units are drawn one at a time, since the end waits for the longest: 252 of 2080 x 6144 with
    // 1-32 tokens, second product, 357 by eights, 310 one by one.  More dealt out: fifteen sixteenths 378.
    // Between an eighth more than one round and two rounds all are dealt out, in fours over the workgroups, whose wavefronts take them as they come free: the
    // tickets of such a second round, one each or several at a time, cost more than they even out.  Layers of two products, tickets / this, us: 173 experts
    // of 736 x 1056, 1301 tokens 85 / 73; 122 of 1600 x 2576, 3441 tokens 193 / 181; 18 of 1920 x 2496, 3996 tokens, Zipf, asymmetric grid 189 / 173;
    // 128 of 768 x 3072 with 100 tokens each 241 / 232; of 44 layers of all shapes 1.02 on average, 1.18 and 0.98 at the ends.  A few units more than one round
    // are better drawn: 30 of 1896 x 2320, 2687 tokens, Zipf 153 / 158.  (One by one over the workgroups: 128 of 768 x 3072 with 100 257.  More
    // rounds this way, and tickets for the last eighth: 170 of 768 x 3072 with 16 141 / 150.)  Not beside a longer chain, where workgroups start
    // late and the others have to be able to take their units: kMmSpread is not set, or the few-token kernel has more than half an item for every tile
    // (309 of 1776 x 2696, 3022 tokens, Zipf 326 / 312; with fewer, 216 of 1248 x 4352, 1335 tokens, uniform, asymmetric 323 / 331).  Nor where the fours leave
    // wavefronts without a unit for longer than the tickets cost, some 28 steps: 82 of 1808 x 6192, 3361 tokens, Zipf, asymmetric, 0.43 of a round of 97 steps
    // 524 / 479; 65 of 2000 x 4912, 3986, Zipf, 80 % zeros, 0.38 of 77 404 / 389; not so 98 of 1792 x 3696, 2110, Zipf, 0.44 of 58 227 / 239.
    // The single-matrix call deals all of them out, round robin over the workgroups first, then over their wavefronts: few units spread
    // over many compute units.
    const int grid = (int)gridDim.x, wg = (int)blockIdx.x;
    bool evenly = listed && (a.mm_spread & kMmSpread) && !late && 2 * few <= n_items && !in_step && total >= all_waves + all_waves / 8 && total <= 2 * all_waves;
    if (evenly) {
        const int places = 2 * total <= 3 * all_waves ? all_waves + all_waves / 2 : 2 * all_waves;  // (three or four fours a workgroup)
        evenly = (places - total) * (a.cols / kMmKc) <= 28 * all_waves;
    }
    int dealt = total;
    if (late || (listed && total > all_waves)) {
        dealt = late ? 0 : all_waves;
        if (!in_step && !evenly) dealt = max((total - total / 8) / all_waves * all_waves, dealt);
    }
    const int some = max(min((total - dealt) / (2 * grid), min(96 * kMmKc / a.cols, waves)), 1);
    int g = wave * grid + wg;
    if (listed) g = wg * waves + wave;
    auto in_fours = [&](int j) { return ((j >> 2) * grid + wg) * 4 + (j & 3); };  // unit j of the workgroup
    if (evenly) g = in_fours(wave);
    if (spread) {
        // Neighbours (of one tile, as a rule) go to different workgroups, so that those with tiles of many tokens share a compute unit with others: two by two,
        // since they read the same activations, where that makes no workgroup's share larger.  Layers, us, neighbours together / this: 65 experts of
        // 920 x 1336, 1735 tokens, Zipf 75.5 / 70.5; 62 of 1128 x 6120, 1572 tokens 190 / 178; 32 of 768 x 3072, 1200 tokens, Zipf 88.5 / 85.5.  (One by one always:
        // 128 of 768 x 3072 with 64 tokens each 146 / 154.)
        const int most = (total + wgs - 1) / wgs, twos = (total + 2 * wgs - 1) / (2 * wgs);
        g = 2 * twos == most ? ((wave >> 1) * wgs + wg) * 2 + (wave & 1) : wave * wgs + wg;
    }
    for (bool first = g < dealt;; first = false) {
        if (!first) {
            if (in_step) {
                // The wavefronts of a workgroup take eight consecutive units together and start them together:
                // where the activations are not stored by token blocks (the first product of a layer) their
                // operand loads touch a line per token, and eight wavefronts that ask for the same lines at the
                // same time are served by one fetch.  (Measured both ways: a layer with few, crowded experts is
                // 3 % faster in step, one with many experts of 8-32 tokens 7 % faster without.)
                __syncthreads();
                if (threadIdx.x == 0) *next_base = dealt + atomicAdd(a.work_counter, waves);
                __syncthreads();
                if (*next_base >= total) break;
                g = *next_base + wave;
                if (g >= total) continue;
            } else {
                g += g < dealt ? all_waves : 0;
                if (evenly) {
                    int j = 0;
                    if (lane == 0) j = atomicAdd(taken, 1);
                    g = in_fours(waves + __builtin_amdgcn_readfirstlane(j));
                } else if (g >= dealt) {
                    if (dealt >= total) break;
                    g = dealt + pool_draw(pool, a.work_counter, some, total - dealt);
                }
            }
        }
        if (g >= total) break;
        const int idx = g / a.mm_row_blocks;
        const int rblk = g - idx * a.mm_row_blocks;
        Item it;
        if (listed) {
            // (scalar loads: nothing writes the list during the launch)
            typedef const __attribute__((address_space(4))) Item *cp_item;
            cp_item p = (cp_item)(uintptr_t)(a.items + idx);
            it.expert = p->expert;
            it.slot0 = p->slot0;
            it.ntok = p->ntok;
        } else {
            it.expert = 0;
            it.slot0 = idx * kMmTokens;
            it.ntok = a.batch - idx * kMmTokens;
        }
        const int expert = it.expert, slot0 = it.slot0;
        const int ntok = min(it.ntok, kMmTokens);
        if (expert < 0 || expert >= a.n_experts || ntok < 1) continue;
        const qmoe_matrix M = matrix_of(a, expert);
        unsigned long long again;
        if (ntok <= 16)
            again = mm_item<1, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
        else if (ntok <= 32)
            again = mm_item<2, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
        else
            again = mm_item<4, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
        if (again) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (other lanes write the same places again)
            mm_again<EPI, ASYM>(a, M, rblk, slot0, ntok, again);
        }
    }
}

}  // namespace

size_t mm_lds_bytes(int n_order)
{
    return mm_table_bytes(n_order) + (size_t)kMmThreads * (kMmRowBytes + kMmWindowBytes) + 32;
}

qmoe_status launch_product_mm(ProductArgs a, const MmPlan &mp, hipStream_t s)
{
    a.mm_row_blocks = (a.rows + 63) / 64;  // units of 64 rows, one wavefront each
    auto launch = [&](auto kernel) -> qmoe_status {
        const qmoe_status st = allow_lds(kernel, mp.smem, true);
        if (st != QMOE_OK) return st;
        hipLaunchKernelGGL(kernel, dim3(mp.grid), dim3(kMmThreads), mp.smem, s, a);
        return QMOE_OK;
    };
    qmoe_status st;
    if (a.minmax)
        st = a.epilogue ? launch(k_product_mm<1, 1>) : launch(k_product_mm<0, 1>);
    else
        st = a.epilogue ? launch(k_product_mm<1, 0>) : launch(k_product_mm<0, 0>);
    if (st != QMOE_OK) return st;
    QMOE_HIP_TRY(hipGetLastError());
    return QMOE_OK;
}

}  // namespace qmoe
