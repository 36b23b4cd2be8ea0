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
// the columns 64 at a time.  Every lane keeps a ring of 128 one-byte columns of its
// row in LDS and decodes its codewords into it sequentially, as far ahead as the
// ring allows (so the lanes of a wavefront, whose codewords end at different
// columns, seldom wait for each other); then the wavefront multiplies the 64
// columns that are complete, for the 64 rows its lanes decoded, with the tokens'
// activations on the matrix cores, fp32 accumulators in registers.  The
// ring holds the weights as the high byte of bf16 +-2.0 (0x40 / 0xC0, low byte
// zero), expanded to bf16 by a byte permute when a fragment is read; the factor 2
// is taken out again, exactly, when a row is written.
// Only device-order streams (whole table in LDS) take this path.
//
// What bounds it: nothing alone.  Of a wavefront's step 48 % goes by in the decoder's rounds (about 4.5 of them, 270 cycles
// each, with 24 vector instructions and about 35 cycles of the LDS that eight wavefronts share), 30 % in the multiply (a quarter of
// that waiting for activations), the rest at the window, the set-up and the results (rows of 2080 and 6144 columns, sparsities mixed); the
// LDS holds two wavefronts per SIMD (ring, window and table), too few to hide each other's waits altogether.  A step's activations are loaded
// straight into the registers the product reads, a codeword piece only by the lanes that need one (asking again for what is there
// costs a line per lane).  (Activations asked for a step ahead: 1164 us instead of 1000 where the wait for the window's piece then
// waits for them too, 1013 where it is moved behind the multiply.)
// (Slower, measured: two lanes per row with rings of 256 columns, two codewords a round, a ring stored by columns and read
// transposed, codewords four by four in the window.)

constexpr int kMmKc = 64;                      // columns per step
constexpr int kMmRing = 2 * kMmKc;             // columns a lane's ring holds
constexpr int kMmAhead = kMmRing - 28 - 1;     // a codeword may start this far past the step's first column (its run then ends
                                               // below column kc + 128, the first one that shares a ring byte with the step)
constexpr int kMmWRowBytes = kMmRing + 16;     // 36 banks per row: 16 consecutive rows read 16 bytes each (two lanes, 8 bytes apiece) without conflict

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// eight ring bytes (high bytes of bf16) -> eight bf16
__device__ __forceinline__ bf16x8 mm_expand(uint32_t d0, uint32_t d1)
{
    u32x4 o;
    o.x = __builtin_amdgcn_perm(0u, d0, 0x010c000cu);
    o.y = __builtin_amdgcn_perm(0u, d0, 0x030c020cu);
    o.z = __builtin_amdgcn_perm(0u, d1, 0x010c000cu);
    o.w = __builtin_amdgcn_perm(0u, d1, 0x030c020cu);
    bf16x8 r;
    __builtin_memcpy(&r, &o, 16);
    return r;
}

__device__ __forceinline__ bf16x8 mm_expand_minmax(uint32_t d0, uint32_t d1, uint32_t hi, uint32_t lo)
{
    const u32x4 o = select_minmax(d0, d1, hi, lo);
    bf16x8 r;
    __builtin_memcpy(&r, &o, 16);
    return r;
}

using lw_u8 = __attribute__((address_space(3))) unsigned char *;
using lw_u64 = __attribute__((address_space(3))) unsigned long long *;
using lw_u32x4 = __attribute__((address_space(3))) u32x4 *;
using lp_u64 = const __attribute__((address_space(3))) unsigned long long *;
using lp_u32x4 = const __attribute__((address_space(3))) u32x4 *;
using lp_i32 = const __attribute__((address_space(3))) int *;
using lp_f32 = const __attribute__((address_space(3))) float *;

// ---- the ring decoder ----
//
// One lane = one row.  A lane's codewords pass through a window of two 16-byte pieces (sixteen
// codewords) in LDS, the next piece is in flight in a register; the codeword two places ahead
// is read from the window and the table entry one place ahead is looked up while the current
// entry is applied.  Applying an entry is three one-byte stores into the lane's ring of 128
// columns: field z goes to ring column (column + position) mod 128 with the value bits of the
// field shifted to the top of the byte (0x40: +2.0, 0xC0: -2.0 as the high byte of bf16) or, for
// the asymmetric grid, as they are (byte selectors 2 / 6); an unused field (0) comes first and
// writes its zero at the run's first column before any real weight of the same run.
//
// (A struct of plain scalars and free functions that are always inlined: the state stays in
// registers.)
constexpr uint32_t kMmWinAhead = 2 * 15;  // the window holds 16 codewords (32 bytes), and a round reads two ahead of the one it applies
constexpr int kMmWinBytes = 32;   // a lane's window: two 16-byte pieces, on 32 bytes

// The table comes first in the LDS, at address 0 (launch_product_mm sees to that), and what follows it begins on 32 bytes: a window's
// address takes the place in it by an OR.
static_assert(kMmWinBytes == 32 && kMmThreads * kMmWRowBytes % kMmWinBytes == 0, "windows on their own size: ring_rounds and ring_code_at keep bits 1..4");
static_assert(kMmRing == 1 << 7, "ring_rounds takes seven bits of a column");
__host__ __device__ inline size_t mm_table_bytes(int n_order) { return ((size_t)n_order * 4 + 31) & ~(size_t)31; }

struct RingDecoder {
    // (bytes into the lane's codewords, counted from its first piece)
    uint32_t ci;                // one past the next codeword
    uint32_t end;               // one past the row's last codeword's end
    uint32_t lim;               // the lane may go on while ci < lim: codewords are left, and the window reaches one past them
    uint32_t wbase;             // first codeword of the window's first piece (a multiple of 16)
    uint32_t pos8;              // 8 * (column where the next run starts)
    uint32_t ent, flips, code;  // the pipeline: entry of the next codeword as read, the sign flips of its code, code of the one after
    uintptr_t pp, last, pstr;   // first piece of the window, the lane's last piece, bytes from a piece to the next
    u32x4 fut;                  // the piece after the window, in flight
    uint32_t wrow, slot;        // LDS byte addresses of the lane's ring and window
};

__device__ __forceinline__ u32x4 ring_piece_at(const RingDecoder &d, uintptr_t at)
{
    // pieces past the lane's last one re-read the last (never used: `end` comes first)
    return *(gp_u32x4)(at < d.last ? at : d.last);
}

__device__ __forceinline__ void ring_store_piece(const RingDecoder &d, uint32_t half_bytes, const u32x4 &v)
{
    lw_u64 w = (lw_u64)(uintptr_t)(d.slot + half_bytes);
    w[0] = (unsigned long long)v.x | ((unsigned long long)v.y << 32);
    w[1] = (unsigned long long)v.z | ((unsigned long long)v.w << 32);
}

__device__ __forceinline__ uint32_t ring_code_at(const RingDecoder &d, uint32_t at)
{
    return (uint32_t)(*(lp_u16)(uintptr_t)(d.slot + (at & 30u)));
}

// LDS byte offset of a code's table entry: the index that order_entry2 takes, times four.  (Signed, so that the second candidate
// needs no saturation: below the crossing it is the smaller one, and the median with the last entry is then the first.)
__device__ __forceinline__ uint32_t ring_entry_at(uint32_t code, int minus_groups12, int last4)
{
    int at;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(at) : "v"(code & ~3u), "v"((int)(code << 2) + minus_groups12), "s"(last4));
    return (uint32_t)at;
}

// The table in LDS has its entries' bytes in another order than the one in memory: field 1, field 0, field 2, length.  What the two
// low bits of a code flip, the signs of fields 1 and 2, is then bits 2 and 18, and one product of the code's low byte
// puts both there (its other bits are left to the caller's mask).
__device__ __forceinline__ uint32_t ring_entry_bytes(uint32_t e) { return __builtin_amdgcn_perm(e, e, 0x00030102u); }
constexpr uint32_t kMmFlips = 0x00040004u;

__device__ __forceinline__ uint32_t ring_flips(uint32_t code)
{
    uint32_t f;
    asm("v_mul_u32_u24_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD"
        : "=v"(f) : "v"(code), "s"(0x00020004u));
    return f;
}

// The lane's row (none: an empty stream), its window filled, its ring cleared.
__device__ __forceinline__ void ring_setup(RingDecoder &d, const qmoe_matrix &M, int row, bool row_live, uint32_t wrow,
                                           uint32_t slot)
{
    const RowStream rst = row_stream(M, row, row_live);
    d.end = 2u * (rst.sub + rst.left) + 2u;
    d.lim = min(d.end, kMmWinAhead);
    d.pp = rst.pp;
    d.last = rst.last;
    d.pstr = rst.pstride;
    d.ci = 2u * rst.sub + 2u;
    d.wrow = wrow;
    d.slot = slot;
    {
        const u32x4 p0 = ring_piece_at(d, d.pp), p1 = ring_piece_at(d, d.pp + d.pstr);
        ring_store_piece(d, 0u, p0);
        ring_store_piece(d, 16u, p1);
    }
    d.fut = ring_piece_at(d, d.pp + 2u * d.pstr);
    d.wbase = 0;
    d.pos8 = 0;
#pragma unroll
    for (int i = 0; i < kMmRing / 8; i++) ((lw_u64)(uintptr_t)wrow)[i] = 0ull;
}

// Fill the pipeline.  Nothing is in flight afterwards, so that the wait at the top of a round is
// for the two reads of the round before and not for the three stores issued after them.
__device__ __forceinline__ void ring_prime(RingDecoder &d, int minus_groups12, int last4)
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t c0 = ring_code_at(d, d.ci - 2u);
    d.code = ring_code_at(d, d.ci);
    d.ent = *(lp_u32)(uintptr_t)ring_entry_at(c0, minus_groups12, last4);
    d.flips = ring_flips(c0);
    asm volatile("" : "+v"(d.ent), "+v"(d.code));
}

// Rounds of one codeword per lane, until no lane of the wavefront that may go on (ci < lim) is before column end8 / 8.  A lane
// that sits out -- its codewords in the window used up, or too far ahead (pos8 > lim8) -- does so for the rest of the call.
//
// The pipeline: a round's two reads, the code two codewords ahead and the entry one ahead, go out before its stores and are
// used in the next round, the code first (it makes an address, the entry waits behind it).  The LDS works in order, so that
// lgkmcnt(3) is the wait for them and not for the three stores issued after them.
//
// In assembly because lanes leave by the execution mask, which only shrinks: the compiler's loop either selects old
// or new state for every lane that sat out (four instructions, and the lane's reads and stores are done in vain) or rebuilds the mask by
// scalar instructions and branches.  24 vector instructions, 5 of the LDS and 3 others; 32, 5 and 4 before: 256 experts of 2080 x 6144
// with 1-32 tokens each 1071 -> 1001 us, 128 experts of 768 x 3072 with 31 tokens each 224 -> 219 us.  (The same instructions field
// after field, not side by side: 1016 us.  Fields without a weight kept from storing: 1028 us.)
template <int ASYM>
__device__ __forceinline__ void ring_rounds(RingDecoder &d, int minus_groups12, int last4, uint32_t lim8, uint32_t end8)
{
    uint32_t e, t0, t1, t2, w0, w1, w2;
    unsigned long long all;
#define QMOE_ROUNDS(value) \
    asm volatile("s_mov_b64 %[all], exec\n\t" \
                 "v_cmpx_lt_u32_e32 vcc, %[ci], %[lim]\n\t" \
                 "v_cmpx_ge_u32_e32 vcc, %[lim8], %[pos]\n\t" \
                 "0:\n\t" \
                 "s_waitcnt lgkmcnt(4)\n\t" \
                 "v_and_b32_e32 %[t0], -4, %[code]\n\t" \
                 "v_lshl_add_u32 %[t1], %[code], 2, %[k12]\n\t" \
                 "v_add_u32_e32 %[ci], 2, %[ci]\n\t" \
                 "v_med3_i32 %[t0], %[t0], %[t1], %[last4]\n\t" \
                 "v_and_or_b32 %[t1], %[ci], 30, %[slot]\n\t" \
                 "s_waitcnt lgkmcnt(3)\n\t" \
                 "v_bitop3_b32 %[e], %[flips], %[ent], %[mask] bitop3:0x6c\n\t" \
                 "v_mul_u32_u24_sdwa %[flips], %[code], %[mul] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t" \
                 "ds_read_u16 %[code], %[t1]\n\t" \
                 "ds_read_b32 %[ent], %[t0]\n\t" \
                 "v_add_u32_sdwa %[t0], %[e], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t" \
                 "v_add_u32_sdwa %[t1], %[e], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:DWORD\n\t" \
                 "v_add_u32_sdwa %[t2], %[e], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD\n\t" \
                 "v_add_u32_sdwa %[pos], %[e], %[pos] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t" \
                 "v_bfe_u32 %[w0], %[t0], 3, 7\n\t" \
                 "v_bfe_u32 %[w1], %[t1], 3, 7\n\t" \
                 "v_bfe_u32 %[w2], %[t2], 3, 7\n\t" \
                 value("%[t0]") \
                 value("%[t1]") \
                 value("%[t2]") \
                 "v_add_u32_e32 %[w0], %[w0], %[ring]\n\t" \
                 "v_add_u32_e32 %[w1], %[w1], %[ring]\n\t" \
                 "v_add_u32_e32 %[w2], %[w2], %[ring]\n\t" \
                 "ds_write_b8 %[w0], %[t0]\n\t" \
                 "ds_write_b8 %[w1], %[t1]\n\t" \
                 "ds_write_b8 %[w2], %[t2]\n\t" \
                 "v_cmpx_lt_u32_e32 vcc, %[ci], %[lim]\n\t" \
                 "v_cmpx_ge_u32_e32 vcc, %[lim8], %[pos]\n\t" \
                 "v_cmp_gt_u32_e32 vcc, %[end8], %[pos]\n\t" \
                 "s_cbranch_vccnz 0b\n\t" \
                 "s_waitcnt lgkmcnt(3)\n\t" \
                 "s_mov_b64 exec, %[all]\n\t" \
                 : [ci] "+v"(d.ci), [pos] "+v"(d.pos8), [ent] "+v"(d.ent), [flips] "+v"(d.flips), [code] "+v"(d.code), \
                   [e] "=&v"(e), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [w0] "=&v"(w0), [w1] "=&v"(w1), [w2] "=&v"(w2), \
                   [all] "=&s"(all) \
                 : [lim] "v"(d.lim), [ring] "v"(d.wrow), [slot] "v"(d.slot), [lim8] "s"(lim8), [end8] "s"(end8), \
                   [k12] "s"(minus_groups12), [last4] "s"(last4), [mask] "s"(kMmFlips), [mul] "s"(0x00020004u) \
                 : "vcc", "memory")
#define QMOE_AS_IS(t) "v_and_b32_e32 " t ", 6, " t "\n\t"
#define QMOE_ON_TOP(t) "v_lshlrev_b32_e32 " t ", 5, " t "\n\t"
    if constexpr (ASYM) QMOE_ROUNDS(QMOE_AS_IS);
    else QMOE_ROUNDS(QMOE_ON_TOP);
#undef QMOE_AS_IS
#undef QMOE_ON_TOP
#undef QMOE_ROUNDS
}

// Decode until every lane of the wavefront has passed column kc + 64.  A lane that is there
// already keeps going as long as its next run starts at most kMmAhead columns past kc (its run
// then ends below column kc + 128, the first one that shares a ring byte with the step), so
// the lanes of a wavefront, whose codewords end at different columns, seldom wait for each
// other.  `after_wait` runs once, right after the step's wait for global memory: the place
// to issue loads that are wanted when the step has been decoded.
template <int ASYM, class AfterWait>
__device__ __forceinline__ void ring_decode_step(RingDecoder &d, int minus_groups12, int last4, int kc,
                                                 AfterWait &&after_wait)
{
    const uint32_t lim8 = 8u * (uint32_t)(kc + kMmAhead), end8 = 8u * (uint32_t)(kc + kMmKc);
    bool first = true;
    do {
        // Slide the window by one piece where its first piece is used up (a third of the lanes in a step, as a
        // rule), and ask for the next one there.
        {
            const bool s8 = d.ci - d.wbase >= 16u;  // (not below the new first piece afterwards, so that the next such test holds)
            asm volatile("" : "+v"(d.fut));  // (the wait belongs here, ahead of after_wait's loads)
            if (first) {
                first = false;
                after_wait();
            }
            if (s8) {
                ring_store_piece(d, d.wbase & 16u, d.fut);
                d.wbase += 16u;
                d.pp += d.pstr;
                d.fut = ring_piece_at(d, d.pp + 2u * d.pstr);
            }
            d.lim = min(d.end, d.wbase + kMmWinAhead);
        }
        if (__any(d.ci < d.lim && d.pos8 < end8)) ring_rounds<ASYM>(d, minus_groups12, last4, lim8, end8);
    } while (__any(d.ci < d.end && d.pos8 < end8));
}

// The half of the ring that held step c becomes columns kc + 128 .. kc + 191: cleared after
// the step's reads.
__device__ __forceinline__ void ring_clear_half(const RingDecoder &d, int c)
{
#pragma unroll
    for (int i = 0; i < kMmKc / 8; i++) ((lw_u64)(uintptr_t)(d.wrow + (uint32_t)((c & 1) * kMmKc)))[i] = 0ull;
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
// MB: blocks of 16 tokens in the tile (1, 2 or 4).  D[token][row] += X[token][k] * W^T[k][row]
// with v_mfma_f32_16x16x32_bf16: operand lane l holds 8 consecutive k (group l / 16) of token
// or row l % 16; accumulator v of lane l is token 4 * (l / 16) + v, row l % 16 of the block.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int MB, int EPI, int ASYM>
__device__ __forceinline__ void mm_item(const ProductArgs &a, const qmoe_matrix &M, int rblk, int slot0, int ntok,
                                        uint32_t wt, uint32_t win)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lg = lane >> 4;

    // The second product writes to the tokens' own rows of the output, scaled by their gates.  Lane t asks
    // for token t's row and gate now, among the other trips to memory of the set-up (two registers for the
    // length of the item); the lanes swap them when the results are written.
    int tok_own = 0;
    float gate_own = 1.0f;
    if constexpr (EPI == 0) {
        const int t = min(lane, ntok - 1);
        tok_own = a.perm ? a.perm[slot0 + t] : slot0 + t;
    }

    // ---- this lane's row (the wavefront's 64 rows are block `rblk` of the matrix) and its codewords
    const int r0 = rblk * 64;
    const int row = r0 + lane;
    const bool row_live = row < a.rows;
    RingDecoder dec;
    ring_setup(dec, M, row, row_live, wt + (uint32_t)(tid * kMmWRowBytes), win + (uint32_t)(tid * kMmWinBytes));
    if constexpr (EPI == 0) gate_own = a.gate ? a.gate[tok_own] : 1.0f;

    // ---- this lane's part of the activations: token 16 * mb + l16, columns 8 * lg .. 8 * lg + 7 of every 32
    uintptr_t xsrc[MB];
    uint32_t xmul2[MB];  // bytes from one column's value to the next column's: 2, or (tiled) 2 * the block's tokens
    const bool x_col = 8 * lg + 8 <= a.cols;
#pragma unroll
    for (int mb = 0; mb < MB; mb++) {
        const int t = 16 * mb + l16;
        const bool x_ok = t < ntok;
        xmul2[mb] = 2u;
        // (a lane whose columns do not exist -- fewer than 8 * lg + 8 columns -- reads column 0 and drops it;
        // a lane without a token reads the block's first token, or row 0)
        const size_t col0 = x_col ? 8 * (size_t)lg : (size_t)0;
        if (EPI == 0 && a.x_tiled) {
            const int tb = min(16, ntok - 16 * mb);  // tokens in this block (<= 0: no such block)
            const size_t block0 = tb > 0 ? (size_t)(slot0 + 16 * mb) : (size_t)slot0;
            const size_t j = x_ok ? (size_t)l16 : (size_t)0;
            xmul2[mb] = 2u * (uint32_t)__builtin_amdgcn_readfirstlane(max(tb, 1));
            xsrc[mb] = reinterpret_cast<uintptr_t>(a.x) + 2 * (block0 * (size_t)a.ldx + 8 * j) + col0 * (size_t)xmul2[mb];
        } else {
            size_t xrow = 0;
            if (x_ok) {
                const int tok = a.perm ? a.perm[slot0 + t] : slot0 + t;
                xrow = a.x_by_slot ? (size_t)(slot0 + t) : (size_t)tok;
            }
            xsrc[mb] = reinterpret_cast<uintptr_t>(a.x) + 2 * (xrow * (size_t)a.ldx + col0);
        }
    }
    // A step's activations are asked for before its weights are decoded and arrive meanwhile.  What a lane without a token brings is some other row's and multiplies into a result nobody writes.
    // Only a last step of fewer than 64 columns looks at its columns: a lane past the last one reads column 8 * lg and
    // drops it.
    const int x_last = x_col ? a.cols - 8 * lg - 8 : 0;  // last column offset this lane may read at
    u32x4 xa[MB][2];
    uint32_t x_end[MB];  // x_last in bytes
#pragma unroll
    for (int mb = 0; mb < MB; mb++) x_end[mb] = (uint32_t)x_last * xmul2[mb];
    auto fetch_x = [&](int k) {
#pragma unroll
        for (int mb = 0; mb < MB; mb++)
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
                xa[mb][ks] = *(gp_u32x4)(xsrc[mb] + (uintptr_t)min((uint32_t)(k + 32 * ks) * xmul2[mb], x_end[mb]));
    };

    f32x4 acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; mb++)
#pragma unroll
        for (int nb = 0; nb < 4; nb++) acc[mb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // asymmetric grid: the grid points of the four rows whose weights this lane feeds to the matrix cores
    uint32_t g_hi[4] = {0u, 0u, 0u, 0u}, g_lo[4] = {0u, 0u, 0u, 0u};
    if constexpr (ASYM) {
#pragma unroll
        for (int nb = 0; nb < 4; nb++) {
            const int rl = 16 * nb + l16;
            uint32_t pair = 0u;  // a row past the end, or a matrix without a pair array, multiplies as zeros
            if (r0 + rl < a.rows && M.minmax_bf16) pair = ((gp_u32)M.minmax_bf16)[r0 + rl];
            g_hi[nb] = pair << 16;
            g_lo[nb] = pair & 0xFFFF0000u;
        }
    }
    const uint32_t wfrag = wt + (uint32_t)((64 * wave + l16) * kMmWRowBytes + 8 * lg);
    const int nsteps = (a.cols + kMmKc - 1) / kMmKc;
    const int minus_groups12 = -12 * a.n_groups, last4 = 4 * (a.n_order - 1);

    ring_prime(dec, minus_groups12, last4);

    for (int c = 0; c < nsteps; c++) {
        const int kc = c * kMmKc;
        // ---- decode until every lane has passed column kc + 64
        ring_decode_step<ASYM>(dec, minus_groups12, last4, kc, [&]() { fetch_x(kc); });
        // the rows this wavefront multiplies are the ones its own lanes wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // (all of the step's weights are asked for before the first is used: 1000 us, 988 now for 256 experts of 2080 x 6144)
        unsigned long long wd[2][4];
        {
            const uint32_t wf = wfrag + (uint32_t)((c & 1) * kMmKc);
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
#pragma unroll
                for (int nb = 0; nb < 4; nb++) wd[ks][nb] = *(lp_u64)(uintptr_t)(wf + (uint32_t)(nb * 16 * kMmWRowBytes + 32 * ks));
            __builtin_amdgcn_sched_barrier(0);
        }

        if (kc + kMmKc > a.cols) {
            asm volatile("");  // (a branch, not selects in every step)
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int ks = 0; ks < 2; ks++) xa[mb][ks] = x_col && kc + 32 * ks <= x_last ? xa[mb][ks] : u32x4{0u, 0u, 0u, 0u};
        }

        // ---- multiply step c
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            bf16x8 bw[4], ax[MB];
#pragma unroll
            for (int nb = 0; nb < 4; nb++) {
                const unsigned long long d = wd[ks][nb];
                if constexpr (ASYM)
                    bw[nb] = mm_expand_minmax((uint32_t)d, (uint32_t)(d >> 32), g_hi[nb], g_lo[nb]);
                else
                    bw[nb] = mm_expand((uint32_t)d, (uint32_t)(d >> 32));
            }
#pragma unroll
            for (int mb = 0; mb < MB; mb++) __builtin_memcpy(&ax[mb], &xa[mb][ks], 16);
#pragma unroll
            for (int mb = 0; mb < MB; mb++)
#pragma unroll
                for (int nb = 0; nb < 4; nb++)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax[mb], bw[nb], acc[mb][nb], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        ring_clear_half(dec, c);
    }

    // accumulator v of lane l: token 16 * mb + 4 * (l / 16) + v, row 16 * nb + l % 16 of the wavefront's 64
    // (second product: output row and gate of each of the lane's tokens, from the lane that holds them)
    int tok_of[MB][4];
    float gate_of[MB][4];
    if constexpr (EPI == 0) {
#pragma unroll
        for (int mb = 0; mb < MB; mb++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int t = 16 * mb + 4 * lg + v;  // < 64
                tok_of[mb][v] = __shfl(tok_own, t, 64);
                gate_of[mb][v] = __shfl(gate_own, t, 64);
            }
    }
#pragma unroll
    for (int nb = 0; nb < 4; nb++) {
        const int r = r0 + 16 * nb + l16;
        if (r < a.rows) {
            // symmetric grid: the weights were +-2; asymmetric: they were the grid points themselves
            const float scale = ASYM ? 1.0f : 0.5f * half_bits_to_float(((gp_u16)M.scale_f16)[r]);
#pragma unroll
            for (int mb = 0; mb < MB; mb++) {
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int t = 16 * mb + 4 * lg + v;
                    if (t < ntok) {
                        const float val = acc[mb][nb][v] * scale;
                        if constexpr (EPI == 0) {
                            reinterpret_cast<float *>(a.out)[(size_t)tok_of[mb][v] * a.ld_out + r] = gate_of[mb][v] * val;
                        } else {
                            const float h = val > 0.0f ? val : 0.0f;
                            size_t at = (size_t)(slot0 + t) * a.ld_out + r;
                            if (a.out_tiled) {
                                const int tb = min(16, ntok - 16 * mb);
                                at = (size_t)(slot0 + 16 * mb) * a.ld_out + ((size_t)(r >> 3) * tb + (4 * lg + v)) * 8 + (r & 7);
                            }
                            reinterpret_cast<uint16_t *>(a.out)[at] = float_to_bf16_bits(h);
                        }
                    }
                }
            }
        }
    }
}

template <int EPI, int ASYM>
__global__ __launch_bounds__(kMmThreads) void k_product_mm(const ProductArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const size_t table_bytes = mm_table_bytes(a.n_order);
    uint32_t *table_w = reinterpret_cast<uint32_t *>(smem);
    unsigned char *wt = smem + table_bytes;                           // [512][kMmWRowBytes] rings
    unsigned char *win = wt + (size_t)kMmThreads * kMmWRowBytes;      // [512][kMmWinBytes] codeword windows

    // A unit of work is 64 rows of one (expert, token tile) item, and a wavefront takes it alone: after
    // the table is staged the wavefronts of a workgroup share nothing and meet at no barrier, so one
    // wavefront's set-up (a chain of trips to memory) runs under the others' arithmetic, a matrix
    // whose rows are no multiple of 512 leaves no wavefront idle, and the units are small enough to
    // pack well.  A layer call brings a list of items and a device counter that hands the units out;
    // the single-matrix call has neither: its items are the tiles of 64 consecutive tokens of
    // `single`, its units dealt out round robin.
    const bool listed = a.items != nullptr;
    const int n_items = listed ? min(*a.n_items_dev, a.max_items) : (a.batch + kMmTokens - 1) / kMmTokens;
    const int total = (int)min((long long)n_items * a.mm_row_blocks, 0x7FFFFFFFLL);
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, waves = kMmThreads / 64;
    // No more workgroups than fill all their wavefronts stay (a workgroup holds its compute unit's LDS whole,
    // so one that runs half empty keeps the other kernels of a layer call off that compute unit); the
    // single-matrix call, which is after latency, spreads its units over as many compute units as it can.
    if (total <= 0 || (int)blockIdx.x >= (listed ? (total + waves - 1) / waves : total)) return;
    int *next_base = reinterpret_cast<int *>(win + (size_t)kMmThreads * kMmWinBytes);  // [1], in-step hand-out only
    int *tok_sums = next_base + 1;                                                      // [2]
    if (threadIdx.x < 2) tok_sums[threadIdx.x] = 0;
    stage_words(table_w, a.order_table, a.n_order, ring_entry_bytes);
    __syncthreads();
    // In step or each wavefront for itself (see the loop)?  In step when most of the tokens sit in tiles of
    // more than 32: those read 4-8 KB of activations per wavefront and step.
    bool in_step = false;
    if (listed && a.mm_in_step) {
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
    // (round robin over the workgroups first, then over their wavefronts: few units spread over many compute units)
    int g_static = wave * (int)gridDim.x + (int)blockIdx.x;
    for (;;) {
        int g = g_static;
        if (in_step) {
            // The wavefronts of a workgroup take eight consecutive units together and start them together:
            // where the activations are not stored by token blocks (the first product of a layer) their
            // operand loads touch a line per token, and eight wavefronts that ask for the same lines at the
            // same time are served by one fetch.  (Measured both ways: a layer with few, crowded experts is
            // 3 % faster in step, one with many experts of 8-32 tokens 7 % faster without.)
            __syncthreads();
            if (threadIdx.x == 0) *next_base = atomicAdd(a.work_counter, waves);
            __syncthreads();
            const int base = *next_base;
            if (base >= total) break;
            g = base + wave;
            if (g >= total) continue;
        } else if (listed) {
            int got = 0;
            if (lane == 0) got = atomicAdd(a.work_counter, 1);
            g = __builtin_amdgcn_readfirstlane(got);
        }
        g_static += (int)gridDim.x * waves;
        if (g >= total) break;
        const int idx = g / a.mm_row_blocks;
        const int rblk = g - idx * a.mm_row_blocks;
        Item it;
        if (listed) {
            it = a.items[idx];
        } else {
            it.expert = 0;
            it.slot0 = idx * kMmTokens;
            it.ntok = a.batch - idx * kMmTokens;
        }
        const int expert = it.expert, slot0 = it.slot0;
        const int ntok = min(it.ntok, kMmTokens);
        if (expert < 0 || expert >= a.n_experts || ntok < 1) continue;
        const qmoe_matrix M = a.mats ? a.mats[expert] : a.single;
        if (ntok <= 16)
            mm_item<1, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
        else if (ntok <= 32)
            mm_item<2, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
        else
            mm_item<4, EPI, ASYM>(a, M, rblk, slot0, ntok, wt_addr, win_addr);
    }
}

}  // namespace

size_t mm_lds_bytes(int n_order)
{
    return mm_table_bytes(n_order) + (size_t)kMmThreads * kMmWRowBytes +
           (size_t)kMmThreads * kMmWinBytes + 16;
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
