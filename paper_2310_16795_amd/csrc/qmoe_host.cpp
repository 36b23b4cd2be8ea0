// Host side of the library: dictionary generation (Section 4.3.2, Algorithm 1),
// entry layouts, the longest-prefix trie encoder and stream validation
// (Section 4.3.3 "Encoding").  No GPU code in this file.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <map>
#include <queue>
#include <thread>

#include <pthread.h>

#if defined(__SSE2__)
#include <emmintrin.h>
#endif

#include "qmoe_internal.h"
#include "qmoe_hooks.h"

namespace qmoe {

Tuning &tuning()
{
    static Tuning t;
    return t;
}

namespace {

// A candidate sequence of Algorithm 1, symbols packed two bits apiece
// (symbol j at bits 2j..2j+1), plus the counts its probability depends on.
struct Candidate {
    uint64_t syms;   // up to 28 symbols
    uint64_t rank3;  // the symbol string as a base-3 number (first symbol most significant)
    double logp;     // zeros*ln(p0) + nonzeros*ln(q), from the integer counts
    uint8_t npairs, zeros, nonzeros;
};

// priority_queue keeps the element for which "less" is false against all others on top
struct PopsLater {
    bool operator()(const Candidate &a, const Candidate &b) const
    {
        if (a.logp != b.logp) return a.logp < b.logp;
        return a.rank3 > b.rank3;
    }
};

inline int sym_at(uint64_t syms, int j) { return (int)((syms >> (2 * j)) & 3u); }

void pack_words(uint64_t syms, int npairs, uint32_t *w)
{
    // each word: count in the low nibble, then its 14 symbols from bit 4 up
    w[0] = (uint32_t)npairs | (uint32_t)((syms & ((1ull << 28) - 1)) << 4);
    w[1] = (uint32_t)npairs | (uint32_t)(((syms >> 28) & ((1ull << 28) - 1)) << 4);
}

// Device numbering of the codewords: group the sign variants of the last two non-zeros
// of each run under one table entry (see qmoe_internal.h).
// What the two low bits of a device code toggle in its table entry: the sign bits of
// fields 1 and 2.  The kernels apply it to every code; single entries are stored with it
// applied once already.
inline uint32_t order_flips(uint32_t code)
{
    return ((code & 1u) << 18) | ((code & 2u) << 25);
}

void build_device_order(qmoe_dict *d)
{
    d->order_table.clear();
    d->order_map.clear();
    d->n_groups = 0;
    if (d->max_nonzeros > kRunMaxNonzeros) return;
    const int n = d->n_entries;
    struct Nz { int pos; bool neg; };
    // key: run length, positions, and the sign of the first non-zero when there are three
    std::map<std::vector<int>, std::vector<int>> groups;  // key -> member code by free-sign bits, -1 = missing
    std::vector<std::vector<Nz>> nz((size_t)n);
    for (int k = 0; k < n; k++) {
        const uint32_t e = d->run[k];
        for (int j = 0; j < kRunMaxNonzeros; j++) {
            const uint32_t f = (e >> (8 + 8 * j)) & 0xFFu;
            if (f) nz[k].push_back(Nz{(int)(f >> 3), ((f >> 1) & 3u) == 3u});
        }
        const size_t c = nz[k].size();
        if (c < 2) continue;
        std::vector<int> key{(int)(e & 0xFFu)};
        for (const Nz &z : nz[k]) key.push_back(z.pos);
        if (c == 3) key.push_back(nz[k][0].neg ? 1 : 0);
        const int bits = (nz[k][c - 2].neg ? 1 : 0) | (nz[k][c - 1].neg ? 2 : 0);
        std::vector<int> &m = groups[key];
        if (m.empty()) m.assign(4, -1);
        if (m[bits] < 0) m[bits] = k;  // duplicates in a hand-made table stay single entries
    }
    std::vector<uint32_t> table;
    std::vector<int> device_of((size_t)n, -1);
    for (const auto &kv : groups) {
        const std::vector<int> &m = kv.second;
        if (m[0] < 0 || m[1] < 0 || m[2] < 0 || m[3] < 0) continue;
        const int g = (int)table.size();
        const int k = m[0];  // both free signs positive
        const size_t c = nz[k].size();
        uint32_t e = d->run[k] & 0xFFu;
        if (c == 3) e |= (((uint32_t)nz[k][0].pos << 3) | ((nz[k][0].neg ? 3u : 1u) << 1)) << 8;
        e |= (((uint32_t)nz[k][c - 2].pos << 3) | (1u << 1)) << 16;
        e |= (((uint32_t)nz[k][c - 1].pos << 3) | (1u << 1)) << 24;
        table.push_back(e);
        for (int b = 0; b < 4; b++) device_of[m[b]] = 4 * g + b;
    }
    const int n_groups = (int)table.size();
    int next = 4 * n_groups;
    for (int k = 0; k < n; k++) {
        if (device_of[k] >= 0) continue;
        device_of[k] = next++;
        // fields right-aligned like those of the groups: unused ones (0) come first
        uint32_t e = d->run[k];
        while ((e >> 8) != 0u && (e >> 24) == 0u) e = (e & 0xFFu) | ((e & 0xFFFFFF00u) << 8);
        table.push_back(e ^ order_flips((uint32_t)device_of[k]));
    }
    int absent = -1;  // codes that name no entry all map to one empty single entry
    if (n < kTableEntries) {
        absent = next++;
        table.push_back(0u ^ order_flips((uint32_t)absent));
    }
    if ((int)table.size() > kMaxOrderTable || next > kTableEntries) return;
    d->order_map.assign(kTableEntries, (uint16_t)(absent >= 0 ? absent : 0));
    for (int k = 0; k < n; k++) d->order_map[k] = (uint16_t)device_of[k];
    d->order_table = std::move(table);
    d->n_groups = n_groups;
}

// The run coder's tables (see qmoe_internal.h), from the trie; left empty when the dictionary does not
// qualify: an entry with more than three non-zeros, or a prefix of an entry that is no entry.
void build_run_coder(qmoe_dict *d)
{
    d->rc_depth.clear();
    d->rc_first.clear();
    d->rc_codes.clear();
    d->rc_depth0 = 0;
    if (d->max_nonzeros > kRunMaxNonzeros || d->code.size() < 2) return;
    for (size_t i = 1; i < d->code.size(); i++)
        if (d->code[i] < 0) return;
    struct Step { int node, pairs, k, pos[3], neg[3]; };
    std::vector<std::vector<uint16_t>> chain(kRcPatterns);  // codewords of a pattern in order of their pairs
    std::vector<Step> todo{Step{0, 0, 0, {0, 0, 0}, {0, 0, 0}}};
    std::vector<int> shortest(kRcPatterns, 0);
    while (!todo.empty()) {
        const Step s = todo.back();
        todo.pop_back();
        if (s.node) {
            int i = kRcZero;
            const int c2 = s.k >= 2 ? s.pos[1] * (s.pos[1] - 1) / 2 + s.pos[0] : 0;
            if (s.k == 1) i = kRcOne + 2 * s.pos[0] + s.neg[0];
            if (s.k == 2) i = kRcTwo + 4 * c2 + (s.neg[0] | s.neg[1] << 1);
            if (s.k == 3)
                i = kRcThree + 8 * (s.pos[2] * (s.pos[2] - 1) * (s.pos[2] - 2) / 6 + c2) +
                    (s.neg[0] | s.neg[1] << 1 | s.neg[2] << 2);
            if (chain[i].empty()) shortest[i] = s.pairs;
            chain[i].push_back((uint16_t)d->code[s.node]);  // a parent comes off the stack before its children: in order
        }
        for (int pair = 0; pair < 9; pair++) {
            const int nx = d->child[(size_t)s.node * 9 + pair];
            if (nx < 0) continue;
            Step c = s;
            c.node = nx;
            c.pairs++;
            const int sym[2] = {pair / 3, pair % 3};
            for (int j = 0; j < 2; j++)
                if (sym[j]) {
                    c.pos[c.k] = 2 * s.pairs + j;
                    c.neg[c.k++] = sym[j] == 1;
                }
            todo.push_back(c);
        }
    }
    d->rc_depth.assign(kRcDepthBytes, 0);
    d->rc_first.assign(kRcPatterns, 0);
    for (int i = 0; i < kRcPatterns; i++) {
        d->rc_first[i] = (uint32_t)d->rc_codes.size() - (uint32_t)shortest[i];
        d->rc_codes.insert(d->rc_codes.end(), chain[i].begin(), chain[i].end());
    }
    auto depth = [&](int i) { return chain[i].empty() ? 0 : shortest[i] + (int)chain[i].size() - 1; };
    for (int i = 0; i < kRcTwo; i++) d->rc_depth[i / 2] |= (uint8_t)(depth(i) << 4 * (i & 1));
    for (int p2 = 1; p2 < 30; p2++)
        for (int p1 = 0; p1 < p2; p1++)
            for (int s = 0; s < 4; s++) {
                const int c2 = p2 * (p2 - 1) / 2 + p1;
                const int d2 = p2 < 28 ? depth(kRcTwo + 4 * c2 + s) : 0, d1 = p1 < 28 ? depth(kRcOne + 2 * p1 + (s & 1)) : 0;
                d->rc_depth[kRcDepth3Bytes + 4 * c2 + s] = (uint8_t)(d2 | d1 << 4);
            }
    d->rc_depth0 = depth(kRcZero);
}

// Derive everything the codec and the kernels need from the interchange words.
qmoe_status finish_dict(qmoe_dict *d)
{
    const int n = d->n_entries;
    d->run.assign(kTableEntries, 0u);
    d->max_nonzeros = 0;
    d->max_pairs = 0;
    for (int k = 0; k < n; k++) {
        const uint32_t w0 = d->words[2 * k], w1 = d->words[2 * k + 1];
        const int np = (int)(w0 & 15u);
        if (np < 1 || np > 14 || (int)(w1 & 15u) != np) return QMOE_E_BAD_SYMBOL;
        d->max_pairs = std::max(d->max_pairs, np);
        uint32_t run = (uint32_t)(8 * 2 * np);
        int nnz = 0;
        for (int j = 0; j < kMaxSyms; j++) {
            const uint32_t w = j < 14 ? w0 : w1;
            const int s = (int)((w >> (4 + 2 * (j % 14))) & 3u);
            if (s == 3) return QMOE_E_BAD_SYMBOL;
            if (j >= 2 * np && s != 0) return QMOE_E_BAD_SYMBOL;
            if (s != 0) {
                if (nnz < kRunMaxNonzeros) {
                    const uint32_t weight = (s == 2) ? 1u : 3u;  // 2-bit signed: +1 / -1
                    run |= (((uint32_t)j << 3) | (weight << 1)) << (8 + 8 * nnz);
                }
                nnz++;
            }
        }
        d->max_nonzeros = std::max(d->max_nonzeros, nnz);
        d->run[k] = run;
    }
    build_device_order(d);
    // trie: node 0 is the root; an entry's node is reached by its pairs in order
    d->child.assign(9, -1);
    d->code.assign(1, -1);
    for (int k = 0; k < n; k++) {
        const uint32_t w0 = d->words[2 * k], w1 = d->words[2 * k + 1];
        const int np = (int)(w0 & 15u);
        int node = 0;
        for (int j = 0; j < np; j++) {
            const uint32_t w = j < 7 ? w0 : w1;
            const int pr = (int)((w >> (4 + 4 * (j % 7))) & 15u);  // two symbols = 4 bits
            const int pair = 3 * (pr & 3) + (pr >> 2);             // first symbol is the low one
            int nx = d->child[(size_t)node * 9 + pair];
            if (nx < 0) {
                nx = (int)d->code.size();
                d->code.push_back(-1);
                d->child.resize(d->child.size() + 9, -1);
                d->child[(size_t)node * 9 + pair] = nx;
            }
            node = nx;
        }
        if (d->code[node] < 0) d->code[node] = k;  // duplicates: the earlier (more probable) index wins
    }
    build_run_coder(d);
    return QMOE_OK;
}

inline int pair_of(int8_t a, int8_t b)
{
    // value -> symbol: 0 -> 0, -1 -> 1, +1 -> 2 ; returns -1 for anything else
    const int sa = a == 0 ? 0 : (a == -1 ? 1 : (a == 1 ? 2 : -1));
    const int sb = b == 0 ? 0 : (b == -1 ? 1 : (b == 1 ? 2 : -1));
    return (sa < 0 || sb < 0) ? -1 : 3 * sa + sb;
}

// One row as two bit strings (bit c: value c is non-zero; it is negative), four spare bytes zero behind
// each.  False when a value is not -1, 0 or +1.
bool row_bits(const int8_t *row, int cols, uint8_t *nz, uint8_t *neg)
{
    int c = 0, bad = 0;
    auto up_to_16 = [&] {
        uint16_t n = 0, m = 0;
        for (int j = 0; j < 16 && c + j < cols; j++) {
            const int v = row[c + j];
            bad |= v < -1 || v > 1;
            n |= (uint16_t)((v != 0) << j);
            m |= (uint16_t)((v < 0) << j);
        }
        std::memcpy(nz + c / 8, &n, 2);
        std::memcpy(neg + c / 8, &m, 2);
        c += 16;
    };
#if defined(__SSE2__)
    for (; c + 16 <= cols; c += 16) {
        const __m128i v = _mm_loadu_si128(reinterpret_cast<const __m128i *>(row + c));
        const __m128i is0 = _mm_cmpeq_epi8(v, _mm_setzero_si128()), is1 = _mm_cmpeq_epi8(v, _mm_set1_epi8(1)),
                      ism = _mm_cmpeq_epi8(v, _mm_set1_epi8(-1));
        bad |= _mm_movemask_epi8(_mm_or_si128(_mm_or_si128(is0, is1), ism)) ^ 0xFFFF;
        const uint16_t n = (uint16_t)~_mm_movemask_epi8(is0), m = (uint16_t)_mm_movemask_epi8(ism);
        std::memcpy(nz + c / 8, &n, 2);
        std::memcpy(neg + c / 8, &m, 2);
    }
    if (c < cols) up_to_16();
#else
    while (c < cols) up_to_16();
#endif
    std::memset(nz + c / 8, 0, 8);
    std::memset(neg + c / 8, 0, 8);
    return bad == 0;
}

// The codewords of rows by the run coder (longest prefix from the places of the next three non-zeros, see
// qmoe_internal.h): about sixty instructions a codeword in place of a dependent table read per pair of
// values.  A codeword's length is needed before the next one can be looked for, so four rows take turns:
// their chains overlap (4096 x 1024 values on one thread: 24 ms by the trie, 4.2 ms row by row, 3.0 ms so).
constexpr int kRowsAtOnce = 4;

struct RowParse {
    const uint8_t *nz, *neg;
    uint16_t *out;
    int i = 0, n = 0;  // pairs done, codewords written; i = -1: no entry fits
};

// The longest entry at pair i of a row: its codeword, and its pairs in *pairs (0: no entry fits).
__attribute__((always_inline)) inline uint16_t longest_run(const uint8_t *depth3, const uint32_t *first, const uint16_t *codes,
                                                           int depth0, int np, const RowParse &r, int i, int *pairs)
{
    const uint8_t *depth2 = depth3 + kRcDepth3Bytes;
    uint64_t w64, m64;
    std::memcpy(&w64, r.nz + (i >> 2), 8);
    std::memcpy(&m64, r.neg + (i >> 2), 8);
    // positions 28..31 stand in for non-zeros that are not there
    uint32_t w = ((uint32_t)(w64 >> (2 * (i & 3))) & 0x0FFFFFFFu) | 0xF0000000u;
    const uint32_t m = (uint32_t)(m64 >> (2 * (i & 3))) & 0x0FFFFFFFu;
    const int p1 = __builtin_ctz(w);
    w &= w - 1;
    const int p2 = __builtin_ctz(w);
    w &= w - 1;
    const int p3 = __builtin_ctz(w);
    w &= w - 1;
    const int p4 = __builtin_ctz(w);
    const int s2 = (int)((m >> p1 & 1) | (m >> p2 & 1) << 1), s3 = s2 | (int)(m >> p3 & 1) << 2;
    const int c2 = p2 * (p2 - 1) / 2 + p1, i3 = 8 * (p3 * (p3 - 1) * (p3 - 2) / 6 + c2) + s3;
    const int limit = std::min(14, np - i);
    const int both = depth2[4 * c2 + s2];
    const int l3 = std::min(std::min(depth3[std::min(i3, kRcTwo) >> 1] >> 4 * (s2 & 1) & 15, limit), p4 >> 1);
    const int l2 = std::min(std::min(both & 15, limit), p3 >> 1), l1 = std::min(std::min(both >> 4, limit), p2 >> 1);
    // the deepest of the four that is there at all (selects: which one it is cannot be predicted)
    int len = std::min(std::min(depth0, limit), p1 >> 1), at = kRcZero;
    at = l1 > p1 >> 1 ? kRcOne + 2 * p1 + (s2 & 1) : at;
    len = l1 > p1 >> 1 ? l1 : len;
    at = l2 > p2 >> 1 ? kRcTwo + 4 * c2 + s2 : at;
    len = l2 > p2 >> 1 ? l2 : len;
    at = l3 > p3 >> 1 ? kRcThree + i3 : at;
    len = l3 > p3 >> 1 ? l3 : len;
    *pairs = len;
    return len < 1 ? 0 : codes[first[at] + (uint32_t)len];
}

void encode_rows_runs(const qmoe_dict *d, int np, RowParse *rows, int n_rows)
{
    const uint8_t *depth3 = d->rc_depth.data();
    const uint32_t *first = d->rc_first.data();
    const uint16_t *codes = d->rc_codes.data();
    const int depth0 = d->rc_depth0;
    if (n_rows == kRowsAtOnce) {
        const RowParse a = rows[0], b = rows[1], c = rows[2], e = rows[3];
        int ia = a.i, ib = b.i, ic = c.i, ie = e.i, n = 0;
        auto live = [np](int i) { return (unsigned)i < (unsigned)np; };
        while (live(ia) && live(ib) && live(ic) && live(ie)) {
            int la, lb, lc, le;
            a.out[n] = longest_run(depth3, first, codes, depth0, np, a, ia, &la);
            b.out[n] = longest_run(depth3, first, codes, depth0, np, b, ib, &lb);
            c.out[n] = longest_run(depth3, first, codes, depth0, np, c, ic, &lc);
            e.out[n] = longest_run(depth3, first, codes, depth0, np, e, ie, &le);
            ia = la ? ia + la : -1;
            ib = lb ? ib + lb : -1;
            ic = lc ? ic + lc : -1;
            ie = le ? ie + le : -1;
            n++;
        }
        rows[0].i = ia; rows[1].i = ib; rows[2].i = ic; rows[3].i = ie;
        for (int k = 0; k < kRowsAtOnce; k++) rows[k].n = n;
    }
    for (int k = 0; k < n_rows; k++) {
        RowParse &r = rows[k];
        int i = r.i, n = r.n;
        while ((unsigned)i < (unsigned)np) {
            int len;
            r.out[n++] = longest_run(depth3, first, codes, depth0, np, r, i, &len);
            i = len ? i + len : -1;
        }
        r.i = i;
        r.n = n;
    }
}

// What a thread keeps from one piece of a matrix to the next.
struct EncodeScratch {
    std::vector<uint8_t> strings;    // non-zero and sign bits of the rows in work
    std::vector<uint16_t> lines;     // their codewords
};

// Encode rows [r0, r1) into out (appended), counts[r - r0] = codewords of row r.
qmoe_status encode_rows(const qmoe_dict *d, const int8_t *tern, int cols, int r0, int r1, EncodeScratch *scratch,
                        std::vector<uint16_t> *out, uint32_t *counts, bool store)
{
    const int32_t *child = d->child.data();
    const int32_t *code = d->code.data();
    const int np = cols / 2;
    const bool runs = !d->rc_depth.empty();
    const size_t bits = (size_t)cols / 8 + 32;
    std::vector<uint8_t> &strings = scratch->strings;
    std::vector<uint16_t> &lines = scratch->lines;
    RowParse work[kRowsAtOnce];
    int done_to = r0;                // rows below it are in work, or done
    if (runs) {
        strings.resize(2 * kRowsAtOnce * bits);
        lines.resize((size_t)kRowsAtOnce * np);
    }
    for (int r = r0; r < r1; r++) {
        const int8_t *row = tern + (size_t)r * cols;
        if (runs) {
            if (r == done_to) {
                const int take = std::min(kRowsAtOnce, r1 - r);
                for (int k = 0; k < take; k++) {
                    uint8_t *nz = strings.data() + 2 * k * bits, *neg = nz + bits;
                    work[k] = RowParse{nz, neg, lines.data() + (size_t)k * np};
                    if (!row_bits(row + (size_t)k * cols, cols, nz, neg)) work[k].i = -1;
                }
                encode_rows_runs(d, np, work, take);
                done_to = r + take;
            }
            const RowParse &w = work[(r - r0) % kRowsAtOnce];
            if (w.i >= 0) {
                if (store) out->insert(out->end(), w.out, w.out + w.n);
                counts[r - r0] = (uint32_t)w.n;
                continue;
            }
        }
        // other dictionaries, and rows that do not encode (the walk says which error comes first)
        uint32_t n = 0;
        int i = 0;
        while (i < np) {
            int node = 0, best = -1, best_len = 0, depth = 0;
            while (i + depth < np) {
                const int pr = pair_of(row[2 * (i + depth)], row[2 * (i + depth) + 1]);
                if (pr < 0) return QMOE_E_BAD_SYMBOL;
                const int nx = child[(size_t)node * 9 + pr];
                if (nx < 0) break;
                node = nx;
                depth++;
                if (code[node] >= 0) {
                    best = code[node];
                    best_len = depth;
                }
            }
            if (best < 0) return QMOE_E_UNENCODABLE;
            if (store) out->push_back((uint16_t)best);
            n++;
            i += best_len;
        }
        counts[r - r0] = n;
    }
    return QMOE_OK;
}

// One call of qmoe_encode_host: threads that take pieces of some rows each, in order, and then, when all pieces are parsed and
// their places known, copy their own codewords there.
//
// What bounds it: a thread's start (7 us where this was measured), and page faults of the results.  So every thread starts up to
// two others before its first piece, on stacks small enough that the C library keeps them from call to call, pieces are small enough that
// the late ones find work left, and nobody copies for the others.  4096 x 1024 values at 92 % zeros, 16 threads: 256 us (1436 with
// one thread), 345 with sixteen even shares, threads started one after the other and one thread that put the parts together.
class HostEncoder {
public:
    HostEncoder(const qmoe_dict *dict, const int8_t *ternary, int n_rows, int n_cols, uint16_t *out, size_t out_cap, uint32_t *offsets,
                size_t *total, int n_threads)
        : d(dict), tern(ternary), rows(n_rows), cols(n_cols), codes(out), cap(out_cap), row_off(offsets), n_codes(total), threads(n_threads)
    {
        // (eight pieces a thread, of whole groups of the rows that are parsed together)
        const int even = (rows + 8 * threads - 1) / (8 * threads);
        piece = std::min(256, (even + kRowsAtOnce - 1) / kRowsAtOnce * kRowsAtOnce);
        n_pieces = (rows + piece - 1) / piece;
        counts.resize((size_t)rows);
        status.assign((size_t)n_pieces, QMOE_OK);
    }

    qmoe_status run()
    {
        work(0);
        return result;
    }

private:
    struct Start {
        HostEncoder *encoder;
        int t;
    };
    struct Part {
        int r0;
        size_t at, n;  // in the thread's own codewords
    };

    static void *begin(void *p)
    {
        const Start s = *static_cast<Start *>(p);
        s.encoder->work(s.t);
        return nullptr;
    }

    void work(int t)
    {
        // (a thread that cannot be started leaves its pieces to the others)
        pthread_t child[2];
        Start start[2];
        int started = 0;
        for (int k = 1; k <= 2; k++) {
            if (2 * t + k >= threads) break;
            pthread_attr_t attr;
            if (pthread_attr_init(&attr) != 0) break;
            start[started] = Start{this, 2 * t + k};
            if (pthread_attr_setstacksize(&attr, kStackBytes) == 0 && pthread_create(&child[started], &attr, begin, &start[started]) == 0)
                started++;
            pthread_attr_destroy(&attr);
        }
        std::vector<uint16_t> own;
        std::vector<Part> parts;
        EncodeScratch scratch;
        for (int p; (p = next_piece.fetch_add(1, std::memory_order_relaxed)) < n_pieces;) {
            // (a piece behind one that failed does not matter; one before it may fail earlier in the matrix)
            if (p < first_failed.load(std::memory_order_relaxed)) {
                const int r0 = p * piece, r1 = std::min(rows, r0 + piece);
                const size_t at = own.size();
                try {
                    if (codes && own.capacity() == 0) own.reserve((size_t)(rows / threads + piece) * (size_t)(cols / 16 + 4));
                    status[p] = encode_rows(d, tern, cols, r0, r1, &scratch, &own, counts.data() + r0, codes != nullptr);
                    parts.push_back(Part{r0, at, own.size() - at});
                } catch (const std::bad_alloc &) {
                    status[p] = QMOE_E_NOMEM;
                }
                if (status[p] != QMOE_OK) {
                    int seen = first_failed.load(std::memory_order_relaxed);
                    while (p < seen && !first_failed.compare_exchange_weak(seen, p, std::memory_order_relaxed)) {}
                }
            }
            if (pieces_done.fetch_add(1, std::memory_order_acq_rel) + 1 == n_pieces) finish();
        }
        if (!parts.empty() && codes && wait_for_places()) {
            for (const Part &p : parts)
                if (p.n) std::memcpy(codes + row_off[p.r0], own.data() + p.at, p.n * sizeof(uint16_t));
        }
        for (int k = 0; k < started; k++) pthread_join(child[k], nullptr);
    }

    // by the thread that parsed the last piece
    void finish()
    {
        result = place_rows();
        {
            std::lock_guard<std::mutex> lock(mutex);
            places.store(result == QMOE_OK ? 1 : -1, std::memory_order_release);
        }
        known.notify_all();
    }

    qmoe_status place_rows()
    {
        const int failed = first_failed.load(std::memory_order_relaxed);
        if (failed < n_pieces) return status[failed];
        uint64_t total = 0;
        for (int r = 0; r < rows; r++) {
            row_off[r] = (uint32_t)total;
            total += counts[r];
        }
        if (total > 0xFFFFFFFFull) return QMOE_E_LIMIT;
        row_off[rows] = (uint32_t)total;
        *n_codes = (size_t)total;
        return codes && cap < total ? QMOE_E_BUFFER_TOO_SMALL : QMOE_OK;
    }

    // The others are at their last pieces: seldom worth going to sleep for.
    bool wait_for_places()
    {
        for (int k = 0; k < 64; k++) {
            const int v = places.load(std::memory_order_acquire);
            if (v) return v > 0;
            std::this_thread::yield();
        }
        std::unique_lock<std::mutex> lock(mutex);
        known.wait(lock, [&]() { return places.load(std::memory_order_acquire) != 0; });
        return places.load(std::memory_order_acquire) > 0;
    }

    static constexpr size_t kStackBytes = 1 << 20;
    const qmoe_dict *d;
    const int8_t *tern;
    int rows, cols;
    uint16_t *codes;
    size_t cap;
    uint32_t *row_off;
    size_t *n_codes;
    int threads, piece = 0, n_pieces = 0;
    std::vector<uint32_t> counts;      // of a row
    std::vector<qmoe_status> status;   // of a piece
    std::atomic<int> next_piece{0}, pieces_done{0}, first_failed{0x7FFFFFFF}, places{0};  // places: 1 known, -1 there are none
    std::mutex mutex;
    std::condition_variable known;
    qmoe_status result = QMOE_OK;
};

}  // namespace
}  // namespace qmoe

using namespace qmoe;

extern "C" {

const char *qmoe_strerror(qmoe_status s)
{
    switch (s) {
    case QMOE_OK: return "ok";
    case QMOE_E_INVALID_ARG: return "invalid argument";
    case QMOE_E_BUFFER_TOO_SMALL: return "output buffer too small";
    case QMOE_E_BAD_SYMBOL: return "symbol outside the ternary alphabet";
    case QMOE_E_CORRUPT_STREAM: return "corrupt codeword stream";
    case QMOE_E_WORKSPACE: return "workspace missing, misaligned or too small";
    case QMOE_E_HIP: return "HIP call failed";
    case QMOE_E_UNENCODABLE: return "input not encodable with this dictionary";
    case QMOE_E_NOMEM: return "out of host memory";
    case QMOE_E_NO_DEVICE_DICT: return "dictionary not uploaded to the device";
    case QMOE_E_LIMIT: return "size beyond the supported limit";
    default: return "unknown status";
    }
}

qmoe_status qmoe_dict_create(double p0, int max_pairs, int n_entries, qmoe_dict **out)
{
    if (!out || !(p0 > 0.0 && p0 < 1.0) || max_pairs < 1 || max_pairs > 14 || n_entries < 1 ||
        n_entries > kTableEntries)
        return QMOE_E_INVALID_ARG;
    *out = nullptr;
    qmoe_dict *d = new (std::nothrow) qmoe_dict;
    if (!d) return QMOE_E_NOMEM;
    try {
        d->words.assign(2 * (size_t)kTableEntries, 0u);
        const double lp0 = std::log(p0), lq = std::log((1.0 - p0) / 2.0);
        std::priority_queue<Candidate, std::vector<Candidate>, PopsLater> queue;
        queue.push(Candidate{0, 0, 0.0, 0, 0, 0});
        int count = 0;
        while (count < n_entries && !queue.empty()) {
            const Candidate s = queue.top();
            queue.pop();
            if (s.npairs >= 1) {  // never above max_pairs: such candidates are not queued
                pack_words(s.syms, s.npairs, &d->words[2 * (size_t)count]);
                count++;
            }
            if (s.npairs == max_pairs) continue;  // longer sequences can never be appended
            for (int t1 = 0; t1 < 3; t1++)
                for (int t2 = 0; t2 < 3; t2++) {
                    Candidate c = s;
                    c.syms |= ((uint64_t)t1 | ((uint64_t)t2 << 2)) << (4 * s.npairs);
                    c.rank3 = s.rank3 * 9 + (uint64_t)(3 * t1 + t2);
                    c.npairs = (uint8_t)(s.npairs + 1);
                    c.zeros = (uint8_t)(s.zeros + (t1 == 0) + (t2 == 0));
                    c.nonzeros = (uint8_t)(s.nonzeros + (t1 != 0) + (t2 != 0));
                    c.logp = (double)c.zeros * lp0 + (double)c.nonzeros * lq;
                    queue.push(c);
                }
        }
        d->n_entries = count;
        const qmoe_status st = finish_dict(d);
        if (st != QMOE_OK) {
            delete d;
            return st;
        }
    } catch (const std::bad_alloc &) {
        delete d;
        return QMOE_E_NOMEM;
    }
    *out = d;
    return QMOE_OK;
}

qmoe_status qmoe_dict_from_words(const uint32_t *words, int n_entries, qmoe_dict **out)
{
    if (!out || !words || n_entries < 1 || n_entries > kTableEntries) return QMOE_E_INVALID_ARG;
    *out = nullptr;
    qmoe_dict *d = new (std::nothrow) qmoe_dict;
    if (!d) return QMOE_E_NOMEM;
    try {
        d->words.assign(2 * (size_t)kTableEntries, 0u);
        std::memcpy(d->words.data(), words, 2 * sizeof(uint32_t) * (size_t)n_entries);
        d->n_entries = n_entries;
        const qmoe_status st = finish_dict(d);
        if (st != QMOE_OK) {
            delete d;
            return st;
        }
    } catch (const std::bad_alloc &) {
        delete d;
        return QMOE_E_NOMEM;
    }
    *out = d;
    return QMOE_OK;
}

qmoe_status qmoe_dict_words(const qmoe_dict *d, const uint32_t **words, int *n_entries)
{
    if (!d || !words || !n_entries) return QMOE_E_INVALID_ARG;
    *words = d->words.data();
    *n_entries = d->n_entries;
    return QMOE_OK;
}

int qmoe_dict_max_nonzeros(const qmoe_dict *d) { return d ? d->max_nonzeros : QMOE_E_INVALID_ARG; }

size_t qmoe_dict_device_bytes(void) { return kDevDictBytes; }

qmoe_status qmoe_dict_device_order(const qmoe_dict *d, const uint16_t **code_map, const uint32_t **table,
                                   int *n_groups, int *n_table)
{
    if (!d || !code_map || !table || !n_groups || !n_table) return QMOE_E_INVALID_ARG;
    *code_map = d->order_map.empty() ? nullptr : d->order_map.data();
    *table = d->order_table.empty() ? nullptr : d->order_table.data();
    *n_groups = d->n_groups;
    *n_table = (int)d->order_table.size();
    return QMOE_OK;
}

void qmoe_dict_destroy(qmoe_dict *d) { delete d; }

qmoe_status qmoe_encode_host(const qmoe_dict *d, const int8_t *tern, int rows, int cols, uint16_t *codes,
                             size_t codes_cap, uint32_t *row_off, size_t *n_codes)
{
    if (!d || !tern || !row_off || !n_codes || rows < 1 || cols < 2 || (cols & 1))
        return QMOE_E_INVALID_ARG;
    int nthreads = tuning().host_threads;
    if (nthreads <= 0) {
        if (const char *env = std::getenv("QMOE_HOST_THREADS")) nthreads = std::atoi(env);
        if (nthreads <= 0) {
            // A thread for every 30 us of one thread's time (0.36 ns a value, 3 by the trie, and 30 ns a row).  With 1, 4, 8, 16 threads, us: 1024 x 2
            // values 18, 56, 67, 119; 500 x 600 176, 82, 108, 103; 2000 x 1100 877, 294, 213, 202.
            nthreads = (int)std::min(16u, std::max(1u, std::thread::hardware_concurrency()));
            nthreads = (int)std::min((double)nthreads, ((double)rows * cols * (d->rc_depth.empty() ? 3.0 : 0.36) + (double)rows * 30.0) / 30000.0);
        }
    }
    nthreads = std::max(1, std::min(nthreads, (rows + 63) / 64));
    try {
        return HostEncoder(d, tern, rows, cols, codes, codes_cap, row_off, n_codes, nthreads).run();
    } catch (const std::bad_alloc &) {
        return QMOE_E_NOMEM;
    }
}

qmoe_status qmoe_validate_host(const qmoe_dict *d, const uint16_t *codes, const uint32_t *row_off, int rows,
                               int cols)
{
    if (!d || !codes || !row_off || rows < 1 || cols < 2 || (cols & 1)) return QMOE_E_INVALID_ARG;
    if (row_off[0] != 0) return QMOE_E_CORRUPT_STREAM;
    for (int r = 0; r < rows; r++) {
        if (row_off[r + 1] < row_off[r]) return QMOE_E_CORRUPT_STREAM;
        int64_t idx = 0;
        for (uint32_t k = row_off[r]; k < row_off[r + 1]; k++) {
            const uint32_t c = codes[k];
            if ((int)c >= d->n_entries) return QMOE_E_CORRUPT_STREAM;
            idx += 2 * (int64_t)(d->words[2 * (size_t)c] & 15u);
            if (idx > cols) return QMOE_E_CORRUPT_STREAM;
        }
        if (idx != cols) return QMOE_E_CORRUPT_STREAM;
    }
    return QMOE_OK;
}

// ---- lane-interleaved device layout of a codeword stream (see include/qmoe.h) ----
namespace {

// rows [*ra, *rb) of lane g when `rows` rows are dealt evenly over `lanes` lanes
inline void lane_rows(int rows, int lanes, int g, int *ra, int *rb)
{
    const int base = rows / lanes, extra = rows - base * lanes;
    *ra = g * base + std::min(g, extra);
    *rb = *ra + base + (g < extra ? 1 : 0);
}

qmoe_status lane_layout_walk(const uint32_t *row_off, int rows, int lanes, uint32_t *wave_off, size_t *n_pieces)
{
    if (!row_off || rows < 1 || lanes < 64 || (lanes % 64) || lanes > 16320) return QMOE_E_INVALID_ARG;
    unsigned long long total = 0;
    for (int w = 0; w < lanes / 64; w++) {
        if (wave_off) wave_off[w] = (uint32_t)total;
        uint32_t most = 0;
        for (int g = 64 * w; g < 64 * w + 64; g++) {
            int ra, rb;
            lane_rows(rows, lanes, g, &ra, &rb);
            if (row_off[rb] < row_off[ra]) return QMOE_E_CORRUPT_STREAM;
            most = std::max(most, (row_off[rb] - row_off[ra] + 7u) / 8u);
        }
        total += 64ull * most;
        if (total > 0xFFFFFFFFull) return QMOE_E_LIMIT;
    }
    if (wave_off) wave_off[lanes / 64] = (uint32_t)total;
    *n_pieces = (size_t)total;
    return QMOE_OK;
}

}  // namespace

qmoe_status qmoe_lane_layout_size(const uint32_t *row_off, int rows, int lanes, size_t *n_pieces)
{
    if (!n_pieces) return QMOE_E_INVALID_ARG;
    return lane_layout_walk(row_off, rows, lanes, nullptr, n_pieces);
}

qmoe_status qmoe_lane_layout_build(const uint16_t *codes, const uint32_t *row_off, int rows, int lanes, uint16_t *out,
                                   size_t out_pieces, uint32_t *wave_off)
{
    if (!codes || !out || !wave_off) return QMOE_E_INVALID_ARG;
    size_t need = 0;
    const qmoe_status st = lane_layout_walk(row_off, rows, lanes, wave_off, &need);
    if (st != QMOE_OK) return st;
    if (out_pieces < need) return QMOE_E_BUFFER_TOO_SMALL;
    std::memset(out, 0, 16 * need);
    for (int g = 0; g < lanes; g++) {
        int ra, rb;
        lane_rows(rows, lanes, g, &ra, &rb);
        const uint32_t k0 = row_off[ra], n = row_off[rb] - k0;
        const size_t first = (size_t)wave_off[g / 64] + (size_t)(g % 64);  // piece p of the lane sits at first + 64 p
        for (uint32_t i = 0; i < n; i++) out[8 * (first + 64 * (size_t)(i / 8)) + (i % 8)] = codes[k0 + i];
    }
    return QMOE_OK;
}

qmoe_status qmoe_lane_layout_unpack(const uint16_t *pieces, const uint32_t *wave_off, const uint32_t *row_off, int rows,
                                    int lanes, uint16_t *codes, size_t codes_cap)
{
    if (!pieces || !wave_off || !row_off || !codes || rows < 1 || lanes < 64 || (lanes % 64)) return QMOE_E_INVALID_ARG;
    if (codes_cap < row_off[rows]) return QMOE_E_BUFFER_TOO_SMALL;
    for (int g = 0; g < lanes; g++) {
        int ra, rb;
        lane_rows(rows, lanes, g, &ra, &rb);
        const uint32_t k0 = row_off[ra], n = row_off[rb] - k0;
        const size_t first = (size_t)wave_off[g / 64] + (size_t)(g % 64);
        for (uint32_t i = 0; i < n; i++) codes[k0 + i] = pieces[8 * (first + 64 * (size_t)(i / 8)) + (i % 8)];
    }
    return QMOE_OK;
}

qmoe_status qmoe_set_tuning(const char *key, int value)
{
    if (!key) return QMOE_E_INVALID_ARG;
    Tuning &t = tuning();
    if (!std::strcmp(key, "threads")) t.threads = value;
    else if (!std::strcmp(key, "rows_per_item")) t.rows_per_item = value;
    else if (!std::strcmp(key, "token_tile")) t.token_tile = value;
    else if (!std::strcmp(key, "lds_dict_entries")) t.lds_dict_entries = value;
    else if (!std::strcmp(key, "grid_per_cu")) t.grid_per_cu = value;
    else if (!std::strcmp(key, "host_threads")) t.host_threads = value;
    else if (!std::strcmp(key, "blocks_first")) t.blocks_first = value;
    else if (!std::strcmp(key, "blocks_second")) t.blocks_second = value;
    else if (!std::strcmp(key, "mfma_min_tokens")) t.mfma_min_tokens = value;
    else if (!std::strcmp(key, "overlap")) t.overlap = value;
    else return QMOE_E_INVALID_ARG;
    return QMOE_OK;
}

qmoe_status qmoe_hook_set(const char *key, int value)
{
    if (!key) return QMOE_E_INVALID_ARG;
    Tuning &t = tuning();
    if (!std::strcmp(key, "phases")) t.phases = value;
    else if (!std::strcmp(key, "stage_out")) t.stage_out = value;
    else if (!std::strcmp(key, "rows")) t.rows = value;
    else if (!std::strcmp(key, "encode_rows")) t.encode_rows = value;
    else return QMOE_E_INVALID_ARG;
    return QMOE_OK;
}

}  // extern "C"
