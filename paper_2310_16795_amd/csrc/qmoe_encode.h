// What the launch code hands to the device encoder (qmoe_encode.hip).  Not part of the C ABI.
#pragma once

#include "qmoe_dev.h"

namespace qmoe {

struct EncodeArgs {
    const int8_t *tern;   // [rows][cols], values -1 / 0 / +1
    int rows, cols;
    const int32_t *child, *code;
    uint32_t *row_off;    // [rows+1]
    uint16_t *codes;
    unsigned long long codes_cap;
    int *status;          // [2]: first error (qmoe_status, 0 = none), a row it happened in
};

struct RunCoderArgs {
    EncodeArgs e;
    const uint32_t *depth;   // depth tables (kRcDepthBytes bytes), nullptr: the dictionary has no run coder
    const uint32_t *first;   // [kRcPatterns]
    const uint16_t *codes;   // codeword of pattern i with D pairs: codes[first[i] + D]
    int depth0;              // depth of the pattern without a non-zero
    int cus, max_lds;
    // launch shape, set by launch_encode
    int lanes_log2;          // lanes per row
    int seg_pairs;           // pairs a lane parses (a multiple of 32)
    int row0, row_end;       // rows of the launch: whole groups of 64 >> lanes_log2, but for the last
    int groups, groups_per_wg, groups_extra;  // (the first groups_extra tickets stand for a group more)
    int bit_words, mask_words, row_lds;  // LDS of a row: (non-zero, sign) words, boundary words, bytes together
};

constexpr int kRcTicketBytes = 16;  // LDS behind the depth tables: the workgroup's ticket

qmoe_status launch_encode(const RunCoderArgs &a, hipStream_t s);

}  // namespace qmoe
