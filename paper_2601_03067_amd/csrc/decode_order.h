// Which workgroup of the paged decode kernels (decode.hip) works on what; arithmetic alone, for the device and for the host.
#pragma once
#include "common.h"

namespace kvfuse {

// What this workgroup works on.  Workgroups go to the eight XCDs in turn, and each XCD has an L2 of its own: all that read the
// blocks of one (layer, KV head) are put on one XCD, eight such groups at a time, requests side by side before the next split of them, so that what
// requests share is read while it is there.  The second half of the requests starts at the last split that has tokens: else
// a common prefix, which comes out of L2, and what is each request's own, which does not, would be read one after the other (20 requests
// of 1742 tokens, 16 groups, 31.4 / 28.5; from the last split whether it has tokens or not, 17 ragged requests 399 / 389).  The groups
// that are left, fewer than eight, alternate (a power of two of them then also shares as few XCDs as it can).
// In the order of the grid several splits scatter a group over all XCDs, and of two splits every other XCD gets the second, which is empty for
// most of ragged requests.  us, in the order of the grid / like this: 48 ragged requests of 512 to 8192 tokens, 8 groups, 142 / 135;
// 18 requests of 5797 tokens, 16 groups, 119 / 99; 2 of 27945 tokens, 16 groups, 72.5 / 55.5; binary32, 17 ragged ones up to 3812 tokens, 96 groups
// of four KV heads a layer, 492 / 389; about the line below, 24 requests of 1024 tokens, 8 groups, 21.4 / 18.4, of 1200 21.3 / 21.4, of 1500
// 26.9 / 26.4, of 2000 31.6 / 30.4; 11 groups 27.2 / 23.1, 29.5 / 26.9, 34.4 / 31.0, 44.4 / 39.5; one request level.  Contexts below 1024 tokens stay in the grid's order (22 requests of 760 tokens, 4 groups, 15.3 /
// 15.9; 494 of 107, 44 groups, 157 / 163), and so do all-head blocks, whose tokens all heads of a layer read (7 requests of 10813 tokens
// 80 / 82; 139 of 438 20.8 / 18.9), and three, five, six or seven groups, which would not keep to an XCD (three: 38.7 / 40.3).
// (Fewer than 2^32 workgroups: neither the layers nor the requests' KV heads of a call are more than 65535, and splits are taken where
// there are fewer than 2048 of both.)
// The lengths are the device's, and may have outgrown the max_blocks that the grid and the states' room are sized for: such a request
// takes its splits in either order like any other, and what lies beyond them is not read.
struct DecodeOrder {
    bool by_xcd;
    uint32_t nsplit;
    GroupsByXcd groups;
    Divisor requests, heads, split_tokens;

    struct Place {
        int split, b, kvh, li;
    };
    // of workgroup (x, y, z) of a grid of splits, requests x KV heads, layers
    __host__ __device__ __forceinline__ Place place(uint32_t x, uint32_t y, uint32_t z, const int32_t *ctx_len) const
    {
        uint32_t split = x, b, li = z, kvh;
        if (by_xcd) {
            uint32_t group, rest;
            groups.place(x + nsplit * (y + requests.d * heads.d * z), group, rest);
            split = requests.of(rest);
            b = rest - split * requests.d;
            if (2 * b >= requests.d) {
                const int32_t last = ctx_len[b] > 0 ? ctx_len[b] - 1 : 0;
                const uint32_t before = split_tokens.of((uint32_t)last);           // splits before the last one with tokens
                const uint32_t full = before < nsplit ? before : nsplit - 1;
                split = split > full ? split : full - split;
            }
            li = heads.of(group);
            kvh = group - li * heads.d;
        } else {
            b = heads.of(y);
            kvh = y - b * heads.d;
        }
        return {(int)split, (int)b, (int)kvh, (int)li};
    }
};

}  // namespace kvfuse
