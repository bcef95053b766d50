// What a forward pass prepares once for its layers, as device code of the
// prologue launch (forward.hip).
#pragma once

#include "agg_common.hpp"

namespace tag {

// omask[r][u] = (present, bits) over the local devices of u's topology.
// A block takes (op tile t, kMaskCands candidates from r0): the tile's op<-dev CSR range
// is read once for the group; four lanes per op row walk its entries and OR
// device bits in registers, and the four partial masks meet by shuffles.
constexpr int kMaskCands = 4;
static_assert(kMaskCands == 4 && kOpTile * 4 == 256, "one lane per quarter row and per stored candidate");

__device__ __forceinline__ void pack_op_masks(const AggArgs &A, int32_t t, int32_t r0) {
    typedef unsigned long long u64;
    const int32_t u0 = A.tiles[3 * t], nu = A.tiles[3 * t + 1], g = A.tiles[3 * t + 2];
    const int32_t d0 = A.dev_off[g];
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;   // op row of the tile, quarter
    u64 pres = 0ull, bits[kMaskCands];
#pragma unroll
    for (int k = 0; k < kMaskCands; ++k) bits[k] = 0ull;
    if (i < nu) {
        const int32_t e1 = A.rp[1][u0 + i + 1];
        for (int32_t e = A.rp[1][u0 + i] + q; e < e1; e += 4) {
            const u64 m = 1ull << (A.col[1][e] - d0);
            const int64_t id = A.eid[1][e];
            pres |= m;
#pragma unroll
            for (int k = 0; k < kMaskCands; ++k)
                if (r0 + k < A.R && A.x_od[(int64_t)(r0 + k) * A.s_od + id]) bits[k] |= m;
        }
    }
    // lanes 4i .. 4i + 3 of one wavefront hold the quarters of row i
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
        pres |= __shfl_xor(pres, o);
#pragma unroll
        for (int k = 0; k < kMaskCands; ++k) bits[k] |= __shfl_xor(bits[k], o);
    }
    if (i < nu && r0 + q < A.R) {   // lane q stores candidate r0 + q
        u64 b = bits[0];
#pragma unroll
        for (int k = 1; k < kMaskCands; ++k) b = q == k ? bits[k] : b;
        const int64_t mi = 2 * ((int64_t)(r0 + q) * A.n_op + u0 + i);
        A.omask[mi] = pres;
        A.omask[mi + 1] = b;
    }
}

// The op tiles' descriptors, in parts of kOpTile / A.tile_sub rows (so an
// op-destination block finds its CSR range and device group in one load
// round), and the op<-op edge features in CSR order (so it loads them without
// the edge-id gather): items i0, i0 + stride, ...
__device__ __forceinline__ void prep_tiles_x(const AggArgs &A, int64_t nnz0, int32_t xrep, int64_t i0, int64_t stride) {
    const int64_t nt = (int64_t)A.n_tiles * A.tile_sub, n = nt + (int64_t)xrep * nnz0;
    const int32_t rows = kOpTile / A.tile_sub;
    for (int64_t i = i0; i < n; i += stride) {
        if (i < nt) {
            const int32_t t = (int32_t)i / A.tile_sub, part = (int32_t)i % A.tile_sub;
            const int32_t g = A.tiles[3 * t + 2], left = A.tiles[3 * t + 1] - part * rows;
            const int32_t nu = left < 0 ? 0 : left < rows ? left : rows;
            const int32_t u0 = A.tiles[3 * t] + (nu > 0 ? part * rows : 0);
            const int32_t eb = A.rp[0][u0], d0 = A.dev_off[g];
            int32_t *o = A.tile_ext + 8 * i;
            o[0] = u0; o[1] = nu; o[2] = g; o[3] = eb; o[4] = A.rp[0][u0 + nu] - eb;
            o[5] = d0; o[6] = A.dev_off[g + 1] - d0; o[7] = 0;
        } else {
            const int64_t j = i - nt, r = j / nnz0, e = j % nnz0;
            A.xcsr[j] = A.x_oo[r * A.s_oo + A.eid[0][e]];
        }
    }
}

}  // namespace tag
