// Row-gathered fp32 GEMM with bias/ReLU epilogue on MFMA 16x16x4:
//   C[m][n] = act(bias[n] + sum_k A[row(m)][k] B[n][k]),  row(m) = row_map ? row_map[m] : m
// Used where the contraction is small and dense: the node encoders
// (K = raw feature width) and the decoder projections (K = f).  Any K and N
// (guarded loads); a negative row_map entry reads a zero row.
//
// In the op encoder C (rows x f) is the largest stream.  A block covers 128
// columns (all of C's row for f <= 128, so A is read once), and the epilogue
// stages the finished tile in LDS and writes whole rows with 16-byte stores
// when C's pitch and alignment allow.
#include <algorithm>

#include "gemm_small.hpp"

namespace tag {
namespace {

using namespace sgemm;

template <int SM, int SK, int WM>
__global__ void __launch_bounds__(256) small_gemm(SmallGemm G, int vec) {
    __shared__ __align__(16) float lds[Tile<SM, SK, WM>::LDS];
    block<SM, SK, WM>(G, vec, blockIdx.x, blockIdx.y, lds,
                      [&](int64_t m) { return G.row_map ? G.row_map[m] : (int32_t)m; });
}

// Node encoders of many rows (K <= 64, columns a multiple of 64): wavefronts
// that run over 16-row units on their own, the weights of the block's NJ * 16
// columns in LDS as exact bf16 split planes (staged once per block, so blocks
// are persistent), the unit's raw features read straight into operand
// registers (lane l: row l % 16, features 8 (l / 16) .. + 7 of a 32-wide step)
// with the next unit's in flight, eight part products per step on bf16 MFMAs
// (the fp32 contraction up to fp32 rounding, at half of the matrix-core time of
// 16x16x4 products; the two more than the transform's six cost nothing
// measurable beside the writes).  Products are taken as
// C^T, so a lane owns four columns of its row; rows leave through the
// wavefront's LDS stage as whole 256-byte segments.  Bound by the HBM write of
// C.  K = 42: 768,000 rows x 256 fp32 columns 330 -> 221 us (4.1 TB/s),
// 2,560,000 x 256 bf16 860 -> 508 us, 6,144,000 x 128 fp32 1.25 -> 0.92 ms (4.5
// TB/s) against 64-row blocks on 16x16x4 products.
template <int NJ, int KP, bool BF>
__global__ void __launch_bounds__(512, 4) enc_rows(SmallGemm G, int halves) {
    constexpr int NS = (KP + 31) / 32;   // 32-wide steps; KP = 32, 48 or 64 features have room in LDS
    // plane row stride (bf16 elements): rows 16-byte aligned, eight rows on distinct banks
    constexpr int KS = KP == 48 ? 48 : KP + 8;
    constexpr int SP = 64 + 4;   // stage row stride (floats)
    __shared__ __attribute__((aligned(16))) uint16_t W[3][NJ * 16 * KS + 8];   // + eight zeros
    __shared__ __attribute__((aligned(16))) float bias[NJ * 16], stage[8][16 * SP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
    // the column halves of a row share an XCD (and its L2)
    const uint32_t lb = xcd_swizzle(blockIdx.x, gridDim.x);
    const int n0 = (int)(lb % halves) * NJ * 16, K = G.K;
    {
        constexpr int NP = NJ * 16 * KP / 2 / 512;   // weight pairs per thread, their loads issued together
        float w[NP][2];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int i = threadIdx.x + 512 * q, k = 2 * (i % (KP / 2));
            const float *b = G.B + (int64_t)(n0 + i / (KP / 2)) * G.ldb;
            w[q][0] = k < K ? b[k] : 0.f;
            w[q][1] = k + 1 < K ? b[k + 1] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int i = threadIdx.x + 512 * q, o = i / (KP / 2) * KS + 2 * (i % (KP / 2));
            unsigned p[3];
            split3(w[q][0], w[q][1], p);
#pragma unroll
            for (int z = 0; z < 3; ++z) *reinterpret_cast<unsigned *>(&W[z][o]) = p[z];
        }
    }
    if (threadIdx.x < 24) W[threadIdx.x / 8][NJ * 16 * KS + threadIdx.x % 8] = 0;
    for (int i = threadIdx.x; i < NJ * 16; i += 512) bias[i] = G.bias ? G.bias[n0 + i] : 0.f;
    __syncthreads();
    const int64_t units = (G.rows + 15) / 16, step = (int64_t)(gridDim.x / halves) * 8;
    float x[NS][8];
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // rows of K floats: 4-byte aligned
    auto load = [&](int64_t unit) {
        const int64_t r = unit * 16 + lr;
        const float *p = G.A + (r < G.rows ? r : G.rows - 1) * G.lda;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 32 * s + 8 * lg;
            if (K >= 32 * (s + 1)) {
                const f4u a = *reinterpret_cast<const f4u *>(p + k), b = *reinterpret_cast<const f4u *>(p + k + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[s][i] = a[i]; x[s][4 + i] = b[i]; }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[s][i] = k + i < K ? p[k + i] : 0.f;
            }
        }
    };
    // the lane's slice of a weight row in each step (past KP: the zeros)
    int woff[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) woff[s] = 32 * s + 8 * lg < KP ? lr * KS + 32 * s + 8 * lg : -1;
    int64_t unit = (int64_t)(lb / halves) * 8 + wave;
    if (unit < units) load(unit);
    float *st = stage[wave];
    for (; unit < units; unit += step) {
        // (the weights are read afresh for every unit: held in registers across
        // the loop they would not fit)
        asm volatile("" ::: "memory");
        bf8 a[NS][3];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            unsigned p[4][3];
#pragma unroll
            for (int i = 0; i < 4; ++i) split3(x[s][2 * i], x[s][2 * i + 1], p[i]);
#pragma unroll
            for (int z = 0; z < 3; ++z) a[s][z] = as_bf8(p[0][z], p[1][z], p[2][z], p[3][z]);
        }
        if (unit + step < units) load(unit + step);
        // Smallest first, the large products of every step last.  With six products,
        // step by step, more pre-activations near zero fell on the wrong side of the
        // ReLU: encoder gradients of 64 candidates of 1,200 ops, 16 seeds, were 9.3e-6
        // from float64 (geometric mean) against 7.1e-6 on fp32 products, 7.7e-6 so.
        constexpr int NP = 8, PW[NP] = {2, 1, 2, 1, 0, 1, 0, 0}, PX[NP] = {1, 2, 0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int hh = 0; hh < NJ / 4; ++hh) {
            f4 acc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[j] = f4{0.f, 0.f, 0.f, 0.f};
                bf8 b[NS][3];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const int o = woff[s] < 0 ? NJ * 16 * KS : woff[s] + (4 * hh + j) * 16 * KS;
#pragma unroll
                    for (int z = 0; z < 3; ++z) b[s][z] = *reinterpret_cast<const bf8 *>(&W[z][o]);
                }
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[s][PW[p]], a[s][PX[p]], acc[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 b = *reinterpret_cast<const float4 *>(&bias[(4 * hh + j) * 16 + 4 * lg]);
                float4 v = make_float4(acc[j][0] + b.x, acc[j][1] + b.y, acc[j][2] + b.z, acc[j][3] + b.w);
                if (G.relu) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
                *reinterpret_cast<float4 *>(st + lr * SP + 16 * j + 4 * lg) = v;
            }
            // (a wavefront's own stage: its writes come before its reads)
            if constexpr (!BF) {
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int rr = 4 * it + lg;
                    const float4 v = *reinterpret_cast<const float4 *>(st + rr * SP + 4 * lr);
                    if (unit * 16 + rr < G.rows)
                        *reinterpret_cast<float4 *>(static_cast<float *>(G.C) + (unit * 16 + rr) * G.ldc + n0 + 64 * hh + 4 * lr) = v;
                }
            } else {
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int rr = 8 * it + (lane >> 3), c = 8 * (lane & 7);
                    const f4 lo = *reinterpret_cast<const f4 *>(st + rr * SP + c);
                    const f4 hi = *reinterpret_cast<const f4 *>(st + rr * SP + c + 4);
                    if (unit * 16 + rr < G.rows)
                        *reinterpret_cast<u4v *>(static_cast<uint16_t *>(G.C) + (unit * 16 + rr) * G.ldc + n0 + 64 * hh + c) =
                            u4v{pack_bf2(lo[0], lo[1]), pack_bf2(lo[2], lo[3]), pack_bf2(hi[0], hi[1]), pack_bf2(hi[2], hi[3])};
                }
            }
        }
    }
}

template <int NJ, int KP>
void launch_enc(const SmallGemm &G, hipStream_t st) {
    const int halves = G.N / (NJ * 16);
    const int64_t units = (G.rows + 15) / 16;
    // two blocks of eight wavefronts per CU
    const int64_t slots = std::min<int64_t>((units + 7) / 8, std::max(1, 512 / halves));
    const unsigned blocks = (unsigned)(slots * halves);
    if (G.c_bf16) enc_rows<NJ, KP, true><<<blocks, 512, 0, st>>>(G, halves);
    else enc_rows<NJ, KP, false><<<blocks, 512, 0, st>>>(G, halves);
}

template <int NJ>
void launch_enc_k(const SmallGemm &G, hipStream_t st) {
    if (G.K <= 32) launch_enc<NJ, 32>(G, st);
    else if (G.K <= 48) launch_enc<NJ, 48>(G, st);
    else launch_enc<NJ, 64>(G, st);
}

// rows from which an encoder takes enc_rows: at least one unit for each
// wavefront of an eighth of the chip; below, staging the weights costs more than
// the rows (1,024 rows: 4.7 us in 16-row blocks of small_gemm)
constexpr int64_t kEncRows = 8192;

template <int SM, int SK, int WM>
void launch_tile(const SmallGemm &G, int vec, hipStream_t st) {
    dim3 grid((unsigned)((G.rows + SM - 1) / SM), (unsigned)((G.N + SN - 1) / SN));
    small_gemm<SM, SK, WM><<<grid, 256, 0, st>>>(G, vec);
}

}  // namespace

namespace {
enum class Route { kFew, kTiles, kEncoder, kSplit };

Route route_of(const SmallGemm &G) {
    // wide contractions of many rows (the decoder's projections for a whole
    // group of every candidate): split products (42,496 + 16,384 rows: 70
    // against 112 us).  Fewer rows than 128 blocks of 64 leave the chip idle
    // either way and keep the 16-row blocks.
    if (G.K >= 64 && G.rows >= 8192 && !G.c_bf16) return Route::kSplit;
    if (G.K <= 64 && G.rows >= kEncRows && vec_ok(G) && !G.row_map && G.N % 64 == 0) return Route::kEncoder;
    // fewer than 256 blocks of 64 rows (the decoder projections, the device
    // encoder): 16-row blocks and 32-wide k-chunks, so that more compute units
    // work and fewer dependent load rounds separate the chunks
    return (G.rows + 63) / 64 < 256 ? Route::kFew : Route::kTiles;
}
}  // namespace

bool small_gemm_few(const SmallGemm &G) { return route_of(G) == Route::kFew; }

void launch_small_gemm(const SmallGemm &G, hipStream_t st) {
    if (G.rows <= 0 || G.N <= 0) return;
    switch (route_of(G)) {
        case Route::kSplit: {
            SplitGemm S{};
            S.A = G.A; S.lda = G.lda; S.row_map = G.row_map;
            S.B = G.B; S.ldb = G.ldb;
            S.M = G.rows; S.N = G.N; S.K = S.k_per = G.K;
            S.ones_col = -1;
            S.bias = G.bias; S.relu = G.relu;
            S.C = static_cast<float *>(G.C); S.ldc = G.ldc;
            launch_split_gemm(S, true, true, 1, st);
            break;
        }
        case Route::kEncoder:
            if (G.N % 128 == 0) launch_enc_k<8>(G, st);
            else launch_enc_k<4>(G, st);
            break;
        case Route::kFew: launch_tile<kFewM, kFewK, 1>(G, vec_ok(G), st); break;
        case Route::kTiles: launch_tile<64, 16, 2>(G, vec_ok(G), st); break;
    }
}

}  // namespace tag
