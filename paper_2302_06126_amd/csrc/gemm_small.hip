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
// columns in LDS (staged once per block, so blocks are persistent), the unit's
// raw features read straight into operand registers with the next unit's in
// flight.  fp32 16x16x4 products in the order of the 16-row blocks (k ascending,
// then the bias), so a row's values do not depend on how many rows a call has.
// Products are taken as C^T, so a lane owns four columns of its row; rows leave
// through the wavefront's LDS stage as whole 256-byte segments.
// Bound by the HBM write of C where C outgrows the last-level cache, with the matrix
// cores busy for about two thirds of it: against 64-row blocks, K = 42: 2,560,000
// rows x 256 bf16 columns 848 -> 598 us, fp32 1.03 -> 0.86 ms (3.1 TB/s), 1,500,000 x
// 128 fp32 299 -> 249 us.  (On exact bf16 splits the last was 237 us and the first
// 548, but sums in another order round other hidden values to the next bf16, and an
// infinite feature became a NaN and by the ReLU a zero.)
template <int NJ, int KP, bool BF>
__global__ void __launch_bounds__(512, 4) enc_rows(SmallGemm G, int halves) {
    constexpr int NS = KP / 4;   // products per 16 x 16 tile; KP = 16, 32, 48 or 64 features
    // LDS weight row of a column: for each lane group lg its operands k = lg, 4 + lg, 8 + lg, ...
    // one after the other (read four at a time); the stride keeps eight rows on distinct banks
    constexpr int WS = KP + 4;
    constexpr int SP = 64 + 4;   // stage row stride (floats)
    __shared__ __attribute__((aligned(16))) float W[NJ * 16 * WS], bias[NJ * 16], stage[8][16 * SP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
    // the column halves of a row share an XCD (and its L2)
    const uint32_t lb = xcd_swizzle(blockIdx.x, gridDim.x);
    const int n0 = (int)(lb % halves) * NJ * 16, K = G.K;
    {
        constexpr int NP = NJ * 16 * KP / 512;   // weights per thread, their loads issued together
        float w[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int i = threadIdx.x + 512 * q, k = i % KP;
            w[q] = k < K ? G.B[(int64_t)(n0 + i / KP) * G.ldb + k] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int i = threadIdx.x + 512 * q, k = i % KP;
            W[i / KP * WS + (k & 3) * NS + (k >> 2)] = w[q];
        }
    }
    for (int i = threadIdx.x; i < NJ * 16; i += 512) bias[i] = G.bias ? G.bias[n0 + i] : 0.f;
    __syncthreads();
    const int64_t units = (G.rows + 15) / 16, step = (int64_t)(gridDim.x / halves) * 8;
    // lane l's operands: row l % 16 of the unit, features l / 16, 4 + l / 16, ... (zero from K on)
    float x[NS];
    auto load = [&](int64_t unit) {
        const int64_t r = unit * 16 + lr;
        const float *p = G.A + (r < G.rows ? r : G.rows - 1) * G.lda;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 4 * s + lg;
            x[s] = k < K ? p[k] : 0.f;
        }
    };
    const float *wl = W + lr * WS + lg * NS;
    int64_t unit = (int64_t)(lb / halves) * 8 + wave;
    if (unit < units) load(unit);
    float *st = stage[wave];
    for (; unit < units; unit += step) {
        // (the weights are read afresh for every unit: held in registers across
        // the loop they would not fit)
        asm volatile("" ::: "memory");
        float a[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) a[s] = x[s];
        if (unit + step < units) load(unit + step);
#pragma unroll
        for (int hh = 0; hh < NJ / 4; ++hh) {
            f4 acc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s4 = 0; s4 < NS; s4 += 4) {
                f4 b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const f4 *>(wl + (4 * hh + j) * 16 * WS + s4);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][s], a[s4 + s], acc[j], 0, 0, 0);
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
    if (G.K <= 16) launch_enc<NJ, 16>(G, st);
    else if (G.K <= 32) launch_enc<NJ, 32>(G, st);
    else if (G.K <= 48) launch_enc<NJ, 48>(G, st);
    else launch_enc<NJ, 64>(G, st);
}

// Rows from which an encoder takes enc_rows.  64 columns: where the 16-row
// blocks end (20,000 to 1,500,000 rows of 8 to 64 features, 64-row tiles | here:
// 42 features 14.9 | 10.7 us at 60,000, 37.6 | 25.1 at 200,000, 247 | 152 at
// 1,500,000; no case slower).  More columns: where the writes of C no longer stay
// in the last-level cache (42 features, 128 columns 31 | 34 us at 140,000,
// 74 | 77 at 400,000, 114 | 103 at 550,000; 256 columns 94 | 101 at 270,000,
// 227 | 193 at 550,000; bf16 27 | 31 for 140,000 x 128, 171 | 141 for 550,000 x
// 256); with fewer, wavefronts of two or three units leave the chip uneven.
inline int64_t enc_rows_from(int N) { return N <= 64 ? 16384 : int64_t(1) << 19; }

template <int SM, int SK, int WM>
void launch_tile(const SmallGemm &G, int vec, hipStream_t st) {
    dim3 grid((unsigned)((G.rows + SM - 1) / SM), (unsigned)((G.N + SN - 1) / SN));
    small_gemm<SM, SK, WM><<<grid, 256, 0, st>>>(G, vec);
}

}  // namespace

namespace {
enum class Route { kFew, kTiles, kEncoder, kSplit };

Route route_of(const SmallGemm &G) {
    // encoders (the contractions with a ReLU) keep fp32 products in one order
    // whatever their size; their kernel takes whole 64-column blocks of aligned rows
    if (G.relu && G.K <= 64 && G.rows >= enc_rows_from(G.N) && vec_ok(G) && !G.row_map && G.N % 64 == 0)
        return Route::kEncoder;
    // wide contractions of many rows (the decoder's projections for a whole
    // group of every candidate): split products (42,496 + 16,384 rows: 70
    // against 112 us).  Fewer rows than 128 blocks of 64 leave the chip idle
    // either way and keep the 16-row blocks.
    if (!G.relu && !G.bias && G.K >= 64 && G.rows >= 8192 && !G.c_bf16) return Route::kSplit;
    // fewer than 256 blocks of 64 rows (the decoder projections, the encoders of
    // small calls): 16-row blocks and 32-wide k-chunks, so that more compute units
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
