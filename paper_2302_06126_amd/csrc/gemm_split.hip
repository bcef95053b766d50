// General fp32 GEMM on the bf16 matrix cores: C[m][n] = sum_k a(m, k) b(n, k),
// both operands split exactly into three bf16 parts as
// they are staged, six part products per 16x16x32 step (the fp32 contraction
// up to fp32 rounding, as in the relation transform, at 3/8 of the matrix-core
// time of fp32 16x16x4 products).  Used where K is at least one 32-wide step:
// the decoder's projections of many rows and the training step's gradients of
// the hidden rows and of the weights (split over K).  Operands and results that
// are not finite give what fp32 products give.
//
// Bound by the staging (loads, splits, LDS) more than by the products: a block
// of TM x TN outputs keeps one k-step of split planes in LDS (48 KiB at 128 x
// 128, three blocks per CU) with the next step's loads in flight, so that
// other blocks' products cover it.  Decoder projections of 42,496 and 16,384
// rows (K = 256, 256 columns): 112 us on fp32 16x16x4 products (small_gemm),
// 70 us here.
#include "agg_common.hpp"

namespace tag {
namespace {

constexpr int BK = 32;

// planes of R rows x 32 k: unpadded 64-byte rows, chunk c of row r at c ^ sw(r)
__device__ __forceinline__ int sw(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }

// Eight consecutive k of one row per (thread, q).  KC: the operand is stored
// [row][k]; four threads cover a row's step.  Otherwise [k][row]: the threads
// of a wavefront read consecutive rows.
template <int ROWS, bool KC>
struct Stager {
    static constexpr int NQ = ROWS * 4 / 256;   // 8-wide chunks per thread
    static_assert(NQ >= 1, "at least 64 rows");
    float x[NQ][8];
    static __device__ __forceinline__ int row(int q) {
        const int i = threadIdx.x + 256 * q;
        return KC ? i >> 2 : i % ROWS;
    }
    static __device__ __forceinline__ int chunk(int q) {
        const int i = threadIdx.x + 256 * q;
        return KC ? i & 3 : i / ROWS;
    }
    // src(q): the row's first element (nullptr: a row of zeros); one(q): a row of ones
    template <typename Src, typename One>
    __device__ __forceinline__ void load(Src src, One one, int64_t ld, int64_t k0, int64_t ke, bool vec) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int64_t k = k0 + 8 * chunk(q);
            const float *p = src(q);
            const float fill = one(q) ? 1.f : 0.f;
            if (KC) {
                if (p && vec && k + 8 <= ke) {
                    const float4 a = *reinterpret_cast<const float4 *>(p + k);
                    const float4 b = *reinterpret_cast<const float4 *>(p + k + 4);
                    x[q][0] = a.x; x[q][1] = a.y; x[q][2] = a.z; x[q][3] = a.w;
                    x[q][4] = b.x; x[q][5] = b.y; x[q][6] = b.z; x[q][7] = b.w;
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[q][i] = k + i < ke ? (p ? p[k + i] : fill) : 0.f;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[q][i] = k + i < ke ? (p ? p[(k + i) * ld] : fill) : 0.f;
            }
        }
    }
    // neg: sign bit to flip in every element
    __device__ __forceinline__ void store(uint16_t (*planes)[ROWS * BK], unsigned neg) const {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            unsigned p[4][3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = __uint_as_float(__float_as_uint(x[q][2 * i]) ^ neg);
                const float b = __uint_as_float(__float_as_uint(x[q][2 * i + 1]) ^ neg);
                split3(a, b, p[i]);
            }
            const int off = row(q) * BK + 8 * (chunk(q) ^ sw(row(q)));
#pragma unroll
            for (int z = 0; z < 3; ++z)
                *reinterpret_cast<u4v *>(&planes[z][off]) = u4v{p[0][z], p[1][z], p[2][z], p[3][z]};
        }
    }
};

// four wavefronts, each half of the tile's rows x half of its columns
template <int TM, int TN, bool AKC, bool BKC>
__global__ void __launch_bounds__(256) gemm_s3(SplitGemm G) {
    constexpr int WM = 2, WN = 4 / WM, NI = TM / WM / 16, NJ = TN / WN / 16;
    __shared__ __attribute__((aligned(16))) uint16_t As[3][TM * BK], Bs[3][TN * BK];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / WN, wn = wave % WN;
    const int64_t m0 = (int64_t)blockIdx.x * TM, n0 = (int64_t)blockIdx.y * TN;
    const int64_t kb = (int64_t)blockIdx.z * G.k_per, ke = G.K < kb + G.k_per ? G.K : kb + G.k_per;
    const bool vec = G.vec != 0;
    Stager<TM, AKC> sa;
    Stager<TN, BKC> sb;
    // each thread's rows (nullptr past the end or for a negative row_map entry)
    const float *pa[Stager<TM, AKC>::NQ], *pb[Stager<TN, BKC>::NQ];
    bool ob[Stager<TN, BKC>::NQ];
#pragma unroll
    for (int q = 0; q < Stager<TM, AKC>::NQ; ++q) {
        int64_t m = m0 + sa.row(q);
        if (m >= G.M) m = -1;
        else if (G.row_map) m = G.row_map[m];
        pa[q] = m < 0 ? nullptr : G.A + (AKC ? m * G.lda : m);
    }
#pragma unroll
    for (int q = 0; q < Stager<TN, BKC>::NQ; ++q) {
        const int64_t n = n0 + sb.row(q);
        ob[q] = n == G.ones_col;
        pb[q] = n < G.N && !ob[q] ? G.B + (BKC ? n * G.ldb : n) : nullptr;
    }
    auto load = [&](int64_t k0) {
        sa.load([&](int q) { return pa[q]; }, [](int) { return false; }, G.lda, k0, ke, vec);
        sb.load([&](int q) { return pb[q]; }, [&](int q) { return ob[q]; }, G.ldb, k0, ke, vec);
    };
    f4 acc[NJ][NI];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[j][i] = f4{0.f, 0.f, 0.f, 0.f};
    int aoff[NI], boff[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int r = wm * (TM / WM) + i * 16 + (lane & 15);
        aoff[i] = r * BK + 8 * ((lane >> 4) ^ sw(r));
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = wn * (TN / WN) + j * 16 + (lane & 15);
        boff[j] = r * BK + 8 * ((lane >> 4) ^ sw(r));
    }
    // Contractions over rows (A not k-contiguous) are long, split, and of terms
    // that cancel.  The bf16 products round their sums towards minus infinity, a
    // bias that grows with the number of steps where the sum grows with its root,
    // so every other step is taken with A and the accumulators negated (both
    // exact; the first step's sign alternates between splits).  A gradient-like
    // 300,000 x 128 by 300,000 x 64, relative to float64: 8.3e-7 (mean -7.8e-7 of
    // the rms) without, 3.5e-7 (4e-9) with, 4.2e-7 on fp32 products; 640,000 x 256
    // by 128 3.0e-6, 1.0e-6, 1.3e-6.  It costs 2 to 6% (14% at 64 x 64 tiles: 76,800 x
    // 256 by 43, 27.9 | 31.8 us, 37.5 on fp32 products).  Over channels (at most
    // 1,024 of them) the splits are nearer than fp32 products either way.
    constexpr bool ALT = !AKC;
    unsigned par = ALT ? (unsigned)blockIdx.z & 1u : 0u;
    auto negate = [&] {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) acc[j][i] = -acc[j][i];
    };
    if (kb < ke) load(kb);
    for (int64_t k0 = kb; k0 < ke; k0 += BK) {
        sa.store(As, ALT ? par << 31 : 0u);
        sb.store(Bs, 0u);
        if (ALT && k0 != kb) negate();
        __syncthreads();
        if (k0 + BK < ke) load(k0 + BK);
        bf8 a[NI][3];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int z = 0; z < 3; ++z) a[i][z] = *reinterpret_cast<const bf8 *>(&As[z][aoff[i]]);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            bf8 b[3];
#pragma unroll
            for (int z = 0; z < 3; ++z) b[z] = *reinterpret_cast<const bf8 *>(&Bs[z][boff[j]]);
            constexpr int PB[6] = {2, 1, 0, 1, 0, 0}, PA[6] = {0, 1, 2, 0, 1, 0};   // smallest first
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[PB[p]], a[i][PA[p]], acc[j][i], 0, 0, 0);
        }
        __syncthreads();
        par ^= 1u;
    }
    if (ALT && par == 0u) negate();   // the last step's sign was 1
    // Infinities and NaN do not survive a split (inf - inf in its parts), nor do
    // values that round to an infinite bf16: outputs that are not finite are
    // stored and then taken again, below.
    auto finite = [](float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; };
    bool redo = false;
    // lane l of block (j, i): row 16 i + l % 16, columns 16 j + 4 (l / 16) .. + 3
    float *C = G.C + (int64_t)blockIdx.z * G.c_split;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int64_t n = n0 + wn * (TN / WN) + j * 16 + 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int64_t m = m0 + wm * (TM / WM) + i * 16 + (lane & 15);
            if (m >= G.M || n >= G.N) continue;
            float *p = C + m * G.ldc + n;
#pragma unroll
            for (int v = 0; v < 4; ++v) redo |= !finite(acc[j][i][v]);
            if (G.cvec && n + 4 <= G.N) {
                *reinterpret_cast<f4 *>(p) = acc[j][i];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < G.N) p[v] = acc[j][i][v];
            }
        }
    }
    if (!redo) return;
    // the lane's own outputs once more, those that are not finite as plain fp32
    // sums (up to the first NaN, which stays)
#pragma unroll 1
    for (int e = 0; e < NJ * NI * 4; ++e) {
        const int64_t m = m0 + wm * (TM / WM) + (e >> 2) % NI * 16 + (lane & 15);
        const int64_t n = n0 + wn * (TN / WN) + (e >> 2) / NI * 16 + 4 * (lane >> 4) + (e & 3);
        if (m >= G.M || n >= G.N || finite(C[m * G.ldc + n])) continue;
        const int64_t row = G.row_map ? (int64_t)G.row_map[m] : m;
        float s = 0.f;
        for (int64_t k = kb; k < ke && s == s; ++k) {
            const float a = row < 0 ? 0.f : G.A[AKC ? row * G.lda + k : k * G.lda + row];
            const float b = n == G.ones_col ? 1.f : G.B[BKC ? n * G.ldb + k : k * G.ldb + n];
            s = fmaf(a, b, s);
        }
        C[m * G.ldc + n] = s;
    }
}

template <int TM, int TN>
void launch_tile(const SplitGemm &G, bool a_kc, bool b_kc, int64_t splits, hipStream_t st) {
    const dim3 grid((unsigned)((G.M + TM - 1) / TM), (unsigned)((G.N + TN - 1) / TN), (unsigned)splits);
    if (!a_kc) {   // (sums over rows come in a few hundred 64-row tiles)
        if constexpr (TM == 64) gemm_s3<TM, TN, false, false><<<grid, 256, 0, st>>>(G);
    } else if (b_kc) gemm_s3<TM, TN, true, true><<<grid, 256, 0, st>>>(G);
    else gemm_s3<TM, TN, true, false><<<grid, 256, 0, st>>>(G);
}

bool al16(const void *p, int64_t ld) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0; }

}  // namespace

// Tiles of 128 x 128 where they give every CU its three blocks, else smaller
// ones (64 columns also where N fits them)
void launch_split_gemm(SplitGemm G, bool a_kc, bool b_kc, int64_t splits, hipStream_t st) {
    if (G.M <= 0 || G.N <= 0) return;
    G.vec = (!a_kc || al16(G.A, G.lda)) && (!b_kc || al16(G.B, G.ldb));
    G.cvec = al16(G.C, G.ldc) && G.c_split % 4 == 0;
    const int64_t b128 = ((G.M + 127) / 128) * ((G.N + 127) / 128) * splits;
    if (G.N <= 64) launch_tile<64, 64>(G, a_kc, b_kc, splits, st);
    else if (!a_kc || G.M <= 64 || b128 < 768) launch_tile<64, 128>(G, a_kc, b_kc, splits, st);
    else launch_tile<128, 128>(G, a_kc, b_kc, splits, st);
}

}  // namespace tag
