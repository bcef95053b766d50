// Readings of the layer equation of Section 4.2.1 that the paper leaves open,
// on a generic fp32 path:
//  * five directed relations: op<-op along the tensor (row = consumer),
//    op<-op against it (row = producer), op<-device, device<-op and
//    device<-device, each with its own W = [W^h | W^e], b, a, adst and
//    softmax (the default reading has three undirected link types);
//  * ReLU after the fully connected edge encoders (default: affine);
//  * K attention heads over all f channels, each with its own attention
//    vectors, averaged (default: K concatenated heads of f/K channels).
// Per layer: W^h h of every node for every relation that touches its type
// (MFMA GEMMs, no folded bias), the edge terms W^e e + b folded to U x + c'
// (affine encoders) or as tables (ReLU encoders), then 16 lanes per
// destination row walk each incoming relation's entries with an online
// softmax per head and write h' = sum_r gamma_r agg_r once.
#include <algorithm>

#include "agg_common.hpp"
#include "fwd_internal.hpp"
#include "transform.hpp"

namespace tag {
namespace {

constexpr int kVarMaxAvgHeads = 8;

__global__ void fill_zero(float *p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0.f;
}

// ------------------------------------------------------------ edge terms
// te[row][c] = b[c] + sum_k W^e[c][k] act(A[k] . x_row + cA[k]); one block
// per table row, the encoded edge vector staged in LDS.
struct EdgeTermArgs {
    const float *We;      // W of the relation: row c at We + c * 2F, W^e = columns [F, 2F)
    const float *b;       // [F]
    const float *A;       // encoder [F][d]
    const float *cA;      // encoder bias [F]
    int d, F, relu;
    // raw feature of table row i: od (d = 1, two rows): x = i; otherwise
    // x = feat[(i / n_links) * stride + (i % n_links) * d + t]
    const float *feat;
    int64_t n_links, stride;
    int bits;             // 1: the rows are the placement bits 0 and 1
    float *te;            // [rows][F]
};

__global__ void __launch_bounds__(256) var_edge_terms(EdgeTermArgs a) {
    __shared__ float enc[256];
    const int64_t i = blockIdx.x;
    const int F = a.F;
    float x0, x1 = 0.f;
    if (a.bits) {
        x0 = (float)i;
    } else {
        const float *xr = a.feat + (i / a.n_links) * a.stride + (i % a.n_links) * a.d;
        x0 = xr[0];
        if (a.d == 2) x1 = xr[1];
    }
    for (int k = threadIdx.x; k < F; k += blockDim.x) {
        float e = a.cA[k] + a.A[(size_t)k * a.d] * x0;
        if (a.d == 2) e = fmaf(a.A[(size_t)k * a.d + 1], x1, e);
        enc[k] = a.relu ? fmaxf(e, 0.f) : e;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < F; c += blockDim.x) {
        const float *wr = a.We + (size_t)c * 2 * F + F;
        float s = a.b[c];
        for (int k = 0; k < F; ++k) s = fmaf(wr[k], enc[k], s);
        a.te[i * F + c] = s;
    }
}

// Affine encoders fold as in the default reading: W^e (A x + c) + b = U x + c'
// per (layer, relation), so no per-link table is written or gathered.  One
// wavefront per (layer, relation, channel).
struct VarFoldArgs {
    const float *layer_w, *layer_b;
    const float *A[3], *c[3];
    int F, NR;
    int type[5];          // link type (0 op-op, 1 op-device, 2 device-device) of each relation
    float *U, *cp;        // [L * NR][F][2], [L * NR][F]
};

__global__ void __launch_bounds__(64) var_fold(VarFoldArgs a) {
    const int F = a.F, lr = blockIdx.x / F, c = blockIdx.x % F, ty = a.type[lr % a.NR];
    const int d = ty == 2 ? 2 : 1;
    const float *W = a.layer_w + (size_t)lr * F * 2 * F + (size_t)c * 2 * F + F;   // row c of W^e
    float u0 = 0.f, u1 = 0.f, s = 0.f;
    for (int k = threadIdx.x; k < F; k += 64) {
        const float we = W[k];
        u0 = fmaf(we, a.A[ty][(size_t)k * d], u0);
        if (d == 2) u1 = fmaf(we, a.A[ty][(size_t)k * d + 1], u1);
        s = fmaf(we, a.c[ty][k], s);
    }
    u0 = head_sum<64>(u0); u1 = head_sum<64>(u1); s = head_sum<64>(s);
    if (threadIdx.x == 0) {
        a.U[((size_t)lr * F + c) * 2] = u0;
        a.U[((size_t)lr * F + c) * 2 + 1] = u1;
        a.cp[(size_t)lr * F + c] = a.layer_b[(size_t)lr * F + c] + s;
    }
}

// ------------------------------------------------------------ aggregation
enum EdgeKind { kBits = 0, kOne = 1, kTwo = 2, kTable = 3 };   // placement bit, one or two raw features, table row

struct VarRel {
    int bucket;              // CSR bucket holding the destination rows
    int dir;                 // bucket 0 only: 0 every entry, 1 forward (row = consumer), 2 backward
    int kind;                // EdgeKind
    const float *ysrc;       // W^h h of the sources: row (rep * n_src + v) at ysrc + row * 2F
    const float *ydst;       // W^h h of the destinations: row (rep * n_dst + u)
    int64_t n_src;
    const float *te;         // edge-term table (ReLU encoders): two rows for kBits, else [replicas][links][F]
    int64_t te_rep;          // replica stride of te in rows (0: shared)
    const float *U, *cp;     // folded affine terms (te == nullptr)
    const float *x;          // raw link features of kOne / kTwo
    int64_t s_x;
    const float *as, *ad;    // attention vectors ([F], or [K][F] for averaged heads)
    float gamma;
    const float *part;       // records of var_part for this relation's rows (nullptr: walked here)
};

struct VarArgs {
    int R, F, K;
    float slope;
    int64_t n_dst;           // destination rows per replica
    const int32_t *rp[4], *col[4], *eid[4];
    const int32_t *oo_head;
    const uint8_t *x_od;
    int64_t s_od;
    int n_rel;
    VarRel rel[3];
    float *out;              // [R * n_dst][F]
    int chunk, max_rec;      // entries per record of var_part, records per row (layout)
    float *part;             // var_part's output
    int rpg;                 // rows per 16 lanes (agg_var)
};

// A destination row belongs to 16 lanes, lane q owning channels [q CPL,
// (q + 1) CPL).  Concatenated heads (AVG false): NH = max(1, K / 16) heads per
// lane, a head spanning max(1, 16 / K) lanes; averaged heads (AVG): every lane
// tracks all NH = K heads over its channels.
template <int CPL, int NH, bool AVG>
struct VarState {
    static constexpr int NA = AVG ? NH : 1;
    float mx[NH], den[NH], acc[NA][CPL];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int h = 0; h < NH; ++h) { mx[h] = -INFINITY; den[h] = 0.f; }
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[k][c] = 0.f;
    }
    // head of (local head h, channel c)
    static __device__ __forceinline__ constexpr int head_of(int c) { return c / (CPL / NH > 0 ? CPL / NH : 1); }
};

// sum over the lph (power of two <= 16) lanes of a head, wave-uniform lph
__device__ __forceinline__ float lanes_sum(float v, int lph) {
    if (lph == 16) return row_sum<16>(v);
    if (lph == 8) return row_sum<8>(v);
    if (lph == 4) return row_sum<4>(v);
    if (lph == 2) return row_sum<2>(v);
    return v;
}

// a lane's channel constants of one relation: the edge terms of placement bit
// 0 and 1, or c' and U, and (concatenated heads) the attention vectors
template <int KIND, int CPL, bool AVG>
struct VarConst {
    float t0[CPL], t1[CPL], t2[CPL], a[CPL], ad[CPL];
    __device__ __forceinline__ void load(const VarRel &V, int F, int c0) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            t0[c] = t1[c] = t2[c] = a[c] = ad[c] = 0.f;
            if (KIND == kBits) {
                t0[c] = V.te ? V.te[c0 + c] : V.cp[c0 + c];
                t1[c] = V.te ? V.te[F + c0 + c] : V.cp[c0 + c] + V.U[2 * (c0 + c)];
            } else if (KIND != kTable) {
                t0[c] = V.cp[c0 + c];
                t1[c] = V.U[2 * (c0 + c)];
                if (KIND == kTwo) t2[c] = V.U[2 * (c0 + c) + 1];
            }
            if (!AVG) {
                a[c] = V.as[c0 + c];
                ad[c] = V.ad[c0 + c];
            }
        }
    }
};

// Entries [beg, end) of destination row u, EB at a time: the batch's source
// rows and link features load together while the next batch's indices do,
// and the running softmax is rescaled once per batch.
template <int KIND, int CPL, int NH, bool AVG>
__device__ __forceinline__ void var_stream(const VarArgs &A, const VarRel &V, const VarConst<KIND, CPL, AVG> &k,
                                           int32_t rep, int32_t u, int32_t beg, int32_t end, int c0, int lph,
                                           VarState<CPL, NH, AVG> &st) {
    constexpr int EB = CPL * (AVG ? NH : 1) > 32 ? 2 : 4;
    const int F = A.F, ldy = 2 * F;
    float qd[NH];            // destination terms
    {
        float yd[CPL];
        load_ch<CPL, false>(V.ydst, ((int64_t)rep * A.n_dst + u) * ldy + c0, yd);
#pragma unroll
        for (int h = 0; h < NH; ++h) qd[h] = 0.f;
        if constexpr (AVG) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) qd[h] = fmaf(V.ad[h * F + c0 + c], yd[c], qd[h]);
                qd[h] = row_sum<16>(qd[h]);
            }
        } else {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int h = VarState<CPL, NH, AVG>::head_of(c);
                qd[h] = fmaf(k.ad[c], yd[c], qd[h]);
            }
#pragma unroll
            for (int h = 0; h < NH; ++h) qd[h] = lanes_sum(qd[h], lph);
        }
    }
    const float *ys = V.ysrc + (int64_t)rep * V.n_src * ldy;
    const uint8_t *xb = KIND == kBits ? A.x_od + (int64_t)rep * A.s_od : nullptr;
    const float *xf = (KIND == kOne || KIND == kTwo) ? V.x + (int64_t)rep * V.s_x : nullptr;
    const float *tt = KIND == kTable ? V.te + (int64_t)rep * V.te_rep * F : nullptr;
    const int32_t *cl = A.col[V.bucket], *ei = A.eid[V.bucket];
    int32_t v[EB], id[EB];
    auto load_idx = [&](int32_t e) {
#pragma unroll
        for (int i = 0; i < EB; ++i) {
            const int32_t j = min(e + i, end - 1);
            v[i] = cl[j];
            id[i] = ei[j];
        }
    };
    load_idx(beg);
    for (int32_t e = beg; e < end; e += EB) {
        float m[EB][CPL], x0[EB], x1[EB];
        bool ok[EB];
#pragma unroll
        for (int i = 0; i < EB; ++i) {
            load_ch<CPL, false>(ys, (int64_t)v[i] * ldy + c0, m[i]);
            x0[i] = x1[i] = 0.f;
            ok[i] = e + i < end;
            if (KIND == kBits) x0[i] = xb[id[i]] ? 1.f : 0.f;
            if (KIND == kOne) x0[i] = xf[id[i]];
            if (KIND == kTwo) { x0[i] = xf[2 * (int64_t)id[i]]; x1[i] = xf[2 * (int64_t)id[i] + 1]; }
            if (V.dir) ok[i] = ok[i] && ((A.oo_head[id[i]] == u) == (V.dir == 1));
        }
        float te[KIND == kTable ? EB : 1][CPL];
        if constexpr (KIND == kTable) {
#pragma unroll
            for (int i = 0; i < EB; ++i) load_ch<CPL, false>(tt, (int64_t)id[i] * F + c0, te[i]);
        }
        load_idx(min(e + EB, end - 1));
#pragma unroll
        for (int i = 0; i < EB; ++i) {
            // entries past the end or of the other direction weigh nothing
            // and hold a zero message
            const float top = ok[i] ? INFINITY : 0.f;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                float z = m[i][c];
                if constexpr (KIND == kBits) z += x0[i] != 0.f ? k.t1[c] : k.t0[c];
                else if constexpr (KIND == kTable) z += te[i][c];
                else if constexpr (KIND == kTwo) z += fmaf(k.t2[c], x1[i], fmaf(k.t1[c], x0[i], k.t0[c]));
                else z += fmaf(k.t1[c], x0[i], k.t0[c]);
                m[i][c] = __builtin_amdgcn_fmed3f(z, 0.f, top);
            }
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            float s2[EB];
            if constexpr (AVG) {
                float av[CPL];
#pragma unroll
                for (int c = 0; c < CPL; ++c) av[c] = V.as[h * F + c0 + c];
#pragma unroll
                for (int i = 0; i < EB; ++i) {
                    float p = 0.f;
#pragma unroll
                    for (int c = 0; c < CPL; ++c) p = fmaf(av[c], m[i][c], p);
                    s2[i] = row_sum<16>(p);
                }
            } else {
#pragma unroll
                for (int i = 0; i < EB; ++i) {
                    float p = 0.f;
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        if (VarState<CPL, NH, AVG>::head_of(c) == h) p = fmaf(k.a[c], m[i][c], p);
                    s2[i] = lanes_sum(p, lph);
                }
            }
            float nm = st.mx[h];
#pragma unroll
            for (int i = 0; i < EB; ++i) {
                const float s = s2[i] + qd[h];
                s2[i] = ok[i] ? (s > 0.f ? s : A.slope * s) * kLog2e : -INFINITY;
                nm = fmaxf(nm, s2[i]);
            }
            const float ref = nm == -INFINITY ? 0.f : nm;   // (no entry yet: every weight is exp2(-inf) = 0)
            const float sc = __builtin_amdgcn_exp2f(st.mx[h] - ref);
            float p[EB], ps = 0.f;
#pragma unroll
            for (int i = 0; i < EB; ++i) { p[i] = __builtin_amdgcn_exp2f(s2[i] - ref); ps += p[i]; }
            st.den[h] = fmaf(st.den[h], sc, ps);
            st.mx[h] = nm;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (!AVG && VarState<CPL, NH, AVG>::head_of(c) != h) continue;
                float &r = st.acc[AVG ? h : 0][c];
                r *= sc;
#pragma unroll
                for (int i = 0; i < EB; ++i) r = fmaf(p[i], m[i][c], r);
            }
        }
    }
}

// Record of a part of a row: K maxima, K sums, then the accumulated channels
// ([F], or [K][F] for averaged heads).
template <bool AVG>
__host__ __device__ __forceinline__ int64_t var_rec(int F, int K) { return 2 * K + (int64_t)(AVG ? K : 1) * F; }

// Long rows (device <- op: one entry per op) in parts of `chunk` entries,
// 16 lanes per (replica, part, row), rows fastest so that the rows of one
// replica's part read the same source rows at about the same time.
template <int KIND, int CPL, int NH, bool AVG>
__global__ void __launch_bounds__(256) var_part(VarArgs A) {
    const VarRel &V = A.rel[0];
    const int lane = threadIdx.x & 15;
    const int64_t w = (int64_t)xcd_swizzle(blockIdx.x, gridDim.x) * 16 + (threadIdx.x >> 4);
    if (w >= (int64_t)A.R * A.max_rec * A.n_dst) return;
    const int32_t u = (int32_t)(w % A.n_dst), part = (int32_t)((w / A.n_dst) % A.max_rec);
    const int32_t rep = (int32_t)(w / (A.n_dst * A.max_rec));
    const int32_t rb = A.rp[V.bucket][u], re = A.rp[V.bucket][u + 1], beg = rb + part * A.chunk;
    if (beg >= re) return;
    const int K = A.K, lph = AVG ? 16 : (K < 16 ? 16 / K : 1), c0 = lane * CPL;
    VarState<CPL, NH, AVG> st;
    st.init();
    VarConst<KIND, CPL, AVG> k;
    k.load(V, A.F, c0);
    var_stream<KIND>(A, V, k, rep, u, beg, min(beg + A.chunk, re), c0, lph, st);
    float *r = A.part + (((int64_t)rep * A.n_dst + u) * A.max_rec + part) * var_rec<AVG>(A.F, K);
    if (lane % lph == 0) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int hd = AVG ? h : (NH > 1 ? lane * NH + h : lane / lph);
            r[hd] = st.mx[h];
            r[K + hd] = st.den[h];
        }
    }
#pragma unroll
    for (int q = 0; q < VarState<CPL, NH, AVG>::NA; ++q)
#pragma unroll
        for (int c = 0; c < CPL; ++c) r[2 * K + (int64_t)q * A.F + c0 + c] = st.acc[q][c];
}

// the records of a row walked in parts, merged in order
template <int CPL, int NH, bool AVG>
__device__ __forceinline__ void var_merge(const VarArgs &A, const VarRel &V, int64_t row, int n, int lane, int lph,
                                          VarState<CPL, NH, AVG> &st) {
    const int F = A.F, K = A.K, c0 = lane * CPL;
    const int64_t rec = var_rec<AVG>(F, K);
    const float *r = V.part + row * A.max_rec * rec;
    for (int q = 0; q < n; ++q, r += rec) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int hd = AVG ? h : (NH > 1 ? lane * NH + h : lane / lph);
            const float rm = r[hd], nm = fmaxf(st.mx[h], rm), ref = nm == -INFINITY ? 0.f : nm;
            const float s0 = __builtin_amdgcn_exp2f(st.mx[h] - ref), s1 = __builtin_amdgcn_exp2f(rm - ref);
            st.den[h] = fmaf(st.den[h], s0, r[K + hd] * s1);
            st.mx[h] = nm;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (!AVG && VarState<CPL, NH, AVG>::head_of(c) != h) continue;
                float &x = st.acc[AVG ? h : 0][c];
                x = fmaf(x, s0, r[2 * K + (int64_t)(AVG ? h : 0) * F + c0 + c] * s1);
            }
        }
    }
}

// Relation ri of the rows row0 .. row0 + nrow - 1 (of all replicas), added
// into the lane's channels of the LDS rows `o`
template <int KIND, int CPL, int NH, bool AVG>
__device__ __forceinline__ void var_rows(const VarArgs &A, int ri, int64_t row0, int nrow, int lane, float *o) {
    const VarRel &V = A.rel[ri];
    const int F = A.F, K = A.K, lph = AVG ? 16 : (K < 16 ? 16 / K : 1), c0 = lane * CPL;
    VarConst<KIND, CPL, AVG> k;
    k.load(V, F, c0);
    int32_t rep = (int32_t)(row0 / A.n_dst), u = (int32_t)(row0 % A.n_dst);
    const float g = AVG ? V.gamma / K : V.gamma;
    // (lane i holds row i's range)
    const int32_t ul = (int32_t)((row0 + min(lane, nrow - 1)) % A.n_dst);
    const int32_t begs = A.rp[V.bucket][ul], ends = A.rp[V.bucket][ul + 1];
#pragma unroll 1
    for (int i = 0; i < nrow; ++i) {
        const int32_t beg = __shfl(begs, i, 16), end = __shfl(ends, i, 16);
        if (beg < end) {
            VarState<CPL, NH, AVG> st;
            st.init();
            if (V.part) var_merge(A, V, row0 + i, (end - beg + A.chunk - 1) / A.chunk, lane, lph, st);
            else var_stream<KIND>(A, V, k, rep, u, beg, end, c0, lph, st);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const float inv = st.den[h] > 0.f ? g / st.den[h] : 0.f;   // (no entry of this direction: 0)
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    if (AVG || VarState<CPL, NH, AVG>::head_of(c) == h)
                        o[i * F + c0 + c] = fmaf(st.acc[AVG ? h : 0][c], inv, o[i * F + c0 + c]);
            }
        }
        if (++u == A.n_dst) { u = 0; ++rep; }
    }
}

// Destination rows, 16 lanes per `rpg` consecutive (replica, row) pairs: each
// incoming relation's entries (or, for rows walked in parts, their records),
// with the relation's channel constants loaded once for the group's rows,
// summed in LDS; every row is written once.  Bound by load latency and vector
// issue: four row groups per wavefront with F / 16 channels per lane, four
// entries in flight each.  One wavefront per row with F / 64 channels per
// lane, one entry at a time, and per-link edge-term tables took 1.67 ms for a
// layer's two launches (1,200 ops, 16 devices, 64 candidates, f = 128); this
// form takes 0.21 ms with the parts.
constexpr int kVarRows = 4;   // rows per 16 lanes where there are enough of them

// SET: the link kinds the rows meet besides placement bits (an instance holds
// registers for its own kinds only): 0 op rows, 1 device rows, 2 tables
template <int CPL, int NH, bool AVG, int SET>
__global__ void __launch_bounds__(256) agg_var(VarArgs A) {
    extern __shared__ __attribute__((aligned(16))) float var_out[];   // [16 groups][rpg][F]
    const int lane = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int64_t rows = (int64_t)A.R * A.n_dst;
    const int64_t row0 = ((int64_t)xcd_swizzle(blockIdx.x, gridDim.x) * 16 + grp) * A.rpg;
    if (row0 >= rows) return;
    const int nrow = (int)min((int64_t)A.rpg, rows - row0), F = A.F, c0 = lane * CPL;
    float *o = var_out + grp * A.rpg * F;   // (each lane touches only its own channels: no barrier)
    for (int i = 0; i < nrow; ++i)
#pragma unroll
        for (int c = 0; c < CPL; ++c) o[i * F + c0 + c] = 0.f;
#pragma unroll 1
    for (int ri = 0; ri < A.n_rel; ++ri) {
        const int kind = A.rel[ri].kind;
        if (kind == kBits) var_rows<kBits, CPL, NH, AVG>(A, ri, row0, nrow, lane, o);
        else var_rows<SET == 0 ? kOne : SET == 1 ? kTwo : kTable, CPL, NH, AVG>(A, ri, row0, nrow, lane, o);
    }
    for (int i = 0; i < nrow; ++i) {
        float *d = A.out + (row0 + i) * F + c0;
        const float *q = o + i * F + c0;
#pragma unroll
        for (int c = 0; c < CPL; c += 4) *reinterpret_cast<float4 *>(d + c) = *reinterpret_cast<const float4 *>(q + c);
    }
}

// ------------------------------------------------------------ planning
// Rows of the device <- op bucket longer than kPartMin entries are walked in
// parts (at most kMaxParts, at least kPartMin entries each): a device row has
// one entry per op, so one walk per row would leave R n_dev short of the
// chip's wavefronts and each of them a serial chain over every op.
constexpr int kPartMin = 64, kMaxParts = 16;

int var_chunk(const tag_graph *g) {
    const int d = g->max_degree[2];
    return std::max(kPartMin, (d + kMaxParts - 1) / kMaxParts);
}
int var_parts(const tag_graph *g) {   // 0: rows are short, walked whole
    const int d = g->max_degree[2];
    return d > kPartMin ? (d + var_chunk(g) - 1) / var_chunk(g) : 0;
}

struct VarLayout {
    float *H_op[2], *H_dev[2];
    float *zero;                 // [F] zeros (no bias added by the transform)
    float *Y_op[2], *Y_dev[2];   // [rows][2F]; the second pair for five relations only
    float *U, *cp;               // folded affine edge encoders
    float *te_oo[2], *te_od[2], *te_dd;   // edge-term tables (ReLU encoders)
    float *part;
};

size_t carve_var(const tag_graph *g, const tag_model_dims *d, int32_t R, void *base, VarLayout *L) {
    Carver c(base);
    const size_t F = d->f, N = (size_t)R * g->n_op, M = (size_t)R * g->n_dev;
    const bool five = d->relations == 5, table = d->edge_act == 1;
    const int NR = five ? 5 : 3;
    for (int i = 0; i < 2; ++i) {
        L->H_op[i] = c.take<float>(N * F + 1);
        L->H_dev[i] = c.take<float>(M * F + 1);
    }
    L->zero = c.take<float>(F);
    for (int i = 0; i < 2; ++i) {
        L->Y_op[i] = i == 0 || five ? c.take<float>(N * 2 * F + 1) : nullptr;
        L->Y_dev[i] = i == 0 || five ? c.take<float>(M * 2 * F + 1) : nullptr;
    }
    L->U = c.take<float>((size_t)d->layers * NR * F * 2);
    L->cp = c.take<float>((size_t)d->layers * NR * F);
    const int64_t rec = d->head_mode == 1 ? var_rec<true>(d->f, d->heads) : var_rec<false>(d->f, d->heads);
    // a layer's op-op tables have been read when its device rows' parts are written: one place for both
    // (tables sized for per-replica features: the caller's strides decide at run time)
    const size_t oo = table ? (size_t)R * g->e_oo * F : 0, parts = M * var_parts(g) * rec;
    float *p = c.take<float>(std::max((five ? 2 : 1) * oo, parts) + 1);
    L->part = p;
    for (int i = 0; i < 2; ++i) {
        const bool on = table && (i == 0 || five);
        L->te_oo[i] = on ? p + i * oo : nullptr;
        L->te_od[i] = on ? c.take<float>(2 * F) : nullptr;
    }
    L->te_dd = table ? c.take<float>((size_t)R * g->e_dd * F + 1) : nullptr;
    return c.used;
}

// Y = H [W_first ; W_second]^T (W^h blocks of two relations) of the op and
// device rows into [rows][2F], no bias, one launch
void var_transform(const tag_model_dims *d, const float *H_op, int64_t rows_op, const float *W1, const float *W2,
                   float *Y_op, const float *H_dev, int64_t rows_dev, const float *V1, const float *V2, float *Y_dev,
                   const float *zero, hipStream_t st) {
    const int F = d->f;
    GemmArgs ga{};
    ga.F = F;
    ga.prep.jph = 0;
    ga.prep.K = d->heads;
    ga.prep.cp_same[0] = ga.prep.cp_same[1] = zero;
    ga.prep.cp_od = zero;
    ga.tiles0 = transform_row_tiles(rows_op);
    ga.side[0] = GemmSide{H_op, rows_op, W1, W2, 2 * F, Y_op};
    ga.side[1] = GemmSide{H_dev, rows_dev, V1, V2, 2 * F, Y_dev};
    launch_transform(ga, false, st);
}

void var_edge_table(const tag_model_dims *d, const float *W, const float *b, const float *A, const float *cA, int dr,
                    const float *feat, int64_t n_links, int64_t stride, int64_t reps, bool bits, float *te,
                    hipStream_t st) {
    const int64_t rows = bits ? 2 : reps * n_links;
    if (rows == 0) return;
    EdgeTermArgs a{W, b, A, cA, dr, d->f, d->edge_act == 1 ? 1 : 0, feat, std::max<int64_t>(n_links, 1), stride,
                   bits ? 1 : 0, te};
    var_edge_terms<<<(unsigned)rows, 256, 0, st>>>(a);
}

// The rows of relation 0 of `A` in parts (when A.part is set), then every row
template <int CPL, int NH, bool AVG>
void launch_agg_var(VarArgs A, hipStream_t st) {
    const int64_t rows = (int64_t)A.R * A.n_dst;
    if (rows == 0) return;
    if (A.part) var_part<kBits, CPL, NH, AVG><<<(unsigned)((rows * A.max_rec + 15) / 16), 256, 0, st>>>(A);
    // several rows per group only where that leaves a few blocks per CU
    A.rpg = rows >= 16 * kVarRows * 1024 ? kVarRows : 1;
    const unsigned blocks = (unsigned)((rows + 16 * A.rpg - 1) / (16 * A.rpg));
    const size_t lds = 16 * A.rpg * A.F * sizeof(float);
    const int kind = A.rel[A.n_rel - 1].kind == kBits ? A.rel[0].kind : A.rel[A.n_rel - 1].kind;
    if (kind == kOne) agg_var<CPL, NH, AVG, 0><<<blocks, 256, lds, st>>>(A);
    else if (kind == kTwo) agg_var<CPL, NH, AVG, 1><<<blocks, 256, lds, st>>>(A);
    else agg_var<CPL, NH, AVG, 2><<<blocks, 256, lds, st>>>(A);
}

template <int CPL>
void dispatch_var_heads(bool avg, int K, const VarArgs &A, hipStream_t st) {
    if (avg) {
        if (K == 1) launch_agg_var<CPL, 1, true>(A, st);
        else if (K == 2) launch_agg_var<CPL, 2, true>(A, st);
        else if (K == 4) launch_agg_var<CPL, 4, true>(A, st);
        else launch_agg_var<CPL, 8, true>(A, st);
    } else {
        if (K <= 16) launch_agg_var<CPL, 1, false>(A, st);
        else if (K == 32) launch_agg_var<CPL, 2, false>(A, st);
        else launch_agg_var<CPL, 4, false>(A, st);
    }
}

void dispatch_agg_var(int F, bool avg, const VarArgs &A, hipStream_t st) {
    if (F == 64) dispatch_var_heads<4>(avg, A.K, A, st);
    else if (F == 128) dispatch_var_heads<8>(avg, A.K, A, st);
    else dispatch_var_heads<16>(avg, A.K, A, st);
}

}  // namespace

bool is_variant(const tag_model_dims *d) {
    return (d->relations != 0 && d->relations != 3) || d->edge_act != 0 || d->head_mode != 0;
}

tag_status check_variant(const tag_model_dims *d) {
    if (d->relations != 0 && d->relations != 3 && d->relations != 5) TAG_FAIL(TAG_EINVAL, "relations must be 3 or 5");
    if (d->edge_act != 0 && d->edge_act != 1) TAG_FAIL(TAG_EINVAL, "edge_act must be 0 or 1");
    if (d->head_mode != 0 && d->head_mode != 1) TAG_FAIL(TAG_EINVAL, "head_mode must be 0 or 1");
    if (!is_variant(d)) return TAG_OK;
    if (d->dtype != TAG_F32) TAG_FAIL(TAG_ESHAPE, "the relations / edge_act / head_mode variants run in fp32");
    if (d->sigma != 0) TAG_FAIL(TAG_ESHAPE, "the relations / edge_act / head_mode variants use ReLU messages");
    if (d->head_mode == 1 && d->heads > kVarMaxAvgHeads) TAG_FAIL(TAG_ESHAPE, "averaged heads: at most 8 heads");
    return TAG_OK;
}

size_t variant_workspace(const tag_graph *g, const tag_model_dims *d, int32_t R) {
    VarLayout L;
    return carve_var(g, d, R, nullptr, &L);
}

tag_status forward_variant(const tag_graph *g, const tag_model_dims *dims, const tag_weights *w,
                           const tag_features *x, void *workspace, size_t ws_bytes, float *E_op, float *E_dev,
                           hipStream_t stream) {
    const int32_t R = x->n_replicas;
    VarLayout L;
    if (carve_var(g, dims, R, nullptr, &L) > ws_bytes)
        TAG_FAIL(TAG_ENOSPACE, "workspace too small (see tag_gnn_workspace)");
    carve_var(g, dims, R, workspace, &L);
    const int F = dims->f, K = dims->heads, NL = dims->layers;
    const bool five = dims->relations == 5, avg = dims->head_mode == 1, table = dims->edge_act == 1;
    const int NR = five ? 5 : 3;
    const size_t asz = (size_t)(avg ? K : 1) * F;
    const int64_t N = (int64_t)R * g->n_op, M = (int64_t)R * g->n_dev;
    const int64_t reps_oo = x->stride_oo ? R : 1, reps_dd = x->stride_dd ? R : 1;
    // relation indices: op<-op (one or two), op<-device, device<-op, device<-device
    const int r_f = 0, r_b = five ? 1 : 0, r_od = five ? 2 : 1, r_do = five ? 3 : 1, r_dd = five ? 4 : 2;
    fill_zero<<<1, 256, 0, stream>>>(L.zero, F);   // a kernel, not a memset node, so the call stays capturable
    if (!table) {
        VarFoldArgs fa{w->layer_w, w->layer_b, {w->enc_edge_w[0], w->enc_edge_w[1], w->enc_edge_w[2]},
                       {w->enc_edge_b[0], w->enc_edge_b[1], w->enc_edge_b[2]}, F, NR, {}, L.U, L.cp};
        fa.type[r_f] = fa.type[r_b] = 0;
        fa.type[r_od] = fa.type[r_do] = 1;
        fa.type[r_dd] = 2;
        var_fold<<<NL * NR * F, 64, 0, stream>>>(fa);
    }

    // encoders: h0 = ReLU(A x + c) (fp32)
    SmallGemm eo{x->x_op, dims->f_op, N, nullptr, dims->f_op, w->enc_op_w, dims->f_op, F, w->enc_op_b, 1, L.H_op[0], F, 0};
    SmallGemm ed{x->x_dev, dims->f_dev, M, nullptr, dims->f_dev, w->enc_dev_w, dims->f_dev, F, w->enc_dev_b, 1,
                 L.H_dev[0], F, 0};
    prof_begin(TAG_STAGE_ENCODE, stream);
    launch_small_gemm(eo, stream);
    launch_small_gemm(ed, stream);
    prof_end(TAG_STAGE_ENCODE, stream);

    VarArgs base{};
    base.R = R; base.F = F; base.K = K;
    base.slope = dims->leaky_slope;
    for (int b = 0; b < 4; ++b) { base.rp[b] = g->rowptr[b]; base.col[b] = g->col[b]; base.eid[b] = g->eid[b]; }
    base.oo_head = g->oo_head;
    base.x_od = x->x_od; base.s_od = x->stride_od;
    base.chunk = var_chunk(g);
    base.max_rec = var_parts(g);
    // where each relation's transform lies: op rows [f ; od] or [f ; b], [od ; do]; device rows [dd ; od], [do ; do]
    float *const Yo = L.Y_op[0], *const Yo2 = L.Y_op[five ? 1 : 0], *const Yd = L.Y_dev[0];
    const float *y_od_op = five ? Yo2 : Yo + F, *y_do_op = Yo2 + F;
    const float *y_do_dev = five ? L.Y_dev[1] : Yd + F;
    for (int l = 0; l < NL; ++l) {
        const float *W[5], *bb[5], *as[5], *ad[5], *U[5], *cp[5];
        for (int r = 0; r < NR; ++r) {
            const size_t lr = (size_t)l * NR + r;
            W[r] = w->layer_w + lr * F * 2 * F;
            bb[r] = w->layer_b + lr * F;
            as[r] = w->att_src + lr * asz;
            ad[r] = w->att_dst + lr * asz;
            U[r] = L.U + lr * F * 2;
            cp[r] = L.cp + lr * F;
        }
        const float *Hop = L.H_op[l & 1], *Hdev = L.H_dev[l & 1];
        prof_begin(TAG_STAGE_TRANSFORM, stream);
        var_transform(dims, Hop, N, W[r_f], five ? W[r_b] : W[r_od], Yo, Hdev, M, W[r_dd], W[r_od], Yd, L.zero, stream);
        if (five)
            var_transform(dims, Hop, N, W[r_od], W[r_do], Yo2, Hdev, M, W[r_do], W[r_do], L.Y_dev[1], L.zero, stream);
        prof_end(TAG_STAGE_TRANSFORM, stream);
        if (table) {   // edge-term tables
            var_edge_table(dims, W[r_f], bb[r_f], w->enc_edge_w[0], w->enc_edge_b[0], 1, x->x_oo, g->e_oo,
                           x->stride_oo, reps_oo, false, L.te_oo[0], stream);
            var_edge_table(dims, W[r_od], bb[r_od], w->enc_edge_w[1], w->enc_edge_b[1], 1, nullptr, 0, 0, 1, true,
                           L.te_od[0], stream);
            if (five) {
                var_edge_table(dims, W[r_b], bb[r_b], w->enc_edge_w[0], w->enc_edge_b[0], 1, x->x_oo, g->e_oo,
                               x->stride_oo, reps_oo, false, L.te_oo[1], stream);
                var_edge_table(dims, W[r_do], bb[r_do], w->enc_edge_w[1], w->enc_edge_b[1], 1, nullptr, 0, 0, 1, true,
                               L.te_od[1], stream);
            }
            var_edge_table(dims, W[r_dd], bb[r_dd], w->enc_edge_w[2], w->enc_edge_b[2], 2, x->x_dd, g->e_dd,
                           x->stride_dd, reps_dd, false, L.te_dd, stream);
        }
        const bool last = l == NL - 1;
        const int five_i = five ? 1 : 0;
        auto rel = [&](int r, int bucket, int dir, int kind, const float *ys, const float *yd, int64_t n_src,
                       const float *te, int64_t te_rep, const float *feat, int64_t s_x, float gamma) {
            return VarRel{bucket, dir, table && kind != kBits ? kTable : kind, ys, yd, n_src, te, te_rep, U[r], cp[r],
                          feat, s_x, as[r], ad[r], gamma, nullptr};
        };
        const int64_t rep_oo = reps_oo > 1 ? g->e_oo : 0, rep_dd = reps_dd > 1 ? g->e_dd : 0;
        // op destinations
        VarArgs A = base;
        A.n_dst = g->n_op;
        A.out = last ? E_op : L.H_op[(l + 1) & 1];
        int n = 0;
        A.rel[n++] = rel(r_f, 0, five ? 1 : 0, kOne, Yo, Yo, g->n_op, L.te_oo[0], rep_oo, x->x_oo, x->stride_oo,
                         dims->gamma_same);
        if (five)
            A.rel[n++] = rel(r_b, 0, 2, kOne, Yo + F, Yo + F, g->n_op, L.te_oo[1], rep_oo, x->x_oo, x->stride_oo,
                             dims->gamma_same);
        A.rel[n++] = rel(r_od, 1, 0, kBits, Yd + F, y_od_op, g->n_dev, L.te_od[0], 0, nullptr, 0, dims->gamma_cross);
        A.n_rel = n;
        prof_begin(TAG_STAGE_AGG_OP_OP, stream);
        dispatch_agg_var(F, avg, A, stream);
        prof_end(TAG_STAGE_AGG_OP_OP, stream);
        // device destinations
        VarArgs B = base;
        B.n_dst = g->n_dev;
        B.out = last ? E_dev : L.H_dev[(l + 1) & 1];
        B.rel[0] = rel(r_do, 2, 0, kBits, y_do_op, y_do_dev, g->n_op, L.te_od[five_i], 0, nullptr, 0,
                       dims->gamma_cross);
        B.rel[1] = rel(r_dd, 3, 0, kTwo, Yd, Yd, g->n_dev, L.te_dd, rep_dd, x->x_dd, x->stride_dd, dims->gamma_same);
        B.n_rel = 2;
        if (B.max_rec > 0) {
            B.part = L.part;
            B.rel[0].part = L.part;
        }
        prof_begin(TAG_STAGE_AGG_DEV_MERGE, stream);
        dispatch_agg_var(F, avg, B, stream);
        prof_end(TAG_STAGE_AGG_DEV_MERGE, stream);
    }
    return launch_status("tag_gnn_forward");
}

}  // namespace tag
