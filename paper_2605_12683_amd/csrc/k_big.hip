// Latent dimensions 65..128 (padded width 128) on the stored-Jacobian path of the shallow PLRNN:
// the same operations as the M <= 64 kernels (k_dense.hip, k_shallow.hip, the carry walk), laid
// out for a 128 x 128 chain matrix that one wave cannot hold.
//
//   k_chunk_product_big   one 4-wave workgroup per chain: wave w holds columns 32w..32w+31 of the
//                         chunk product P <- E_t P in matrix-core accumulators (split, the B
//                         operand of the next step), E_t split into LDS; the chunk-local solution
//                         u <- E_t u + rhs on the vector units through LDS
//   k_carry_big           one 256-thread block per walk: carries across the chunks, one level,
//                         or two with k_carry_group_big (group maps on the matrix cores)
//   k_fixup_big           one 128-thread block per chain: each chunk re-run from its carry
//   k_resjac_big          residual, masks (the fixed-order float32 decision) and F, one row per
//                         wave, W1 and W2 in LDS
//   k_jacform_big         J~ = diag(A p) + W1 diag(m) (W2 P) on the matrix cores, 4 waves per
//                         row, two column tiles each
//   k_grads_big           per-block partial sums of the shallow gradients (layout of
//                         k_grads_shplrnn), summed by k_reduce_rows
// E_t is J_t, or J_t^T when flipped (the bare scan's other orientation), as in k_dense.hip.
#include "common.h"
#include "launch.h"
#include "split16.h"

namespace deer {

constexpr int BG = 128;   // padded width

// element (row, col) of E_t (J_t row-major per step, zero outside M x M)
template <bool FLIP>
__device__ __forceinline__ float eload(const float *__restrict__ Jp, int M, int row, int col) {
    if (row >= M || col >= M) return 0.f;
    return FLIP ? Jp[(size_t)col * M + row] : Jp[(size_t)row * M + col];
}

// Products of 128 x 128 matrices along a chain, Q <- E_t Q from the identity, on the bf16 matrix
// cores with operands in three exact parts (split16.h), one 4-wave workgroup per chain.  Wave w holds
// columns 32 w .. 32 w + 31 of Q in accumulators, which after the split are the next step's B operand;
// E_t is split by the workgroup into LDS in the A operand's layout (96 KB: one buffer, written between
// two barriers), the next step's loads in flight while the matrix cores work on this one.
// 384 instructions of 16 x 16 x 32 per wave and step take 3.0 us (512 of 16 x 16 x 4 in fp32 7.1 us),
// after which reading E_t (64 KB a step on every CU) and the splits count as much.
struct BigProd {
    v4u es[8][4][3][64];   // [row tile][k block][hi, mid, lo][es_slot(lane)]
    float ub[2][BG];
};

// Staging without a transpose: a load takes 128 bytes of each of 8 rows (16 rows of 64 bytes took 2.3
// us a step with few blocks, this 1.4 us) and the lane group g of a row's 8-byte pieces is spread
// over both halves of the banks; with a transpose a load takes 64 bytes of each of 4 source rows.
__device__ __forceinline__ int es_slot(int lane) { return lane ^ ((lane >> 1) & 8); }

template <bool TRN>
struct BigChain {
    BigProd &s;
    int wv, lane, g, c;
    v4f acc[8][2];            // acc[I][Jt][r]: row 16 I + 4 g + r, column 32 wv + 16 Jt + c
    float4 pre[16];           // the next E: columns col(k) .. + 3 of row(k)

    __device__ __forceinline__ explicit BigChain(BigProd &sm) : s(sm) {
        wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        lane = threadIdx.x & 63;
        g = lane >> 4;
        c = lane & 15;
#pragma unroll
        for (int I = 0; I < 8; ++I)
#pragma unroll
            for (int Jt = 0; Jt < 2; ++Jt)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[I][Jt][r] = (16 * I + 4 * g + r == 32 * wv + 16 * Jt + c) ? 1.f : 0.f;
    }
    __device__ __forceinline__ int row(int k) const {
        return TRN ? 16 * (2 * wv + (k >> 3)) + c : 32 * wv + 8 * (k >> 2) + (lane >> 3);
    }
    __device__ __forceinline__ int col(int k) const { return TRN ? 16 * (k & 7) + 4 * g : 32 * (k & 3) + 4 * (lane & 7); }
    // the loaded rows, split, into LDS (between two barriers)
    __device__ __forceinline__ void stage_store() {
        typedef uint32_t v2u __attribute__((ext_vector_type(2)));
        if constexpr (TRN) {
#pragma unroll
            for (int k = 0; k < 16; k += 2) {
                v4u o[3];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 v = pre[k + h];
                    uint32_t a[3], b[3];
                    split_pair(v.x, v.y, a);
                    split_pair(v.z, v.w, b);
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        o[q][2 * h] = a[q];
                        o[q][2 * h + 1] = b[q];
                    }
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) s.es[2 * wv + (k >> 3)][(k & 7) >> 1][q][es_slot(lane)] = o[q];
            }
        } else {
            const int gg = lane & 3, e2 = (lane >> 2) & 1, cr = lane >> 3;   // lane group, slot half, row mod 8
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float4 v = pre[k];
                uint32_t a[3], b[3];
                split_pair(v.x, v.y, a);
                split_pair(v.z, v.w, b);
                const int sl = es_slot(16 * gg + 8 * ((k >> 2) & 1) + cr);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    reinterpret_cast<v2u *>(&s.es[2 * wv + (k >> 3)][k & 3][q][sl])[e2] = (v2u){a[q], b[q]};
            }
        }
    }
    // Q <- E Q
    __device__ __forceinline__ void multiply() {
        v4u bq[3][2][4];
#pragma unroll
        for (int Jt = 0; Jt < 2; ++Jt)
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t part[3];
                    split_pair(acc[I][Jt][2 * h], acc[I][Jt][2 * h + 1], part);
#pragma unroll
                    for (int q = 0; q < 3; ++q) bq[q][Jt][I >> 1][2 * (I & 1) + h] = part[q];
                }
#pragma unroll
        for (int I0 = 0; I0 < 8; I0 += 2) {
            __builtin_amdgcn_sched_barrier(0);   // else operands read early spill
#pragma unroll
            for (int I = I0; I < I0 + 2; ++I)
#pragma unroll
                for (int Jt = 0; Jt < 2; ++Jt) acc[I][Jt] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                v4u aq[2][3];
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int q = 0; q < 3; ++q) aq[n][q] = s.es[I0 + n][kk][q][es_slot(lane)];
#pragma unroll
                for (int o = 2; o >= 0; --o)   // parts of one order of magnitude, the smallest first
#pragma unroll
                    for (int qa = o; qa >= 0; --qa)
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int Jt = 0; Jt < 2; ++Jt)
                                acc[I0 + n][Jt] = mfma_b(aq[n][qa], bq[o - qa][Jt][kk], acc[I0 + n][Jt]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // row 32 wv + lane % 32 of E u for the u of buffer buf (both halves of the wave hold it)
    __device__ __forceinline__ float apply(int buf) {
        const int I = 2 * wv + ((lane & 31) >> 4), hh = lane >> 5;
        float p0 = 0.f, p1 = 0.f;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
            const int kk = 2 * hh + k2;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4u w[3];
#pragma unroll
                for (int e = 0; e < 3; ++e) w[e] = s.es[I][kk][e][es_slot(16 * q + c)];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 y = *reinterpret_cast<const float4 *>(&s.ub[buf][32 * kk + 16 * h + 4 * q]);
                    float x[4];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {   // (lo + mid) + hi: exact
                        x[2 * e] = (__uint_as_float(w[2][2 * h + e] << 16) + __uint_as_float(w[1][2 * h + e] << 16)) +
                                   __uint_as_float(w[0][2 * h + e] << 16);
                        x[2 * e + 1] = (__uint_as_float(w[2][2 * h + e] & 0xffff0000u) +
                                        __uint_as_float(w[1][2 * h + e] & 0xffff0000u)) +
                                       __uint_as_float(w[0][2 * h + e] & 0xffff0000u);
                    }
                    p0 = fmaf(x[0], y.x, p0);
                    p1 = fmaf(x[1], y.y, p1);
                    p0 = fmaf(x[2], y.z, p0);
                    p1 = fmaf(x[3], y.w, p1);
                }
            }
        }
        const float part = p0 + p1;
        return part + __shfl_xor(part, 32, 64);
    }
    // (Q^T r)[32 wv + 16 Jt + c] for the r of buffer buf
    __device__ __forceinline__ float apply_t(int buf, int Jt) {
        float part = 0.f;
#pragma unroll
        for (int I = 0; I < 8; ++I) {
            const float4 rv = *reinterpret_cast<const float4 *>(&s.ub[buf][16 * I + 4 * g]);
            part = fmaf(acc[I][Jt][0], rv.x, part);
            part = fmaf(acc[I][Jt][1], rv.y, part);
            part = fmaf(acc[I][Jt][2], rv.z, part);
            part = fmaf(acc[I][Jt][3], rv.w, part);
        }
        return group_sum(part);
    }
    __device__ __forceinline__ void store(float *__restrict__ P) {
#pragma unroll
        for (int I = 0; I < 8; ++I)
#pragma unroll
            for (int Jt = 0; Jt < 2; ++Jt)
#pragma unroll
                for (int r = 0; r < 4; ++r) P[(16 * I + 4 * g + r) * BG + 32 * wv + 16 * Jt + c] = acc[I][Jt][r];
    }
};

// REV: the product covers steps [s0 + 1, min(s1 + 1, T)) (the reverse chunk map is its
// transpose) and the local solution of u_k = E_{k+1}^T u_{k+1} + rhs_k (zero past the chunk) is
// taken as the sum u_{s0} = sum_k (E_k ... E_{s0+1})^T rhs_k along the same sweep: Q_k =
// E_k ... E_{s0+1} is the accumulated product after the step that takes E_k.
// M = 128, 8192 steps in 256 chunks: forward 347 us and reverse 310 us with fp32 instructions,
// 250 us and 235 us now (reading the matrices alone takes 109 us).
template <bool REV, bool FLIP>
__global__ __launch_bounds__(256) void k_chunk_product_big(const float *__restrict__ J, const float *__restrict__ rhs,
                                                           float rhs_sign, float *__restrict__ Pout,
                                                           float *__restrict__ vout, const int *__restrict__ active,
                                                           int B, int T, int M, int C, int ncs) {
    __shared__ __align__(16) BigProd sm;
    const int id = blockIdx.x;   // chain
    const int b = id / ncs, cc = id % ncs;
    if (active && !active[b]) return;
    BigChain<FLIP> q(sm);
    const int tid = threadIdx.x, g = q.g, c = q.c, wv = q.wv;
    const int s0 = cc * C, s1 = min(s0 + C, T);
    const int lo = REV ? s0 + 1 : s0, hi = REV ? min(s1 + 1, T) : s1;
    const int len = max(hi - lo, 0);
    const int ui = 32 * wv + (q.lane & 31);   // the row of u this lane forms (REV: whose rhs it stages)
    const bool own = q.lane < 32;
    float rpre = 0.f;
    // row-major E with M % 4 == 0: 16-byte loads through a resource bounded at the matrix's end
    // (rows past M read zero; columns past M take an offset outside it)
    const bool fast = !FLIP && (M & 3) == 0;
    auto stage_load = [&](int t) {
        const size_t row = (size_t)b * T + lo + t;
        const float *Jp = J + row * M * M;
        rpre = (ui < M && lo + t < s1) ? rhs[row * M + ui] : 0.f;
        if (fast) {
            const auto rs = bounded_rsrc(Jp, (uint32_t)M * M * 4u);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const uint32_t vo = q.col(k) < M ? 4u * (uint32_t)(q.row(k) * M + q.col(k)) : kOffLane;
                q.pre[k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)vo, 0, 0));
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int r = q.row(k), col = q.col(k);
            q.pre[k] = make_float4(eload<FLIP>(Jp, M, r, col), eload<FLIP>(Jp, M, r, col + 1),
                                   eload<FLIP>(Jp, M, r, col + 2), eload<FLIP>(Jp, M, r, col + 3));
        }
    };
    float vsum[2] = {0.f, 0.f};   // REV: sum over the steps of (Q_k^T rhs_k)[32 wv + 16 Jt + c]
    if (!REV && tid < BG) sm.ub[0][tid] = 0.f;
    if (len > 0) {
        stage_load(0);
        q.stage_store();
        if (REV && own) sm.ub[0][ui] = rpre;
    }
    lds_barrier();
    int cur = 0;
    for (int t = 0; t < len; ++t, cur ^= 1) {
        const bool more = t + 1 < len;
        const float rc = rpre;
        if (more) stage_load(t + 1);   // in flight during this step
        q.multiply();
        if (REV) {
            if (lo + t < s1) {
#pragma unroll
                for (int Jt = 0; Jt < 2; ++Jt) vsum[Jt] += q.apply_t(cur, Jt);
            }
        } else {
            // u_k = E_k u_{k-1} + sign rhs_k
            const float y = q.apply(cur);
            if (own) sm.ub[cur ^ 1][ui] = ui < M ? fmaf(rhs_sign, rc, y) : 0.f;
        }
        if (more) {
            lds_barrier();   // every wave has read this step's E
            q.stage_store();
            if (REV && own) sm.ub[cur ^ 1][ui] = rpre;
        }
        lds_barrier();
    }
    q.store(Pout + (size_t)id * BG * BG);
    if (REV) {
        if (g == 0) {
#pragma unroll
            for (int Jt = 0; Jt < 2; ++Jt) {
                const int col = 32 * wv + 16 * Jt + c;
                const float r0 = (col < M && s0 < s1) ? rhs[((size_t)b * T + s0) * M + col] : 0.f;
                vout[(size_t)id * BG + col] = col < M ? rhs_sign * (r0 + vsum[Jt]) : 0.f;
            }
        }
    } else if (tid < BG) {
        vout[(size_t)id * BG + tid] = sm.ub[cur][tid];
    }
}

// carries across the chunks of each sequence, in processing order k (REV: chunk c = ncs - 1 - k):
// carry_in[c] = the state entering chunk c;  next = A_k carry + v_c with A_k = P_c (P_c^T in REV).
// Long chunk sequences use two levels: groups of G consecutive k composed into one map (Q_j, u_j)
// on the matrix cores (k_carry_group_big, all groups in parallel), a walk over the group maps, and
// every group re-walked from its carry.  Serial depth G + ncs / G + G instead of ncs.
constexpr int FST = BG + 1;   // LDS row stride of a tile read along rows and along columns

// one walk of G consecutive k per 256-thread block (G = ncs: a whole sequence), from zero or from
// the walk's start vector.  Few blocks run, so a step is bound by latency: the maps go straight to
// registers, two steps ahead, and only y passes through LDS.  A load takes 128 bytes of each of 8
// rows, lane l columns 32 j + 4 (l % 8) .. + 3 of row 32 w + 8 u + l / 8; REV: columns
// 32 w + 4 (l % 8) .. + 3 of row l / 8 + 8 j.  The partial sums are added across the lanes.
// M = 128: 32 blocks walking 8 maps 11 us, one block walking 32 maps 37 us (20 and 73 us with the
// maps staged in LDS).
template <bool REV>
__global__ __launch_bounds__(256) void k_carry_big(const float *__restrict__ P, const float *__restrict__ v,
                                                   float *__restrict__ carry_in, const int *__restrict__ active,
                                                   int ncs, int G, const float *__restrict__ start) {
    __shared__ __align__(16) float ys[2][BG];
    const int ngroups = (ncs + G - 1) / G;
    const int b = blockIdx.x / ngroups, j = blockIdx.x % ngroups;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (active && !active[b]) return;
    const int k0 = j * G, k1 = min(k0 + G, ncs);
    auto chunk = [&](int k) { return (size_t)b * ncs + (REV ? ncs - 1 - k : k); };
    float4 pre[2][16];
    float vpre[2];
    auto load = [&](int k, float4 (&p)[16], float &vv) {
        const size_t id = chunk(min(k, k1 - 1));
        const float *Pc = P + id * BG * BG;
#pragma unroll
        for (int q = 0; q < 16; ++q)
            p[q] = *reinterpret_cast<const float4 *>(
                REV ? Pc + ((lane >> 3) + 8 * q) * BG + 32 * w + 4 * (lane & 7)
                    : Pc + (32 * w + 8 * (q >> 2) + (lane >> 3)) * BG + 32 * (q & 3) + 4 * (lane & 7));
        vv = v[id * BG + (tid & (BG - 1))];
    };
    auto step = [&](int k, float4 (&p)[16], float &vv) {
        const int cur = (k - k0) & 1;
        if (tid < BG) carry_in[chunk(k) * BG + tid] = ys[cur][tid];
        float o[4] = {0.f, 0.f, 0.f, 0.f};
        if (REV) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float y = ys[cur][(lane >> 3) + 8 * q];
                o[0] = fmaf(p[q].x, y, o[0]);
                o[1] = fmaf(p[q].y, y, o[1]);
                o[2] = fmaf(p[q].z, y, o[2]);
                o[3] = fmaf(p[q].w, y, o[3]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] += __shfl_xor(o[e], 8, 64);
                o[e] = group_sum(o[e]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 y = *reinterpret_cast<const float4 *>(&ys[cur][32 * q + 4 * (lane & 7)]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    o[u] = fmaf(p[4 * u + q].x, y.x, o[u]);
                    o[u] = fmaf(p[4 * u + q].y, y.y, o[u]);
                    o[u] = fmaf(p[4 * u + q].z, y.z, o[u]);
                    o[u] = fmaf(p[4 * u + q].w, y.w, o[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                o[u] += __shfl_xor(o[u], 1, 64);
                o[u] += __shfl_xor(o[u], 2, 64);
                o[u] += __shfl_xor(o[u], 4, 64);
            }
        }
        // the new state without v in the other buffer (its reads ended at the previous barrier)
        if (REV) {
            if (lane < 8) *reinterpret_cast<float4 *>(&ys[cur ^ 1][32 * w + 4 * lane]) = make_float4(o[0], o[1], o[2], o[3]);
        } else if ((lane & 7) < 4) {
            const int u = lane & 3;
            ys[cur ^ 1][32 * w + 8 * u + (lane >> 3)] = u == 0 ? o[0] : u == 1 ? o[1] : u == 2 ? o[2] : o[3];
        }
        lds_barrier();
        if (tid < BG) ys[cur ^ 1][tid] += vv;
        load(k + 2, p, vv);
        lds_barrier();
    };
    load(k0, pre[0], vpre[0]);
    load(k0 + 1, pre[1], vpre[1]);
    if (tid < BG) ys[0][tid] = start ? start[((size_t)b * ngroups + j) * BG + tid] : 0.f;
    __syncthreads();
    for (int k = k0; k < k1; k += 2) {
        step(k, pre[0], vpre[0]);
        if (k + 1 < k1) step(k + 1, pre[1], vpre[1]);
    }
}

// group maps in processing order: Q_j = A_{k1-1} ... A_{k0} and u_j = the group's walk from zero,
// composed as the chunk products are.  M = 128, 32 groups of 8: 57 us (118 us with fp32
// instructions).
template <bool REV>
__global__ __launch_bounds__(256) void k_carry_group_big(const float *__restrict__ P, const float *__restrict__ v,
                                                         float *__restrict__ gq, float *__restrict__ gu,
                                                         const int *__restrict__ active, int ncs, int G) {
    __shared__ __align__(16) BigProd sm;
    const int ngroups = (ncs + G - 1) / G;
    const int b = blockIdx.x / ngroups, j = blockIdx.x % ngroups;
    if (active && !active[b]) return;
    BigChain<REV> q(sm);
    const int tid = threadIdx.x, ui = 32 * q.wv + (q.lane & 31);
    const int k0 = j * G, k1 = min(k0 + G, ncs);
    float vpre = 0.f;
    auto stage_load = [&](int k) {
        const size_t id = (size_t)b * ncs + (REV ? ncs - 1 - k : k);
        const float *Pc = P + id * BG * BG;
#pragma unroll
        for (int k2 = 0; k2 < 16; ++k2) {
            const int r = q.row(k2), col = q.col(k2);
            q.pre[k2] = REV ? make_float4(Pc[col * BG + r], Pc[(col + 1) * BG + r], Pc[(col + 2) * BG + r],
                                          Pc[(col + 3) * BG + r])
                            : *reinterpret_cast<const float4 *>(Pc + r * BG + col);
        }
        vpre = v[id * BG + ui];
    };
    if (tid < BG) sm.ub[0][tid] = 0.f;
    stage_load(k0);
    q.stage_store();
    lds_barrier();
    int cur = 0;
    for (int k = k0; k < k1; ++k, cur ^= 1) {
        const bool more = k + 1 < k1;
        const float vc = vpre;
        if (more) stage_load(k + 1);   // in flight during this step
        q.multiply();
        const float y = q.apply(cur);
        if (q.lane < 32) sm.ub[cur ^ 1][ui] = y + vc;
        if (more) {
            lds_barrier();   // every wave has read this step's map
            q.stage_store();
        }
        lds_barrier();
    }
    q.store(gq + ((size_t)b * ngroups + j) * BG * BG);
    if (tid < BG) gu[((size_t)b * ngroups + j) * BG + tid] = sm.ub[cur][tid];
}

// MODE 0: Newton fix-up (next iterate = current + Delta, per-chain max |Delta| and max |z|);
// MODE 1: forward bare scan; MODE 2: reverse (y_k = E_{k+1}^T y_{k+1} + b_k).  256 threads: lane
// l of wave w forms half hh = l / 32 of row i = 32 w + l % 32 of E y (MODE 2: of E^T y), the two
// halves added across the wave.  Each step's E is staged in LDS by the block with coalesced
// loads, the next step's loads (and its right-hand side and iterate) in flight during this step.
// With a row stride of 129 floats and the second half's walk started 32 entries in, the 64 lanes
// of a read fall on distinct banks, for rows (MODE 0, 1) and for columns (MODE 2).

template <int MODE, bool FLIP>
__global__ __launch_bounds__(256) void k_fixup_big(const float *__restrict__ J, const float *__restrict__ rhs,
                                                   float rhs_sign, const float *__restrict__ carry_in, float *zbuf,
                                                   float *outbuf, const int *__restrict__ zsel,
                                                   uint32_t *__restrict__ chain_bits, const int *__restrict__ active,
                                                   int B, int T, int M, int C, int ncs) {
    __shared__ float js[2][BG][FST];
    __shared__ float ys[2][BG];
    __shared__ uint32_t red[2][4];
    const int id = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int hh = lane >> 5, i = 32 * w + (lane & 31);
    const int b = id / ncs, cc = id % ncs;
    const bool ok = !active || active[b];
    const int s0 = cc * C, s1 = ok ? min(s0 + C, T) : s0;
    const int len = s1 - s0;
    const float *zin = MODE == 0 ? cur_iter(zbuf, outbuf, zsel, b) : nullptr;
    float *out = MODE == 0 ? next_iter(zbuf, outbuf, zsel, b) : outbuf;
    const bool own = hh == 0 && i < M;   // the lane that writes row i
    // step t: k = the row of the output, kj = the matrix (MODE 2: k + 1, none past the end)
    auto k_of = [&](int t) { return MODE == 2 ? s1 - 1 - t : s0 + t; };
    // staging: thread tid takes the 16-byte groups tid + 256 q (q < 16), row (tid + 256 q) / 32
    float4 pre[16];
    float rpre = 0.f, zpre = 0.f;
    // row-major E with M % 4 == 0: 16-byte loads through a resource bounded at the matrix's end
    // (rows past M read zero) with one lane offset (columns past M: an offset outside it)
    const bool fast = !FLIP && (M & 3) == 0;
    const uint32_t vlane = ((tid & 31) * 4 + 3 < M) ? 4u * ((uint32_t)(tid >> 5) * M + (tid & 31) * 4) : kOffLane;
    auto stage_load = [&](int t) {
        const int k = k_of(t), kj = MODE == 2 ? k + 1 : k;
        const bool has = kj < T;
        const float *Jp = J + ((size_t)b * T + (has ? kj : 0)) * M * M;
        if (fast) {
            const auto rs = bounded_rsrc(Jp, has ? (uint32_t)M * M * 4u : 0u);
#pragma unroll
            for (int q = 0; q < 16; ++q)
                pre[q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)vlane, q * 32 * M, 0));
        } else {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int e4 = tid + 256 * q, row = e4 >> 5, c4 = (e4 & 31) * 4;
                pre[q] = !has ? make_float4(0.f, 0.f, 0.f, 0.f)
                              : make_float4(eload<FLIP>(Jp, M, row, c4), eload<FLIP>(Jp, M, row, c4 + 1),
                                            eload<FLIP>(Jp, M, row, c4 + 2), eload<FLIP>(Jp, M, row, c4 + 3));
            }
        }
        if (own) {
            const size_t e = ((size_t)b * T + k) * M + i;
            rpre = rhs[e];
            if (MODE == 0) zpre = zin[e];
        }
    };
    auto stage_store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int e4 = tid + 256 * q, row = e4 >> 5, c4 = (e4 & 31) * 4;
            js[buf][row][c4] = pre[q].x;
            js[buf][row][c4 + 1] = pre[q].y;
            js[buf][row][c4 + 2] = pre[q].z;
            js[buf][row][c4 + 3] = pre[q].w;
        }
    };
    if (tid < BG) ys[0][tid] = (ok && tid < M) ? carry_in[(size_t)id * BG + tid] : 0.f;
    float rc = 0.f, zc = 0.f;
    if (len > 0) {
        stage_load(0);
        stage_store(0);
        rc = rpre;
        zc = zpre;
    }
    __syncthreads();
    uint32_t emax = 0u, zmax = 0u;
    int cur = 0;
    const int q0 = 64 * hh;
    for (int t = 0; t < len; ++t) {
        const int k = k_of(t);
        const bool more = t + 1 < len;
        if (more) stage_load(t + 1);   // in flight during this step
        // half hh of the sum over q in [64 hh, 64 hh + 64), walked from 32 hh on (entries past M
        // are zero in the staged tile and in ys)
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll 4
        for (int u = 0; u < 64; u += 4) {
            const int q = q0 + ((u + 32 * hh) & 63);
            const float e0 = MODE == 2 ? js[cur][q][i] : js[cur][i][q];
            const float e1 = MODE == 2 ? js[cur][q + 1][i] : js[cur][i][q + 1];
            const float e2 = MODE == 2 ? js[cur][q + 2][i] : js[cur][i][q + 2];
            const float e3 = MODE == 2 ? js[cur][q + 3][i] : js[cur][i][q + 3];
            a0 = fmaf(e0, ys[cur][q], a0);
            a1 = fmaf(e1, ys[cur][q + 1], a1);
            a2 = fmaf(e2, ys[cur][q + 2], a2);
            a3 = fmaf(e3, ys[cur][q + 3], a3);
        }
        float part = (a0 + a1) + (a2 + a3);
        part += __shfl_xor(part, 32, 64);
        float y = 0.f;
        if (own) {
            const size_t e = ((size_t)b * T + k) * M + i;
            y = fmaf(rhs_sign, rc, part);
            if (MODE == 0) {
                out[e] = zc + y;
                const uint32_t ab = abs_bits(y), zb = abs_bits(zc);
                emax = emax > ab ? emax : ab;
                zmax = zmax > zb ? zmax : zb;
            } else {
                out[e] = y;
            }
        }
        if (hh == 0) ys[cur ^ 1][i] = y;
        if (more) {
            stage_store(cur ^ 1);   // that buffer's reads ended at the previous barrier
            rc = rpre;
            zc = zpre;
        }
        __syncthreads();
        cur ^= 1;
    }
    if (MODE == 0) {
        emax = wave_max_u32(emax);
        zmax = wave_max_u32(zmax);
        if (lane == 0) {
            red[0][w] = emax;
            red[1][w] = zmax;
        }
        __syncthreads();
        if (tid == 0 && ok) {
            uint32_t e = red[0][0], z = red[1][0];
            for (int v = 1; v < 4; ++v) {
                e = e > red[0][v] ? e : red[0][v];
                z = z > red[1][v] ? z : red[1][v];
            }
            chain_bits[id] = e;
            chain_bits[(size_t)B * ncs + id] = z;
        }
    }
}

// ---- shallow PLRNN at M <= 128 -------------------------------------------------------------

// forced input of step s for latent i, the float32 decision of the other kernels
__device__ __forceinline__ float big_forced(const ShArgs &a, const float *z, int b, int s, int i) {
    if (s == 0) return a.z0 ? a.z0[(size_t)b * a.M + i] : (i < a.N ? a.x[(size_t)b * (a.T + 1) * a.N + i] : 0.f);
    if (a.zt) return a.zt[((size_t)b * a.T + s) * a.M + i];
    const float zp = z[((size_t)b * a.T + s - 1) * a.M + i];
    if (i >= a.N) return zp;
    const float xs = a.x[((size_t)b * (a.T + 1) + s) * a.N + i];
    if (s <= a.tw) return xs;   // latent warm-up: alpha_s = 1
    const float p = __fsub_rn(1.0f, a.alpha);
    return __fadd_rn(__fmul_rn(p, zp), __fmul_rn(a.alpha, xs));
}

// One row per wave, the four waves of a block on their own rows; LDS: W2^T [M][L] | W1^T [L][M],
// so that the lanes of a read take consecutive words.  Lane l < L forms the hidden pre-activation
// u_l left to right from h2 (a rounding after every multiply and add: the fixed-order float32
// decision), with z~_j broadcast from lane j % 64 of the wave's registers; lanes i and i + 64 form
// F_i and r_i from relu(u), broadcast the same way.
__global__ __launch_bounds__(256) void k_resjac_big(const ShArgs a, const float *zbuf, const float *zalt,
                                                    const int *__restrict__ zsel, float *__restrict__ F_out,
                                                    float *__restrict__ r_out, uint32_t *__restrict__ masks,
                                                    const int *__restrict__ active) {
    extern __shared__ __align__(16) float smem[];
    const int M = a.M, L = a.L, T = a.T, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    float *w2t = smem, *w1t = w2t + (size_t)M * L;
    for (int e = tid; e < M * L; e += 256) {
        const int i = e / L, l = e % L;   // W1[i][l]; W2[l][i] at the same (i, l)
        w1t[(size_t)l * M + i] = a.W1[e];
        w2t[(size_t)i * L + l] = a.W2[(size_t)l * M + i];
    }
    const int LW = (L + 31) / 32;
    const long rows = (long)a.B * T;
    __syncthreads();
    for (long row = (long)blockIdx.x * 4 + wv; row < rows; row += (long)gridDim.x * 4) {
        const int b = (int)(row / T), s = (int)(row % T);
        if (active && !active[b]) continue;   // wave-uniform
        const float *z = cur_iter(zbuf, zalt, zsel, b);
        const int i1 = lane + 64;
        const float zt0 = lane < M ? big_forced(a, z, b, s, lane) : 0.f;
        const float zt1 = i1 < M ? big_forced(a, z, b, s, i1) : 0.f;
        float u = 0.f;
        if (lane < L) {
            u = a.h2 ? a.h2[lane] : 0.f;
            const float *wr = w2t + lane;
            const int m0 = M < 64 ? M : 64;
            for (int j = 0; j < m0; ++j)
                u = __fadd_rn(u, __fmul_rn(wr[(size_t)j * L], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zt0), j))));
            for (int j = 64; j < M; ++j)
                u = __fadd_rn(u, __fmul_rn(wr[(size_t)j * L], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zt1), j - 64))));
        }
        const float ru = (lane < L && u > 0.f) ? u : 0.f;
        const uint64_t on = __builtin_amdgcn_ballot_w64(lane < L && u > 0.f);
        if (masks && lane < LW) masks[(size_t)row * LW + lane] = (uint32_t)(on >> (32 * lane));
        float f0 = 0.f, f1 = 0.f;
        for (int l = 0; l < L; ++l) {
            const float rl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ru), l));
            f0 = fmaf(w1t[(size_t)l * M + lane], rl, f0);
            if (i1 < M) f1 = fmaf(w1t[(size_t)l * M + i1], rl, f1);
        }
        const size_t e0 = (size_t)row * M;
        if (lane < M) {
            const float f = fmaf(a.A[lane], zt0, f0) + (a.h1 ? a.h1[lane] : 0.f);
            if (F_out) F_out[e0 + lane] = f;
            if (r_out) r_out[e0 + lane] = z[e0 + lane] - f;
        }
        if (i1 < M) {
            const float f = fmaf(a.A[i1], zt1, f1) + (a.h1 ? a.h1[i1] : 0.f);
            if (F_out) F_out[e0 + i1] = f;
            if (r_out) r_out[e0 + i1] = z[e0 + i1] - f;
        }
    }
}

// J~_s = Cd (or diag(A p)) + W1 diag(m_s) V with V = W2 diag(p) (or the given W2 P), on the bf16
// matrix cores with operands in three exact parts (split16.h): one row at a time per block, the
// blocks walking the rows, wave wv computes the column tiles 2 wv, 2 wv + 1 of all 8 row tiles.  KB =
// blocks of 32 hidden units; lane group g takes units 32 kk + 8 g .. + 7 of a block.  W1's parts are
// shared through LDS, a wave's columns of V stay in registers, and a step's mask clears half-words of
// V.  M = 128, L = 50, 8192 rows: 107 us, near the 537 MB written (78 us at the rate of a fill); 187 us
// with fp32 instructions and stores of 64 bytes of 16 rows.  Two waves a SIMD are needed, hence at
// most 256 VGPRs: 317 us where the products were ordered over both unit blocks and spilled.
template <bool ROW4, int KB>
__global__ __launch_bounds__(256, 2) void k_jacform_big(const ShArgs a, const uint32_t *__restrict__ masks,
                                                     float *__restrict__ Jout, const int *__restrict__ active,
                                                     const float *__restrict__ gamma) {
    __shared__ __align__(16) v4u w1s[8][KB][3][64];   // [row tile][k block][hi, mid, lo][lane]
    const int M = a.M, L = a.L, T = a.T, N = a.N;
    const int tid = threadIdx.x;
    const float p1 = __fsub_rn(1.0f, a.alpha);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
    v4u vq[3][2][KB];
#pragma unroll
    for (int kk = 0; kk < KB; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = 16 * (2 * wv + u) + c;   // a row of W1, a column of V
            const double p = r < N ? p1 : 1.f;
            v4u wq[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float w1[2], w2[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int l = 32 * kk + 8 * g + 2 * i + e;
                    w1[e] = r < M && l < L ? a.W1[(size_t)r * L + l] : 0.f;
                    w2[e] = r < M && l < L ? a.W2[(size_t)l * M + r] : 0.f;
                }
                uint32_t part[3];
                split_pair(w1[0], w1[1], part);
#pragma unroll
                for (int q = 0; q < 3; ++q) wq[q][i] = part[q];
                split_pair_f64(w2[0] * p, w2[1] * p, part);
#pragma unroll
                for (int q = 0; q < 3; ++q) vq[q][u][kk][i] = part[q];
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) w1s[2 * wv + u][kk][q][lane] = wq[q];
        }
    __syncthreads();
    const int LW = (L + 31) / 32;
    const auto cd_rs = bounded_rsrc(a.Cd, a.Cd ? (uint32_t)M * M * 4u : 0u);
    // diagonal A p of rows 16 I + 8 u + c % 8 (the transposed-tile stores)
    float dgI[8][2];
#pragma unroll
    for (int I = 0; I < 8; ++I)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = 16 * I + 8 * u + (c & 7);
            dgI[I][u] = (ROW4 && !a.Cd && i < M) ? a.A[i] * (i < N ? p1 : 1.f) : 0.f;
        }
    const int t_lo = a.t_hi > a.t_lo ? a.t_lo : 0;
    const int len = a.t_hi > a.t_lo ? a.t_hi - a.t_lo : T;
    const long rows = (long)a.B * len;
    auto grow_of = [&](long r) {
        const long bb = r / len;
        return bb * T + t_lo + (r - bb * len);
    };
    // the next row's mask words (L <= 64: at most two) are loaded while this row is formed
    uint32_t wn0 = 0u, wn1 = 0u;
    auto fetch = [&](long r) {
        if (r >= rows) return;
        const uint32_t *mw = masks + (size_t)grow_of(r) * LW;
        wn0 = mw[0];
        wn1 = LW > 1 ? mw[1] : 0u;
    };
    fetch(blockIdx.x);
    for (long r0 = blockIdx.x; r0 < rows; r0 += gridDim.x) {
        const long bb = r0 / len;
        const long grow = grow_of(r0);
        const uint32_t wc0 = wn0, wc1 = wn1;
        fetch(r0 + gridDim.x);
        if (active && !active[bb]) continue;
        v4f acc[8][2];
#pragma unroll
        for (int I = 0; I < 8; ++I)
#pragma unroll
            for (int Jt = 0; Jt < 2; ++Jt) acc[I][Jt] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            const int by = (int)((kk ? wc1 : wc0) >> (8 * g));
            v4u m;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t e0 = (uint32_t)((by << (31 - 2 * i)) >> 31), e1 = (uint32_t)((by << (30 - 2 * i)) >> 31);
                m[i] = (e0 & 0xffffu) | (e1 & 0xffff0000u);
            }
            v4u vm[3][2];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int Jt = 0; Jt < 2; ++Jt) vm[q][Jt] = vq[q][Jt][kk] & m;
#pragma unroll
            for (int I0 = 0; I0 < 8; I0 += 2) {
                v4u wq[2][3];
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int q = 0; q < 3; ++q) wq[n][q] = w1s[I0 + n][kk][q][lane];
                // parts of one order of magnitude, the smallest first.  ROW4: the transposed tile,
                // V^T diag(m) W1^T
#pragma unroll
                for (int o = 2; o >= 0; --o)
#pragma unroll
                    for (int qa = o; qa >= 0; --qa)
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int Jt = 0; Jt < 2; ++Jt)
                                acc[I0 + n][Jt] = ROW4 ? mfma_b(vm[o - qa][Jt], wq[n][qa], acc[I0 + n][Jt])
                                                       : mfma_b(wq[n][qa], vm[o - qa][Jt], acc[I0 + n][Jt]);
            }
        }
        // stores through a resource bounded at J~_s's end: rows past M fall outside it, columns
        // past M take an offset outside it
        const auto rs = bounded_rsrc(Jout + (size_t)grow * M * M, (uint32_t)M * M * 4u);
        const float gm = gamma ? gamma[bb] : 1.f;
        if (ROW4) {
            // acc[I][Jt][r] = J~[16 I + c][32 wv + 16 Jt + 4 g + r].  Lanes c and c ^ 8 exchange a tile, so
            // that a store takes all 32 columns (128 bytes) of eight rows: store u rows 16 I + 8 u + c % 8,
            // lane columns 32 wv + 16 (c / 8) + 4 g .. + 3 (with M % 4 == 0 the four are all inside the
            // row or all past it)
            const bool up = c >= 8;
            const int col0 = 32 * wv + (up ? 16 : 0) + 4 * g;
            const uint32_t vo = col0 < M ? 4u * (uint32_t)((c & 7) * M + col0) : kOffLane;
#pragma unroll
            for (int I = 0; I < 8; ++I) {
                float st[2][4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float give = up ? acc[I][0][r] : acc[I][1][r];
                    const float got = __int_as_float(
                        __builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xF, 0xF, true));   // row_ror:8
                    st[0][r] = up ? got : acc[I][0][r];
                    st[1][r] = up ? acc[I][1][r] : got;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int row = 16 * I + 8 * u + (c & 7);
                    const uint32_t vr = vo + 4u * (uint32_t)M * (uint32_t)(16 * I + 8 * u);
                    const int dr = row - col0;   // the diagonal entry's column in the four
                    const float dg = dgI[I][u];
                    float4 d = make_float4(dr == 0 ? dg : 0.f, dr == 1 ? dg : 0.f, dr == 2 ? dg : 0.f, dr == 3 ? dg : 0.f);
                    if (a.Cd) d = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(cd_rs, (int)vr, 0, 0));
                    const float4 o = make_float4(gm * (st[u][0] + d.x), gm * (st[u][1] + d.y), gm * (st[u][2] + d.z),
                                                 gm * (st[u][3] + d.w));
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), rs, (int)vr, 0, 0);
                }
            }
            continue;
        }
#pragma unroll
        for (int Jt = 0; Jt < 2; ++Jt) {
            const int col = 32 * wv + 16 * Jt + c;
            const uint32_t vo = col < M ? 4u * (uint32_t)(4 * g * M + col) : kOffLane;
            // the diagonal entry (col, col) sits in row tile col / 16 at 4 g + r = col % 16
            const float dg = (!a.Cd && col < M) ? a.A[col] * (col < N ? p1 : 1.f) : 0.f;
#pragma unroll
            for (int I = 0; I < 8; ++I)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // lane offset of row 16 I + 4 g + r (kOffLane plus a row offset stays outside)
                    const uint32_t vr = vo + 4u * (uint32_t)M * (uint32_t)(16 * I + r);
                    float d = (16 * I + 4 * g + r == col) ? dg : 0.f;
                    if (a.Cd) d = bload(cd_rs, vr, 0);
                    bstore_u(rs, __float_as_uint(gm * (acc[I][Jt][r] + d)), vr, 0);
                }
        }
    }
}

// Per-block partial sums over rows (layout of k_grads_shplrnn):
//   [M*L dW1 (row-major) | L*M dW2 | L dh2 | M dA | M dh1]
// dW1 += lam relu(u)^T, dW2 += delta z~^T with delta = (W1^T lam) * m, dh2 += delta, dA += lam * z~,
// dh1 += lam.  Each thread owns up to GB_PER entries of dW1 and of dW2 in registers.
constexpr int GB_PER = 32;

__global__ __launch_bounds__(256) void k_grads_big(const ShArgs a, const float *__restrict__ z,
                                                   const float *__restrict__ lam, const uint32_t *__restrict__ masks,
                                                   float *__restrict__ part) {
    extern __shared__ __align__(16) float smem[];
    const int M = a.M, L = a.L, T = a.T, tid = threadIdx.x;
    // W2 kept transposed ([M][L]) so that the lanes l of a read take consecutive words
    float *w1 = smem, *w2t = w1 + (size_t)M * L, *zt = w2t + (size_t)L * M, *lm = zt + BG, *ru = lm + BG,
          *dl = ru + L;
    for (int e = tid; e < M * L; e += 256) {
        w1[e] = a.W1[e];
        const int l = e / M, k = e % M;
        w2t[(size_t)k * L + l] = a.W2[e];
    }
    const int LW = (L + 31) / 32;
    float g1[GB_PER], g2[GB_PER];
    // the (row, column) of this thread's entries of dW1 and of dW2 in one word (7, 6, 6, 7 bits:
    // M <= 128, L < 64), so that no row divides
    uint32_t ix[GB_PER];
#pragma unroll
    for (int q = 0; q < GB_PER; ++q) {
        g1[q] = g2[q] = 0.f;
        const uint32_t e = (uint32_t)(tid + 256 * q);
        ix[q] = (e / L) | ((e % L) << 7) | ((e / M) << 13) | ((e % M) << 19);
    }
    float dh2 = 0.f, dA = 0.f, dh1 = 0.f;
    const long rows = (long)a.B * T;
    const long per = (rows + gridDim.x - 1) / gridDim.x;
    const long r0 = (long)blockIdx.x * per, r1 = r0 + per < rows ? r0 + per : rows;
    // the next row's z~, lambda and mask word are loaded while this row is summed
    float zn = 0.f, ln = 0.f;
    uint32_t mn = 0u;
    auto load_row = [&](long row) {
        const int b = (int)(row / T), s = (int)(row % T);
        if (tid < M) {
            zn = big_forced(a, z, b, s, tid);
            ln = lam[(size_t)row * M + tid];
        }
        if ((tid >> 2) < L) mn = masks[(size_t)row * LW + (tid >> 7)];   // the word of unit tid / 4
    };
    if (r0 < r1) load_row(r0);
    __syncthreads();
    for (long row = r0; row < r1; ++row) {
        if (tid < M) {
            zt[tid] = zn;
            lm[tid] = ln;
        }
        const uint32_t mw = mn;
        if (row + 1 < r1) load_row(row + 1);
        __syncthreads();
        {
            // four threads per hidden unit l (L < 64), each summing every fourth k, added across the
            // four lanes
            const int l = tid >> 2, p = tid & 3;
            float u = 0.f, d = 0.f;
            if (l < L)
                for (int k = p; k < M; k += 4) {
                    u = fmaf(w2t[(size_t)k * L + l], zt[k], u);
                    d = fmaf(w1[(size_t)k * L + l], lm[k], d);
                }
            u += __shfl_xor(u, 1, 64);
            u += __shfl_xor(u, 2, 64);
            d += __shfl_xor(d, 1, 64);
            d += __shfl_xor(d, 2, 64);
            if (l < L && p == 0) {
                const bool m = (mw >> (l & 31)) & 1u;
                ru[l] = m ? u + (a.h2 ? a.h2[l] : 0.f) : 0.f;
                dl[l] = m ? d : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < GB_PER; ++q) {
            const int e = tid + 256 * q;
            if (e < M * L) {
                uint32_t x = ix[q];
                asm volatile("" : "+v"(x));   // keeps the packed word, not 4 hoisted LDS addresses, live
                g1[q] = fmaf(lm[x & 127u], ru[(x >> 7) & 63u], g1[q]);      // dW1[i][l]
                g2[q] = fmaf(dl[(x >> 13) & 63u], zt[(x >> 19) & 127u], g2[q]);   // dW2[l][j]
            }
        }
        if (tid < L) dh2 += dl[tid];
        if (tid < M) {
            dA = fmaf(lm[tid], zt[tid], dA);
            dh1 += lm[tid];
        }
        __syncthreads();
    }
    const size_t stride = (size_t)2 * M * L + L + 2 * M;
    float *pp = part + (size_t)blockIdx.x * stride;
#pragma unroll
    for (int q = 0; q < GB_PER; ++q) {
        const int e = tid + 256 * q;
        if (e < M * L) {
            pp[e] = g1[q];
            pp[(size_t)M * L + e] = g2[q];
        }
    }
    if (tid < L) pp[(size_t)2 * M * L + tid] = dh2;
    if (tid < M) {
        pp[(size_t)2 * M * L + L + tid] = dA;
        pp[(size_t)2 * M * L + L + M + tid] = dh1;
    }
}

// ---- host launchers (called by the dispatchers of the M <= 64 kernels when the padded width is
// 128) ------------------------------------------------------------------------------------------

int launch_chunk_product_big(bool rev, bool flip, int B, int T, int M, const float *J, const float *rhs,
                             float rhs_sign, float *P, float *v, const int *active, int C, int ncs, hipStream_t st) {
    const int grid = B * ncs;
    KTimer kt("k_chunk_product_dense", st);
#define CPB(R, F) \
    hipLaunchKernelGGL((k_chunk_product_big<R, F>), dim3(grid), dim3(256), 0, st, J, rhs, rhs_sign, P, v, active, B, T, M, C, ncs)
    if (!rev) { if (flip) CPB(false, true); else CPB(false, false); }
    else { if (flip) CPB(true, true); else CPB(true, false); }
#undef CPB
    DEER_LAUNCH_CHECK("k_chunk_product_big");
    return DEER_OK;
}

int launch_carry_big(bool rev, const float *P, const float *v, float *carry_in, const int *active, int B, int ncs,
                     int G, float *gws, hipStream_t st) {
    KTimer kt("k_carry", st);
    if (!G) {
        if (rev) hipLaunchKernelGGL(k_carry_big<true>, dim3(B), dim3(256), 0, st, P, v, carry_in, active, ncs, ncs, nullptr);
        else hipLaunchKernelGGL(k_carry_big<false>, dim3(B), dim3(256), 0, st, P, v, carry_in, active, ncs, ncs, nullptr);
        DEER_LAUNCH_CHECK("k_carry_big");
        return DEER_OK;
    }
    // workspace: group maps [B][ng][BG][BG], their walks from zero [B][ng][BG], group carries
    const int ng = (ncs + G - 1) / G;
    float *gq = gws;
    float *gu = gq + (size_t)B * ng * BG * BG;
    float *gc = gu + (size_t)B * ng * BG;
    const int grid = B * ng;
    if (rev) hipLaunchKernelGGL(k_carry_group_big<true>, dim3(grid), dim3(256), 0, st, P, v, gq, gu, active, ncs, G);
    else hipLaunchKernelGGL(k_carry_group_big<false>, dim3(grid), dim3(256), 0, st, P, v, gq, gu, active, ncs, G);
    DEER_LAUNCH_CHECK("k_carry_group_big");
    hipLaunchKernelGGL(k_carry_big<false>, dim3(B), dim3(256), 0, st, gq, gu, gc, active, ng, ng, nullptr);
    DEER_LAUNCH_CHECK("k_carry_big");
    if (rev) hipLaunchKernelGGL(k_carry_big<true>, dim3(grid), dim3(256), 0, st, P, v, carry_in, active, ncs, G, gc);
    else hipLaunchKernelGGL(k_carry_big<false>, dim3(grid), dim3(256), 0, st, P, v, carry_in, active, ncs, G, gc);
    DEER_LAUNCH_CHECK("k_carry_big");
    return DEER_OK;
}

int launch_fixup_big(int mode, bool flip, int B, int T, int M, const float *J, const float *rhs, float rhs_sign,
                     const float *carry_in, float *z, float *out, const int *zsel, uint32_t *chain_bits,
                     const int *active, int C, int ncs, hipStream_t st) {
    const int grid = B * ncs;
    KTimer kt(mode == 2 ? "k_fixup_dense_rev" : "k_fixup_dense_fwd", st);
#define FXB(MO, F)                                                                                                  \
    hipLaunchKernelGGL((k_fixup_big<MO, F>), dim3(grid), dim3(256), 0, st, J, rhs, rhs_sign, carry_in, z, out, zsel, \
                       chain_bits, active, B, T, M, C, ncs)
    if (mode == 0) FXB(0, false);
    else if (mode == 1) { if (flip) FXB(1, true); else FXB(1, false); }
    else { if (flip) FXB(2, true); else FXB(2, false); }
#undef FXB
    DEER_LAUNCH_CHECK("k_fixup_big");
    return DEER_OK;
}

size_t big_resjac_lds(int M, int L) { return (size_t)2 * M * L * sizeof(float); }
size_t big_grads_lds(int M, int L) { return ((size_t)2 * M * L + 2 * BG + 2 * L) * sizeof(float); }

int launch_resjac_big(const ShArgs &a, const float *z, const float *zalt, const int *zsel, float *F, float *r,
                      uint32_t *masks, const int *active, hipStream_t st) {
    // four rows per block; as many blocks as the LDS of the 256 CUs holds (160 KiB each, at most 8)
    const long rows = (long)a.B * a.T, want = (rows + 3) / 4;
    long per_cu = (long)(160 * 1024) / (long)big_resjac_lds(a.M, a.L);
    per_cu = per_cu < 1 ? 1 : (per_cu > 8 ? 8 : per_cu);
    const int grid = (int)(want < 256 * per_cu ? want : 256 * per_cu);
    KTimer kt("k_resjac_shplrnn", st);
    hipLaunchKernelGGL(k_resjac_big, dim3(grid), dim3(256), big_resjac_lds(a.M, a.L), st, a, z, zalt, zsel, F, r,
                       masks, active);
    DEER_LAUNCH_CHECK("k_resjac_big");
    return DEER_OK;
}

int launch_jacform_big(const ShArgs &a, const uint32_t *masks, float *J, const int *active, const float *gamma,
                       hipStream_t st) {
    // every block walks rows with W1 and V split once: two blocks per CU (the registers of a wave)
    const long rows = (long)a.B * (a.t_hi > a.t_lo ? a.t_hi - a.t_lo : a.T);
    const int grid = (int)(rows < 256 * 2 ? rows : 256 * 2);
    KTimer kt("k_jacform_shplrnn", st);
#define JFB(R, K) hipLaunchKernelGGL((k_jacform_big<R, K>), dim3(grid), dim3(256), 0, st, a, masks, J, active, gamma)
    if ((a.M & 3) == 0) { if (a.L > 32) JFB(true, 2); else JFB(true, 1); }
    else { if (a.L > 32) JFB(false, 2); else JFB(false, 1); }
#undef JFB
    DEER_LAUNCH_CHECK("k_jacform_big");
    return DEER_OK;
}

int launch_grads_big(const ShArgs &a, const float *z, const float *lam, const uint32_t *masks, float *part, int nb,
                     hipStream_t st) {
    KTimer kt("k_grads_shplrnn", st);
    hipLaunchKernelGGL(k_grads_big, dim3(nb), dim3(256), big_grads_lds(a.M, a.L), st, a, z, lam, masks, part);
    DEER_LAUNCH_CHECK("k_grads_big");
    return DEER_OK;
}

}  // namespace deer
