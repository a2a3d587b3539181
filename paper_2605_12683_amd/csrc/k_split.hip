// Vanilla PLRNN, 16 < M <= 64: the Newton pass's first two kernels (eqs. GTF_residual,
// GTF_DEER_update) and the adjoint's (eq. backward_recursion).
//
//   k_newton_local_plrnn   residual r_t = z_t - F(z~_{t-1}), ReLU masks m_t and the chunk-local
//                          solution v_c (from a zero carry), 16 chunks as matrix-core columns;
//                          says which chunks' masks changed since the pass before
//   k_chunk_product_split  P_c = J~_e ... J~_s of a chunk from the masks, J~_t = gamma (diag(A) +
//                          W diag(m_t)) diag(p), on the bf16 matrix cores with split operands
//   k_adjoint_walk_plrnn   the adjoint down a chunk: its local solution and the masks, or from the
//                          carry the adjoint and the parameter gradients
//
// P_c depends on the masks and the damping only.  Near the solution few ReLU decisions change
// from one Newton update to the next, so a chunk whose masks and damping are those its stored
// product was formed with keeps it: the same bits, without the 2 M^3 flops per step.
#include "common.h"
#include "launch.h"
#include "newton_ctl.h"
#include "split16.h"

namespace deer {

// mask word of 32 latents from its eight nibbles, one per byte
__device__ __forceinline__ uint32_t pack_nibbles(const uint8_t *n8) {
    const uint2 n = *reinterpret_cast<const uint2 *>(n8);
    uint32_t lo = n.x, hi = n.y;
    lo = (lo | (lo >> 4)) & 0x00ff00ffu;
    lo = (lo | (lo >> 8)) & 0xffffu;
    hi = (hi | (hi >> 4)) & 0x00ff00ffu;
    hi = (hi | (hi >> 8)) & 0xffffu;
    return lo | (hi << 16);
}

// ---------------------------------------------------------------------------------------
// residual, masks, local solution.  Block = 16 chunks (column c) x MP / 16 waves; wave w owns the
// row tile w: lane (g, c) the latents i0 = 16 w + 4 g .. i0 + 3 of chunk c.  Per step every lane
// puts relu(z~) and m p u of its latents in LDS (double-buffered, one barrier a step), and two
// products with the rows of W (A fragments in registers, fp32 matrix cores) follow:
//   F = A z~ + W relu(z~) + h,  r = z - F;     u <- gamma (A p u + W (m p u)) - r
// The rows of z and x of PD steps are in flight in a register double buffer: 8 steps of 16-byte loads,
// or 4 of scalar loads, whose addresses take more registers.  Bound by the chain of a step, half of it
// fp32 matrix instructions (32 a wave at M = 64), the rest the exchange through LDS and the barrier
// (M = 64, 32 x 131072 steps: 0.92 ms; z and x read, r and the masks written at 3.5 TB/s).  VEC: M and
// N multiples of 4 and x, z 16-byte aligned.
// The masks of four steps are put together from LDS and stored by one wave, which reads the
// words they replace ahead and reports any difference in changed[chunk].
// ---------------------------------------------------------------------------------------
template <int MP, bool VEC, bool WU>
__global__ __launch_bounds__(MP * 4) void k_newton_local_plrnn(
    const float *__restrict__ A, const float *__restrict__ W, const float *__restrict__ h, float alpha, int N,
    const float *__restrict__ x, const float *__restrict__ z0, const float *zbuf, const float *zalt,
    const int *__restrict__ zsel, float *__restrict__ r_out, uint32_t *__restrict__ masks, int *__restrict__ changed,
    float *__restrict__ vout, const int *__restrict__ active, const float *__restrict__ gamma, int B, int T, int M, int C,
    int ncs, int tw, uint32_t *mark, uint32_t pass_no) {
    constexpr int NW = MP / 16, NS = MP / 4, DQ = MP + 4, MW = MP / 32, PD = VEC ? 8 : 4, MR = 2 * PD;
    __shared__ __align__(16) float rls[2][16 * DQ], uls[2][16 * DQ];   // [buffer][chunk][latent]
    __shared__ __align__(16) uint8_t mls[MR][16][MP / 4];              // mask nibbles of the last 2 PD steps
    __shared__ int chs[2][16];
    if (mark && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(mark, pass_no, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int nchains = B * ncs;
    const int id = blockIdx.x * 16 + c;
    const bool exists = id < nchains;
    const int b = exists ? id / ncs : 0, cc = exists ? id % ncs : 0;
    const bool ok = exists && (!active || active[b]);
    const int s0 = cc * C;
    const int len = ok ? max(min(C, T - s0), 0) : 0;
    int maxlen = len;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) maxlen = max(maxlen, __shfl_xor(maxlen, off, 64));
    maxlen = __builtin_amdgcn_readfirstlane(maxlen);
    if (maxlen == 0) return;   // uniform over the block: no chunk of it runs
    float aw[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = 16 * (s / 4) + 4 * g + (s % 4), row = 16 * wv + c;
        aw[s] = (row < M && k < M) ? W[row * M + k] : 0.f;
    }
    const int i0 = 16 * wv + 4 * g;
    float Av[4], hv[4], pv[4];
    bool fo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool lat = i0 + q < M;
        Av[q] = lat ? A[i0 + q] : 0.f;
        hv[q] = lat && h ? h[i0 + q] : 0.f;
        pv[q] = p_of(i0 + q, N, alpha);
        fo[q] = i0 + q < N;
    }
    const float gm = gamma ? gamma[b] : 1.f;
    const float *z = cur_iter(zbuf, zalt, zsel, b);
    const size_t rowb = (size_t)b * T + s0;             // first row of the chunk in z
    const size_t rowx = (size_t)b * (T + 1) + s0;       // x row of step s0
    float zp[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = i0 + q;
        zp[q] = 0.f;
        if (len > 0 && i < M) {
            if (s0 == 0) zp[q] = z0 ? z0[(size_t)b * M + i] : (fo[q] ? x[rowx * N + i] : 0.f);
            else zp[q] = z[(rowb - 1) * M + i];
        }
    }
    float u[4] = {0.f, 0.f, 0.f, 0.f};
    // branch-free: a step past the chunk reads its first row, a latent past M (an unforced one)
    // latent 0; what does not apply is zeroed
    float4 zq[PD], xq[PD];
    auto fetch = [&](int t, float4 &zn, float4 &xn) {
        const bool run = t < len;
        const size_t o = run ? t : 0;
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (VEC) {
            const float4 zv = *reinterpret_cast<const float4 *>(z + (rowb + o) * M + (i0 < M ? i0 : 0));
            zn = run && i0 < M ? zv : zero;
            if (N > 0) {
                const float4 xv = *reinterpret_cast<const float4 *>(x + (rowx + o) * N + (i0 < N ? i0 : 0));
                xn = run && i0 < N ? xv : zero;
            } else {
                xn = zero;
            }
        } else {
            float zv[4], xv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float a = z[(rowb + o) * M + (i0 + q < M ? i0 + q : 0)];
                const float d = N > 0 ? x[(rowx + o) * N + (fo[q] ? i0 + q : 0)] : 0.f;
                zv[q] = run && i0 + q < M ? a : 0.f;
                xv[q] = run && fo[q] ? d : 0.f;
            }
            zn = make_float4(zv[0], zv[1], zv[2], zv[3]);
            xn = make_float4(xv[0], xv[1], xv[2], xv[3]);
        }
    };
#pragma unroll
    for (int k = 0; k < PD; ++k) fetch(k, zq[k], xq[k]);
    // masks in store: of each tile of PD steps wave w < PD / 4 takes steps 4 w .. 4 w + 3, lane (g, c)
    // step 4 w + g of chunk c
    uint32_t diff = 0u;
    for (int t0 = 0; t0 < maxlen; t0 += PD) {
        const int td = t0 + 4 * wv + g;
        const bool duty = wv < PD / 4 && td < len;
        uint32_t old0 = 0u, old1 = 0u;
        if (duty) {
            old0 = masks[(rowb + td) * MW];
            if (MW > 1) old1 = masks[(rowb + td) * MW + 1];
        }
        float4 zn2[PD], xn2[PD];
#pragma unroll
        for (int k = 0; k < PD; ++k) fetch(t0 + PD + k, zn2[k], xn2[k]);
#pragma unroll
        for (int k = 0; k < PD; ++k) {
            const int t = t0 + k;
            if (t >= maxlen) break;
            const int cur = k & 1;   // PD is even: buffer parity follows t
            const int s = s0 + t;
            const float zc[4] = {zq[k].x, zq[k].y, zq[k].z, zq[k].w}, xc[4] = {xq[k].x, xq[k].y, xq[k].z, xq[k].w};
            const bool warm = WU && s <= tw;
            float zt[4], rz[4], mu[4], uo[4];
            uint32_t nib = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float f = __fadd_rn(__fmul_rn(pv[q], zp[q]), __fmul_rn(alpha, xc[q]));
                if (WU && warm) f = xc[q];
                zt[q] = (s == 0 || !fo[q]) ? zp[q] : f;
                const bool pos = zt[q] > 0.f;
                nib |= pos ? 1u << q : 0u;
                rz[q] = pos ? zt[q] : 0.f;
                uo[q] = (WU && warm && fo[q]) ? 0.f : pv[q] * u[q];   // P_s u
                mu[q] = pos ? uo[q] : 0.f;
            }
            *reinterpret_cast<float4 *>(&rls[cur][c * DQ + i0]) = make_float4(rz[0], rz[1], rz[2], rz[3]);
            *reinterpret_cast<float4 *>(&uls[cur][c * DQ + i0]) = make_float4(mu[0], mu[1], mu[2], mu[3]);
            mls[t & (MR - 1)][c][4 * wv + g] = (uint8_t)nib;
            lds_barrier();
            v4f f0 = {0.f, 0.f, 0.f, 0.f}, f1 = f0, y0 = f0, y1 = f0;
#pragma unroll
            for (int j = 0; j < NS / 4; ++j) {
                const float4 dr = *reinterpret_cast<const float4 *>(&rls[cur][c * DQ + 16 * j + 4 * g]);
                const float4 du = *reinterpret_cast<const float4 *>(&uls[cur][c * DQ + 16 * j + 4 * g]);
                y0 = mfma16x16x4(aw[4 * j + 0], du.x, y0);
                f0 = mfma16x16x4(aw[4 * j + 0], dr.x, f0);
                y1 = mfma16x16x4(aw[4 * j + 1], du.y, y1);
                f1 = mfma16x16x4(aw[4 * j + 1], dr.y, f1);
                y0 = mfma16x16x4(aw[4 * j + 2], du.z, y0);
                f0 = mfma16x16x4(aw[4 * j + 2], dr.z, f0);
                y1 = mfma16x16x4(aw[4 * j + 3], du.w, y1);
                f1 = mfma16x16x4(aw[4 * j + 3], dr.w, f1);
            }
            float rr[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float F = fmaf(Av[q], zt[q], f0[q] + f1[q]) + hv[q];
                rr[q] = zc[q] - F;
                const float un = fmaf(gm, fmaf(Av[q], uo[q], y0[q] + y1[q]), -rr[q]);
                u[q] = t < len ? un : u[q];
                zp[q] = zc[q];
            }
            if (t < len) {
                float *ro = r_out + (rowb + t) * M + i0;
                if constexpr (VEC) {
                    if (i0 < M) *reinterpret_cast<float4 *>(ro) = make_float4(rr[0], rr[1], rr[2], rr[3]);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (i0 + q < M) ro[q] = rr[q];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PD; ++k) {
            zq[k] = zn2[k];
            xq[k] = xn2[k];
        }
        // the ring holds two tiles, so the next tile's nibbles go to the other half of it
        if (duty) {
            uint32_t w[MW];
#pragma unroll
            for (int k = 0; k < MW; ++k) {
                w[k] = pack_nibbles(&mls[td & (MR - 1)][c][8 * k]);
                masks[(rowb + td) * MW + k] = w[k];
            }
            diff |= (w[0] ^ old0) | (MW > 1 ? w[MW - 1] ^ old1 : 0u);
        }
    }
    if (ok) {
#pragma unroll
        for (int q = 0; q < 4; ++q) vout[(size_t)id * MP + i0 + q] = u[q];
    }
    int dv = diff != 0u;
    dv |= __shfl_xor(dv, 16, 64);
    dv |= __shfl_xor(dv, 32, 64);
    if (wv < 2 && g == 0) chs[wv][c] = dv;   // wave 1 found none where PD is 4
    lds_barrier();
    if (wv == 0 && g == 0 && ok) changed[id] = chs[0][c] | chs[1][c];
}

// ---------------------------------------------------------------------------------------
// chunk products.  One chunk per wave.  The accumulators of a step hold P in the 16 x 16 tiles
// (I, Jt); lane (g, c) element r is P[16 I + 4 g + r][16 Jt + c].  With the k slots of a 16x16x32
// instruction numbered k = 32 kk + 16 (e >> 2) + 4 g + (e & 3) (e the slot within the lane) these
// accumulators, split, are the next step's B operand: no data moves between lanes.
//
// A operand: gamma (W + diag A) diag(p), formed in float64 and split once, in LDS (MP = 64: 24 KB,
// shared by the four chunks of a block, all of one sequence and so of one damping); per step the
// columns whose ReLU is off are cleared, the diagonal keeping A (v_bfi between the two).
//
// Per step at M = 64: 192 matrix instructions (1.52 us on a SIMD) and about 490 vector ones
// (splitting 4096 entries, masks), where fp32 matrix instructions took 256 (3.55 us).  M = 64,
// 32 x 131072 steps: 8.4 ms for every chunk (2.05 us a step on a SIMD; 20.3 ms in fp32 with the local
// solution in the same kernel), and with the products that are kept 50 ms for the nine passes of a
// solve (125 ms for eight passes in fp32).
// REV: the adjoint's range, J~_{hi-1} ... J~_{s0+1}, hi = min(s1 + 1, T).
// ---------------------------------------------------------------------------------------
template <int MP>
constexpr int kSplitWaves = MP == 64 ? 4 : 1;   // chunks per block

template <int MP, bool REV, bool WU>
__global__ __launch_bounds__(kSplitWaves<MP> * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_chunk_product_split(
    const float *__restrict__ A, const float *__restrict__ W, float alpha, int N, const uint32_t *__restrict__ masks,
    const int *__restrict__ changed, float *__restrict__ pgam, float *__restrict__ Pout, const int *__restrict__ active,
    const float *__restrict__ gamma, int B, int T, int M, int C, int ncs, int tw) {
    constexpr int NI = MP / 16, KK = MP / 32, MW = MP / 32, NW = kSplitWaves<MP>;
    constexpr int IB = MP == 32 ? 2 : 1;   // row tiles formed together: four independent sums
    __shared__ __align__(16) v4u wls[NI][KK][3][64];   // [row tile][k block][hi, mid, lo][lane]
    __shared__ __align__(16) uint2 dls[NI][3][64];     // diag A alone: slots 0..3 of k tile I, for rows whose ReLU is off
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int nb = (ncs + NW - 1) / NW;
    const int b = blockIdx.x / nb, cc = (int)(blockIdx.x % nb) * NW + wv;
    if (active && !active[b]) return;
    const int id = b * ncs + cc, s0 = cc * C;
    const float gm = gamma ? gamma[b] : 1.f;
    // kept: the stored product is that of these masks and this damping
    const bool todo = cc < ncs && (REV || !changed || changed[id] || pgam[id] != gm);
    if constexpr (NW > 1) {
        if (!__syncthreads_or(todo)) return;
    } else {
        if (!todo) return;
    }
    for (int I = wv; I < NI; I += NW) {
        const int row = 16 * I + c;
        const double ad = row < M ? (double)A[row] * gm * p_of(row, N, alpha) : 0.0;
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                double w[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int k = 16 * j + 4 * g + 2 * h2 + e;
                    w[e] = (row < M && k < M) ? (double)W[row * M + k] * gm * p_of(k, N, alpha) : 0.0;
                    w[e] += k == row ? ad : 0.0;
                }
                uint32_t part[3];
                split_pair_f64(w[0], w[1], part);
#pragma unroll
                for (int q = 0; q < 3; ++q) reinterpret_cast<uint32_t *>(&wls[I][j >> 1][q][lane])[2 * (j & 1) + h2] = part[q];
            }
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            uint32_t part[3];
            split_pair_f64(c == 4 * g + 2 * h2 ? ad : 0.0, c == 4 * g + 2 * h2 + 1 ? ad : 0.0, part);
#pragma unroll
            for (int q = 0; q < 3; ++q) reinterpret_cast<uint32_t *>(&dls[I][q][lane])[h2] = part[q];
        }
    }
    if constexpr (NW > 1) __syncthreads();
    else wave_lds_sync();
    if (!todo) return;
    const int s1 = min(s0 + C, T);
    const int lo = REV ? s0 + 1 : s0, hi = REV ? min(s1 + 1, T) : s1;
    const int len = __builtin_amdgcn_readfirstlane(hi - lo);
    // columns kept in a latent warm-up step (P_1 drops the observed ones)
    uint32_t om[NI][2];
    if constexpr (WU) {
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const int k = 16 * j + 4 * g + 2 * h2;
                om[j][h2] = (k < N ? 0u : 0xffffu) | (k + 1 < N ? 0u : 0xffff0000u);
            }
    }

    v4f acc[NI][NI];
#pragma unroll
    for (int Jt = 0; Jt < NI; ++Jt)
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[I][Jt][r] = (16 * I + 4 * g + r == 16 * Jt + c) ? 1.f : 0.f;
    // mask words of 64 steps at a time, one step per lane, the next 64 in flight
    const size_t rowm = (size_t)b * T + lo;
    uint32_t mc[MW], mn[MW];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int k = 0; k < MW; ++k) mn[k] = t0 + lane < len ? masks[(rowm + t0 + lane) * MW + k] : 0u;
    };
    fetch(0);
    for (int t = 0; t < len; ++t) {
        if ((t & 63) == 0) {
#pragma unroll
            for (int k = 0; k < MW; ++k) mc[k] = mn[k];
            fetch(t + 64);
        }
        // P to the B operand
        v4u bq[3][KK][NI];
#pragma unroll
        for (int Jt = 0; Jt < NI; ++Jt)
#pragma unroll
            for (int I = 0; I < NI; ++I)
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    uint32_t part[3];
                    split_pair(acc[I][Jt][2 * h2], acc[I][Jt][2 * h2 + 1], part);
#pragma unroll
                    for (int q = 0; q < 3; ++q) bq[q][I >> 1][Jt][2 * (I & 1) + h2] = part[q];
                }
        // all ones in the half of each slot whose ReLU is on
        uint32_t pm[NI][2];
#pragma unroll
        for (int k = 0; k < MW; ++k) {
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)mc[k], t & 63) >> (4 * g);
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2)
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    const uint32_t l = (uint32_t)__builtin_amdgcn_sbfe((int)w, 16 * j2 + 2 * h2, 1);
                    const uint32_t u = (uint32_t)__builtin_amdgcn_sbfe((int)w, 16 * j2 + 2 * h2 + 1, 1);
                    pm[2 * k + j2][h2] = (l & 0xffffu) | (u & 0xffff0000u);
                }
        }
        uint32_t keep[NI][2];
        if constexpr (WU) {
            const bool warm = lo + t <= tw;
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    keep[j][h2] = warm ? om[j][h2] : 0xffffffffu;
                    pm[j][h2] &= keep[j][h2];
                }
        }
#pragma unroll
        for (int I0 = 0; I0 < NI; I0 += IB) {
            __builtin_amdgcn_sched_barrier(0);   // else the next tile's operands are formed early and spill
            v4f s[IB][NI];
#pragma unroll
            for (int n = 0; n < IB; ++n)
#pragma unroll
                for (int Jt = 0; Jt < NI; ++Jt) s[n][Jt] = (v4f){0.f, 0.f, 0.f, 0.f};
            v4u aq[IB][KK][3];
#pragma unroll
            for (int n = 0; n < IB; ++n)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int I = I0 + n;
                    const uint2 d2 = dls[I][q][lane];
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        const v4u w = wls[I][kk][q][lane];
#pragma unroll
                        for (int e2 = 0; e2 < 4; ++e2) {
                            const int j = 2 * kk + (e2 >> 1), h2 = e2 & 1;
                            uint32_t d = 0u;
                            if (j == I) {
                                d = h2 ? d2.y : d2.x;
                                if (WU) d &= keep[j][h2];
                            }
                            aq[n][kk][q][e2] = (pm[j][h2] & w[e2]) | (~pm[j][h2] & d);
                        }
                    }
                }
#pragma unroll
            for (int o = 2; o >= 0; --o)   // parts (qa, qb) of one order of magnitude, the smallest first
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                    for (int qa = o; qa >= 0; --qa)
#pragma unroll
                        for (int n = 0; n < IB; ++n)
#pragma unroll
                            for (int Jt = 0; Jt < NI; ++Jt) s[n][Jt] = mfma_b(aq[n][kk][qa], bq[o - qa][kk][Jt], s[n][Jt]);
#pragma unroll
            for (int n = 0; n < IB; ++n)
#pragma unroll
                for (int Jt = 0; Jt < NI; ++Jt) acc[I0 + n][Jt] = s[n][Jt];
        }
    }
    float *P = Pout + (size_t)id * MP * MP;
#pragma unroll
    for (int Jt = 0; Jt < NI; ++Jt)
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) P[(16 * I + 4 * g + r) * MP + 16 * Jt + c] = acc[I][Jt][r];
    if (!REV && pgam && lane == 0) pgam[id] = gm;
}

// ---------------------------------------------------------------------------------------
// the adjoint's walk of a chunk, lam_k = J~_{k+1}^T lam_{k+1} + g_k for k = s1 - 1 .. s0 (eq.
// backward_recursion), in the layout of k_newton_local_plrnn: 16 chunks as columns, wave w the row
// tile w of W^T, lam through double-buffered LDS, one barrier a step.
//   FINAL false: from a zero lam; the result is the chunk's local solution v_c.  The masks (formed
//     here from z and x, every row read once) are written for the chunk products.
//   FINAL true: from the carry; lam is written and the parameter gradients
//     dW += lam_k relu(z~_k)^T,  dA += lam_k o z~_k,  dh += lam_k
//     are summed over the block's 16 chunks (dW on the matrix cores, the chunks as the k
//     dimension), two steps at a time in fp32 and those sums in float64, one partial
//     gpart[block][MP][MP + 2] per block.
// z~_k = forced(z_{k-1}, x_k) serves the gradient of step k and is the mask of step k - 1's Jacobian
// term; the same rows give the MSE seed of step k - 1.  Bound by the chain of a step as
// k_newton_local_plrnn is (M = 64, 32 x 131072 steps: 0.83 ms, and 1.14 ms with the gradients; the
// lane-per-latent kernel with the gradient products on the vector units took 3.8 ms).  Rows in flight:
// 8 steps where only z and x are read in 16-byte loads, else 4 (three rows a step, or the gradient
// sums, leave no registers for more).
// ---------------------------------------------------------------------------------------
template <int MP, bool VEC, bool WU, bool GIN, bool FINAL>
__global__ __launch_bounds__(MP * 4) __attribute__((amdgpu_waves_per_eu(2))) void k_adjoint_walk_plrnn(
    const float *__restrict__ A, const float *__restrict__ W, float alpha, int N, const float *__restrict__ x,
    const float *__restrict__ z0, const float *__restrict__ z, const float *__restrict__ gin, float seed_scale,
    const float *__restrict__ carry_in, float *__restrict__ out, uint32_t *__restrict__ masks,
    float *__restrict__ gpart, int B, int T, int M, int C, int ncs, int tw) {
    constexpr int NW = MP / 16, NS = MP / 4, DQ = MP + 4, MW = MP / 32, PD = VEC && !GIN && !FINAL ? 8 : 4, MR = 2 * PD;
    __shared__ __align__(16) float lls[2][16 * DQ], rls[FINAL ? 2 : 1][16 * DQ];   // lam, relu(z~): [buffer][chunk][latent]
    __shared__ __align__(16) uint8_t mls[FINAL ? 1 : MR][16][MP / 4];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int nchains = B * ncs;
    const int id = blockIdx.x * 16 + c;
    const bool ok = id < nchains;
    const int b = ok ? id / ncs : 0, cc = ok ? id % ncs : 0;
    const int s0 = cc * C, s1 = min(s0 + C, T);
    const int len = ok ? max(s1 - s0, 0) : 0;
    int maxlen = len;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) maxlen = max(maxlen, __shfl_xor(maxlen, off, 64));
    maxlen = __builtin_amdgcn_readfirstlane(maxlen);
    float aw[NS];   // rows of W^T
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = 16 * (s / 4) + 4 * g + (s % 4), row = 16 * wv + c;
        aw[s] = (row < M && k < M) ? W[k * M + row] : 0.f;
    }
    const int i0 = 16 * wv + 4 * g;
    float Av[4], pv[4];
    bool fo[4], la[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        la[q] = i0 + q < M;
        Av[q] = la[q] ? A[i0 + q] : 0.f;
        pv[q] = p_of(i0 + q, N, alpha);
        fo[q] = i0 + q < N;
    }
    const size_t rowb = (size_t)b * T, rowx = (size_t)b * (T + 1);
    // z~_s of this lane's latents from the rows z_{s-1} (zr) and x_s (xr)
    auto forced = [&](int s, const float (&zr)[4], const float (&xr)[4], float (&zt)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float f = __fadd_rn(__fmul_rn(pv[q], zr[q]), __fmul_rn(alpha, xr[q]));
            if (WU && s <= tw) f = xr[q];
            zt[q] = (s == 0 || !fo[q]) ? zr[q] : f;
        }
    };
    // rows of step t (k = s1 - 1 - t): z_{k-1} (z_0 itself, given or [x_0; 0], for k = 0), x_k and
    // the cotangent g_k; branch-free as in the forward kernel
    auto fetch = [&](int t, float4 &zn, float4 &xn, float4 &gn) {
        const bool run = t < len;
        const int k = run ? s1 - 1 - t : s0;
        float zv[4], xv[4], gv[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (VEC) {
            const int iz = i0 < M ? i0 : 0, ix = i0 < N ? i0 : 0;
            const float4 x4 = N > 0 ? *reinterpret_cast<const float4 *>(x + (rowx + k) * N + ix) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 z4 = *reinterpret_cast<const float4 *>(z + (rowb + (k > 0 ? k - 1 : 0)) * M + iz);
            xv[0] = x4.x, xv[1] = x4.y, xv[2] = x4.z, xv[3] = x4.w;
            zv[0] = z4.x, zv[1] = z4.y, zv[2] = z4.z, zv[3] = z4.w;
            if constexpr (GIN) {
                const float4 g4 = *reinterpret_cast<const float4 *>(gin + (rowb + k) * M + iz);
                gv[0] = g4.x, gv[1] = g4.y, gv[2] = g4.z, gv[3] = g4.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                xv[q] = N > 0 ? x[(rowx + k) * N + (fo[q] ? i0 + q : 0)] : 0.f;
                zv[q] = z[(rowb + (k > 0 ? k - 1 : 0)) * M + (la[q] ? i0 + q : 0)];
                if constexpr (GIN) gv[q] = gin[(rowb + k) * M + (la[q] ? i0 + q : 0)];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            xv[q] = run && fo[q] ? xv[q] : 0.f;
            if (k == 0) zv[q] = z0 ? z0[(size_t)b * M + (la[q] ? i0 + q : 0)] : xv[q];
            zv[q] = run && la[q] ? zv[q] : 0.f;
            gv[q] = run && la[q] ? gv[q] : 0.f;
        }
        zn = make_float4(zv[0], zv[1], zv[2], zv[3]);
        xn = make_float4(xv[0], xv[1], xv[2], xv[3]);
        gn = make_float4(gv[0], gv[1], gv[2], gv[3]);
    };
    // entering step k = s1 - 1: z_k, x_{k+1} (MSE seed) and the mask z~_{k+1} > 0
    float zk[4], xk[4], zn1[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        zk[q] = len > 0 && la[q] ? z[(rowb + s1 - 1) * M + i0 + q] : 0.f;
        xk[q] = len > 0 && fo[q] ? x[(rowx + s1) * N + i0 + q] : 0.f;
    }
    forced(s1, zk, xk, zn1);
    float lam[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) lam[q] = FINAL && ok && la[q] ? carry_in[(size_t)id * MP + i0 + q] : 0.f;
    *reinterpret_cast<float4 *>(&lls[0][c * DQ + i0]) = make_float4(lam[0], lam[1], lam[2], lam[3]);
    v4f dw[NW];
    float dA[4], dh[4];
    double dws[NW][4], dAs[4], dhs[4];
    if constexpr (FINAL) {
#pragma unroll
        for (int J = 0; J < NW; ++J) {
            dw[J] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) dws[J][q] = 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dA[q] = dh[q] = 0.f;
            dAs[q] = dhs[q] = 0.0;
        }
    }
    // dW += lam relu(z~)^T of the step whose rows are in buffer `buf`
    auto grad = [&](int buf) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float lv = lls[buf][(4 * s + g) * DQ + 16 * wv + c];
#pragma unroll
            for (int J = 0; J < NW; ++J)
                dw[J] = mfma16x16x4(lv, rls[buf][(4 * s + g) * DQ + 16 * J + c], dw[J]);
        }
    };
    auto flush = [&]() {
#pragma unroll
        for (int J = 0; J < NW; ++J) {
#pragma unroll
            for (int q = 0; q < 4; ++q) dws[J][q] += (double)dw[J][q];
            dw[J] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dAs[q] += (double)dA[q];
            dhs[q] += (double)dh[q];
            dA[q] = dh[q] = 0.f;
        }
    };
    float4 zq[PD], xq[PD], gq[PD];
#pragma unroll
    for (int k = 0; k < PD; ++k) fetch(k, zq[k], xq[k], gq[k]);
    lds_barrier();
    for (int t0 = 0; t0 < maxlen; t0 += PD) {
        float4 zn2[PD], xn2[PD], gn2[PD];
#pragma unroll
        for (int k = 0; k < PD; ++k) fetch(t0 + PD + k, zn2[k], xn2[k], gn2[k]);
#pragma unroll
        for (int k8 = 0; k8 < PD; ++k8) {
            const int t = t0 + k8;
            if (t >= maxlen) break;
            const int cur = k8 & 1;   // PD is even: buffer parity follows t
            const bool run = t < len;
            const int k = s1 - 1 - t;
            const float zr[4] = {zq[k8].x, zq[k8].y, zq[k8].z, zq[k8].w}, xr[4] = {xq[k8].x, xq[k8].y, xq[k8].z, xq[k8].w};
            const float gr[4] = {gq[k8].x, gq[k8].y, gq[k8].z, gq[k8].w};
            v4f y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
            for (int j = 0; j < NS / 4; ++j) {
                const float4 d = *reinterpret_cast<const float4 *>(&lls[cur][c * DQ + 16 * j + 4 * g]);
                y0 = mfma16x16x4(aw[4 * j + 0], d.x, y0);
                y1 = mfma16x16x4(aw[4 * j + 1], d.y, y1);
                y0 = mfma16x16x4(aw[4 * j + 2], d.z, y0);
                y1 = mfma16x16x4(aw[4 * j + 3], d.w, y1);
            }
            if (FINAL && t > 0) grad(cur);   // step t - 1
            if (FINAL && (t & 1)) flush();   // short fp32 sums: their rounding is what is left
            float zt[4], rz[4];
            forced(k, zr, xr, zt);
            uint32_t nib = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool pos = zt[q] > 0.f;
                nib |= pos ? 1u << q : 0u;
                rz[q] = pos ? zt[q] : 0.f;
                const bool jon = k + 1 < T && !(WU && fo[q] && k + 1 <= tw);   // P_{k+1} = P_1 drops observed rows
                const float y = jon ? pv[q] * fmaf(Av[q], lam[q], zn1[q] > 0.f ? y0[q] + y1[q] : 0.f) : 0.f;
                float gk;
                if constexpr (GIN) gk = gr[q];
                else gk = fo[q] && (!WU || k >= tw) ? seed_scale * (zk[q] - xk[q]) : 0.f;   // warm-up states: no seed
                lam[q] = run && la[q] ? y + gk : (FINAL ? 0.f : lam[q]);
                if constexpr (FINAL) {
                    dA[q] = fmaf(lam[q], run ? zt[q] : 0.f, dA[q]);
                    dh[q] += lam[q];
                }
                zk[q] = zr[q];
                xk[q] = xr[q];
                zn1[q] = zt[q];
            }
            *reinterpret_cast<float4 *>(&lls[cur ^ 1][c * DQ + i0]) = make_float4(lam[0], lam[1], lam[2], lam[3]);
            if constexpr (FINAL) {
                *reinterpret_cast<float4 *>(&rls[cur ^ 1][c * DQ + i0]) =
                    run ? make_float4(rz[0], rz[1], rz[2], rz[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
                if (out && run) {
                    float *lo = out + (rowb + k) * M + i0;
                    if constexpr (VEC) {
                        if (i0 < M) *reinterpret_cast<float4 *>(lo) = make_float4(lam[0], lam[1], lam[2], lam[3]);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (la[q]) lo[q] = lam[q];
                    }
                }
            } else {
                mls[t & (MR - 1)][c][4 * wv + g] = (uint8_t)nib;
            }
            lds_barrier();
        }
#pragma unroll
        for (int k = 0; k < PD; ++k) {
            zq[k] = zn2[k];
            xq[k] = xn2[k];
            gq[k] = gn2[k];
        }
        if constexpr (!FINAL) {
            const int td = t0 + 4 * wv + g;
            if (wv < PD / 4 && td < len) {
#pragma unroll
                for (int k = 0; k < MW; ++k)
                    masks[(rowb + s1 - 1 - td) * MW + k] = pack_nibbles(&mls[td & (MR - 1)][c][8 * k]);
            }
        }
    }
    if constexpr (!FINAL) {
        if (ok) {
#pragma unroll
            for (int q = 0; q < 4; ++q) out[(size_t)id * MP + i0 + q] = lam[q];
        }
    } else {
        if (maxlen > 0) grad(maxlen & 1);   // the last step
        flush();
        float *gp = gpart + (size_t)blockIdx.x * MP * (MP + 2);
#pragma unroll
        for (int J = 0; J < NW; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) gp[(i0 + r) * (MP + 2) + 16 * J + c] = (float)dws[J][r];
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // the 16 chunks' sums
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                dAs[q] += __shfl_xor(dAs[q], off, 64);
                dhs[q] += __shfl_xor(dhs[q], off, 64);
            }
            if (c == 0) {
                gp[(i0 + q) * (MP + 2) + MP] = (float)dAs[q];
                gp[(i0 + q) * (MP + 2) + MP + 1] = (float)dhs[q];
            }
        }
    }
}

// ---- launchers ---------------------------------------------------------------------------
int adjoint_walk_blocks(int B, int ncs) { return (B * ncs + 15) / 16; }

// 16-byte rows of z and x: every row a multiple of four floats on a 16-byte boundary
static bool rows16(const PlrnnArgs &a, const float *z, const float *zalt) {
    return a.M % 4 == 0 && a.N % 4 == 0 && (((uintptr_t)a.x | (uintptr_t)z | (uintptr_t)zalt) & 15u) == 0;
}

int launch_newton_local_plrnn(const PlrnnArgs &a, const float *z, const float *zalt, const int *zsel, float *r,
                              uint32_t *masks, int *changed, float *v, const int *active, const float *gamma, int C,
                              int ncs, uint32_t *mark, uint32_t pass_no, hipStream_t st) {
    const int grid = (a.B * ncs + 15) / 16;
    const bool vec = rows16(a, z, zalt);
    KTimer kt("k_newton_local_plrnn", st);
#define NL(MPV, VV, WUV)                                                                                              \
    hipLaunchKernelGGL((k_newton_local_plrnn<MPV, VV, WUV>), dim3(grid), dim3(MPV * 4), 0, st, a.A, a.W, a.h, a.alpha, \
                       a.N, a.x, a.z0, z, zalt, zsel, r, masks, changed, v, active, gamma, a.B, a.T, a.M, C, ncs, a.tw, \
                       mark, pass_no)
#define NLW(MPV, VV) if (a.tw > 0) NL(MPV, VV, true); else NL(MPV, VV, false)
    if (padded_dim(a.M) == 32) {
        if (vec) NLW(32, true); else NLW(32, false);
    } else {
        if (vec) NLW(64, true); else NLW(64, false);
    }
#undef NLW
#undef NL
    DEER_LAUNCH_CHECK("k_newton_local_plrnn");
    return DEER_OK;
}

int launch_adjoint_walk_plrnn(const PlrnnArgs &a, bool fin, const float *g, float seed_scale, const float *z,
                              const float *carry, float *out, uint32_t *masks, float *gpart, int C, int ncs,
                              hipStream_t st) {
    const int grid = adjoint_walk_blocks(a.B, ncs);
    const bool vec = rows16(a, z, z) && (((uintptr_t)g | (fin ? (uintptr_t)out : 0)) & 15u) == 0;
    KTimer kt(fin ? "k_fixup_rev_plrnn" : "k_adjoint_local_plrnn", st);
#define AW(MPV, VV, WUV, GV, FV)                                                                                       \
    hipLaunchKernelGGL((k_adjoint_walk_plrnn<MPV, VV, WUV, GV, FV>), dim3(grid), dim3(MPV * 4), 0, st, a.A, a.W, a.alpha, \
                       a.N, a.x, a.z0, z, g, seed_scale, carry, out, masks, gpart, a.B, a.T, a.M, C, ncs, a.tw)
#define AWF(MPV, VV, WUV, GV) if (fin) AW(MPV, VV, WUV, GV, true); else AW(MPV, VV, WUV, GV, false)
#define AWG(MPV, VV, WUV) if (g) { AWF(MPV, VV, WUV, true); } else { AWF(MPV, VV, WUV, false); }
#define AWW(MPV, VV) if (a.tw > 0) { AWG(MPV, VV, true) } else { AWG(MPV, VV, false) }
    if (padded_dim(a.M) == 32) {
        if (vec) { AWW(32, true) } else { AWW(32, false) }
    } else {
        if (vec) { AWW(64, true) } else { AWW(64, false) }
    }
#undef AWW
#undef AWG
#undef AWF
#undef AW
    DEER_LAUNCH_CHECK("k_adjoint_walk_plrnn");
    return DEER_OK;
}

int launch_chunk_product_split(const PlrnnArgs &a, bool rev, const uint32_t *masks, const int *changed, float *pgam,
                               float *P, const int *active, const float *gamma, int C, int ncs, hipStream_t st) {
    KTimer kt(rev ? "k_chunk_product_split_rev" : "k_chunk_product_split", st);
#define CPS(MPV, RV, WUV)                                                                                              \
    hipLaunchKernelGGL((k_chunk_product_split<MPV, RV, WUV>),                                                            \
                       dim3(a.B * ((ncs + kSplitWaves<MPV> - 1) / kSplitWaves<MPV>)), dim3(kSplitWaves<MPV> * 64), 0, st, \
                       a.A, a.W, a.alpha, a.N, masks, changed, pgam, P, active, gamma, a.B, a.T, a.M, C, ncs, a.tw)
#define CPSW(MPV, RV) if (a.tw > 0) CPS(MPV, RV, true); else CPS(MPV, RV, false)
    if (padded_dim(a.M) == 32) {
        if (rev) CPSW(32, true); else CPSW(32, false);
    } else {
        if (rev) CPSW(64, true); else CPSW(64, false);
    }
#undef CPSW
#undef CPS
    DEER_LAUNCH_CHECK("k_chunk_product_split");
    return DEER_OK;
}

}  // namespace deer
