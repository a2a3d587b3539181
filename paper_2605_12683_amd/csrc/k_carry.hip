// Carries across chunks, padded widths 32 and 64.
//   forward: carry_in[c] = y_end(c-1),  y_end(c) = P_c y_end(c-1) + v_c
//   reverse: carry_in[c] = lam_{s1(c)}, lam_{s0(c)} = P_c^T lam_{s1(c)} + v_c
// In processing order k (k = c forward, c = ncs - 1 - k reverse) both read
//   carry_in[c(k)] = cur_k,  cur_{k+1} = A_k cur_k + v_{c(k)},  A_k = P_c or P_c^T.
// Two levels: groups of G consecutive k are composed into one map (Q_j, u_j), all groups at once
// (k_carry_maps), then one block per group walks the maps of the groups before it and its own
// chunks (k_carry_walk).  Walking the group maps again in every block costs less than a kernel of
// its own for them.  Serial depth G products + ncs / G + G matrix-vector steps.
#include "common.h"
#include "launch.h"

namespace deer {

// ---------------------------------------------------------------------------------------
// group maps.  Wave w < MP / 16 owns 16 columns of Q, the last wave u as column 0.  A map is the A
// operand of fp32 16x16x4 products whose accumulators are the next step's B operand (k-step 4 j + q
// takes column 16 j + 4 g + q in lane group g), so a step is matrix instructions only; the
// maps of the next PF steps are in flight.  Latency-bound: M = 32, 32 maps: 15 us (fp32 products on the
// vector units through LDS: 45 us).
// ---------------------------------------------------------------------------------------
template <int MP, bool REV>
__global__ __launch_bounds__((MP / 16 + 1) * 64) void k_carry_maps(const float *__restrict__ P,
                                                                   const float *__restrict__ v,
                                                                   float *__restrict__ gq, float *__restrict__ gu,
                                                                   const int *__restrict__ active, int ncs, int G) {
    constexpr int NI = MP / 16;
    const int ng = (ncs + G - 1) / G;
    const int b = blockIdx.x / ng, j = blockIdx.x % ng;
    if (active && !active[b]) return;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const bool vec = w == NI;
    const int k0 = j * G, k1 = min(k0 + G, ncs);
    constexpr int PF = MP == 32 ? 4 : 2;   // maps in flight
    float4 an[PF][NI][NI], vn[PF][NI];
    auto fetch = [&](int k, float4 (&a)[NI][NI], float4 (&vv)[NI]) {
        const int cc = REV ? ncs - 1 - k : k;
        const size_t id = (size_t)b * ncs + cc;
        const float *Pc = P + id * MP * MP;
#pragma unroll
        for (int I = 0; I < NI; ++I) {
#pragma unroll
            for (int jj = 0; jj < NI; ++jj) {
                if constexpr (!REV) {
                    a[I][jj] = *reinterpret_cast<const float4 *>(Pc + (16 * I + c) * MP + 16 * jj + 4 * g);
                } else {
                    const float *q = Pc + (16 * jj + 4 * g) * MP + 16 * I + c;
                    a[I][jj] = make_float4(q[0], q[MP], q[2 * MP], q[3 * MP]);
                }
            }
            vv[I] = *reinterpret_cast<const float4 *>(v + id * MP + 16 * I + 4 * g);
        }
    };
    v4f acc[NI];
#pragma unroll
    for (int I = 0; I < NI; ++I)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[I][r] = (!vec && 16 * I + 4 * g + r == 16 * w + c) ? 1.f : 0.f;
    const bool add = vec && c == 0;
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(min(k0 + p, k1 - 1), an[p], vn[p]);
    for (int kt = k0; kt < k1; kt += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            if (kt + p >= k1) break;
            const float4 (&a)[NI][NI] = an[p], (&vv)[NI] = vn[p];
            v4f s[NI];
#pragma unroll
            for (int I = 0; I < NI; ++I)
                s[I] = (v4f){add ? vv[I].x : 0.f, add ? vv[I].y : 0.f, add ? vv[I].z : 0.f, add ? vv[I].w : 0.f};
#pragma unroll
            for (int jj = 0; jj < NI; ++jj) {
#pragma unroll
                for (int I = 0; I < NI; ++I) s[I] = mfma16x16x4(a[I][jj].x, acc[jj][0], s[I]);
#pragma unroll
                for (int I = 0; I < NI; ++I) s[I] = mfma16x16x4(a[I][jj].y, acc[jj][1], s[I]);
#pragma unroll
                for (int I = 0; I < NI; ++I) s[I] = mfma16x16x4(a[I][jj].z, acc[jj][2], s[I]);
#pragma unroll
                for (int I = 0; I < NI; ++I) s[I] = mfma16x16x4(a[I][jj].w, acc[jj][3], s[I]);
            }
#pragma unroll
            for (int I = 0; I < NI; ++I) acc[I] = s[I];
            fetch(min(kt + p + PF, k1 - 1), an[p], vn[p]);
        }
    }
    const size_t gid = (size_t)b * ng + j;
    if (!vec) {
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) gq[(gid * MP + 16 * I + 4 * g + r) * MP + 16 * w + c] = acc[I][r];
    } else if (c == 0) {
#pragma unroll
        for (int I = 0; I < NI; ++I)
            *reinterpret_cast<float4 *>(gu + gid * MP + 16 * I + 4 * g) = make_float4(acc[I][0], acc[I][1], acc[I][2], acc[I][3]);
    }
}

// ---------------------------------------------------------------------------------------
// walk.  One wave per group j of sequence b: from zero through the maps of the groups 0 .. j - 1,
// then through its own chunks, writing each chunk's carry.  A lane holds KC = MP * MP / 64 entries of
// one row of a map (MP = 32: half a row; the two halves are added across the wave), the vector is
// read from LDS, and the maps of the next PF steps are in flight (M = 32, 20 groups and 32 chunks:
// 12.7 us in one launch; the two walks took 26 us in two).
// ---------------------------------------------------------------------------------------
template <int MP, bool REV>
__global__ __launch_bounds__(64) void k_carry_walk(const float *__restrict__ P, const float *__restrict__ v,
                                                   const float *__restrict__ gq, const float *__restrict__ gu,
                                                   float *__restrict__ carry_in, const int *__restrict__ active, int ncs,
                                                   int G) {
    constexpr int KC = MP * MP / 64, PF = MP == 32 ? 4 : 2;
    __shared__ __align__(16) float cs[MP];
    const int ng = (ncs + G - 1) / G;
    const int b = blockIdx.x / ng, j = blockIdx.x % ng;
    if (active && !active[b]) return;
    const int lane = threadIdx.x, i = lane % MP, q0 = lane / MP * KC;
    const int k0 = j * G, k1 = min(k0 + G, ncs), n = j + (k1 - k0);   // steps: groups, then chunks
    float m[PF][KC], vv[PF];
    auto fetch = [&](int t, float (&mt)[KC], float &vt) {
        const bool grp = t < j;
        const int k = k0 + (t - j);
        const int cc = REV ? ncs - 1 - k : k;
        const size_t id = grp ? (size_t)b * ng + t : (size_t)b * ncs + cc;
        const float *A = (grp ? gq : P) + id * MP * MP;
        vt = (grp ? gu : v)[id * MP + i];
        if (!REV || grp) {
#pragma unroll
            for (int q = 0; q < KC / 4; ++q) {
                const float4 a = *reinterpret_cast<const float4 *>(A + i * MP + q0 + 4 * q);
                mt[4 * q] = a.x;
                mt[4 * q + 1] = a.y;
                mt[4 * q + 2] = a.z;
                mt[4 * q + 3] = a.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < KC; ++q) mt[q] = A[(q0 + q) * MP + i];
        }
    };
    float cur = 0.f;
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(min(p, n - 1), m[p], vv[p]);
    for (int t0 = 0; t0 < n; t0 += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const int t = t0 + p;
            if (t >= n) break;
            if (lane < MP) {
                cs[i] = cur;
                if (t >= j) {
                    const int k = k0 + (t - j), cc = REV ? ncs - 1 - k : k;
                    carry_in[((size_t)b * ncs + cc) * MP + i] = cur;
                }
            }
            wave_lds_sync();
            float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
            for (int q = 0; q < KC / 4; ++q) {
                const float4 x = *reinterpret_cast<const float4 *>(&cs[q0 + 4 * q]);
                a0 = fmaf(m[p][4 * q], x.x, a0);
                a1 = fmaf(m[p][4 * q + 1], x.y, a1);
                a2 = fmaf(m[p][4 * q + 2], x.z, a2);
                a3 = fmaf(m[p][4 * q + 3], x.w, a3);
            }
            float s = (a0 + a1) + (a2 + a3);
            if constexpr (MP == 32) s += __shfl_xor(s, 32, 64);
            cur = s + vv[p];
            wave_lds_sync();   // every lane has read cs
            fetch(min(t + PF, n - 1), m[p], vv[p]);
        }
    }
}

// G = 0: one level (a walk over all chunks)
int launch_carry_mid(int MP, bool rev, const float *P, const float *v, float *carry_in, const int *active, int B, int ncs,
                     int G, float *gws, hipStream_t st) {
    if (G <= 0) G = ncs;
    const int ng = (ncs + G - 1) / G;
    float *gq = gws, *gu = gws ? gws + (size_t)B * ng * MP * MP : nullptr;
    KTimer kt("k_carry", st);
#define CM(MPV, R)                                                                                                   \
    {                                                                                                                \
        if (ng > 1)                                                                                                  \
            hipLaunchKernelGGL((k_carry_maps<MPV, R>), dim3(B * ng), dim3((MPV / 16 + 1) * 64), 0, st, P, v, gq, gu,    \
                               active, ncs, G);                                                                      \
        hipLaunchKernelGGL((k_carry_walk<MPV, R>), dim3(B * ng), dim3(64), 0, st, P, v, (const float *)gq,             \
                           (const float *)gu, carry_in, active, ncs, G);                                             \
    }
    if (MP == 32) {
        if (rev) CM(32, true) else CM(32, false)
    } else {
        if (rev) CM(64, true) else CM(64, false)
    }
#undef CM
    DEER_LAUNCH_CHECK("k_carry");
    return DEER_OK;
}

}  // namespace deer
