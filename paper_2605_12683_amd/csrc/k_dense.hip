// Chunked associative scan over affine pairs (J_t, b_t) with the Jacobians stored in HBM
// ([B, T, M, M], row-major per step): the bare scan of deer_scan(DEER_SCAN_DENSE) and the
// linear solve of every shallow-PLRNN Newton update (scheduled-sampling appendix, the pair
// (A_t, b_t) and its composition; eq. GTF_DEER_update; eq. backward_recursion).
//
//   k_chunk_product_dense   per chunk: P_c = J_e ... J_s and the chunk's local solution v_c from a
//                           zero carry on the matrix cores (fp32 MFMA, A operand = J_t streamed
//                           from HBM, B operand = the accumulators themselves)
//   k_fixup_dense           the chunk re-run from its carry: forward (Newton: z += Delta and
//                           max|Delta|; bare scan: y written) or reverse (y_{t-1} = J_t^T y_t + b)
// Carries across chunks: k_carry.hip (M <= 16: k_plrnn.hip).
#include "common.h"
#include "launch.h"

namespace deer {

template <int MP>
struct DGeo {
    static constexpr int NCH = 64 / MP;
};

// ---------------------------------------------------------------------------------------
// chunk products with the chunk-local solution, all four (direction, transpose) combinations.  The
// chunk is swept in processing order (forward: k = s0 .., reverse: k = s1 - 1 ..) with the step's
// matrix A_k = op(J_k) (reverse: op(J_{k+1})), op the transpose when TR:
//   Q <- A_k Q,   u <- A_k u + rhs_sign * rhs_k.
// One chain per wave; the B operand is [Q | u] (MP / 16 column tiles plus one whose column 0 is u), so
// one set of A fragments advances both, and neither LDS nor barriers are needed.  With the
// k-permutation kappa(4j+q, g) = 16j + 4g + q the accumulators are the next step's B operand, and
// the four values a lane needs for k-steps 4j..4j+3 are one 16-byte vector of row 16I + c (TR: four
// rows of column 16I + c).  The matrices of the next PF steps are in flight: a chunk is short and
// one wave or two run on a SIMD, so a step otherwise waits for its load (M = 32, 4 x 8000 steps:
// 58 us forward and 51 us reverse; with one step in flight and two chains a wave 70 us, and 155 us
// with the local solution of the reverse on the vector units).
// The first matrix of a sequence multiplies a zero state: it is loaded but not used.
// P is stored as the carries take it: Q forward, Q^T reverse.
// ---------------------------------------------------------------------------------------
template <int MP, bool REV, bool TR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MP == 64 ? 1 : 2))) void k_chunk_product_dense(
    const float *__restrict__ J, const float *__restrict__ rhs, float rhs_sign, float *__restrict__ Pout,
    float *__restrict__ vout, const int *__restrict__ active, int B, int T, int M, int C, int ncs) {
    constexpr int NI = MP / 16, PF = MP == 16 ? 8 : MP == 32 ? 4 : 2;
    const int lane = threadIdx.x, g = lane >> 4, c = lane & 15;
    const int id = blockIdx.x, b = id / ncs, s0 = (id % ncs) * C;
    if (active && !active[b]) return;
    const int s1 = min(s0 + C, T), len = s1 - s0;
    const bool vec = !TR && M == MP;   // full 16-byte rows, no padding
    float an[PF][NI][NI][4], rn[PF][NI][4];
    auto fetch = [&](int t, float (&a)[NI][NI][4], float (&r)[NI][4]) {
        const int k = REV ? s1 - 1 - t : s0 + t;
        const size_t row = (size_t)b * T + k;
        const float *Jp = J + ((size_t)b * T + (REV ? min(k + 1, T - 1) : k)) * M * M;
#pragma unroll
        for (int I = 0; I < NI; ++I) {
#pragma unroll
            for (int jj = 0; jj < NI; ++jj) {
                if (vec) {
                    const float4 v4 = *reinterpret_cast<const float4 *>(Jp + (16 * I + c) * M + 16 * jj + 4 * g);
                    a[I][jj][0] = v4.x;
                    a[I][jj][1] = v4.y;
                    a[I][jj][2] = v4.z;
                    a[I][jj][3] = v4.w;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {   // from a valid address, zeroed outside M x M
                        const int row2 = 16 * I + c, col = 16 * jj + 4 * g + q;
                        const bool in = row2 < M && col < M;
                        const float x = Jp[in ? (TR ? col * M + row2 : row2 * M + col) : 0];
                        a[I][jj][q] = in ? x : 0.f;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 16 * I + 4 * g + q;
                const float x = rhs[row * M + (i < M ? i : 0)];
                r[I][q] = c == 0 && i < M ? x : 0.f;
            }
        }
    };
    v4f acc[NI + 1][NI];
#pragma unroll
    for (int tt = 0; tt <= NI; ++tt)
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[tt][I][r] = (tt < NI && 16 * I + 4 * g + r == 16 * tt + c) ? 1.f : 0.f;
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(min(p, len - 1), an[p], rn[p]);
    for (int t0 = 0; t0 < len; t0 += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const int t = t0 + p;
            if (t >= len) break;
            const int k = REV ? s1 - 1 - t : s0 + t;
            if (REV ? k + 1 < T : k > 0) {
#pragma unroll
                for (int tt = 0; tt <= NI; ++tt) {
                    v4f s[NI];
#pragma unroll
                    for (int I = 0; I < NI; ++I) s[I] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int jj = 0; jj < NI; ++jj)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int I = 0; I < NI; ++I) s[I] = mfma16x16x4(an[p][I][jj][q], acc[tt][jj][q], s[I]);
#pragma unroll
                    for (int I = 0; I < NI; ++I) acc[tt][I] = s[I];
                }
            }
#pragma unroll
            for (int I = 0; I < NI; ++I)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[NI][I][q] = fmaf(rhs_sign, rn[p][I][q], acc[NI][I][q]);
            fetch(min(t + PF, len - 1), an[p], rn[p]);
        }
    }
    float *P = Pout + (size_t)id * MP * MP;
#pragma unroll
    for (int tt = 0; tt < NI; ++tt)
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            if constexpr (REV) {
                *reinterpret_cast<float4 *>(P + (16 * tt + c) * MP + 16 * I + 4 * g) =
                    make_float4(acc[tt][I][0], acc[tt][I][1], acc[tt][I][2], acc[tt][I][3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) P[(16 * I + 4 * g + r) * MP + 16 * tt + c] = acc[tt][I][r];
            }
        }
    if (c == 0) {
#pragma unroll
        for (int I = 0; I < NI; ++I)
            *reinterpret_cast<float4 *>(vout + (size_t)id * MP + 16 * I + 4 * g) =
                make_float4(acc[NI][I][0], acc[NI][I][1], acc[NI][I][2], acc[NI][I][3]);
    }
}

// MODE 0: forward Newton fix-up (next iterate = current + Delta, in place when the two buffers
//         coincide; per-chain max |Delta| and max |z|)
// MODE 1: forward bare scan (y written)
// MODE 2: reverse (y_k = J_{k+1}^T y_{k+1} + b_k written)
// FLIP (modes 1, 2): the other orientation of the stored matrices, as in k_chunk_product_dense
template <int MP, int MODE, bool FLIP>
__global__ __launch_bounds__(64) void k_fixup_dense(const float *__restrict__ J, const float *__restrict__ rhs,
                                                    float rhs_sign, const float *__restrict__ carry_in,
                                                    float *zbuf, float *outbuf, const int *__restrict__ zsel,
                                                    uint32_t *__restrict__ chain_bits,
                                                    const int *__restrict__ active, int B, int T, int M, int C,
                                                    int ncs) {
    using G = DGeo<MP>;
    __shared__ __align__(16) float lds[64];
    const int lane = threadIdx.x, n = lane / MP, i = lane % MP;
    const int id = blockIdx.x * G::NCH + n;
    const bool ok0 = id < B * ncs;
    const int b = ok0 ? id / ncs : 0, cc = ok0 ? id % ncs : 0;
    const bool ok = ok0 && (!active || active[b]);
    const int s0 = cc * C, s1 = ok ? min(s0 + C, T) : s0;
    // MODE 0: iterate buffers (zbuf, outbuf) selected per sequence; MODE 1, 2: y = outbuf
    const float *zin = MODE == 0 ? cur_iter(zbuf, outbuf, zsel, b) : nullptr;
    float *out = MODE == 0 ? next_iter(zbuf, outbuf, zsel, b) : outbuf;
    float y = (ok && i < M) ? carry_in[(size_t)id * MP + i] : 0.f;
    uint32_t emax = 0u, zmax = 0u;
    const int maxlen = __builtin_amdgcn_readfirstlane(C);
    // the row (column, reverse) of J~ a step uses, its right-hand side and the iterate are
    // loaded one step ahead
    auto fetch = [&](int t, float *jv, float &bv, float &zv) {
        const int k = MODE == 2 ? s1 - 1 - t : s0 + t;
        const bool run = (MODE == 2 ? k >= s0 : k < s1) && i < M;
        const size_t e = ((size_t)b * T + k) * M + i;
        if ((MODE != 2) == FLIP) {
            // column i of J_k (forward, flipped) or of J_{k+1} (reverse)
            const int kj = MODE == 2 ? k + 1 : k;
            const bool has = run && kj < T;
            const float *Jc = J + ((size_t)b * T + kj) * M * M + i;
#pragma unroll
            for (int q = 0; q < MP; ++q) jv[q] = (has && q < M) ? Jc[(size_t)q * M] : 0.f;
        } else if (MODE != 2) {
            const float *Jr = J + (((size_t)b * T + k) * M + i) * M;
            if ((M & 3) == 0) {   // 16-byte aligned rows: vector loads
                const float4 *J4 = reinterpret_cast<const float4 *>(Jr);
#pragma unroll
                for (int q = 0; q < MP / 4; ++q) {
                    const float4 v4 = (run && 4 * q < M) ? J4[q] : make_float4(0.f, 0.f, 0.f, 0.f);
                    jv[4 * q] = v4.x;
                    jv[4 * q + 1] = v4.y;
                    jv[4 * q + 2] = v4.z;
                    jv[4 * q + 3] = v4.w;
                }
            } else {
#pragma unroll
                for (int q = 0; q < MP; ++q) jv[q] = (run && q < M) ? Jr[q] : 0.f;
            }
        } else {
            // row i of J_{k+1} (reverse, flipped)
            const bool has = run && k + 1 < T;
            const float *Jr = J + (((size_t)b * T + k + 1) * M + i) * M;
#pragma unroll
            for (int q = 0; q < MP; ++q) jv[q] = (has && q < M) ? Jr[q] : 0.f;
        }
        bv = run ? rhs[e] : 0.f;
        zv = (MODE == 0 && run) ? zin[e] : 0.f;
    };
    float jn[MP], bn, zn;
    fetch(0, jn, bn, zn);
    for (int t = 0; t < maxlen; ++t) {
        const int k = MODE == 2 ? s1 - 1 - t : s0 + t;
        const bool run = (MODE == 2 ? k >= s0 : k < s1) && i < M;
        float jc[MP];
#pragma unroll
        for (int q = 0; q < MP; ++q) jc[q] = jn[q];
        const float bc = bn, zc = zn;
        fetch(t + 1, jn, bn, zn);
        lds[lane] = y;
        lds_barrier();
        float acc = 0.f;
        {
            const float *l = lds + n * MP;
#pragma unroll
            for (int q = 0; q < MP; ++q) acc = fmaf(jc[q], l[q], acc);
        }
        lds_barrier();
        if (run) {
            const size_t e = ((size_t)b * T + k) * M + i;
            y = fmaf(rhs_sign, bc, acc);
            if (MODE == 0) {
                const float zo = zc;
                out[e] = zo + y;
                const uint32_t ab = abs_bits(y), zb = abs_bits(zo);
                emax = emax > ab ? emax : ab;
                zmax = zmax > zb ? zmax : zb;
            } else {
                out[e] = y;
            }
        }
    }
    if (MODE == 0) {
#pragma unroll
        for (int off = MP / 2; off > 0; off >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)emax, off, 64);
            const uint32_t oz = (uint32_t)__shfl_xor((int)zmax, off, 64);
            emax = emax > o ? emax : o;
            zmax = zmax > oz ? zmax : oz;
        }
        if (ok && i == 0) {   // per-chain maxima, reduced per sequence by k_seq_max
            chain_bits[id] = emax;
            chain_bits[(size_t)B * ncs + id] = zmax;
        }
    }
}

int launch_chunk_product_dense(bool rev, int B, int T, int M, const float *J, const float *rhs, float rhs_sign,
                               float *P, float *v, const int *active, int C, int ncs, hipStream_t st, bool flip) {
    const int MP = padded_dim(M);
    if (MP == 128) return launch_chunk_product_big(rev, flip, B, T, M, J, rhs, rhs_sign, P, v, active, C, ncs, st);
    KTimer kt("k_chunk_product_dense", st);
#define CPD(MPV, R, TRV)                                                                                             \
    hipLaunchKernelGGL((k_chunk_product_dense<MPV, R, TRV>), dim3(B * ncs), dim3(64), 0, st, J, rhs, rhs_sign, P, v,   \
                       active, B, T, M, C, ncs)
#define CPW(R, TRV) { if (MP == 16) CPD(16, R, TRV); else if (MP == 32) CPD(32, R, TRV); else CPD(64, R, TRV); }
    const bool tr = rev != flip;   // the direction's default orientation, or the other
    if (rev) {
        if (tr) CPW(true, true) else CPW(true, false)
    } else {
        if (tr) CPW(false, true) else CPW(false, false)
    }
#undef CPW
#undef CPD
    DEER_LAUNCH_CHECK("k_chunk_product_dense");
    return DEER_OK;
}

int launch_fixup_dense(int mode, int B, int T, int M, const float *J, const float *rhs, float rhs_sign,
                       const float *carry_in, float *z, float *out, const int *zsel, uint32_t *chain_bits,
                       const int *active, int C, int ncs, hipStream_t st, bool flip) {
    const int MP = padded_dim(M);
    if (MP == 128)
        return launch_fixup_big(mode, flip, B, T, M, J, rhs, rhs_sign, carry_in, z, out, zsel, chain_bits, active, C,
                                ncs, st);
    const int nch = B * ncs;
    const int grid = (nch + (64 / MP) - 1) / (64 / MP);
    KTimer kt(mode == 2 ? "k_fixup_dense_rev" : "k_fixup_dense_fwd", st);
#define FXD(MPV, MO, FL)                                                                                          \
    hipLaunchKernelGGL((k_fixup_dense<MPV, MO, FL>), dim3(grid), dim3(64), 0, st, J, rhs, rhs_sign, carry_in, z, out, \
                       zsel, chain_bits, active, B, T, M, C, ncs)
#define FXD3(MO, FL) \
    if (MP == 16) FXD(16, MO, FL); else if (MP == 32) FXD(32, MO, FL); else FXD(64, MO, FL);
    if (mode == 0) { FXD3(0, false) }
    else if (mode == 1) { if (flip) { FXD3(1, true) } else { FXD3(1, false) } }
    else { if (flip) { FXD3(2, true) } else { FXD3(2, false) } }
#undef FXD3
#undef FXD
    DEER_LAUNCH_CHECK("k_fixup_dense");
    return DEER_OK;
}

}  // namespace deer
