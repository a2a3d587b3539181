// Shallow PLRNN Newton update without a stored Jacobian (eq. shplrnn_nonlinear with V = W2,
// b = h2; eq. GTF_DEER_update).  The forced Jacobian of step t,
//   J~_t = gamma (diag(A p) + W1 diag(m_t) W2 diag(p)),   m_t = (W2 z~_{t-1} + h2 > 0),
// is never written to HBM: the residual kernel leaves the hidden masks m_t (L bits per step),
// and the two kernels here rebuild what they need of J~_t from them and from W1, W2.
//
//   k_chunk_aggregates_sh    per chunk, J~_t^T formed on the matrix cores (K = L, the masks
//        applied to the W1 operand) lands in exactly the register layout of an A operand of
//        J~_t, so the composition P <- J~_t P follows at once.  A wave owns one chunk and forms
//        the Jacobians of NT consecutive steps per pass over the W1 / W2 tiles in LDS.
//   k_fixup_shjvp            the chunk re-run from its carry with J~_t applied as a
//        Jacobian-vector product, Delta_t = gamma (A p Delta + W1 (m_t (W2 (p Delta)))) + s r_t.
//        A block runs 16 chains as the 16 columns of two matrix-core products per step; its 4
//        waves split the hidden units, hold their slices of W2 diag(p) and W1 as A fragments in
//        registers for the whole chunk, and sum their partial W1 products through LDS.  The same
//        walk from a zero carry gives the chunk-local solutions (in k_chunk_aggregates_sh).
// Per step this replaces 4 M^2 bytes written and read twice by 4 L / 8 bytes of masks.
#include "common.h"
#include "launch.h"
#include "newton_ctl.h"
#include "split16.h"

namespace deer {

static int shf_LP(int L) { return (L + 15) / 16 * 16; }

// l tiles per wave of the walks (4 waves share the (L + 15) / 16 tiles)
static int shf_nlw(int L) {
    const int nlt = (L + 15) / 16;
    const int per = (nlt + 3) / 4;
    return per <= 1 ? 1 : per <= 2 ? 2 : per <= 4 ? 4 : per <= 8 ? 8 : 0;
}

// groups of four waves in a block of k_chunk_aggregates_sh: the split weights of the largest sizes
// (nlw MP = 128: up to 96 KB) leave one block on a CU, which then has two
static constexpr int shf_groups(int MP, int nlw) { return nlw * MP == 128 ? 2 : 1; }

// chunk products: W1 and W2 in three parts in blocks of 32 units, and the mask table; local walk: per
// group double-buffered partial sums of the four waves and the maxima
size_t shfused_product_lds(int M, int L) {
    const size_t MP = padded_dim(M), prod = 12 * MP * ((L + 31) / 32 * 32) + 256 * sizeof(v4u);
    const size_t walk = (2 * 4 * (MP / 16) * 64 * sizeof(v4f) + 4 * 16 * 2 * sizeof(uint32_t)) * shf_groups((int)MP, shf_nlw(L));
    return prod > walk ? prod : walk;
}

size_t shf_resjac_lds(int M, int L);

bool shfused_supported(int M, int L) {
    const int MP = padded_dim(M);
    if (MP > 64 || L <= 0) return false;
    if (shf_resjac_lds(M, L) > 80 * 1024) return false;   // two blocks per CU
    const int nlw = shf_nlw(L);
    // fix-up A fragments in registers: NLW * (MP / 4) + (MP / 16) * 4 NLW floats per lane
    return nlw > 0 && nlw * (MP / 4 + MP / 4) <= 64;
}

// ---------------------------------------------------------------------------------------
// chunk products on the bf16 matrix cores with operands in three exact parts (split16.h).  Per step
//   J^T tile (I, Jt) = sum_l (W2 diag p)[l, 16 I + .] m_l W1[16 Jt + ., l]
// from the two weights, split once per block into LDS (the parts of eight l per lane and tile) with
// W1's half-words cleared where the unit is off; a block of 32 units takes the lane's eight mask bits
// through a 256-entry table of half-word masks.  A lane of the accumulator holds J[16 Jt + c][16 I +
// 4 g + r], which is slot (I & 1, r) of k block I >> 1 of an A operand with the k slots numbered as in
// k_chunk_product_split, so with the diagonal added and split again it composes at once, P <- J~ P.
// A wave owns one chunk and forms the Jacobians of NT consecutive steps together (one read of the
// weights from LDS for all of them).
//
// A chunk whose masks are those of the pass before (masks_prev) and whose damping is that of its
// stored product keeps it; masks_prev null: every product is formed.
// forward: P_c = J~_{s1-1} ... J~_{s0};  REV (the adjoint): J~_{hi-1} ... J~_{s0+1}, hi = min(s1 + 1, T).
//
// M = 32, L = 256: a step is 216 matrix instructions (1.72 us on a SIMD) and about 450 vector ones,
// where fp32 matrix instructions took 320 (4.4 us); 8 x 65536 steps: 1.2 ms for every chunk of the
// adjoint against 2.6 ms in fp32.
// ---------------------------------------------------------------------------------------
template <int MP, int NT, int NWV, bool REV, bool WU>
__device__ __forceinline__ void sh_chunk_product(const ShArgs &a, const uint32_t *__restrict__ masks,
                                                 const uint32_t *__restrict__ masks_prev,
                                                 const float *__restrict__ gamma, float *__restrict__ pgam,
                                                 float *__restrict__ Pout, const int *__restrict__ active, int C,
                                                 int ncs, int LB, int block, v4u *smem4) {
    constexpr int NI = MP / 16, KK = (MP + 31) / 32, NV = (NT * 16 + 63) / 64;
    constexpr int NTB = NT * NI < 4 ? NT : 4 / NI;   // steps whose sums run together: four independent ones
    v4u *wa = smem4;                       // [LB][NI][part][64]  (W2 diag p)^T
    v4u *wb = smem4 + LB * NI * 192;       // [LB][NI][part][64]  W1
    v4u *lut = smem4 + 2 * LB * NI * 192;  // [256] half-word masks of eight bits
    const int M = a.M, L = a.L, T = a.T, N = a.N, LW = (L + 31) / 32;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int id = block * NWV + wv;
    const bool exists = id < a.B * ncs;
    const int b = exists ? id / ncs : 0, s0 = exists ? (id % ncs) * C : 0;
    const int s1 = min(s0 + C, T);
    const float gm = gamma ? gamma[b] : 1.f;
    bool todo = exists && (!active || active[b]);
    if (!REV && masks_prev && todo && pgam[id] == gm) {
        const size_t w0 = ((size_t)b * T + s0) * LW;
        const int nw = (s1 - s0) * LW;
        uint32_t d = 0u;
        for (int e = lane; e < nw; e += 64) d |= masks[w0 + e] ^ masks_prev[w0 + e];
        todo = __builtin_amdgcn_ballot_w64(d != 0u) != 0ull;
    }
    if (!__syncthreads_or(todo)) return;
    // table: half-word k of entry e is all ones where bit k of e is set
    if (tid < 256) {
        v4u t;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            t[k] = ((tid >> (2 * k)) & 1 ? 0xffffu : 0u) | ((tid >> (2 * k + 1)) & 1 ? 0xffff0000u : 0u);
        lut[tid] = t;
    }
    for (int e = tid; e < LB * NI * 64; e += NWV * 64) {
        const int ln = e & 63, I = (e >> 6) % NI, kb = (e >> 6) / NI;
        const int i = 16 * I + (ln & 15), l0 = 32 * kb + 8 * (ln >> 4);
        const double p = p_of(i, N, a.alpha);
        v4u pa[3], pb[3];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            float w2[2], w1[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int l = l0 + 2 * e2 + k;
                const bool ok = i < M && l < L;
                w2[k] = ok ? a.W2[(size_t)l * M + i] : 0.f;
                w1[k] = ok ? a.W1[(size_t)i * L + l] : 0.f;
            }
            uint32_t part[3];
            split_pair_f64(w2[0] * p, w2[1] * p, part);
#pragma unroll
            for (int q = 0; q < 3; ++q) pa[q][e2] = part[q];
            split_pair(w1[0], w1[1], part);
#pragma unroll
            for (int q = 0; q < 3; ++q) pb[q][e2] = part[q];
        }
        const int o = (kb * NI + I) * 192 + ln;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            wa[o + 64 * q] = pa[q];
            wb[o + 64 * q] = pb[q];
        }
    }
    __syncthreads();
    if (!todo) return;

    float dgr[NI][4];   // the diagonal of row 16 Jt + c, in the lane and slot that hold it
#pragma unroll
    for (int Jt = 0; Jt < NI; ++Jt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * Jt + c;
            dgr[Jt][r] = (c == 4 * g + r && row < M) ? (float)((double)a.A[row] * gm * p_of(row, N, a.alpha)) : 0.f;
        }
    v4f acc[NI][NI];
#pragma unroll
    for (int tt = 0; tt < NI; ++tt)
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[I][tt][r] = (16 * I + 4 * g + r == 16 * tt + c) ? 1.f : 0.f;
    const int lo = REV ? s0 + 1 : s0, hi = REV ? min(s1 + 1, T) : s1;
    const int len = __builtin_amdgcn_readfirstlane(hi - lo);
    // mask words of NT steps, one per lane, the next NT steps' in flight
    const uint32_t *mrow = masks + ((size_t)b * T + lo) * LW;
    uint32_t mc[NV], mn[NV];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int e = 64 * k + lane;
            mn[k] = (e < NT * LW && t0 * LW + e < len * LW) ? mrow[t0 * LW + e] : 0u;
        }
    };
    if (len > 0) fetch(0);
    for (int t0 = 0; t0 < len; t0 += NT) {
        const int nv = min(NT, len - t0);
#pragma unroll
        for (int k = 0; k < NV; ++k) mc[k] = mn[k];
        fetch(t0 + NT);
        v4f jt[NT][NI][NI];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int I = 0; I < NI; ++I)
#pragma unroll
                for (int Jt = 0; Jt < NI; ++Jt) jt[nt][I][Jt] = (v4f){0.f, 0.f, 0.f, 0.f};
        for (int kb = 0; kb < LB; ++kb) {
            v4u oa[NI][3];
#pragma unroll
            for (int I = 0; I < NI; ++I)
#pragma unroll
                for (int q = 0; q < 3; ++q) oa[I][q] = wa[((kb * NI + I) * 3 + q) * 64 + lane];
            v4u pm[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int e = nt * LW + kb;   // steps past the chunk have zero masks (and are not composed)
                uint32_t w;
                if (NV == 1 || e < 64) w = (uint32_t)__builtin_amdgcn_readlane((int)mc[0], e & 63);
                else w = (uint32_t)__builtin_amdgcn_readlane((int)mc[NV - 1], e & 63);
                pm[nt] = lut[(w >> (8 * g)) & 255u];
            }
#pragma unroll
            for (int Jt = 0; Jt < NI; ++Jt) {
                v4u ob[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) ob[q] = wb[((kb * NI + Jt) * 3 + q) * 64 + lane];
#pragma unroll
                for (int n0 = 0; n0 < NT; n0 += NTB) {
                    v4u bm[NTB][3];
#pragma unroll
                    for (int n = 0; n < NTB; ++n)
#pragma unroll
                        for (int q = 0; q < 3; ++q) bm[n][q] = ob[q] & pm[n0 + n];
#pragma unroll
                    for (int o = 2; o >= 0; --o)   // parts of one order of magnitude, the smallest first
#pragma unroll
                        for (int qa = o; qa >= 0; --qa)
#pragma unroll
                            for (int n = 0; n < NTB; ++n)
#pragma unroll
                                for (int I = 0; I < NI; ++I)
                                    jt[n0 + n][I][Jt] = mfma_b(oa[I][qa], bm[n][o - qa], jt[n0 + n][I][Jt]);
                }
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt >= nv) break;
            const int t = t0 + nt;
            // P to the B operand
            v4u bq[3][KK][NI];
#pragma unroll
            for (int tt = 0; tt < NI; ++tt)
#pragma unroll
                for (int I = 0; I < 2 * KK; ++I)
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2) {
                        uint32_t part[3] = {0u, 0u, 0u};
                        if (I < NI) split_pair(acc[I < NI ? I : 0][tt][2 * h2], acc[I < NI ? I : 0][tt][2 * h2 + 1], part);
#pragma unroll
                        for (int q = 0; q < 3; ++q) bq[q][I >> 1][tt][2 * (I & 1) + h2] = part[q];
                    }
            // a latent warm-up step's P_1 drops the observed latents' columns
            const bool warm = WU && lo + t <= a.tw;
#pragma unroll
            for (int Jt = 0; Jt < NI; ++Jt) {
                if constexpr (NI == 4) __builtin_amdgcn_sched_barrier(0);   // else operands formed early spill
                v4u aq[3][KK];
#pragma unroll
                for (int I = 0; I < 2 * KK; ++I)
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2) {
                        uint32_t part[3] = {0u, 0u, 0u};
                        if (I < NI) {
                            const int Ic = I < NI ? I : 0, k = 16 * I + 4 * g + 2 * h2;
                            float v0 = jt[nt][Ic][Jt][2 * h2], v1 = jt[nt][Ic][Jt][2 * h2 + 1];
                            v0 = I == Jt ? fmaf(v0, gm, dgr[Jt][2 * h2]) : v0 * gm;
                            v1 = I == Jt ? fmaf(v1, gm, dgr[Jt][2 * h2 + 1]) : v1 * gm;
                            if (WU && warm) {
                                v0 = k < N ? 0.f : v0;
                                v1 = k + 1 < N ? 0.f : v1;
                            }
                            split_pair(v0, v1, part);
                        }
#pragma unroll
                        for (int q = 0; q < 3; ++q) aq[q][I >> 1][2 * (I & 1) + h2] = part[q];
                    }
                v4f s[NI];
#pragma unroll
                for (int tt = 0; tt < NI; ++tt) s[tt] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int o = 2; o >= 0; --o)
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                        for (int qa = o; qa >= 0; --qa)
#pragma unroll
                            for (int tt = 0; tt < NI; ++tt) s[tt] = mfma_b(aq[qa][kk], bq[o - qa][kk][tt], s[tt]);
#pragma unroll
                for (int tt = 0; tt < NI; ++tt) acc[Jt][tt] = s[tt];
            }
        }
    }
    float *P = Pout + (size_t)id * MP * MP;
#pragma unroll
    for (int tt = 0; tt < NI; ++tt)
#pragma unroll
        for (int I = 0; I < NI; ++I)
#pragma unroll
            for (int r = 0; r < 4; ++r) P[(16 * I + 4 * g + r) * MP + 16 * tt + c] = acc[I][tt][r];
    if (!REV && pgam && lane == 0) pgam[id] = gm;
}

// ---------------------------------------------------------------------------------------
// fix-ups.  Block = 16 chains (column c = lane & 15) x 4 waves; wave w owns the l tiles
// lt = NLW w + k.  Per step, with y tiles dl[I] (lane (g, c) element r = y[16I + 4g + r] of
// chain c, replicated in all 4 waves):
//   forward (Newton, REV false), J~_t y at step k = s0 + t, masks of step k:
//     u[k] = (W2 diag(p))[tile lt, :] y,  u *= m,  p2[I] = W1[tile I, wave's tiles] u
//     next = gamma (p2 + A p y) - r_k; z_k += next, per-chain max |Delta| and max |z|
//   reverse (adjoint, REV true), J~_{k+1}^T y at step k = s1 - 1 - t, masks of step k + 1:
//     u[k] = W1^T[tile lt, :] y,  u *= m,  p2[I] = (W2 diag(p))^T[tile I, wave's tiles] u
//     next = (p2 + A p y) + s g_k  (no J term when k + 1 = T); y_k written
// A = the first factor's rows as A fragments, B = y or u in the k-permuted accumulator layout.
// LOCAL: from y = 0 instead of the carry, the chunk's last y (the local solution) written to
// outbuf[chain][MP] and nothing else.
// The waves' contributions (wave 0 adds the diagonal and the right-hand side) are summed in
// LDS in a fixed order, so every wave holds the same next y.  NG groups of four waves may share a
// block, each with its own 16 chains and LDS and all with the steps of the longest.
// ---------------------------------------------------------------------------------------
template <int MP>
struct ShWalkLds {
    v4f red[2][4][MP / 16][64];
    uint32_t mx[4][16][2];
};

template <int MP, int NLW, int NG, bool REV, bool LOCAL>
__device__ __forceinline__ void shjvp_walk(const ShArgs &a, const uint32_t *__restrict__ masks,
                                           const float *__restrict__ rhs, float rhs_sign,
                                           const float *__restrict__ gamma, const float *__restrict__ carry_in,
                                           float *zbuf, float *outbuf, const int *__restrict__ zsel,
                                           uint32_t *__restrict__ chain_bits, const int *__restrict__ active, int C,
                                           int ncs, const FusedCtl &fc, int block, ShWalkLds<MP> *smg) {
    constexpr int NI = MP / 16, NS = MP / 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = NG > 1 ? wave >> 2 : 0, wv = wave & 3,
              lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    auto &red = smg[grp].red;
    auto &mx = smg[grp].mx;
    const int M = a.M, L = a.L, T = a.T, N = a.N;
    const int LW = (L + 31) / 32, nlt = (L + 15) / 16;
    // a1: rows l = 16 lt + c, k = i = 16 j + 4 g + q;  a2: rows i = 16 I + c, k = l = 16 lt + 4 g + q
    float a1[NLW][NS], a2[NI][4 * NLW];
#pragma unroll
    for (int k = 0; k < NLW; ++k) {
        const int lt = wv * NLW + k, l = 16 * lt + c;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = 16 * (s / 4) + 4 * g + (s % 4);
            const bool e = lt < nlt && l < L && i < M;
            a1[k][s] = !e ? 0.f : REV ? a.W1[(size_t)i * L + l] : a.W2[(size_t)l * M + i] * p_of(i, N, a.alpha);
        }
    }
#pragma unroll
    for (int I = 0; I < NI; ++I)
#pragma unroll
        for (int k = 0; k < NLW; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int lt = wv * NLW + k, i = 16 * I + c, l = 16 * lt + 4 * g + q;
                const bool e = lt < nlt && i < M && l < L;
                a2[I][4 * k + q] =
                    !e ? 0.f : REV ? a.W2[(size_t)l * M + i] * p_of(i, N, a.alpha) : a.W1[(size_t)i * L + l];
            }
    const int nchains = a.B * ncs;
    const int id = (block * NG + grp) * 16 + c;
    const bool exists = id < nchains;
    const int b = exists ? id / ncs : 0, cc = exists ? id % ncs : 0;
    const bool ok = exists && (!active || active[b]);
    const int s0 = cc * C;
    const int len = ok ? max(min(s0 + C, T) - s0, 0) : 0;
    // steps of the block: the longest of its chains (the same value in every wave)
    int maxlen = len;
    if constexpr (NG > 1) {   // lane l: chain l % 32 of the block
        static_assert(NG == 2, "two groups of 16 chains");
        const int id2 = block * 32 + (lane & 31), b2 = id2 < nchains ? id2 / ncs : 0, s2 = id2 < nchains ? id2 % ncs * C : 0;
        maxlen = id2 < nchains && (!active || active[b2]) ? max(min(s2 + C, T) - s2, 0) : 0;
    }
#pragma unroll
    for (int off = 1; off < 16 * NG; off <<= 1) maxlen = max(maxlen, __shfl_xor(maxlen, off, 64));
    maxlen = __builtin_amdgcn_readfirstlane(maxlen);
    const float gm = gamma ? gamma[b] : 1.f;
    const float *zin = REV || LOCAL ? nullptr : cur_iter(zbuf, outbuf, zsel, b);
    float *zout = REV || LOCAL ? outbuf : next_iter(zbuf, outbuf, zsel, b);
    float dg[NI][4];
    v4f dl[NI];
#pragma unroll
    for (int I = 0; I < NI; ++I)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * g + r;
            dg[I][r] = i < M ? a.A[i] * p_of(i, N, a.alpha) : 0.f;
            dl[I][r] = (!LOCAL && ok && i < M) ? carry_in[(size_t)id * MP + i] : 0.f;
        }
    const size_t rowb = (size_t)b * T;
    // row of step t of this chain, and whether its Jacobian exists (reverse: J~_{k+1}, k + 1 < T)
    auto krow = [&](int t) { return REV ? s0 + len - 1 - t : s0 + t; };
    // per step: mask words of the wave's tiles; the right-hand side and (forward) the iterate
    // of the element r = w of every tile (wave w adds the diagonal and right-hand side of that
    // element and writes it), one step ahead
    uint32_t mn[NLW];
    float rn[NI], zn[NI];
    auto fetch = [&](int t) {
        const bool run = t < len;
        const int k = krow(t);
        const int mrow = REV ? k + 1 : k;
        const bool hasj = run && mrow < T;
#pragma unroll
        for (int kk = 0; kk < NLW; ++kk) {
            const int lt = wv * NLW + kk;
            mn[kk] = (hasj && lt < nlt) ? masks[(rowb + mrow) * LW + (lt >> 1)] : 0u;
        }
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            const int i = 16 * I + 4 * g + wv;
            const bool e = run && i < M;
            rn[I] = e ? rhs[(rowb + k) * M + i] : 0.f;
            zn[I] = (!REV && !LOCAL && e) ? zin[(rowb + k) * M + i] : 0.f;
        }
    };
    fetch(0);
    uint32_t emax = 0u, zmax = 0u;
    for (int t = 0; t < maxlen; ++t) {
        uint32_t mc[NLW];
        float rcur[NI], zcur[NI];
#pragma unroll
        for (int k = 0; k < NLW; ++k) mc[k] = mn[k];
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            rcur[I] = rn[I];
            zcur[I] = zn[I];
        }
        const int kcur = krow(t);
        // the Jacobian term of this step: always forward; reverse unless k + 1 = T
        const bool hasj = !REV || kcur + 1 < T;
        // latent warm-up step of this lane's chain (P_1 in J~_k, forward, or J~_{k+1}, reverse):
        // the observed latents' entries of y enter neither W2 diag(p) y nor the diagonal term
        // (forward), or the output's observed rows vanish (reverse)
        const bool wdrop = a.tw > 0 && (REV ? kcur + 1 : kcur) <= a.tw && t < len;
        if (!REV && a.tw > 0) {
#pragma unroll
            for (int I = 0; I < NI; ++I)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (wdrop && 16 * I + 4 * g + r < N) dl[I][r] = 0.f;
        }
        fetch(t + 1);
        v4f u[NLW];
#pragma unroll
        for (int k = 0; k < NLW; ++k) {
            v4f s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q4 = 0; q4 < NS; ++q4) s = mfma16x16x4(a1[k][q4], dl[q4 / 4][q4 % 4], s);
            const int sh = 16 * ((wv * NLW + k) & 1) + 4 * g;
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] = select_bit(mc[k], sh + r, s[r]);
            u[k] = s;
        }
        v4f p2[NI];
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            v4f s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < NLW; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) s = mfma16x16x4(a2[I][4 * k + q], u[k][q], s);
            p2[I] = s;
        }
        const int buf = t & 1;
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            v4f ct;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool own = r == wv;
                const bool jon = hasj && !(REV && wdrop && 16 * I + 4 * g + r < N);
                const float jv = jon ? gm * (own ? fmaf(dg[I][r], dl[I][r], p2[I][r]) : p2[I][r]) : 0.f;
                ct[r] = own ? fmaf(rhs_sign, rcur[I], jv) : jv;
            }
            red[buf][wv][I][lane] = ct;
        }
        lds_barrier();
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            v4f s = red[buf][0][I][lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const v4f o = red[buf][w][I][lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) s[r] = s[r] + o[r];
            }
            if (!LOCAL || t < len) dl[I] = s;   // local: past the chunk its last y stays
        }
        if (!LOCAL && t < len) {
#pragma unroll
            for (int I = 0; I < NI; ++I) {
                const int i = 16 * I + 4 * g + wv;
                if (i < M) {
                    const v4f d = dl[I];
                    const float y = wv == 0 ? d[0] : wv == 1 ? d[1] : wv == 2 ? d[2] : d[3];
                    if (REV) {
                        zout[(rowb + kcur) * M + i] = y;
                    } else {
                        const float zo = zcur[I];
                        zout[(rowb + kcur) * M + i] = zo + y;
                        const uint32_t ab = abs_bits(y), zb = abs_bits(zo);
                        emax = emax > ab ? emax : ab;
                        zmax = zmax > zb ? zmax : zb;
                    }
                }
            }
        }
    }
    if (LOCAL && ok) {
#pragma unroll
        for (int I = 0; I < NI; ++I) {
            const v4f d = dl[I];
            outbuf[(size_t)id * MP + 16 * I + 4 * g + wv] = wv == 0 ? d[0] : wv == 1 ? d[1] : wv == 2 ? d[2] : d[3];
        }
    }
    if (REV || LOCAL) return;
    // per-chain maxima: the lane groups, then the 4 waves (through the LDS of the last step,
    // whose reads are done once every wave has passed this barrier)
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)emax, off, 64);
        const uint32_t oz = (uint32_t)__shfl_xor((int)zmax, off, 64);
        emax = emax > o ? emax : o;
        zmax = zmax > oz ? zmax : oz;
    }
    if (g == 0) {
        mx[wv][c][0] = emax;
        mx[wv][c][1] = zmax;
    }
    lds_barrier();
    if (wv != 0) return;
    if (g == 0 && ok) {
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            emax = emax > mx[w][c][0] ? emax : mx[w][c][0];
            zmax = zmax > mx[w][c][1] ? zmax : mx[w][c][1];
        }
        if (!fc.seq) {   // reduced per sequence by the pass-end control
            chain_bits[id] = emax;
            chain_bits[(size_t)nchains + id] = zmax;
        }
    }
    if (!fc.seq) return;
    // fused pass-end control (chains of a sequence that is not running do not arrive)
    block16_arrive(fc, emax, zmax, ok, b, ncs, lane);
}

template <int MP, int NLW, bool REV>
__global__ __launch_bounds__(256) void k_fixup_shjvp(const ShArgs a, const uint32_t *__restrict__ masks,
                                                     const float *__restrict__ rhs, float rhs_sign,
                                                     const float *__restrict__ gamma,
                                                     const float *__restrict__ carry_in, float *zbuf, float *outbuf,
                                                     const int *__restrict__ zsel, uint32_t *__restrict__ chain_bits,
                                                     const int *__restrict__ active, int C, int ncs, FusedCtl fc) {
    __shared__ ShWalkLds<MP> sm;
    shjvp_walk<MP, NLW, 1, REV, false>(a, masks, rhs, rhs_sign, gamma, carry_in, zbuf, outbuf, zsel, chain_bits, active, C,
                                       ncs, fc, blockIdx.x, &sm);
}

// ---------------------------------------------------------------------------------------
// A chunk's aggregates: the first blocks walk the local solutions (16 chunks for every four waves), the
// others form the chunk products (a chunk a wave).  The two need nothing of each other, and on a short sequence
// neither fills the chip: M = 4, L = 50, 32768 steps take 24 us together (20 + 15 us one after the
// other).  M = 32, L = 256, 8 x 65536 steps: 1.02 ms a pass on average (with the products that are
// kept) against 1.94 ms in fp32.
// ---------------------------------------------------------------------------------------
template <int MP, int NT, int NLW, bool REV, bool WU>
__global__ __launch_bounds__(256 * shf_groups(MP, NLW)) __attribute__((amdgpu_waves_per_eu(2))) void k_chunk_aggregates_sh(
    const ShArgs a, const uint32_t *__restrict__ masks, const uint32_t *__restrict__ masks_prev,
    const float *__restrict__ rhs, float rhs_sign, const float *__restrict__ gamma, float *__restrict__ pgam,
    float *__restrict__ Pout, float *__restrict__ vout, const int *__restrict__ active, int C, int ncs, int LB,
    int nwalk) {
    extern __shared__ __align__(16) v4u smem4[];
    constexpr int NG = shf_groups(MP, NLW);
    if ((int)blockIdx.x < nwalk)
        shjvp_walk<MP, NLW, NG, REV, true>(a, masks, rhs, rhs_sign, gamma, nullptr, nullptr, vout, nullptr, nullptr, active,
                                           C, ncs, FusedCtl{}, blockIdx.x, reinterpret_cast<ShWalkLds<MP> *>(smem4));
    else
        sh_chunk_product<MP, NT, 4 * NG, REV, WU>(a, masks, masks_prev, gamma, pgam, Pout, active, C, ncs, LB,
                                                  blockIdx.x - nwalk, smem4);
}

// ---------------------------------------------------------------------------------------
// residual and hidden masks of a Newton pass on the matrix cores.  A wave owns a tile of 16
// rows (b, s), the 16 columns of its products; W2 (row l, column i), W1 (row i, column l) and
// h2 sit in LDS and serve as A operands.  Per 16-unit hidden tile lt:
//   u   = W2[tile lt, :] z~ + h2     B = z~ of the rows (lane (g, c): z~[row c][16j + 4g + q])
//   m   = u > 0 (the 4 lane groups' bits ORed into the row's mask word), v = relu(u)
//   F  += W1[:, tile lt] v           B = v in its accumulator layout
// and F = A z~ + F + h1, r = z - F.  No barrier inside the loop over tiles.  The sums round as
// the matrix cores do, so a decision with u within rounding of 0 may differ from the
// fixed-order float32 one of k_resjac_shplrnn; these masks serve only the Newton passes (the
// masks a caller receives and the adjoint's come from k_resjac_shplrnn).
// ---------------------------------------------------------------------------------------
static int shf_LQ(int L) { return shf_LP(L) + 4; }

size_t shf_resjac_lds(int M, int L) {
    const int MP = padded_dim(M), LP = shf_LP(L);
    return ((size_t)LP * (MP + 4) + (size_t)MP * shf_LQ(L) + LP) * sizeof(float);
}

template <int MP>
__global__ __launch_bounds__(256) void k_resjac_shmfma(const ShArgs a, const float *zbuf, const float *zalt,
                                                       const int *__restrict__ zsel, float *__restrict__ r_out,
                                                       uint32_t *__restrict__ masks, const int *__restrict__ active,
                                                       int LP, uint32_t *mark, uint32_t pass_no) {
    constexpr int NI = MP / 16, MQ = MP + 4;
    extern __shared__ __align__(16) float smem[];
    // the pass's first kernel: block 0 marks its start (every earlier pass is complete)
    if (mark && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(mark, pass_no, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int M = a.M, L = a.L, T = a.T, N = a.N, LQ = LP + 4;
    float *w2s = smem;             // [LP][MQ]
    float *w1s = w2s + LP * MQ;    // [MP][LQ]
    float *h2s = w1s + MP * LQ;    // [LP]
    const int tid = threadIdx.x;
    for (int e = tid; e < LP * MQ; e += 256) {
        const int l = e / MQ, i = e % MQ;
        w2s[e] = (l < L && i < M) ? a.W2[(size_t)l * M + i] : 0.f;
    }
    for (int e = tid; e < MP * LQ; e += 256) {
        const int i = e / LQ, l = e % LQ;
        w1s[e] = (i < M && l < L) ? a.W1[(size_t)i * L + l] : 0.f;
    }
    for (int e = tid; e < LP; e += 256) h2s[e] = (e < L && a.h2) ? a.h2[e] : 0.f;
    __syncthreads();
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int LW = (L + 31) / 32, nlt = LP / 16;
    const float p = __fsub_rn(1.0f, a.alpha);
    float dA[NI][4], h1v[NI][4];
#pragma unroll
    for (int I = 0; I < NI; ++I)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * g + r;
            dA[I][r] = i < M ? a.A[i] : 0.f;
            h1v[I][r] = (i < M && a.h1) ? a.h1[i] : 0.f;
        }
    const long total = (long)a.B * T;
    const long ntiles = (total + 15) / 16;
    const long nw = (long)gridDim.x * 4;
    // The inputs of a tile for row c, latents i = 16j + 4g + q: z_{s-1} (or the initial state at
    // s = 0) and x_s, combined into z~ as k_resjac_shplrnn does, and z_s.  Every lane loads from a
    // valid address (rows past the end, inactive sequences and latents past M read row 0 /
    // latent 0 and are zeroed after), so the loads carry no branches and the next tile's, issued
    // at the top of a tile, are waited for only when the tile ends.
    struct RowIn {   // (sequence, step) of row c of a tile and the sequence's control words
        int b, s, sel, act;
        bool inr;
    };
    struct TileIn {
        float zp[NI][4], xs[NI][4], zc[NI][4];
        int s;
        bool ok;
    };
    // stage 1, two tiles ahead: the row's position and its control words (loads in flight)
    auto rowin = [&](long tile, RowIn &ri) {
        const long rowc = tile * 16 + c;
        ri.b = 0;
        ri.s = 0;
        ri.inr = tile < ntiles && rowc < total;
        if (ri.inr) row_at(row_base(tile * 16, T), c, T, ri.b, ri.s);
        ri.sel = zsel ? zsel[ri.b] : 0;
        ri.act = active ? active[ri.b] : 1;
    };
    // stage 2, one tile ahead: the inputs, at addresses from the control words loaded a tile ago
    auto fetch = [&](const RowIn &ri, TileIn &in) {
        const int b = ri.b, s = ri.s;
        in.ok = ri.inr && ri.act != 0;
        in.s = s;
        const float *z = ri.sel ? zalt : zbuf;
        const size_t rp = (size_t)b * T + (s > 0 ? s - 1 : 0), rc = (size_t)b * T + s;
        const size_t xr = ((size_t)b * (T + 1) + s) * (size_t)(N > 0 ? N : 1);
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 16 * j + 4 * g + q, ic = i < M ? i : 0;
                const float zpv = z[rp * M + ic];
                const float z0v = a.z0 ? a.z0[(size_t)b * M + ic] : 0.f;
                in.zp[j][q] = s > 0 ? zpv : z0v;
                in.xs[j][q] = N > 0 ? a.x[xr + (i < N ? i : 0)] : 0.f;
                in.zc[j][q] = z[rc * M + ic];
            }
    };
    const long t0w = (long)blockIdx.x * 4 + wv;
    RowIn r1, r2;
    TileIn cur, nxt;
    rowin(t0w, r1);
    fetch(r1, cur);
    rowin(t0w + nw, r1);
    for (long tile = t0w; tile < ntiles; tile += nw) {
        rowin(tile + 2 * nw, r2);
        fetch(r1, nxt);
        const long rowc = tile * 16 + c;
        const bool rok = cur.ok;
        const int s = cur.s;
        float zt[NI][4], zc[NI][4];
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 16 * j + 4 * g + q;
                float v;
                if (s == 0)   // the initial state: z0, or [x_0; 0]
                    v = a.z0 ? cur.zp[j][q] : (i < N ? cur.xs[j][q] : 0.f);
                else if (i < N && s <= a.tw)   // latent warm-up: alpha_s = 1
                    v = cur.xs[j][q];
                else
                    v = i < N ? __fadd_rn(__fmul_rn(p, cur.zp[j][q]), __fmul_rn(a.alpha, cur.xs[j][q])) : cur.zp[j][q];
                const bool e = rok && i < M;
                zt[j][q] = e ? v : 0.f;
                zc[j][q] = e ? cur.zc[j][q] : 0.f;
            }
        // a tile whose sequences have all stopped (a pass queued past their convergence) does no
        // work (the branch is wave-uniform)
        if (__builtin_amdgcn_ballot_w64(rok) != 0ull) {
            v4f F[NI];
    #pragma unroll
            for (int I = 0; I < NI; ++I) F[I] = (v4f){0.f, 0.f, 0.f, 0.f};
            for (int w = 0; w < LW; ++w) {
                uint32_t word = 0u;
    #pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int lt = 2 * w + h;
                    if (lt >= nlt) break;
                    const float4 hq = *reinterpret_cast<const float4 *>(h2s + 16 * lt + 4 * g);
                    v4f u = {hq.x, hq.y, hq.z, hq.w};
    #pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        const float4 aq = *reinterpret_cast<const float4 *>(w2s + (16 * lt + c) * MQ + 16 * j + 4 * g);
                        u = mfma16x16x4(aq.x, zt[j][0], u);
                        u = mfma16x16x4(aq.y, zt[j][1], u);
                        u = mfma16x16x4(aq.z, zt[j][2], u);
                        u = mfma16x16x4(aq.w, zt[j][3], u);
                    }
    #pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool on = u[r] > 0.f;
                        word |= (on ? 1u : 0u) << (16 * h + 4 * g + r);
                        u[r] = on ? u[r] : 0.f;
                    }
    #pragma unroll
                    for (int I = 0; I < NI; ++I) {
                        const float4 aq = *reinterpret_cast<const float4 *>(w1s + (16 * I + c) * LQ + 16 * lt + 4 * g);
                        F[I] = mfma16x16x4(aq.x, u[0], F[I]);
                        F[I] = mfma16x16x4(aq.y, u[1], F[I]);
                        F[I] = mfma16x16x4(aq.z, u[2], F[I]);
                        F[I] = mfma16x16x4(aq.w, u[3], F[I]);
                    }
                }
                word |= (uint32_t)__shfl_xor((int)word, 16, 64);
                word |= (uint32_t)__shfl_xor((int)word, 32, 64);
                if (g == 0 && rok) masks[(size_t)rowc * LW + w] = word;
            }
            if (rok) {
    #pragma unroll
                for (int I = 0; I < NI; ++I)
    #pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * I + 4 * g + r;
                        if (i < M) r_out[(size_t)rowc * M + i] = zc[I][r] - (fmaf(dA[I][r], zt[I][r], F[I][r]) + h1v[I][r]);
                    }
            }
        }
        cur = nxt;
        r1 = r2;
    }
}

int launch_resjac_shmfma(const ShArgs &a, const float *z, const float *zalt, const int *zsel, float *r,
                         uint32_t *masks, const int *active, hipStream_t st, uint32_t *mark, uint32_t pass_no) {
    const int MP = padded_dim(a.M);
    if (!shfused_supported(a.M, a.L) || a.zt) return DEER_ERR_INVALID_ARG;
    const size_t lds = shf_resjac_lds(a.M, a.L);
    if (lds > 80 * 1024) return DEER_ERR_INVALID_ARG;
    const long ntiles = ((long)a.B * a.T + 15) / 16;
    // two resident blocks per CU (LDS), each wave walking its share of the tiles
    const long want = (ntiles + 3) / 4;
    const int grid = (int)(want < 512 ? want : 512);
    const int LP = shf_LP(a.L);
    KTimer kt("k_resjac_shmfma", st);
#define RJM(MPV) \
    hipLaunchKernelGGL((k_resjac_shmfma<MPV>), dim3(grid), dim3(256), lds, st, a, z, zalt, zsel, r, masks, active, LP, \
                       mark, pass_no)
    if (MP == 16) RJM(16); else if (MP == 32) RJM(32); else RJM(64);
#undef RJM
    DEER_LAUNCH_CHECK("k_resjac_shmfma");
    return DEER_OK;
}

int launch_chunk_aggregates_sh(bool rev, const ShArgs &a, const uint32_t *masks, const uint32_t *masks_prev,
                               const float *rhs, float rhs_sign, const float *gamma, float *pgam, float *P, float *v,
                               const int *active, int C, int ncs, hipStream_t st) {
    const int MP = padded_dim(a.M);
    if (!shfused_supported(a.M, a.L) || (rev && (gamma || active))) return DEER_ERR_INVALID_ARG;
    const int LB = (a.L + 31) / 32, nlw = shf_nlw(a.L), ng = shf_groups(MP, nlw);
    const int nwalk = (a.B * ncs + 16 * ng - 1) / (16 * ng), grid = nwalk + (a.B * ncs + 4 * ng - 1) / (4 * ng);
    const size_t lds = shfused_product_lds(a.M, a.L);
    KTimer kt(rev ? "k_chunk_aggregates_sh_rev" : "k_chunk_aggregates_sh", st);
#define CPS(MPV, NTV, NL, RV, WUV)                                                                                   \
    hipLaunchKernelGGL((k_chunk_aggregates_sh<MPV, NTV, NL, RV, WUV>), dim3(grid), dim3(256 * ng), lds, st, a, masks,   \
                       masks_prev, rhs, rhs_sign, gamma, pgam, P, v, active, C, ncs, LB, nwalk)
#define CPW(MPV, NTV, NL, RV) { if (a.tw > 0) CPS(MPV, NTV, NL, RV, true); else CPS(MPV, NTV, NL, RV, false); }
#define CPR(MPV, NTV, NL) { if (rev) CPW(MPV, NTV, NL, true) else CPW(MPV, NTV, NL, false) }
    // shfused_supported bounds NLW * MP / 2 (the walk's A fragments per lane) by 64
    if (MP == 16) {
        if (nlw == 1) CPR(16, 8, 1) else if (nlw == 2) CPR(16, 8, 2) else if (nlw == 4) CPR(16, 8, 4) else CPR(16, 8, 8)
    } else if (MP == 32) {
        if (nlw == 1) CPR(32, 4, 1) else if (nlw == 2) CPR(32, 4, 2) else CPR(32, 4, 4)
    } else {
        if (nlw == 1) CPR(64, 1, 1) else CPR(64, 1, 2)
    }
#undef CPR
#undef CPW
#undef CPS
    DEER_LAUNCH_CHECK("k_chunk_aggregates_sh");
    return DEER_OK;
}

int launch_fixup_shjvp(bool rev, const ShArgs &a, const uint32_t *masks, const float *rhs, float rhs_sign,
                       const float *gamma, const float *carry_in, float *z, float *out, const int *zsel,
                       uint32_t *chain_bits, const int *active, int C, int ncs, hipStream_t st, const FusedCtl *fc) {
    const int MP = padded_dim(a.M);
    if (!shfused_supported(a.M, a.L) || (fc && (rev || !active))) return DEER_ERR_INVALID_ARG;
    const FusedCtl fcv = fc ? *fc : FusedCtl{};
    const int nch = a.B * ncs;
    const int grid = (nch + 15) / 16;
    const int nlw = shf_nlw(a.L);
    KTimer kt(rev ? "k_fixup_shjvp_rev" : "k_fixup_shjvp", st);
#define FXL(MPV, NL, RV)                                                                                             \
    hipLaunchKernelGGL((k_fixup_shjvp<MPV, NL, RV>), dim3(grid), dim3(256), 0, st, a, masks, rhs, rhs_sign, gamma,     \
                       carry_in, z, out, zsel, chain_bits, active, C, ncs, fcv)
#define FXJ(MPV, NL) { if (rev) FXL(MPV, NL, true); else FXL(MPV, NL, false); }
    if (MP == 16) {
        if (nlw == 1) FXJ(16, 1) else if (nlw == 2) FXJ(16, 2) else if (nlw == 4) FXJ(16, 4) else FXJ(16, 8)
    } else if (MP == 32) {
        if (nlw == 1) FXJ(32, 1) else if (nlw == 2) FXJ(32, 2) else FXJ(32, 4)
    } else {
        if (nlw == 1) FXJ(64, 1) else FXJ(64, 2)
    }
#undef FXJ
#undef FXL
    DEER_LAUNCH_CHECK("k_fixup_shjvp");
    return DEER_OK;
}

}  // namespace deer
