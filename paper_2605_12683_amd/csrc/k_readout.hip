// Read-out MLP of the diagonal SSM and its mean-squared loss (the LSSM's observation model;
// linear-SSM appendix), forward and backward in one pass over the states:
//   s_t = Wa Re(h_t) + ca            (H hidden units)
//   y_t = Wb relu(s_t) + cb          (No outputs)
//   L   = sum_{b,t} ||y_t - x_{t+1}||^2 / (B No T)        (0-based rows: target row t + 1)
//   dy_t = 2 (y_t - x_{t+1}) / (B No T),  ds_t = (Wb^T dy_t) * 1[s_t > 0]
//   g_t = dL/dRe h_t = Wa^T ds_t     (the cotangent of the reverse scan)
//   dWa = sum ds_t Re(h_t)^T, dca = sum ds_t, dWb = sum dy_t relu(s_t)^T, dcb = sum dy_t
//
// The three products with Wa are dense [16 rows x 64] x [64 x 128] contractions on the fp16 matrix
// cores with split operands (split16.h).  A wave takes 16 consecutive (b, t) rows at a time, row c
// of the tile in the lanes (., c):
//   GEMM1  S^T = Wa H^T     B = Re h straight from the loads (slot 2 i + p of k block kk is channel
//                           32 kk + 8 i + 2 g + p, so a load instruction takes 64 bytes of every row)
//   GEMM2  G^T = Wa^T dS^T  B = dS^T in the layout it is formed in (no data movement); a lane ends
//                           with four consecutive channels of its row
//   GEMM3  dWa^T += H^T dS^T, shared by the eight waves of a block: after every round (each wave one
//                           tile) wave w accumulates hidden units 16 w .. 16 w + 15 over the 128
//                           rows, which go through LDS 64 at a time as half-words, rows packed in
//                           pairs by a lane exchange
// dS^T = Wb^T dy is one fp32 16x16x4 instruction per 16 hidden units (four outputs).
// Scales, all powers of two: Wa and Wb once; every row's h and dy by their own largest entry (a
// column of the B operands, so rows do not meet); for GEMM3, whose k index is the row, the split
// halves are brought to the round's largest row (exact but for bits below 2^-38 of it) and the
// round's sums are added in fp32.  In GEMM1 Wa has a third part and is exact: its split error would
// be the same in every row and add up in dWb and dcb.
// A row of h or a Wa with infinities or NaN has no split: such preactivations are formed in plain
// fp32 (an infinite state still makes the loss infinite or NaN), and such rows do not set a round's
// scale.
// Bound by the issue of vector instructions (splits, ReLU and masks, packing for GEMM3) in turn with
// the matrix cores, at the two waves per SIMD that 153 KB of LDS and 256 VGPRs leave.
// N = 64, H = 128, 2^22 rows: 1.44 ms; with fp32 matrix instructions (222 ns of a SIMD for the 16
// that 6 of these at 127 ns / 16 replace) 2.34 ms.
#include "common.h"
#include "launch.h"
#include "split16.h"

namespace deer {

namespace {
constexpr int RH = 128;          // hidden units (padded)
constexpr int RM = 64;           // state channels (padded)
constexpr int RNO = 4;           // outputs (padded)
constexpr int RW = 8;            // waves per block (one per 16 hidden units in GEMM3)
constexpr int BS = 17;           // LDS row stride of the [hidden][row] tile of dWb
constexpr int RPS = RH * RM + RNO * RH + RH + RNO + 1;   // partial floats per wave
constexpr int RPS_PAD = (RPS + 63) & ~63;

// lane c of a pair of rows (c, c ^ 1): the partner's register, and the half-words of one column packed
// in row order (even lanes the first half-word's column, odd lanes the second's)
__device__ __forceinline__ uint32_t pair_sel(bool odd) { return odd ? 0x03020706u : 0x05040100u; }
__device__ __forceinline__ uint32_t pair_rows(uint32_t own, uint32_t sel) {
    const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
    return __builtin_amdgcn_perm(other, own, sel);
}
// both half-words times a power of two
__device__ __forceinline__ uint32_t scale_halves(uint32_t v, v2h f) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2h, v) * f);
}
}  // namespace

template <bool GRADS>
__global__ __launch_bounds__(RW * 64) void k_readout(const RoArgs ra, const float *__restrict__ h,
                                                     const float *__restrict__ x, int B, int T, float scale,
                                                     float *__restrict__ gout, uint32_t *__restrict__ masks,
                                                     float *__restrict__ part) {
    __shared__ __align__(16) v4u w1[8][2][3][64];    // Wa: [hidden tile][k block][hi, lo, rest][lane]
    __shared__ __align__(16) v4u w2[4][4][2][64];    // Wa^T: [channel tile][k block][hi, lo][lane]
    __shared__ __align__(16) v4u h3[GRADS ? 2 : 1][4][2][64];   // GEMM3, 64 rows: [k block][channel tile][hi, lo][lane]
    __shared__ __align__(16) v4u d3[GRADS ? 2 : 1][8][2][64];   //                 [k block][hidden tile][hi, lo][lane]
    __shared__ __align__(16) float4 wb4[RH];         // Wb of a hidden unit, the four outputs
    __shared__ __align__(16) float cas[RH];
    __shared__ __align__(16) float buf[GRADS ? RW : 1][32][BS];
    __shared__ __align__(16) float4 dyv[GRADS ? RW : 1][16];
    __shared__ float lsw[RW], mxs[RW][2];
    __shared__ int rsc[2][RW][2];                    // round parity, wave: smallest shifts of its rows
    const int M = ra.M, H = ra.H, No = ra.No;
    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, g = lane >> 4, c = lane & 15;
    const float m1 = opaque_m1();
    {
        float xa = 0.f, xb = 0.f;
        int nf = 0;
        for (int e = tid; e < H * M; e += RW * 64) {
            const float v = fabsf(ra.Wa[e]);
            const bool fin = v < __builtin_inff();
            nf |= fin ? 0 : 1;
            xa = fmaxf(xa, fin ? v : 0.f);
        }
        for (int e = tid; e < RH; e += RW * 64) {
            float w[RNO];
            float n = 0.f;
#pragma unroll
            for (int o = 0; o < RNO; ++o) {
                w[o] = (o < No && e < H) ? ra.Wb[o * H + e] : 0.f;
                n += fabsf(w[o]);
            }
            wb4[e] = make_float4(w[0], w[1], w[2], w[3]);
            xb = fmaxf(xb, n);
            cas[e] = (e < H && ra.ca) ? ra.ca[e] : 0.f;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            xa = fmaxf(xa, __shfl_xor(xa, off, 64));
            xb = fmaxf(xb, __shfl_xor(xb, off, 64));
        }
        if (lane == 0) {
            mxs[wv][0] = xa;
            mxs[wv][1] = xb;
            rsc[0][wv][0] = 0;
        }
        if (nf) rsc[0][wv][0] = 1;
    }
    __syncthreads();
    float xa = 0.f, xb = 0.f;
    int nfw = 0;   // Wa holds infinities or NaN
#pragma unroll
    for (int w = 0; w < RW; ++w) {
        nfw |= rsc[0][w][0];
        xa = fmaxf(xa, mxs[w][0]);
        xb = fmaxf(xb, mxs[w][1]);
    }
    nfw = __builtin_amdgcn_readfirstlane(nfw);
    const int sa = min(9 - exp_of(xa), 100), sw = min(12 - exp_of(xb), 100);
    {
        // wave w: hidden tile w of Wa, and two of the 16 (channel tile, k block) pairs of Wa^T
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            v4u hi, lo, rest;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float w[2], v[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int hid = 16 * wv + c, ch = 32 * kk + 8 * i + 2 * g + p;
                    w[p] = (hid < H && ch < M) ? ldexpf(ra.Wa[hid * M + ch], sa) : 0.f;
                }
                uint32_t a, b;
                split_pair(w[0], w[1], m1, a, b);
                hi[i] = a;
                lo[i] = b;
                const v2h ah = __builtin_bit_cast(v2h, a), bh2 = __builtin_bit_cast(v2h, b);
#pragma unroll
                for (int p = 0; p < 2; ++p) v[p] = (w[p] - (float)ah[p]) - (float)bh2[p];   // exact
                rest[i] = __builtin_bit_cast(uint32_t, v2h{(_Float16)v[0], (_Float16)v[1]});
            }
            w1[wv][kk][0][lane] = hi;
            w1[wv][kk][1][lane] = lo;
            w1[wv][kk][2][lane] = rest;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = wv >> 1, kk = 2 * (wv & 1) + u;
            v4u hi, lo;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float w[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int e = 2 * i + p, ch = 16 * q + c, hid = 16 * (2 * kk + (e >> 2)) + 4 * g + (e & 3);
                    w[p] = (hid < H && ch < M) ? ldexpf(ra.Wa[hid * M + ch], sa) : 0.f;
                }
                uint32_t a, b;
                split_pair(w[0], w[1], m1, a, b);
                hi[i] = a;
                lo[i] = b;
            }
            w2[q][kk][0][lane] = hi;
            w2[q][kk][1][lane] = lo;
        }
    }
    float wbA[8];   // A operand of dS^T: Wb[o = g][16 n + c], scaled
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int hid = 16 * n + c;
        wbA[n] = (g < No && hid < H) ? ldexpf(ra.Wb[g * H + hid], sw) : 0.f;
    }
    float cb[RNO];
#pragma unroll
    for (int o = 0; o < RNO; ++o) cb[o] = (o < No && ra.cb) ? ra.cb[o] : 0.f;
    __syncthreads();

    const long rows = (long)B * T;
    const long ntiles = (rows + 15) / 16;
    const int HW = (H + 31) / 32;
    const bool odd = (c & 1) != 0;
    const uint32_t psel = pair_sel(odd);
    const uint32_t one2 = __builtin_bit_cast(uint32_t, v2h{(_Float16)1.f, (_Float16)1.f});
    const v4u ones = c == 0 ? (v4u){one2, one2, one2, one2} : (v4u){0u, 0u, 0u, 0u};   // A operand: row 0 all ones

    v4f acc3[4];                    // dWa^T tiles [channel tile q] of hidden tile n = wv
    float dwb[4][RNO], dca = 0.f, dcb[RNO], lsum = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc3[q] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < RNO; ++o) {
        dcb[o] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dwb[k][o] = 0.f;
    }

    // Re h of a tile, loaded one tile ahead: lane (g, c) the channels 32 kk + 8 i + 2 g (+ 1) of row c,
    // through a buffer resource that ends at the last row (rows past the end and channels past M load 0
    // without branches; the whole offset is in the VGPR, so the range check covers it).  Even M: one
    // 16-byte load takes both channels.
    const bool even = (M & 1) == 0;
    float hv[2][4][2];
    auto load_tile = [&](long tl) {
        const long rb = tl < ntiles ? tl * 16 : rows;
        const long left = rows - rb;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(h + rb * M * 2), (short)0,
                                                          (int)(left < 16 ? left * M * 8 : 16L * M * 8), 0x00020000);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ch = 32 * kk + 8 * i + 2 * g;
                const int vo = ch < M ? (c * M + ch) * 8 : (int)0x80000000;
                if (even) {
                    const float4 v = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, 0, 0));
                    hv[kk][i][0] = v.x;
                    hv[kk][i][1] = v.z;
                } else {
                    const int vo1 = ch + 1 < M ? (c * M + ch + 1) * 8 : (int)0x80000000;
                    hv[kk][i][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, vo, 0, 0));
                    hv[kk][i][1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, vo1, 0, 0));
                }
            }
    };
    // rounds are block-uniform (GEMM3 needs every wave at its barriers); a wave whose tile
    // lies past the end works on zero rows, which contribute nothing
    load_tile((long)blockIdx.x * RW + wv);
    int par = 0;
    for (long base = (long)blockIdx.x * RW; base < ntiles; base += (long)gridDim.x * RW, par ^= 1) {
        const long tile = base + wv;
        const long r0 = tile * 16;
        // the row's scale and its split states
        uint32_t mx = 0u;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = max(max(mx, abs_bits(hv[kk][i][0])), abs_bits(hv[kk][i][1]));
        {
            auto p = __builtin_amdgcn_permlane32_swap(mx, mx, false, false);
            mx = max(p[0], p[1]);
            auto q = __builtin_amdgcn_permlane16_swap(mx, mx, false, false);
            mx = max(q[0], q[1]);
        }
        const int ph = min(13 - exp_of(__uint_as_float(mx)), 126);   // below -114: the row is not finite
        const float fh = pow2i(ph);
        v4u bh[2], bl[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t a, b;
                split_pair(hv[kk][i][0] * fh, hv[kk][i][1] * fh, m1, a, b);
                bh[kk][i] = a;
                bl[kk][i] = b;
            }
        load_tile(tile + (long)gridDim.x * RW);

        // GEMM1: acc1[n][r] at lane (g, c) = S^T[hidden 16n + 4g + r][row c]
        v4f acc1[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) acc1[n] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
            for (int n0 = 0; n0 < 8; n0 += 4) {
                v4u ah[4], al[4], ar[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    ah[n] = w1[n0 + n][kk][0][lane];
                    al[n] = w1[n0 + n][kk][1][lane];
                    ar[n] = w1[n0 + n][kk][2][lane];
                }
#pragma unroll
                for (int n = 0; n < 4; ++n) acc1[n0 + n] = mfma_h(ar[n], bh[kk], acc1[n0 + n]);
#pragma unroll
                for (int n = 0; n < 4; ++n) acc1[n0 + n] = mfma_h(al[n], bh[kk], acc1[n0 + n]);
#pragma unroll
                for (int n = 0; n < 4; ++n) acc1[n0 + n] = mfma_h(ah[n], bl[kk], acc1[n0 + n]);
#pragma unroll
                for (int n = 0; n < 4; ++n) acc1[n0 + n] = mfma_h(ah[n], bh[kk], acc1[n0 + n]);
            }
        }
        // bias, ReLU, mask bits (bit 4n + r of the lane's hidden units), outputs y (partial over the
        // lane's 32 hidden units, then over the 4 lane groups)
        const float fs = ldexpf(1.f, -(ph + sa));
        uint32_t mb = 0u;
        float yp[RNO] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const float4 cq = *reinterpret_cast<const float4 *>(&cas[16 * n + 4 * g]);
            const float cv[4] = {cq.x, cq.y, cq.z, cq.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float s = fmaf(acc1[n][r], fs, cv[r]);
                const bool pos = s > 0.f;
                const float rl = pos ? s : 0.f;
                acc1[n][r] = rl;
                mb |= (pos ? 1u : 0u) << (4 * n + r);
                const float4 w = wb4[16 * n + 4 * g + r];
                yp[0] = fmaf(w.x, rl, yp[0]);
                yp[1] = fmaf(w.y, rl, yp[1]);
                yp[2] = fmaf(w.z, rl, yp[2]);
                yp[3] = fmaf(w.w, rl, yp[3]);
            }
        }
#pragma unroll
        for (int o = 0; o < RNO; ++o) yp[o] = group_sum(yp[o]);
        const long row = r0 + c;
        const bool rok = row < rows;
        const bool plain = nfw || ph < -114;
        if (__any(plain)) {
            // preactivations of rows that have no split, again
            const float *hq = h + (rok ? row : rows - 1) * M * 2;
            if (plain) mb = 0u;
            float yq[RNO] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k = 0; k < 32; ++k) {
                const int hid = 16 * (k >> 2) + 4 * g + (k & 3);
                float v = 0.f;
                if (plain && hid < H) {
#pragma unroll 1
                    for (int ch = 0; ch < M; ++ch) v = fmaf(ra.Wa[hid * M + ch], hq[2 * ch], v);
                }
                v += cas[hid];
                const bool pos = v > 0.f;
                v = pos ? v : 0.f;
                if (plain) mb |= (pos ? 1u : 0u) << k;
                const float4 w = wb4[hid];
                yq[0] = fmaf(w.x, v, yq[0]);
                yq[1] = fmaf(w.y, v, yq[1]);
                yq[2] = fmaf(w.z, v, yq[2]);
                yq[3] = fmaf(w.w, v, yq[3]);
#pragma unroll
                for (int n = 0; n < 8; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (plain && 4 * n + r == k) acc1[n][r] = v;
            }
#pragma unroll
            for (int o = 0; o < RNO; ++o) {
                const float v = group_sum(yq[o]);
                if (plain) yp[o] = v;
            }
        }
        if (masks) {
            // word w holds hidden units 32w .. 32w + 31, i.e. tiles n = 2w, 2w + 1
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t word = (((mb >> (8 * w)) & 15u) << (4 * g)) | (((mb >> (8 * w + 4)) & 15u) << (16 + 4 * g));
                word |= (uint32_t)__shfl_xor((int)word, 16, 64);
                word |= (uint32_t)__shfl_xor((int)word, 32, 64);
                if (g == w && w < HW && rok) masks[row * HW + w] = word;
            }
        }
        float err[RNO];
        {
            // target row t + 1 of sequence b for row = b T + t: x row index row + b + 1, with
            // b from the tile's first row (one scalar division) and the sequence boundaries
            // inside the tile (rows past the end read row 1 of a valid sequence, unused)
            const uint32_t Tu = (uint32_t)T;
            const uint32_t b0 = __builtin_amdgcn_readfirstlane((uint32_t)(r0 < rows ? r0 : 0) / Tu);
            const uint32_t rowu = rok ? (uint32_t)row : b0 * Tu;
            uint32_t bq = b0;
            for (int k = 0; k < 16 && rowu >= (bq + 1) * Tu; ++k) ++bq;
            const float *xt = x + ((size_t)rowu + bq + 1) * No;
#pragma unroll
            for (int o = 0; o < RNO; ++o) {
                const bool ok = rok && o < No;
                err[o] = ok ? (yp[o] + cb[o]) - xt[o] : 0.f;
                if (g == 0) lsum = fmaf(err[o], err[o], lsum);
            }
        }
        if constexpr (GRADS) {
            // dWb, dcb: relu(s) of 32 hidden units at a time through LDS, lane l then owns hidden unit
            // l % 32 and half of the rows
            if (g == 0) {
                dyv[wv][c] = make_float4(scale * err[0], scale * err[1], scale * err[2], scale * err[3]);
#pragma unroll
                for (int o = 0; o < RNO; ++o) dcb[o] += scale * err[o];
            }
            wave_lds_sync();
            float4 dr[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) dr[k] = dyv[wv][8 * (lane >> 5) + k];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) buf[wv][16 * n + 4 * g + r][c] = acc1[2 * p + n][r];
                wave_lds_sync();
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float a = buf[wv][lane & 31][8 * (lane >> 5) + k];
                    dwb[p][0] = fmaf(dr[k].x, a, dwb[p][0]);
                    dwb[p][1] = fmaf(dr[k].y, a, dwb[p][1]);
                    dwb[p][2] = fmaf(dr[k].z, a, dwb[p][2]);
                    dwb[p][3] = fmaf(dr[k].w, a, dwb[p][3]);
                }
                wave_lds_sync();
            }
        }
        // dS^T = (Wb^T err) * mask in the GEMM1 accumulator layout, scaled by 2^(sd + sw): below 2^14
        const uint32_t em = max(max(abs_bits(err[0]), abs_bits(err[1])), max(abs_bits(err[2]), abs_bits(err[3])));
        const int sd = em >= 0x7f800000u ? -127 : max(min(-exp_of(__uint_as_float(em)), 126), -126);   // -127: not finite
        const float eg = (g == 0 ? err[0] : g == 1 ? err[1] : g == 2 ? err[2] : err[3]) * pow2i(max(sd, -126));
        v4u dh[4], dl[4];   // B operand of GEMM2: k block kk holds hidden tiles 2 kk, 2 kk + 1
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const v4f d = mfma16x16x4(wbA[n], eg, (v4f){0.f, 0.f, 0.f, 0.f});
            float dm[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) dm[r] = select_bit(mb, 4 * n + r, d[r]);
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                uint32_t a, b;
                split_pair(dm[2 * h2], dm[2 * h2 + 1], m1, a, b);
                dh[n >> 1][2 * (n & 1) + h2] = a;
                dl[n >> 1][2 * (n & 1) + h2] = b;
            }
        }
        // GEMM2: acc2[q][r] at lane (g, c) = G[row c][channel 16q + 4g + r]
        v4f acc2[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc2[q] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            v4u ah[4], al[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ah[q] = w2[q][kk][0][lane];
                al[q] = w2[q][kk][1][lane];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) acc2[q] = mfma_h(al[q], dh[kk], acc2[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc2[q] = mfma_h(ah[q], dl[kk], acc2[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc2[q] = mfma_h(ah[q], dh[kk], acc2[q]);
        }
        {
            // stores through a resource that ends at the last row (later rows dropped), channels past M
            // outside it
            const long left = rows - r0 < 0 ? 0 : (rows - r0 < 16 ? rows - r0 : 16);
            const auto rs = __builtin_amdgcn_make_buffer_rsrc(gout + (r0 < rows ? r0 : 0) * M, (short)0,
                                                              (int)(left * M * 4), 0x00020000);
            const float fg = ldexpf(1.f, -(sd + sw + sa));   // apart from scale: their product may be subnormal
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = 16 * q + 4 * g;
                if ((M & 3) == 0) {
                    const v4u v = {__float_as_uint(acc2[q][0] * fg * scale), __float_as_uint(acc2[q][1] * fg * scale),
                                   __float_as_uint(acc2[q][2] * fg * scale), __float_as_uint(acc2[q][3] * fg * scale)};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs, ch < M ? (c * M + ch) * 4 : (int)0x80000000, 0, 0);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc2[q][r] * fg * scale), rs,
                                                              ch + r < M ? (c * M + ch + r) * 4 : (int)0x80000000, 0, 0);
                }
            }
        }
        if constexpr (GRADS) {
            // rows packed in pairs (in place: GEMM1 and GEMM2 are done with these)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int k1 = 0; k1 < 2; ++k1) {
                    bh[k1][i] = pair_rows(bh[k1][i], psel);
                    bl[k1][i] = pair_rows(bl[k1][i], psel);
                }
#pragma unroll
                for (int k2 = 0; k2 < 4; ++k2) {
                    dh[k2][i] = pair_rows(dh[k2][i], psel);
                    dl[k2][i] = pair_rows(dl[k2][i], psel);
                }
            }
            // the round's largest row (smallest shift) of h and of dy
            const bool hfin = ph >= -114, dfin = sd >= -126;
            int th = hfin ? ph : 1000, td = dfin ? sd : 1000;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                th = min(th, __shfl_xor(th, off, 64));
                td = min(td, __shfl_xor(td, off, 64));
            }
            if (lane == 0) {
                rsc[par][wv][0] = th;
                rsc[par][wv][1] = td;
            }
            lds_barrier();
#pragma unroll
            for (int w = 0; w < RW; ++w) {
                th = min(th, rsc[par][w][0]);
                td = min(td, rsc[par][w][1]);
            }
            // per row: to the round's scale; a packed register holds rows (c & ~1, c | 1)
            const int dph = hfin ? th - ph : 0, dsd = dfin ? td - sd : 0;
            const int dph2 = __builtin_amdgcn_update_dpp(0, dph, 0xB1, 0xF, 0xF, true);
            const int dsd2 = __builtin_amdgcn_update_dpp(0, dsd, 0xB1, 0xF, 0xF, true);
            const v2h sh2 = {(_Float16)ldexpf(1.f, odd ? dph2 : dph), (_Float16)ldexpf(1.f, odd ? dph : dph2)};
            const v2h sd2 = {(_Float16)ldexpf(1.f, odd ? dsd2 : dsd), (_Float16)ldexpf(1.f, odd ? dsd : dsd2)};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int k1 = 0; k1 < 2; ++k1) {
                    bh[k1][i] = scale_halves(bh[k1][i], sh2);
                    bl[k1][i] = scale_halves(bl[k1][i], sh2);
                }
#pragma unroll
                for (int k2 = 0; k2 < 4; ++k2) {
                    dh[k2][i] = scale_halves(dh[k2][i], sd2);
                    dl[k2][i] = scale_halves(dl[k2][i], sd2);
                }
            }
            v4f s3[4], sdc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) s3[q] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if ((wv >> 2) == half) {
                    // rows 16 (wv % 4) + c of the 64: k block (wv % 4) / 2, slot (lane group gr, e = c % 8)
                    const int kk = (wv & 3) >> 1, gr = 2 * (wv & 1) + (c >> 3), e = c & 7;
                    // dword of the slot pair (e & ~1) of lane (gr, col): even lanes write the first
                    // half-word's column, odd lanes the second's
                    auto at = [&](v4u *blk, int col) { return reinterpret_cast<uint32_t *>(blk + gr * 16 + col) + (e >> 1); };
                    const int p = odd ? 1 : 0;
#pragma unroll
                    for (int k1 = 0; k1 < 2; ++k1)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int q = 2 * k1 + (i >> 1), col = 8 * (i & 1) + 2 * g + p;
                            *at(h3[kk][q][0], col) = bh[k1][i];
                            *at(h3[kk][q][1], col) = bl[k1][i];
                        }
#pragma unroll
                    for (int k2 = 0; k2 < 4; ++k2)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int n = 2 * k2 + (i >> 1), col = 4 * g + 2 * (i & 1) + p;
                            *at(d3[kk][n][0], col) = dh[k2][i];
                            *at(d3[kk][n][1], col) = dl[k2][i];
                        }
                }
                lds_barrier();
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const v4u xh = d3[kk][wv][0][lane], xl = d3[kk][wv][1][lane];
                    v4u ah[4], al[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        ah[q] = h3[kk][q][0][lane];
                        al[q] = h3[kk][q][1][lane];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) s3[q] = mfma_h(al[q], xh, s3[q]);
                    sdc = mfma_h(ones, xl, sdc);
#pragma unroll
                    for (int q = 0; q < 4; ++q) s3[q] = mfma_h(ah[q], xl, s3[q]);
                    sdc = mfma_h(ones, xh, sdc);
#pragma unroll
                    for (int q = 0; q < 4; ++q) s3[q] = mfma_h(ah[q], xh, s3[q]);
                }
                // the next half (or the next round, past its first barrier) overwrites h3 and d3
                if (half == 0) lds_barrier();
            }
            // in two factors, as the largest h and the largest dy need not meet in a row
            const float f3 = ldexpf(1.f, -th), f4 = ldexpf(1.f, -(td + sw));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc3[q][r] = fmaf(s3[q][r] * f3, f4, acc3[q][r]);
            dca = fmaf(sdc[0], f4, dca);   // row 0: lanes g = 0
        }
    }

    // per-block partials: [dWa (RH x RM) | dWb (RNO x RH) | dca (RH) | dcb (RNO) | sum err^2];
    // every wave writes its hidden rows of dWa and dca, the rest is summed over the block's waves
    float *pb = part + (long)blockIdx.x * RPS_PAD;
#pragma unroll
    for (int o = 0; o < RNO; ++o) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) dcb[o] += GRADS ? __shfl_xor(dcb[o], off, 64) : 0.f;
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) lsum += __shfl_xor(lsum, off, 64);
    if constexpr (GRADS) {
        constexpr int RV = RNO * RH + RNO + 1;
        static_assert(RW * RV * sizeof(float) <= sizeof(d3), "block sums fit in the dS tiles");
        lds_barrier();   // every wave is past its reads of d3
        float *red = reinterpret_cast<float *>(&d3[0][0][0][0]);
        float *rw = red + wv * RV;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) pb[(16 * wv + c) * RM + 16 * q + 4 * g + r] = scale * acc3[q][r];
        if (g == 0) pb[RH * RM + RNO * RH + 16 * wv + c] = scale * dca;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int o = 0; o < RNO; ++o) {
                const float t = dwb[p][o] + __shfl_xor(dwb[p][o], 32, 64);
                if (lane < 32) rw[o * RH + 32 * p + lane] = t;
            }
        if (lane < RNO) {
            float v = dcb[0];
#pragma unroll
            for (int o = 1; o < RNO; ++o)
                if (lane == o) v = dcb[o];
            rw[RNO * RH + lane] = v;
        }
        if (lane == 0) rw[RV - 1] = lsum;
        __syncthreads();
        for (int e = tid; e < RV; e += RW * 64) {
            float t = 0.f;
#pragma unroll
            for (int w2s = 0; w2s < RW; ++w2s) t += red[w2s * RV + e];
            pb[e < RNO * RH ? RH * RM + e : RH * RM + RH + e] = t;   // dcb and the loss follow dca
        }
    } else {
        if (lane == 0) lsw[wv] = lsum;
        __syncthreads();
        if (tid == 0) {
            float t = 0.f;
#pragma unroll
            for (int w2s = 0; w2s < RW; ++w2s) t += lsw[w2s];
            pb[RPS - 1] = t;
        }
    }
}

// float64 sums of the per-block partials: stage 1 over slices of the blocks, stage 2 over slices
constexpr int RO_SLICES = 256;

__global__ __launch_bounds__(256) void k_readout_sum1(const float *__restrict__ part, int nwaves, int only_loss,
                                                      double *__restrict__ part2) {
    const int sl = blockIdx.x;
    const int w0 = (int)((long)nwaves * sl / RO_SLICES), w1 = (int)((long)nwaves * (sl + 1) / RO_SLICES);
    for (int e = only_loss ? RPS - 1 + (int)threadIdx.x : (int)threadIdx.x; e < RPS; e += 256) {
        double s0 = 0.0, s1 = 0.0;
        int w = w0;
        for (; w + 1 < w1; w += 2) {
            s0 += (double)part[(size_t)w * RPS_PAD + e];
            s1 += (double)part[(size_t)(w + 1) * RPS_PAD + e];
        }
        if (w < w1) s0 += (double)part[(size_t)w * RPS_PAD + e];
        part2[(size_t)sl * RPS + e] = s0 + s1;
    }
}

__global__ __launch_bounds__(256) void k_readout_sum2(const double *__restrict__ part2, RoGrads gr, int M, int H,
                                                      int No, float loss_scale, float *__restrict__ loss) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= RPS) return;
    if (!loss && e == RPS - 1) return;
    if (!gr.Wa && !gr.Wb && !gr.ca && !gr.cb && e != RPS - 1) return;
    double s = 0.0;
    for (int sl = 0; sl < RO_SLICES; ++sl) s += part2[(size_t)sl * RPS + e];
    if (e < RH * RM) {
        const int i = e / RM, k = e % RM;
        if (gr.Wa && i < H && k < M) gr.Wa[i * M + k] = (float)s;
    } else if (e < RH * RM + RNO * RH) {
        const int o = (e - RH * RM) / RH, i = (e - RH * RM) % RH;
        if (gr.Wb && o < No && i < H) gr.Wb[o * H + i] = (float)s;
    } else if (e < RH * RM + RNO * RH + RH) {
        const int i = e - RH * RM - RNO * RH;
        if (gr.ca && i < H) gr.ca[i] = (float)s;
    } else if (e < RPS - 1) {
        const int o = e - RH * RM - RNO * RH - RH;
        if (gr.cb && o < No) gr.cb[o] = (float)s;
    } else {
        loss[0] = (float)(s * (double)loss_scale);
    }
}

// persistent grid: as many blocks as are resident at once (one pass over the tiles)
static int readout_grid(long rows) {
    static int resident = 0;
    if (!resident) {
        int dev = 0, cus = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_readout<true>, RW * 64, 0) != hipSuccess || per < 1)
            per = 1;
        resident = cus * per;
    }
    const long ntiles = (rows + 15) / 16;
    const long want = (ntiles + RW - 1) / RW;
    return (int)(want < resident ? want : resident);
}

size_t readout_ws_bytes(int B, int T) {
    const int grid = readout_grid((long)B * T);
    const size_t p1 = ((size_t)grid * RPS_PAD * sizeof(float) + 255) & ~(size_t)255;
    return p1 + (size_t)RO_SLICES * RPS * sizeof(double);
}

int launch_readout(const RoArgs &ra, int B, int T, const float *h, const float *x, float *g, uint32_t *masks,
                   float *loss, const RoGrads &gr, void *ws, hipStream_t st) {
    const int grid = readout_grid((long)B * T);
    const size_t p1 = ((size_t)grid * RPS_PAD * sizeof(float) + 255) & ~(size_t)255;
    float *part = (float *)ws;
    double *part2 = (double *)((char *)ws + p1);
    const float scale = 2.0f / ((float)B * (float)ra.No * (float)T);
    const bool grads = gr.Wa || gr.ca || gr.Wb || gr.cb;
    {
        KTimer _kt("k_readout", st);
        if (grads)
            hipLaunchKernelGGL(k_readout<true>, dim3(grid), dim3(RW * 64), 0, st, ra, h, x, B, T, scale, g, masks, part);
        else
            hipLaunchKernelGGL(k_readout<false>, dim3(grid), dim3(RW * 64), 0, st, ra, h, x, B, T, scale, g, masks,
                               part);
    }
    DEER_LAUNCH_CHECK("k_readout");
    if (grads || loss) {
        KTimer _kt("k_readout_sum", st);
        hipLaunchKernelGGL(k_readout_sum1, dim3(RO_SLICES), dim3(256), 0, st, (const float *)part, grid,
                           grads ? 0 : 1, part2);
        hipLaunchKernelGGL(k_readout_sum2, dim3((RPS + 255) / 256), dim3(256), 0, st, (const double *)part2, gr, ra.M,
                           ra.H, ra.No, 0.5f * scale, loss);
        DEER_LAUNCH_CHECK("k_readout_sum");
    }
    return DEER_OK;
}

}  // namespace deer
