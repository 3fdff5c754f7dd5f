// fp32 storage path: projections and attention on the fp32 matrix instruction (v_mfma_f32_16x16x4), every product and
// sum in fp32.
//
// What bounds it: the models that run in fp32 are small (two layers of width 256 over 128 suffix tokens: 0.35 GFLOP,
// 10 MB), so a pass is a chain of dependent launches that each last about as long as their memory round trips.  The
// kernels are therefore cut for latency: many small workgroups, every operand requested at once straight into the
// registers the matrix instruction reads, the k range of a projection and the key range of an attention tile split
// over the wavefronts of a workgroup, and RMSNorm, rotation, SwiGLU and the residual add done where the operands pass
// by.  Measured on that model: 487 -> 62 us per pass (12 launches instead of 20; in a kernel trace 3 to 6 us a projection, 8 us
// the attention; the launches alone take the host about 47 us).
#include "kernels.h"
#include <algorithm>
#include <cfloat>

namespace cs {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------------------------------------
// C[M,N] = A[M,K] . W[N,K]^T.  A workgroup owns a tile of 16 BLK x 16 BLK; its NW wavefronts take the 16-wide k groups
// of the tile in turn (wavefront w the groups w, w + NW, ...) and their partial products are added through LDS in
// wavefront order.  A lane holds k 16 kg + 4 (lane / 16) .. + 3 of row lane % 16 of a block as one 16-byte load per
// operand; the four matrix instructions of a group take its components in turn (which k meets which is the same for
// both operands, so their order is free).
// NORM: A holds rows of the residual stream, not yet normalised.  The gain is applied on the way in; the workgroup
// passes over whole rows, so it knows their sum of squares too, and 1 / rms scales the result rows at the end.
// Column pairs: with the SwiGLU and the rotating epilogue the first half of a tile's columns are gate rows (or columns
// of a head's first half) and the second half their partners.
template <int EPI, bool NORM, int BLK, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmF32 p) {
    constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_ROPE;
    constexpr int NE = BLK * 16, HALF = NE / 2;
    constexpr int UN = BLK == 1 ? 4 : 2;                  // k groups requested together
    __shared__ float red[NW][NE][NE + 1];
    __shared__ float ssq[NW][NE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fg = lane >> 4;
    const int m0 = blockIdx.x * NE, t = blockIdx.y;
    int rA = t * NE, rB = rA + HALF;                      // weight rows of the two halves of the tile's columns
    const int half_hd = p.hd >> 1;
    int head = 0, o0 = 0;
    if constexpr (EPI == EPI_SWIGLU) {                    // rows interleaved 32 gate / 32 up
        const int f0 = t * HALF;
        rA = 64 * (f0 >> 5) + (f0 & 31);
        rB = rA + 32;
    } else if constexpr (EPI == EPI_ROPE) {
        const int per_head = half_hd / HALF;
        head = t / per_head;
        o0 = (t - head * per_head) * HALF;
        rA = head * p.hd + o0;
        rB = rA + half_hd;
    }
    const float *ap[BLK], *wp[BLK];
#pragma unroll
    for (int i = 0; i < BLK; ++i) {
        const int col = 16 * i + fr;
        ap[i] = p.A + (size_t)min(m0 + 16 * i + fr, p.M - 1) * p.K + 4 * fg;   // rows past M repeat the last one
        wp[i] = p.W + (size_t)(col < HALF ? rA + col : rB + col - HALF) * p.K + 4 * fg;
    }
    f32x4 acc[BLK][BLK];
    float sq[BLK];
#pragma unroll
    for (int i = 0; i < BLK; ++i) {
        sq[i] = 0.f;
#pragma unroll
        for (int j = 0; j < BLK; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int nkg = p.K >> 4;
    for (int kb = wave; kb < nkg; kb += NW * UN) {
        f32x4 a[UN][BLK], w[UN][BLK], g[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int kg = kb + NW * u;
            if (kg < nkg) {                               // wave-uniform
#pragma unroll
                for (int i = 0; i < BLK; ++i) {
                    a[u][i] = *reinterpret_cast<const f32x4 *>(ap[i] + 16 * kg);
                    w[u][i] = *reinterpret_cast<const f32x4 *>(wp[i] + 16 * kg);
                }
                if constexpr (NORM) g[u] = *reinterpret_cast<const f32x4 *>(p.g + 16 * kg + 4 * fg);
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (kb + NW * u >= nkg) break;
            if constexpr (NORM) {
#pragma unroll
                for (int i = 0; i < BLK; ++i) {
                    sq[i] += a[u][i][0] * a[u][i][0] + a[u][i][1] * a[u][i][1] + a[u][i][2] * a[u][i][2] + a[u][i][3] * a[u][i][3];
                    a[u][i] *= g[u];
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < BLK; ++i)
#pragma unroll
                    for (int j = 0; j < BLK; ++j) acc[i][j] = mma_f32(a[u][i][c], w[u][j][c], acc[i][j]);
        }
    }
    // a block's result: column lane % 16, rows 4 (lane / 16) + e
#pragma unroll
    for (int i = 0; i < BLK; ++i) {
#pragma unroll
        for (int j = 0; j < BLK; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave][16 * i + 4 * fg + e][16 * j + fr] = acc[i][j][e];
        if constexpr (NORM) {
            sq[i] += __shfl_xor(sq[i], 16);
            sq[i] += __shfl_xor(sq[i], 32);
            if (fg == 0) ssq[wave][16 * i + fr] = sq[i];
        }
    }
    __syncthreads();
    constexpr int N_EL = NE * (PAIR ? HALF : NE);
    for (int idx = threadIdx.x; idx < N_EL; idx += 64 * NW) {
        const int r = idx / (PAIR ? HALF : NE), c = idx % (PAIR ? HALF : NE), m = m0 + r;
        if (m >= p.M) continue;
        float v = 0.f, v2 = 0.f, rinv = 1.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            v += red[w][r][c];
            if constexpr (PAIR) v2 += red[w][r][c + HALF];
        }
        if constexpr (NORM) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += ssq[w][r];
            rinv = 1.0f / sqrtf(s / (float)p.K + p.eps);
            v *= rinv;
            v2 *= rinv;
        }
        if constexpr (EPI == EPI_SWIGLU) {
            p.out[(size_t)m * (p.N >> 1) + t * HALF + c] = v / (1.0f + expf(-v)) * v2;
        } else if constexpr (EPI == EPI_ROPE) {
            const RopeArgs &ro = p.rope;
            const bool is_q = head < ro.Hq, is_v = head >= ro.Hq + ro.Hkv;
            const int hh = is_q ? head : is_v ? head - ro.Hq - ro.Hkv : head - ro.Hq;
            float *dst = reinterpret_cast<float *>(is_q ? ro.q : is_v ? ro.v : ro.k) +
                         ((size_t)m * (is_q ? ro.Hq : ro.Hkv) + hh) * p.hd + o0 + c;
            float lo = v, hi = v2;
            if (!is_v) {
                const float cs = ro.cos_t[(size_t)m * half_hd + o0 + c], sn = ro.sin_t[(size_t)m * half_hd + o0 + c];
                lo = v * cs - v2 * sn;
                hi = v2 * cs + v * sn;
            }
            dst[0] = lo;
            dst[half_hd] = hi;
        } else {
            float *o = p.out + (size_t)m * p.N + t * NE + c;
            *o = EPI == EPI_RESID_F32 ? *o + v : v;
        }
    }
}

// 16 x 16 tiles while they leave the chip room (up to two of them a CU), 32 x 32 beyond, which read half the operand bytes per flop.  Those have
// eight wavefronts while they are about half of one to two a CU (513 to 2048 tiles of 16 x 16) and a k range of up to 512 is one or two rounds
// of theirs: 128 rows, 256 x 2048, gate/up, 8.1 -> 6.0 us.  The line is the right one in the lower half, too, though not every CU has a tile there - whole pass
// of two layers, 16 x 16 against 32 x 32 from 513 tiles on: 640 tiles (80 rows, 2048 columns) at K 256 61.0 : 58.2 us, at K 512 71.6 : 68.8, 896 tiles at
// K 512 79.3 : 72.7, 832 tiles (208 rows, 1024 columns, the QKV of 624 with it) at K 256 64.7 : 60.8; nowhere slower between 513 and 1023.  Longer k ranges:
// 16 x 16 up to 2048 tiles, k split over eight wavefronts instead of four.
template <int EPI, bool NORM>
static hipError_t launch_gemm_f32_epi(const GemmF32 &p, hipStream_t s) {
    const long tiles16 = (long)((p.M + 15) / 16) * (p.N / 16);
    if (tiles16 > 512 && tiles16 <= 2048 && p.K <= 512) {
        const dim3 grid((p.M + 31) / 32, p.N / 32);
        gemm_f32_kernel<EPI, NORM, 2, 8><<<grid, 512, 0, s>>>(p);
    } else if (tiles16 <= 2048) {
        const dim3 grid((p.M + 15) / 16, p.N / 16);
        if (p.K >= 512) gemm_f32_kernel<EPI, NORM, 1, 8><<<grid, 512, 0, s>>>(p);
        else gemm_f32_kernel<EPI, NORM, 1, 4><<<grid, 256, 0, s>>>(p);
    } else {
        const dim3 grid((p.M + 31) / 32, p.N / 32);
        gemm_f32_kernel<EPI, NORM, 2, 4><<<grid, 256, 0, s>>>(p);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmF32 &p, int epi, hipStream_t s) {
    if (p.M < 1 || p.N % 64 != 0 || p.K % 16 != 0 || (epi == EPI_ROPE && (p.hd % 32 != 0 || p.N % p.hd != 0))) return hipErrorInvalidValue;
    switch (epi) {
        case EPI_STORE_F32: return p.g ? launch_gemm_f32_epi<EPI_STORE_F32, true>(p, s) : launch_gemm_f32_epi<EPI_STORE_F32, false>(p, s);
        case EPI_RESID_F32: return p.g ? hipErrorInvalidValue : launch_gemm_f32_epi<EPI_RESID_F32, false>(p, s);
        case EPI_SWIGLU: return p.g ? launch_gemm_f32_epi<EPI_SWIGLU, true>(p, s) : launch_gemm_f32_epi<EPI_SWIGLU, false>(p, s);
        case EPI_ROPE: return p.g ? launch_gemm_f32_epi<EPI_ROPE, true>(p, s) : hipErrorInvalidValue;
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------------------
// Attention.  One workgroup per (16 query rows, kv head, trace); the rows are the (suffix token, q head of the group)
// pairs of the trace, row = t * G + g.  Its wavefronts take the 16-key tiles in turn, each with a running (max, sum, O)
// of its own (online softmax), and merge through LDS in wavefront order at the end.  Scores are computed transposed,
// S^T = K . Q^T, so a lane owns one query (lane % 16) and ends up holding the probabilities of keys 4 (lane / 16) .. + 3,
// which is what O^T += V^T . P^T wants of it.
__device__ __forceinline__ size_t key_block(const AttnArgs &a, int b, int j) {   // block-table index of cached key j (of the last column past it)
    return (size_t)b * a.max_blocks + min((unsigned)j / (unsigned)a.block_size, (unsigned)a.max_blocks - 1u);
}
__device__ __forceinline__ const float *key_row(const AttnArgs &a, const float *pages, const float *suf, int L, int cu_b, int c, int j, int blk) {
    if (j < L) {
        blk = min(max(blk, 0), a.n_blocks - 1);
        return pages + (((size_t)blk * a.Hkv + c) * a.block_size + (unsigned)j % (unsigned)a.block_size) * a.hd;
    }
    int t = min(cu_b + (j - L), a.T - 1);
    return suf + ((size_t)t * a.Hkv + c) * a.hd;
}
// Wave-uniform loads of what no kernel of this launch writes: into scalar registers, apart from the vector memory counter.
typedef __attribute__((address_space(4))) const int32_t scalar_i32;
__device__ __forceinline__ int scalar_load(const int32_t *p) { return *(scalar_i32 *)(uintptr_t)p; }

// What bounds it is a chain of round trips: lengths, block-table entries, keys and values, once per round of 16 NW keys.  So the
// entries are asked for before the lengths are known, the next round's before this one's products, twelve wavefronts take 192 keys in a round
// where the grid leaves a CU to a workgroup, and four of them merge the results, four dims a lane.  Where a tile's keys lie in one block, its entry
// and address are wave-uniform.  Launch, 4 traces of 128 + 32 keys, 4 heads of 64: 11 -> 7.8 us; whole pass (two layers), 4 traces of 512 + 64: 100 -> 80 us,
// 16: 155 -> 142; head size 128, 32 of 2048 + 32, 4 / 2 heads: 568 -> 367, the same with blocks of 5: 600 -> 392.
// (Wavefronts per SIMD given: left alone, the branch for values that are not finite takes registers of a wavefront's worth.  At head size 128 it
// is two, 174 and 185 registers: with three, 168, keys asked for ahead and addresses spilled, 20 and 48 bytes - 367 and 426 us in those two cases, 16 of
// 4096 + 100 with 2 / 2 heads and blocks of 5 584 for 506.)
// PAGE: block_size is a multiple of 16, so the 16 keys of a tile lie in one block.
template <int HD, int NW, bool PAGE>
__global__ __launch_bounds__(64 * NW, HD == 128 ? 2 : NW == 12 ? 3 : 4) void attn_f32_kernel(AttnArgs a) {
    constexpr int NK = HD / 16, OS = HD + 4;
    __shared__ __attribute__((aligned(16))) float om[NW][16][OS];       // O of a wavefront, [query][dim]
    __shared__ float mls[NW][2][16];
    asm volatile("" : : "s"(a.q), "s"(a.ksuf), "s"(a.vsuf), "s"(a.k_pages), "s"(a.v_pages), "s"(a.block_table), "s"(a.cu), "s"(a.plens), "s"(a.out), "s"(a.scale),
                 "s"(a.block_size), "s"(a.max_blocks), "s"(a.n_blocks), "s"(a.T), "s"(a.Hq), "s"(a.Hkv));
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fg = lane >> 4;
    const int c = blockIdx.y, G = a.Hq / a.Hkv;
    for (int b = blockIdx.z; b < a.B; b += gridDim.z) {
        // Block-table entries of the round to come: one for the 16 keys of a tile, or one for this lane's key and for each of its four values.
        int blk[PAGE ? 1 : 5];
        auto fetch_blocks = [&](int j0) __attribute__((always_inline)) {
            if constexpr (PAGE) {
                blk[0] = scalar_load(a.block_table + key_block(a, b, j0));
            } else {
                blk[0] = a.block_table[key_block(a, b, j0 + fr)];
    #pragma unroll
                for (int e = 0; e < 4; ++e) blk[1 + e] = a.block_table[key_block(a, b, j0 + 4 * fg + e)];
            }
        };
        fetch_blocks(16 * wave);
        const int cu_0 = scalar_load(a.cu + b), cu_1 = scalar_load(a.cu + b + 1), len = scalar_load(a.plens + b);
        asm volatile("" : : "s"(cu_0), "s"(cu_1), "s"(len));   // (in one round)
        const int cu_b = min(max(cu_0, 0), a.T - 1), S = min(max(cu_1, cu_b + 1), a.T) - cu_b;
        const int L = min(max(len, 0), a.max_blocks * a.block_size);
        const int row0 = blockIdx.x * 16, n_rows = G * S;
        if (row0 >= n_rows) continue;                         // a shorter trace (uniform)
        const int r = min(row0 + fr, n_rows - 1), tt = r / G, g = r - tt * G;
        const int n_keys = L + tt + 1;                        // keys this lane's query sees
        const int n_all = L + min(row0 + 15, n_rows - 1) / G + 1;
        f32x4 q[NK];
        const float *qr = reinterpret_cast<const float *>(a.q) + ((size_t)(cu_b + tt) * a.Hq + c * G + g) * HD + 4 * fg;
        const float *kp = reinterpret_cast<const float *>(a.k_pages), *vp = reinterpret_cast<const float *>(a.v_pages);
        const float *ks = reinterpret_cast<const float *>(a.ksuf), *vs = reinterpret_cast<const float *>(a.vsuf);
        float m = -INFINITY, l = 0.f;
        f32x4 o[NK];
    #pragma unroll
        for (int i = 0; i < NK; ++i) {
            q[i] = *reinterpret_cast<const f32x4 *>(qr + 16 * i);
            o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        bool scaled = false;
        for (int j0 = 16 * wave; j0 < n_all; j0 += 16 * NW) {
            // keys past the last one are clamped to it, which is a suffix token (no entry is used for it), and masked
            const float *kr, *vr[4];
            if constexpr (PAGE) {
                const int bs = a.block_size;
                const size_t at = (((size_t)min(max(blk[0], 0), a.n_blocks - 1) * a.Hkv + c) * bs + (unsigned)j0 % (unsigned)bs) * HD;
                auto row = [&](const float *pages, const float *suf, int i) {
                    const int j = min(j0 + i, n_all - 1);
                    return j < L ? pages + at + i * HD : suf + ((size_t)min(cu_b + (j - L), a.T - 1) * a.Hkv + c) * HD;
                };
                kr = row(kp, ks, fr) + 4 * fg;
    #pragma unroll
                for (int e = 0; e < 4; ++e) vr[e] = row(vp, vs, 4 * fg + e) + fr;
            } else {
                kr = key_row(a, kp, ks, L, cu_b, c, min(j0 + fr, n_all - 1), blk[0]) + 4 * fg;
    #pragma unroll
                for (int e = 0; e < 4; ++e) vr[e] = key_row(a, vp, vs, L, cu_b, c, min(j0 + 4 * fg + e, n_all - 1), blk[1 + e]) + fr;
            }
            f32x4 k[NK];
            float v[NK][4];
    #pragma unroll
            for (int i = 0; i < NK; ++i) k[i] = *reinterpret_cast<const f32x4 *>(kr + 16 * i);
    #pragma unroll
            for (int i = 0; i < NK; ++i)
    #pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = vr[e][16 * i];
            if (j0 + 16 * NW < n_all) fetch_blocks(j0 + 16 * NW);
            if (!scaled) {                                                    // (here, behind the first round's loads)
    #pragma unroll
                for (int i = 0; i < NK; ++i) q[i] *= a.scale;
                scaled = true;
            }
            f32x4 s2[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};      // two chains: the instruction's latency is 8 cycles a link
    #pragma unroll
            for (int i = 0; i < NK; ++i)
    #pragma unroll
                for (int e = 0; e < 4; ++e) s2[e & 1] = mma_f32(k[i][e], q[i][e], s2[e & 1]);
            f32x4 sc = s2[0] + s2[1];
            float mx = -INFINITY;
    #pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[e] = j0 + 4 * fg + e < n_keys ? sc[e] : -INFINITY;
                mx = fmaxf(mx, sc[e]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx);
            const float ref = m_new == -INFINITY ? 0.f : m_new;               // a tile no key of which this query sees
            const float alpha = m == -INFINITY ? 0.f : expf(m - ref);
            float ps = 0.f;
    #pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[e] = expf(sc[e] - ref);
                ps += sc[e];
            }
            ps += __shfl_xor(ps, 16);
            ps += __shfl_xor(ps, 32);
            l = l * alpha + ps;
            m = m_new;
    #pragma unroll
            for (int i = 0; i < NK; ++i) o[i] *= alpha;
            if (j0 + 16 > L + row0 / G + 1) {                                 // (uniform) a query of the tile does not see all keys
                // Its probability of them is zero, which must not meet a NaN or an infinity: such values are taken out of the
                // matrix product and added for the queries that see them.  Never taken with finite values.
                bool odd = false;
    #pragma unroll
                for (int i = 0; i < NK; ++i)
    #pragma unroll
                    for (int e = 0; e < 4; ++e) odd |= !(fabsf(v[i][e]) <= FLT_MAX);
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0, 0)) {
    #pragma unroll
                    for (int i = 0; i < NK; ++i)
    #pragma unroll
                        for (int e = 0; e < 4; ++e) v[i][e] = fabsf(v[i][e]) <= FLT_MAX ? v[i][e] : 0.f;
    #pragma unroll 1
                    for (int jj = 0; jj < 16; ++jj) {
                        const int e = jj & 3;
                        const float p = __shfl(e == 0 ? sc[0] : e == 1 ? sc[1] : e == 2 ? sc[2] : sc[3], 16 * (jj >> 2) + fr);
                        const int jk = min(j0 + jj, n_all - 1);
                        const float *row = key_row(a, vp, vs, L, cu_b, c, jk, a.block_table[key_block(a, b, jk)]) + 4 * fg;
    #pragma unroll
                        for (int i = 0; i < NK; ++i) {
                            const f32x4 w = *reinterpret_cast<const f32x4 *>(row + 16 * i);
    #pragma unroll
                            for (int d = 0; d < 4; ++d)
                                if (j0 + jj < n_keys && !(fabsf(w[d]) <= FLT_MAX)) o[i][d] += p * w[d];
                        }
                    }
                }
            }
    #pragma unroll
            for (int i = 0; i < NK; ++i)
    #pragma unroll
                for (int e = 0; e < 4; ++e) o[i] = mma_f32(v[i][e], sc[e], o[i]);
        }
        // o[i][e]: dim 16 i + 4 (lane / 16) + e of query lane % 16
    #pragma unroll
        for (int i = 0; i < NK; ++i) *reinterpret_cast<f32x4 *>(&om[wave][fr][16 * i + 4 * fg]) = o[i];
        if (fg == 0) {
            mls[wave][0][fr] = m;
            mls[wave][1][fr] = l;
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < 16 * HD / 4; idx += 64 * NW) {
            const int rr = idx / (HD / 4), d = idx % (HD / 4) * 4;
            if (row0 + rr >= n_rows) continue;
            float M = -INFINITY;
    #pragma unroll
            for (int w = 0; w < NW; ++w) M = fmaxf(M, mls[w][0][rr]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            float lt = 0.f;
    #pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float mw = mls[w][0][rr];
                const f32x4 ow = *reinterpret_cast<const f32x4 *>(&om[w][rr][d]);
                if (mw == -INFINITY) continue;
                const float wgt = expf(mw - M);
                acc += wgt * ow;
                lt += wgt * mls[w][1][rr];
            }
            const int t = (row0 + rr) / G;
            *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + ((size_t)(cu_b + t) * a.Hq + c * G + (row0 + rr - t * G)) * HD + d) =
                f32x4{acc[0] / lt, acc[1] / lt, acc[2] / lt, acc[3] / lt};
        }
        __syncthreads();                                      // om and mls are free for the next trace
    }
}

hipError_t launch_attn_f32(const AttnArgs &a, int max_S, hipStream_t s) {
    const dim3 grid(((a.Hq / a.Hkv) * max_S + 15) / 16, a.Hkv, std::min(a.B, 32768));
    const bool page = a.block_size % 16 == 0;
    auto run = [&](auto kern, auto general, int threads) { (page ? kern : general)<<<grid, threads, 0, s>>>(a); };
    if (a.hd == 64 && (long)grid.x * grid.y * grid.z <= 256) run(attn_f32_kernel<64, 12, true>, attn_f32_kernel<64, 12, false>, 768);
    else if (a.hd == 64) run(attn_f32_kernel<64, 8, true>, attn_f32_kernel<64, 8, false>, 512);
    else if (a.hd == 128) run(attn_f32_kernel<128, 4, true>, attn_f32_kernel<128, 4, false>, 256);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace cs
