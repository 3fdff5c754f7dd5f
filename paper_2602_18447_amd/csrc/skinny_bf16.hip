// Projections of a pass over few rows (at most SK_MAX_ROWS tokens: generation steps, one interactive trace, a handful
// of short steps), bf16 or fp16 operands on the 16x16x32 matrix instruction.
//
// What bounds them: each weight matrix is read once from HBM against operands that fit the L2, so the floor of a
// launch is that stream (6 MB: 3.3 us, 28 MB: 6.2 us, 55 MB: 10.2 us, measured with a bare read loop), and below about
// 30 MB the chain of memory round trips inside the launch, not the stream, decides its time.  Hence:
//  - a workgroup owns all rows of one tile of 16 CT columns and its wavefronts split the k range between them: no operand
//    is shared inside a workgroup, so the main loop has no barrier.  A wavefront's weight k-tiles travel global -> LDS
//    directly into a ring of its own (whole 128-byte lines; read straight into the registers of the matrix instruction
//    they would be 16-byte pieces of 16 rows, at a quarter of the rate: 26 against 15 us for the gate/up projection over
//    32 rows).  Activations are kept in fragment order (frag_index): the 16 rows x 32 k of a matrix operand are 1 KiB in
//    lane order, so they do go straight to registers, each load one contiguous kilobyte;
//  - everything the epilogue reads (residual rows, gains, rotary tables, cache rows) is requested in front of the main
//    loop, so that it arrives under the weights;
//  - RMSNorm costs no launch: a residual projection writes, next to the fp32 rows, the 16-bit operand
//    x * gain * (power of two near 1 / rms of the row as it was before the update, whatever the level of the residual
//    stream) and the sum of squares of each of its 16-column tiles; the projection that consumes it scales its result
//    rows by the exact 1 / rms over that power of two.  A row that one update grows or shrinks so far that its operand
//    leaves the format's range is told by the consumer (the producer gives the partial sum of squares of a tile with such
//    an element a negative sign), which then multiplies once more with that row's operand taken from the fp32 row and the
//    power of two of its own rms: elements are then at most sqrt(width) * gain, as after an RMSNorm of its own;
//  - where one workgroup per tile would leave the chip idle (long k over few columns) the k range is cut into S slices;
//    they leave fp32 partial products and the slice that arrives last (a counter per tile) adds them in slice order and
//    runs the epilogue: the order is fixed, whoever performs it, so results are bit-identical from run to run.
// Values handed over inside one launch travel as device-scope relaxed atomic stores and loads (written through to, and
// served from, the memory side of the per-XCD L2 caches); no cache is written back or invalidated as a whole.
#include "kernels.h"
#include "xwg.h"
#include <algorithm>
#include <type_traits>

namespace cs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define CS_LDS_AS __attribute__((address_space(3)))

namespace {

// 64 lanes x 16 bytes from a wave-uniform base plus a byte offset per lane into LDS at lds_dst + 16 * lane.  Inline
// assembly with a memory clobber: the compiler neither moves memory accesses across it nor waits for it; completion is
// waited for explicitly with wait_vm.
__device__ __forceinline__ void dma16_base(const char *base, unsigned off, unsigned lds_dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(lds_dst), "v"(off), "s"(base) : "memory");
}
// Barrier for LDS data only.  (__syncthreads() also waits until every store to global memory is acknowledged, about a
// microsecond.)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }
// the value of the lane N further in the row of 16 lanes, and the sum over the row
template <int N>
__device__ __forceinline__ float row_ror(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum16(float v) {
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    return v + row_ror<1>(v);
}
// at most N vector memory operations of this wavefront still outstanding (they complete in issue order)
template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

template <bool F16>
__device__ inline f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Weight rows behind the 16 columns of tile t.  Column 4 g + e (g, e = 0..3) is row rA + 4 g + e of a plain tile; where
// columns come in pairs (SwiGLU: gate and up of the same activation; rotation: a column of a head's first half and its
// partner) it is row rA + 2 g + e for e < 2 and the partner rB + 2 g + e - 2 for the others, so that a lane, which ends up
// with columns 4 g .. 4 g + 3 of a row, holds both halves of two pairs.
template <int EPI>
__device__ inline void tile_rows(int t, int &rA, int &rB) {
    if constexpr (EPI == SK_EPI_SWIGLU) {       // rows interleaved 32 gate / 32 up
        const int f0 = 8 * t;
        rA = 64 * (f0 >> 5) + (f0 & 31);
        rB = rA + 32;
    } else if constexpr (EPI == SK_EPI_ROPE) {  // the rows of a head are ordered [0..31 | 64..95 | 32..63 | 96..127]
        const int head = t >> 3, o0 = 8 * (t & 7);
        rA = head * 128 + (o0 < 32 ? o0 : 32 + o0);
        rB = rA + 32;
    } else {
        rA = 16 * t;
        rB = rA;
    }
}
// row of tile row r (= 4 g + e) relative to rA
template <int EPI>
__device__ inline int tile_row(int r, int rB_minus_rA) {
    if constexpr (EPI == SK_EPI_RESID) return r;
    else return 2 * (r >> 2) + (r & 1) + ((r >> 1) & 1) * rB_minus_rA;
}
__device__ inline unsigned pack2(float a, float b, int fmt) {   // fmt 3: IEEE half (saturating), else bf16
    if (fmt == 3) return (unsigned)__half_as_ushort(to_half_sat(a)) | ((unsigned)__half_as_ushort(to_half_sat(b)) << 16);
    return (unsigned)__bfloat16_as_ushort(__float2bfloat16(a)) | ((unsigned)__bfloat16_as_ushort(__float2bfloat16(b)) << 16);
}
// Of an operand x * gain * f: the largest magnitude that may be stored (half: the format's; bf16: one that leaves the
// products' sums finite), and the smallest f * rms of the row that leaves its elements' precision (half: the step of
// 2^-24 below 2^-14, against elements near f * rms).
__device__ constexpr float operand_max(bool f16) { return f16 ? 65504.0f : 0x1p96f; }
__device__ constexpr float operand_min_rms(bool f16) { return f16 ? 0x1p-4f : 0x1p-64f; }
// power of two at or below r, within what keeps products and quotients of two of them finite
__device__ inline float pow2_of(float r) { return __uint_as_float(__float_as_uint(fminf(fmaxf(r, 0x1p-60f), 0x1p60f)) & 0x7f800000u); }
__device__ inline unsigned pack2_lo(float a, float b, unsigned hi) {   // second bf16 terms
    return pack2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u), 1);
}

}  // namespace

// Row blocks whose partial products (1 KiB each and wavefront) are added in one pass: as many as 64 KiB of LDS hold (128 KiB
// where a workgroup has a CU to itself).
constexpr int skinny_rb(int mb, int ct, int nw) {
    int rb = mb;
    while (rb > 1 && (nw * rb * ct * 1024 > (nw == 8 && ct >= 4 ? 131072 : 65536) || mb % rb != 0)) --rb;
    return rb;
}

// MB: blocks of 16 rows; CT: 16-column tiles of a workgroup; NW wavefronts; D: k-tiles of a group.  A wavefront works in
// groups of D k-tiles: the weights of group g + 1 are on their way while group g is multiplied.  (A gate/up
// projection of one row block and tile in one buffer: three workgroups of 48 KiB fit a CU if their registers let them; with
// two it takes 14.7 instead of 12.4 us.)
template <int EPI, bool F16, int MB, int CT, int NW, int D, int NBUF>
__global__ __launch_bounds__(64 * NW, EPI == SK_EPI_SWIGLU && MB * CT == 1 && NBUF == 1 ? 6 : 2) void skinny_kernel(SkinnyGemm a) {
    constexpr int NT = 64 * NW;
    constexpr int RB = skinny_rb(MB, CT, NW);            // row blocks per pass of the reduction
    constexpr int NCH = MB / RB, NBK = RB * CT, EPB = (NBK + NW - 1) / NW;     // passes; 16 x 16 blocks of one, and per wavefront
    static_assert(MB % RB == 0, "reduction passes");
    constexpr int GB = D * CT * 2048;                    // bytes of a group's weights
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];    // [NW][n_buf groups]; then the partial products
    // RESID: power of two of the row's operand.  Others: factor of its result, negative where the operand given does not hold the
    // row; row_sc: power of two of the operand that does.
    __shared__ float row_f[16 * MB], row_sc[EPI == SK_EPI_RESID ? 1 : 16 * MB];
    __shared__ volatile int s_last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fg = lane >> 4;
    // everything below in one round of scalar loads instead of one per branch
    asm volatile("" : : "s"(a.X), "s"(a.W), "s"(a.K), "s"(a.n_ct), "s"(a.S), "s"(a.ms), "s"(a.ssq_in), "s"(a.sc_in), "s"(a.ssq_n), "s"(a.x),
                 "s"(a.xg_out), "s"(a.g_next), "s"(a.rope.cos_t), "s"(a.rope.sin_t), "s"(a.kv_row));
    // Workgroup -> (column tile, k slice, block of rows): the ms row blocks of a tile and slice, which read the same weights,
    // are 8 ids apart, on one XCD and its L2.
    const int n_t = a.n_ct / CT;
    const int ts = (int)(blockIdx.x / (8 * a.ms)) * 8 + (int)(blockIdx.x & 7), mi = (int)(blockIdx.x >> 3) % a.ms;
    if (ts >= n_t * a.S) return;
    const int s = ts / n_t, t = ts - s * n_t;                              // k slice, column tile
    const int r0 = 16 * MB * mi, M = min(a.M - r0, 16 * MB);               // rows r0 .. r0 + M - 1 (M >= 1: the launcher)
    const int nk = a.K >> 6;
    const int kt0 = (int)((long)s * nk / a.S), nks = (int)((long)(s + 1) * nk / a.S) - kt0;
    const int nkw = nks > wave ? (nks - wave + NW - 1) / NW : 0;           // k-tiles kt0 + wave, + NW, ... of this wavefront

    // ---- what the epilogue needs, requested first.  In a pass wavefront w finishes the 16 x 16 blocks w, w + NW, ...; a
    // lane has row fr and columns 4 fg .. 4 fg + 3 of a block.
    auto row_of = [&](int ch, int j) { return 16 * (RB * ch + min(wave + NW * j, NBK - 1) / CT) + fr; };
    auto tile_of = [&](int j) { return t * CT + min(wave + NW * j, NBK - 1) % CT; };
    f32x4 pre[NCH][EPB];         // RESID: the residual row's columns; ROPE: cos, cos, sin, sin of the lane's two pairs
    int kvr[NCH][EPB];
    uint2 gain[EPB];             // (kept as loaded: converted here, it would be waited for here)
#pragma unroll
    for (int j = 0; j < EPB; ++j) {
        const int tt = tile_of(j), col = tt * 16 + 4 * fg, o = 8 * (tt & 7) + 2 * fg;
        if constexpr (EPI == SK_EPI_RESID) gain[j] = *reinterpret_cast<const uint2 *>((a.xg_out ? a.g_next : a.W) + col);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            const int row = r0 + min(row_of(ch, j), M - 1);
            if constexpr (EPI == SK_EPI_RESID) pre[ch][j] = *reinterpret_cast<const f32x4 *>(a.x + (size_t)row * (a.n_ct * 16) + col);
            if constexpr (EPI == SK_EPI_ROPE) {
                const float2 cs = *reinterpret_cast<const float2 *>(a.rope.cos_t + (size_t)row * 64 + o);
                const float2 sn = *reinterpret_cast<const float2 *>(a.rope.sin_t + (size_t)row * 64 + o);
                pre[ch][j] = f32x4{cs.x, cs.y, sn.x, sn.y};
                kvr[ch][j] = a.kv_row ? a.kv_row[row] : -1;
            }
        }
    }
    // Partial sums of squares per row: 16 threads a row take every 16th partial; added up under the first group's loads.
    // Room for 96 of them (width 1536), for 320 (width 5120) where a thread has one row; what is beyond is summed here.
    constexpr int NP = (16 * MB * 16 + NT - 1) / NT;                       // passes over the rows
    constexpr int NSQ = NP == 1 ? 20 : 6;
    const bool want_f = EPI != SK_EPI_RESID || a.xg_out != nullptr;
    float sqv[NP][NSQ], sc_prev[NP], sq_far[NP];
    float sq_min[NP];                                                      // negative: a partial says that its operand left the range
    if (want_f) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = r0 + min(p * (NT / 16) + (tid >> 4), M - 1);
            sq_far[p] = sq_min[p] = 0.f;
            for (int i = (tid & 15) + 16 * NSQ; i < a.ssq_n; i += 16) {
                const float v = a.ssq_in[(size_t)row * a.ssq_n + i];
                sq_far[p] += fabsf(v);
                sq_min[p] = fminf(sq_min[p], v);
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = r0 + min(p * (NT / 16) + (tid >> 4), M - 1);
            const float *sp = a.ssq_in + (size_t)row * a.ssq_n;
#pragma unroll
            for (int e = 0; e < 6; ++e) sqv[p][e] = sp[min((tid & 15) + 16 * e, a.ssq_n - 1)];
            if constexpr (NSQ > 6) {
#pragma unroll
                for (int e = 6; e < NSQ; ++e) sqv[p][e] = 0.f;
                if (a.ssq_n > 96) {                                        // uniform
#pragma unroll
                    for (int e = 6; e < NSQ; ++e) sqv[p][e] = sp[min((tid & 15) + 16 * e, a.ssq_n - 1)];
                }
            }
            sc_prev[p] = a.sc_in[row];
        }
    }
    auto row_factors = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = p * (NT / 16) + (tid >> 4);
            float sq = sq_far[p];
#pragma unroll
            for (int e = 0; e < NSQ; ++e) {
                const float v = (tid & 15) + 16 * e < a.ssq_n ? sqv[p][e] : 0.f;
                sq += fabsf(v);
                sq_min[p] = fminf(sq_min[p], v);
            }
            sq = sum16(sq);
            const float rinv = 1.0f / sqrtf(sq / (float)a.d_norm + a.eps);
            float f;
            if constexpr (EPI == SK_EPI_RESID) {
                f = pow2_of(rinv);
                if (t == 0 && s == 0 && (tid & 15) == 0 && row < M) a.sc_out[r0 + row] = f;
            } else {
                const bool any_left = (__builtin_amdgcn_ballot_w64(sq_min[p] < 0.f) >> (lane & 48) & 0xffff) != 0;
                const bool own = any_left || sc_prev[p] < operand_min_rms(F16) * rinv;
                const float sc = own ? pow2_of(rinv) : sc_prev[p];
                f = own ? -(rinv / sc) : rinv / sc;
                if ((tid & 15) == 0 && row < 16 * MB) row_sc[row] = sc;
            }
            if ((tid & 15) == 0 && row < 16 * MB) row_f[row] = f;
        }
    };

    // ---- main loop
    const char *wbase[CT];
    int wdiff = 0;
#pragma unroll
    for (int i = 0; i < CT; ++i) {
        int rA, rB;
        tile_rows<EPI>(t * CT + i, rA, rB);
        wbase[i] = reinterpret_cast<const char *>(a.W) + (size_t)rA * a.K * 2;
        wdiff = rB - rA;                                                   // the same for every tile
    }
    // Direct loads: one instruction fills 8 rows x 128 bytes; lane l sits at row l / 8, 16-byte slot l % 8 and fetches the
    // k-vector that the swizzle (slot = vector ^ ((row >> 1) & 7), row counted inside the tile) puts there.
    const int lr = lane >> 3;
    const unsigned w_offA = (unsigned)(tile_row<EPI>(lr, wdiff) * a.K) * 2u + (unsigned)(((lane & 7) ^ ((lr >> 1) & 7)) * 16);
    const unsigned w_offB = (unsigned)(tile_row<EPI>(8 + lr, wdiff) * a.K) * 2u + (unsigned)(((lane & 7) ^ (((8 + lr) >> 1) & 7)) * 16);
    const int n_buf = min(NBUF, (nk + a.S * NW * D - 1) / (a.S * NW * D)); // groups in the ring (launcher: the same)
    unsigned char *ring = smem + wave * n_buf * GB;
    const unsigned ring0 = (unsigned)(size_t)(CS_LDS_AS unsigned char *)ring;
    const int n_grp = (nkw + D - 1) / D;
    auto issue_w = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int dd = 0; dd < D; ++dd)
            if (g * D + dd < nkw) {                                        // wave-uniform
                const unsigned ko = (unsigned)(kt0 + wave + NW * (g * D + dd)) * 128u;
#pragma unroll
                for (int q = 0; q < CT; ++q) {
                    const unsigned dst = ring0 + (NBUF == 2 ? (g & 1) * GB : 0) + (dd * CT + q) * 2048;
                    dma16_base(wbase[q] + ko, w_offA, dst);
                    dma16_base(wbase[q] + ko, w_offB, dst + 1024);
                }
            }
    };
    // this lane's 16 bytes of a fragment block of activations (rows past M repeat the last one)
    unsigned xoff[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
        xoff[i] = ((unsigned)i * (unsigned)(a.K >> 5) * 64u + (unsigned)(fg * 16 + min(fr, max(M - 1 - 16 * i, 0)))) * 16u;
    int w_frag[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w_frag[ks] = fr * 128 + (((4 * ks + fg) ^ ((fr >> 1) & 7)) << 4);
    f32x4 acc[MB][CT];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int q = 0; q < CT; ++q) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char *xbase = reinterpret_cast<const char *>(a.X) + (size_t)(MB * mi) * (a.K >> 5) * 1024;
    // Activations of group g; k-tiles past the end repeat the last one, their products are skipped.
    auto load_x = [&](int g, bf16x8 (&xf)[D][MB][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int dd = 0; dd < D; ++dd) {
            const char *xb = xbase + (unsigned)(kt0 + wave + NW * min(g * D + dd, nkw - 1)) * 2048u;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                xf[dd][i][0] = *reinterpret_cast<const bf16x8 *>(xb + xoff[i]);
                xf[dd][i][1] = *reinterpret_cast<const bf16x8 *>(xb + xoff[i] + 1024);
            }
        }
    };
    auto multiply = [&](int g, const bf16x8 (&xf)[D][MB][2]) __attribute__((always_inline)) {
        const unsigned char *wg = ring + (NBUF == 2 ? (g & 1) * GB : 0);
#pragma unroll
        for (int dd = 0; dd < D; ++dd) {
            if (g * D + dd < nkw) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int q = 0; q < CT; ++q) {
                        const bf16x8 wf = *reinterpret_cast<const bf16x8 *>(wg + (dd * CT + q) * 2048 + w_frag[ks]);
#pragma unroll
                        for (int i = 0; i < MB; ++i) acc[i][q] = mma16<F16>(wf, xf[dd][i][ks], acc[i][q]);
                    }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");               // the group's slots may be refilled
    };
    // The compiler places the waits for the activations.  It counts its own loads only, not the direct ones, so a use of
    // the group's activations waits until no more memory operations are outstanding than activation loads were issued
    // behind them.  XA groups of activations ahead are as many loads as a group of weights: then that wait never covers the
    // weights that are to stay in flight.
    if constexpr (NBUF == 1 && D == 1 && CT >= 4) {
        // A group's operands go to registers before they are multiplied, so that the next group's weights are on their way meanwhile; its
        // activations follow as the registers of a row block become free.  Whole pass of four layers, graphs, with the wait for the activations behind
        // the next weights and as it is: 1536 / 8960, 96 rows 274.0 -> 271.2 us, 2048 / 11008, 64 rows 362.0 -> 356.5, 4096 / 14336 (two layers), 64 rows 364.5 -> 359.9;
        // gate/up of 96 rows, 1536 / 8960 (55 MB), 19.6 us a launch without any of it, 18.5 now, the reduction in two passes instead of three included.
        bf16x8 xf[MB][2];
        unsigned f16 = (unsigned)fr * 16u;
        auto load_block = [&](int g, int i) __attribute__((always_inline)) {         // (its offset is made here: six of them kept take registers that six
            const unsigned off = (unsigned)fg * 256u + min(f16, (unsigned)max(M - 1 - 16 * i, 0) * 16u);     // row blocks do not have)
            const char *xb = xbase + (size_t)i * (a.K >> 5) * 1024 + (unsigned)(kt0 + wave + NW * g) * 2048u;
            xf[i][0] = *reinterpret_cast<const bf16x8 *>(xb + off);
            xf[i][1] = *reinterpret_cast<const bf16x8 *>(xb + off + 1024);
        };
        if (n_grp > 0) {
#pragma unroll
            for (int i = 0; i < MB; ++i) load_block(0, i);
            issue_w(0);
        }
        for (int g = 0; g < n_grp; ++g) {
            if (g == 0 && want_f) row_factors();
            wait_vm<0>();
            bf16x8 wf[2][CT];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int q = 0; q < CT; ++q) wf[ks][q] = *reinterpret_cast<const bf16x8 *>(ring + q * 2048 + w_frag[ks]);
            // Here the compiler's own waits for the activations belong: it counts those loads only, so behind the next group's direct
            // loads a wait for them would cover these, too.
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    f32x4 x = __builtin_bit_cast(f32x4, xf[i][ks]);
                    asm volatile("" : "+v"(x));
                    xf[i][ks] = __builtin_bit_cast(bf16x8, x);
                }
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f16) : : "memory");
            const bool more = g + 1 < n_grp;                               // wave-uniform
            if (more) issue_w(g + 1);
#pragma unroll
            for (int i = 0; i < MB; ++i) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int q = 0; q < CT; ++q) acc[i][q] = mma16<F16>(wf[ks][q], xf[i][ks], acc[i][q]);
                if (more) load_block(g + 1, i);
            }
        }
    } else if constexpr (NBUF == 1) {
        for (int g = 0; g < n_grp; ++g) {
            bf16x8 xf[D][MB][2];
            load_x(g, xf);
            issue_w(g);
            if (g == 0 && want_f) row_factors();
            wait_vm<0>();
            multiply(g, xf);
        }
    } else if (n_grp > 0) {
        constexpr int XA = (CT + MB - 1) / MB;
        bf16x8 xf[XA + 1][D][MB][2];
#pragma unroll
        for (int u = 0; u < XA; ++u) load_x(u, xf[u]);
        issue_w(0);
        for (int g0 = 0; g0 < n_grp; g0 += XA + 1) {
#pragma unroll
            for (int u = 0; u <= XA; ++u) {
                const int g = g0 + u;
                if (g >= n_grp) break;
                load_x(g + XA, xf[(u + XA) % (XA + 1)]);
                if (g + 1 < n_grp) issue_w(g + 1);
                // issued behind this group's weights: activations, and the next group's weights
                if ((g + 2) * D <= nkw) wait_vm<2 * MB * D + 2 * CT * D>();
                else wait_vm<2 * MB * D>();
                multiply(g, xf[u]);
                if (g == 0 && want_f) row_factors();
            }
        }
    }

    if (n_grp == 0 && want_f) row_factors();                               // a wavefront without k-tiles

    auto epilogue = [&](int ch, int j, f32x4 v) __attribute__((always_inline)) {
        const int row_l = row_of(ch, j), row = r0 + row_l, tt = tile_of(j);
        const bool ok = row_l < M;
        if constexpr (EPI == SK_EPI_RESID) {
            const int N = a.n_ct * 16, col = tt * 16 + 4 * fg;
            v += pre[ch][j];
            if (ok) *reinterpret_cast<f32x4 *>(a.x + (size_t)row * N + col) = v;
            if (a.xg_out) {
                float sq = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                sq += __shfl_xor(sq, 16);
                sq += __shfl_xor(sq, 32);
                const float f = row_f[row_l];
                const float g[4] = {__uint_as_float(gain[j].x << 16), __uint_as_float(gain[j].x & 0xffff0000u), __uint_as_float(gain[j].y << 16),
                                    __uint_as_float(gain[j].y & 0xffff0000u)};
                const float y4[4] = {v[0] * g[0] * f, v[1] * g[1] * f, v[2] * g[2] * f, v[3] * g[3] * f};
                const float top = fmaxf(fmaxf(fabsf(y4[0]), fabsf(y4[1])), fmaxf(fabsf(y4[2]), fabsf(y4[3])));
                if (__builtin_amdgcn_ballot_w64(top > operand_max(a.xg_fmt == 3)) >> fr & 0x0001000100010001ull) sq = -sq;
                if (ok) {
                    const uint2 y = {pack2(y4[0], y4[1], a.xg_fmt), pack2(y4[2], y4[3], a.xg_fmt)};
                    *reinterpret_cast<uint2 *>(reinterpret_cast<bf16 *>(a.xg_out) + frag_index(row, col, N)) = y;
                    if (fg == 0) a.ssq_out[(size_t)row * a.n_ct + tt] = sq;
                }
            }
        } else if constexpr (EPI == SK_EPI_SWIGLU) {
            v *= fabsf(row_f[row_l]);
            const float a0 = v[0] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[0])) * v[2], a1 = v[1] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[1])) * v[3];
            if (ok) *reinterpret_cast<unsigned *>(reinterpret_cast<bf16 *>(a.act) + frag_index(row, tt * 8 + 2 * fg, a.n_ct * 8)) = pack2(a0, a1, a.act_fmt);
        } else {
            v *= fabsf(row_f[row_l]);
            if (!ok) return;
            const RopeArgs &r = a.rope;
            const int head = tt >> 3, o = 8 * (tt & 7) + 2 * fg;
            const bool is_q = head < r.Hq, is_v = head >= r.Hq + r.Hkv;
            const int hh = is_q ? head : is_v ? head - r.Hq - r.Hkv : head - r.Hq;
            const f32x4 p = pre[ch][j];
            if (!is_v) v = f32x4{v[0] * p[0] - v[2] * p[2], v[1] * p[1] - v[3] * p[3], v[2] * p[0] + v[0] * p[2], v[3] * p[1] + v[1] * p[3]};
            const size_t idx = ((size_t)row * (is_q ? r.Hq : r.Hkv) + hh) * 128 + o;
            const unsigned h0 = pack2(v[0], v[1], 1), h1 = pack2(v[2], v[3], 1);
            auto put = [&](void *base, size_t at, unsigned x0, unsigned x1) {
                *reinterpret_cast<unsigned *>(reinterpret_cast<bf16 *>(base) + at) = x0;
                *reinterpret_cast<unsigned *>(reinterpret_cast<bf16 *>(base) + at + 64) = x1;
            };
            put(is_q ? r.q : is_v ? r.v : r.k, idx, h0, h1);
            void *lo = is_q ? r.q_lo : is_v ? r.v_lo : r.k_lo;
            if (lo) put(lo, idx, pack2_lo(v[0], v[1], h0), pack2_lo(v[2], v[3], h1));
            if (!is_q && kvr[ch][j] >= 0)     // the token joins the context: row kv_row % 16 of page kv_row / 16
                put(is_v ? a.v_pages : a.k_pages, (((size_t)(kvr[ch][j] >> 4) * r.Hkv + hh) * 16 + (kvr[ch][j] & 15)) * 128 + o, h0, h1);
        }
    };

    // ---- the wavefronts' products added in wavefront order, RB row blocks at a time, in the registers' own layout
    f32x4 *red = reinterpret_cast<f32x4 *>(smem);                          // [NW][NBK][64]
    f32x4 *plane = a.S > 1 ? reinterpret_cast<f32x4 *>(a.planes) + (size_t)((t * a.ms + mi) * a.S) * (MB * CT * 64) : nullptr;
    lds_barrier();                                                         // every wavefront is done with its ring; row_f is complete
    if constexpr (EPI != SK_EPI_RESID) {
        // Rows whose operand does not hold them: the products once more, every row's operand from its fp32 values (for the
        // other rows of the block the same operand, hence the same result).  Rare, hence cut for few registers: operands
        // straight from memory, addresses of its own.
        bool own = false;
        for (int r = lane; r < 16 * MB; r += 64) own |= row_f[r] < 0.f;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(own) != 0, 0)) {  // the same for every wavefront
            int lane_ = threadIdx.x & 63;
            asm volatile("" : "+v"(lane_));
            const int fr_ = lane_ & 15;
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int q = 0; q < CT; ++q) acc[i][q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int ks = 0; ks < 2 * nkw; ++ks) {
                const int k = 64 * (kt0 + wave + NW * (ks >> 1)) + 32 * (ks & 1) + 8 * (lane_ >> 4);
                const uint4 gv = *reinterpret_cast<const uint4 *>(a.g_next + k);
                const unsigned gw[4] = {gv.x, gv.y, gv.z, gv.w};
                bf16x8 xf[MB];
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const float *xr = a.x + (size_t)(r0 + min(16 * i + fr_, M - 1)) * a.K + k, sc = row_sc[16 * i + fr_];
                    const f32x4 x0 = *reinterpret_cast<const f32x4 *>(xr), x1 = *reinterpret_cast<const f32x4 *>(xr + 4);
                    unsigned y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float xa = e < 2 ? x0[2 * e] : x1[2 * e - 4], xb = e < 2 ? x0[2 * e + 1] : x1[2 * e - 3];
                        y[e] = pack2(xa * __uint_as_float(gw[e] << 16) * sc, xb * __uint_as_float(gw[e] & 0xffff0000u) * sc, F16 ? 3 : 1);
                    }
                    xf[i] = __builtin_bit_cast(bf16x8, make_uint4(y[0], y[1], y[2], y[3]));
                }
#pragma unroll
                for (int q = 0; q < CT; ++q) {
                    int rA, rB;
                    tile_rows<EPI>(t * CT + q, rA, rB);
                    const bf16x8 wf = *reinterpret_cast<const bf16x8 *>(a.W + (size_t)(rA + tile_row<EPI>(fr_, rB - rA)) * a.K + k);
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[i][q] = mma16<F16>(wf, xf[i], acc[i][q]);
                }
            }
        }
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        if (ch > 0) lds_barrier();
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int q = 0; q < CT; ++q) red[(wave * NBK + r * CT + q) * 64 + lane] = acc[ch * RB + r][q];
        lds_barrier();
#pragma unroll
        for (int j = 0; j < EPB; ++j) {
            const int b = wave + NW * j;
            if (b < NBK) {                                                 // wave-uniform
                f32x4 v = red[b * 64 + lane];
#pragma unroll
                for (int w = 1; w < NW; ++w) v += red[(w * NBK + b) * 64 + lane];
                if (a.S == 1) epilogue(ch, j, v);
                else xwg_store4(plane + ((size_t)s * MB * CT + NBK * ch + b) * 64 + lane, v);
            }
        }
    }
    if (a.S > 1) {
        if (!xwg_arrive_last(a.tile_cnt + t * a.ms + mi, a.S, &s_last, tid)) return;
        const XwgLoads planes(plane, (unsigned)(a.S * MB * CT) * 1024u);
        // a pass's blocks at once, four or eight slices of each in flight, added in slice order (a round of loads takes about a microsecond;
        // 96 rows, 8960 x 1536, five slices and two blocks a wavefront: one round instead of four, 17.3 -> 16.4 us with groups of two k-tiles)
        constexpr int IN_FLIGHT = CT >= 3 && EPB <= 2 ? 8 : 4;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            f32x4 v[EPB];
#pragma unroll
            for (int j = 0; j < EPB; ++j) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int sp = 0; sp < a.S; sp += IN_FLIGHT) {
                f32x4 pv[EPB][IN_FLIGHT];
#pragma unroll
                for (int j = 0; j < EPB; ++j)
#pragma unroll
                    for (int q = 0; q < IN_FLIGHT; ++q)
                        pv[j][q] = planes.load4((unsigned)(min(sp + q, a.S - 1) * MB * CT + NBK * ch + min(wave + NW * j, NBK - 1)) * 1024u + lane * 16u);
#pragma unroll
                for (int j = 0; j < EPB; ++j)
#pragma unroll
                    for (int q = 0; q < IN_FLIGHT; ++q)
                        if (sp + q < a.S) v[j] += pv[j][q];
            }
#pragma unroll
            for (int j = 0; j < EPB; ++j)
                if (wave + NW * j < NBK) epilogue(ch, j, v[j]);
        }
    }
}

// Tiling of a projection: blocks of 16 rows per workgroup (mb) and workgroups over the rows (ms), 16-column tiles per
// workgroup (ct), k slices (S).  Times are of single launches over weights that come from HBM, MI355X; those inside a pass differ by up to a
// microsecond.
//  - Wide outputs (gate/up).  One row block: one tile per workgroup, the weights' stream decides (55 MB: 11.7 us).  More
//    rows: the activations, which every workgroup re-reads from the L2, would cost as much as the weights, so a workgroup
//    takes as many tiles as leave about one workgroup per CU (1120 tiles: 5; 32 rows 16.2 -> 12.9 us, 96 rows 25 -> 18.5 us).
//  - Narrow outputs over a k range of fewer than 128 k-tiles: one tile, never cut (a hand-over between slices - store,
//    counter and load at the memory side - is about 3 us); several row blocks are halved over two workgroups, which share
//    the weights through their L2 (96 rows x 2048 columns x 1536: 9.0 -> 6.5 us).  From 256 tiles on two tiles.
//  - Narrow outputs over long k ranges (down): cut so that about one workgroup per CU (about two where there are enough
//    tiles) shares the work; more rows take more tiles per workgroup, again for the activations (8960 x 1536: 9.9 us for one
//    row, 11.5 for 32, 16.4 for 96).
//  - A width made for the other kind of projection (a wide model's QKV or residual projection of 1024 tiles and more, a small
//    model's gate/up): one tile, never cut.  Rotating projections over 128 k-tiles and more: never cut either, one tile, two
//    from 128 tiles on.
SkinnyPlan skinny_plan(int epi, int M, int K, int n_ct) {
    SkinnyPlan p;
    const int b = (M + 15) / 16, nk = K / 64;
    p.ct = 1;
    p.S = 1;
    p.ms = b > 4 ? 2 : 1;
    if ((epi == SK_EPI_SWIGLU) != (n_ct >= 1024)) {
    } else if (epi == SK_EPI_SWIGLU) {
        p.ct = b == 1 ? 1 : n_ct % 5 == 0 && n_ct / 5 <= 256 ? 5 : n_ct % 4 == 0 ? 4 : 1;
        if (p.ct == 5) p.ms = b > 6 ? 2 : 1;
    } else if (nk < 128) {
        p.ct = n_ct >= 256 && n_ct % 2 == 0 ? 2 : 1;
        p.ms = b > (p.ct == 2 ? 2 : 1) ? 2 : 1;
    } else if (n_ct >= 128 || epi == SK_EPI_ROPE) {
        p.ct = n_ct >= 128 && n_ct % 2 == 0 ? 2 : 1;
    } else {
        p.ct = b == 1 ? 1 : b <= 4 ? (n_ct % 3 == 0 ? 3 : 1) : n_ct % 4 == 0 ? 4 : 1;
    }
    p.mb = (b + p.ms - 1) / p.ms;
    if (p.mb == 5) p.mb = 6;
    const int wgs = n_ct / p.ct * p.ms;
    if (epi == SK_EPI_RESID && n_ct < 1024 && nk >= 128 && wgs <= SK_MAX_TILES_CUT)
        p.S = std::max(1, std::min((wgs >= 128 ? 480 : b == 1 ? 208 : 256) / wgs, nk / 8));
    return p;
}
// Tilings there are kernels for (what skinny_plan may return).
constexpr bool has_kernel(int epi, int mb, int ct) {
    if (mb == 6) return epi == SK_EPI_SWIGLU && ct == 5;
    if (mb < 1 || mb > 4) return false;
    return epi == SK_EPI_SWIGLU ? ct == 1 || ct == 4 || ct == 5 : epi == SK_EPI_RESID ? ct >= 1 && ct <= 4 : ct == 1 || ct == 2;
}
bool skinny_has_kernel(int epi, const SkinnyPlan &p) { return has_kernel(epi, p.mb, p.ct); }
size_t skinny_plane_bytes(int epi, int M, int K, int n_ct) {      // the largest over all row counts up to M
    size_t best = 0;
    for (int b = 1; b <= (M + 15) / 16; ++b) {
        const SkinnyPlan p = skinny_plan(epi, 16 * b, K, n_ct);
        if (p.S > 1) best = std::max(best, (size_t)p.S * 16 * p.mb * p.ms * 16 * n_ct * 4);
    }
    return best;
}

template <int EPI, bool F16, int MB, int CT, int NW, int D, int NBUF = 2>
static hipError_t launch_one(const SkinnyGemm &a, hipStream_t s) {
    static std::atomic<uint32_t> attr_done{0};
    auto kern = skinny_kernel<EPI, F16, MB, CT, NW, D, NBUF>;
    constexpr int group = NW * D * CT * 2048, red = NW * skinny_rb(MB, CT, NW) * CT * 1024;
    if (hipError_t e = set_dynamic_lds_once(attr_done, reinterpret_cast<const void *>(kern), std::max(NBUF * group, red)); e != hipSuccess) return e;
    const int n_buf = std::min(NBUF, (a.K / 64 + a.S * NW * D - 1) / (a.S * NW * D));
    const int tiles = a.S * (a.n_ct / CT);
    kern<<<(tiles + 7) / 8 * 8 * a.ms, 64 * NW, std::max(n_buf * group, red), s>>>(a);
    return hipGetLastError();
}

template <int EPI, bool F16, int MB, int CT>
static hipError_t launch_ct(const SkinnyGemm &a, hipStream_t s) {
    constexpr int D2 = MB < 4 ? 2 : 1;                   // (two groups of more activations than this do not fit the registers)
    if constexpr (!has_kernel(EPI, MB, CT)) {
        return hipErrorInvalidValue;
    } else if constexpr (CT >= 3) {
        if constexpr (EPI == SK_EPI_RESID && CT == 4) return launch_one<EPI, F16, MB, CT, 8, 2, 1>(a, s);
        else return launch_one<EPI, F16, MB, CT, 8, 1, 1>(a, s);
    } else if constexpr (CT == 2) {
        return launch_one<EPI, F16, MB, CT, 8, D2>(a, s);
    } else {
        if (a.K <= 64 * 24) return launch_one<EPI, F16, MB, 1, 8, 3, 1>(a, s);       // a wavefront's whole share of the k range at once
        if constexpr (EPI == SK_EPI_RESID && MB < 3)
            if (a.S > 1) return launch_one<EPI, F16, MB, 1, 8, 3>(a, s);
        return launch_one<EPI, F16, MB, 1, 8, D2>(a, s);
    }
}
template <int EPI, bool F16, int MB>
static hipError_t launch_mb(const SkinnyGemm &a, const SkinnyPlan &p, hipStream_t s) {
    switch (p.ct) {
        case 1: return launch_ct<EPI, F16, MB, 1>(a, s);
        case 2: return launch_ct<EPI, F16, MB, 2>(a, s);
        case 3: return launch_ct<EPI, F16, MB, 3>(a, s);
        case 4: return launch_ct<EPI, F16, MB, 4>(a, s);
        case 5: return launch_ct<EPI, F16, MB, 5>(a, s);
    }
    return hipErrorInvalidValue;
}
template <int EPI, bool F16>
static hipError_t launch_epi(const SkinnyGemm &a, const SkinnyPlan &p, hipStream_t s) {
    switch (p.mb) {
        case 1: return launch_mb<EPI, F16, 1>(a, p, s);
        case 2: return launch_mb<EPI, F16, 2>(a, p, s);
        case 3: return launch_mb<EPI, F16, 3>(a, p, s);
        case 4: return launch_mb<EPI, F16, 4>(a, p, s);
        case 6: return launch_mb<EPI, F16, 6>(a, p, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_skinny(SkinnyGemm a, int epi, bool f16, hipStream_t s) {
    if (a.M < 1 || a.M > SK_MAX_ROWS || a.K % 64 != 0 || a.K < 64 || a.n_ct < 1 || !a.X || !a.W) return hipErrorInvalidValue;
    const SkinnyPlan p = skinny_plan(epi, a.M, a.K, a.n_ct);
    if (p.S > 1 && (!a.planes || !a.tile_cnt)) return hipErrorInvalidValue;
    if ((epi != SK_EPI_RESID || a.xg_out) && (!a.ssq_in || a.ssq_n < 1)) return hipErrorInvalidValue;
    a.S = p.S;
    a.ms = p.ms;
    switch (epi) {
        case SK_EPI_ROPE: return f16 ? launch_epi<SK_EPI_ROPE, true>(a, p, s) : launch_epi<SK_EPI_ROPE, false>(a, p, s);
        case SK_EPI_RESID: return f16 ? launch_epi<SK_EPI_RESID, true>(a, p, s) : launch_epi<SK_EPI_RESID, false>(a, p, s);
        case SK_EPI_SWIGLU: return f16 ? launch_epi<SK_EPI_SWIGLU, true>(a, p, s) : launch_epi<SK_EPI_SWIGLU, false>(a, p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace cs
