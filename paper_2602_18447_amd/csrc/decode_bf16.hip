// Kernel of a generation step (Algorithm 1: the generate calls of Stage 1 and of the Stage 3 fallback), one new token
// per trace, beside the projections (skinny_bf16.hip) and the attention (attn_few.hip): the language-model head, a stream
// of its weights from HBM, built around keeping that stream going and touching it once.
#include "kernels.h"
#include <algorithm>

namespace cs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define CS_LDS_AS __attribute__((address_space(3)))

namespace {

constexpr int DEC_THREADS = 512, DEC_WAVES = 8;
constexpr int DEC_KW = 3;                    // k-tiles a wavefront owns at most (24 / 8 wavefronts)
constexpr int DEC_XT = 4096;                 // one activation k-tile: 32 rows x 128 bytes = two ring slots
constexpr int DEC_WT = 2048;                 // one weight k-tile: 16 rows x 128 bytes = one ring slot
constexpr int DEC_RED = DEC_WAVES * 32 * 16 * 4;           // 16 KiB: the 8 partial products of a column tile
constexpr int DEC_NSLOT = 8;                               // weight slots of a wavefront: 16 KiB in flight
constexpr int DEC_RING = DEC_WAVES * DEC_NSLOT * DEC_WT;
static_assert(DEC_MAX_KT == DEC_KW * DEC_WAVES && 2 * DEC_KW <= DEC_NSLOT - 2, "activation k-tiles are staged in the ring");

__device__ inline f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 64 lanes x 16 bytes from per-lane global addresses into LDS at lds_dst + 16 * lane (lds_dst wave-uniform).  Issued
// from inline assembly with a memory clobber: the compiler neither reorders LDS accesses across it nor waits for it;
// completion is waited for explicitly with dec_wait_vm.
__device__ inline void dma16(const void *src, unsigned lds_dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_dst), "v"(src) : "memory");
}
// at most n vector memory operations of this wavefront still outstanding (they complete in issue order)
template <int N>
__device__ inline void dec_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ inline void dec_wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

}  // namespace

// ---- language-model head --------------------------------------------------------------------------------------------
// Running (max, first index of the max, sum of exp(z - max)) of a row of logits.
struct DecHeadAcc {
    float m;
    int idx;
    float s;
};
__device__ inline DecHeadAcc dec_head_merge(DecHeadAcc a, DecHeadAcc b) {   // lowest index on equal maxima
    DecHeadAcc r;
    const bool a_first = a.m > b.m || (a.m == b.m && a.idx < b.idx);
    r.m = a_first ? a.m : b.m;
    r.idx = a_first ? a.idx : b.idx;
    r.s = (a.m == -INFINITY ? 0.f : a.s * __expf(a.m - r.m)) + (b.m == -INFINITY ? 0.f : b.s * __expf(b.m - r.m));
    return r;
}

// The language-model head at one position per trace: logits of 16-column tiles of the vocabulary, reduced on the spot.
// A workgroup of 8 wavefronts walks the tiles j, j + nwg, ...; wavefront w owns the k-tiles w, w + 8, w + 16 (at most
// three): it keeps their activations (32 rows, two bf16 terms) in registers as MFMA operands and streams the matching
// weight k-tiles (16 rows x 128 bytes) through a private ring of LDS slots filled by direct global -> LDS loads, so the
// main loop has no workgroup barrier and 16 KiB per wavefront stay in flight across tile borders.  Per tile the 8 partial
// 32 x 16 products are added in wavefront order through LDS; a thread keeps the running (max, first index of the max,
// sum of exponentials) of its columns, so the [M, vocab] logits are never written.
__global__ __launch_bounds__(DEC_THREADS) void dec_head_kernel(DecHead a) {
    constexpr int NSLOT = DEC_NSLOT, SLOT0 = 2 * DEC_KW;                // slot of unit 0
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = blockIdx.x;
    const int nk = a.K >> 6;
    const int nkw = nk > wave ? (nk - wave + DEC_WAVES - 1) / DEC_WAVES : 0;     // k-tiles of this wavefront (<= 3)
    const int n_my = (a.n_ct - j + a.nwg - 1) / a.nwg;                  // column tiles j, j + nwg, ...
    const int total = n_my * nkw;                                       // (tile, k-tile) units of this wavefront
    unsigned char *ring = smem + wave * NSLOT * DEC_WT;                 // this wavefront's slots
    float *red = reinterpret_cast<float *>(smem + DEC_RING);
    const unsigned ring0 = (unsigned)(size_t)(CS_LDS_AS unsigned char *)ring;

    // Direct-load roles: one instruction fills 8 rows x 128 bytes; lane l sits at row l / 8, 16-byte slot l % 8 and
    // fetches the k-vector that the swizzle (slot = vector ^ ((row >> 1) & 7), row counted inside the tile) puts there.
    const int lr = lane >> 3, lslot = lane & 7;
    // Unit u = (column tile u / nkw, the wavefront's k-tile u % nkw) goes through slot (SLOT0 + u) % NSLOT.
    auto issue_unit = [&](int u) {
        int ti = u / nkw, i = u - ti * nkw;
        int t = j + ti * a.nwg, kt = wave + DEC_WAVES * i;
        unsigned dst = ring0 + ((u + SLOT0) % NSLOT) * DEC_WT;
        int vecA = lslot ^ ((lr >> 1) & 7), vecB = lslot ^ (((8 + lr) >> 1) & 7);
        dma16(a.W + (size_t)(16 * t + lr) * a.K + (size_t)kt * 64 + vecA * 8, dst);
        dma16(a.W + (size_t)(16 * t + 8 + lr) * a.K + (size_t)kt * 64 + vecB * 8, dst + 1024);
    };
    // activation k-tile i of this wavefront (term: 0 = hi, 1 = lo half of a two-term row) to LDS address dst
    auto issue_x = [&](int i, int term, unsigned dst) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            int row = 8 * r4 + lr;
            int vec = lslot ^ ((row >> 1) & 7);
            const bf16 *src = a.X + (size_t)min(row, a.M - 1) * 2 * a.K + (size_t)term * a.K +
                              (size_t)(wave + DEC_WAVES * i) * 64 + vec * 8;            // rows past M repeat the last row
            dma16(src, dst + r4 * 1024);
        }
    };
    // fragment addresses: 16 x 16 x 32 MFMA, lane l supplies row l % 16 and the k-vector l / 16 of a 32-wide k-step
    const int fr = lane & 15, fg = lane >> 4;
    int w_off[2], x_off[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        w_off[ks] = fr * 128 + (((4 * ks + fg) ^ ((fr >> 1) & 7)) << 4);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            int row = 16 * rb + fr;
            x_off[ks][rb] = row * 128 + (((4 * ks + fg) ^ ((row >> 1) & 7)) << 4);
        }
    }
    bf16x8 xf[2][DEC_KW][2][2];
    // the activations go through slots 0..5 into registers, once per term; the first two weight units are on their way
    // in slots 6, 7
#pragma unroll
    for (int term = 0; term < 2; ++term) {
#pragma unroll
        for (int i = 0; i < DEC_KW; ++i)
            if (i < nkw) issue_x(i, term, ring0 + i * DEC_XT);
        if (term == 0) {
            if (0 < total) issue_unit(0);
            if (1 < total) issue_unit(1);
        }
        // the staged k-tiles were issued before the weight units of this term (if any): they land first
        if (term == 0 && total >= 2) dec_wait_vm<4>();
        else if (term == 0 && total == 1) dec_wait_vm<2>();
        else dec_wait_vm<0>();
#pragma unroll
        for (int i = 0; i < DEC_KW; ++i)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
                    xf[term][i][ks][rb] = i < nkw ? *reinterpret_cast<const bf16x8 *>(ring + i * DEC_XT + x_off[ks][rb]) : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        dec_wait_lds();
    }
#pragma unroll
    for (int u = 2; u < NSLOT; ++u)
        if (u < total) issue_unit(u);

    const int row = tid >> 4, c = tid & 15;                             // this thread's element of a 32 x 16 tile
    DecHeadAcc hacc = {-INFINITY, 0x7fffffff, 0.f};                     // this thread's columns so far
    int u = 0;
    for (int ti = 0; ti < n_my; ++ti) {
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int i = 0; i < DEC_KW; ++i) {
            if (i < nkw) {
                const int after = min(NSLOT - 1, total - 1 - u);        // units issued after this one
                switch (after) {
                    case 7: dec_wait_vm<14>(); break;
                    case 6: dec_wait_vm<12>(); break;
                    case 5: dec_wait_vm<10>(); break;
                    case 4: dec_wait_vm<8>(); break;
                    case 3: dec_wait_vm<6>(); break;
                    case 2: dec_wait_vm<4>(); break;
                    case 1: dec_wait_vm<2>(); break;
                    default: dec_wait_vm<0>(); break;
                }
                const unsigned char *wsl = ring + ((u + SLOT0) % NSLOT) * DEC_WT;
                bf16x8 wf[2];
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) wf[ks] = *reinterpret_cast<const bf16x8 *>(wsl + w_off[ks]);
                dec_wait_lds();                                         // the slot is in registers: refill it
                if (u + NSLOT < total) issue_unit(u + NSLOT);
#pragma unroll
                for (int term = 0; term < 2; ++term)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        acc[0] = mma16(xf[term][i][ks][0], wf[ks], acc[0]);
                        acc[1] = mma16(xf[term][i][ks][1], wf[ks], acc[1]);
                    }
                ++u;
            }
        }
        // accumulator layout: column lane % 16, rows 16 rb + 4 (lane / 16) + e
        float *mine = red + wave * 512;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) mine[(16 * rb + 4 * fg + e) * 16 + fr] = acc[rb][e];
        __syncthreads();
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) v += red[w * 512 + tid];   // wavefront order: fixed
        __syncthreads();                                                // red is free for the next tile
        // logit of (row, vocabulary entry 16 t + c) into the thread's running statistics (its entries ascend)
        if (v > hacc.m) {
            hacc.s = (hacc.m == -INFINITY ? 0.f : hacc.s * __expf(hacc.m - v)) + 1.0f;
            hacc.m = v;
            hacc.idx = 16 * (j + ti * a.nwg) + c;
        } else {
            hacc.s += __expf(v - hacc.m);
        }
    }
    // the 16 threads of a row, then one record per (workgroup, row) for the kernel that finishes the rows
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        DecHeadAcc o = {__shfl_xor(hacc.m, off), __shfl_xor(hacc.idx, off), __shfl_xor(hacc.s, off)};
        hacc = dec_head_merge(hacc, o);
    }
    if (c == 0) {
        float *rec = a.part + ((size_t)j * DEC_MAX_ROWS + row) * 4;
        rec[0] = hacc.m;
        rec[1] = __int_as_float(hacc.idx);
        rec[2] = hacc.s;
    }
}

hipError_t launch_dec_head(const DecHead &a, hipStream_t s) {
    if (a.M < 1 || a.M > DEC_MAX_ROWS || a.K % 64 != 0 || a.K > 64 * DEC_MAX_KT || a.nwg < 1 || a.nwg > 256 || a.n_ct < a.nwg || !a.X || !a.part)
        return hipErrorInvalidValue;
    static std::atomic<uint32_t> attr_done{0};
    constexpr int smem = DEC_RING + DEC_RED;
    if (hipError_t e = set_dynamic_lds_once(attr_done, reinterpret_cast<const void *>(dec_head_kernel), smem); e != hipSuccess) return e;
    dec_head_kernel<<<a.nwg, DEC_THREADS, smem, s>>>(a);
    return hipGetLastError();
}

// The rows of the language-model head: the records of all workgroups of dec_head_kernel merged in
// workgroup order per row (one wavefront per row).
__global__ __launch_bounds__(64) void dec_head_final_kernel(const float *__restrict__ part, int nwg, const float *__restrict__ verdict_logits,
                                                             int n_verdict, int32_t *__restrict__ token, float *__restrict__ max_logit,
                                                             float *__restrict__ lse, float *__restrict__ conf_full) {
    const int b = blockIdx.x, lane = threadIdx.x;
    DecHeadAcc acc = {-INFINITY, 0x7fffffff, 0.f};
    for (int g = lane; g < nwg; g += 64) {
        const float *rec = part + ((size_t)g * DEC_MAX_ROWS + b) * 4;
        acc = dec_head_merge(acc, DecHeadAcc{rec[0], __float_as_int(rec[1]), rec[2]});
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        DecHeadAcc o = {__shfl_xor(acc.m, off), __shfl_xor(acc.idx, off), __shfl_xor(acc.s, off)};
        acc = dec_head_merge(acc, o);
    }
    if (lane == 0) {
        float l = acc.m + logf(acc.s);
        token[b] = acc.idx;
        max_logit[b] = acc.m;
        lse[b] = l;
        if (conf_full && verdict_logits) {
            float zv = verdict_logits[(size_t)b * n_verdict];
            for (int v = 1; v < n_verdict; ++v) zv = fmaxf(zv, verdict_logits[(size_t)b * n_verdict + v]);
            conf_full[b] = expf(zv - l);
        }
    }
}

hipError_t launch_dec_head_final(const float *part, int nwg, int B, const float *verdict_logits, int n_verdict, int32_t *token,
                                 float *max_logit, float *lse, float *conf_full, hipStream_t s) {
    dec_head_final_kernel<<<B, 64, 0, s>>>(part, nwg, verdict_logits, n_verdict, token, max_logit, lse, conf_full);
    return hipGetLastError();
}

}  // namespace cs
