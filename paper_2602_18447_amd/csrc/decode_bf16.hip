// Kernels of a generation step (Algorithm 1: the generate calls of Stage 1 and of the Stage 3 fallback), one new token
// per trace, beside the projections (skinny_bf16.hip): attention with one query row per head, and the language-model
// head.  Both are streams from HBM - cached keys / values, the head's weights - and are built around keeping that
// stream going and touching it once.
#include "kernels.h"
#include "xwg.h"
#include <algorithm>

namespace cs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(8))) short i16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

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

__device__ inline unsigned short to_fmt(float v, int fmt) {   // fmt 3: IEEE half (saturating), else bf16
    return fmt == 3 ? __half_as_ushort(to_half_sat(v)) : __bfloat16_as_ushort(__float2bfloat16(v));
}

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

// The rows of the language-model head: the records of all workgroups of dec_gemm_kernel<DEC_EPI_HEAD> merged in
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

// ---- attention ------------------------------------------------------------------------------------------------------
// One workgroup per (trace, kv head, piece of n_iter x 256 cached keys); in each round of 256 keys wavefront w takes PAGES
// 16-token pages and keeps a running (max, sum, O) over its rounds.  Keys go straight from global memory into the
// registers of the score product's first operand (lane l: token l % 16 of a page, head-dim elements 32 ks + 8 (l / 16) ..
// + 7), values go global -> LDS (rows of 256 bytes) and come back through transposing reads as the first operand of
// O^T += V^T . P^T.  The 16-byte vector v of token k sits at slot v ^ (2 (k & 7)) of its row, so that the 32 bytes x 8
// consecutive tokens that half a wavefront reads at a time fall into different banks; the lane that fills a slot
// fetches the matching global vector.
// Transposing reads (ds_read_b64_tr_b16): in a group of 16 lanes, lane i supplies the address of 4 consecutive 16-bit
// elements and receives element i % 4 of what lanes i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4 addressed.
// The new token is not part of the pieces: the first wavefront of the last piece adds it to its state.
//
// What bounds it: few (trace, kv head) pairs, the chain of round trips in a workgroup - page ids, keys and values, the
// arrival counter, the other pieces' results: the page ids are asked for before the length is known, and the last
// workgroup's wavefronts merge the pieces side by side as they merged their own results.  One trace, 4096 keys: 14.7 us
// when the pieces were merged one after the other by every thread.  Many pairs: the stream of keys and values (32 traces x 2
// heads x 2048 keys, 67 MB), for which two workgroups of four wavefronts share a CU with 128 KiB each in flight.
constexpr int DEC_ATTN_SMEM = 65536;

// The wavefronts' results [row][128] (om, stride floats per wavefront) and (max, sum) at om[1024 + row], om[1040 + row]
// merged for (row, columns 4 c4 .. + 3), in wavefront order.
template <int NW>
__device__ __forceinline__ f32x4 dec_combine(const float *om, int stride, int row, int c4, float &M, float &l) {
    float mw[NW];
    M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mw[w] = om[w * stride + 1024 + row];
        M = fmaxf(M, mw[w]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float wgt = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - M);
        const f32x4 o = *reinterpret_cast<const f32x4 *>(om + w * stride + row * 128 + 4 * c4);
        if (mw[w] != -INFINITY) {                        // a wavefront without keys left nothing
            acc += wgt * o;
            l += wgt * om[w * stride + 1040 + row];
        }
    }
    return acc;
}

template <int NW, int PAGES>
__global__ __launch_bounds__(64 * NW, 2) void dec_attn_kernel(DecAttn a) {
    static_assert(NW * PAGES * 16 == DEC_PIECE && NW * PAGES * 4096 == DEC_ATTN_SMEM && PAGES % 2 == 0, "256 keys a round");
    constexpr int WLDS = PAGES * 4096;                   // a wavefront's values, later its results
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ volatile int s_last;
    asm volatile("" : : "s"(a.q), "s"(a.q_lo), "s"(a.ksuf), "s"(a.vsuf), "s"(a.k_pages), "s"(a.v_pages), "s"(a.table), "s"(a.plens), "s"(a.out),
                 "s"(a.part_o), "s"(a.part_ml), "s"(a.max_pieces), "s"(a.n_iter));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid: x = (piece, kv head), pieces from the last one of the longest trace down; y = trace
    const int h = blockIdx.x % a.Hkv, b = blockIdx.y;
    const int p = a.max_pieces - 1 - blockIdx.x / a.Hkv;
    const int piece_keys = DEC_PIECE * a.n_iter;
    const int32_t *bt = a.table + (size_t)b * a.max_blocks;
    int entry[PAGES];                                                   // page ids of the first round
#pragma unroll
    for (int i = 0; i < PAGES; ++i) entry[i] = bt[min((piece_keys >> 4) * p + wave * PAGES + i, a.max_blocks - 1)];
    const int L = min(max(a.plens[b], 0), a.max_L);                     // cached keys; the new token sees all of them and itself
    const int n_p = max((L + piece_keys - 1) / piece_keys, 1);          // pieces of this trace
    if (p >= n_p) return;                                               // uniform: a shorter trace
    const int G = a.G;
    unsigned char *vst = smem + wave * WLDS;
    const unsigned lds_v = (unsigned)(size_t)(CS_LDS_AS unsigned char *)vst;
    const int fr = lane & 15, fg = lane >> 4;
    const bf16 *ks_row = a.ksuf + ((size_t)b * a.Hkv + h) * 128, *vs_row = a.vsuf + ((size_t)b * a.Hkv + h) * 128;
    // q operand: lane l holds query row l % 16 (rows >= G repeat the last one; they are never stored), head-dim elements
    // 32 ks + 8 (l / 16) .. + 7
    bf16x8 q_hi[4], q_lo[4];
    const size_t qo = ((size_t)b * a.Hq + (size_t)h * G + min(fr, G - 1)) * 128 + 8 * fg;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        q_hi[ks] = *reinterpret_cast<const bf16x8 *>(a.q + qo + 32 * ks);
        q_lo[ks] = *reinterpret_cast<const bf16x8 *>(a.q_lo + qo + 32 * ks);
    }
    float m_w = -INFINITY, l_w = 0.f;                                   // running maximum (log2 units) and sum of this wavefront
    f32x4 o_acc[8];
#pragma unroll
    for (int hb = 0; hb < 8; ++hb) o_acc[hb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < a.n_iter; ++it) {
        const int key0 = piece_keys * p + DEC_PIECE * it + 16 * PAGES * wave;   // this wavefront's keys of this round
        if (key0 >= L) break;                                           // wave-uniform; later rounds lie further out
        if (it > 0) {
#pragma unroll
            for (int i = 0; i < PAGES; ++i) entry[i] = bt[min((key0 >> 4) + i, a.max_blocks - 1)];
        }
        const int lrow = lane >> 4, lslot = lane & 15;
        // tokens at or past L are masked; what is fetched for them is the new token's row, so that page rows that were
        // never written are not read
        bf16x8 kf[PAGES][4];
#pragma unroll
        for (int kb = 0; kb < PAGES; ++kb) {
            const int tok0 = key0 + 16 * kb;
            const int id = tok0 < L ? min(max(entry[kb], 0), a.n_blocks - 1) : 0;
            const size_t page = ((size_t)id * a.Hkv + h) * 16 * 128;
            // values: instruction jj fills tokens 4 jj .. 4 jj + 3 of the page; lane l: token 4 jj + l / 16, slot l % 16
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int kl = 4 * jj + lrow;
                const int vvec = lslot ^ (2 * (kl & 7));
                dma16(tok0 + kl < L ? a.v_pages + page + kl * 128 + vvec * 8 : vs_row + vvec * 8, lds_v + kb * 4096 + jj * 1024);
            }
            // keys: token fr of the page, 16 bytes per k-step
            const bf16 *krow = tok0 + fr < L ? a.k_pages + page + fr * 128 : ks_row;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kf[kb][ks] = *reinterpret_cast<const bf16x8 *>(krow + 32 * ks + 8 * fg);
        }
        // scores: S^T[token][query row]; lane l ends up with query row l % 16, tokens 4 (l / 16) + e of each page
        f32x4 sc[PAGES];
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < PAGES; ++kb) {
            sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                sc[kb] = mma16(kf[kb][ks], q_hi[ks], sc[kb]);
                sc[kb] = mma16(kf[kb][ks], q_lo[ks], sc[kb]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = (key0 + 16 * kb + 4 * fg + e < L) ? sc[kb][e] * a.scale_log2 : -INFINITY;
                sc[kb][e] = v;
                mx = fmaxf(mx, v);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // running maximum: finite from the first round on (token key0 < L is visible to every query row)
        const float m_new = fmaxf(m_w, mx);
        const float alpha = m_w == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_w - m_new);
        m_w = m_new;
        float ps = 0.f;
#pragma unroll
        for (int kb = 0; kb < PAGES; ++kb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[kb][e] = __builtin_amdgcn_exp2f(sc[kb][e] - m_new);
                ps += sc[kb][e];
            }
        ps += __shfl_xor(ps, 16);
        ps += __shfl_xor(ps, 32);
        l_w = l_w * alpha + ps;
        if (it > 0) {
#pragma unroll
            for (int hb = 0; hb < 8; ++hb) o_acc[hb] *= alpha;
        }
        dec_wait_vm<0>();                                // the values have landed
        // probabilities as the second operand of O^T += V^T . P^T over two pages: k index 8 (l / 16) + i <-> token
        // 4 (l / 16) + i of the first page (i < 4) or the second (i >= 4), which is what the lane already holds; two bf16
        // terms.  V^T operand: group l / 16 reads tokens 4 (l / 16) .. + 3 of a page; lane i of the group points at token
        // i / 4, head-dim elements 16 hb + 4 (i % 4) .. + 3 and receives the four tokens of element 16 hb + i
        const int vrow = 4 * fg + (fr >> 2), q4 = fr & 3;
#pragma unroll
        for (int pp = 0; pp < PAGES / 2; ++pp) {
            bf16x8 p_hi, p_lo;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float pr = sc[2 * pp + (i >> 2)][i & 3];
                __bf16 hi = (__bf16)pr;
                p_hi[i] = hi;
                p_lo[i] = (__bf16)(pr - (float)hi);
            }
#pragma unroll
            for (int hb = 0; hb < 8; ++hb) {
                const unsigned char *p0 = vst + pp * 8192 + vrow * 256 + (((2 * hb + (q4 >> 1)) ^ (2 * (vrow & 7))) << 4) + ((q4 & 1) << 3);
                i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CS_LDS_AS i16x4 *)p0);
                i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CS_LDS_AS i16x4 *)(p0 + 4096));
                bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                o_acc[hb] = mma16(vf, p_hi, o_acc[hb]);
                o_acc[hb] = mma16(vf, p_lo, o_acc[hb]);
            }
        }
        dec_wait_lds();                                  // the value region may be refilled (or reused below)
    }
    if (p == n_p - 1 && wave == 0) {                     // the new token
        f32x4 sn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {                 // (its key in all 16 rows of the operand)
            const bf16x8 kn = *reinterpret_cast<const bf16x8 *>(ks_row + 32 * ks + 8 * fg);
            sn = mma16(kn, q_hi[ks], sn);
            sn = mma16(kn, q_lo[ks], sn);
        }
        const float v = sn[0] * a.scale_log2, m_new = fmaxf(m_w, v);
        const float alpha = m_w == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_w - m_new), pr = __builtin_amdgcn_exp2f(v - m_new);
        m_w = m_new;
        l_w = l_w * alpha + pr;
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            const uint2 vn = *reinterpret_cast<const uint2 *>(vs_row + 16 * hb + 4 * fg);
            const f32x4 vf = {__uint_as_float(vn.x << 16), __uint_as_float(vn.x & 0xffff0000u), __uint_as_float(vn.y << 16), __uint_as_float(vn.y & 0xffff0000u)};
            o_acc[hb] = o_acc[hb] * alpha + pr * vf;
        }
    }
    // ---- the wavefronts' results, each in its own value region, combined in wavefront order
    constexpr int OM = WLDS / 4;
    float *om = reinterpret_cast<float *>(vst);
    if (m_w != -INFINITY && fr < G) {
#pragma unroll
        for (int hb = 0; hb < 8; ++hb)
            *reinterpret_cast<f32x4 *>(om + fr * 128 + 16 * hb + 4 * fg) = o_acc[hb];   // rows 16 hb + 4 (l / 16) + e
    }
    if (fg == 0 && fr < DEC_MAX_G) {
        om[1024 + fr] = m_w;
        om[1040 + fr] = l_w;
    }
    auto lds_barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); };
    lds_barrier();
    const float *all = reinterpret_cast<const float *>(smem);
    const int row = tid >> 5, c4 = tid & 31;                            // this thread's part of the result (row < G)
    auto store_out = [&](f32x4 acc, float l) {
        const float inv = 1.0f / l;
        unsigned short *o = reinterpret_cast<unsigned short *>(a.out) + frag_index(b, (h * G + row) * 128 + 4 * c4, a.Hq * 128);
        ushort4 v = {to_fmt(acc[0] * inv, a.out_fmt), to_fmt(acc[1] * inv, a.out_fmt), to_fmt(acc[2] * inv, a.out_fmt), to_fmt(acc[3] * inv, a.out_fmt)};
        *reinterpret_cast<ushort4 *>(o) = v;
    };
    const size_t item0 = (size_t)b * a.max_pieces * a.Hkv + h;          // piece p: item0 + p Hkv
    if (row < G) {
        float M, l;
        const f32x4 acc = dec_combine<NW>(all, OM, row, c4, M, l);
        if (n_p == 1) {
            store_out(acc, l);
        } else {
            const size_t at = (item0 + (size_t)p * a.Hkv) * DEC_MAX_G + row;
            xwg_store4(reinterpret_cast<f32x4 *>(a.part_o + at * 128) + c4, acc);
            if (c4 == 0) {
                xwg_store(a.part_ml + at * 2, M);
                xwg_store(a.part_ml + at * 2 + 1, l);
            }
        }
    }
    if (n_p == 1) return;
    // ---- the pieces of this (trace, kv head): the last workgroup to arrive merges them.  Wavefront w takes the pieces w,
    // w + NW, ... in turn; a lane has columns 4 (lane % 32) .. + 3 of the rows lane / 32, + 2, ...
    if (!xwg_arrive_last(a.ctl + DEC_CTL_ATTN + b * a.Hkv + h, n_p, &s_last, tid)) return;
    constexpr int RP = DEC_MAX_G / 2;
    const int rl = lane >> 5, cl = lane & 31;
    float mm[RP], ll[RP];
    f32x4 oo[RP];
#pragma unroll
    for (int i = 0; i < RP; ++i) { mm[i] = -INFINITY; ll[i] = 0.f; oo[i] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    for (int pp = wave; pp < n_p; pp += NW) {
        f32x4 ov[RP];
        float mv[RP], lv[RP];
        const size_t at = (item0 + (size_t)pp * a.Hkv) * DEC_MAX_G;
#pragma unroll
        for (int i = 0; i < RP; ++i) {
            const int r = min(2 * i + rl, G - 1);
            ov[i] = xwg_load4(reinterpret_cast<const f32x4 *>(a.part_o + (at + r) * 128) + cl);
            mv[i] = xwg_load(a.part_ml + (at + r) * 2);
            lv[i] = xwg_load(a.part_ml + (at + r) * 2 + 1);
        }
        xwg_wait4(ov);
#pragma unroll
        for (int i = 0; i < RP; ++i) {
            const float M = fmaxf(mm[i], mv[i]);                        // (every piece has a key: its maximum is finite)
            const float wo = mm[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mm[i] - M), wn = __builtin_amdgcn_exp2f(mv[i] - M);
            oo[i] = oo[i] * wo + wn * ov[i];
            ll[i] = ll[i] * wo + wn * lv[i];
            mm[i] = M;
        }
    }
#pragma unroll
    for (int i = 0; i < RP; ++i) {
        const int r = 2 * i + rl;
        if (r < G) {
            *reinterpret_cast<f32x4 *>(om + r * 128 + 4 * cl) = oo[i];
            if (cl == 0) { om[1024 + r] = mm[i]; om[1040 + r] = ll[i]; }
        }
    }
    lds_barrier();
    if (row < G) {
        float M, l;
        const f32x4 acc = dec_combine<NW>(all, OM, row, c4, M, l);
        store_out(acc, l);
    }
}

// Rounds of 256 keys a workgroup makes: the fewest (a power of two up to 16) that keep the grid at about the two workgroups
// a CU holds - with many (trace, kv head) pairs, pieces of 256 keys make several rounds of short workgroups whose fixed
// costs (dispatch, lengths and page ids, the merge) add up.
static int dec_attn_rounds(int B, int Hkv, int max_L) {
    int n = 1;
    while (n < 16 && (long)B * Hkv * ((max_L + DEC_PIECE * n - 1) / (DEC_PIECE * n)) > 576) n *= 2;
    return n;
}

hipError_t launch_dec_attn(DecAttn a, hipStream_t s) {
    if (a.B < 1 || a.G < 1 || a.G > DEC_MAX_G || a.Hkv < 1 || a.B * a.Hkv > DEC_CTL_TILE - DEC_CTL_ATTN || !a.q_lo) return hipErrorInvalidValue;
    a.n_iter = dec_attn_rounds(a.B, a.Hkv, a.max_L);
    a.max_pieces = std::max((a.max_L + DEC_PIECE * a.n_iter - 1) / (DEC_PIECE * a.n_iter), 1);
    const dim3 grid(a.max_pieces * a.Hkv, a.B);
    static std::atomic<uint32_t> attr8{0}, attr4{0};
    // up to about one workgroup per CU: eight wavefronts, the shorter chain; beyond, four, of which two workgroups fit a CU
    if ((long)grid.x * grid.y <= 288) {
        if (hipError_t e = set_dynamic_lds_once(attr8, reinterpret_cast<const void *>(dec_attn_kernel<8, 2>), DEC_ATTN_SMEM); e != hipSuccess) return e;
        dec_attn_kernel<8, 2><<<grid, 512, DEC_ATTN_SMEM, s>>>(a);
    } else {
        if (hipError_t e = set_dynamic_lds_once(attr4, reinterpret_cast<const void *>(dec_attn_kernel<4, 4>), DEC_ATTN_SMEM); e != hipSuccess) return e;
        dec_attn_kernel<4, 4><<<grid, 256, DEC_ATTN_SMEM, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace cs
