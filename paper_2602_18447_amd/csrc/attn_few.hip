// Attention of a pass over few suffix tokens (generation steps, one or a few traces being verified), bf16 operands on
// the matrix cores, fp32 online softmax.  The passes over more tokens have attn_bf16.hip.
//
// There are few query rows - 6 per kv head and token on the smaller model - and the chip has to be filled from the
// keys: a workgroup takes a tile of 16 or 32 query rows of one (context unit, kv head) and one piece of its cached keys;
// where a trace brings several suffix tokens, the suffix keys are one more piece, and where it brings one, the first
// wavefront of the last piece adds that one key.  Inside a workgroup every wavefront walks its own run of 16-token pages,
// two per round, and keeps its own (max, sum, O): no workgroup barrier before the results are combined.  The workgroup
// that finishes a tile last merges the pieces, in piece order (the even and then the odd ones where the rows are few), so the
// result does not depend on which one that is.
//
// Keys and values travel global -> LDS directly, rows of 256 bytes: reading the score product's operand straight from
// memory instead takes 16 rows per load, four different rows in neighbouring lanes, which the address unit works off
// four times slower.  A round's region of keys is refilled as soon as its operands are in registers, the region of
// values after the value product.
//  * Key k keeps its 16-byte vector v at slot v ^ (k & 15): the 16 keys a read takes at one v lie in 16 slots.
//  * Token k keeps value vector v at slot v ^ (2 (k & 7)), so that the 32 bytes x 8 consecutive tokens that half a
//    wavefront reads at a time (transposing reads) fall into different banks.
//  * Transposing reads (ds_read_b64_tr_b16): in a group of 16 lanes, lane i supplies the address of 4 consecutive 16-bit
//    elements and receives element i % 4 of what lanes i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4 addressed.
#include "kernels.h"
#include "xwg.h"
#include <algorithm>
#include <type_traits>

namespace cs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(8))) short i16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define CS_LDS_AS __attribute__((address_space(3)))

namespace {

constexpr int NW = 8;                // wavefronts of a workgroup; their regions leave room for one workgroup per CU

__device__ inline f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// 64 lanes x 16 bytes from per-lane global addresses into LDS at lds_dst + 16 * lane (lds_dst wave-uniform).  Issued from
// inline assembly with a memory clobber: the compiler neither reorders memory accesses across it nor waits for it;
// completion is waited for with wait_vm.
__device__ inline void dma16(const void *src, unsigned lds_dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_dst), "v"(src) : "memory");
}
// the same from a wave-uniform address plus 32-bit byte offsets
__device__ inline void dma16_base(const void *base, unsigned off, unsigned lds_dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_dst), "v"(off), "s"(base) : "memory");
}
template <int N>
__device__ inline void wait_vm() {   // at most N vector memory operations of this wavefront still outstanding (issue order)
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

__device__ inline unsigned short to_fmt(float v, int fmt) {   // fmt 3: IEEE half (saturating), else bf16
    return fmt == 3 ? __half_as_ushort(to_half_sat(v)) : __bfloat16_as_ushort(__float2bfloat16(v));
}
// over the four lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ inline float quad_max(float v) {
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float quad_sum(float v) {
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}
// Wave-uniform loads of what no kernel of this launch writes: into scalar registers, apart from the vector memory counter.
typedef __attribute__((address_space(4))) const int32_t scalar_i32;
__device__ inline int scalar_load(const int32_t *p) { return *(scalar_i32 *)(uintptr_t)p; }
__device__ inline float exp2_from(float m, float ref) { return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - ref); }

// A row of results keeps its 16-byte vector v at slot v ^ (row & 15): a wavefront stores one vector of 16 rows at a time.
__device__ inline int om_at(int row, int v) { return row * 128 + 4 * (v ^ (row & 15)); }
// The wavefronts' results [row][128] (om, 4096 floats per wavefront) and (max, sum) s_ml merged for (row, columns 4 c4 ..
// + 3), in wavefront order; a wavefront without keys for the row left a maximum of -inf.
template <int ROWS>
__device__ inline f32x4 combine(const float *om, const float (&s_ml)[NW][ROWS][2], int row, int c4, float &M, float &l) {
    M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, s_ml[w][row][0]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float mw = s_ml[w][row][0];
        const f32x4 o = *reinterpret_cast<const f32x4 *>(om + w * 4096 + om_at(row, c4));
        if (mw != -INFINITY) {
            const float wgt = __builtin_amdgcn_exp2f(mw - M);
            acc += wgt * o;
            l += wgt * s_ml[w][row][1];
        }
    }
    return acc;
}

}  // namespace

// RB: blocks of 16 query rows.  TERMS == 2: q and the probabilities carried as two bf16 terms, in the suffix piece also keys
// and values.  ONE: every trace has one suffix token (tile = trace); second terms of its key and value where they are given.
// What bounds it: at few tiles the chain of round trips - tile or length, page ids, keys and values, arrival counter, the
// other pieces - and at many the stream of keys and values, for which each wavefront has 16 KiB in flight.
template <int RB, int TERMS, bool ONE>
__global__ __launch_bounds__(64 * NW, 2) void few_attn_kernel(FewAttn a) {
    constexpr int ROWS = 16 * RB, WLDS = 16384;          // a wavefront's keys and values of a round, later its results
    static_assert(ROWS * 512 <= WLDS, "results fit the region");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ float s_ml[NW][ROWS][2];
    __shared__ volatile int s_last;
    asm volatile("" : : "s"(a.q), "s"(a.q_lo), "s"(a.ksuf), "s"(a.vsuf), "s"(a.k_pages), "s"(a.v_pages), "s"(a.table), "s"(a.plens), "s"(a.out),
                 "s"(a.part_o), "s"(a.part_ml), "s"(a.pieces), "s"(a.wave_pages), "s"(a.tiles), "s"(a.n_tiles), "s"(a.inv_G));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid: pieces from the last one of the longest context down.  With several tiles per context, the tiles that read the
    // same piece follow each other, and each XCD (workgroup id % 8) takes an eighth of that list: its cache serves all but
    // the first of them.
    const int groups = a.pieces * a.Hkv;
    int tile, grp;
    if constexpr (ONE) {
        tile = blockIdx.x / groups;
        grp = blockIdx.x - tile * groups;
    } else {
        const int i = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        grp = i / a.n_tiles;
        tile = i - grp * a.n_tiles;
        if (grp >= groups) return;
    }
    const int p = a.pieces - 1 - grp / a.Hkv, h = grp % a.Hkv;
    const int ppw = a.wave_pages, piece_keys = 16 * NW * ppw, G = a.G;
    FewTile t;
    int page0, n_p;
    bool suf = false;
    int entry[2];
    auto fetch_ids = [&](int pg) {                                      // page ids of the round that starts at page pg
#pragma unroll
        for (int i = 0; i < 2; ++i) entry[i] = scalar_load(a.table + (size_t)t.b0 * a.max_blocks + min(pg + i, a.max_blocks - 1));
    };
    if constexpr (ONE) {
        t.b0 = tile; t.cu0 = tile; t.row0 = 0; t.n_rows = G; t.k_start = tile; t.n_keys = 1;
        page0 = (p * NW + wave) * ppw;
        fetch_ids(page0);                                               // (asked for before the length is known)
        t.L = min(max(scalar_load(a.plens + tile), 0), a.max_L);
        n_p = max((t.L + piece_keys - 1) / piece_keys, 1);
    } else {
        const int32_t *tp = reinterpret_cast<const int32_t *>(a.tiles + tile);
        t.b0 = scalar_load(tp); t.cu0 = scalar_load(tp + 1); t.row0 = scalar_load(tp + 2); t.n_rows = scalar_load(tp + 3);
        t.L = scalar_load(tp + 4); t.k_start = scalar_load(tp + 5); t.n_keys = scalar_load(tp + 6);
        // the suffix is piece 0; with a.fold there is one piece, the context and then the suffix
        n_p = a.fold ? 1 : (t.L + piece_keys - 1) / piece_keys + 1;
        suf = p == 0 && !a.fold;
        page0 = ((a.fold ? p : p - 1) * NW + wave) * ppw;
        if (!suf) fetch_ids(page0);
    }
    if (p >= n_p || t.n_rows <= 0) return;                              // uniform: a shorter context, an unused tile
    unsigned char *kst = smem + wave * WLDS, *vst = kst + 8192;
    const unsigned lds_k = (unsigned)(size_t)(CS_LDS_AS unsigned char *)kst, lds_v = lds_k + 8192;
    const int fr = lane & 15, fg = lane >> 4;

    // first key of this wavefront's round 0 and the end of its keys: cached rows, or suffix tokens counted from k_start
    int key_lo = suf ? 32 * wave : 16 * page0;
    int key_hi = suf ? min(t.n_keys, key_lo + 32) : min(t.L, key_lo + 16 * ppw);
    const size_t suf_row = (size_t)a.Hkv * 128;
    const bf16 *new_k = a.ksuf + ((size_t)t.k_start * a.Hkv + h) * 128, *new_v = a.vsuf + ((size_t)t.k_start * a.Hkv + h) * 128;
    const int lrow = lane >> 4, lslot = lane & 15;
    // one round's 32 rows, two pages: instruction jj fills tokens 4 jj .. 4 jj + 3 of a page; lane l: token 4 jj + l / 16,
    // slot l % 16.  Tokens at or past the end are masked; a suffix row is fetched for them, so that page rows that were
    // never written are not read.
    unsigned k_off[4], v_off[4];                                        // of this lane's vectors in a page's rows
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int kl = 4 * jj + lrow;
        k_off[jj] = kl * 256 + ((lslot ^ kl) << 4);
        v_off[jj] = kl * 256 + ((lslot ^ (2 * (kl & 7))) << 4);
    }
    auto issue = [&](const bf16 *pages, const bf16 *fresh, unsigned dst, int key0, const unsigned (&off)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int tok0 = key0 + 16 * kb;
            const bf16 *page = pages + ((size_t)min(max(entry[kb], 0), a.n_blocks - 1) * a.Hkv + h) * 16 * 128;
            if (!suf && tok0 + 16 <= key_hi) {                          // wave-uniform
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) dma16_base(page, off[jj], dst + kb * 4096 + jj * 1024);
            } else {
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int k = tok0 + 4 * jj + lrow, vec = (off[jj] & 255) >> 1;
                    const bf16 *row = suf ? fresh + min(k, t.n_keys - 1) * suf_row : k < key_hi ? page + (k & 15) * 128 : fresh;
                    dma16(row + vec, dst + kb * 4096 + jj * 1024);
                }
            }
        }
    };
    auto first_round = [&]() __attribute__((always_inline)) {
        if (key_lo < key_hi) {                                          // wave-uniform
            issue(a.k_pages, new_k, lds_k, key_lo, k_off);
            issue(a.v_pages, new_v, lds_v, key_lo, v_off);
        }
    };
    first_round();
    // q operand: lane l holds query row l % 16 of a block (rows past the end repeat the last one; they are never stored),
    // head-dim elements 32 ks + 8 (l / 16) .. + 7.  Asked for behind the first round: it comes from a cache, the keys do not.
    bf16x8 q_hi[RB][4], q_lo[TERMS == 2 ? RB : 1][4];
    int tok[RB];                                                        // packed suffix token of the row
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = min(t.row0 + 16 * rb + fr, t.n_rows - 1), tt = ONE ? 0 : (int)((unsigned)r * (unsigned)a.inv_G >> 20);      // r / G
        tok[rb] = t.cu0 + tt;
        const size_t qo = ((size_t)tok[rb] * a.Hq + (size_t)h * G + (r - tt * G)) * 128 + 8 * fg;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            q_hi[rb][ks] = *reinterpret_cast<const bf16x8 *>(a.q + qo + 32 * ks);
            if constexpr (TERMS == 2) q_lo[rb][ks] = *reinterpret_cast<const bf16x8 *>(a.q_lo + qo + 32 * ks);
        }
    }
    float m_w[RB], l_w[RB];                                             // running maximum (log2 units) and sum of this wavefront
    f32x4 o_acc[RB][8];
    int k_lo[RB];                                                       // first suffix token the row sees (suffix piece)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_w[rb] = -INFINITY;
        l_w[rb] = 0.f;
        k_lo[rb] = 0;
        if (suf || (!ONE && a.fold)) k_lo[rb] = min(a.cu[min(max(a.tok_trace[tok[rb]], 0), a.B - 1)], tok[rb]);
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) o_acc[rb][hb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // O^T += V^T . P^T over two pages; k index 8 (l / 16) + i <-> token 4 (l / 16) + i of the first page (i < 4) or the
    // second (i >= 4), which is what the lane holds of P.  V^T operand: group l / 16 reads tokens 4 (l / 16) .. + 3 of a
    // page; lane i of the group points at token i / 4, head-dim elements 16 hb + 4 (i % 4) .. + 3 and receives the four
    // tokens of element 16 hb + i
    const int vrow = 4 * fg + (fr >> 2), q4 = fr & 3;
    auto values = [&](const unsigned char *base, const bf16x8 (&ph)[RB], const bf16x8 (&pl)[RB], bool second) __attribute__((always_inline)) {
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            const unsigned char *p0 = base + vrow * 256 + (((2 * hb + (q4 >> 1)) ^ (2 * (vrow & 7))) << 4) + ((q4 & 1) << 3);
            i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CS_LDS_AS i16x4 *)p0);
            i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((CS_LDS_AS i16x4 *)(p0 + 4096));
            bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                o_acc[rb][hb] = mma16(vf, ph[rb], o_acc[rb][hb]);
                if (second) o_acc[rb][hb] = mma16(vf, pl[rb], o_acc[rb][hb]);
            }
        }
    };
    // the keys of the piece; with a.fold the suffix after the context
    for (int again = !ONE && a.fold;; again = 0) {
        for (int key0 = key_lo; key0 < key_hi; key0 += 32) {                // wave-uniform
            const bool more = key0 + 32 < key_hi;
            if (more) fetch_ids((key0 >> 4) + 2);
            wait_vm<8>();                                                   // the keys have landed; the values may not have
            const bool lo_terms = TERMS == 2 && !ONE && suf;
            auto refill_keys = [&]() __attribute__((always_inline)) {
                wait_lds();                                                 // the keys' region is free
                if (more) issue(a.k_pages, new_k, lds_k, key0 + 32, k_off);
                else if (lo_terms) issue(a.v_pages, a.vsuf_lo + (new_v - a.vsuf), lds_k, key0, v_off);     // second terms of the values
            };
            // scores: S^T[token][query row]; lane l ends up with query row l % 16, tokens 4 (l / 16) + e of each page.
            // (Two terms of two blocks of rows leave no registers for all of a round's keys.)
            constexpr bool HOLD = RB * TERMS < 4;
            auto key_frag = [&](int kb, int ks) { return *reinterpret_cast<const bf16x8 *>(kst + kb * 4096 + fr * 256 + (((4 * ks + fg) ^ fr) << 4)); };
            bf16x8 kf[HOLD ? 2 : 1][4];
            if constexpr (HOLD) {
#pragma unroll
                for (int i = 0; i < 8; ++i) kf[i >> 2][i & 3] = key_frag(i >> 2, i & 3);
                refill_keys();
            }
            f32x4 sc[RB][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                if constexpr (!HOLD) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) kf[0][ks] = key_frag(kb, ks);
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    sc[rb][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        sc[rb][kb] = mma16(kf[HOLD ? kb : 0][ks], q_hi[rb][ks], sc[rb][kb]);
                        if constexpr (TERMS == 2) sc[rb][kb] = mma16(kf[HOLD ? kb : 0][ks], q_lo[rb][ks], sc[rb][kb]);
                    }
                }
            }
            if constexpr (!HOLD) refill_keys();
            if (lo_terms) {                                                 // second terms of the keys
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const bf16 *kr = a.ksuf_lo + (new_k - a.ksuf) + min(key0 + 16 * kb + fr, t.n_keys - 1) * suf_row + 8 * fg;
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) kf[0][ks] = *reinterpret_cast<const bf16x8 *>(kr + 32 * ks);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) sc[rb][kb] = mma16(kf[0][ks], q_hi[rb][ks], sc[rb][kb]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            bf16x8 p_hi[RB], p_lo[RB];
            const bool whole = !suf && key0 + 32 <= key_hi;                 // wave-uniform: every row sees every key
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if (!whole) {                                               // keys k_min .. k_end - 1 are seen
                    const int k_min = suf ? k_lo[rb] - t.k_start : 0, k_end = suf ? min(tok[rb] - t.k_start + 1, key_hi) : key_hi;
                    const unsigned n_seen = max(k_end - k_min, 0);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const unsigned k = (unsigned)(key0 + 16 * (i >> 2) + 4 * fg + (i & 3) - k_min);
                        sc[rb][i >> 2][i & 3] = k < n_seen ? sc[rb][i >> 2][i & 3] : -INFINITY;
                    }
                }
                float mx = sc[rb][0][0];
#pragma unroll
                for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sc[rb][i >> 2][i & 3]);
                const float m_new = fmaxf(m_w[rb], quad_max(mx) * a.scale_log2), ref = m_new == -INFINITY ? 0.f : m_new;
                if (__builtin_amdgcn_ballot_w64(m_new > m_w[rb]) != 0) {
                    const float alpha = exp2_from(m_w[rb], ref);
                    l_w[rb] *= alpha;
#pragma unroll
                    for (int hb = 0; hb < 8; ++hb) o_acc[rb][hb] *= alpha;
                }
                m_w[rb] = m_new;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float pr = __builtin_amdgcn_exp2f(fmaf(sc[rb][i >> 2][i & 3], a.scale_log2, -ref));
                    l_w[rb] += pr;
                    const __bf16 hi = (__bf16)pr;
                    p_hi[rb][i] = hi;
                    if constexpr (TERMS == 2) p_lo[rb][i] = (__bf16)(pr - (float)hi);
                }
            }
            if (more || lo_terms) wait_vm<8>(); else wait_vm<0>();          // the values have landed
            values(vst, p_hi, p_lo, TERMS == 2);
            if (lo_terms) {
                wait_vm<0>();
                values(kst, p_hi, p_lo, false);
            }
            wait_lds();                                                     // the values' region is free
            if (more) issue(a.v_pages, new_v, lds_v, key0 + 32, v_off);
        }
        if (!again) break;
        suf = true;
        key_lo = 32 * wave;
        key_hi = min(t.n_keys, key_lo + 32);
        first_round();
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) l_w[rb] = quad_sum(l_w[rb]);        // (a lane has added up its own tokens)
    if (ONE && p == n_p - 1 && wave == 0) {                             // the new token
        f32x4 sn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {                                // (its key in all 16 rows of the operand)
            const bf16x8 kn = *reinterpret_cast<const bf16x8 *>(new_k + 32 * ks + 8 * fg);
            sn = mma16(kn, q_hi[0][ks], sn);
            if constexpr (TERMS == 2) {
                sn = mma16(kn, q_lo[0][ks], sn);
                if (a.ksuf_lo) sn = mma16(*reinterpret_cast<const bf16x8 *>(a.ksuf_lo + (new_k - a.ksuf) + 32 * ks + 8 * fg), q_hi[0][ks], sn);
            }
        }
        const float v = sn[0] * a.scale_log2, m_new = fmaxf(m_w[0], v);
        const float alpha = exp2_from(m_w[0], m_new), pr = __builtin_amdgcn_exp2f(v - m_new);
        m_w[0] = m_new;
        l_w[0] = l_w[0] * alpha + pr;
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            const uint2 vn = *reinterpret_cast<const uint2 *>(new_v + 16 * hb + 4 * fg);
            f32x4 vf = {__uint_as_float(vn.x << 16), __uint_as_float(vn.x & 0xffff0000u), __uint_as_float(vn.y << 16), __uint_as_float(vn.y & 0xffff0000u)};
            if (TERMS == 2 && a.vsuf_lo) {
                const uint2 vl = *reinterpret_cast<const uint2 *>(a.vsuf_lo + (new_v - a.vsuf) + 16 * hb + 4 * fg);
                vf += f32x4{__uint_as_float(vl.x << 16), __uint_as_float(vl.x & 0xffff0000u), __uint_as_float(vl.y << 16), __uint_as_float(vl.y & 0xffff0000u)};
            }
            o_acc[0][hb] = o_acc[0][hb] * alpha + pr * vf;
        }
    }
    // ---- the wavefronts' results, each in its own region, combined in wavefront order
    const int rows = min(ROWS, t.n_rows - t.row0);                      // rows of this tile that exist
    float *om = reinterpret_cast<float *>(kst);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = 16 * rb + fr;
        if (m_w[rb] != -INFINITY && row < rows) {
#pragma unroll
            for (int hb = 0; hb < 8; ++hb) *reinterpret_cast<f32x4 *>(om + om_at(row, 4 * hb + fg)) = o_acc[rb][hb];
        }
        if (fg == 0) {
            s_ml[wave][row][0] = m_w[rb];
            s_ml[wave][row][1] = l_w[rb];
        }
    }
    lds_barrier();
    const float *all = reinterpret_cast<const float *>(smem);
    auto store_out = [&](int row, int c4, f32x4 acc, float l) {
        const float inv = 1.0f / l;
        const int r = t.row0 + row, tt = ONE ? 0 : (int)((unsigned)r * (unsigned)a.inv_G >> 20);
        unsigned short *o = reinterpret_cast<unsigned short *>(a.out) + frag_index(t.cu0 + tt, (h * G + r - tt * G) * 128 + 4 * c4, a.Hq * 128);
        ushort4 v = {to_fmt(acc[0] * inv, a.out_fmt), to_fmt(acc[1] * inv, a.out_fmt), to_fmt(acc[2] * inv, a.out_fmt), to_fmt(acc[3] * inv, a.out_fmt)};
        *reinterpret_cast<ushort4 *>(o) = v;
    };
    const int c4 = tid & 31;
    const size_t rec0 = ((size_t)tile * a.Hkv + h) * a.pieces;          // piece p: rec0 + p
#pragma unroll
    for (int row = tid >> 5; row < ROWS; row += 2 * NW) {
        if (row >= rows) break;
        float M, l;
        const f32x4 acc = combine<ROWS>(all, s_ml, row, c4, M, l);
        if (n_p == 1) {
            store_out(row, c4, acc, l);
        } else {
            const size_t at = (rec0 + p) * ROWS + row;
            xwg_store4(reinterpret_cast<f32x4 *>(a.part_o + at * 128) + c4, acc);
            if (c4 == 0) {
                xwg_store(a.part_ml + at * 2, M);
                xwg_store(a.part_ml + at * 2 + 1, l);
            }
        }
    }
    if (n_p == 1) return;
    // ---- the pieces of this tile and kv head: the last workgroup to arrive merges them.  A thread has columns 4 c4 .. + 3 of a row (of two where
    // there are 32) and adds the pieces up in order, 12 or 8 of them in flight, 4 where that is all, weighed by their common maximum (a running one chains their
    // exponentials: generate one token at 4096 keys, 17 pieces, 1388 -> 1340 us a step); up to 8 rows take half of the threads each for the even and
    // the odd pieces, whose sums meet in LDS.  What bounds it is a round of loads from the memory side (about a microsecond) and what is loaded, so
    // the rounds are few, little else is between them and the result, and with 32 rows the last one is of about the size of what is left.  Whole launch in a pass
    // against wavefronts that took every eighth piece two at a time and met in LDS: one trace of 2048 keys and 96 tokens (5 pieces) 16.6 -> 15.4 us,
    // 32 traces of 2048 keys and one token (4) 19.0 -> 18.4, one of 4096 (17) 12.6 -> 11.7.
    if (!xwg_arrive_last(a.arrived + tile * a.Hkv + h, n_p, &s_last, tid)) return;
    const bool halves = ONE && rows <= 8;                               // uniform
    const int odd = halves ? tid >> 8 : 0, step = halves ? 2 : 1, row0 = halves ? (tid >> 5) & 7 : tid >> 5;
    const XwgLoads parts(a.part_o + rec0 * ROWS * 128, (unsigned)(n_p * ROWS) * 512u), stats(a.part_ml + rec0 * ROWS * 2, (unsigned)(n_p * ROWS) * 8u);
    float mm[RB], ll[RB];
    f32x4 oo[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) { mm[i] = -INFINITY; ll[i] = 0.f; oo[i] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    // the pieces from first on, FLY at a time, in rounds that begin before end; rest: such a round may go past the last piece
    auto add_pieces = [&](int first, int end, auto fly, auto rest) __attribute__((always_inline)) {
        constexpr int FLY = decltype(fly)::value;
        for (int pp = first; pp < end; pp += FLY * step) {
            f32x4 ov[FLY][RB];
            float2 ml[FLY][RB];
#pragma unroll
            for (int q = 0; q < FLY; ++q)
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const unsigned rec = (decltype(rest)::value ? min(pp + q * step, n_p - 1) : pp + q * step) * ROWS + min(row0 + 16 * i, rows - 1);
                    ov[q][i] = parts.load4(rec * 512u + c4 * 16u);
                    ml[q][i] = stats.load2(rec * 8u);
                }
#pragma unroll
            for (int i = 0; i < RB; ++i) {                                  // (every row sees a key of every piece)
                float M = mm[i];
#pragma unroll
                for (int q = 0; q < FLY; ++q) M = fmaxf(M, ml[q][i].x);     // (past the end: the last piece again)
                const float wo = exp2_from(mm[i], M);
                oo[i] *= wo;
                ll[i] *= wo;
                mm[i] = M;
#pragma unroll
                for (int q = 0; q < FLY; ++q) {
                    const bool here = !decltype(rest)::value || pp + q * step < n_p;      // (nothing of the repeated piece: it may hold an infinity)
                    const float wn = here ? __builtin_amdgcn_exp2f(ml[q][i].x - M) : 0.f;
                    oo[i] += wn * (here ? ov[q][i] : f32x4{0.f, 0.f, 0.f, 0.f});
                    if (!decltype(rest)::value && q > 0) {               // (unfused, as behind the select: the same bits whatever the round)
#pragma clang fp contract(off)
                        ll[i] += wn * ml[q][i].y;
                    } else {
                        ll[i] += here ? wn * ml[q][i].y : 0.f;
                    }
                }
            }
        }
    };
    if constexpr (RB == 1) {
        if (n_p <= 4 * step) add_pieces(odd, n_p, std::integral_constant<int, 4>{}, std::true_type{});
        else add_pieces(odd, n_p, std::integral_constant<int, 12>{}, std::true_type{});
    } else {
        // The rest in a round of about its size: what is loaded for nothing takes its share of the CU's stream, too.  33 pieces of 32 rows read as
        // 40, four layers of 1536 x 8960, 3 x 5 tokens of 16000 keys, 272 us, as 34 265; 17 as 24, 32 tokens of 8000 keys, 254, as 18 245.  (With 16 rows
        // and fewer, half and a quarter of the bytes, a second size of the round costs as much as it saves.)
        const int whole = n_p / 8 * 8, left = n_p - whole;
        add_pieces(0, whole, std::integral_constant<int, 8>{}, std::false_type{});
        if (left > 6) add_pieces(whole, n_p, std::integral_constant<int, 8>{}, std::true_type{});
        else if (left > 4) add_pieces(whole, n_p, std::integral_constant<int, 6>{}, std::true_type{});
        else if (left > 2) add_pieces(whole, n_p, std::integral_constant<int, 4>{}, std::true_type{});
        else if (left > 0) add_pieces(whole, n_p, std::integral_constant<int, 2>{}, std::true_type{});
    }
    if (halves) {
        f32x4 *meet = reinterpret_cast<f32x4 *>(smem);                  // [8 rows][32]
        if (odd == 1) {
            meet[row0 * 32 + c4] = oo[0];
            if (c4 == 0) { s_ml[0][row0][0] = mm[0]; s_ml[0][row0][1] = ll[0]; }
        }
        lds_barrier();
        if (odd == 1) return;
        const float m2 = s_ml[0][row0][0], M = fmaxf(mm[0], m2);
        const float wo = __builtin_amdgcn_exp2f(mm[0] - M), wn = exp2_from(m2, M);
        oo[0] = oo[0] * wo + wn * meet[row0 * 32 + c4];
        ll[0] = ll[0] * wo + wn * s_ml[0][row0][1];
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
        if (row0 + 16 * i < rows) store_out(row0 + 16 * i, c4, oo[i], ll[i]);
}

namespace {
template <int RB, int TERMS, bool ONE>
hipError_t launch(const FewAttn &a, int grid, hipStream_t s) {
    constexpr int smem = NW * 16384;
    static std::atomic<uint32_t> attr{0};
    if (hipError_t e = set_dynamic_lds_once(attr, reinterpret_cast<const void *>(few_attn_kernel<RB, TERMS, ONE>), smem); e != hipSuccess) return e;
    few_attn_kernel<RB, TERMS, ONE><<<grid, 64 * NW, smem, s>>>(a);
    return hipGetLastError();
}
}  // namespace

int few_attn_rows(bool one) { return one ? 16 : 32; }
int64_t few_attn_tiles(const int32_t *h_cu, int B, const int32_t *h_group_start, int n_units, int G, bool one) {
    if (one) return B;
    int64_t n = 0;
    if (!h_group_start) n_units = B;
    for (int i = 0; i < n_units; ++i) {
        const int b0 = h_group_start ? h_group_start[i] : i, b1 = h_group_start ? h_group_start[i + 1] : i + 1;
        n += ((int64_t)G * (h_cu[b1] - h_cu[b0]) + few_attn_rows(false) - 1) / few_attn_rows(false);
    }
    return n;
}
constexpr int FEW_SLOTS = 256;       // workgroups that are resident at once
static_assert(FEW_RECORDS >= FEW_SLOTS, "a record per workgroup where a tile has several pieces");

// Pieces of the longest context (and the suffix, where there are several suffix tokens): as many as fill the chip once; a
// wavefront takes an even number of pages, because the round of a single page costs nearly what one of two does (one trace
// of 4096 keys: 32 pieces of one page per wavefront 12.5 us, 16 of two 10.6 us, 11 of three 12.2 us, 8 of four 12.1 us).
// A tile has one piece or n_tiles * Hkv * pieces <= FEW_SLOTS, so FEW_RECORDS partial results are enough.
void few_attn_pieces(FewAttn &a, bool one) {
    const int suffix = one ? 0 : 1, want = std::max(FEW_SLOTS / (a.n_tiles * a.Hkv) - suffix, 1);
    const int pages = std::max((a.max_L + 15) / 16, 1);
    a.wave_pages = 2 * ((pages - 1) / (2 * NW * want) + 1);
    a.pieces = (pages - 1) / (NW * a.wave_pages) + 1;
    a.fold = !one && a.pieces == 1;
    if (!a.fold) a.pieces += suffix;
}

hipError_t launch_few_attn(FewAttn a, hipStream_t s) {
    const bool one = a.tiles == nullptr, two = a.q_lo != nullptr;
    if (a.B < 1 || !few_attn_takes(a.n_tiles, a.Hkv, a.G, a.T, one) || (one && a.B != a.n_tiles) || (!one && two && (!a.ksuf_lo || !a.vsuf_lo)))
        return hipErrorInvalidValue;
    static_assert(SK_MAX_ROWS * FEW_MAX_G * FEW_MAX_G < 1 << 20, "r / G from a product");
    a.inv_G = (1 << 20) / a.G + 1;                       // r / G for r < 128 G: r G < 2^20
    few_attn_pieces(a, one);
    const int items = a.pieces * a.Hkv * a.n_tiles, grid = one ? items : (items + 7) / 8 * 8;
    if (one) return two ? launch<1, 2, true>(a, grid, s) : launch<1, 1, true>(a, grid, s);
    return two ? launch<2, 2, false>(a, grid, s) : launch<2, 1, false>(a, grid, s);
}

}  // namespace cs
