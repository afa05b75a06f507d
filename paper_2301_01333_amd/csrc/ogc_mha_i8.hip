// Int8 scaled dot-product attention for gfx950 (the Int8 rows of Table I, Section VII): both batch matmuls on the
// int8 matrix instruction, the scalar, the mask and the softmax in between, one kernel, scores never leaving the
// compute unit.
//
// Definition (per batch entry, head and query i; q, k, v int8 with zero point 0):
//   S[j]  = sum_c q[i][c] k[j][c]                         int32
//   s[j]  = S[j] * (q_scale*k_scale*scale) + mask[j]      fp32, here in the base-2 logarithm domain
//   e[j]  = 2^(s[j] - max_j s[j])
//   P[j]  = rne(127 e[j])                                 7 bits unsigned: the signed int8 operand of the second product
//   A[c]  = sum_j P[j] v[j][c],  L = sum_j P[j]           int32
//   o[c]  = clamp(rne((float(A[c]) / float(L)) * (v_scale/o_scale)), -128, 127)
// The normalisation uses the integer sum of the QUANTIZED numerators and comes after the integer product, so nothing
// has to be rescaled while the keys stream by; the price is that the row maximum must be known before the first
// numerator is quantized: the kernel makes two passes over the keys, the first computing scores and their maximum
// only (the first product on the int8 matrix pipe is cheap next to the softmax arithmetic of the second pass).
//
// One workgroup = 4 wavefronts = 128 queries of one (batch, head), a lane owns one query; both products are computed
// transposed (S^T = K Q^T, O^T = V^T P^T) so that, in the 32x32 accumulator layout, a lane's 16 scores of a 32-key
// group become, after quantization, exactly its 16 bytes of the second product's operand: V^T goes to LDS with the
// key index permuted to the order in which the accumulator registers hold the keys.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <type_traits>

#include "ogc_mha.h"

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

#define MHA8_DEV static __device__ __forceinline__

struct MhaI8Args {
    const uint8_t* q;
    const uint8_t* k;
    const uint8_t* v;
    const float* mask;
    uint8_t* o;
    long long sq[3], sk[3], sv[3], so[3];  // element (= byte) strides: batch, head, token
    int batch, heads, seq;
    int q_tiles;    // ceil(seq / 128)
    int xcd_order;  // 1: the query tiles of one (batch, head) are placed on one XCD
    uint32_t tiles_magic, heads_magic;  // reciprocals of q_tiles and heads (0: divide)
    int far;        // 1: a unit's rows span more than 32 bits of byte offset
    float c1;       // q_scale * k_scale * scale * log2(e)
    float r;        // v_scale / o_scale
};

MHA8_DEV void swap32_i8(uint32_t& a, uint32_t& b) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
MHA8_DEV float other_half_f(float x) {
    uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
    swap32_i8(a, b);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? a : b);
}
MHA8_DEV int other_half_i(int x) {
    uint32_t a = (uint32_t)x, b = a;
    swap32_i8(a, b);
    return (int)((threadIdx.x & 32) ? a : b);
}

// a mask value in the base-2 domain; the lowest stay finite (-infinity is for keys beyond the sequence), NaN passes
MHA8_DEV float base2_mask(float m) {
    return (m < -2.3e38f ? -2.3e38f : m) * 1.44269504088896340736f;
}

// The plain kernel: keys and values through registers, both passes over 64-key blocks.  For launches that do not fill the
// chip (stream_case below).  D32 = head_dim / 32.  Key blocks of 64 (two 32-key groups).
template <int D32> __global__ __launch_bounds__(256, 2) void ogc_mha_i8_kernel(MhaI8Args a) {
    constexpr int D = D32 * 32, KB = 64, SB = 2;
    constexpr int KSTR = D + 16;    // bytes per key row of K in LDS (padded: consecutive rows start 4 banks apart)
    constexpr int VSTR = KB + 16;   // bytes per channel row of V^T in LDS
    constexpr int CH = D / 16;      // 16-byte chunks per token row
    constexpr int UNITS = KB * CH;  // 16-byte chunks per block of keys (or values)
    constexpr int KU = (UNITS + 255) / 256;
    __shared__ __attribute__((aligned(16))) uint8_t k_lds[KB * KSTR];
    __shared__ __attribute__((aligned(16))) uint8_t vt_lds[D * VSTR];
    __shared__ __attribute__((aligned(16))) float m_lds[KB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, col = lane & 31;
    int bh, qt;
    if (a.xcd_order) {
        const int L = blockIdx.x, x = L & 7, r = L >> 3;
        bh = x + 8 * (r / a.q_tiles);
        qt = r % a.q_tiles;
    } else {
        bh = blockIdx.x / a.q_tiles;
        qt = blockIdx.x % a.q_tiles;
    }
    const int b = bh / a.heads, hd = bh % a.heads, S = a.seq;
    const uint8_t* kbase = a.k + b * a.sk[0] + hd * a.sk[1];
    const uint8_t* vbase = a.v + b * a.sv[0] + hd * a.sv[1];
    const long long kss = a.sk[2], vss = a.sv[2];

    // this lane's query row as the second operand of the first product: bytes 32 i + 16 h .. + 15 of the row
    const int query = (qt * 4 + wave) * 32 + col;
    v4i qreg[D32];
    {
        const int qrow = query < S ? query : S - 1;
        const uint8_t* qp = a.q + b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2];
#pragma unroll
        for (int i = 0; i < D32; ++i) qreg[i] = *(const v4i*)(qp + i * 32 + h * 16);
    }

    v4i kreg[KU], vreg[KU];
    float mreg = 0.0f;   // the mask value as loaded; scaled when it is written to LDS (scaling here would wait for the load,
                         // and with it for every key / value load issued just before)
    bool mpad = false;   // the key lies beyond the sequence
    auto prefetch = [&](int key0, bool with_v) {
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int u = tid + 256 * i, key = key0 + u / CH, part = u % CH;
            const bool on = (UNITS % 256 == 0 || u < UNITS) && key < S;
            kreg[i] = on ? *(const v4i*)(kbase + key * kss + part * 16) : (v4i){0, 0, 0, 0};
            if (with_v) vreg[i] = on ? *(const v4i*)(vbase + key * vss + part * 16) : (v4i){0, 0, 0, 0};
        }
        if (tid < KB) {
            const int key = key0 + tid;
            mpad = key >= S;
            mreg = 0.0f;
            if (!mpad && a.mask) mreg = a.mask[(long long)b * S + key];
        }
    };
    auto fill_lds = [&](bool with_v) {
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int u = tid + 256 * i;
            if (UNITS % 256 == 0 || u < UNITS) {
                const int kk = u / CH, part = u % CH;
                *(v4i*)(k_lds + kk * KSTR + part * 16) = kreg[i];
                if (with_v) {
                    // key kk of the block sits, inside its group of 32, at offset 8g + 4hh + e; the accumulator
                    // registers of a lane in half hh hold it as byte 4g + e: position 16hh + 4g + e
                    const int ko = kk & 31, pos = (kk & 32) + 16 * ((ko >> 2) & 1) + 4 * (ko >> 3) + (ko & 3);
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        vt_lds[(16 * part + j) * VSTR + pos] = (uint8_t)((uint32_t)vreg[i][j >> 2] >> (8 * (j & 3)));
                }
            }
        }
        if (tid < KB) m_lds[tid] = mpad ? -INFINITY : base2_mask(mreg);
    };
    // scores of the current block in the base-2 domain, scalar and mask applied: t[sb][4g+e] <-> key 32 sb + 8g + 4h + e
    auto scores = [&](float (&t)[SB][16]) {
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            const uint8_t* krow = k_lds + (sb * 32 + col) * KSTR + h * 16;
            v16i acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
            for (int i = 0; i < D32; ++i) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(krow + i * 32), qreg[i], acc, 0, 0, 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f mk = *(const v4f*)(m_lds + sb * 32 + 8 * g + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) t[sb][4 * g + e] = __builtin_fmaf((float)acc[4 * g + e], a.c1, mk[e]);
            }
        }
    };

    const int nkb = (S + KB - 1) / KB;
    // ---- pass 1: the row maximum
    float row_max = -INFINITY;
    prefetch(0, false);
    for (int kb = 0; kb < nkb; ++kb) {
        __syncthreads();
        fill_lds(false);
        __syncthreads();
        if (kb + 1 < nkb) prefetch((kb + 1) * KB, false);
        float t[SB][16];
        scores(t);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb)
#pragma unroll
            for (int r = 0; r < 16; ++r) row_max = fmaxf(row_max, t[sb][r]);
    }
    row_max = fmaxf(row_max, other_half_f(row_max));  // key 0 always exists: finite

    // ---- pass 2: numerators, quantized, and the second product
    v16i oacc[D32];
#pragma unroll
    for (int d = 0; d < D32; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0;
    uint32_t row_sum = 0;  // this lane's keys only; the halves are added at the end
    prefetch(0, true);
    for (int kb = 0; kb < nkb; ++kb) {
        __syncthreads();
        fill_lds(true);
        __syncthreads();
        if (kb + 1 < nkb) prefetch((kb + 1) * KB, true);
        float t[SB][16];
        scores(t);
#pragma unroll
        for (int sb = 0; sb < SB; ++sb) {
            uint32_t dw[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t w = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ex = __builtin_amdgcn_exp2f(t[sb][4 * g + e] - row_max);   // in [0, 1]; a key past the end: 0
                    w = __builtin_amdgcn_cvt_pk_u8_f32(ex * 127.0f, e, w);                 // round to nearest even
                }
                dw[g] = w;
                row_sum = __builtin_amdgcn_sad_u8(w, 0u, row_sum);                         // + the four bytes
            }
            const v4i pw = {(int)dw[0], (int)dw[1], (int)dw[2], (int)dw[3]};
#pragma unroll
            for (int d = 0; d < D32; ++d) {
                const v4i vv = *(const v4i*)(vt_lds + (d * 32 + col) * VSTR + sb * 32 + 16 * h);
                oacc[d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vv, pw, oacc[d], 0, 0, 0);
            }
        }
    }

    // ---- normalise, requantize, store: after the half exchange a lane holds 16 consecutive channels of its query
    const int total = (int)row_sum + other_half_i((int)row_sum);
    const float lf = (float)total;
    uint8_t* op = a.o + b * a.so[0] + hd * a.so[1] + (long long)query * a.so[2];
#pragma unroll
    for (int d = 0; d < D32; ++d) {
        uint32_t dw[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float tt = ((float)oacc[d][4 * g + e] / lf) * a.r;
                const int qi = (int)__builtin_rintf(fminf(fmaxf(tt, -128.0f), 127.0f));
                w |= ((uint32_t)qi & 0xffu) << (8 * e);
            }
            dw[g] = w;
        }
        swap32_i8(dw[0], dw[2]);
        swap32_i8(dw[1], dw[3]);
        if (query < S) *(v4i*)(op + d * 32 + 16 * h) = (v4i){(int)dw[0], (int)dw[2], (int)dw[1], (int)dw[3]};
    }
}

typedef __attribute__((address_space(3))) uint8_t mha8_lds_u8;
typedef __attribute__((address_space(3))) uint32_t mha8_lds_u32;
typedef __attribute__((address_space(3))) float mha8_lds_f32;
typedef __attribute__((address_space(3))) v4i mha8_lds_v4i;
typedef __attribute__((address_space(3))) v4f mha8_lds_v4f;
typedef __attribute__((address_space(3))) v2i mha8_lds_v2i;

constexpr int MHA8_UNIT = 64;        // keys per unit: two groups of 32
constexpr int MHA8_LDS_KEYS = 4096;  // addends held in LDS; longer sequences replace them every 64 units
constexpr int MHA8_SLOTS = 3;        // units of keys, and of values, in LDS: one in use, two on their way
constexpr float MHA8_NEAR = 8192.0f; // scores (base-2 domain) that may go without an addend

template <int D32> struct Mha8 {
    static constexpr int D = D32 * 32, CH = D / 16;  // bytes and 16-byte pieces of a row
    static constexpr int UNIT_BYTES = MHA8_UNIT * D, RING = 2 * MHA8_SLOTS * UNIT_BYTES;
    // Position of piece c of row r inside the row: c ^ swz(r).  A read of the first product takes the same piece of eight
    // consecutive keys, one of the second (byte transpose) 16-byte pieces of the keys 8 a + 4 h + (0..3), a = 0, 1: these
    // permutations put the eight pieces on distinct groups of four banks, for rows of 32, 64, 96 and 128 bytes.
    static __device__ __forceinline__ int kswz(int r) { return D32 == 4 ? (r & 7) : D32 == 2 ? ((r >> 1) & 3) : ((r >> 2) & 1); }
    static __device__ __forceinline__ int vswz(int r) {
        return D32 == 4 ? ((r & 3) | ((r >> 1) & 4)) : D32 == 2 ? (((r >> 1) & 1) | ((r >> 2) & 2)) : ((r >> 3) & 1);
    }
};

template <int N> MHA8_DEV void mha8_wait_and_meet() {  // all but the N newest loads have landed, LDS accesses are done, then the workgroup meets
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The streaming kernel.  D32 = head_dim / 32.
//
// What it spends most on, and what follows from that: the vector ALU (49 % of the SIMDs' cycles issue to it, 16 % of the
// matrix pipe's are busy, 37 % of the LDS cycles are conflicts; 128 x 8 x 384 x 128).  Per score it owes a conversion, a multiply-add, an
// exponential and a packing conversion in the second pass; the plain kernel spends three times that, and its byte-wise
// transposed LDS writes of the values conflict for two thirds of the LDS cycles.  Here
//   * keys and values go from global memory straight into LDS, two units ahead; V^T leaves LDS through the transposing
//     read (ds_read_b64_tr_b8: 8 keys x 16 channels per 16 lanes, the keys' rows chosen by the lanes' addresses);
//   * a group of 32 keys whose mask entries are all zero (most of them) takes its maximum over the integer scores, two
//     per instruction, and needs no addend per score: the scale is positive, so the order is the same; the multiply by
//     127 and the row maximum ride in the exponent's multiply-add (2^(x + log2 127) is 127 * 2^x).  log2(127) - maximum is
//     one fp32 value, rounded at the maximum's magnitude, so this form is kept to scores below 2^13 (MHA8_NEAR): there it
//     is off by 2^-11 at most, a numerator cannot pass 127.1, and over whole rows as many numerators round apart from
//     exact ones as by the definition's order (512 keys near the top of the range: 2.9e-3 and 3.5e-3 of them at 2^13,
//     9e-5 and 1e-4 at 264, where scales of 4 / 127 end);
//   * all other groups go by the definition's order, the plain kernel's: the score with its mask, minus the maximum,
//     exponentiated, times 127.  The difference is exact at the maximum, whatever its size, so a row that is masked alike
//     has numerators of at most 127 too (a byte of 128 and more is negative to the matrix instruction);
//   * a unit whose mask entries are so low that no int8 product can make up for it is left out of both passes: its
//     numerators round to zero whatever q and k hold.  With |S| <= 16384 d, and some key's mask 0 or more, key j has none
//     if mask[j] + 2 * 16384 d c1 + 16 < 0 (base-2 domain; a numerator is zero from 2^-8 on).
// Measured (same card, padding masks of half the length to all of it, plain / this): batch 128 x 8 heads x 384 tokens x 128:
// 167 -> 105 us (460 -> 735 TOP/s); 128 x 16 x 512 x 64: 241 -> 171 (without a mask 242 -> 187); 1 x 8 x 8192 x 128: 505 -> 290.
// Both passes in one loop body (less code) was 15 % slower: the accumulators of the second live through the first.
template <int D32> __global__ __launch_bounds__(256, D32 == 4 ? 2 : 3) void ogc_mha_i8_stream_kernel(MhaI8Args a) {
    typedef Mha8<D32> B;
    constexpr int D = B::D, U = B::UNIT_BYTES;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    mha8_lds_u8* const lds = (mha8_lds_u8*)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD takes a contiguous run of (batch, head) pairs: the query tiles of a pair share its L2
    const uint32_t wg = blockIdx.x, lin = a.xcd_order ? (wg & 7) * (gridDim.x >> 3) + (wg >> 3) : wg;
    const int bh = a.tiles_magic ? __umulhi(lin, a.tiles_magic) : lin / a.q_tiles, qt = (int)lin - bh * a.q_tiles;
    const int b = a.heads_magic ? __umulhi(bh, a.heads_magic) : bh / a.heads, hd = bh - b * a.heads, S = a.seq;
    const int n = (S + MHA8_UNIT - 1) / MHA8_UNIT;
    const uint8_t* kbase = a.k + b * a.sk[0] + hd * a.sk[1];
    const uint8_t* vbase = a.v + b * a.sv[0] + hd * a.sv[1];
    const long long kss = a.sk[2], vss = a.sv[2];

    // this lane's query row as the second operand of the first product: bytes 32 i + 16 h .. + 15 of the row
    const int query = (qt * 4 + wave) * 32 + col;
    v4i qreg[D32];
    {
        const int qrow = query < S ? query : S - 1;
        const uint8_t* qp = a.q + b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2];
#pragma unroll
        for (int i = 0; i < D32; ++i) qreg[i] = *(const v4i*)(qp + i * 32 + h * 16);
    }

    // ---- addends (mask in the base-2 domain, -infinity beyond the sequence), what kind of group they make, which units count
    mha8_lds_f32* const add = (mha8_lds_f32*)(lds + B::RING);
    const int add_keys = n * MHA8_UNIT < MHA8_LDS_KEYS ? n * MHA8_UNIT : MHA8_LDS_KEYS;
    // per unit: bits 0, 1: groups with a nonzero addend; bit 2: an addend that counts beside one of 0 or more; bit 3: one of those
    mha8_lds_u32* const kinds = (mha8_lds_u32*)(add + add_keys);
    const float floor = a.c1 > 0.0f ? -(2.0f * 16384.0f * D * a.c1 + 16.0f) : -INFINITY;
    // a scale that is not positive does not keep the order of the scores, a large one not the precision of the short form
    const bool near = a.c1 > 0.0f && 16384.0f * D * a.c1 <= MHA8_NEAR;
    auto fill = [&](int first, int count) {  // keys first .. first + count - 1 (whole units, at most MHA8_LDS_KEYS)
        const float* mrow = a.mask + (long long)b * S;
#pragma unroll 1
        for (int j0 = first + tid; j0 < first + count; j0 += 1024) {  // a wavefront has one unit at a time
            float t[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = a.mask && j0 + 256 * i < S ? base2_mask(mrow[j0 + 256 * i]) : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = j0 + 256 * i;
                if (j >= first + count) break;
                const float v = j < S ? t[i] : -INFINITY;
                add[j & (MHA8_LDS_KEYS - 1)] = v;
                const uint64_t nz = __builtin_amdgcn_ballot_w64(v != 0.0f), on = __builtin_amdgcn_ballot_w64(!(v < floor));
                const uint64_t top = __builtin_amdgcn_ballot_w64(v >= 0.0f);
                if (lane == 0)
                    kinds[(j / MHA8_UNIT) & 63] = ((uint32_t)nz ? 1u : 0u) | ((uint32_t)(nz >> 32) ? 2u : 0u) | (on ? 4u : 0u) | (top ? 8u : 0u);
            }
        }
        __syncthreads();
    };
    const bool whole = n * MHA8_UNIT <= MHA8_LDS_KEYS;  // all addends fit: units can be left out
    // one bit per unit, in scalar registers (longer sequences: the 64 units whose addends are in LDS; every unit counts)
    uint64_t counts = ~0ull, odd0 = ~0ull, odd1 = ~0ull;
    int total = n, first_unit = 0;
    auto read_kinds = [&]() {
        const uint32_t kd = lane < n ? kinds[lane] : 0u;
        odd0 = __builtin_amdgcn_ballot_w64((kd & 1) != 0);
        odd1 = __builtin_amdgcn_ballot_w64((kd & 2) != 0);
        if (!near) odd0 = odd1 = ~0ull;
        const bool bounded = __builtin_amdgcn_ballot_w64((kd & 8) != 0) != 0;  // the row maximum is that of a score at least
        counts = __builtin_amdgcn_ballot_w64(lane < n && (!bounded || (kd & 4) != 0));
    };
    auto next_unit = [&](int u) { return whole ? u + 1 + __builtin_ctzll((counts >> u) >> 1 | 1ull << 63) : u + 1; };  // (past the last: unused)

    // ---- direct loads: 2 * D32 of 1 KiB for a unit's keys, as many for its values, dealt round the wavefronts.  Load m
    // covers the pieces 64 m + lane of the unit's LDS image.
    uint32_t voff[D32];  // byte offset of the lane's piece from the unit's first row; !a.far: it fits 32 bits
#pragma unroll
    for (int i = 0; i < D32; ++i) {
        const int ld = i * 4 + wave;
        const bool is_v = ld >= 2 * D32;
        const int p = (ld - (is_v ? 2 * D32 : 0)) * 64 + lane, r = p / B::CH;
        voff[i] = (uint32_t)r * (uint32_t)(is_v ? vss : kss) + ((p % B::CH) ^ (is_v ? B::vswz(r) : B::kswz(r))) * 16;
    }
    int lu = 0, li = 0;                // next unit to load, and its number in the order of use (0 .. 2 total - 1)
    uint32_t lslot = 0;
    int newest = 0;                    // the newest issue(): 1 keys of a whole unit, 2 keys and values of one, 0 anything else
    auto issue = [&]() {
        newest = 0;
        if (li >= 2 * total) return;
        const bool with_v = li >= total, full = (lu + 1) * MHA8_UNIT <= S;
#pragma unroll
        for (int i = 0; i < D32; ++i) {
            const int ld = i * 4 + wave;
            const bool is_v = ld >= 2 * D32;
            if (is_v && !with_v) continue;
            const long long rs = is_v ? vss : kss;
            const uint8_t* g = (is_v ? vbase : kbase) + (long long)(lu * MHA8_UNIT) * rs;
            const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds0 + (is_v ? MHA8_SLOTS * U + (ld - 2 * D32) * 1024 : ld * 1024) + lslot);
            if (full && !a.far) {
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(voff[i]), "s"(g) : "memory", "m0");
                continue;
            }
            int l = lane;
            asm volatile("" : "+v"(l));  // nothing of this rare branch is kept in registers across the main loop
            const int p = (ld - (is_v ? 2 * D32 : 0)) * 64 + l, r = p / B::CH;
            if (lu * MHA8_UNIT + r < S) {
                const uint8_t* gl = g + r * rs + ((p % B::CH) ^ (is_v ? B::vswz(r) : B::kswz(r))) * 16;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(gl) : "memory", "m0");
            } else {  // rows beyond the sequence are zero
                *(mha8_lds_v4i*)(uintptr_t)(m0 + l * 16) = (v4i){l >> 6, l >> 6, l >> 6, l >> 6};
            }
        }
        if (full) newest = with_v ? 2 : 1;
        lslot = lslot == 2 * U ? 0 : lslot + U;
        ++li;
        lu = li == total ? first_unit : next_unit(lu);
    };
    // Before unit i is used: its loads were issued two steps ago; those of the step before may still be under way, D32 per
    // wavefront with values, at least D32 / 2 without.
    auto arrive = [&]() {
        if (newest == 2) mha8_wait_and_meet<D32>();
        else if (newest == 1) mha8_wait_and_meet<D32 / 2>();
        else mha8_wait_and_meet<0>();
    };
    // Units 0 and 1, which hardly ever turn out not to count, while the mask is looked at; once more if they do not.
    // (The code is kept short here and below, one copy of each part: small calls wait for instructions more than for data.)
    for (bool known = !whole;; known = true) {
#pragma unroll 1
        for (int i = 0; i < 2; ++i) issue();
        if (known) break;
        if (!a.mask && near) {  // every unit counts, and only the last can have addends (read behind later barriers)
            odd0 = S - (n - 1) * MHA8_UNIT < 32 ? 1ull << (n - 1) : 0;
            odd1 = S % MHA8_UNIT ? 1ull << (n - 1) : 0;
            if (S % MHA8_UNIT && tid < MHA8_UNIT) add[(n - 1) * MHA8_UNIT + tid] = (n - 1) * MHA8_UNIT + tid < S ? 0.0f : -INFINITY;
            break;
        }
        fill(0, add_keys);
        read_kinds();
        total = __builtin_popcountll(counts);
        first_unit = __builtin_ctzll(counts);
        if ((counts & 3) == (n > 1 ? 3u : 1u)) {
            lu = total > 2 ? next_unit(1) : first_unit;  // as issue() would have left it
            break;
        }
        mha8_wait_and_meet<0>();
        lu = first_unit, li = 0, lslot = 0;
    }

    // ---- operand addresses in the first slot
    const uint32_t kaddr = lds0 + col * D;  // + the piece's position
    const int ksw = B::kswz(col), tr = (lane & 15) >> 1;
    // row that this lane supplies to the transposing read: key 8 (tr / 4) + 4 h + tr % 4 of a group (+ 16 in the second read)
    const int vrow = 8 * (tr >> 2) + 4 * h + (tr & 3);
    const uint32_t vaddr = lds0 + MHA8_SLOTS * U + vrow * D + (lane & 1) * 8;
    const int vpiece = ((lane >> 4) & 1) ^ B::vswz(vrow);
    auto scores = [&](uint32_t slot, int g) {  // rows = keys 32 g .. 32 g + 31 of the unit, columns = queries
        v16i s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0;
#pragma unroll
        for (int i = 0; i < D32; ++i) {
            const v4i kf = *(const mha8_lds_v4i*)(uintptr_t)(kaddr + slot + g * 32 * D + (((2 * i + h) ^ ksw) * 16));
            s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf, qreg[i], s, 0, 0, 0);
        }
        return s;
    };
    auto read_addends = [&](int u, int g, v4f (&mk)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            mk[q] = *(const mha8_lds_v4f*)(add + ((u * MHA8_UNIT & (MHA8_LDS_KEYS - 1)) + g * 32 + 8 * q + 4 * h));
    };
    auto odd = [&](int u, int g) { return (((g ? odd1 : odd0) >> (u & 63)) & 1) != 0; };

    // longer sequences: the next MHA8_LDS_KEYS addends (no wavefront reads the last ones any more)
    auto turn = [&](int u) {
        if (whole || u % (MHA8_LDS_KEYS / MHA8_UNIT) != 0) return;
        const int left = (n - u) * MHA8_UNIT;
        fill(u * MHA8_UNIT, left < MHA8_LDS_KEYS ? left : MHA8_LDS_KEYS);
        read_kinds();
    };

    // ---- pass 1: the row maximum
    uint32_t slot = 0;
    int imax = -2147483647 - 1;
    float fmx = -INFINITY;
    int u = first_unit;
#pragma unroll 1
    for (int i = 0; i < total; ++i) {
        arrive();
        issue();
        turn(u);
        v16i s[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) s[g] = scores(slot, g);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (!odd(u, g)) {
#pragma unroll
                for (int r = 0; r < 16; ++r) imax = s[g][r] > imax ? s[g][r] : imax;
            } else {
                v4f mk[4];
                read_addends(u, g, mk);
#pragma unroll
                for (int r = 0; r < 16; ++r) fmx = fmaxf(fmx, __builtin_fmaf((float)s[g][r], a.c1, mk[r >> 2][r & 3]));
            }
        }
        slot = slot == 2 * U ? 0 : slot + U;
        u = next_unit(u);
    }
    if (imax != -2147483647 - 1) fmx = fmaxf(fmx, (float)imax * a.c1);
    const float row_max = fmaxf(fmx, other_half_f(fmx));  // finite: key 0 exists
    const float k0 = 6.98868468677216586f - row_max;      // log2(127) - the maximum

    // ---- pass 2: numerators, quantized, and the second product
    v16i oacc[D32];
#pragma unroll
    for (int d = 0; d < D32; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0;
    uint32_t row_sum = 0;  // this lane's keys only; the halves are added at the end
    u = first_unit;
#pragma unroll 1
    for (int i = 0; i < total; ++i) {
        arrive();
        issue();
        turn(u);
        v16i s[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) s[g] = scores(slot, g);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            v4i vf[D32];
#pragma unroll
            for (int d = 0; d < D32; ++d) {
                const uint32_t at = vaddr + slot + g * 32 * D + (((2 * d) ^ vpiece) * 16);
                const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((mha8_lds_v2i*)(uintptr_t)at);
                const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((mha8_lds_v2i*)(uintptr_t)(at + 16 * D));
                vf[d] = (v4i){lo[0], lo[1], hi[0], hi[1]};
            }
            uint32_t dw[4];
            auto numerators = [&](auto with_mask_c) {
                v4f mk[4];
                if constexpr (decltype(with_mask_c)::value) read_addends(u, g, mk);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t w = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x;  // in [0, 127]; a key past the end: 0
                        if constexpr (decltype(with_mask_c)::value)
                            x = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[g][4 * q + e], a.c1, mk[q][e]) - row_max) * 127.0f;
                        else
                            x = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[g][4 * q + e], a.c1, k0));
                        w = __builtin_amdgcn_cvt_pk_u8_f32(x, e, w);  // round to nearest even
                    }
                    dw[q] = w;
                    row_sum = __builtin_amdgcn_sad_u8(w, 0u, row_sum);  // + the four bytes
                }
            };
            if (!odd(u, g)) numerators(std::integral_constant<bool, false>{});
            else numerators(std::integral_constant<bool, true>{});
            const v4i pw = {(int)dw[0], (int)dw[1], (int)dw[2], (int)dw[3]};
#pragma unroll
            for (int d = 0; d < D32; ++d) oacc[d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[d], pw, oacc[d], 0, 0, 0);
        }
        slot = slot == 2 * U ? 0 : slot + U;
        u = next_unit(u);
    }

    // ---- normalise, requantize, store: after the half exchange a lane holds 16 consecutive channels of its query
    const int sum = (int)row_sum + other_half_i((int)row_sum);
    const float lf = (float)sum;
    uint8_t* op = a.o + b * a.so[0] + hd * a.so[1] + (long long)query * a.so[2];
#pragma unroll
    for (int d = 0; d < D32; ++d) {
        uint32_t dw[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float tt = ((float)oacc[d][4 * g + e] / lf) * a.r;
                const int qi = (int)__builtin_rintf(fminf(fmaxf(tt, -128.0f), 127.0f));
                w |= ((uint32_t)qi & 0xffu) << (8 * e);
            }
            dw[g] = w;
        }
        swap32_i8(dw[0], dw[2]);
        swap32_i8(dw[1], dw[3]);
        if (query < S) *(v4i*)(op + d * 32 + 16 * h) = (v4i){(int)dw[0], (int)dw[2], (int)dw[1], (int)dw[3]};
    }
}

namespace {

bool stride_ok_i8(const int64_t s[3]) {
    for (int i = 0; i < 3; ++i)
        if (s[i] < 0 || s[i] % 16 != 0) return false;
    return true;
}

// The ring, the addends, the units' kinds: at most 66 KiB (head_dim 128, 4096 keys and more).
template <int D32> void launch_i8(const MhaI8Args& a, bool stream, dim3 grid, hipStream_t s) {
    if (!stream) {
        hipLaunchKernelGGL((ogc_mha_i8_kernel<D32>), grid, dim3(256), 0, s, a);
        return;
    }
    const int keys = (a.seq + MHA8_UNIT - 1) / MHA8_UNIT * MHA8_UNIT;
    const size_t lds = Mha8<D32>::RING + (size_t)(keys < MHA8_LDS_KEYS ? keys : MHA8_LDS_KEYS) * 4 + 64 * 4;
    if (lds > 65536) {  // said at every such launch: the limit belongs to the current device
        if (hipFuncSetAttribute((const void*)ogc_mha_i8_stream_kernel<D32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return;  // reported by the caller
    }
    hipLaunchKernelGGL((ogc_mha_i8_stream_kernel<D32>), grid, dim3(256), lds, s, a);
}

// The streaming kernel or the plain one.  The former does less per score and starts slower (three times the code, the
// mask looked at before the first score), about 2 us on a launch that does not fill the chip.  Measured both ways, plain /
// streaming, us, batch x heads x seq, padding mask:
//   d = 64:  1x16x64 5.3 / 6.8;  64x12x64 8.9 / 9.6;  256x12x64 26.5 / 25.7;  32x12x128 9.2 / 9.9;  128x12x128 22.9 / 21.0;
//            8x8x256 9.6 / 10.2;  32x12x197 18.5 / 15.1;  1x8x384 12.0 / 10.0;  8x8x384 12.6 / 12.5;  128x16x512 241 / 171
//   d = 128: 8x12x64 7.8 / 8.3;  1x16x128 10.2 / 9.8;  32x12x128 15.5 / 14.2;  8x8x384 21.4 / 17.4;  128x8x384 167 / 105
bool stream_case(const ogc_mha_desc* d) {
    const int64_t tiles = (int64_t)d->batch * d->heads * ((d->seq + 127) / 128);
    return d->seq >= (d->head_dim >= 96 ? 128 : 320) || tiles * d->seq >= 128 * 1024;
}

}  // namespace

extern "C" {

ogc_status ogc_mha_i8_validate(const ogc_mha_desc* d, const ogc_mha_quant* qp) {
    if (!d || !qp) return OGC_ERR_INVALID_ARG;
    if (d->dtype != OGC_I8) return OGC_ERR_INVALID_ARG;
    if (d->softmax != OGC_SOFTMAX_STABLE && d->softmax != OGC_SOFTMAX_FAST) return OGC_ERR_INVALID_ARG;
    if (!isfinite(d->scale)) return OGC_ERR_INVALID_ARG;
    const float sc[4] = {qp->q_scale, qp->k_scale, qp->v_scale, qp->o_scale};
    for (int i = 0; i < 4; ++i)
        if (!(sc[i] > 0.0f) || !isfinite(sc[i])) return OGC_ERR_INVALID_ARG;
    if (d->batch <= 0 || d->heads <= 0 || d->seq <= 0 || d->head_dim <= 0) return OGC_ERR_SHAPE;
    if (d->seq > 65536 || (int64_t)d->batch * d->heads > 65535) return OGC_ERR_SHAPE;
    // the numerators are quantized against the row maximum: without the max reduction they have no fixed range
    if (d->softmax == OGC_SOFTMAX_FAST) return OGC_ERR_UNSUPPORTED;
    if (d->head_dim != 32 && d->head_dim != 64 && d->head_dim != 96 && d->head_dim != 128) return OGC_ERR_UNSUPPORTED;
    if (!stride_ok_i8(d->q_stride) || !stride_ok_i8(d->k_stride) || !stride_ok_i8(d->v_stride) || !stride_ok_i8(d->o_stride))
        return OGC_ERR_ALIGNMENT;
    return OGC_OK;
}

ogc_status ogc_mha_run_i8(const ogc_mha_desc* d, const ogc_mha_quant* qp, const void* q, const void* k, const void* v,
                          const float* mask, void* o, void* stream) {
    const ogc_status st = ogc_mha_i8_validate(d, qp);
    if (st != OGC_OK) return st;
    if (!q || !k || !v || !o) return OGC_ERR_INVALID_ARG;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return OGC_ERR_ALIGNMENT;
    if ((uintptr_t)mask & 3) return OGC_ERR_ALIGNMENT;
    MhaI8Args a;
    a.q = (const uint8_t*)q;
    a.k = (const uint8_t*)k;
    a.v = (const uint8_t*)v;
    a.mask = mask;
    a.o = (uint8_t*)o;
    for (int i = 0; i < 3; ++i) {
        a.sq[i] = d->q_stride[i];
        a.sk[i] = d->k_stride[i];
        a.sv[i] = d->v_stride[i];
        a.so[i] = d->o_stride[i];
    }
    a.batch = d->batch;
    a.heads = d->heads;
    a.seq = d->seq;
    a.q_tiles = (d->seq + 127) / 128;
    const int bh = d->batch * d->heads;
    a.xcd_order = (bh % 8 == 0) ? 1 : 0;
    auto magic = [](uint64_t m, uint64_t v) { return v == 1 || m * v >= 1ull << 32 ? 0u : (uint32_t)((1ull << 32) / v + 1); };  // exact there
    a.tiles_magic = magic((uint64_t)bh * a.q_tiles, a.q_tiles);
    a.heads_magic = magic(bh, d->heads);
    a.far = a.sk[2] > (1ll << 31) / MHA8_UNIT || a.sv[2] > (1ll << 31) / MHA8_UNIT;
    a.c1 = ((qp->q_scale * qp->k_scale) * d->scale) * 1.44269504088896340736f;  // fp32 products, left to right
    a.r = qp->v_scale / qp->o_scale;                                             // one fp32 division
    const dim3 grid((unsigned)(bh * a.q_tiles));
    hipStream_t s = (hipStream_t)stream;
    switch (d->head_dim / 32) {
    case 1: launch_i8<1>(a, stream_case(d), grid, s); break;
    case 2: launch_i8<2>(a, stream_case(d), grid, s); break;
    case 3: launch_i8<3>(a, stream_case(d), grid, s); break;
    default: launch_i8<4>(a, stream_case(d), grid, s); break;
    }
    return hipGetLastError() == hipSuccess ? OGC_OK : OGC_ERR_DEVICE;
}

const char* ogc_mha_i8_kernel_name(const ogc_mha_desc* d) {
    if (!d || d->dtype != OGC_I8) return nullptr;
    if (d->batch > 0 && d->heads > 0 && d->seq > 0 && stream_case(d)) {
        switch (d->head_dim) {
        case 32: return "ogc_mha_i8_stream_kernel<1>";
        case 64: return "ogc_mha_i8_stream_kernel<2>";
        case 96: return "ogc_mha_i8_stream_kernel<3>";
        case 128: return "ogc_mha_i8_stream_kernel<4>";
        }
    }
    switch (d->head_dim) {
    case 32: return "ogc_mha_i8_kernel<1>";
    case 64: return "ogc_mha_i8_kernel<2>";
    case 96: return "ogc_mha_i8_kernel<3>";
    case 128: return "ogc_mha_i8_kernel<4>";
    }
    return nullptr;
}

}  // extern "C"
