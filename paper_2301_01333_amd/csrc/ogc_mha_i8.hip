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

#include "ogc_lds_limit.h"
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
    int key_slots;  // streaming kernel: units of keys that LDS holds
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

// The plain kernel: keys and values through registers, both passes over 64-key blocks.  For launches of 32 and 64 channels that
// do not fill the chip (stream_case below).  D32 = head_dim / 32.  Key blocks of 64 (two 32-key groups).
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
constexpr int MHA8_VSLOTS = 3;       // units of values in LDS: one in use, two on their way
constexpr float MHA8_NEAR = 8192.0f; // scores (base-2 domain) that may go without an addend

template <int D32> struct Mha8 {
    static constexpr int D = D32 * 32, CH = D / 16;  // bytes and 16-byte pieces of a row
    static constexpr int UNIT_BYTES = MHA8_UNIT * D;
    static constexpr int RESIDENT = D32 == 1 ? 6 : D32 == 2 ? 5 : D32 == 3 ? 4 : 3;  // workgroups that the registers of a compute unit hold
    // Position of piece c of row r inside the row: c ^ swz(r).  LDS takes a 16-byte read in groups of 16 lanes and has 64 banks:
    // a read of the first product takes the same piece of sixteen consecutive keys, one of the second (byte transpose) 16-byte
    // pieces of the keys 8 a + 4 h + (0..3), a = 0, 1.  With these permutations, for rows of 32, 64, 96 and 128 bytes, the
    // former takes 4.1 clocks (8.0 with the pieces of eight keys apart), the latter 3.4 to 4.1.
    static __device__ __forceinline__ int kswz(int r) { return D32 == 4 ? ((r >> 1) & 7) : D32 == 2 ? ((r >> 2) & 3) : ((r >> 3) & 1); }
    static __device__ __forceinline__ int vswz(int r) {
        return D32 == 4 ? ((r & 3) | ((r >> 1) & 4)) : D32 == 2 ? (((r >> 1) & 1) | ((r >> 2) & 2)) : ((r >> 3) & 1);
    }
};

// All but the n newest loads have landed (or a few more), LDS accesses are done, then the workgroup meets.
MHA8_DEV void mha8_wait_and_meet(int n) {
    if (n >= 4) {
        if (n >= 18) asm volatile("s_waitcnt vmcnt(18)" ::: "memory");
        else if (n >= 12) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else if (n >= 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else if (n >= 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    } else if (n >= 2) {
        if (n == 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    } else {
        if (n == 1) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The streaming kernel.  D32 = head_dim / 32.
//
// What bounds it, and what follows from that: the vector ALU (65 % of the SIMDs' cycles at 128 x 16 x 512 x 64, 49 % at 128 x 8 x
// 384 x 128; the matrix pipe 20 to 25 %), the way of the first keys from HBM, and how many workgroups a compute unit has to
// cover that with.  Per score it owes a conversion, a multiply-add, an exponential and a packing conversion in the second pass.
//   * Keys and values go from global memory straight into LDS; V^T leaves it through the transposing read
//     (ds_read_b64_tr_b8: 8 keys x 16 channels per 16 lanes, the keys' rows chosen by the lanes' addresses).
//   * The first half of the keys, the queries and the mask are asked for at once; then all keys for which LDS has slots.
//     Where that is all that count, the second pass finds them there and loads values only.  Slots for 128 channels and 384 tokens: three
//     workgroups on a compute unit 192 keys each, two 384, one 1024.
//   * Registers are kept to 80 / 96 / 128 / 168 (32 / 64 / 96 / 128 channels) for 6 / 5 / 4 / 3 workgroups on a compute unit
//     (Mha8::RESIDENT): one group of 32 keys at a time in the second pass, one place where its product is taken, so that the
//     accumulators stay in place.  96 channels miss their 128 by three registers, spilled between the passes; the build sees to it
//     that no loop reloads one.  128 channels in 128 registers for four: 88 -> 103 us, slots for two units of keys only.
//     Workgroups of six or eight wavefronts share their loads among more queries and are slower all the same: six leave two
//     SIMDs with a wavefront too many for a second workgroup (131 us), eight of 128 channels spill (109).
//   * A group of 32 keys whose mask entries are all zero (most of them) takes its maximum over the integer scores, two
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
// Measured (same card, padding masks of half the length to all of it, inputs from HBM; two workgroups on a compute unit, slots for
// three units of keys, keys twice, a division per output / this): batch 128 x 8 heads x 384 tokens x 128: 125 -> 88 us (619 ->
// 880 TOP/s); 128 x 16 x 512 x 64: 189 -> 166; 16 x 8 x 1024 x 96: 79 -> 60; 64 x 8 x 384 x 32: 32.7 -> 26.1; 1 x 8 x 384 x 128: 16.3 -> 14.8.
// Without any arithmetic over the keys 62 of the 88 us are left: loads, barriers, a workgroup's start and its end.
// Both passes in one loop body (less code) was 15 % slower: the accumulators of the second live through the first.
template <int D32> __global__ __launch_bounds__(256, Mha8<D32>::RESIDENT) void ogc_mha_i8_stream_kernel(MhaI8Args a) {
    typedef Mha8<D32> B;
    constexpr int D = B::D, U = B::UNIT_BYTES;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    mha8_lds_u8* const lds = (mha8_lds_u8*)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = 4, threads = NW * 64, PW = (2 * D32 + NW - 1) / NW;  // PW: 1 KiB loads of a wavefront for a unit's keys (or values)
    // each XCD takes a contiguous run of (batch, head) pairs: the query tiles of a pair share its L2
    const uint32_t wg = blockIdx.x, lin = a.xcd_order ? (wg & 7) * (gridDim.x >> 3) + (wg >> 3) : wg;
    const int bh = a.tiles_magic ? __umulhi(lin, a.tiles_magic) : lin / a.q_tiles, qt = (int)lin - bh * a.q_tiles;
    const int b = a.heads_magic ? __umulhi(bh, a.heads_magic) : bh / a.heads, hd = bh - b * a.heads, S = a.seq;
    const int n = (S + MHA8_UNIT - 1) / MHA8_UNIT;
    const uint8_t* kbase = a.k + b * a.sk[0] + hd * a.sk[1];
    const uint8_t* vbase = a.v + b * a.sv[0] + hd * a.sv[1];
    const long long kss = a.sk[2], vss = a.sv[2];
    const uint32_t ring = (uint32_t)a.key_slots * U;  // bytes of the keys' slots; the values' follow

    // this lane's query row as the second operand of the first product: bytes 32 i + 16 h .. + 15 of the row
    const bool idle = (qt * 4 + wave) * 32 >= S;  // (loads its share and meets the others)
    const int query = (qt * 4 + wave) * 32 + col;
    v4i qreg[D32];
    {
        const int qrow = query < S ? query : S - 1;
        const uint8_t* qp = a.q + b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2];
#pragma unroll
        for (int i = 0; i < D32; ++i) qreg[i] = *(const v4i*)(qp + i * 32 + h * 16);
    }
    // ... and the first of the mask
    const float* const mrow = a.mask + (long long)b * S;
    float mfirst[4];
    auto read_mask = [&](int from, float (&t)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = a.mask && from + tid + threads * i < S ? mrow[from + tid + threads * i] : 0.0f;
    };
    read_mask(0, mfirst);

    // ---- direct loads.  A unit's keys are 2 * D32 KiB, dealt round the wavefronts from the first on, its values from the last.
    // Load m covers the pieces 64 m + lane of the unit's LDS image.
    const int first[2] = {wave, NW - 1 - wave};  // this wavefront's first load of a unit's keys, values
    uint32_t voff[2][PW];  // byte offset of the lane's piece from the unit's first row; !a.far: it fits 32 bits
#pragma unroll
    for (int is_v = 0; is_v < 2; ++is_v)
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const int p = (first[is_v] + i * NW) * 64 + lane, r = p / B::CH;
            voff[is_v][i] = (uint32_t)r * (uint32_t)(is_v ? vss : kss) + ((p % B::CH) ^ (is_v ? B::vswz(r) : B::kswz(r))) * 16;
        }
    int loads = 0;  // direct loads of this wavefront so far
    auto load = [&](int is_v, int unit, uint32_t slot) {
        const long long rs = is_v ? vss : kss;
        const uint8_t* g = (is_v ? vbase : kbase) + (long long)(unit * MHA8_UNIT) * rs;
        const bool full = (unit + 1) * MHA8_UNIT <= S;
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const int ld = first[is_v] + i * NW;
            if (ld >= 2 * D32) break;
            const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds0 + slot + ld * 1024);
            if (full && !a.far) {
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(voff[is_v][i]), "s"(g) : "memory", "m0");
                ++loads;  // (not so below, where no lane may take part: such a load is awaited with those after it)
                continue;
            }
            int l = lane;
            asm volatile("" : "+v"(l));  // nothing of this rare branch is kept in registers across the main loop
            const int p = ld * 64 + l, r = p / B::CH;
            if (unit * MHA8_UNIT + r < S) {
                const uint8_t* gl = g + r * rs + ((p % B::CH) ^ (is_v ? B::vswz(r) : B::kswz(r))) * 16;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(gl) : "memory", "m0");
            } else {  // rows beyond the sequence are zero
                *(mha8_lds_v4i*)(uintptr_t)(m0 + l * 16) = (v4i){l >> 6, l >> 6, l >> 6, l >> 6};
            }
        }
    };

    // ---- addends (mask in the base-2 domain, -infinity beyond the sequence), what kind of group they make, which units count
    mha8_lds_f32* const add = (mha8_lds_f32*)(lds + ring + MHA8_VSLOTS * U);
    const int add_keys = n * MHA8_UNIT < MHA8_LDS_KEYS ? n * MHA8_UNIT : MHA8_LDS_KEYS;
    // per unit: bits 0, 1: groups with a nonzero addend; bit 2: an addend that counts beside one of 0 or more; bit 3: one of those
    mha8_lds_u32* const kinds = (mha8_lds_u32*)(add + add_keys);
    const float floor = a.c1 > 0.0f ? -(2.0f * 16384.0f * D * a.c1 + 16.0f) : -INFINITY;
    // a scale that is not positive does not keep the order of the scores, a large one not the precision of the short form
    const bool near = a.c1 > 0.0f && 16384.0f * D * a.c1 <= MHA8_NEAR;
    auto fill = [&](int from, int count, float (&t)[4]) {  // keys from .. from + count - 1 (whole units, at most MHA8_LDS_KEYS); t: their first
#pragma unroll 1
        for (int f = from; f < from + count; f += 4 * threads) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = f + tid + threads * i;  // a wavefront has one unit at a time
                if (j >= from + count) break;
                const float v = j < S ? base2_mask(t[i]) : -INFINITY;
                add[j & (MHA8_LDS_KEYS - 1)] = v;
                const uint64_t nz = __builtin_amdgcn_ballot_w64(v != 0.0f), on = __builtin_amdgcn_ballot_w64(!(v < floor));
                const uint64_t top = __builtin_amdgcn_ballot_w64(v >= 0.0f);
                if (lane == 0)
                    kinds[(j / MHA8_UNIT) & 63] = ((uint32_t)nz ? 1u : 0u) | ((uint32_t)(nz >> 32) ? 2u : 0u) | (on ? 4u : 0u) | (top ? 8u : 0u);
            }
            if (f + 4 * threads < from + count) read_mask(f + 4 * threads, t);
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

    // ---- the order of use: the keys of the units that count, and once more if they do not all stay in LDS, then (with the
    // second round) the values.  Use j of the keys is in slot j mod key_slots, use j of the values in slot j mod MHA8_VSLOTS.
    int ku = 0, kj = 0, kuses = 1 << 30, vu = 0, vj = 0;  // next to load, its number in the order, and how many there are
    uint32_t kslot = 0, vslot = 0;
    int kstamp = 0, vstamp = 0;  // lane j mod 64: `loads` behind use j
    auto load_keys = [&]() {
        if (kj >= kuses) return;
        load(0, ku, kslot);
        kstamp = lane == (kj & 63) ? loads : kstamp;
        kslot = kslot + U == ring ? 0 : kslot + U;
        ++kj;
        ku = kj == total ? first_unit : next_unit(ku);
    };
    auto load_values = [&]() {
        if (vj >= total) return;
        load(1, vu, ring + vslot);
        vstamp = lane == (vj & 63) ? loads : vstamp;
        vslot = vslot == (MHA8_VSLOTS - 1) * U ? 0 : vslot + U;
        ++vj;
        vu = next_unit(vu);
    };
    // The first half of the units, which hardly ever turn out not to count, while the mask is on its way; once more if they do not.
    // (One copy of each part: small calls wait for instructions more than for data.)
    const int half = n < 3 ? n : (n + 1) / 2, ahead = half < a.key_slots ? half : a.key_slots;
#pragma unroll 1
    for (int i = 0; i < ahead; ++i) load_keys();

#pragma unroll
    for (int i = 0; i < D32; ++i) asm volatile("" : "+v"(qreg[i]));  // (awaited here, not behind all loads below)
    if (!a.mask && near && whole) {  // every unit counts, and only the last can have addends (read behind later barriers)
        odd0 = S - (n - 1) * MHA8_UNIT < 32 ? 1ull << (n - 1) : 0;
        odd1 = S % MHA8_UNIT ? 1ull << (n - 1) : 0;
        if (S % MHA8_UNIT && tid < MHA8_UNIT) add[(n - 1) * MHA8_UNIT + tid] = (n - 1) * MHA8_UNIT + tid < S ? 0.0f : -INFINITY;
    } else if (whole) {
        fill(0, add_keys, mfirst);
        read_kinds();
        total = __builtin_popcountll(counts);
        first_unit = __builtin_ctzll(counts);
        if ((~counts & ((2ull << (ahead - 1)) - 1)) == 0) {
            ku = next_unit(ahead - 1);  // as load_keys() would have left it
        } else {
            mha8_wait_and_meet(0);
            ku = first_unit, kj = 0, kslot = 0;
        }
        vu = first_unit;
    }
    const bool stay = total <= a.key_slots;  // one round of loads for the keys
    kuses = stay ? total : 2 * total;
    if (kj >= total) ku = first_unit;
#pragma unroll 1
    while (kj < (kuses < a.key_slots ? kuses : a.key_slots)) load_keys();

    // ---- operand addresses in the first slot
    const uint32_t kaddr = lds0 + col * D;  // + the piece's position
    const int ksw = B::kswz(col), tr = (lane & 15) >> 1;
    // row that this lane supplies to the transposing read: key 8 (tr / 4) + 4 h + tr % 4 of a group (+ 16 in the second read)
    const int vrow = 8 * (tr >> 2) + 4 * h + (tr & 3);
    const uint32_t vaddr = lds0 + ring + vrow * D + (lane & 1) * 8;
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
    auto read_addends = [&](int u, int g, int q) {  // of the keys 8 q + 4 h .. + 3 of the group
        return *(const mha8_lds_v4f*)(add + ((u * MHA8_UNIT & (MHA8_LDS_KEYS - 1)) + g * 32 + 8 * q + 4 * h));
    };
    auto odd = [&](int u, int g) { return (((g ? odd1 : odd0) >> (u & 63)) & 1) != 0; };

    // longer sequences: the next MHA8_LDS_KEYS addends (no wavefront reads the last ones any more)
    auto turn = [&](int u) {
        if (whole || u % (MHA8_LDS_KEYS / MHA8_UNIT) != 0) return;
        const int left = (n - u) * MHA8_UNIT;
        float t[4];
        read_mask(u * MHA8_UNIT, t);
        fill(u * MHA8_UNIT, left < MHA8_LDS_KEYS ? left : MHA8_LDS_KEYS, t);
        read_kinds();
    };

    // ---- pass 1: the row maximum.  Behind the barrier no wavefront reads the use before any more: its slot is loaded again.
    uint32_t slot = 0;
    int imax = -2147483647 - 1;
    float fmx = -INFINITY;
    int u = first_unit;
#pragma unroll 1
    for (int i = 0; i < total; ++i) {
        mha8_wait_and_meet(loads - __builtin_amdgcn_readlane(kstamp, i & 63));
        if (i) load_keys();
        if (i < MHA8_VSLOTS) load_values();
        turn(u);
        const uint32_t at_k = slot;
        const int at = u;
        slot = slot + U == ring ? 0 : slot + U;
        u = next_unit(u);
        if (idle) continue;
        v16i s[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) s[g] = scores(at_k, g);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (!odd(at, g)) {
#pragma unroll
                for (int r = 0; r < 16; ++r) imax = s[g][r] > imax ? s[g][r] : imax;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f mk = read_addends(at, g, q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) fmx = fmaxf(fmx, __builtin_fmaf((float)s[g][4 * q + e], a.c1, mk[e]));
                }
            }
        }
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
    if (stay) slot = 0;
    uint32_t vat = 0;
#pragma unroll 1
    for (int i = 0; i < total; ++i) {
        const int kst = stay ? 0 : __builtin_amdgcn_readlane(kstamp, (total + i) & 63), vst = __builtin_amdgcn_readlane(vstamp, i & 63);
        mha8_wait_and_meet(loads - (kst > vst ? kst : vst));
        load_keys();
        if (i) load_values();
        turn(u);
        const uint32_t at_k = slot, at_v = vat;
        const int at = u;
        slot = slot + U == ring ? 0 : slot + U;
        vat = vat == (MHA8_VSLOTS - 1) * U ? 0 : vat + U;
        u = next_unit(u);
        if (idle) continue;
        auto numerators = [&](int g, const v16i& s, auto with_mask_c) {
            constexpr int AT_ONCE = D32 == 4 ? 4 : D32 == 2 ? 1 : 2;  // quads of addends read together: as the registers allow
            v4i w4;
            v4f mk[AT_ONCE];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t w = 0;
                if constexpr (decltype(with_mask_c)::value) {
                    if (q % AT_ONCE == 0)
#pragma unroll
                        for (int x = 0; x < AT_ONCE; ++x) mk[x] = read_addends(at, g, q + x);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x;  // in [0, 127]; a key past the end: 0
                    if constexpr (decltype(with_mask_c)::value)
                        x = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[4 * q + e], a.c1, mk[q % AT_ONCE][e]) - row_max) * 127.0f;
                    else
                        x = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[4 * q + e], a.c1, k0));
                    w = __builtin_amdgcn_cvt_pk_u8_f32(x, e, w);  // round to nearest even
                }
                w4[q] = (int)w;
                if constexpr (decltype(with_mask_c)::value && AT_ONCE < 4) __builtin_amdgcn_sched_barrier(0);
                row_sum = __builtin_amdgcn_sad_u8(w, 0u, row_sum);  // + the four bytes
            }
            return w4;
        };
        auto second = [&](int g, const v4i& pw) {
#pragma unroll
            for (int d = 0; d < D32; ++d) {
                const uint32_t from = vaddr + at_v + g * 32 * D + (((2 * d) ^ vpiece) * 16);
                const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((mha8_lds_v2i*)(uintptr_t)from);
                const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((mha8_lds_v2i*)(uintptr_t)(from + 16 * D));
                oacc[d] = __builtin_amdgcn_mfma_i32_32x32x32_i8((v4i){lo[0], lo[1], hi[0], hi[1]}, pw, oacc[d], 0, 0, 0);
            }
        };
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const v16i s = scores(at_k, g);
            v4i pw;
            if (!odd(at, g)) pw = numerators(g, s, std::integral_constant<bool, false>{});
            else pw = numerators(g, s, std::integral_constant<bool, true>{});
            second(g, pw);
        }
    }
    if (idle) return;

    // ---- normalise, requantize, store: after the half exchange a lane holds 16 consecutive channels of its query.
    // float(A) / float(L) by the reciprocal: y = 1 / L rounded once, q = A y, q + (A - q L) y, the last two fused.  This is the
    // quotient rounded once, the division's own result: with u the unit in the last place of A / L and y = (1 + e) / L, q is within
    // 1.5 u, so the remainder is exact and the sum before its rounding is |A / L - q| |e| < 1.5 * 2^-24 u away from A / L, which
    // is more than u / 2 L away from any midpoint of two fp32 values.  For L below 2^22 that is enough (and up to 2^23, beyond the
    // longest sequence, it still holds: a q beside the midpoint leaves an error below 2^-24 u, and for one farther off |e| would
    // have to pass (1 - 1.5 * 2^-24) 2^-24, which no such L reaches).  As a division, 64 of them a lane, it was half of the
    // vector ALU's work at 384 tokens.  Longer sequences divide, with time to spare; without that second body the compiler of
    // the 96-channel kernel reloads a spilled register in the loop over the keys.
    const int sum = (int)row_sum + other_half_i((int)row_sum);
    const float lf = (float)sum, y = 1.0f / lf;
    uint8_t* op = a.o + b * a.so[0] + hd * a.so[1] + (long long)query * a.so[2];
    auto finish = [&](auto quotient) {
#pragma unroll
        for (int d = 0; d < D32; ++d) {
            uint32_t dw[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float tt = quotient((float)oacc[d][4 * g + e]) * a.r;
                    // + 1.5 * 2^23 rounds to an integer, to even at ties, whose low byte is that of the sum's bits
                    w[e] = __builtin_bit_cast(uint32_t, fminf(fmaxf(tt, -128.0f), 127.0f) + 12582912.0f);
                }
                dw[g] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(w[3], w[2], 0x0c0c0400u), __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0400u), 0x05040100u);
            }
            swap32_i8(dw[0], dw[2]);
            swap32_i8(dw[1], dw[3]);
            if (query < S) *(v4i*)(op + d * 32 + 16 * h) = (v4i){(int)dw[0], (int)dw[2], (int)dw[1], (int)dw[3]};
        }
    };
    if (S <= 32768) {
        finish([&](float x) {
            const float q = x * y;
            return __builtin_fmaf(__builtin_fmaf(-q, lf, x), y, q);
        });
    } else {
        finish([&](float x) { return x / lf; });
    }
}

namespace {

// A number below 2^32 / v times this, shifted right by 32, is it divided by v (0: divide).
uint32_t magic_i8(uint64_t m, uint64_t v) { return v == 1 || m * v >= 1ull << 32 ? 0u : (uint32_t)((1ull << 32) / v + 1); }

bool stride_ok_i8(const int64_t s[3]) {
    for (int i = 0; i < 3; ++i)
        if (s[i] < 0 || s[i] % 16 != 0) return false;
    return true;
}

constexpr size_t MHA8_CU_LDS = 160 * 1024;

// Bytes of LDS beside the keys' slots: the values' slots, the addends, the units' kinds.
template <int D32> size_t side_lds(int seq) {
    const int keys = (seq + MHA8_UNIT - 1) / MHA8_UNIT * MHA8_UNIT;
    return MHA8_VSLOTS * Mha8<D32>::UNIT_BYTES + (size_t)(keys < MHA8_LDS_KEYS ? keys : MHA8_LDS_KEYS) * 4 + 64 * 4;
}

template <int D32> void launch_i8(MhaI8Args& a, bool stream, unsigned tiles, hipStream_t s) {
    if constexpr (D32 <= 2) {
        if (!stream) {
            hipLaunchKernelGGL((ogc_mha_i8_kernel<D32>), dim3(tiles), dim3(256), 0, s, a);
            return;
        }
    }
    // As many slots for keys, up to all units (60: their stamps are lanes), as leave the LDS of a compute unit to the
    // workgroups that its registers hold, or to those that it gets if the launch has fewer; three at least.
    const int units = (a.seq + MHA8_UNIT - 1) / MHA8_UNIT, all = units < 60 ? units : 60;
    const size_t side = side_lds<D32>(a.seq);
    unsigned each = (tiles + 255) / 256;
    if (each > (unsigned)Mha8<D32>::RESIDENT) each = Mha8<D32>::RESIDENT;
    auto fit = [&]() { return (int)(((long long)(MHA8_CU_LDS / each) - (long long)side) / Mha8<D32>::UNIT_BYTES); };
    while (each > 1 && fit() < (all < 3 ? all : 3)) --each;
    a.key_slots = fit() < all ? fit() : all;
    const size_t lds = (size_t)a.key_slots * Mha8<D32>::UNIT_BYTES + side;
    if (lds > 65536) {  // raised to the same for all launches, once on a device (host time of a call 3.92 -> 3.89 us)
        static OgcLdsLimit limit;
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess) return;  // (errors are reported by the caller)
        const void* const kern = (const void*)ogc_mha_i8_stream_kernel<D32>;
        if (limit.raise(dev, MHA8_CU_LDS, [&]() { return (int)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)MHA8_CU_LDS); }) != 0) return;
    }
    hipLaunchKernelGGL((ogc_mha_i8_stream_kernel<D32>), dim3(tiles), dim3(256), lds, s, a);
}

// The streaming kernel or the plain one.  The former does less per score and starts slower (three times the code, the
// mask looked at before the first score), half a microsecond on a launch that does not fill the chip; with 96 and 128 channels the
// plain one's values, byte by byte into LDS, cost more than that in every launch.  With 32 and 64 channels one line through the
// sizes: near it either kernel is up to 8 % the better one (1x4x300 of 64 channels, 8x4x300 of 32 and 8x8x384 of 64 below are on the wrong
// side).  Measured both ways, plain / streaming, us, batch x heads x seq, padding mask:
//   d = 32:  16x16x100 6.8 / 7.3;  8x8x256 9.2 / 9.4;  32x12x128 8.7 / 8.2;  128x16x60 16.1 / 12.1;  8x4x300 10.6 / 10.3;  4x8x700 19.9 / 17.3
//   d = 64:  1x16x64 4.9 / 5.5;  32x8x48 5.5 / 6.1;  16x16x100 7.3 / 7.9;  8x8x256 9.8 / 10.2;  8x16x200 10.1 / 9.7;  32x12x128 10.6 / 9.8;
//            64x12x64 10.1 / 8.0;  16x16x256 15.4 / 13.5;  1x4x300 10.7 / 9.8;  1x8x384 12.3 / 12.0;  8x8x384 12.8 / 13.2
//   d = 96:  4x4x64 6.3 / 6.2;  1x4x100 7.9 / 7.5;  64x8x100 15.6 / 12.1;   d = 128:  1x4x48 7.0 / 6.6;  1x8x100 10.1 / 8.4;  8x8x384 22.8 / 16.8
bool stream_case(const ogc_mha_desc* d) {
    const int64_t tiles = (int64_t)d->batch * d->heads * ((d->seq + 127) / 128);
    return d->head_dim >= 96 || d->seq >= 320 || tiles * d->seq >= 40 * 1024;
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
    a.key_slots = 0;
    a.tiles_magic = magic_i8((uint64_t)bh * a.q_tiles, a.q_tiles);
    a.heads_magic = magic_i8(bh, d->heads);
    a.far = a.sk[2] > (1ll << 31) / MHA8_UNIT || a.sv[2] > (1ll << 31) / MHA8_UNIT;
    a.c1 = ((qp->q_scale * qp->k_scale) * d->scale) * 1.44269504088896340736f;  // fp32 products, left to right
    a.r = qp->v_scale / qp->o_scale;                                             // one fp32 division
    const unsigned tiles = (unsigned)(bh * a.q_tiles);
    hipStream_t s = (hipStream_t)stream;
    switch (d->head_dim / 32) {
    case 1: launch_i8<1>(a, stream_case(d), tiles, s); break;
    case 2: launch_i8<2>(a, stream_case(d), tiles, s); break;
    case 3: launch_i8<3>(a, stream_case(d), tiles, s); break;
    default: launch_i8<4>(a, stream_case(d), tiles, s); break;
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
    }
    return nullptr;
}

}  // extern "C"
