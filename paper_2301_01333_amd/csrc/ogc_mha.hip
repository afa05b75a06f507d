// Fused scaled dot-product attention for gfx950 (the MHA subgraph of Section VII / Table I): both batch
// matmuls, the scalar, the mask and the softmax in one kernel, scores never leaving the compute unit.
//
// One workgroup = 4 wavefronts = 128 queries of one (batch, head); a wavefront owns 32 queries (64, as two
// groups of 32, in the bf16 variant for head dimensions up to 64).  Keys and values stream through LDS 32 at a time
// (bf16: straight from global memory, see ogc_mha_bf16.h; fp32: prefetched one block ahead in registers).  Both products
// are computed TRANSPOSED so that a lane owns one query:
//
//   S^T[key][query] = K * Q^T     first MFMA operand = 32 keys x k from LDS, second = Q^T, held in registers
//   O^T[c][query]   = V^T * P^T   first operand = 32 channels x keys from LDS (V is transposed on its way into LDS,
//                                 or out of it), second = the softmax weights exactly where the first product left them
//
// In the 32x32 accumulator layout lane l holds column (query) l%32 and rows 8g + 4(l/32) + e, g,e = 0..3.  The
// softmax reductions of a query are therefore 16 values inside a lane plus one exchange with lane l^32, the
// running maximum / sum / rescale factors are per-lane scalars, and the weights feed the second product without
// any data movement: the reduction axis of that product (keys) may be summed in any order, so V^T is simply
// taken with its key index permuted to the order in which the accumulator registers hold the keys.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <atomic>
#include <type_traits>

#include "ogc_mha.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

#define MHA_DEV static __device__ __forceinline__

struct MhaArgs {
    const uint8_t* q;
    const uint8_t* k;
    const uint8_t* v;
    const float* mask;
    uint8_t* o;
    long long sq[3], sk[3], sv[3], so[3];  // element strides: batch, head, token
    int batch, heads, seq;
    int q_tiles;       // ceil(seq / queries per workgroup)
    int xcd_order;     // 1: workgroups of one (batch, head) are placed on one XCD
    uint32_t tiles_magic, heads_magic;  // bf16: reciprocals of q_tiles and heads for div_magic
    float scale_log2;  // scale * log2(e)
    float inv_scale;   // bf16, mask in LDS: 1 / scale, and the bound its quotient is held to
    float addend_max;
};

constexpr float LOG2E = 1.44269504088896340736f;

MHA_DEV void swap32(uint32_t& a, uint32_t& b) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
// value of x in the other half of the wavefront (lane ^ 32)
MHA_DEV float other_half(float x) {
    uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
    swap32(a, b);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? a : b);
}
MHA_DEV uint32_t pack_bf16(float lo, float hi) {  // round to nearest even, two values per register
    v2bf r = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, r);
}

// n / d; m = floor(2^32 / d) + 1 where that is exact for every n in use (n * d < 2^32, and d > 1), else 0
MHA_DEV uint32_t div_magic(uint32_t n, uint32_t d, uint32_t m) { return m ? __umulhi(n, m) : n / d; }

#include "ogc_mha_bf16.h"

constexpr int MHA_F32_KEYS = 32;    // keys per block of the fp32 body
constexpr int MHA_BF16_WHOLE = 64;  // a bf16 sequence of whole blocks of this many keys without a mask needs no addend

// The fp32 body.  PLAIN: no mask, whole key blocks and a positive scalar, so no key needs an addend.
template <int D32, int FAST, int PLAIN> MHA_DEV void mha_f32_body(const MhaArgs& a) {
    constexpr int KB = MHA_F32_KEYS, D = D32 * 32;
    constexpr int KSTR = D * 4 + 16;   // bytes per key row of K in LDS (padded)
    constexpr int VSTR = KB * 4 + 16;  // bytes per channel row of V^T in LDS (padded)
    constexpr int CH = D * 4 / 16;     // 16-byte chunks per token row
    constexpr int KU = KB * CH / 256;  // 16-byte chunks of K per thread
    constexpr int VU = D32;            // chunks of V per thread
    __shared__ __attribute__((aligned(16))) uint8_t k_lds[KB * KSTR];
    __shared__ __attribute__((aligned(16))) uint8_t vt_lds[D * VSTR];
    __shared__ __attribute__((aligned(16))) float m_lds[KB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, col = lane & 31;
    int bh, qt;
    if (a.xcd_order) {  // consecutive workgroup ids go round the 8 XCDs: keep one (batch, head) on one of them
        const int L = blockIdx.x, x = L & 7, r = L >> 3;
        bh = x + 8 * (r / a.q_tiles);
        qt = r % a.q_tiles;
    } else {
        bh = blockIdx.x / a.q_tiles;
        qt = blockIdx.x % a.q_tiles;
    }
    const int b = bh / a.heads, hd = bh % a.heads, S = a.seq;
    const uint8_t* kbase = a.k + (b * a.sk[0] + hd * a.sk[1]) * 4;
    const uint8_t* vbase = a.v + (b * a.sv[0] + hd * a.sv[1]) * 4;
    const long long kss = a.sk[2] * 4, vss = a.sv[2] * 4;

    // ---- this lane's query row as the second MFMA operand, resident for the whole kernel
    constexpr int QN = D / 8;
    const int query = (qt * 4 + wave) * 32 + col;
    v4i qreg[QN];
    v16f oacc[D32];
    float run_max = -INFINITY, run_sum = 0.0f;  // run_sum: this lane's keys only, halves are added at the end
    {
        const int qrow = query < S ? query : S - 1;
        const uint8_t* qp = a.q + (b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2]) * 4;
#pragma unroll
        for (int i = 0; i < QN; ++i) qreg[i] = *(const v4i*)(qp + i * 32 + h * 16);
#pragma unroll
        for (int d = 0; d < D32; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[d][r] = 0.0f;
    }

    // ---- prefetch registers for one block of keys / values / mask
    v4i kreg[KU], vreg[VU];
    float mreg = 0.0f;   // the mask value as loaded; scaled when it is written to LDS (scaling here would wait for the load,
                         // and with it for every key / value load issued just before)
    bool mpad = false;   // the key lies beyond the sequence
    auto prefetch = [&](int key0) {
        const bool full = key0 + KB <= S;  // uniform: every key of the block exists, no row needs a zero fill
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int u = tid + 256 * i, key = key0 + u / CH, part = u % CH;
            kreg[i] = (full || key < S) ? *(const v4i*)(kbase + key * kss + part * 16) : (v4i){0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < VU; ++i) {
            const int u = tid + 256 * i, key = key0 + (u & 31), c = u >> 5;
            vreg[i] = (full || key < S) ? *(const v4i*)(vbase + key * vss + c * 16) : (v4i){0, 0, 0, 0};
        }
        if (tid < KB) {
            const int key = key0 + tid;
            mpad = key >= S;
            mreg = 0.0f;
            if (!mpad && a.mask) mreg = a.mask[(long long)b * S + key];
        }
    };
    auto fill_lds = [&]() {
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int u = tid + 256 * i;
            *(v4i*)(k_lds + (u / CH) * KSTR + (u % CH) * 16) = kreg[i];
        }
#pragma unroll
        for (int i = 0; i < VU; ++i) {
            const int u = tid + 256 * i, kl = u & 31, c = u >> 5;
#pragma unroll
            for (int j = 0; j < 4; ++j) *(int*)(vt_lds + (4 * c + j) * VSTR + kl * 4) = vreg[i][j];
        }
        if (tid < KB) m_lds[tid] = mpad ? -INFINITY : mreg * LOG2E;
    };

    const int nkb = (S + KB - 1) / KB;
    prefetch(0);
    for (int kb = 0; kb < nkb; ++kb) {
        __syncthreads();  // every wavefront is done with the previous block
        fill_lds();
        __syncthreads();
        if (kb + 1 < nkb) prefetch((kb + 1) * KB);

        // ---- scores, transposed: rows = keys, columns = queries
        v16f sacc;
        {
            const v16f zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            const uint8_t* krow = k_lds + col * KSTR + h * 16;
#pragma unroll
            for (int i = 0; i < QN; ++i) {
                const v4f kf = *(const v4f*)(krow + i * 32), qf = __builtin_bit_cast(v4f, qreg[i]);
                sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.x, qf.x, i ? sacc : zero, 0, 0, 0);
                sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.y, qf.y, sacc, 0, 0, 0);
                sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.z, qf.z, sacc, 0, 0, 0);
                sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.w, qf.w, sacc, 0, 0, 0);
            }
        }
        // ---- scalar, mask, running maximum (base-2 logarithm domain; a key beyond the sequence carries
        // -infinity).  A block of valid keys without a mask needs no per-key addend: the maximum is taken on
        // the raw products and the scalar rides in the exponent's multiply-add.
        const float c = a.scale_log2;
        float cand = -INFINITY;
        if constexpr (PLAIN) {
            if constexpr (!FAST) {
#pragma unroll
                for (int r = 0; r < 16; ++r) cand = fmaxf(cand, sacc[r]);
                cand *= c;
            }
        } else {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f mk = *(const v4f*)(m_lds + 8 * g + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = __builtin_fmaf(sacc[4 * g + e], c, mk[e]);
                    sacc[4 * g + e] = t;
                    if constexpr (!FAST) cand = fmaxf(cand, t);
                }
            }
        }
        float off = 0.0f;
        if constexpr (!FAST) {
            // The reference point of the exponentials only has to be NEAR the maximum: it moves when a block
            // exceeds it by more than 2^8, so most blocks skip the rescaling of the output accumulators.  The
            // result is the same function (numerator and denominator carry the same factor); weights reach
            // 256 at most, far from any overflow.  Key 0 of block 0 is always valid: the first block sets it.
            cand = fmaxf(cand, other_half(cand));
            const bool need = cand > run_max + 8.0f;
            if (__builtin_amdgcn_ballot_w64(need) != 0) {
                const float new_max = need ? cand : run_max;
                const float alpha = __builtin_amdgcn_exp2f(run_max - new_max);
                run_max = new_max;
                run_sum *= alpha;
#pragma unroll
                for (int d = 0; d < D32; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
            }
            off = -run_max;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float x;
            if constexpr (PLAIN) x = __builtin_fmaf(sacc[r], c, off);
            else x = FAST ? sacc[r] : sacc[r] + off;
            sacc[r] = __builtin_amdgcn_exp2f(x);
        }
        // ---- O^T += V^T P^T
#pragma unroll
        for (int r = 0; r < 16; ++r) run_sum += sacc[r];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int d = 0; d < D32; ++d) {
                const v4f vv = *(const v4f*)(vt_lds + (d * 32 + col) * VSTR + (8 * g + 4 * h) * 4);
                oacc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv.x, sacc[4 * g], oacc[d], 0, 0, 0);
                oacc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv.y, sacc[4 * g + 1], oacc[d], 0, 0, 0);
                oacc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv.z, sacc[4 * g + 2], oacc[d], 0, 0, 0);
                oacc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv.w, sacc[4 * g + 3], oacc[d], 0, 0, 0);
            }
    }

    // ---- normalise and store: after the half exchange a lane holds 16 consecutive channels of its query
    const float total = run_sum + other_half(run_sum);
    const float inv = 1.0f / total;
    uint8_t* op = a.o + (b * a.so[0] + hd * a.so[1] + (long long)query * a.so[2]) * 4;
#pragma unroll
    for (int d = 0; d < D32; ++d) {
        uint32_t dw[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) dw[g][e] = __builtin_bit_cast(uint32_t, oacc[d][4 * g + e] * inv);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            swap32(dw[0][e], dw[2][e]);
            swap32(dw[1][e], dw[3][e]);
        }
        if (query < S) {
            uint8_t* dst = op + (d * 32 + 16 * h) * 4;
            const int order[4] = {0, 2, 1, 3};
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(v4i*)(dst + 16 * g) = (v4i){(int)dw[order[g]][0], (int)dw[order[g]][1], (int)dw[order[g]][2], (int)dw[order[g]][3]};
        }
    }
}

// Wavefronts per SIMD the registers are held to: one 32-query group with head_dim <= 64 fits three.
constexpr int mha_waves(int dt, int d32, int qs) { return dt == OGC_BF16 && qs == 1 && d32 <= 2 ? 3 : 2; }

// DT: OGC_F32 / OGC_BF16.  D32 = head_dim / 32.  FAST: softmax without the running maximum.  PLAIN: no mask, the
// sequence is a whole number of key blocks and the scalar is positive, so no key needs an addend.
// QS: 32-query groups per wavefront (1 or 2).  With 2, every key / value operand read from LDS feeds two matrix
// instructions (one per group).
template <int DT, int D32, int FAST, int PLAIN, int QS>
__global__ __launch_bounds__(256, mha_waves(DT, D32, QS)) void ogc_mha_kernel(MhaArgs a) {
    if constexpr (DT == OGC_BF16) {
        extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
        mha_bf16_body<D32, FAST, PLAIN ? MHA_NO_ADDEND : MHA_ADDEND_IN_LDS, QS>(a, (mha_lds_u8*)smem);
    } else {
        mha_f32_body<D32, FAST, PLAIN>(a);
    }
}

// bf16 calls that do not fit the other forms: scalars that are not positive or have no fp32 reciprocal, token strides
// beyond 32 bits of byte offset.
template <int D32, int FAST> __global__ __launch_bounds__(256, 2) void ogc_mha_general_kernel(MhaArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    mha_bf16_body<D32, FAST, MHA_ADDEND_GENERAL, 1>(a, (mha_lds_u8*)smem);
}

namespace {

// Bytes of LDS of a bf16 launch: the ring, and the addends where the mode keeps them there.
size_t bf16_lds(int d32, int seq, int plain) {
    const int keys = seq <= MHA_UNIT ? 2 * MHA_UNIT : (seq + MHA_UNIT - 1) / MHA_UNIT * MHA_UNIT;  // at least two units
    return (size_t)2 * 4 * MHA_UNIT * d32 * 64 + (plain ? 0 : (size_t)(keys < MHA_LDS_KEYS ? keys : MHA_LDS_KEYS) * 4);
}

// One launch with dynamic LDS; the limit is raised once per kernel that can ask for more than 64 KiB (head_dim 128: up to
// 80 KiB).  Two threads at once only repeat it.
template <int DT, int D32, int FAST, int PLAIN, int QS> hipError_t launch_one(const MhaArgs& a, dim3 grid, hipStream_t st) {
    auto kern = ogc_mha_kernel<DT, D32, FAST, PLAIN, QS>;
    const size_t lds = DT == OGC_BF16 ? bf16_lds(D32, a.seq, PLAIN) : 0;
    static std::atomic<bool> raised{false};
    if (lds > 65536 && !raised.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)bf16_lds(D32, MHA_LDS_KEYS, PLAIN));
        if (e != hipSuccess) return e;
        raised.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, a);
    return hipGetLastError();
}
template <int DT, int D32, int QS> hipError_t launch_fast(int fast, int plain, const MhaArgs& a, dim3 grid, hipStream_t st) {
    if (fast && plain) return launch_one<DT, D32, 1, 1, QS>(a, grid, st);
    if (fast) return launch_one<DT, D32, 1, 0, QS>(a, grid, st);
    if (plain) return launch_one<DT, D32, 0, 1, QS>(a, grid, st);
    return launch_one<DT, D32, 0, 0, QS>(a, grid, st);
}
template <int DT> hipError_t launch_dim(int d32, int qs, int fast, int plain, const MhaArgs& a, dim3 grid, hipStream_t st) {
    if (qs == 2) {  // bf16 with head_dim <= 64 only (query_groups)
        if constexpr (DT == OGC_BF16) return d32 == 1 ? launch_fast<DT, 1, 2>(fast, plain, a, grid, st) : launch_fast<DT, 2, 2>(fast, plain, a, grid, st);
    }
    switch (d32) {
    case 1: return launch_fast<DT, 1, 1>(fast, plain, a, grid, st);
    case 2: return launch_fast<DT, 2, 1>(fast, plain, a, grid, st);
    case 3: return launch_fast<DT, 3, 1>(fast, plain, a, grid, st);
    default: return launch_fast<DT, 4, 1>(fast, plain, a, grid, st);
    }
}
template <int D32> void launch_general_dim(int fast, const MhaArgs& a, dim3 grid, hipStream_t st) {
    if (fast) hipLaunchKernelGGL((ogc_mha_general_kernel<D32, 1>), grid, dim3(256), bf16_lds(D32, a.seq, 1), st, a);
    else hipLaunchKernelGGL((ogc_mha_general_kernel<D32, 0>), grid, dim3(256), bf16_lds(D32, a.seq, 1), st, a);
}
hipError_t launch_general(int d32, int fast, const MhaArgs& a, dim3 grid, hipStream_t st) {
    switch (d32) {
    case 1: launch_general_dim<1>(fast, a, grid, st); break;
    case 2: launch_general_dim<2>(fast, a, grid, st); break;
    case 3: launch_general_dim<3>(fast, a, grid, st); break;
    default: launch_general_dim<4>(fast, a, grid, st); break;
    }
    return hipGetLastError();
}

// no mask, whole key blocks only, positive scalar
bool plain_case(const ogc_mha_desc* d, const float* mask) {
    const int kb = d->dtype == OGC_BF16 ? MHA_BF16_WHOLE : MHA_F32_KEYS;
    return mask == nullptr && d->seq % kb == 0 && d->scale > 0.0f;
}

// bf16 calls that take the general kernel.  A lane's piece is addressed by 32 bits of byte offset from its unit's first
// row; the addend in LDS is the mask divided by the scalar.
bool general_case(const ogc_mha_desc* d, const float* mask) {
    if (d->dtype != OGC_BF16) return false;
    const int64_t most = (int64_t)1 << 31;
    if (d->k_stride[2] * 2 > most / MHA_UNIT || d->v_stride[2] * 2 > most / MHA_UNIT) return true;
    if (plain_case(d, mask)) return false;
    return !(d->scale >= 1e-30f && d->scale <= 1e30f);
}

// 32-query groups per wavefront.  Two where the registers allow it (bf16, head_dim <= 64) and the sequence is long
// enough to keep the four wavefronts of a workgroup busy: the bf16 kernel is then no longer bound by LDS reads.
int query_groups(const ogc_mha_desc* d) {
    const bool can = d->dtype == OGC_BF16 && d->head_dim <= 64;
    if (d->query_groups != 0) return (d->query_groups == 2 && can) ? 2 : 1;
    return (can && d->seq >= 256) ? 2 : 1;
}

bool stride_ok(const int64_t s[3], int elt) {
    for (int i = 0; i < 3; ++i)
        if (s[i] < 0 || (s[i] * elt) % 16 != 0) return false;
    return true;
}

}  // namespace

extern "C" {

ogc_status ogc_mha_validate(const ogc_mha_desc* d) {
    if (!d) return OGC_ERR_INVALID_ARG;
    if (d->dtype != OGC_F32 && d->dtype != OGC_BF16 && d->dtype != OGC_I8) return OGC_ERR_INVALID_ARG;
    if (d->softmax != OGC_SOFTMAX_STABLE && d->softmax != OGC_SOFTMAX_FAST) return OGC_ERR_INVALID_ARG;
    if (d->query_groups < 0 || d->query_groups > 2) return OGC_ERR_INVALID_ARG;
    if (!isfinite(d->scale)) return OGC_ERR_INVALID_ARG;
    if (d->batch <= 0 || d->heads <= 0 || d->seq <= 0 || d->head_dim <= 0) return OGC_ERR_SHAPE;
    if (d->seq > 65536 || (int64_t)d->batch * d->heads > 65535) return OGC_ERR_SHAPE;
    if (d->dtype == OGC_I8) return OGC_ERR_UNSUPPORTED;
    if (d->head_dim != 32 && d->head_dim != 64 && d->head_dim != 96 && d->head_dim != 128) return OGC_ERR_UNSUPPORTED;
    const int e = d->dtype == OGC_F32 ? 4 : 2;
    if (!stride_ok(d->q_stride, e) || !stride_ok(d->k_stride, e) || !stride_ok(d->v_stride, e) || !stride_ok(d->o_stride, e))
        return OGC_ERR_ALIGNMENT;
    return OGC_OK;
}

ogc_status ogc_mha_run(const ogc_mha_desc* d, const void* q, const void* k, const void* v, const float* mask, void* o,
                       void* stream) {
    const ogc_status st = ogc_mha_validate(d);
    if (st != OGC_OK) return st;
    if (!q || !k || !v || !o) return OGC_ERR_INVALID_ARG;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return OGC_ERR_ALIGNMENT;
    if ((uintptr_t)mask & 3) return OGC_ERR_ALIGNMENT;
    MhaArgs a;
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
    const bool general = general_case(d, mask);
    const int qs = general ? 1 : query_groups(d);
    a.q_tiles = (d->seq + 128 * qs - 1) / (128 * qs);
    const int bh = d->batch * d->heads;
    auto magic = [](uint64_t n, uint64_t v) { return v == 1 || n * v >= 1ull << 32 ? 0u : (uint32_t)((1ull << 32) / v + 1); };
    a.tiles_magic = magic((uint64_t)bh * a.q_tiles, a.q_tiles);
    a.heads_magic = magic(bh, d->heads);
    a.xcd_order = (bh % 8 == 0) ? 1 : 0;
    a.scale_log2 = d->scale * 1.44269504088896340736f;
    a.inv_scale = 1.0f / d->scale;
    a.addend_max = 3.0e38f / fmaxf(1.0f, a.scale_log2);
    const dim3 grid((unsigned)(bh * a.q_tiles));
    const int plain = plain_case(d, mask);
    const hipError_t e = general ? launch_general(d->head_dim / 32, d->softmax, a, grid, (hipStream_t)stream)
                       : d->dtype == OGC_F32 ? launch_dim<OGC_F32>(d->head_dim / 32, qs, d->softmax, plain, a, grid, (hipStream_t)stream)
                                             : launch_dim<OGC_BF16>(d->head_dim / 32, qs, d->softmax, plain, a, grid, (hipStream_t)stream);
    return e == hipSuccess ? OGC_OK : OGC_ERR_DEVICE;
}

const char* ogc_mha_kernel_name(const ogc_mha_desc* d, int32_t has_mask) {
    if (ogc_mha_validate(d) != OGC_OK) return nullptr;
    static char names[2][4][2][2][2][48], general[4][2][48];
    if (general_case(d, has_mask ? (const float*)d : nullptr)) {
        char* g = general[d->head_dim / 32 - 1][d->softmax];
        if (!g[0]) snprintf(g, 48, "ogc_mha_general_kernel<%d, %d>", d->head_dim / 32, d->softmax);
        return g;
    }
    const int plain = plain_case(d, has_mask ? (const float*)d : nullptr), qs = query_groups(d);
    char* s = names[d->dtype == OGC_BF16][d->head_dim / 32 - 1][d->softmax][plain][qs - 1];
    if (!s[0]) snprintf(s, 48, "ogc_mha_kernel<%d, %d, %d, %d, %d>", d->dtype, d->head_dim / 32, d->softmax, plain, qs);
    return s;
}

}  // extern "C"
