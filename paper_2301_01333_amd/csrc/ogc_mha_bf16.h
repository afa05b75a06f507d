// The bf16 body of the fused attention kernel (included by ogc_mha.hip; see there for the operation and the transposed
// products).  One workgroup = 4 wavefronts, QS groups of 32 queries each; keys and values stream through LDS in units
// of 32 keys.
//
// What bounds it, and what follows from that.  Per unit, 32 queries and d = 64 a wavefront owes 256 clocks of matrix
// instructions and, per score, one multiply-add, one exponential, half a conversion and half a row-sum instruction:
// about 256 clocks of vector-ALU issue as well.  Everything else has to go:
//   * keys and values go from global memory straight into LDS (global_load_lds_dwordx4: no staging registers, no LDS
//     writes), PF units ahead of their use; rows keep their order, only the 16-byte pieces inside a row are permuted
//     (by the lane that loads them) so that the operand reads are free of bank conflicts;
//   * V^T operands come out of LDS through the transposing read (ds_read_b64_tr_b16: 4 keys x 16 channels per 16
//     lanes), whose four keys are exactly the four consecutive keys a register quad of the score accumulator holds;
//   * a mask (and the -infinity of keys beyond the sequence) is the initial value of the score accumulator, divided
//     by the scalar once per workgroup, so it costs no arithmetic per score.  Such an accumulator is rounded at the size
//     of the mask once per matrix instruction, so this is for tiles whose references end up near zero: some key's addend
//     is within 2^10 of it (base 2) and none lies above.  Up to there the outputs of rows masked alike are as near to 64 bits
//     as with the mask added last (0.00228 of their norm both ways at -700); at -10000 they were 0.00244 against 0.00231, at
//     -100000 0.0067 against 0.0038.  The other tiles (batch entries that are masked throughout) take a loop of their own;
//   * the reference point of the exponentials is not the running maximum of every unit.  A unit is exponentiated
//     against the reference there is, and only if the row sum of the result (needed anyway) passes 2^8, or is no
//     number, is the unit's maximum taken, the reference moved and the unit exponentiated again.  The same function:
//     numerator and denominator carry the same factor, and every weight stays at or below 2^8.  A reference beyond 2^24
//     (scores whose spacing in fp32 is no longer small against 1) always takes that way, which subtracts exactly;
//   * the scores of the next unit and the second product of the one before are computed next to the exponentials of
//     this one: the matrix pipe and the vector ALU work side by side inside a wavefront.
// Measured against the staged body (64-key blocks through registers, maximum of every block, transposing LDS writes), both
// on one card: batch 128 x 16 heads x 512 tokens x 64, padding mask: 210 -> 193 us (655 -> 713 TFLOP/s); 64 x 16 x 512 x 32:
// 77 -> 58; 64 x 16 x 512 x 96: 174 -> 158; 1 x 8 x 8192 x 128: 310 -> 270.  More, and where it is the slower, at stream_case.
// Counters at the first of these: vector ALU 48 % of the SIMDs' cycles, matrix pipe 31 %.  About 30 of its us are the tensors' way
// from HBM, and 16 units are too few to hide a workgroup's first loads and its end behind its one neighbour on the
// compute unit: 8 x 16 x 2048 x 64, the same arithmetic, takes 146 us.  Tried: workgroups that walk over several tiles
// with the loads running on across them (no faster: the clock gives way), one query group per wavefront for long
// sequences (LDS reads, 196 us), four pairs of weights between matrix instructions (182).
#ifndef OGC_MHA_BF16_H
#define OGC_MHA_BF16_H

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) uint8_t mha_lds_u8;
typedef __attribute__((address_space(3))) v4i mha_lds_v4i;
typedef __attribute__((address_space(3))) v4s mha_lds_v4s;
typedef __attribute__((address_space(3))) v4f mha_lds_v4f;

constexpr int MHA_LDS_KEYS = 4096;  // longer sequences replace half of them every 64 units
constexpr int MHA_UNIT = 32;  // keys per unit
constexpr int MHA_PF = 2;     // units in flight ahead of the one in use
constexpr float MHA_ADDEND_NEAR = 1024.0f;  // addends (base-2 domain) of keys that may hold a tile's references near zero
constexpr int MHA_READ_AHEAD = 3;  // pairs of weights between an operand's LDS read and its first matrix instruction

template <int D32> struct MhaB {
    static constexpr int D = D32 * 32, ROW = D * 2, CH = ROW / 16;  // bytes and 16-byte pieces per row
    static constexpr int UNIT_BYTES = MHA_UNIT * ROW, SLOTS = 4;
    static constexpr int RING = 2 * SLOTS * UNIT_BYTES;  // keys, then values
    // Position of piece c of key row r inside the row.  A read takes the same piece of eight consecutive keys (first
    // product) or two neighbouring pieces of four consecutive ones (second): with these the eight 16-byte pieces fall
    // on distinct groups of four banks, for rows of 64, 128, 192 and 256 bytes.
    static constexpr bool WIDE_ROWS = CH % 8 == 0;
    static __device__ __forceinline__ int kswz(int r) { return WIDE_ROWS ? (r & 7) : ((r >> 1) & 3); }
    static __device__ __forceinline__ int vswz(int r) { return WIDE_ROWS ? 2 * (r & 3) : 2 * ((r >> 1) & 1); }
};

template <int N> MHA_DEV void mha_wait_and_meet() {  // all but the N newest loads have landed, LDS accesses are done, then the workgroup meets
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// D32 = head_dim / 32.  PLAIN: no mask, whole units, so no key needs an addend.  The scalar is positive.
template <int D32, int FAST, int PLAIN, int QS> MHA_DEV void mha_stream_body(const MhaArgs& a, mha_lds_u8* lds) {
    typedef MhaB<D32> B;
    constexpr int D = B::D, QN = D / 16, NL = D32;  // NL: 1 KiB loads per wavefront and unit (keys and values together)
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroup ids go round the 8 XCDs.  Each XCD takes a contiguous run of (batch, head) pairs, so that the query tiles
    // of a pair share its L2, and so that it works on all the heads of a batch entry at a time: the heads of a token are
    // neighbours in memory, and an XCD that saw only every eighth of them would use only some of its L2's channels.
    const uint32_t wg = blockIdx.x, lin = a.xcd_order ? (wg & 7) * (gridDim.x >> 3) + (wg >> 3) : wg;
    const int bh = div_magic(lin, a.q_tiles, a.tiles_magic), qt = (int)lin - bh * a.q_tiles;
    const int b = div_magic(bh, a.heads, a.heads_magic), hd = bh - b * a.heads, S = a.seq;
    const int n = S > MHA_UNIT ? (S + MHA_UNIT - 1) / MHA_UNIT : 2;  // at least two: the second may hold no key
    const uint8_t* kbase = a.k + (b * a.sk[0] + hd * a.sk[1]) * 2;
    const uint8_t* vbase = a.v + (b * a.sv[0] + hd * a.sv[1]) * 2;
    const long long kss = a.sk[2] * 2, vss = a.sv[2] * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    // ---- direct loads.  The 4 * D32 loads of a unit's keys (the first half) and values go round the wavefronts.
    // Load m of 64 pieces covers the pieces 64 m + lane of the unit's linear LDS image.
    uint32_t voff[NL];   // byte offset of the lane's piece from the unit's first row (32 bits: checked by the host)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int ld = i * 4 + wave;
        const bool is_v = ld >= 2 * D32;
        const int p = (ld - (is_v ? 2 * D32 : 0)) * 64 + lane, r = p / B::CH, slot = p % B::CH;
        const int piece = slot ^ (is_v ? B::vswz(r) : B::kswz(r));
        voff[i] = (uint32_t)r * (uint32_t)(is_v ? vss : kss) + piece * 16;
    }
    // keys of unit ku into the slot at ko (bytes), values of unit vu into the one at vo; units that do not exist are left out
    auto issue = [&](int ku, uint32_t ko, int vu, uint32_t vo) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int ld = i * 4 + wave;
            const bool is_v = ld >= 2 * D32;
            const int u = is_v ? vu : ku;
            if (u < 0 || u >= n) continue;
            const long long rs = is_v ? vss : kss;
            const uint8_t* g = (is_v ? vbase : kbase) + (long long)(u * MHA_UNIT) * rs;
            const uint32_t dst = lds0 + (is_v ? B::SLOTS * B::UNIT_BYTES + vo + (ld - 2 * D32) * 1024 : ko + ld * 1024);
            const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst);
            auto load = [&]() {
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(voff[i]), "s"(g) : "memory", "m0");
            };
            if ((u + 1) * MHA_UNIT <= S) load();
            else {  // rows beyond the sequence are zero
                int l = lane;
                asm volatile("" : "+v"(l));  // nothing of this rare branch is kept in registers across the main loop
                if (u * MHA_UNIT + ((ld - (is_v ? 2 * D32 : 0)) * 64 + l) / B::CH < S) load();
                else *(mha_lds_v4i*)(uintptr_t)(dst + l * 16) = (v4i){l >> 6, l >> 6, l >> 6, l >> 6};
            }
        }
    };

    // ---- this lane's query rows as the second operand of the first product
    int query[QS];
    v4i qreg[QS][QN];
    v16f oacc[QS][D32];
    float ref[QS], run_sum[QS];  // run_sum: this lane's keys only, the halves are added at the end
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
        query[qs] = (qt * 4 + wave) * (32 * QS) + qs * 32 + col;
        const int qrow = query[qs] < S ? query[qs] : S - 1;
        const uint8_t* qp = a.q + (b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2]) * 2;
#pragma unroll
        for (int i = 0; i < QN; ++i) qreg[qs][i] = *(const v4i*)(qp + i * 32 + h * 16);
#pragma unroll
        for (int d = 0; d < D32; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[qs][d][r] = 0.0f;
        ref[qs] = run_sum[qs] = 0.0f;
    }

    // ---- first loads, oldest first: K0 | K1 V0 | K2 V1
    constexpr uint32_t U = B::UNIT_BYTES;
    issue(0, 0, -1, 0);
    issue(1, U, 0, 0);
    issue(2, 2 * U, 1, U);
    // an addend per key in LDS, -infinity beyond the sequence: mask times `by` (1 / scalar, or log2(e) in the last loop below)
    typedef __attribute__((address_space(3))) float lds_f32;
    lds_f32* const add = (lds_f32*)(lds + B::RING);
    const float* mrow = a.mask + (long long)b * S;
    auto each_mask = [&](int first, int count, auto use) {  // use(key, mask) for keys first .. first + count - 1, four loads in flight
        for (int j0 = first + tid; j0 < first + count; j0 += 1024) {
            float m[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) m[i] = a.mask && j0 + 256 * i < S ? mrow[j0 + 256 * i] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (j0 + 256 * i < first + count) use(j0 + 256 * i, m[i]);
        }
    };
    auto fill_addends = [&](int first, int count, float by, float most) {  // a multiple of MHA_UNIT, at most MHA_LDS_KEYS
        each_mask(first, count, [&](int j, float m) { add[j & (MHA_LDS_KEYS - 1)] = j < S ? finite_mask(m * by, most) : -INFINITY; });
    };
    const int add_keys = n * MHA_UNIT < MHA_LDS_KEYS ? n * MHA_UNIT : MHA_LDS_KEYS;
    // May addends start accumulators?  Only if some key holds the references near zero and none lifts them far above it.
    lds_f32* const votes = (lds_f32*)(lds + 3 * U);  // (the slot of the fourth unit's keys, which are loaded later)
    if constexpr (!PLAIN) {
        bool some = false, high = false;
        each_mask(0, n * MHA_UNIT, [&](int j, float m) {
            if (j < add_keys) add[j] = j < S ? finite_mask(m * a.inv_scale, a.addend_max) : -INFINITY;
            some = some || (j < S && !(fabsf(m * LOG2E) > MHA_ADDEND_NEAR));
            high = high || m * LOG2E > MHA_ADDEND_NEAR;
        });
        const uint64_t somes = __builtin_amdgcn_ballot_w64(some), highs = __builtin_amdgcn_ballot_w64(high);
        if (!FAST && lane == 0) votes[wave] = highs ? -8.0f : somes ? 1.0f : 0.0f;
    }
    if (3 * MHA_UNIT <= S) mha_wait_and_meet<FAST ? 2 * NL : NL>();
    else mha_wait_and_meet<0>();

    const float c = a.scale_log2;
    float exact_c = c;  // for weights by rounded products; 1 in the last loop below
    // ---- operand addresses in the first slot.  The other pieces of a row follow by exclusive or: a slot begins at a
    // multiple of the row's size, and the permutation is an exclusive or itself.
    const uint32_t kaddr = lds0 + col * B::ROW + ((h ^ B::kswz(col)) * 16);
    const int vr = (lane & 15) >> 2;  // key offset inside a quad whose row this lane supplies to the transposing read
    const uint32_t vaddr = lds0 + B::SLOTS * B::UNIT_BYTES + (4 * h + vr) * B::ROW + (lane & 1) * 8 +
                           (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ B::vswz(4 * h + vr)) * 16);

    // operand i of the first product: 32 keys x 16 channels
    auto read_keys = [&](uint32_t ko, int i) {
        // pieces 8 and up of a 256-byte row: the permutation leaves bit 3 alone; 64- and 192-byte rows: bits 2 and 3
        const uint32_t at = B::WIDE_ROWS ? ((kaddr + ko) ^ ((i & 3) * 32)) + (i >> 2) * 128 : ((kaddr + ko) ^ ((i & 1) * 32)) + (i >> 1) * 64;
        return *(const mha_lds_v4i*)(uintptr_t)at;
    };
    auto read_addend = [&](int u, v16f& init) {
        if constexpr (!PLAIN) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f m = *(const mha_lds_v4f*)(add + ((u * MHA_UNIT & (MHA_LDS_KEYS - 1)) + 8 * g + 4 * h));
#pragma unroll
                for (int e = 0; e < 4; ++e) init[4 * g + e] = m[e];
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) init[r] = 0.0f;
        }
    };
    // operand jd of the second: 32 channels (d) x the 16 keys of group j
    auto read_values = [&](uint32_t vo, int jd) {
        const int j = jd / D32, d = jd % D32;
        const uint32_t at = (B::WIDE_ROWS ? ((vaddr + vo) ^ ((d & 1) * 64)) + (d >> 1) * 128 : (vaddr + vo) + d * 64) + 16 * j * B::ROW;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mha_lds_v4s*)(uintptr_t)at);
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mha_lds_v4s*)(uintptr_t)(at + 8 * B::ROW));
        return (v8s){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    // one matrix instruction of the first product (instruction t = operand piece t / QS, query group t % QS) ...
    auto mma_score = [&](int t, const v4i (&kf)[QN], const v16f& init, v16f (&s)[QS]) {
        const int i = t / QS, qs = t % QS;
        s[qs] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, kf[i]), __builtin_bit_cast(v8bf, qreg[qs][i]),
                                                        i ? s[qs] : init, 0, 0, 0);
    };
    // ... and of the second (t = (16-key group, channel block, query group))
    auto mma_value = [&](int t, const v8s (&vf)[2 * D32], const uint32_t (&w)[QS][8]) {
        const int qs = t % QS, jd = t / QS, j = jd / D32, d = jd % D32;
        const v4i pw = {(int)w[qs][4 * j], (int)w[qs][4 * j + 1], (int)w[qs][4 * j + 2], (int)w[qs][4 * j + 3]};
        oacc[qs][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, vf[jd]), __builtin_bit_cast(v8bf, pw),
                                                              oacc[qs][d], 0, 0, 0);
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    // two weights of a unit (rounded to bf16, packed) and their share of the row sum over this lane's 16 keys
    // (SPLIT: the product is rounded before the reference is taken off, as the reference itself was: the two cancel
    // exactly at the maximum, however large they are)
    auto weight_pair = [&](auto split_c, const v16f& s, int t, float off, uint32_t& w, float& sum) {
        constexpr bool SPLIT = decltype(split_c)::value;
        auto power = [&](float x) { return FAST ? x * c : SPLIT ? x * exact_c + off : __builtin_fmaf(x, c, off); };
        const float p0 = __builtin_amdgcn_exp2f(power(s[2 * t])), p1 = __builtin_amdgcn_exp2f(power(s[2 * t + 1]));
        const v2bf pr = {(__bf16)p0, (__bf16)p1};
        w = __builtin_bit_cast(uint32_t, pr);
        asm volatile("" : "+v"(w));  // the compiler would move the arithmetic to the next step, where the weights are used
        sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, w), (v2bf){(__bf16)1.0f, (__bf16)1.0f}, t ? sum : 0.0f, false);
    };
    auto slot = [](int u) { return (uint32_t)(u & (B::SLOTS - 1)) * U; };
    // One step: weights of unit u (scores s -> w), next to the scores of unit u + 1 (-> next; NEXT) and the second
    // product of unit u - 1 (weights wp; PREV).
    auto step = [&](auto prev_c, auto next_c, int u, v16f (&s)[QS], v16f (&next)[QS], const uint32_t (&wp)[QS][8], uint32_t (&w)[QS][8]) {
        constexpr bool PREV = decltype(prev_c)::value, NEXT = decltype(next_c)::value;
        // K[u+1] was issued two steps ago, V[u-1] three; only the loads of the step before may still be in flight, and a
        // wavefront has NL of those only if that step's key unit exists and is whole
        if ((u + MHA_PF + 1) * MHA_UNIT <= S) mha_wait_and_meet<NL>();
        else mha_wait_and_meet<0>();
        issue(u + 3, slot(u + 3), u + 2, slot(u + 2));  // over K[u-1] and V[u-2], which no one reads any more
        if constexpr (NEXT && !PLAIN) {
            // unit u + 1 opens a new half (the first two are there): over the half before unit u's
            constexpr int HALF = MHA_LDS_KEYS / 2;
            const int first = (u + 1) * MHA_UNIT;
            if (first % HALF == 0 && first >= MHA_LDS_KEYS) {
                fill_addends(first, n * MHA_UNIT - first < HALF ? n * MHA_UNIT - first : HALF, a.inv_scale, a.addend_max);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
        }
        v4i kf[QN];
        v8s vf[2 * D32];
        v16f init;
        // Matrix instructions, the second product's first, spread evenly between the pairs of weights.  An operand is
        // read from LDS AHEAD pairs before its first use (the value of an unread operand costs no register).
        constexpr int NP = PREV ? 2 * D32 * QS : 0, NK = NEXT ? QN * QS : 0, PAIRS = 8 * QS, AHEAD = MHA_READ_AHEAD;
        auto first_pair = [](int m) { return ((m + 1) * PAIRS + NP + NK - 1) / (NP + NK > 0 ? NP + NK : 1) - 1; };  // the pair after which instruction m issues
        float sum[QS];
#pragma unroll
        for (int t = -AHEAD; t < PAIRS; ++t) {
            if constexpr (PREV) {
#pragma unroll
                for (int jd = 0; jd < 2 * D32; ++jd)
                    if (first_pair(jd * QS) == t + AHEAD || (t == -AHEAD && first_pair(jd * QS) < 0)) vf[jd] = read_values(slot(u - 1), jd);
            }
            if constexpr (NEXT) {
                if (first_pair(NP) == t + AHEAD) read_addend(u + 1, init);
#pragma unroll
                for (int i = 0; i < QN; ++i)
                    if (first_pair(NP + i * QS) == t + AHEAD) kf[i] = read_keys(slot(u + 1), i);
            }
            if (t < 0) continue;
            if (t % 2 == 0) {  // two pairs side by side (of the two query groups, if there are two): their chains overlap
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int x = t; x < t + 2; ++x) weight_pair(no, s[x % QS], x / QS, -ref[x % QS], w[x % QS][x / QS], sum[x % QS]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int m = (NP + NK) * t / PAIRS; m < (NP + NK) * (t + 1) / PAIRS; ++m) {
                if (m < NP) mma_value(m, vf, wp);
                else mma_score(m - NP, kf, init, next);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!FAST) {
            bool far = false;
#pragma unroll
            for (int qs = 0; qs < QS; ++qs) far = far || !(sum[qs] <= 256.0f) || !(fabsf(ref[qs]) <= 16777216.0f);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, D32 == 1)) {  // (32 channels: spills, laid out as unlikely)
#pragma unroll
                for (int qs = 0; qs < QS; ++qs) {
                    // the scores once more: keeping them until here would cost 16 registers a group
                    v16f t;
                    if constexpr (!NEXT) {
                        t = s[qs];  // no next scores: the registers are there
                    } else {
                        read_addend(u, t);
#pragma unroll
                        for (int i = 0; i < QN; ++i)
                            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, read_keys(slot(u), i)),
                                                                        __builtin_bit_cast(v8bf, qreg[qs][i]), t, 0, 0, 0);
                    }
                    float cand = t[0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) cand = fmaxf(cand, t[r]);
                    cand = fmaxf(cand, other_half(cand)) * c;
                    const float new_ref = fmaxf(cand, ref[qs]);
                    const float alpha = __builtin_amdgcn_exp2f(ref[qs] - new_ref);
                    ref[qs] = new_ref;
                    run_sum[qs] *= alpha;
#pragma unroll
                    for (int d = 0; d < D32; ++d)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[qs][d][r] *= alpha;
#pragma unroll
                    for (int p = 0; p < 8; ++p) weight_pair(yes, t, p, -new_ref, w[qs][p], sum[qs]);
                }
            }
        }
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) run_sum[qs] += sum[qs];
    };

    v16f s0[QS], s1[QS];
    uint32_t w0[QS][8], w1[QS][8];
    auto first_scores = [&](int u, v16f (&s)[QS]) {
        v4i kf[QN];
        v16f init;
#pragma unroll
        for (int i = 0; i < QN; ++i) kf[i] = read_keys(slot(u), i);
        read_addend(u, init);
#pragma unroll
        for (int t = 0; t < QN * QS; ++t) mma_score(t, kf, init, s);
    };
    auto top = [](const v16f& x, const v16f& y) {  // the maximum of two units' scores, this lane's query
        float t = fmaxf(x[0], y[0]);
#pragma unroll
        for (int r = 1; r < 16; ++r) t = fmaxf(t, fmaxf(x[r], y[r]));
        return fmaxf(t, other_half(t));
    };
    auto last = [&](uint32_t (&w)[QS][8]) {  // the second product of the last unit
        mha_wait_and_meet<0>();
        v8s vf[2 * D32];
#pragma unroll
        for (int jd = 0; jd < 2 * D32; ++jd) vf[jd] = read_values(slot(n - 1), jd);
#pragma unroll
        for (int t = 0; t < 2 * D32 * QS; ++t) mma_value(t, vf, w);
    };
    const v4f v = !PLAIN && !FAST ? *(const mha_lds_v4f*)votes : (v4f){1.0f, 0.0f, 0.0f, 0.0f};
    first_scores(0, s0);
    if constexpr (!FAST) first_scores(1, s1);
    const bool late = !PLAIN && !FAST && __builtin_amdgcn_readfirstlane((int)(v[0] + v[1] + v[2] + v[3])) <= 0;
    if (__builtin_expect(!late, 1)) {
        if constexpr (FAST) {
            step(no, yes, 0, s0, s1, w1, w0);
        } else {
            // The first reference: the maximum of the first two units (key 0 is always valid).  The further keys it has seen,
            // the more often a row's largest weight is exactly 1, which bf16 holds: with one unit, outputs were 0.5 % further
            // from 64 bits than the staged body's (0.00230 against 0.00229 of their norm), with two they are as near.  The
            // second unit's scores stand alone for that, 1 to 2 % of the time at 512 keys.
#pragma unroll
            for (int qs = 0; qs < QS; ++qs) ref[qs] = top(s0[qs], s1[qs]) * c;
            step(no, no, 0, s0, s1, w1, w0);
        }
        int u = 1;
        for (; u + 2 < n; u += 2) {
            step(yes, yes, u, s1, s0, w0, w1);
            step(yes, yes, u + 1, s0, s1, w1, w0);
        }
        if (u + 2 == n) {
            step(yes, yes, u, s1, s0, w0, w1);
            step(yes, no, u + 1, s0, s1, w1, w0);
            last(w0);
        } else {
            step(yes, no, u, s1, s0, w0, w1);
            last(w1);
        }
    } else if constexpr (!PLAIN && !FAST) {
        // One unit at a time, each score in the base-2 domain and rounded once, after its product was summed near zero.
        exact_c = 1.0f;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        fill_addends(0, add_keys, LOG2E, MHA_F32_MAX);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        auto scores = [&](int u, int qs) {
            v16f t, m;
#pragma unroll
            for (int r = 0; r < 16; ++r) t[r] = 0.0f;
#pragma unroll
            for (int i = 0; i < QN; ++i)
                t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, read_keys(slot(u), i)),
                                                            __builtin_bit_cast(v8bf, qreg[qs][i]), t, 0, 0, 0);
            read_addend(u, m);
#pragma unroll
            for (int r = 0; r < 16; ++r) t[r] = __builtin_fmaf(t[r], a.scale_log2, m[r]);
            return t;
        };
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) ref[qs] = top(scores(0, qs), scores(1, qs));
#pragma unroll 1
        for (int u = 0; u < n; ++u) {
            // K[u] and V[u] were issued two steps ago at the latest
            if ((u + MHA_PF + 1) * MHA_UNIT <= S) mha_wait_and_meet<NL>();
            else mha_wait_and_meet<0>();
            issue(u + 3, slot(u + 3), u + 2, slot(u + 2));
            if (u * MHA_UNIT % MHA_LDS_KEYS == 0 && u > 0) {
                const int left = n * MHA_UNIT - u * MHA_UNIT;
                fill_addends(u * MHA_UNIT, left < MHA_LDS_KEYS ? left : MHA_LDS_KEYS, LOG2E, MHA_F32_MAX);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
#pragma unroll
            for (int qs = 0; qs < QS; ++qs) {
                const v16f t = scores(u, qs);
                const float cand = top(t, t);
                if (__builtin_amdgcn_ballot_w64(!(cand <= ref[qs] + 8.0f)) != 0) {
                    const float new_ref = fmaxf(cand, ref[qs]), alpha = __builtin_amdgcn_exp2f(ref[qs] - new_ref);
                    ref[qs] = new_ref;
                    run_sum[qs] *= alpha;
#pragma unroll
                    for (int d = 0; d < D32; ++d)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[qs][d][r] *= alpha;
                }
                float sum;
#pragma unroll
                for (int p = 0; p < 8; ++p) weight_pair(yes, t, p, -ref[qs], w0[qs][p], sum);
                run_sum[qs] += sum;
            }
            v8s vf[2 * D32];
#pragma unroll
            for (int jd = 0; jd < 2 * D32; ++jd) vf[jd] = read_values(slot(u), jd);
#pragma unroll
            for (int t = 0; t < 2 * D32 * QS; ++t) mma_value(t, vf, w0);
        }
    }

    // ---- normalise and store: after the half exchange a lane holds 16 consecutive channels of its query
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
        const float inv = 1.0f / (run_sum[qs] + other_half(run_sum[qs]));
        uint8_t* op = a.o + (b * a.so[0] + hd * a.so[1] + (long long)query[qs] * a.so[2]) * 2;
#pragma unroll
        for (int d = 0; d < D32; ++d) {
            uint32_t dw[4][2];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                dw[g][0] = pack_bf16(oacc[qs][d][4 * g] * inv, oacc[qs][d][4 * g + 1] * inv);
                dw[g][1] = pack_bf16(oacc[qs][d][4 * g + 2] * inv, oacc[qs][d][4 * g + 3] * inv);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                swap32(dw[0][j], dw[2][j]);
                swap32(dw[1][j], dw[3][j]);
            }
            if (query[qs] < S) {
                uint8_t* dst = op + (d * 32 + 16 * h) * 2;
                *(v4i*)dst = (v4i){(int)dw[0][0], (int)dw[0][1], (int)dw[2][0], (int)dw[2][1]};
                *(v4i*)(dst + 16) = (v4i){(int)dw[1][0], (int)dw[1][1], (int)dw[3][0], (int)dw[3][1]};
            }
        }
    }
}

#endif
