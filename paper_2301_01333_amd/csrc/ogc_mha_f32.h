// The fp32 body of the fused attention kernel for heads of up to 96 channels (included by ogc_mha.hip; see there for the
// operation and the transposed products).  One workgroup = 4 wavefronts = 128 queries; keys and values in blocks of 32.
//
// The fp32 matrix instruction runs at a sixteenth of the bf16 one's rate, and the staged body was bound by it.  An fp32 value is
// the sum of three bf16 values without any error (8 + 8 + 8 bits), so a product of two is nine bf16 products, of which
// the three smallest are left out: six instructions at sixteen times the rate.  The pieces are rounded to nearest, so that what is
// left out is 2^-24 of a product at most and of either sign (pieces that are cut: 2^-21, always of the product's sign, which
// does not average out: 8.9e-7 against 3.4e-7 for operands of +-1.0078124).  The five small products of
// a sum are added up first and the large ones on top of them, a block of 32 keys at a time: the bf16 instruction truncates what
// it adds to a larger sum, and in one running sum that added up (9.6e-6 at 4096 products of one sign against 1.0e-6 for the
// fp32 instruction; sums kept apart 3.7e-7).  Error against 64 bits, relative 2-norm, fp32 instruction / this: 512 x 64 5.2e-7 /
// 2.2e-7, 1024 x 96 7.2e-7 / 3.0e-7, 160 x 32 3.2e-7 / 1.4e-7; operands of one magnitude (+-1.0078124, +-1.1) 512 x 64 5.9e-7 / 3.4e-7
// and 8.1e-7 / 2.8e-7, with the largest pieces there are (+-(1 + 2^-8 - 2^-17)) 5.6e-7 / 3.9e-7; log-normal ones 9.1e-7 / 3.2e-7.
//
// What bounds it: power.  32 x 16 heads x 512 x 64 (206 GFLOP of bf16 instructions): 273 -> 190 us, but 148 us where all
// inputs are one; the clock is at 1.8 GHz, the matrix pipe busy in 51 % and the vector ALU in 55 % of the cycles; fewer vector
// instructions (377 -> 300 a block and wavefront) changed nothing there and gave 10 % where half
// of the chip works.  2 x 8 x 1024 x 64: 80 -> 48 us; 8 x 16 x 512 x 96: 109 -> 78; more at split_case.  Tried: eight wavefronts that
// share the pieces of keys and values (50.2 against 51.1 us at 8 x 16 x 512 x 64, 202 against 197 at 32); 96 and 128 channels with
// 512 registers, one wavefront a SIMD (arrays in scratch memory, ten times as long).
#ifndef OGC_MHA_F32_H
#define OGC_MHA_F32_H

// Three bf16 pieces of fp32 values that add up to them exactly: the nearest bf16 value, the nearest one to what is left (a
// subtraction without rounding), and the rest, which has 7 bits.  Elements 2 t, 2 t + 1 share a register.
struct Pieces8 {
    v4i p[3];
};
MHA_DEV uint32_t upper_halves(float x, float y) {  // of values that have no others
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, y), __builtin_bit_cast(uint32_t, x), 0x07060302u);
}
// one piece of a pair, and what is left of it
MHA_DEV uint32_t next_piece(float& x, float& y) {
    const uint32_t p = pack_bf16(x, y);
    x -= __builtin_bit_cast(float, __builtin_amdgcn_alignbyte(p, 0u, 2u));  // (p << 16, for which the compiler converts x once more)
    y -= __builtin_bit_cast(float, p & 0xffff0000u);
    return p;
}
// The largest / the smallest of m and both magnitudes.  (As a builtin the former takes the masked body for 64 channels to scratch
// memory.  The compiler does not know what the assembly's operands must keep away from: they are loaded, never computed.)
MHA_DEV float widest(float m, float x, float y) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(x), "v"(y));
    return m;
}
MHA_DEV float least(float m, float x, float y) { return __builtin_elementwise_minimum(__builtin_elementwise_minimum(fabsf(x), fabsf(y)), m); }
// orders magnitudes, zero above all others
MHA_DEV uint32_t zero_last(float x) { return (__builtin_bit_cast(uint32_t, x) << 1) - 1u; }
MHA_DEV Pieces8 split8(const v4f& a, const v4f& b) {
    Pieces8 r;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float x = t < 2 ? a[2 * t & 3] : b[2 * t & 3], y = t < 2 ? a[(2 * t & 3) + 1] : b[(2 * t & 3) + 1];
        r.p[0][t] = (int)next_piece(x, y);
        r.p[1][t] = (int)next_piece(x, y);
        r.p[2][t] = (int)upper_halves(x, y);
    }
    return r;
}

template <int D32> struct MhaS {
    typedef MhaB<D32> B;  // a plane (one piece of 32 keys) has the layout of a bf16 unit: 32 rows, swizzled 16-byte pieces
    static constexpr int PLANE = B::UNIT_BYTES, BLOCK = 6 * PLANE;  // three of the keys, three of the values
    static constexpr int MASKS = 2 * BLOCK, BYTES = MASKS + 2 * 32 * 4;
};

// D32 = head_dim / 32 (up to 3).  FAST, PLAIN: as the staged body.
template <int D32, int FAST, int PLAIN> MHA_DEV void mha_split_body(const MhaArgs& a, uint8_t* smem) {
    typedef MhaS<D32> L;
    typedef MhaB<D32> B;
    constexpr int D = D32 * 32, QN = D / 16, KB = 32;
    constexpr bool PIPE = D32 <= 2;  // scores are computed a round ahead (96 channels: no registers for it)
    constexpr int UNITS = KB * B::CH, TU = 2 * UNITS / 256;  // runs of 8 elements in a block's keys, and a thread's share of keys and values
    mha_lds_u8* const lds = (mha_lds_u8*)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wg = blockIdx.x, lin = a.xcd_order ? (wg & 7) * (gridDim.x >> 3) + (wg >> 3) : wg;  // as the streaming body
    const int bh = div_magic(lin, a.q_tiles, a.tiles_magic), qt = (int)lin - bh * a.q_tiles;
    const int b = div_magic(bh, a.heads, a.heads_magic), hd = bh - b * a.heads, S = a.seq;
    const uint8_t* kbase = a.k + (b * a.sk[0] + hd * a.sk[1]) * 4;
    const uint8_t* vbase = a.v + (b * a.sv[0] + hd * a.sv[1]) * 4;
    const long long kss = a.sk[2] * 4, vss = a.sv[2] * 4;

    // ---- this lane's query row as the second operand of the first product, in pieces
    const int query = (qt * 4 + wave) * 32 + col, qrow = query < S ? query : S - 1;
    Pieces8 qp[QN];
    float wide = 0.0f;  // the largest magnitude among queries and values (see the end)
    {
        uint32_t low = ~0u;
        const uint8_t* p = a.q + (b * a.sq[0] + hd * a.sq[1] + qrow * a.sq[2]) * 4 + h * 32;
#pragma unroll
        for (int i = 0; i < QN; ++i) {
            const v4f x = *(const v4f*)(p + i * 64), y = *(const v4f*)(p + i * 64 + 16);
            qp[i] = split8(x, y);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                wide = widest(wide, x[e], y[e]);
                low = min(low, min(zero_last(x[e]), zero_last(y[e])));
            }
        }
        if (low < zero_last(0x1p-110f)) wide = INFINITY;
    }

    // ---- a block of keys and one of values (and mask) on their way: D32 units of 8 elements a thread, keys first.  No branch:
    // rows beyond the sequence repeat its last one (their weights are zero; what is not finite there ends the tile below).
    const int nkb = (S + KB - 1) / KB;
    const bool masked = a.mask != nullptr;
    const float* const mrow = masked ? a.mask + (long long)b * S : (const float*)kbase;
    v4f raw[TU][2];
    float mreg = 0.0f;
    // wavefront-uniform base and 32 bits of offset (checked by the host)
    auto unit_of = [&](int i, bool& is_v, int& r, int& piece) {
        is_v = wave * 64 + 256 * i >= UNITS;
        const int u = lane + (wave * 64 + 256 * i) % UNITS;
        r = u / B::CH, piece = u % B::CH;
    };
    auto prefetch_unit = [&](int i, int kblk, int vblk) {
        bool is_v;
        int r, piece;
        unit_of(i, is_v, r, piece);
        const int blk0 = is_v ? vblk : kblk, blk = blk0 < nkb ? blk0 : nkb - 1, most = S - 1 - blk * KB;
        const uint8_t* g = (is_v ? vbase : kbase) + (long long)(blk * KB) * (is_v ? vss : kss);
        const uint32_t row = PLAIN || r < most ? r : most;
        const uint32_t at = __umul24(row, (uint32_t)(is_v ? vss : kss)) + piece * 32;
        raw[i][0] = *(const v4f*)(g + at);
        raw[i][1] = *(const v4f*)(g + at + 16);
    };
    auto prefetch_mask = [&](int kblk) {
        if constexpr (!PLAIN) {
            const int key = kblk * KB + col;
            mreg = mrow[masked ? (key < S ? key : S - 1) : 0];
        }
    };
    // pieces of elements 2 t, 2 t + 1 of unit i, in two steps; with the last of them the unit goes to LDS
    uint32_t up[3][4];
    float left[2];
    auto fill_step = [&](int i, int t, int step, int kblk, int vblk) {
        if (step == 0) {
            left[0] = raw[i][t >> 1][2 * t & 3], left[1] = raw[i][t >> 1][(2 * t & 3) + 1];
            if (256 * (i + 1) > UNITS) wide = widest(wide, left[0], left[1]);  // (not the units of keys alone)
            up[0][t] = next_piece(left[0], left[1]);
            return;
        }
        up[1][t] = next_piece(left[0], left[1]);
        up[2][t] = upper_halves(left[0], left[1]);
        if (t < 3) return;
        bool is_v;
        int r, piece;
        unit_of(i, is_v, r, piece);
        const uint32_t at = lds0 + ((is_v ? vblk : kblk) & 1) * L::BLOCK + (is_v ? 3 * L::PLANE : 0) + r * B::ROW +
                            (piece ^ (is_v ? B::vswz(r) : B::kswz(r))) * 16;
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *(mha_lds_v4i*)(uintptr_t)(at + p * L::PLANE) = (v4i){(int)up[p][0], (int)up[p][1], (int)up[p][2], (int)up[p][3]};
    };
    auto fill_mask = [&](int kblk, int buf) {
        if constexpr (!PLAIN) {  // every wavefront writes the same 32 values
            const float m = kblk * KB + col >= S ? -INFINITY : masked ? (mreg < MHA_MASK_LOW ? MHA_MASK_LOW : mreg) * LOG2E : 0.0f;
            *(__attribute__((address_space(3))) float*)(uintptr_t)(lds0 + L::MASKS + buf * 128 + col * 4) = m;
        }
    };
    auto prefetch = [&](int kblk, int vblk) {
#pragma unroll
        for (int i = 0; i < TU; ++i) prefetch_unit(i, kblk, vblk);
        prefetch_mask(kblk);
    };
    auto fill = [&](int kblk, int vblk) {
#pragma unroll
        for (int i = 0; i < TU; ++i)
#pragma unroll
            for (int t = 0; t < 8; ++t) fill_step(i, t >> 1, t & 1, kblk, vblk);
        fill_mask(kblk, kblk & 1);
    };
    auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    v16f oacc[D32];
#pragma unroll
    for (int d = 0; d < D32; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0.0f;
    float run_max = -INFINITY, run_sum = 0.0f;
    const float c = a.scale_log2;

    const uint32_t kaddr = lds0 + col * B::ROW + ((h ^ B::kswz(col)) * 16);
    const int vr = (lane & 15) >> 2;
    const uint32_t vaddr = lds0 + 3 * L::PLANE + (4 * h + vr) * B::ROW + (lane & 1) * 8 +
                           (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ B::vswz(4 * h + vr)) * 16);
    auto read_keys = [&](uint32_t o, int i) {
        const uint32_t at = B::WIDE_ROWS ? ((kaddr ^ ((i & 3) * 32)) + (i >> 2) * 128) : ((kaddr ^ ((i & 1) * 32)) + (i >> 1) * 64);
        return __builtin_bit_cast(v8bf, *(const mha_lds_v4i*)(uintptr_t)(at + o));
    };
    auto read_values = [&](uint32_t o, int j, int d) {
        const uint32_t at = (B::WIDE_ROWS ? (vaddr ^ ((d & 1) * 64)) + (d >> 1) * 128 : vaddr + d * 64) + 16 * j * B::ROW + o;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mha_lds_v4s*)(uintptr_t)at);
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mha_lds_v4s*)(uintptr_t)(at + 8 * B::ROW));
        return __builtin_bit_cast(v8bf, (v8s){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    };
    auto mma = [](const v8bf& x, const v4i& y, const v16f& z) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, __builtin_bit_cast(v8bf, y), z, 0, 0, 0); };
    v16f zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;

    // Scores of a block, instruction m of 6 QN: the small products first, the large ones on top of their sum.  The pieces of
    // the next 16 channels are read while these are multiplied.
    constexpr bool KEEP = D32 <= 2;  // the upper pieces stay in registers until the large products
    constexpr int AHEAD = PIPE;
    v8bf kf[1 + AHEAD][3], k0[KEEP ? QN : 1];
    auto read_key_pieces = [&](uint32_t o, int i) {
#pragma unroll
        for (int p = 0; p < 3; ++p) kf[i & AHEAD][p] = read_keys(o + p * L::PLANE, i);
    };
    auto score_step = [&](uint32_t o, int m, v16f& s) {
        if (m < 5 * QN) {
            const int i = m / 5, w = m % 5;
            const v8bf(&f)[3] = kf[i & AHEAD];
            if (w == 0 && AHEAD && i + 1 < QN) read_key_pieces(o, i + 1);
            if (w == 0 && !AHEAD && i) read_key_pieces(o, i);
            if (KEEP && w == 0) k0[KEEP ? i : 0] = f[0];
            s = mma(f[w == 0 ? 2 : (w & 1)], qp[i].p[w == 1 || w == 4 ? 1 : w == 2 ? 2 : 0], m ? s : zero);
        } else {
            const int i = m - 5 * QN;
            s = mma(KEEP ? k0[KEEP ? i : 0] : read_keys(o, i), qp[i].p[0], s);
        }
    };
    // scalar, mask and maximum of four scores (base-2 logarithm domain)
    auto scale_step = [&](int kblk, int g, v16f& s, float& cand) {
        if constexpr (PLAIN) {
            if constexpr (!FAST) {
#pragma unroll
                for (int e = 0; e < 4; ++e) cand = fmaxf(cand, s[4 * g + e]);
            }
        } else {
            const v4f mk = *(const mha_lds_v4f*)(uintptr_t)(lds0 + L::MASKS + (kblk & 1) * 128 + (8 * g + 4 * h) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s[4 * g + e] = __builtin_fmaf(s[4 * g + e], c, mk[e]);
                if constexpr (!FAST) cand = fmaxf(cand, s[4 * g + e]);
            }
        }
    };
    auto row_top = [&](float cand) { return FAST ? 0.0f : fmaxf(cand, other_half(cand)) * (PLAIN ? c : 1.0f); };
    // The sums of a block's last 32 channels are added to the output in the next round, when they are certainly there.
    constexpr bool LATE = PIPE;
    v16f late = zero;
    auto add_late = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[D32 - 1][r] += late[r];
    };
    auto follow = [&](float cand) {  // the reference of the exponentials moves when a block exceeds it by more than 2^8
        if constexpr (!FAST) {
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
                if constexpr (LATE)
#pragma unroll
                    for (int r = 0; r < 16; ++r) late[r] *= alpha;
            }
        }
    };
    // One round: the weights of block u (from its scores s) next to the scores of block u + 1, then the second product of
    // block u next to the pieces of the keys and values to come and the maximum of block u + 1.  Matrix instructions and vector
    // arithmetic alternate in small portions: a wavefront issues in order, and a portion runs while the instruction before it does.
    // PAR: u % 2, so that LDS offsets are constants.
    auto round = [&](auto more_c, auto par_c, int u, v16f& s) {
        constexpr bool MORE = decltype(more_c)::value;
        constexpr int PAR = decltype(par_c)::value;
        v16f next;
        float off = FAST ? 0.0f : -run_max;
        Pieces8 pw[2];
        float w[2];
        auto weight_step = [&](int n) {  // n of 24: three steps a pair of weights
            const int t = n / 3;
            if (n % 3 == 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float x = s[2 * t + e];
                    w[e] = __builtin_amdgcn_exp2f(PLAIN ? __builtin_fmaf(x, c, off) : FAST ? x : x + off);
                    run_sum += w[e];
                }
            } else if (n % 3 == 1) {
                pw[t / 4].p[0][t & 3] = (int)next_piece(w[0], w[1]);
            } else {
                pw[t / 4].p[1][t & 3] = (int)next_piece(w[0], w[1]);
                pw[t / 4].p[2][t & 3] = (int)upper_halves(w[0], w[1]);
            }
        };
        constexpr int NA = MORE && PIPE ? 6 * QN : 1;
        constexpr uint32_t o = PAR * L::BLOCK, o1 = L::BLOCK - o;
        v8bf vf[1 + AHEAD][3], v0[2];
        auto read_value_pieces = [&](int n) {  // n = 2 d + j
#pragma unroll
            for (int p = 0; p < 3; ++p) vf[n & AHEAD][p] = read_values(o + p * L::PLANE, n & 1, n >> 1);
        };
        if constexpr (!PIPE) {
            read_key_pieces(o, 0);
#pragma unroll
            for (int m = 0; m < 6 * QN; ++m) {
                score_step(o, m, s);
                if constexpr (MORE) {
#pragma unroll
                    for (int n = 8 * TU * m / (6 * QN); n < 8 * TU * (m + 1) / (6 * QN); ++n) {
                        fill_step(n / 8, (n & 7) >> 1, n & 1, PAR + 1, PAR + 1);
                        if (n % 8 == 7) prefetch_unit(n / 8, u + 2, u + 2);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (MORE) fill_mask(u + 1, PAR ^ 1);
            if constexpr (MORE) prefetch_mask(u + 2);
            float top = -INFINITY;
#pragma unroll
            for (int g = 0; g < 4; ++g) scale_step(PAR, g, s, top);
            follow(row_top(top));
            off = FAST ? 0.0f : -run_max;
        }
        if constexpr (PIPE && MORE) {
            read_key_pieces(o1, 0);
            __builtin_amdgcn_sched_barrier(0);
            weight_step(0);
            weight_step(1);
            __builtin_amdgcn_sched_barrier(0);
        }
        constexpr int W0 = PIPE && MORE ? 2 : 0;
#pragma unroll
        for (int m = 0; m < NA; ++m) {
            if constexpr (PIPE && MORE) score_step(o1, m, next);
            if (m == (NA < 4 ? 0 : NA - 4)) read_value_pieces(0);
#pragma unroll
            for (int n = W0 + (24 - W0) * m / NA; n < W0 + (24 - W0) * (m + 1) / NA; ++n) weight_step(n);
            if (LATE && m >= 1 && m <= 4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[D32 - 1][4 * (m - 1) + e] += late[4 * (m - 1) + e];
            }
            if (LATE && !MORE) add_late();
            __builtin_amdgcn_sched_barrier(0);
        }
        // O^T += V^T P^T, a block's sum at a time (an accumulator that lived on would round the small products away)
        constexpr int NB = 12 * D32, STEPS = 8 * TU;
        float cand = -INFINITY;
        v16f t0, t1;
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            const int d = m / 12, i = m % 12, j = i < 10 ? i / 5 : i - 10, x = i < 10 ? i % 5 : 5;
            if (AHEAD && i == 1) read_value_pieces(2 * d + 1);
            if (AHEAD && i == 6 && d + 1 < D32) read_value_pieces(2 * d + 2);
            if (!AHEAD && x == 0 && m) read_value_pieces(2 * d + j);
            if (x == 0) v0[j] = vf[j & AHEAD][0];
            const v8bf& f = x == 5 ? v0[j] : vf[j & AHEAD][x == 0 ? 2 : x & 1];
            v16f& t = LATE && (d & 1) ? t1 : t0;
            t = mma(f, pw[j].p[x == 1 || x == 4 ? 1 : x == 2 ? 2 : 0], i ? t : zero);
            if (LATE && d && i >= 2 && i < 6) {
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[d - (d > 0)][4 * (i - 2) + e] += ((d & 1) ? t0 : t1)[4 * (i - 2) + e];
            }
            if constexpr (PIPE && MORE) {
                if (m < 4) scale_step(PAR + 1, m, next, cand);
                if (m == 5) cand = row_top(cand);
#pragma unroll
                for (int n = m < 5 ? 0 : STEPS * (m - 5) / (NB - 5); n < (m < 5 ? 0 : STEPS * (m - 4) / (NB - 5)); ++n) {
                    fill_step(n / 8, (n & 7) >> 1, n & 1, PAR, PAR + 1);
                    if (n % 8 == 7) prefetch_unit(n / 8, u + 3, u + 2);
                }
                if (m == NB - 1) fill_mask(u + 2, PAR);
                if (m == NB - 1) prefetch_mask(u + 3);
            }
            if (i == 11 && !LATE) {
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[d][r] += t[r];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (LATE) late = (D32 - 1) & 1 ? t1 : t0;
        if constexpr (MORE) {
            if constexpr (PIPE) {
                follow(cand);
                s = next;
            }
            meet();
        }
    };

    // K0 | K1 V0: the first scores stand alone
    prefetch(0, 0);
    fill(0, 0);
    prefetch(1, PIPE ? 0 : 1);
    meet();
    v16f s;
    if constexpr (PIPE) {
        read_key_pieces(0, 0);
#pragma unroll
        for (int m = 0; m < 6 * QN; ++m) score_step(0, m, s);
        float cand = -INFINITY;
#pragma unroll
        for (int g = 0; g < 4; ++g) scale_step(0, g, s, cand);
        follow(row_top(cand));
        fill(1, 0);
        prefetch(2, 1);
        meet();
    }
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    int u = 0;
    for (; u + 2 < nkb; u += 2) {
        round(yes, even, u, s);
        round(yes, odd, u + 1, s);
    }
    if (u + 2 == nkb) {
        round(yes, even, u, s);
        round(no, odd, u + 1, s);
    } else {
        round(no, even, u, s);
    }
    if constexpr (LATE) add_late();

    // ---- normalise.  Some tiles are computed once more by the fp32 instruction.  Pieces are multiples of 2^-133 (the instruction
    // takes those below the smallest exponent as they are): what is below 2^-110 is off by 2^-134 at most.
    //   * Infinities: the pieces have no answer to them (infinity less itself is no number; nor is then the sum of the weights).
    //   * Queries below 2^-110, or Q beyond 2^90 over the scalar: smaller keys move a score by 96 x 2^-134 Q times that, 2^-37.
    //   * Values up to V and sums below 2^-94 V: smaller weights, up to 2^16 of them, move a sum by 2^-118 V, 2^-24 of it.  (Values
    //     beyond 2^100 in any case: their sums, and the first piece of the largest of them, are close to infinity.)
    //   * Results below 2^-100: smaller values move them by 2^-134, 2^-34 of them.
    //   * Sums of zero where there are values below the smallest exponent, whose pieces may be zero.
    // One look for the largest and the smallest of all (scalars of up to 2^60: queries and values up to 2^20, sums from 2^-74 on), a
    // closer one at what it finds, for which the wavefronts put together what each saw of the values: 32 x 16 x 512 x 64 with values
    // of 2^21 194 us, 190 without; all computed again 452.
    const float total = run_sum + other_half(run_sum), inv = 1.0f / total;
    float lowest = 1.0f;
#pragma unroll
    for (int d = 0; d < D32; ++d)
#pragma unroll
        for (int r = 0; r < 16; r += 2) lowest = least(lowest, oacc[d][r], oacc[d][r + 1]);
    // (sums from 2^-74 on over a total of up to 2^26 are results from 2^-100 on)
    if (__builtin_expect(__syncthreads_or(!(total > 0.0f && total <= 0x1p26f && wide <= 0x1p20f && lowest >= 0x1p-74f)), 0)) {
        float* const seen = (float*)smem;  // (the barrier above: nothing in LDS is read any more)
#pragma unroll
        for (int i = 1; i < 64; i *= 2) wide = fmaxf(wide, __shfl_xor(wide, i));
        if (lane == 0) seen[wave] = wide;
        __syncthreads();
        wide = fmaxf(fmaxf(seen[0], seen[1]), fmaxf(seen[2], seen[3]));
        const float low = fmaxf(0x1p-74f, wide * 0x1p-94f);
        bool again = !(total > 0.0f && total <= 0x1p120f && wide <= 0x1p100f && wide * fabsf(c) <= 0x1p90f), nothing = false;
#pragma unroll
        for (int d = 0; d < D32; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                again = again || zero_last(oacc[d][r]) < zero_last(low) || zero_last(oacc[d][r] * inv) < zero_last(0x1p-100f);
                nothing = nothing || oacc[d][r] == 0.0f;
            }
        again = again || (nothing && wide > 0x1p20f);
        // Channels of zeros, as padding leaves them, are told from small values by the values themselves, eight loads on their way at
        // a time: 2 x 8 x 1024 x 64 53 us, 47.6 without such channels (61 with one load at a time).
        if (__syncthreads_or(nothing)) {
            constexpr int AT_ONCE = 8;
            const int n = S * (D / 4);
            for (int u = tid; !again && u < n; u += 256 * AT_ONCE) {
                v4f x[AT_ONCE];
#pragma unroll
                for (int t = 0; t < AT_ONCE; ++t) {
                    const int w = u + 256 * t < n ? u + 256 * t : u;
                    x[t] = *(const v4f*)(vbase + (w / (D / 4)) * vss + w % (D / 4) * 16);
                }
#pragma unroll
                for (int t = 0; t < AT_ONCE; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) again = again || zero_last(x[t][e]) < zero_last(0x1p-126f);
            }
        }
        if (__syncthreads_or(again)) {
            typedef MhaStaged<OGC_F32, D32> T;
            mha_staged_body<OGC_F32, D32, FAST, PLAIN, 1, 1>(a, smem, smem + T::K_BYTES, (float*)(smem + T::K_BYTES + T::V_BYTES));
            return;
        }
    }
#pragma unroll
    for (int d = 0; d < D32; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] *= inv;
    uint8_t* op = a.o + (b * a.so[0] + hd * a.so[1] + (long long)query * a.so[2]) * 4;
#pragma unroll
    for (int d = 0; d < D32; ++d) {
        uint32_t dw[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float f = oacc[d][4 * g + e];  // (a bit cast of a vector's element itself reads element 0)
                dw[g][e] = __builtin_bit_cast(uint32_t, f);
            }
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

#endif
