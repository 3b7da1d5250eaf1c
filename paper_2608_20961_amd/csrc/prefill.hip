// treewy_chain_prefill kernel: the gated delta rule over a chain of T tokens,
// in chunks of 32 tokens, the state in registers from chunk to chunk.
//
// Per chunk (the chain form of the verify system, see verify.hip):
//   B[t,i] = beta_t (g_t/g_i) (k_t . k_i) (i < t),  A[t,i] = (g_t/g_i) (q_t . k_i) (i <= t)
//   T = (I + B)^{-1}                                 <- these need no state
//   P = [K; Q] S^T,  R = beta (V - g P_K),  U = T R,  O = g P_Q + A U
//   S <- g_N S + sum_l (g_N/g_l) U_l k_l^T           <- these do
//
// Work split.  The second group is the only serial chain, so a workgroup has
// two kinds of waves.  NS state waves each own 16 columns of d_v (16 rows of
// the state) and do nothing but the second group.  PW chunk waves prepare
// the chunks: chunk wave p takes chunks p, p + PW, ... whole (K/Q rows into
// LDS, decays, the two gram tiles, T, and T and A split into bf16 hi / lo
// planes), each in an LDS slot of its own, so that nothing but the barrier
// that ends each step passes between waves.  In step n the state waves run
// chunk n - PW + 1, the chunk wave whose slot that is leaves it alone (it
// scans the decays of its next chunk, whose rows are on their way into
// registers), and the other PW - 1 chunk waves are each one stage further
// with a later chunk.
//
// A unit is split over 8 / NS workgroups by d_v columns where there are too
// few units to fill the GPU: the columns are independent, the preparation is
// repeated.
#include "device.h"
#include "launch.h"
#include "mfma16.h"

namespace treewy {

namespace {

constexpr int CT = 32;                                   // tokens per chunk

// Order of a contraction index (d_k, or the chunk's tokens) in LDS: within
// each 32, entry 16 h + 4 g + r sits at position 8 g + 4 h + r.  Lane group g
// of a 16x16x32 product then reads, as its eight positions 8 g .. 8 g + 7, the
// entries 4 g + r of two 16-row accumulator tiles: what its registers hold.
//
// LDS of one chunk slot (bytes).  K and Q rows are 256 bytes, in 16-byte
// granules: granule G of row t is stored at G ^ swz(t), so that 16 rows read
// at the same granule, and the four rows by four granules of a transposed
// read, fall on distinct banks.
template <bool F32IN>
struct Slot {
    static constexpr int XROW = D * 2;
    static constexpr int X_BYTES = CT * XROW;
    static constexpr int K_OFF = 0, Q_OFF = X_BYTES;     // K and Q in bf16 ...
    static constexpr int LO = 2 * X_BYTES;               // ... and, past them, their low halves (fp32 tokens)
    static constexpr int PROW = CT * 2;                  // a plane's row: 64 bytes, see plane_at
    static constexpr int PLANE = CT * PROW;
    static constexpr int MS = CT + 4;                    // floats per row of B
    static constexpr int T_OFF = (F32IN ? 4 : 2) * X_BYTES;  // T hi, T lo; before them B in fp32
    static constexpr int A_OFF = T_OFF + CT * MS * 4;        // A hi, A lo
    static constexpr int G_OFF = A_OFF + 2 * PLANE;      // per token: decay g_t,
    static constexpr int BE_OFF = G_OFF + CT * 4;        // beta_t,
    static constexpr int W_OFF = BE_OFF + CT * 4;        // update weight g_N / g_t,
    static constexpr int INV_OFF = W_OFF + CT * 4;       // 1 / mantissa and
    static constexpr int E_OFF = INV_OFF + CT * 4;       // exponent of g_t (see DecayX)
    static constexpr int GN_OFF = E_OFF + CT * 4;        // g_N
    static constexpr int BYTES = GN_OFF + 16;
    static_assert(2 * PLANE <= CT * MS * 4, "T's planes fit where B in fp32 was");
    static_assert(T_OFF % 16 == 0 && A_OFF % 16 == 0 && G_OFF % 16 == 0 && BYTES % 16 == 0, "alignment");
};

// Byte offset of row t, token x in a plane of T or A: rows of four 16-byte
// granules in the order above, granule G at G ^ (swz(t) & 3), so that the lanes
// of two neighbouring groups that a 16-byte read serves together fall on
// distinct banks; no padding of the rows does that (see swz).  With swz, in
// place of rows of 80 bytes: 64 units of 777 fp32 tokens 81.6 -> 78.6 us, of
// 4096 bf16 tokens 168.1 -> 166.0.
__device__ __forceinline__ int plane_at(int t, int x) {
    return t * CT * 2 + ((((x >> 2) & 3) ^ (swz(t) & 3)) << 4) + ((x & 16) >> 1) + (x & 3) * 2;
}

// Waves of a workgroup by role.  Waves go round the CU's four SIMDs; with two
// state waves the workgroup is launched with eight, of which waves 4 and 5
// end at once, so that each state wave has a SIMD to itself and the chunk
// waves share the other two.
template <int NS> constexpr int launched_waves(int pw) { return NS == 2 ? 8 : NS + pw; }

template <bool F32IN, bool SBF, int NS, int PW>
__global__ __launch_bounds__(64 * launched_waves<NS>(PW), (launched_waves<NS>(PW) + 3) / 4) void prefill_kernel(
    const void *S0, const void *__restrict__ q_, const void *__restrict__ k_, const void *__restrict__ v_,
    const float *__restrict__ alpha, const float *__restrict__ beta, int T, int units, void *S_T,
    void *__restrict__ o_) {
    using In = typename std::conditional<F32IN, float, __bf16>::type;
    static_assert(!(SBF && F32IN), "a bf16 state is paired with bf16 inputs");
    static_assert(PW >= 2 && PW <= 4, "a chunk wave has one to three stages of LDS work");
    using L = Slot<F32IN>;
    constexpr int SPLIT = 8 / NS;                        // workgroups per unit
    constexpr int ROW = D * (int)sizeof(In);             // bytes per token row
    constexpr int XP = SPLIT > 1 ? CACHED : STREAM;      // (a unit's other workgroups read the same K/Q rows)
    constexpr int MS = L::MS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[PW * L::BYTES];

    // Whole units: the workgroup runs units u0, u0 + stride, ... as one
    // sequence of chunks, the next unit's chunks being prepared while the
    // state waves finish this one's.  Parts of units: one each, a unit's parts
    // on one XCD (consecutive workgroups go round the eight).
    int u0, part = 0, stride = units;
    if constexpr (SPLIT == 1) {
        u0 = blockIdx.x;
        stride = gridDim.x;
    } else {
        const int x = blockIdx.x & 7, y = blockIdx.x >> 3;
        part = y % SPLIT;
        u0 = (y / SPLIT) * 8 + x;
    }
    if (u0 >= units) return;                             // (uniform across the workgroup)

    const int hw_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (NS == 2 && (hw_wave == 4 || hw_wave == 5)) return;   // (see launched_waves; a wave that has ended is not waited for)
    const int wave = NS == 2 && hw_wave > 5 ? hw_wave - 2 : hw_wave;
    if (wave >= NS + PW) return;
    const int lane = threadIdx.x & 63;
    const int chunks = (T + CT - 1) / CT;
    const int steps = ((units - u0 + stride - 1) / stride) * chunks;   // chunks of all this workgroup's units
    auto tokens_of = [&](int c) { return T - CT * c < CT ? T - CT * c : CT; };
    auto row_of = [&](int u, int c) { return (size_t)u * T + (size_t)CT * c; };   // row of chunk c's first token

    // Every wave passes PW - 1 + steps barriers.
    if (wave < NS) {
        // ---- a state wave ---------------------------------------------------
        const int l16 = lane & 15, g = lane >> 4;
        const int col = 16 * (part * NS + wave) + l16;   // this lane's d_v column (= row of the state)
        // State tile jt: d_k 16 jt + 4 g + [0, 4), as floats or four bf16.
        using SReg = typename std::conditional<SBF, uint2, f32x4>::type;
        constexpr int SB = SBF ? 2 : 4;
        const int s_off = (col * D + 4 * g) * SB;
        SReg S[8], S_next[8];
        auto load_state = [&](int u, SReg (&X)[8]) {
            const rsrc_t rs = make_rsrc(static_cast<const char *>(S0) + (size_t)u * D * D * SB, D * D * SB);
#pragma unroll
            for (int jt = 0; jt < 8; ++jt) {
                if constexpr (SBF) X[jt] = ld_u32x2<CACHED>(rs, s_off + 16 * jt * SB);
                else X[jt] = ld_f32x4<CACHED>(rs, s_off + 16 * jt * SB);
            }
        };
        load_state(u0, S);
        using VT = typename std::conditional<F32IN, float, unsigned short>::type;
        VT vr[8];                                        // V at the accumulator positions, one chunk ahead
        auto load_v = [&](int u, int c) {
            const rsrc_t rv = make_rsrc(static_cast<const In *>(v_) + row_of(u, c) * D, tokens_of(c) * ROW);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int off = ((16 * (r >> 2) + 4 * g + (r & 3)) * D + col) * (int)sizeof(In);
                if constexpr (F32IN) vr[r] = ld_f32(rv, off);
                else vr[r] = __builtin_amdgcn_raw_buffer_load_b16(rv, off, 0, CACHED);
            }
        };
        load_v(u0, 0);
        // Lane part of the address of granule 4 s + g of row 16 m + l16 (s is
        // XORed in at bits 6 and 7), and of this lane's piece of a transposed
        // read: within each 16 lanes, lane 4 j + y points at four entries of
        // token row j and lane i receives column i of the 4 x 16 block.
        const int row_addr = l16 * L::XROW + ((g ^ swz(l16)) << 4);
        const int j4 = l16 >> 2, y = l16 & 3;
        const int tr_addr = (4 * g + j4) * L::XROW + ((y ^ swz(4 * g + j4)) << 4);
        const int plane_addr = plane_at(l16, 4 * g);     // granule g of row l16 of a plane
        for (int i = 0; i < PW - 1; ++i) __syncthreads();
        // (the serial chain: these waves go first at instruction issue)
        __builtin_amdgcn_s_setprio(2);
        int slot = 0;
        for (int u = u0; u < units; u += stride) {
        for (int c = 0; c < chunks; ++c) {
            if (SPLIT == 1 && c == chunks - 1 && u + stride < units) load_state(u + stride, S_next);
            unsigned char *sl = lds + slot * L::BYTES;
            auto row8 = [&](int off, int m, int s) {
                return *reinterpret_cast<const bf16x8 *>(sl + off + 16 * m * L::XROW + (row_addr ^ (s << 6)));
            };
            // P = [K; Q] S^T for this wave's columns; fp32 states (and tokens) as hi + lo.
            f32x4 pk[2] = {}, pq[2] = {};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bf16x8 bh, bl;
                if constexpr (SBF) {
                    bh = __builtin_bit_cast(bf16x8, make_uint4(S[2 * s].x, S[2 * s].y, S[2 * s + 1].x, S[2 * s + 1].y));
                } else {
                    float sv[8];
                    *reinterpret_cast<f32x4 *>(sv) = S[2 * s];
                    *reinterpret_cast<f32x4 *>(sv + 4) = S[2 * s + 1];
                    split8(sv, bh, bl);
                }
                bf16x8 ak[2], aq[2];
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    ak[m] = row8(L::K_OFF, m, s);
                    aq[m] = row8(L::Q_OFF, m, s);
                }
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    pk[m] = mma16(ak[m], bh, pk[m]);
                    pq[m] = mma16(aq[m], bh, pq[m]);
                }
                if constexpr (!SBF) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        pk[m] = mma16(ak[m], bl, pk[m]);
                        pq[m] = mma16(aq[m], bl, pq[m]);
                    }
                }
                if constexpr (F32IN) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        pk[m] = mma16(row8(L::LO + L::K_OFF, m, s), bh, pk[m]);
                        pq[m] = mma16(row8(L::LO + L::Q_OFF, m, s), bh, pq[m]);
                    }
                }
            }
            // R and g P_Q
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const f32x4 g4 = *reinterpret_cast<const f32x4 *>(sl + L::G_OFF + 4 * (16 * m + 4 * g));
                const f32x4 b4 = *reinterpret_cast<const f32x4 *>(sl + L::BE_OFF + 4 * (16 * m + 4 * g));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float vt;
                    if constexpr (F32IN) vt = vr[4 * m + e];
                    else vt = __builtin_bit_cast(float, (uint32_t)vr[4 * m + e] << 16);
                    pk[m][e] = b4[e] * (vt - g4[e] * pk[m][e]);
                    pq[m][e] *= g4[e];
                }
            }
            if (c + 1 < chunks) load_v(u, c + 1);
            else if (u + stride < units) load_v(u + stride, 0);
            // Plane product (T or A, rows 16 m + l16) with tokens x given as the
            // accumulator tiles hold them.
            auto plane_product = [&](int off, bf16x8 bh, bf16x8 bl, f32x4 (&acc)[2]) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const unsigned char *p = sl + off + 16 * m * L::PROW + plane_addr;
                    const bf16x8 ah = *reinterpret_cast<const bf16x8 *>(p);
                    const bf16x8 alo = *reinterpret_cast<const bf16x8 *>(p + L::PLANE);
                    acc[m] = mma16(ah, bh, acc[m]);
                    acc[m] = mma16(ah, bl, acc[m]);
                    acc[m] = mma16(alo, bh, acc[m]);
                }
            };
            bf16x8 xh, xl;
            float x8[8];
            *reinterpret_cast<f32x4 *>(x8) = pk[0];
            *reinterpret_cast<f32x4 *>(x8 + 4) = pk[1];
            split8(x8, xh, xl);
            f32x4 uu[2] = {};
            plane_product(L::T_OFF, xh, xl, uu);         // U = T R
            // S <- g_N S + K^T (w U): the product's rows over d_k are this
            // lane's state entries, so it accumulates onto the scaled state.
            const float gN = *reinterpret_cast<const float *>(sl + L::GN_OFF);
            bf16x8 wh, wl;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const f32x4 w4 = *reinterpret_cast<const f32x4 *>(sl + L::W_OFF + 4 * (16 * m + 4 * g));
#pragma unroll
                for (int e = 0; e < 4; ++e) x8[4 * m + e] = uu[m][e] * w4[e];
            }
            split8(x8, wh, wl);
            auto kt = [&](int off, int jt) {             // rows d_k 16 jt + l16 of K^T at tokens 16 h + 4 g + r
                s16x4 a[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    a[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_s16x4 *)(sl + off + 16 * h * L::XROW + 8 * (jt & 1) + (tr_addr ^ ((jt >> 1) << 6))));
                return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a[0], a[1], 0, 1, 2, 3, 4, 5, 6, 7));
            };
#pragma unroll
            for (int jt = 0; jt < 8; ++jt) {
                f32x4 d;
                if constexpr (SBF) d = bf4_to_f32(S[jt]);
                else d = S[jt];
#pragma unroll
                for (int e = 0; e < 4; ++e) d[e] *= gN;
                const bf16x8 a = kt(L::K_OFF, jt);
                d = mma16(a, wh, d);
                d = mma16(a, wl, d);
                if constexpr (F32IN) d = mma16(kt(L::LO + L::K_OFF, jt), wh, d);
                if constexpr (SBF) S[jt] = f32_to_bf4(d);
                else S[jt] = d;
            }
            *reinterpret_cast<f32x4 *>(x8) = uu[0];
            *reinterpret_cast<f32x4 *>(x8 + 4) = uu[1];
            split8(x8, xh, xl);
            plane_product(L::A_OFF, xh, xl, pq);         // O = g P_Q + A U
            const rsrc_t ro = make_rsrc(static_cast<In *>(o_) + row_of(u, c) * D, tokens_of(c) * ROW);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int off = ((16 * m + 4 * g) * D + col) * (int)sizeof(In);
                if constexpr (F32IN) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) st_f32<CACHED>(ro, off + e * ROW, pq[m][e]);
                } else {
                    // (parts of a line: the default policy lets L2 merge the neighbouring waves')
#pragma unroll
                    for (int e = 0; e < 4; e += 2) {
                        const uint32_t pr = pack_bf2(pq[m][e], pq[m][e + 1]);
                        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)pr, ro, off + e * ROW, 0, CACHED);
                        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(pr >> 16), ro, off + (e + 1) * ROW, 0, CACHED);
                    }
                }
            }
            slot = slot + 1 < PW ? slot + 1 : 0;
            __syncthreads();
        }
        const rsrc_t rn = make_rsrc(static_cast<char *>(S_T) + (size_t)u * D * D * SB, D * D * SB);
#pragma unroll
        for (int jt = 0; jt < 8; ++jt) {
            if constexpr (SBF) st_u32x2<CACHED>(rn, s_off + 16 * jt * SB, S[jt]);
            else st_u32x4<CACHED>(rn, s_off + 16 * jt * SB, __builtin_bit_cast(uint4, S[jt]));
            S[jt] = S_next[jt];
        }
        }                                                // unit
    } else {
        // ---- a chunk wave ---------------------------------------------------
        const int p = wave - NS, l32 = lane & 31, hg = lane >> 5;
        unsigned char *sl = lds + p * L::BYTES;
        float *Bm = reinterpret_cast<float *>(sl + L::T_OFF);
        // Lane part of the address of granule 2 s + hg of row l32 (s is XORed in: bits 5 to 7).
        const int row_addr = l32 * L::XROW + ((hg ^ swz(l32)) << 4);
        constexpr int KN = CT * ROW / 16 / 64;           // 16-byte pieces of K (and of Q) per lane
        uint4 kr[KN], qr[KN];
        float al, be;
        auto load = [&](int u, int c) {
            const int n = tokens_of(c);
            const size_t r0 = row_of(u, c);
            al = ld_f32(make_rsrc(alpha + r0, n * 4), lane * 4);
            be = ld_f32(make_rsrc(beta + r0, n * 4), lane * 4);
            const rsrc_t rk = make_rsrc(static_cast<const In *>(k_) + r0 * D, n * ROW);
            const rsrc_t rq = make_rsrc(static_cast<const In *>(q_) + r0 * D, n * ROW);
#pragma unroll
            for (int i = 0; i < KN; ++i) kr[i] = ld_u32x4<XP>(rk, (lane + 64 * i) * 16);
#pragma unroll
            for (int i = 0; i < KN; ++i) qr[i] = ld_u32x4<XP>(rq, (lane + 64 * i) * 16);
        };
        // 16 bytes of a row into the slot at `off`, d_k in the order above.
        auto stage = [&](int off, int i, const uint4 &x) {
            if constexpr (!F32IN) {
                const int r = (lane >> 4) + 4 * i, c = lane & 15;    // d_k 8c .. 8c + 7
                unsigned char *row = sl + off + r * L::XROW + ((c >> 1) & 1) * 8;
                const int G = 4 * (c >> 2) + 2 * (c & 1);
                *reinterpret_cast<uint2 *>(row + ((G ^ swz(r)) << 4)) = make_uint2(x.x, x.y);
                *reinterpret_cast<uint2 *>(row + (((G + 1) ^ swz(r)) << 4)) = make_uint2(x.z, x.w);
            } else {
                const int r = (lane >> 5) + 2 * i, c = lane & 31;    // d_k 4c .. 4c + 3
                uint2 hi, lo;
                split4(__builtin_bit_cast(f32x4, x), hi, lo);
                unsigned char *row = sl + off + r * L::XROW + ((c >> 2) & 1) * 8 +
                                     (((4 * (c >> 3) + (c & 3)) ^ swz(r)) << 4);
                *reinterpret_cast<uint2 *>(row) = hi;
                *reinterpret_cast<uint2 *>(row + L::LO) = lo;
            }
        };
        // Decays of a chunk of n tokens from its gates in al: inclusive prefix
        // products, in extended range (lane t: token t), and what follows from them.
        float inv = 0.f, bl = 0.f, gt = 0.f, wt = 0.f, gN = 0.f, mt = 0.f, bt = 0.f;
        int pe = 0, et = 0;
        auto scan = [&](int n) {
            float pm = lane < n ? DecayX::mant(al) : 0.f;
            pe = lane < n ? DecayX::expo(al) : 0;
#pragma unroll
            for (int off = 1; off < CT; off <<= 1) {
                const float ym = __shfl_up(pm, off);
                const int ye = __shfl_up(pe, off);
                if (lane >= off && lane < n) DecayX::mul(pm, pe, ym, ye);
            }
            const float mN = __shfl(pm, n - 1);
            const int eN = __shfl(pe, n - 1);
            inv = lane < n ? 1.f / pm : 0.f;
            bl = lane < n ? be : 0.f;
            gt = DecayX::value(pm, pe);
            wt = DecayX::ratio(mN, eN, inv, pe);         // (0 past the chunk)
            gN = DecayX::value(mN, eN);
            mt = __shfl(pm, l32);
            bt = __shfl(bl, l32);
            et = __shfl(pe, l32);
        };
        int passed = 0;                                  // barriers passed
        auto step_end = [&]() {
            __syncthreads();
            ++passed;
        };
        // This wave's chunks: p, p + PW, ... of the workgroup's sequence.
        int u = u0, c = p;
        auto settle = [&](int &u, int &c) {              // chunk c counted from unit u -> unit and chunk
            while (c >= chunks && u < units) {
                c -= chunks;
                u += stride;
            }
        };
        settle(u, c);
        if (u < units) {
            load(u, c);
            scan(tokens_of(c));
        }
        for (int i = 0; i < p; ++i) step_end();
        while (u < units) {
            const int n = tokens_of(c);
            int un = u, cn = c + PW;                     // the next one
            settle(un, cn);
            if (lane < CT) {
                *reinterpret_cast<float *>(sl + L::G_OFF + 4 * lane) = gt;
                *reinterpret_cast<float *>(sl + L::BE_OFF + 4 * lane) = bl;
                *reinterpret_cast<float *>(sl + L::W_OFF + 4 * lane) = wt;
                *reinterpret_cast<float *>(sl + L::INV_OFF + 4 * lane) = inv;
                *reinterpret_cast<int *>(sl + L::E_OFF + 4 * lane) = pe;
                if (lane == 0) *reinterpret_cast<float *>(sl + L::GN_OFF) = gN;
            }
#pragma unroll
            for (int i = 0; i < KN; ++i) stage(L::K_OFF, i, kr[i]);
#pragma unroll
            for (int i = 0; i < KN; ++i) stage(L::Q_OFF, i, qr[i]);
            lds_order();
            if (un < units) load(un, cn);
            // The gram tiles with token t = l32 along the lanes and i down the
            // rows: a lane's entries come in runs of four i of one row of B and A.
            f32x16 gk = {}, gq = {};
#pragma unroll 2
            for (int s = 0; s < 8; ++s) {
                const unsigned char *row = sl + (row_addr ^ (s << 5));
                const bf16x8 ak = *reinterpret_cast<const bf16x8 *>(row + L::K_OFF);
                const bf16x8 aq = *reinterpret_cast<const bf16x8 *>(row + L::Q_OFF);
                gk = mma(ak, ak, gk);
                gq = mma(ak, aq, gq);
                if constexpr (F32IN) {
                    const bf16x8 akl = *reinterpret_cast<const bf16x8 *>(row + L::LO + L::K_OFF);
                    const bf16x8 aql = *reinterpret_cast<const bf16x8 *>(row + L::LO + L::Q_OFF);
                    gk = mma(akl, ak, gk);
                    gk = mma(ak, akl, gk);
                    gq = mma(akl, aq, gq);
                    gq = mma(ak, aql, gq);
                }
            }
            if constexpr (PW == 4) step_end();
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int i0 = acc_row(4 * q4, hg);      // i0 .. i0 + 3
                const f32x4 inv4 = *reinterpret_cast<const f32x4 *>(sl + L::INV_OFF + 4 * i0);
                const int4 e4 = *reinterpret_cast<const int4 *>(sl + L::E_OFF + 4 * i0);
                f32x4 bv, av;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (rows past the chunk's last token come out zero: their gates and keys are)
                    const int i = i0 + e, ei = e == 0 ? e4.x : e == 1 ? e4.y : e == 2 ? e4.z : e4.w;
                    const float rs = DecayX::ratio(mt, et, inv4[e], ei);
                    const float ratio = i < l32 ? rs : (i == l32 ? 1.f : 0.f);
                    bv[e] = i < l32 ? bt * rs * gk[4 * q4 + e] : 0.f;
                    // (rounded to fp32 here: the split below must not fuse this product into its lo)
                    float a = ratio * gq[4 * q4 + e];
                    asm("" : "+v"(a));
                    av[e] = a;
                }
                *reinterpret_cast<f32x4 *>(Bm + l32 * MS + i0) = bv;
                uint2 hi, lo;
                split4(av, hi, lo);
                unsigned char *a = sl + L::A_OFF + plane_at(l32, i0);
                *reinterpret_cast<uint2 *>(a) = hi;
                *reinterpret_cast<uint2 *>(a + L::PLANE) = lo;
            }
            lds_order();
            if constexpr (PW >= 3) step_end();
            // T = (I + B)^{-1}: the two 16-row diagonal blocks by the sweep, on
            // lanes 0 to 31, then the block below them, T10 = -T1 (B10 T0), on
            // the matrix cores, in pairs of bf16 as verify.hip has it for more
            // than 16 ancestors.  For at most 16 that kernel's solve is in
            // fp32: there B10 and B10 T0 stand as three bf16 each (in pairs a last
            // chunk of 17 tokens with close keys came out 4 to 7% further off;
            // in three everywhere whole units took 1 to 2% longer).  The planes
            // go over B's fp32 rows, read before.
            // Lanes 32 to 63 sweep the zeros above the diagonal blocks and
            // write these, and zeros where T10 goes.
            {
                const int bq = (lane >> 4) & 1, tl = lane & 15, g = lane >> 4;
                const float *Bb = hg ? Bm + tl * MS + 16 : Bm + l32 * MS + 16 * bq;
                float b[16], r[16];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const f32x4 v4 = *reinterpret_cast<const f32x4 *>(Bb + 4 * x);
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[4 * x + e] = r[4 * x + e] = v4[e];
                }
                // B10[tl][4 g + e] in slots e of lane group g (slots 4 to 7 stay empty)
                const f32x4 b10 = *reinterpret_cast<const f32x4 *>(Bm + (16 + tl) * MS + 4 * g);
                lds_order();
                sweep16<15>(r, b, tl);
                unsigned char *th = sl + L::T_OFF;
#pragma unroll
                for (int x = 0; x < 4; ++x) {            // entries 16 bq + 4 x + [0, 4)
                    uint2 hi, lo;
                    split4(f32x4{r[4 * x], r[4 * x + 1], r[4 * x + 2], r[4 * x + 3]}, hi, lo);
                    unsigned char *t = th + plane_at(l32, 16 * (bq ^ hg) + 4 * x);
                    *reinterpret_cast<uint2 *>(t) = hi;
                    *reinterpret_cast<uint2 *>(t + L::PLANE) = lo;
                }
                if (lane < n) *reinterpret_cast<unsigned short *>(th + plane_at(lane, lane)) = 0x3F80;   // 1 on the diagonal
                lds_order();
                // Rows 4 g + e of T0, column tl (a transposed read), and of T1, row tl.
                const unsigned char *t0 = th + plane_at(4 * g + (tl >> 2), 4 * (tl & 3));
                const unsigned char *t1 = th + plane_at(16 + tl, 16 + 4 * g);
                const bf16x8 t0h = low8(__builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)t0)));
                const bf16x8 t0l =
                    low8(__builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(t0 + L::PLANE))));
                const bf16x8 t1h = low8(*reinterpret_cast<const uint2 *>(t1));
                const bf16x8 t1l = low8(*reinterpret_cast<const uint2 *>(t1 + L::PLANE));
                // (in pairs; the third parts where at most 16 tokens precede one, see above)
                const bool third = n <= 17;
                uint2 hi, lo, rest;
                split4(b10, hi, lo);
                f32x4 acc = {};
                acc = mma16(low8(hi), t0h, acc);
                acc = mma16(low8(hi), t0l, acc);
                acc = mma16(low8(lo), t0h, acc);         // B10 T0: rows 4 g + e, column tl
                if (third) {
                    split4(b10, hi, lo, rest);
                    acc = mma16(low8(lo), t0l, acc);
                    acc = mma16(low8(rest), t0h, acc);
                }
                const f32x4 b10t0 = acc;
                split4(b10t0, hi, lo);
                acc = f32x4{};
                acc = mma16(t1h, low8(hi), acc);
                acc = mma16(t1h, low8(lo), acc);
                acc = mma16(t1l, low8(hi), acc);
                if (third) {
                    split4(b10t0, hi, lo, rest);
                    acc = mma16(t1l, low8(lo), acc);
                    acc = mma16(t1h, low8(rest), acc);
                }
                split4(-acc, hi, lo);
                unsigned char *w = th + plane_at(16 + 4 * g, tl);   // (rows 16 + 4 g + e: the same granule)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t h2 = e < 2 ? hi.x : hi.y, l2 = e < 2 ? lo.x : lo.y;
                    *reinterpret_cast<unsigned short *>(w + e * L::PROW) = (unsigned short)(e & 1 ? h2 >> 16 : h2);
                    *reinterpret_cast<unsigned short *>(w + e * L::PROW + L::PLANE) = (unsigned short)(e & 1 ? l2 >> 16 : l2);
                }
            }
            step_end();                                  // the slot is whole: the state waves run it in the next step
            if (un < units) scan(tokens_of(cn));
            step_end();                                  // ... and are done with it
            u = un;
            c = cn;
        }
        while (passed < PW - 1 + steps) step_end();
    }
}

template <bool F32IN, bool SBF, int NS, int PW>
hipError_t launch(const void *S0, const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                  int T, int units, int cus, void *S_T, void *o, hipStream_t stream) {
    constexpr int SPLIT = 8 / NS;
    const unsigned grid =
        SPLIT == 1 ? (unsigned)(units < cus ? units : cus) : (unsigned)((units + 7) / 8 * 8 * SPLIT);
    hipLaunchKernelGGL((prefill_kernel<F32IN, SBF, NS, PW>), dim3(grid), dim3(64 * launched_waves<NS>(PW)), 0, stream, S0,
                       q, k, v, alpha, beta, T, units, S_T, o);
    return hipGetLastError();
}

}  // namespace

// One workgroup of this kernel runs on a CU, so a unit goes to four
// workgroups where that fills at most the GPU (a quarter of the CUs' number
// of units), to two up to half, and otherwise the resident workgroups walk
// the units whole.  With bf16 tokens a chunk step takes 1.3 us with a quarter or
// half of a unit per workgroup (one 4096-token sequence of 64 heads: 606 -> 166
// us, against verify.hip's kernel, one workgroup of four like waves per unit;
// bound by the state waves' serial chain) and 2.2 to 2.5 us with a whole one (32
// sequences of 1000 tokens, 64 heads, bf16 state: 807 -> 633 us).  With fp32 tokens
// a step takes 2.9 us (64 units of 777 tokens: 185 -> 78.6 us): there the chunk
// waves set the pace, each loading, splitting and staging 32 KB of K and Q and
// making three products for one, with three slots in LDS instead of four.
//   bf16 tokens, one chunk: the kernels of verify.hip and small.hip, whose chunk is bit for bit a verify
//     (small.hip's limit is one for both calls).
//   Whole units of few chunks: it too, two of its workgroups per CU hide the
//     latency of a short unit (512 units of 64 tokens: 25.4 against 26.5 us; of
//     512 tokens: 124 against 105 us; in one round of at most as many units as
//     CUs two chunks suffice: 256 units of 64 tokens, 17.9 against 16.5 us).
//   fp32 tokens in whole units: it too (the chunk waves' fp32 rows do not fit
//     beside eight state waves; 256 units of 512 tokens: 132 against 135 us in halves).
hipError_t launch_prefill(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                          const float *beta, int T, int B, int H, bool f32_in, bool bf16_state, void *S_T, void *o,
                          int32_t *err, hipStream_t stream) {
    const int units = B * H, cus = compute_units();
    if (small_prefill_fits(T, units, f32_in))
        return launch_small_prefill(S0, q, k, v, alpha, beta, T, B, H, bf16_state, S_T, o, stream);
    const bool quarters = (int64_t)units * 4 <= cus, halves = (int64_t)units * 2 <= cus;
    const int chunks = (T + CT - 1) / CT;
    const bool whole = !f32_in && chunks >= (units <= cus ? 2 : 5);
    if ((!f32_in && chunks == 1) || !(halves || whole))
        return launch_prefill_unit(S0, q, k, v, alpha, beta, T, B, H, f32_in, bf16_state, S_T, o, err, stream);
#define TREEWY_PREFILL(F, S, NS, PW) launch<F, S, NS, PW>(S0, q, k, v, alpha, beta, T, units, cus, S_T, o, stream)
    if (f32_in) return quarters ? TREEWY_PREFILL(true, false, 2, 3) : TREEWY_PREFILL(true, false, 4, 3);
    if (bf16_state)
        return quarters ? TREEWY_PREFILL(false, true, 2, 4)
                        : halves ? TREEWY_PREFILL(false, true, 4, 4) : TREEWY_PREFILL(false, true, 8, 4);
    return quarters ? TREEWY_PREFILL(false, false, 2, 4)
                    : halves ? TREEWY_PREFILL(false, false, 4, 4) : TREEWY_PREFILL(false, false, 8, 4);
#undef TREEWY_PREFILL
}

}  // namespace treewy
