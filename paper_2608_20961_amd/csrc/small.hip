// Few units: drafts of at most 48 nodes (treewy_verify, treewy_commit_verify),
// chains of at most 32 tokens (treewy_chain_prefill) and treewy_commit: the system
// of verify.hip on 16-row tiles, every wave on its own.  Bound by the latency of
// the wave's reads and of its steps.
//
// A wave owns 16 columns of d_v (16 rows of the state) of one unit and needs
// nothing of the other seven: K and Q rows come from memory in operand
// layout, and the gram tiles, the ancestors and T = (I + B)^{-1} are so small
// at 16 nodes that every wave forms its own.  So there is no LDS and no
// barrier, and the chain of a wave is: its reads, the walk and the gram while
// the state arrives, the sweep for T in registers, P, U = T R, O, the stores.
// The four 16-lane rows of a wave hold the tree four times over (lane % 16 =
// node): the sweep broadcasts within a row, and what lane group g needs of
// nodes 4 g .. 4 g + 3 is in its own row.
//
// Contraction order: slots 8 g + e of a 16x16x32 product over d_k are
// d_k 32 s + 8 g + e; over the nodes, slots e < 4 of lane group g are node 4 g +
// e, what an accumulator tile holds, and slots e >= 4 are empty.
#include "device.h"
#include "launch.h"
#include "mfma16.h"

namespace treewy {

namespace {

constexpr int VERIFY = 0, FUSED = 1, PREFILL = 2;
constexpr int NW = 4;                                    // waves per workgroup
constexpr int PARTS = D / 16 / NW;                       // workgroups per unit

// Value x[r] of lane group gg (0 .. 3) in every group, for the four groups of each lane % 16:
// out[4 gg + r].
__device__ __forceinline__ void all_groups(const f32x4 &x, float (&out)[16]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float xr = x[r];
        const int v = __builtin_bit_cast(int, xr);
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // groups 0, 0, 2, 2 and 1, 1, 3, 3
        const int even = p[0], odd = p[1];
        const auto a = __builtin_amdgcn_permlane32_swap(even, even, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(odd, odd, false, false);
        const int g0 = a[0], g2 = a[1], g1 = b[0], g3 = b[1];
        out[r] = __builtin_bit_cast(float, g0);
        out[4 + r] = __builtin_bit_cast(float, g1);
        out[8 + r] = __builtin_bit_cast(float, g2);
        out[12 + r] = __builtin_bit_cast(float, g3);
    }
}

__device__ __forceinline__ void floats8(uint4 a, uint4 b, float (&x)[8]) {
    const f32x4 f = __builtin_bit_cast(f32x4, a), h = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = f[e];
        x[4 + e] = h[e];
    }
}

// A wave's rows of the state: lane (l16, g) holds d_k 32 s + 8 g + [0, 8) of row `col`.
template <bool SBF>
struct State {
    static constexpr int SB = SBF ? 2 : 4, SN = SBF ? 1 : 2;     // bytes per entry, 16-byte pieces per eight
    uint4 x[4][SN];
    int col, g;
    __device__ __forceinline__ State(int col, int g) : col(col), g(g) {}

    __device__ __forceinline__ void load(const void *S0, int u) {
        const rsrc_t rs = make_rsrc(static_cast<const char *>(S0) + (size_t)u * D * D * SB, D * D * SB);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int p = 0; p < SN; ++p) x[s][p] = ld_u32x4<CACHED>(rs, (col * D + 32 * s + 8 * g) * SB + 16 * p);
    }
    __device__ __forceinline__ void get(float (&f)[4][8], float scale) const {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (SBF) {
                const uint32_t w[4] = {x[s][0].x, x[s][0].y, x[s][0].z, x[s][0].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f[s][2 * e] = scale * __builtin_bit_cast(float, w[e] << 16);
                    f[s][2 * e + 1] = scale * __builtin_bit_cast(float, w[e] & 0xffff0000u);
                }
            } else {
                floats8(x[s][0], x[s][SN - 1], f[s]);
#pragma unroll
                for (int e = 0; e < 8; ++e) f[s][e] *= scale;
            }
        }
    }
    __device__ __forceinline__ void put(const float (&f)[4][8]) {   // (a bf16 state is rounded here)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (SBF) {
                x[s][0] = __builtin_bit_cast(uint4, round8(f[s]));
            } else {
                x[s][0] = __builtin_bit_cast(uint4, f32x4{f[s][0], f[s][1], f[s][2], f[s][3]});
                x[s][SN - 1] = __builtin_bit_cast(uint4, f32x4{f[s][4], f[s][5], f[s][6], f[s][7]});
            }
        }
    }
    // Out: an fp32 state's 16-byte pieces go round the lane groups first, so
    // that each store instruction writes 64 bytes of a row together.
    __device__ __forceinline__ void store(void *S_new, int u) const {
        const rsrc_t rn = make_rsrc(static_cast<char *>(S_new) + (size_t)u * D * D * SB, D * D * SB);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (SBF) {
                st_u32x4<CACHED>(rn, (col * D + 32 * s + 8 * g) * SB, x[s][0]);
            } else {                                     // pieces 2 g, 2 g + 1 of eight -> pieces g and 4 + g
                uint32_t a[4] = {x[s][0].x, x[s][0].y, x[s][0].z, x[s][0].w};
                uint32_t c[4] = {x[s][1].x, x[s][1].y, x[s][1].z, x[s][1].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const auto i = __builtin_amdgcn_permlane16_swap(a[e], c[e], false, false);   // pieces 0 1 4 5 | 2 3 6 7
                    const uint32_t i0 = i[0], i1 = i[1];
                    const auto j = __builtin_amdgcn_permlane32_swap(i0, i1, false, false);       // pieces 0 1 2 3 | 4 5 6 7
                    a[e] = j[0];
                    c[e] = j[1];
                }
                const int off = (col * D + 32 * s + 4 * g) * 4;
                st_u32x4<CACHED>(rn, off, make_uint4(a[0], a[1], a[2], a[3]));
                st_u32x4<CACHED>(rn, off + 64, make_uint4(c[0], c[1], c[2], c[3]));
            }
        }
    }
};

// x[i] += u k[i], i = 0 .. 15, where k[2 j], k[2 j + 1] are the values k0, k1 of
// lane L + j of each row of 16 lanes (see fmac_bcast).
template <int L> __device__ __forceinline__ void rank1_half(float (&x0)[8], float (&x1)[8], float k0, float k1, float u) {
#define TW_F(n, m, j) "v_fmac_f32_dpp %" #n ", %" #m ", %[u] row_newbcast:%[i" #j "] row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" TW_F(0, 16, 0) TW_F(1, 17, 0) TW_F(2, 16, 1) TW_F(3, 17, 1) TW_F(4, 16, 2) TW_F(5, 17, 2)
        TW_F(6, 16, 3) TW_F(7, 17, 3) TW_F(8, 16, 4) TW_F(9, 17, 4) TW_F(10, 16, 5) TW_F(11, 17, 5) TW_F(12, 16, 6)
        TW_F(13, 17, 6) TW_F(14, 16, 7) TW_F(15, 17, 7)
        : "+&v"(x0[0]), "+&v"(x0[1]), "+&v"(x0[2]), "+&v"(x0[3]), "+&v"(x0[4]), "+&v"(x0[5]), "+&v"(x0[6]), "+&v"(x0[7]),
          "+&v"(x1[0]), "+&v"(x1[1]), "+&v"(x1[2]), "+&v"(x1[3]), "+&v"(x1[4]), "+&v"(x1[5]), "+&v"(x1[6]), "+&v"(x1[7])
        : "v"(k0), "v"(k1), [u] "v"(u), [i0] "n"(L), [i1] "n"(L + 1), [i2] "n"(L + 2), [i3] "n"(L + 3), [i4] "n"(L + 4),
          [i5] "n"(L + 5), [i6] "n"(L + 6), [i7] "n"(L + 7));
#undef TW_F
}

// NK entries of a path, read together so that one latency covers them: the key
// row, two values a lane, and the pseudo-value of this lane's column.  Lane
// (l16, g) holds d_k 32 (l16 / 4) + 8 g + 2 (l16 % 4) + [0, 2), so the 32 values
// that lane group g needs (those of its state entries) are in its own 16 lanes, and the
// multiply-adds take them by a row broadcast.  (With each lane holding all
// of its 32 values, a key row was four or eight reads and as many registers,
// and a path of 64 entries a chain of 16 or 32 latencies: the fused call of 128
// units of 8 nodes took 21.8 us with bf16 and 30.5 us with fp32 tokens.)
template <bool F32IN, int NK>
struct Keys {
    static constexpr int SZ = F32IN ? 4 : 2;
    using KT = typename std::conditional<F32IN, uint2, uint32_t>::type;
    KT k[NK];
    float u[NK];
    // x += wu k^T
    __device__ __forceinline__ void rank1(float (&x)[4][8], float wu, int e) const {
        float k0, k1;
        if constexpr (F32IN) {
            const uint32_t a = k[e].x, b = k[e].y;
            k0 = __builtin_bit_cast(float, a);
            k1 = __builtin_bit_cast(float, b);
        } else {
            k0 = __builtin_bit_cast(float, k[e] << 16);
            k1 = __builtin_bit_cast(float, k[e] & 0xffff0000u);
        }
        rank1_half<0>(x[0], x[1], k0, k1, wu);
        rank1_half<8>(x[2], x[3], k0, k1, wu);
    }
};

// An accepted path of at most 64 nodes of a draft of at most 64 (lane l = entry
// l; alpha and parent of node = lane).
struct Path {
    rsrc_t rk, ru;
    int len, node, par, row;
    float al, w, ga;                                     // w: of entry l; ga: the product of alpha over the path

    __device__ __forceinline__ void issue(const CommitArgs &cm, int u, int b, int in_size) {
        const int lane = threadIdx.x & 63, np = cm.N_prev;
        row = D * in_size;
        rk = make_rsrc(static_cast<const char *>(cm.k) + (size_t)u * cm.in_stride * row, np * row);
        ru = make_rsrc(cm.U + (size_t)u * cm.u_stride * D, np * D * 4);
        al = ld_f32(make_rsrc(cm.alpha + (size_t)u * cm.in_stride, np * 4), lane * 4);
        // (an opaque zero offset: a uniform load's result would be moved to a scalar register at once)
        len = ld_i32(make_rsrc(cm.path_len + b, 4), opaque(0));
        node = ld_i32(make_rsrc(cm.path + (size_t)b * cm.L_max, cm.L_max * 4), lane * 4);
        const int32_t *pp = cm.parent;
        par = ld_i32(make_rsrc(pp ? pp + (size_t)b * np : nullptr, pp ? np * 4 : 0), lane * 4);
    }
    // Entry l lies in [0, N), follows entry l - 1 in index order and (with a
    // parent array) is its child, entry 0 a child of the committed prefix.  A
    // bad path commits nothing.
    __device__ __forceinline__ void check(const CommitArgs &cm, int b, bool first, int32_t *err) {
        const int lane = threadIdx.x & 63;
        const bool len_ok = len >= 0 && len <= cm.L_max;
        const int n = len_ok ? len : 0;
        const int a = lane < n ? node : -1;
        const int before = __shfl(a, lane > 0 ? lane - 1 : 0);
        const int pa = lane == 0 ? -1 : before;
        const int src = (a >= 0 && a < 64) ? a : lane;
        const int par_a = __shfl(par, src);
        const float al_a = __shfl(al, src);
        bool bad = !len_ok;
        if (lane < n) bad = bad || a < 0 || a >= cm.N_prev || a <= pa || (cm.parent && par_a != pa);
        const bool ok = !__any(bad);
        len = __builtin_amdgcn_readfirstlane(ok ? n : 0);
        if (!ok && first && lane == 0) flag_error(err, b, TREEWY_FLAG_BAD_PATH);
        float x = lane < len ? al_a : 1.f;               // suffix products of the gates
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const float y = __shfl_down(x, off);
            x *= lane + off < 64 ? y : 1.f;
        }
        const float after = __shfl_down(x, 1);
        w = lane < len ? (lane + 1 < 64 ? after : 1.f) : 0.f;
        ga = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
    }
    // Entries l0 .. of the path (past it: an offset past the end, which reads zero).
    template <bool F32IN, int NK>
    __device__ __forceinline__ void load(Keys<F32IN, NK> &x, int l0, int g, int col) const {
        constexpr int OOB = 1 << 30;
        const int l16 = threadIdx.x & 15, off = (32 * (l16 >> 2) + 8 * g + 2 * (l16 & 3)) * x.SZ;
#pragma unroll
        for (int e = 0; e < NK; ++e) {
            const bool live = l0 + e < len;              // (uniform)
            const int a = __builtin_amdgcn_readlane(node, (l0 + e) & 63);
            if constexpr (F32IN) x.k[e] = ld_u32x2<CACHED>(rk, (live ? a * row : OOB) + off);
            else x.k[e] = (uint32_t)ld_i32(rk, (live ? a * row : OOB) + off);
            x.u[e] = ld_f32(ru, live ? (a * D + col) * 4 : OOB);
        }
    }
    __device__ __forceinline__ float weight(int l) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), l & 63));
    }
};

// S <- g_a S + sum_l w_l U_l k_l^T over the path, entry after entry; the first are in `keys`, the others come
// MORE at a time while those before them are added.
constexpr int FIRST = 8, MORE = 16;
template <bool F32IN, bool SBF>
__device__ __forceinline__ void commit_path(State<SBF> &st, const Path &path, const Keys<F32IN, FIRST> &keys) {
    if (path.len == 0) return;                           // (uniform; the state stays as it is, bit for bit)
    Keys<F32IN, MORE> now, next;
    if (path.len > FIRST) path.load(now, FIRST, st.g, st.col);
    float x[4][8];
    st.get(x, path.ga);
#pragma unroll
    for (int e = 0; e < FIRST; ++e)
        if (e < path.len) keys.rank1(x, path.weight(e) * keys.u[e], e);
    for (int l0 = FIRST; l0 < path.len; l0 += MORE) {
        if (l0 + MORE < path.len) path.load(next, l0 + MORE, st.g, st.col);
#pragma unroll
        for (int e = 0; e < MORE; ++e)
            if (l0 + e < path.len) now.rank1(x, path.weight(l0 + e) * now.u[e], e);
        now = next;
    }
    st.put(x);
}

template <bool F32IN, bool SBF, int MODE>
__global__ __launch_bounds__(64 * NW) void small_kernel(
    const void *S0, const void *__restrict__ q_, const void *__restrict__ k_, const void *__restrict__ v_,
    const float *__restrict__ alpha, const float *__restrict__ beta, const int32_t *__restrict__ parent, int N, int H,
    int units, void *__restrict__ o_, float *U, int32_t *__restrict__ err, CommitArgs cm) {
    using In = typename std::conditional<F32IN, float, __bf16>::type;
    static_assert(!(SBF && F32IN), "a bf16 state is paired with bf16 inputs");
    constexpr int ROW = D * (int)sizeof(In);
    // A unit's workgroups sit on one XCD (consecutive workgroups go round the
    // eight), so that its K and Q rows are read from memory once.
    const int bx = blockIdx.x & 7, by = blockIdx.x >> 3;
    const int part = by % PARTS, u = (by / PARTS) * 8 + bx;
    if (u >= units) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int b = u / H, col = 16 * (part * NW + wave) + l16;    // this lane's d_v column (= row of the state)
    State<SBF> st(col, g);
    const bool first = part == 0 && wave == 0;                   // the wave that reports what is malformed
    const size_t node0 = (size_t)u * N;

    // ---- every read of the wave, in the order it needs them -------------------
    const int par = ld_i32(make_rsrc(parent + (size_t)b * N, N * 4), l16 * 4);
    const float al = ld_f32(make_rsrc(alpha + node0, N * 4), l16 * 4);
    const float be = ld_f32(make_rsrc(beta + node0, N * 4), l16 * 4);
    Path path;
    if constexpr (MODE == FUSED) path.issue(cm, u, b, sizeof(In));
    const rsrc_t rk = make_rsrc(static_cast<const In *>(k_) + node0 * D, N * ROW);
    const rsrc_t rq = make_rsrc(static_cast<const In *>(q_) + node0 * D, N * ROW);
    constexpr int XN = F32IN ? 2 : 1;                    // 16-byte pieces per eight entries
    uint4 kx[4][XN], qx[4][XN];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int x = 0; x < XN; ++x) {
            const int off = l16 * ROW + (32 * s + 8 * g) * (int)sizeof(In) + 16 * x;
            kx[s][x] = ld_u32x4<CACHED>(rk, off);
            qx[s][x] = ld_u32x4<CACHED>(rq, off);
        }
    using VT = typename std::conditional<F32IN, float, unsigned short>::type;
    VT vr[4];
    const rsrc_t rv = make_rsrc(static_cast<const In *>(v_) + node0 * D, N * ROW);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int off = ((4 * g + r) * D + col) * (int)sizeof(In);
        if constexpr (F32IN) vr[r] = ld_f32(rv, off);
        else vr[r] = __builtin_amdgcn_raw_buffer_load_b16(rv, off, 0, CACHED);
    }
    __builtin_amdgcn_sched_barrier(0);                   // (the state's reads last: reads return in order)
    st.load(S0, u);
    __builtin_amdgcn_sched_barrier(0);

    // ---- ancestors and cumulative decay by pointer jumping (see verify.hip) -----
    float pm = l16 < N ? DecayX::mant(al) : 0.f;
    int pe = l16 < N ? DecayX::expo(al) : 0;
    int ptr = l16 < N ? par : -1;
    if (ptr < -1 || ptr >= l16) {
        if (first && lane < 16) flag_error(err, b, TREEWY_FLAG_BAD_PARENT);
        ptr = -1;
    }
    int mask = ptr >= 0 ? 1 << ptr : 0;
    while (__any(ptr >= 0)) {
        const int src = (lane & 48) | (ptr >= 0 ? ptr : l16);
        const float pm_s = __shfl(pm, src);
        const int pe_s = __shfl(pe, src);
        const int link = __shfl(mask | (ptr + 1) << 16, src);
        if (ptr >= 0) {
            DecayX::mul(pm, pe, pm_s, pe_s);
            mask |= link & 0xffff;
            ptr = (link >> 16) - 1;
        }
    }
    const float inv = 1.f / pm, bt = l16 < N ? be : 0.f, gt = DecayX::value(pm, pe);
    // ... of the nodes 4 g + r (lane group g's accumulator rows)
    float inv4[4], g4[4], b4[4];
    int e4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int src = (lane & 48) | (4 * g + r);
        inv4[r] = __shfl(inv, src);
        e4[r] = __shfl(pe, src);
        g4[r] = __shfl(gt, src);
        b4[r] = __shfl(bt, src);
    }

    Keys<F32IN, FIRST> keys;
    if constexpr (MODE == FUSED) {
        path.check(cm, b, first, err);
        path.load(keys, 0, g, col);
    }

    // ---- gram tiles: lane t = l16, rows i = 4 g + r -------------------------------
    bf16x8 kh[4], kl[F32IN ? 4 : 1], qh[4], ql[F32IN ? 4 : 1];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if constexpr (F32IN) {
            float x[8];
            floats8(kx[s][0], kx[s][XN - 1], x);
            split8(x, kh[s], kl[s]);
            floats8(qx[s][0], qx[s][XN - 1], x);
            split8(x, qh[s], ql[s]);
        } else {
            kh[s] = __builtin_bit_cast(bf16x8, kx[s][0]);
            qh[s] = __builtin_bit_cast(bf16x8, qx[s][0]);
        }
    }
    f32x4 gk = {}, gq = {};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        gk = mma16(kh[s], kh[s], gk);
        gq = mma16(kh[s], qh[s], gq);
        if constexpr (F32IN) {
            gk = mma16(kl[s], kh[s], gk);
            gk = mma16(kh[s], kl[s], gk);
            gq = mma16(kl[s], qh[s], gq);
            gq = mma16(kh[s], ql[s], gq);
        }
    }
    f32x4 Bt, At;                                        // B[t][4 g + r], A[t][4 g + r]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * g + r;
        const bool strict = (mask >> i) & 1;
        const float rs = DecayX::ratio(pm, pe, inv4[r], e4[r]);
        const float ratio = strict ? rs : (i == l16 ? 1.f : 0.f);
        Bt[r] = strict ? bt * ratio * gk[r] : 0.f;
        float a = ratio * gq[r];
        asm("" : "+v"(a));                               // (rounded to fp32 before it is split)
        At[r] = a;
    }
    uint2 hi, lo;
    split4(At, hi, lo);
    const bf16x8 Ah = low8(hi), Al = low8(lo);

    // ---- T, row t = l16, by the sweep; its entries 4 g + r as an operand ----------
    bf16x8 Th, Tl;
    {
        float bb[16], r[16];
        all_groups(Bt, bb);
#pragma unroll
        for (int j = 0; j < 16; ++j) r[j] = bb[j];
        sweep16<15>(r, bb, l16);
        f32x4 t4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (values first: a select of references goes through memory)
            const float r0 = r[e], r1 = r[4 + e], r2 = r[8 + e], r3 = r[12 + e];
            const float a = g & 1 ? r1 : r0, c = g & 1 ? r3 : r2;
            t4[e] = 4 * g + e == l16 && l16 < N ? 1.f : g & 2 ? c : a;
        }
        split4(t4, hi, lo);
        Th = low8(hi);
        Tl = low8(lo);
    }

    // ---- fused: the previous round's path into the state, and the state out --------
    if constexpr (MODE == FUSED) {
        commit_path(st, path, keys);
        st.store(cm.S_new, u);
    }

    // ---- P = [K; Q] S^T: lane column col, rows t = 4 g + r -------------------------
    f32x4 pk = {}, pq = {};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        bf16x8 bh, bl;
        if constexpr (SBF) {
            bh = __builtin_bit_cast(bf16x8, st.x[s][0]);
        } else {
            float x[8];
            floats8(st.x[s][0], st.x[s][st.SN - 1], x);
            split8(x, bh, bl);
        }
        pk = mma16(kh[s], bh, pk);
        pq = mma16(qh[s], bh, pq);
        if constexpr (!SBF) {
            pk = mma16(kh[s], bl, pk);
            pq = mma16(qh[s], bl, pq);
        }
        if constexpr (F32IN) {
            pk = mma16(kl[s], bh, pk);
            pq = mma16(ql[s], bh, pq);
        }
    }
    // ---- R, U = T R, O = g P_Q + A U -------------------------------------------------
    f32x4 R;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float vt;
        if constexpr (F32IN) vt = vr[r];
        else vt = __builtin_bit_cast(float, (uint32_t)vr[r] << 16);
        R[r] = b4[r] * (vt - g4[r] * pk[r]);
        pq[r] *= g4[r];
    }
    auto product = [&](bf16x8 ah, bf16x8 alo, const f32x4 &x, f32x4 acc) {
        uint2 h, l;
        split4(x, h, l);
        acc = mma16(ah, low8(h), acc);
        acc = mma16(ah, low8(l), acc);
        return mma16(alo, low8(h), acc);
    };
    const f32x4 uu = product(Th, Tl, R, f32x4{});
    const rsrc_t ru = make_rsrc(U + node0 * D, N * D * 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) st_f32<CACHED>(ru, ((4 * g + r) * D + col) * 4, uu[r]);
    const f32x4 oo = product(Ah, Al, uu, pq);
    const rsrc_t ro = make_rsrc(static_cast<In *>(o_) + node0 * D, N * ROW);
    // (parts of a line: the default policy lets L2 merge the neighbouring waves')
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const int off = ((4 * g + r) * D + col) * (int)sizeof(In);
        if constexpr (F32IN) {
            st_f32<CACHED>(ro, off, oo[r]);
            st_f32<CACHED>(ro, off + ROW, oo[r + 1]);
        } else {
            const uint32_t pr = pack_bf2(oo[r], oo[r + 1]);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)pr, ro, off, 0, CACHED);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(pr >> 16), ro, off + ROW, 0, CACHED);
        }
    }
}

// x_j of lane group i <-> x_i of lane group j (a 4 x 4 transpose between the four values and the four lane groups).
__device__ __forceinline__ void transpose_groups(float (&x)[4]) {
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float f = x[j];
        v[j] = __builtin_bit_cast(int, f);
    }
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
        const auto p = __builtin_amdgcn_permlane16_swap(v[j], v[j + 1], false, false);
        v[j] = p[0];
        v[j + 1] = p[1];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto p = __builtin_amdgcn_permlane32_swap(v[j], v[j + 2], false, false);
        v[j] = p[0];
        v[j + 2] = p[1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = v[j];
        x[j] = __builtin_bit_cast(float, i);
    }
}

// Drafts of up to 16 NT nodes of bf16 tokens, the same way: NT tiles of 16 nodes.
// In the walk lane = node; its results go through a piece of LDS that belongs
// to the wave.  The diagonal blocks of T are swept at once, block q in lane group
// q (a transpose across the lane groups before and after turns the gram's
// layout into rows and back); T itself is not formed: U comes by forward
// substitution over the tiles, U_a = T_a (R_a - sum over b < a of B_ab U_b), whose
// operands B_ab and A_ab are the gram tiles as the accumulators hold them.  Past
// the first tile T, B, R and U stand as three bf16 each in this solve (24 bits:
// with keys that lie close together the sum cancels most of R, and in pairs the
// error of U was up to 1.6 times verify.hip's): six products in three
// instructions, two to the halves of the contraction (0.1 us more at 48 nodes).
template <bool SBF, int MODE, int NT>
__global__ __launch_bounds__(64 * NW, MODE == FUSED && NT == 3 ? 1 : 2) void tiles_kernel(
    const void *S0, const void *__restrict__ q_, const void *__restrict__ k_, const void *__restrict__ v_,
    const float *__restrict__ alpha, const float *__restrict__ beta, const int32_t *__restrict__ parent, int N, int H,
    int units, void *__restrict__ o_, float *U, int32_t *__restrict__ err, CommitArgs cm) {
    using In = __bf16;
    static_assert(NT == 2 || NT == 3, "at most 48 nodes: with four tiles what every wave repeats outweighs what it saves");
    constexpr int ROW = D * (int)sizeof(In);
    constexpr int N_INV = 0, N_EXP = 1, N_GVAL = 2, N_BETA = 3, N_MANT = 4, N_MASK0 = 5, N_MASK1 = 6, FIELDS = 7;
    __shared__ __attribute__((aligned(16))) int node_s[NW][FIELDS][64];
    __shared__ __attribute__((aligned(16))) unsigned char k_s[MODE == PREFILL ? NW : 1][MODE == PREFILL ? 32 * 256 : 16];
    const int bx = blockIdx.x & 7, by = blockIdx.x >> 3;
    const int part = by % PARTS, u = (by / PARTS) * 8 + bx;
    if (u >= units) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int b = u / H, col = 16 * (part * NW + wave) + l16;
    State<SBF> st(col, g);
    const bool first = part == 0 && wave == 0;
    const size_t node0 = (size_t)u * N;

    // ---- every read of the wave, in the order it needs them -------------------
    int par = lane - 1;                                  // (a chain)
    if constexpr (MODE != PREFILL) par = ld_i32(make_rsrc(parent + (size_t)b * N, N * 4), lane * 4);
    const float al = ld_f32(make_rsrc(alpha + node0, N * 4), lane * 4);
    const float be = ld_f32(make_rsrc(beta + node0, N * 4), lane * 4);
    Path path;
    if constexpr (MODE == FUSED) path.issue(cm, u, b, sizeof(In));
    const rsrc_t rk = make_rsrc(static_cast<const In *>(k_) + node0 * D, N * ROW);
    const rsrc_t rq = make_rsrc(static_cast<const In *>(q_) + node0 * D, N * ROW);
    bf16x8 kh[NT][4], qh[NT][4];
    auto load_rows = [&](bf16x8 (&x)[NT][4], rsrc_t r) {
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                x[a][s] = __builtin_bit_cast(bf16x8, ld_u32x4<CACHED>(r, (16 * a + l16) * ROW + (32 * s + 8 * g) * 2));
    };
    load_rows(kh, rk);
    load_rows(qh, rq);
    unsigned short vr[NT][4];
    const rsrc_t rv = make_rsrc(static_cast<const In *>(v_) + node0 * D, N * ROW);
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            vr[a][r] = __builtin_amdgcn_raw_buffer_load_b16(rv, ((16 * a + 4 * g + r) * D + col) * 2, 0, CACHED);
    __builtin_amdgcn_sched_barrier(0);
    st.load(S0, u);
    __builtin_amdgcn_sched_barrier(0);

    // ---- ancestors and cumulative decay by pointer jumping (lane = node) --------
    float wt = 0.f, gN = 0.f;                            // prefill: the update's weight of token = lane, and g_N
    {
        float pm = lane < N ? DecayX::mant(al) : 0.f;
        int pe = lane < N ? DecayX::expo(al) : 0;
        int ptr = lane < N ? par : -1;
        if (ptr < -1 || ptr >= lane) {
            if (first) flag_error(err, b, TREEWY_FLAG_BAD_PARENT);
            ptr = -1;
        }
        int m0 = ptr >= 0 && ptr < 32 ? 1 << ptr : 0, m1 = ptr >= 32 ? 1 << (ptr - 32) : 0;
        while (__any(ptr >= 0)) {
            const int src = ptr >= 0 ? ptr : lane;
            const float pm_s = __shfl(pm, src);
            const int pe_s = __shfl(pe, src), ptr_s = __shfl(ptr, src), m0_s = __shfl(m0, src);
            const int m1_s = NT > 2 ? __shfl(m1, src) : 0;
            if (ptr >= 0) {
                DecayX::mul(pm, pe, pm_s, pe_s);
                m0 |= m0_s;
                m1 |= m1_s;
                ptr = ptr_s;
            }
        }
        const float inv = 1.f / pm, bt = lane < N ? be : 0.f, gt = DecayX::value(pm, pe);
        if constexpr (MODE == PREFILL) {
            const float mN = __shfl(pm, N - 1);
            const int eN = __shfl(pe, N - 1);
            wt = lane < N ? DecayX::ratio(mN, eN, inv, pe) : 0.f;
            gN = DecayX::value(mN, eN);
        }
        int(&w)[FIELDS][64] = node_s[wave];
        w[N_INV][lane] = __builtin_bit_cast(int, inv);
        w[N_EXP][lane] = pe;
        w[N_GVAL][lane] = __builtin_bit_cast(int, gt);
        w[N_BETA][lane] = __builtin_bit_cast(int, bt);
        w[N_MANT][lane] = __builtin_bit_cast(int, pm);
        w[N_MASK0][lane] = m0;
        w[N_MASK1][lane] = m1;
    }
    lds_order();
    auto field1 = [&](int f, int a) { return node_s[wave][f][16 * a + l16]; };
    auto field4 = [&](int f, int a) { return *reinterpret_cast<const int4 *>(&node_s[wave][f][16 * a + 4 * g]); };
    Keys<false, FIRST> keys;
    if constexpr (MODE == FUSED) {
        path.check(cm, b, first, err);
        path.load(keys, 0, g, col);
    }

    // ---- gram tiles: lane t = 16 a + l16, rows i = 16 bb + 4 g + r, bb <= a --------
    constexpr int PAIRS = NT * (NT + 1) / 2;             // tile (a, bb) at a (a + 1) / 2 + bb
    uint2 Bh[PAIRS], Bm[PAIRS], Bl[PAIRS];               // -B off the diagonal, and A, as operands
    uint2 Ah[PAIRS], Al[PAIRS];
    float Bd[4][4] = {};                                 // B's diagonal tiles
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        const float mt = __builtin_bit_cast(float, field1(N_MANT, a)), bt = __builtin_bit_cast(float, field1(N_BETA, a));
        const int et = field1(N_EXP, a), m0 = field1(N_MASK0, a), m1 = NT > 2 ? field1(N_MASK1, a) : 0;
#pragma unroll
        for (int bb = 0; bb <= a; ++bb) {
            f32x4 gk = {}, gq = {};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                gk = mma16(kh[bb][s], kh[a][s], gk);
                gq = mma16(kh[bb][s], qh[a][s], gq);
            }
            const int4 iv = field4(N_INV, bb), ev = field4(N_EXP, bb);
            const int i4[4] = {iv.x, iv.y, iv.z, iv.w}, e4[4] = {ev.x, ev.y, ev.z, ev.w};
            const int bits = (bb < 2 ? m0 : m1) >> (16 * (bb & 1) + 4 * g);
            const int p = a * (a + 1) / 2 + bb;
            f32x4 Bt, At;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int iv_r = i4[r];
                const bool strict = (bits >> r) & 1, self = a == bb && 4 * g + r == l16;
                const float rs = DecayX::ratio(mt, et, __builtin_bit_cast(float, iv_r), e4[r]);
                const float ratio = strict ? rs : self ? 1.f : 0.f;
                Bt[r] = strict ? bt * ratio * gk[r] : 0.f;
                float x = ratio * gq[r];
                asm("" : "+v"(x));                       // (rounded to fp32 before it is split)
                At[r] = x;
            }
            split4(At, Ah[p], Al[p]);
            if (a == bb) {
#pragma unroll
                for (int r = 0; r < 4; ++r) Bd[a][r] = Bt[r];
            } else {
                split4(-Bt, Bh[p], Bm[p], Bl[p]);
            }
        }
    }

    // ---- the diagonal blocks of T: block q's rows in lane group q ------------------
    uint2 Th[4], Tm[4], Tl[4];
    {
        float bb[16], r[16];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x[4] = {Bd[0][e], Bd[1][e], Bd[2][e], Bd[3][e]};
            transpose_groups(x);                         // group q: its row's entries 4 j + e
#pragma unroll
            for (int j = 0; j < 4; ++j) r[4 * j + e] = bb[4 * j + e] = x[j];
        }
        sweep16<15>(r, bb, l16);
        f32x4 t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float f = r[4 * j + e];
                x[j] = 4 * j + e == l16 && lane < N ? 1.f : f;
            }
            transpose_groups(x);                         // group g: block q's entries 4 g + e
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q][e] = x[q];
        }
#pragma unroll
        for (int q = 0; q < NT; ++q) split4(t[q], Th[q], Tm[q], Tl[q]);
    }

    // ---- fused: the previous round's path into the state, and the state out --------
    if constexpr (MODE == FUSED) {
        commit_path(st, path, keys);
        st.store(cm.S_new, u);
    }

    // ---- P = [K; Q] S^T: lane column col, rows 16 a + 4 g + r -----------------------
    f32x4 pk[NT] = {}, pq[NT] = {};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        bf16x8 bh, bl;
        if constexpr (SBF) {
            bh = __builtin_bit_cast(bf16x8, st.x[s][0]);
        } else {
            float x[8];
            floats8(st.x[s][0], st.x[s][st.SN - 1], x);
            split8(x, bh, bl);
        }
#pragma unroll
        for (int a = 0; a < NT; ++a) {
            pk[a] = mma16(kh[a][s], bh, pk[a]);
            pq[a] = mma16(qh[a][s], bh, pq[a]);
        }
        if constexpr (!SBF) {
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                pk[a] = mma16(kh[a][s], bl, pk[a]);
                pq[a] = mma16(qh[a][s], bl, pq[a]);
            }
        }
    }
    // ---- R, then tile by tile U_a = T_a (R_a - sum B_ab U_b) and O_a = g P_Q + sum A_ab U_b
    auto product = [&](uint2 ah, uint2 alo, uint2 xh, uint2 xl, f32x4 acc) {
        acc = mma16(low8(ah), low8(xh), acc);
        acc = mma16(low8(ah), low8(xl), acc);
        return mma16(low8(alo), low8(xh), acc);
    };
    auto product3 = [&](uint2 ah, uint2 am, uint2 alo, uint2 xh, uint2 xm, uint2 xl, f32x4 acc) {
        acc = mma16(both8(ah, alo), both8(xl, xh), acc);
        acc = mma16(both8(ah, am), both8(xm, xm), acc);
        return mma16(both8(ah, am), both8(xh, xh), acc);
    };
    const rsrc_t ru = make_rsrc(MODE == PREFILL ? nullptr : U + node0 * D, MODE == PREFILL ? 0 : N * D * 4);
    const rsrc_t ro = make_rsrc(static_cast<In *>(o_) + node0 * D, N * ROW);
    uint2 uh[NT], um[NT], ul[NT];
    f32x4 u32[MODE == PREFILL ? NT : 1];
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        const int4 gv = field4(N_GVAL, a), bv = field4(N_BETA, a);
        const int g4[4] = {gv.x, gv.y, gv.z, gv.w}, b4[4] = {bv.x, bv.y, bv.z, bv.w};
        f32x4 R;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float vt = __builtin_bit_cast(float, (uint32_t)vr[a][r] << 16);
            const int gi = g4[r], bi = b4[r];
            const float gr = __builtin_bit_cast(float, gi), br = __builtin_bit_cast(float, bi);
            R[r] = br * (vt - gr * pk[a][r]);
            pq[a][r] *= gr;
        }
#pragma unroll
        for (int bb = 0; bb < a; ++bb) {
            const int p = a * (a + 1) / 2 + bb;
            R = product3(Bh[p], Bm[p], Bl[p], uh[bb], um[bb], ul[bb], R);
        }
        uint2 rh, rm, rl;
        split4(R, rh, rm, rl);
        // (the first tile as small_kernel has it: the same bits)
        const f32x4 uu = a == 0 ? product(Th[a], Tm[a], rh, rm, f32x4{}) : product3(Th[a], Tm[a], Tl[a], rh, rm, rl, f32x4{});
        if constexpr (MODE == PREFILL) u32[a] = uu;
        else
#pragma unroll
            for (int r = 0; r < 4; ++r) st_f32<CACHED>(ru, ((16 * a + 4 * g + r) * D + col) * 4, uu[r]);
        split4(uu, uh[a], um[a], ul[a]);
        f32x4 oo = pq[a];
#pragma unroll
        for (int bb = 0; bb <= a; ++bb) oo = product(Ah[a * (a + 1) / 2 + bb], Al[a * (a + 1) / 2 + bb], uh[bb], um[bb], oo);
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            const int off = ((16 * a + 4 * g + r) * D + col) * (int)sizeof(In);
            const uint32_t pr = pack_bf2(oo[r], oo[r + 1]);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)pr, ro, off, 0, CACHED);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(pr >> 16), ro, off + ROW, 0, CACHED);
        }
    }
    if constexpr (MODE == PREFILL) {
        node_s[wave][N_INV][lane] = __builtin_bit_cast(int, wt);
        float x[4][8];
        st.get(x, gN);
        // The update K^T (w U) on the matrix cores: K's rows through LDS of the
        // wave's own for the transposed reads (granule G of 16 bytes of row t at G ^
        // swz(t)), w U as the accumulators hold it.  Slots e < 4 of lane group g are
        // token 4 g + e, the others token 16 + 4 g + e - 4; row 4 y + r of product
        // (s, h) is d_k 32 s + 8 y + 4 h + r, so its rows 4 g + r land on this
        // lane's entries.
        static_assert(MODE != PREFILL || NT == 2, "32 tokens: one step of the contraction");
        unsigned char *ks = k_s[wave];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                *reinterpret_cast<bf16x8 *>(ks + (16 * a + l16) * 256 + (((4 * s + g) ^ swz(l16)) << 4)) = kh[a][s];
        lds_order();
        float wu[8];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int4 wv = field4(N_INV, a);            // (the weights by now)
            const int w4[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int wi = w4[r];
                wu[4 * a + r] = __builtin_bit_cast(float, wi) * u32[a][r];
            }
        }
        bf16x8 wh, wl;
        split8(wu, wh, wl);
        const int j4 = l16 >> 2, y = l16 & 3;
        const int tr_addr = (4 * g + j4) * 256 + ((y ^ swz(4 * g + j4)) << 4);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned char *at = ks + 8 * h + (tr_addr ^ (s << 6));
                const s16x4 k0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at);
                const s16x4 k1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at + 16 * 256));
                const bf16x8 kt = __builtin_bit_cast(bf16x8, __builtin_shufflevector(k0, k1, 0, 1, 2, 3, 4, 5, 6, 7));
                f32x4 d = {x[s][4 * h], x[s][4 * h + 1], x[s][4 * h + 2], x[s][4 * h + 3]};
                d = mma16(kt, wh, d);
                d = mma16(kt, wl, d);
#pragma unroll
                for (int r = 0; r < 4; ++r) x[s][4 * h + r] = d[r];
            }
        st.put(x);
        st.store(cm.S_new, u);
    }
}

// treewy_commit: the accepted path into the state, by the same waves.
template <bool F32IN, bool SBF>
__global__ __launch_bounds__(64 * NW) void small_commit_kernel(const void *S0, int H, int units, int32_t *__restrict__ err,
                                                               CommitArgs cm) {
    const int bx = blockIdx.x & 7, by = blockIdx.x >> 3;
    const int part = by % PARTS, u = (by / PARTS) * 8 + bx;
    if (u >= units) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int b = u / H, col = 16 * (part * NW + wave) + (lane & 15);
    Path path;
    path.issue(cm, u, b, F32IN ? 4 : 2);
    State<SBF> st(col, g);
    st.load(S0, u);
    __builtin_amdgcn_sched_barrier(0);
    path.check(cm, b, part == 0 && wave == 0, err);
    Keys<F32IN, FIRST> keys;
    path.load(keys, 0, g, col);
    commit_path(st, path, keys);
    st.store(cm.S_new, u);
}

// A unit's workgroups, eight units at a time (see the kernels' unit and part).
unsigned grid_of(int units) { return (unsigned)(((int64_t)units + 7) / 8 * 8 * PARTS); }

template <bool F32IN, bool SBF, int MODE>
hipError_t launch(const void *S0, const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                  const int32_t *parent, int N, int B, int H, void *o, float *U, int32_t *err, const CommitArgs &cm,
                  hipStream_t stream) {
    hipLaunchKernelGGL((small_kernel<F32IN, SBF, MODE>), dim3(grid_of(B * H)), dim3(64 * NW), 0, stream, S0, q, k, v, alpha,
                       beta, parent, N, H, B * H, o, U, err, cm);
    return hipGetLastError();
}

template <bool SBF, int MODE, int NT>
hipError_t launch_tiles(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                        const float *beta, const int32_t *parent, int N, int B, int H, void *o, float *U, int32_t *err,
                        const CommitArgs &cm, hipStream_t stream) {
    hipLaunchKernelGGL((tiles_kernel<SBF, MODE, NT>), dim3(grid_of(B * H)), dim3(64 * NW), 0, stream, S0, q, k, v, alpha,
                       beta, parent, N, H, B * H, o, U, err, cm);
    return hipGetLastError();
}

template <int MODE>
hipError_t dispatch(const void *S0, const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                    const int32_t *parent, int N, int B, int H, bool f32_in, bool bf16_state, void *o, float *U,
                    int32_t *err, const CommitArgs &cm, hipStream_t stream) {
#define TREEWY_TILES(S, NT)                                                                                          \
    launch_tiles<S, MODE, NT>(S0, q, k, v, alpha, beta, parent, N, B, H, o, U, err, cm, stream)
    if constexpr (MODE == PREFILL) {
        return bf16_state ? TREEWY_TILES(true, 2) : TREEWY_TILES(false, 2);
    } else {
        if (N > 16) {                                    // (bf16 tokens: see small_verify_fits)
            if (bf16_state) return N <= 32 ? TREEWY_TILES(true, 2) : TREEWY_TILES(true, 3);
            return N <= 32 ? TREEWY_TILES(false, 2) : TREEWY_TILES(false, 3);
        }
        if (bf16_state) return launch<false, true, MODE>(S0, q, k, v, alpha, beta, parent, N, B, H, o, U, err, cm, stream);
        if (f32_in) return launch<true, false, MODE>(S0, q, k, v, alpha, beta, parent, N, B, H, o, U, err, cm, stream);
        return launch<false, false, MODE>(S0, q, k, v, alpha, beta, parent, N, B, H, o, U, err, cm, stream);
    }
#undef TREEWY_TILES
}

}  // namespace

// Where these kernels are used: with few units a call is one wave's chain of
// dependent steps and a launch, and eight short waves per unit beat four long
// ones; with many, what every wave repeats (K and Q, the gram, the solve) costs
// more.  us a call, from a graph, this against the others' (fp32 state):
//   verify: 8-node chains in 32 units 4.1 against 6.2, 128 units 4.2 against 6.4;
//     32 nodes, bf16 tokens, in 128 units 6.5 against 8.0, 192 units 10.0 against
//     7.9; 39 and 48 nodes in 128 units 8.0 and 8.5 against 11.1 and 11.2, 192
//     units 12.3 and 13.2 against 11.4 and 11.7; 64 nodes in four tiles 11.2
//     against 10.6 already at 64 units, 24 nodes with fp32 tokens 8.7 against 8.5;
//   the fused call, paths of 4 entries: 8-node chains in 32 units 5.9 against 9.8, 128
//     units 7.1 against 10.2; 32 nodes in 128 units 9.3 against 11.7, 192 units 13.9
//     against 12.0; paths of 64 entries, 8 nodes in 128 units: 15.0 against 16.9 with
//     bf16 and 15.8 against 19.2 with fp32 tokens;
//   prefill of 20 tokens: 64 units 7.7 against 9.8, 128 units 9.0 against 10.3, 192
//     units 12.0 against 10.7;
//   commit, paths of 0, 1 and 4 entries: 32 units 3.7, 4.1 and 4.4 against 3.7, 4.5
//     and 5.3, 128 units 4.6, 5.3 and 5.6 against 4.5, 5.4 and 6.2, 192 units 6.9, 7.5
//     and 7.7 against 4.8, 5.6 and 6.6 (the state's rows pass in 64-byte pieces).
// One limit for verify, the fused call and a one-chunk prompt: their kernels of
// one family do the same arithmetic, so a fused call that commits nothing, and
// a prompt of one chunk, give verify's outputs bit for bit at every number of
// units.  Past it a draft of at most 16 nodes could gain still (8-node chains in
// 256 units: verify 5.9 against 7.1, fused 9.7 against 11.8) where a prompt of 16
// tokens loses (192 units 11.8 against 11.0), and with fp32 tokens 16-node trees in
// 192 units lose too (9.2 against 8.2).
static bool few_units(int units) { return 2 * (int64_t)units <= compute_units(); }
bool small_verify_fits(int N, int units, bool f32_in) { return N <= (f32_in ? 16 : 48) && few_units(units); }
bool small_prefill_fits(int T, int units, bool f32_in) { return T <= 32 && !f32_in && few_units(units); }
bool small_commit_fits(int N, int L_max, int units) { return N <= 64 && L_max <= 64 && few_units(units); }

hipError_t launch_small_verify(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                               const float *beta, const int32_t *parent, int N, int B, int H, bool f32_in,
                               bool bf16_state, void *o, float *U, int32_t *err, hipStream_t stream) {
    return dispatch<VERIFY>(S0, q, k, v, alpha, beta, parent, N, B, H, f32_in, bf16_state, o, U, err, CommitArgs{}, stream);
}

hipError_t launch_small_commit_verify(const void *S_old, const void *q, const void *k, const void *v, const float *alpha,
                                      const float *beta, const int32_t *parent, int N, int B, int H, bool f32_in,
                                      bool bf16_state, void *o, float *U, int32_t *err, const CommitArgs &cm,
                                      hipStream_t stream) {
    return dispatch<FUSED>(S_old, q, k, v, alpha, beta, parent, N, B, H, f32_in, bf16_state, o, U, err, cm, stream);
}

hipError_t launch_small_prefill(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                                const float *beta, int T, int B, int H, bool bf16_state, void *S_T, void *o,
                                hipStream_t stream) {
    CommitArgs cm = {};
    cm.S_new = S_T;
    return dispatch<PREFILL>(S0, q, k, v, alpha, beta, nullptr, T, B, H, false, bf16_state, o, nullptr, nullptr, cm, stream);
}

hipError_t launch_small_commit(const void *S0, int B, int H, bool f32_k, bool bf16_state, int32_t *err,
                               const CommitArgs &cm, hipStream_t stream) {
    const dim3 grid(grid_of(B * H)), block(64 * NW);
#define TREEWY_COMMIT(F, S) hipLaunchKernelGGL((small_commit_kernel<F, S>), grid, block, 0, stream, S0, H, B * H, err, cm)
    if (f32_k) {
        if (bf16_state) TREEWY_COMMIT(true, true);
        else TREEWY_COMMIT(true, false);
    } else {
        if (bf16_state) TREEWY_COMMIT(false, true);
        else TREEWY_COMMIT(false, false);
    }
#undef TREEWY_COMMIT
    return hipGetLastError();
}

}  // namespace treewy
