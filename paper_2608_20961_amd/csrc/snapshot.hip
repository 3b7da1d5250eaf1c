// Full-state-snapshotting baseline (the paper's approach (i), "storeall"):
// run the gated delta rule (eq. 1) node by node and write every node's full
// state, so that rollback is a copy of one snapshot.  Kept deliberately as the
// store-all data flow, for the memory and bandwidth comparison with
// reconstruct-on-commit; it is not the method.
//
// The rows of a state are independent, so every wave runs ROWS rows of one unit
// through all nodes on its own: lanes 0 to 31 hold rows 0 .. ROWS / 2 - 1 of
// these at columns 4 (lane % 32) .. + 3, lanes 32 to 63 the others, so that each
// store instruction of a node's state writes whole lines.  Nothing passes
// between waves: the dot products over a row sum across its 32 lanes by DPP.
// A node's vectors are fetched two nodes ahead, and a node whose parent is not
// the node before it has the parent's state (its own elements, stored earlier
// by the same lanes) fetched one node ahead.  Bound by the states' writes and
// reloads.  One workgroup per unit, with two barriers a node and nothing
// fetched ahead, took 154 us for 128 units of 32 nodes on half the CUs, this
// takes 62 us; 1024 units of 8-node chains 166 -> 124 us (6.0 TB/s); 512 units of
// 60-node trees 537 -> 529 us.  (States read back later are stored through the
// caches, the others past them: with every store past the caches the last
// takes 587 us, with none the chains take 150 us.)
#include "device.h"
#include "launch.h"

namespace treewy {

constexpr int ROWS = 8;                                  // rows per wave
constexpr int PARTS = D / (ROWS * THREADS / 64);         // workgroups per unit

// Sum over the 32 lanes of a half wave, in every lane: quads, pairs of quads
// and halves of 16 by DPP, then the two rows of 16.
__device__ __forceinline__ float sum32(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1, 0, 3, 2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2, 3, 0, 1]
    v += dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror
    const int u = __builtin_bit_cast(int, v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const int r0 = r[0], r1 = r[1];                      // (a bit cast of r[1] itself gives r[0])
    return __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
}

template <bool F32IN>
__global__ __launch_bounds__(THREADS) void snapshot_verify_kernel(
    const float *S0, const void *__restrict__ q_, const void *__restrict__ k_, const void *__restrict__ v_,
    const float *__restrict__ alpha, const float *__restrict__ beta, const int32_t *__restrict__ parent, int N, int H,
    void *__restrict__ o_, float *snaps, int32_t *__restrict__ err) {
    using In = typename std::conditional<F32IN, float, __bf16>::type;
    // (four entries in one access, of arrays that need no more than an element's alignment)
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    typedef __bf16 bf16x4u __attribute__((ext_vector_type(4), aligned(2)));
    using In4 = typename std::conditional<F32IN, f32x4u, bf16x4u>::type;
    constexpr int R = ROWS / 2;                          // rows per lane
    const int u = blockIdx.x / PARTS, part = blockIdx.x % PARTS, b = u / H;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c4 = 4 * (lane & 31);
    const int row = (part * (THREADS / 64) + wave) * ROWS + R * (lane >> 5);   // this lane's first row
    const size_t node0 = (size_t)u * N;
    const In *q = static_cast<const In *>(q_) + node0 * D, *k = static_cast<const In *>(k_) + node0 * D;
    const In *v = static_cast<const In *>(v_) + node0 * D;
    In *o = static_cast<In *>(o_) + node0 * D;
    alpha += node0;
    beta += node0;
    parent += (size_t)b * N;
    const int at = (row * D + c4) * 4;                   // this lane's first byte of a state
    constexpr int STATE = D * D * 4;                     // bytes of a state (N <= 64 of them: offsets fit an int)
    const rsrc_t rs = make_rsrc(S0 + (size_t)u * D * D, STATE);
    const rsrc_t rn = make_rsrc(snaps + node0 * D * D, N * STATE);

    struct Node {
        In4 k, q, v;                                     // columns c4 .. + 3 of k and q, rows row .. + 3 of v
        float al, be;
    };
    static_assert(R == 4, "a lane's rows of v are one load");
    auto fetch = [&](int t, Node &x) {
        x.k = *reinterpret_cast<const In4 *>(k + (size_t)t * D + c4);
        x.q = *reinterpret_cast<const In4 *>(q + (size_t)t * D + c4);
        x.v = *reinterpret_cast<const In4 *>(v + (size_t)t * D + row);
        x.al = alpha[t];
        x.be = beta[t];
    };
    // The parent of node t; a malformed one counts as the committed state.
    auto parent_of = [&](int t) {
        int p = parent[t];
        if (p < -1 || p >= t) {
            if (threadIdx.x == 0 && part == 0) flag_error(err, b, TREEWY_FLAG_BAD_PARENT);
            p = -1;
        }
        return p;
    };
    f32x4 s[R], far[R];                                  // the running state; the next node's parent if it is another
    auto fetch_state = [&](int p, f32x4 (&x)[R]) {
        if (p < 0) {
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = ld_f32x4<CACHED>(rs, at + i * D * 4);
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = ld_f32x4<CACHED>(rn, p * STATE + at + i * D * 4);
        }
    };
    // Nodes whose state some later node reads back (one bit each, N <= 64): these
    // are stored through the caches, the others past them.
    uint64_t again = 0;
    {
        const int p = lane < N ? parent[lane] : lane - 1;
        again = wave_or64(p >= 0 && p < lane - 1 ? 1ull << p : 0ull);
    }
    Node a, c;
    fetch(0, a);
    fetch(N > 1 ? 1 : 0, c);
    parent_of(0);                                        // (the committed state in any case)
    fetch_state(-1, s);
    auto step = [&](int t, Node &x) {                    // node t, its vectors in x; x is refilled for node t + 2
        int p_next = t;
        if (t + 1 < N) {
            p_next = parent_of(t + 1);
            if (p_next != t) fetch_state(p_next, far);
        }
        float kk[4], qq[4], sk[R], sq[R], vv[R];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kk[e] = to_f32(x.k[e]);
            qq[e] = to_f32(x.q[e]);
            vv[e] = to_f32(x.v[e]);
        }
        const float al = x.al, be = x.be;
        if (t + 2 < N) fetch(t + 2, x);
        const float kq = sum32(kk[0] * qq[0] + kk[1] * qq[1] + kk[2] * qq[2] + kk[3] * qq[3]);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            sk[i] = sum32(s[i][0] * kk[0] + s[i][1] * kk[1] + s[i][2] * kk[2] + s[i][3] * kk[3]);
            sq[i] = sum32(s[i][0] * qq[0] + s[i][1] * qq[1] + s[i][2] * qq[2] + s[i][3] * qq[3]);
        }
        In4 out;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float vt = be * (vv[i] - al * sk[i]);  // pseudo-value of the row
#pragma unroll
            for (int e = 0; e < 4; ++e) s[i][e] = fmaf(al, s[i][e], vt * kk[e]);   // eq. 1 via the key rewrite
            out[i] = from_f32<In>(al * sq[i] + vt * kq);
        }
        if ((again >> t) & 1) {
#pragma unroll
            for (int i = 0; i < R; ++i)
                st_u32x4<CACHED>(rn, t * STATE + at + i * D * 4, __builtin_bit_cast(uint4, s[i]));
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i)
                st_u32x4<STREAM>(rn, t * STATE + at + i * D * 4, __builtin_bit_cast(uint4, s[i]));
        }
        if ((lane & 31) == 0) *reinterpret_cast<In4 *>(o + (size_t)t * D + row) = out;
        if (p_next != t) {
#pragma unroll
            for (int i = 0; i < R; ++i) s[i] = far[i];
        }
    };
    for (int t = 0; t < N; t += 2) {
        step(t, a);
        if (t + 1 < N) step(t + 1, c);
    }
}

__global__ __launch_bounds__(THREADS) void snapshot_commit_kernel(
    const float *S0, const float *__restrict__ snaps, const int32_t *__restrict__ accepted, int N,
    int H, float *S_new, int32_t *__restrict__ err) {
    const int tid = threadIdx.x, u = blockIdx.x, b = u / H;
    int a = accepted[b];
    if (a < -1 || a >= N) {
        if (tid == 0 && u % H == 0) flag_error(err, b, TREEWY_FLAG_BAD_PATH);
        a = -1;
    }
    const f32x4 *from = reinterpret_cast<const f32x4 *>(
        a < 0 ? S0 + (size_t)u * D * D : snaps + ((size_t)u * N + a) * D * D);
    f32x4 *dst = reinterpret_cast<f32x4 *>(S_new + (size_t)u * D * D);
    f32x4 s[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = from[tid + THREADS * i];
#pragma unroll
    for (int i = 0; i < 16; ++i) dst[tid + THREADS * i] = s[i];
}

hipError_t launch_snapshot_verify(const float *S0, const void *q, const void *k, const void *v,
                                  const float *alpha, const float *beta, const int32_t *parent,
                                  int N, int B, int H, bool f32_in, void *o, float *snapshots,
                                  int32_t *err, hipStream_t stream) {
    const dim3 grid((unsigned)(B * H) * PARTS), block(THREADS);
    if (f32_in)
        hipLaunchKernelGGL((snapshot_verify_kernel<true>), grid, block, 0, stream, S0, q, k, v, alpha,
                           beta, parent, N, H, o, snapshots, err);
    else
        hipLaunchKernelGGL((snapshot_verify_kernel<false>), grid, block, 0, stream, S0, q, k, v, alpha,
                           beta, parent, N, H, o, snapshots, err);
    return hipGetLastError();
}

hipError_t launch_snapshot_commit(const float *S0, const float *snapshots, const int32_t *accepted,
                                  int N, int B, int H, float *S_new, int32_t *err,
                                  hipStream_t stream) {
    hipLaunchKernelGGL(snapshot_commit_kernel, dim3((unsigned)(B * H)), dim3(THREADS), 0, stream, S0,
                       snapshots, accepted, N, H, S_new, err);
    return hipGetLastError();
}

}  // namespace treewy
