// Kernel launchers behind the C ABI.  Arguments are already validated by the
// caller; each returns the HIP error of the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace treewy {

// The previous round's accepted path, committed inside verify (fused call):
// S0 of this round = g_a S_old + sum_l w_l U_prev[a_l] k_prev[a_l]^T.
struct CommitArgs {
    const float *U;           // [units, N_prev, D] pseudo-values of the previous round
    const void *k;            // [units, N_prev, D] its keys, in the input dtype
    const float *alpha;       // [units, N_prev]
    const int32_t *path;      // [B, L_max] root -> accepted node
    const int32_t *path_len;  // [B]
    const int32_t *parent;    // [B, N_prev] or null (then only range and order are checked)
    void *S_new;              // [units, D, D] in the state dtype; may be S_old
    int L_max, N_prev;
    int in_stride;            // rows per unit in k and alpha (N_prev for whole tensors)
    int u_stride;             // rows per unit in U (N_prev for whole tensors)
};

hipError_t launch_verify(const void *S0, const void *q, const void *k, const void *v,
                         const float *alpha, const float *beta, const int32_t *parent, int N,
                         int B, int H, bool f32_in, bool bf16_state, void *o, float *U, int32_t *err,
                         hipStream_t stream);

// Commit of the previous round's accepted path fused into this round's verify.
hipError_t launch_commit_verify(const void *S_old, const float *U_prev, const void *k_prev,
                                const float *alpha_prev, const int32_t *path, const int32_t *path_len,
                                int L_max, const int32_t *parent_prev, int N_prev, const void *q,
                                const void *k, const void *v, const float *alpha, const float *beta,
                                const int32_t *parent, int N, int B, int H, bool f32_in, bool bf16_state,
                                void *S_new, void *o, float *U, int32_t *err, hipStream_t stream);

// CUs of the current device.
inline int compute_units() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

// The kernels of few units (small.hip), and for which sizes they are used (verify's rule is the fused call's too).
bool small_verify_fits(int N, int units, bool f32_in);
bool small_prefill_fits(int T, int units, bool f32_in);
bool small_commit_fits(int N, int L_max, int units);
hipError_t launch_small_verify(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                               const float *beta, const int32_t *parent, int N, int B, int H, bool f32_in,
                               bool bf16_state, void *o, float *U, int32_t *err, hipStream_t stream);
hipError_t launch_small_commit_verify(const void *S_old, const void *q, const void *k, const void *v, const float *alpha,
                                      const float *beta, const int32_t *parent, int N, int B, int H, bool f32_in,
                                      bool bf16_state, void *o, float *U, int32_t *err, const CommitArgs &cm,
                                      hipStream_t stream);
hipError_t launch_small_prefill(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                                const float *beta, int T, int B, int H, bool bf16_state, void *S_T, void *o,
                                hipStream_t stream);
hipError_t launch_small_commit(const void *S0, int B, int H, bool f32_k, bool bf16_state, int32_t *err,
                               const CommitArgs &cm, hipStream_t stream);

// Chain prefill: T tokens per unit in chunks, one launch, the state in
// registers between chunks; inputs and o are [B, H, T, ...].
hipError_t launch_prefill(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                          const float *beta, int T, int B, int H, bool f32_in, bool bf16_state, void *S_T, void *o,
                          int32_t *err, hipStream_t stream);

// ... by one four-wave workgroup per unit (launch_prefill uses it for some sizes).
hipError_t launch_prefill_unit(const void *S0, const void *q, const void *k, const void *v, const float *alpha,
                               const float *beta, int T, int B, int H, bool f32_in, bool bf16_state, void *S_T,
                               void *o, int32_t *err, hipStream_t stream);

hipError_t launch_commit(const void *S0, const float *U, const void *k, const float *alpha,
                         const int32_t *path, const int32_t *path_len, int L_max,
                         const int32_t *parent, int N, int B, int H, bool f32_k, bool bf16_state,
                         void *S_new, int32_t *err, hipStream_t stream);

hipError_t launch_snapshot_verify(const float *S0, const void *q, const void *k, const void *v,
                                  const float *alpha, const float *beta, const int32_t *parent,
                                  int N, int B, int H, bool f32_in, void *o, float *snapshots,
                                  int32_t *err, hipStream_t stream);

hipError_t launch_snapshot_commit(const float *S0, const float *snapshots, const int32_t *accepted,
                                  int N, int B, int H, float *S_new, int32_t *err,
                                  hipStream_t stream);

hipError_t launch_path_from_node(const int32_t *parent, const int32_t *accepted, int N, int B,
                                 int L_max, int32_t *path, int32_t *path_len, int32_t *err,
                                 hipStream_t stream);

hipError_t launch_accept_greedy(const int32_t *parent, const int32_t *draft, const int32_t *target,
                                const int32_t *root, int N, int B, int L_max, int32_t *path,
                                int32_t *path_len, int32_t *bonus, int32_t *err, hipStream_t stream);

}  // namespace treewy
