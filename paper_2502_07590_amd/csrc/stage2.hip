// Stage 2, order-agnostic form: exact softmax attention over the selected KV only, forward and
// backward (paper Sec. "Sparse Attention with Query Grouping", per-query form; attention formula
// of Sec. "Various Self-Attention Paradigms"), for index rows in ANY order.  The inner loops live in stage2_core.h.
//
// Two layouts: a lane group per row (a wave handles 64 / lanes rows side by side), and a wave per row for small problems and
// for the key-major step, whose lists differ in length.
#include <algorithm>

#include "stage2_core.h"

namespace dsv {

// ------------------------------------------------------------------------------------ forward
template <typename T, int D, int LPR, bool CARE>
__global__ __launch_bounds__(256) void sparse_fwd_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                         const T *__restrict__ V, const int32_t *__restrict__ idx,
                                                         T *__restrict__ O, float *__restrict__ lse, int L,
                                                         float scale, HeadTable tab)
{
    typedef LaneLayout<T, D, LPR> LL;
    constexpr int CH = D / LPR;
    constexpr int RPW = 64 / LPR;  // rows per wave
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / LPR, s = lane % LPR;
    const int64_t iq = (int64_t)blockIdx.x * (4 * RPW) + wave * RPW + grp;
    const bool live = iq < L;
    const int64_t i = live ? iq : L - 1;
    const int64_t head_base = (int64_t)bh * L * D;
    const int32_t *row = idx + tab.off[slot] + i * k;

    const RowChunk<T, CH> q = load_chunk<T, CH, LL::PSB>(Q + head_base + i * D + LL::off(s));
    FwdState<CH> st;
    st.m = -INFINITY;
    st.l = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) st.acc[c] = 0.f;
    __shared__ __align__(16) int32_t stage_all[256 / LPR][kStage];  // one index staging slot per row group
    int32_t *stage = stage_all[threadIdx.x / LPR];
    constexpr bool FOLD = CARE && sizeof(T) == 4;
    __shared__ float sums[FOLD ? (CH + 2) * 256 : 256];
    fwd_sweep<T, D, LPR, CARE, FOLD>(st, q, K + head_base, V + head_base, (uint32_t)LL::off(s), row, 0, k, scale * kLog2e, stage, s,
                               sums + threadIdx.x);

    const float inv = 1.f / st.l;
#pragma unroll
    for (int c = 0; c < CH; ++c) st.acc[c] *= inv;
    if (live) {
        store_chunk<T, CH, LL::PSB>(O + head_base + i * D + LL::off(s), st.acc);
        if (s == 0) lse[(int64_t)bh * L + i] = (st.m + log2f(st.l)) * kLn2;
    }
}

// ------------------------------------------------------------------------------------ backward
// Two gather passes with no floating-point atomics:
//   dq pass    query-major over idx: dQ and the row term Delta_i;
//   dkdv pass  key-major over the transposed index (for each key, the queries that selected it):
//              dK and dV, each output row owned by one wave; keys with an empty list get zeros.
//                dK_j = scale * sum_i dS_ij q_i,  dV_j = sum_i p_ij dO_i,  dS_ij = p_ij (dO_i . v_j - Delta_i)
// Delta_i = dO_i . O_i equals sum_j p_ij dP_ij over the selected keys (dP_ij = dO_i . v_j); the dq
// pass forms it from that sum in fp32, because the stored O is rounded to the storage type and the
// error of dO . O_stored alone would exceed the output tolerance.  One sweep yields both Delta and dQ:
// with D0 = dO_i . O_stored as a centring value,
//   dQ_i = scale * ( sum_j p_ij (dP_ij - D0) k_j  -  (Delta_i - D0) * sum_j p_ij k_j ).
// Delta is kept for the dkdv pass.
template <typename T, int D, int LPR, bool CARE>
__global__ __launch_bounds__(256) void sparse_bwd_dq_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                            const T *__restrict__ V,
                                                            const int32_t *__restrict__ idx, const T *__restrict__ O,
                                                            const float *__restrict__ lse, const T *__restrict__ dO,
                                                            T *__restrict__ dQ, float *__restrict__ delta_out, int L,
                                                            float scale, HeadTable tab)
{
    typedef LaneLayout<T, D, LPR> LL;
    constexpr int CH = D / LPR;
    constexpr int RPW = 64 / LPR;  // rows per wave
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / LPR, s = lane % LPR;
    const int64_t iq = (int64_t)blockIdx.x * (4 * RPW) + wave * RPW + grp;
    const bool live = iq < L;
    const int64_t i = live ? iq : L - 1;
    const int64_t head_base = (int64_t)bh * L * D;
    const int32_t *row = idx + tab.off[slot] + i * k;

    const RowChunk<T, CH> q = load_chunk<T, CH, LL::PSB>(Q + head_base + i * D + LL::off(s));
    const RowChunk<T, CH> go = load_chunk<T, CH, LL::PSB>(dO + head_base + i * D + LL::off(s));
    const RowChunk<T, CH> o = load_chunk<T, CH, LL::PSB>(O + head_base + i * D + LL::off(s));
    const float delta0 = row_sum<LPR>(dot_chunk<T, CH>(go, o));
    DqState<CH> st;
    st.delta = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) { st.a[c] = 0.f; st.b[c] = 0.f; }
    __shared__ __align__(16) int32_t stage_all[256 / LPR][kStage];  // one index staging slot per row group
    int32_t *stage = stage_all[threadIdx.x / LPR];
    constexpr bool FOLD = CARE && sizeof(T) == 4;
    __shared__ float sums[FOLD ? (2 * CH + 1) * 256 : 256];
    dq_sweep<T, D, LPR, FOLD>(st, q, go, K + head_base, V + head_base, (uint32_t)LL::off(s), row, 0, k, scale * kLog2e,
                   lse[(int64_t)bh * L + i] * kLog2e, delta0, stage, s, sums + threadIdx.x);
    if (live) {
        float dq[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) dq[c] = scale * (st.a[c] - (st.delta - delta0) * st.b[c]);
        store_chunk<T, CH, LL::PSB>(dQ + head_base + i * D + LL::off(s), dq);
        if (s == 0) delta_out[(int64_t)bh * L + i] = st.delta;
    }
}

// ------------------------------------------------------------------------------------ a wave per row
// Forms for heads whose K and V rows an L2 holds: the 64 / LPR lane groups of a wave share ONE row (or key), each walks an
// equal part of its index row (or list), and the parts' sums meet in a butterfly over the groups.  No ranges, no partial
// results in memory, no row order: one launch, and 64 / LPR times the waves of the forms above, which is what a short
// sequence lacks (L = 1024, two heads, fp32, k = 128: the forward 33.6 -> 12.7 us, the backward 72.9 -> 25.5 us against the blocked
// forms).  The key-major step takes this form wherever it does not run blocked: lists differ in length by an order of
// magnitude, and a wave that owns 16 of them waits for the longest (L = 32768, four heads, k = 2048, lists as stage 1 makes
// them: 19.8 ms by lane groups, 14.4 by waves).
// This group's part of n positions: whole steps of 4.
template <int LPR> __device__ __forceinline__ void group_part(int n, int grp, int &tb, int &te)
{
    const int per = ((n + 64 / LPR - 1) / (64 / LPR) + 3) & ~3;
    tb = min(grp * per, n);
    te = min(tb + per, n);
}

template <typename T, int D, int LPR, bool CARE>
__global__ __launch_bounds__(256) void sparse_fwd_wave_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                              const T *__restrict__ V, const int32_t *__restrict__ idx,
                                                              T *__restrict__ O, float *__restrict__ lse, int L, float scale,
                                                              HeadTable tab)
{
    typedef LaneLayout<T, D, LPR> LL;
    constexpr int CH = D / LPR;
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int lane = threadIdx.x & 63;
    const int grp = lane / LPR, s = lane % LPR;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= L) return;  // whole wave; nothing synchronises across waves
    const int64_t head_base = (int64_t)bh * L * D;
    const int32_t *row = idx + tab.off[slot] + i * k;
    const RowChunk<T, CH> q = load_chunk<T, CH, LL::PSB>(Q + head_base + i * D + LL::off(s));
    FwdState<CH> st;
    st.m = -INFINITY;
    st.l = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) st.acc[c] = 0.f;
    __shared__ __align__(16) int32_t stage_all[256 / LPR][kStage];
    int tb, te;
    group_part<LPR>(k, grp, tb, te);
    fwd_sweep<T, D, LPR, CARE, false>(st, q, K + head_base, V + head_base, (uint32_t)LL::off(s), row, tb, te, scale * kLog2e,
                               stage_all[threadIdx.x / LPR], s, (float *)nullptr);
    float m = st.m;
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
    const float f = fast_exp2(st.m - m);  // a group without positions: 2^(-inf) = 0
    const float l = group_sum<LPR>(st.l * f);
    const float inv = 1.f / l;
#pragma unroll
    for (int c = 0; c < CH; ++c) st.acc[c] = group_sum<LPR>(st.acc[c] * f) * inv;
    if (grp == 0) {
        store_chunk<T, CH, LL::PSB>(O + head_base + i * D + LL::off(s), st.acc);
        if (s == 0) lse[(int64_t)bh * L + i] = (m + log2f(l)) * kLn2;
    }
}

template <typename T, int D, int LPR, bool CARE>
__global__ __launch_bounds__(256) void sparse_bwd_dq_wave_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                 const T *__restrict__ V, const int32_t *__restrict__ idx,
                                                                 const T *__restrict__ O, const float *__restrict__ lse,
                                                                 const T *__restrict__ dO, T *__restrict__ dQ,
                                                                 float *__restrict__ delta_out, int L, float scale,
                                                                 HeadTable tab)
{
    typedef LaneLayout<T, D, LPR> LL;
    constexpr int CH = D / LPR;
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int lane = threadIdx.x & 63;
    const int grp = lane / LPR, s = lane % LPR;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= L) return;
    const int64_t head_base = (int64_t)bh * L * D;
    const int32_t *row = idx + tab.off[slot] + i * k;
    const RowChunk<T, CH> q = load_chunk<T, CH, LL::PSB>(Q + head_base + i * D + LL::off(s));
    const RowChunk<T, CH> go = load_chunk<T, CH, LL::PSB>(dO + head_base + i * D + LL::off(s));
    const RowChunk<T, CH> o = load_chunk<T, CH, LL::PSB>(O + head_base + i * D + LL::off(s));
    const float delta0 = row_sum<LPR>(dot_chunk<T, CH>(go, o));
    DqState<CH> st;
    st.delta = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) { st.a[c] = 0.f; st.b[c] = 0.f; }
    __shared__ __align__(16) int32_t stage_all[256 / LPR][kStage];
    int tb, te;
    group_part<LPR>(k, grp, tb, te);
    constexpr bool FOLD = CARE && sizeof(T) == 4 && LPR > 8;  // eight parts of a row are short sums as they are
    __shared__ float sums[FOLD ? (2 * CH + 1) * 256 : 256];
    dq_sweep<T, D, LPR, FOLD>(st, q, go, K + head_base, V + head_base, (uint32_t)LL::off(s), row, tb, te, scale * kLog2e,
                        lse[(int64_t)bh * L + i] * kLog2e, delta0, stage_all[threadIdx.x / LPR], s, sums + threadIdx.x);
    const float delta = group_sum<LPR>(st.delta);
    float dq[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) dq[c] = scale * group_sum<LPR>(st.a[c] - (delta - delta0) * st.b[c]);
    if (grp == 0) {
        store_chunk<T, CH, LL::PSB>(dQ + head_base + i * D + LL::off(s), dq);
        if (s == 0) delta_out[(int64_t)bh * L + i] = delta;
    }
}

template <typename T, int D, int LPR>
__global__ __launch_bounds__(256) void sparse_bwd_dkdv_wave_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                   const T *__restrict__ V, const int32_t *__restrict__ idxT,
                                                                   const int64_t *__restrict__ col,
                                                                   const float *__restrict__ lse,
                                                                   const float *__restrict__ delta, const T *__restrict__ dO,
                                                                   T *__restrict__ dK, T *__restrict__ dV, int L, float scale,
                                                                   HeadTable tab)
{
    typedef LaneLayout<T, D, LPR> LL;
    constexpr int CH = D / LPR;
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int lane = threadIdx.x & 63;
    const int grp = lane / LPR, s = lane % LPR;
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= L) return;
    const int64_t head_base = (int64_t)bh * L * D;
    const int64_t *cp = col + (int64_t)bh * (L + 1);
    const int64_t beg = cp[j];
    const int n = (int)(cp[j + 1] - beg);
    const RowChunk<T, CH> kc = load_chunk<T, CH, LL::PSB>(K + head_base + j * D + LL::off(s));
    const RowChunk<T, CH> vc = load_chunk<T, CH, LL::PSB>(V + head_base + j * D + LL::off(s));
    DkdvState<CH> st;
#pragma unroll
    for (int c = 0; c < CH; ++c) { st.dk[c] = 0.f; st.dv[c] = 0.f; }
    __shared__ __align__(16) int32_t stage_all[256 / LPR][kStage];
    int tb, te;
    group_part<LPR>(n, grp, tb, te);
    dkdv_sweep<T, D, LPR, sizeof(T) == 4 && (LPR > 8)>(st, kc, vc, Q + head_base, dO + head_base, lse + (int64_t)bh * L, delta + (int64_t)bh * L,
                          (uint32_t)LL::off(s), idxT + tab.off[slot] + beg, tb, te, scale * kLog2e,
                          stage_all[threadIdx.x / LPR], s);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        st.dk[c] = scale * group_sum<LPR>(st.dk[c]);
        st.dv[c] = group_sum<LPR>(st.dv[c]);
    }
    if (grp == 0) {
        store_chunk<T, CH, LL::PSB>(dK + head_base + j * D + LL::off(s), st.dk);
        store_chunk<T, CH, LL::PSB>(dV + head_base + j * D + LL::off(s), st.dv);
    }
}

// ------------------------------------------------------------------------------------ host
// CARE of the kernels (FINE and FOLD of stage2_core.h): for rows that ranges could have walked.  Calls without the flag never had
// ranges, and go without: 0 to 9 % of the forward, up to 20 % of the dq step of long fp32 rows.
template <typename T, int D, bool CARE>
static dsv_status fwd_c(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                        const void *V, const int32_t *idx, void *O, float *lse, hipStream_t st)
{
    constexpr int LPR = SweepLanes<T, D>::fwd;
    const auto kern = waves ? &sparse_fwd_wave_kernel<T, D, LPR, CARE> : &sparse_fwd_kernel<T, D, LPR, CARE>;
    const int rows = waves ? 4 : 256 / LPR;  // per block
    for (int t = 0; t < n_tabs; ++t) {
        hipLaunchKernelGGL(kern, dim3((p.L + rows - 1) / rows, tabs[t].n), dim3(256), 0, st, (const T *)Q, (const T *)K, (const T *)V, idx,
                           (T *)O, lse, p.L, p.scale, tabs[t]);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

template <typename T, int D>
static dsv_status fwd_t(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                        const void *V, const int32_t *idx, void *O, float *lse, hipStream_t st)
{
    KernelSpan span(DSV_KERNEL_FWD_SWEEP, st);
    return p.flags & DSV_FLAG_SORTED_INDEX ? fwd_c<T, D, true>(p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, st)
                                           : fwd_c<T, D, false>(p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, st);
}

template <typename T, int D, bool CARE>
static dsv_status bwd_dq_c(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                           const void *V, const int32_t *idx, const void *O, const float *lse, const void *dO,
                           void *dQ, float *delta, hipStream_t st)
{
    constexpr int LPR = SweepLanes<T, D>::dq;
    const auto kern = waves ? &sparse_bwd_dq_wave_kernel<T, D, LPR, CARE> : &sparse_bwd_dq_kernel<T, D, LPR, CARE>;
    const int rows = waves ? 4 : 256 / LPR;  // per block
    for (int t = 0; t < n_tabs; ++t) {
        hipLaunchKernelGGL(kern, dim3((p.L + rows - 1) / rows, tabs[t].n), dim3(256), 0, st, (const T *)Q, (const T *)K, (const T *)V, idx,
                           (const T *)O, lse, (const T *)dO, (T *)dQ, delta, p.L, p.scale, tabs[t]);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

template <typename T, int D>
static dsv_status bwd_dq_t(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                           const void *V, const int32_t *idx, const void *O, const float *lse, const void *dO,
                           void *dQ, float *delta, hipStream_t st)
{
    KernelSpan span(DSV_KERNEL_DQ_SWEEP, st);
    if constexpr (sizeof(T) == 4) {
        if (p.flags & DSV_FLAG_SORTED_INDEX)
            return bwd_dq_c<T, D, true>(p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, dO, dQ, delta, st);
    }
    return bwd_dq_c<T, D, false>(p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, dO, dQ, delta, st);
}

template <typename T, int D>
static dsv_status bwd_dkdv_t(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const void *Q, const void *K,
                             const void *V, const int32_t *idxT, const int64_t *col, const float *lse,
                             const float *delta, const void *dO, void *dK, void *dV, hipStream_t st)
{
    KernelSpan span(DSV_KERNEL_DKDV_SWEEP, st);
    for (int t = 0; t < n_tabs; ++t) {
        hipLaunchKernelGGL((sparse_bwd_dkdv_wave_kernel<T, D, SweepLanes<T, D>::dq>), dim3((p.L + 3) / 4, tabs[t].n), dim3(256), 0, st,
                           (const T *)Q, (const T *)K, (const T *)V, idxT, col, lse, delta, (const T *)dO, (T *)dK, (T *)dV, p.L,
                           p.scale, tabs[t]);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

#define DSV_DISPATCH_TD(FN, ...)                                        \
    do {                                                                \
        if (p.dtype == DSV_BF16) {                                      \
            if (p.d == 64) return FN<bf16_t, 64>(__VA_ARGS__);          \
            if (p.d == 128) return FN<bf16_t, 128>(__VA_ARGS__);        \
        } else if (p.dtype == DSV_F32) {                                \
            if (p.d == 64) return FN<float, 64>(__VA_ARGS__);           \
            if (p.d == 128) return FN<float, 128>(__VA_ARGS__);         \
        }                                                               \
        return DSV_EUNSUPPORTED;                                        \
    } while (0)

dsv_status launch_sparse_fwd(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                             const void *V, const int32_t *idx, void *O, float *lse, hipStream_t st)
{
    DSV_DISPATCH_TD(fwd_t, p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, st);
}

dsv_status launch_bwd_dq(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                         const void *V, const int32_t *idx, const void *O, const float *lse, const void *dO, void *dQ,
                         float *delta, hipStream_t st)
{
    DSV_DISPATCH_TD(bwd_dq_t, p, tabs, n_tabs, waves, Q, K, V, idx, O, lse, dO, dQ, delta, st);
}

dsv_status launch_bwd_dkdv(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const void *Q, const void *K,
                           const void *V, const int32_t *idxT, const int64_t *col, const float *lse, const float *delta,
                           const void *dO, void *dK, void *dV, hipStream_t st)
{
    DSV_DISPATCH_TD(bwd_dkdv_t, p, tabs, n_tabs, Q, K, V, idxT, col, lse, delta, dO, dK, dV, st);
}

}  // namespace dsv
