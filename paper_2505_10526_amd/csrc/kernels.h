// Internal interface between the translation units of libmassv_verify: launches (every launch_* function only enqueues on `st` and
// returns a massv_status) and the device code that two of them share.
#pragma once

#include "common.h"
#include <hip/hip_ext.h>

namespace massv {

// ---- one-shot kernel timing hook (api.hip) ----
// massv_trace_kernel() arms a request on the calling thread; the next launch of that kernel goes out
// through hipExtLaunchKernelGGL with the caller's two events, which then carry the kernel's own begin
// and end timestamps (the same clock a profiler's kernel trace reports), and the request is disarmed.
struct TraceRequest { int kid; hipEvent_t start, stop; };
TraceRequest& trace_request();

template <typename K, typename... Args>
inline void launch_traced(int kid, K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, Args... args) {
    TraceRequest& t = trace_request();
    if (kid >= 0 && t.kid == kid) {
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, st, t.start, t.stop, 0, args...);
        t.kid = -1;
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, st, args...);
    }
}

// ---- small row-wise kernels (elementwise.hip) ----
// Row m of X -> RMSNorm -> operand-order output (see packed_index), by a workgroup of kNormPackThreads; g == nullptr: no
// normalisation, the row is only re-laid out.  H % 8 == 0.
constexpr int kNormPackThreads = 1024;
__device__ inline void rmsnorm_pack_row(const bf16_t* __restrict__ x, const bf16_t* __restrict__ g, bf16_t* __restrict__ y,
                                        int H, float eps, int mt_count, int m) {
    const int tid = threadIdx.x;
    const bf16x8* xr = reinterpret_cast<const bf16x8*>(x + (size_t)m * H);
    const int groups = H / 8;
    float rstd = 1.f;
    if (g) {
        float ss = 0.f;
        for (int k8 = tid; k8 < groups; k8 += kNormPackThreads) {
            const bf16x8 v = xr[k8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float f = (float)v[e]; ss += f * f; }
        }
        ss = wave_sum(ss);
        __shared__ float part[16];
        if ((tid & 63) == 0) part[tid >> 6] = ss;
        __syncthreads();
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) tot += part[w];
        rstd = 1.0f / sqrtf(tot / (float)H + eps);
    }
    for (int k8 = tid; k8 < groups; k8 += kNormPackThreads) {
        bf16x8 v = xr[k8];
        if (g) {
            const bf16x8 gv = reinterpret_cast<const bf16x8*>(g)[k8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (bf16_t)((float)v[e] * rstd * (float)gv[e]);
        }
        *reinterpret_cast<bf16x8*>(y + packed_index(m, k8 * 8, mt_count)) = v;
    }
}
// bf16 only: y[m,:] = x[m,:] * g / sqrt(mean(x[m,:]^2) + eps), output in operand order (packed_index); g == nullptr re-lays the rows out without normalising.
int launch_rmsnorm_packed(const void* x, const void* g, void* y, int M, int H, float eps, hipStream_t st);
// Rotates the q and k heads of qkv[M][(n_q+2n_kv)*d] by pos[m], writes q to
// q_out[M][n_q][d] and the k / v rows of token (b,i) to cache row kv_len[b]+i.
// q_norm / k_norm [d] (nullptr = none): RMSNorm of every query / key head before the rotation.
int launch_rope_append(const void* qkv, const int32_t* pos, const int32_t* kv_len, void* q_out,
                       void* k_cache, void* v_cache, const void* q_norm, const void* k_norm, float eps,
                       const massv_attn_desc& a, float theta, hipStream_t st);
// bf16: sums the K slabs of the q/k/v projection's partial sums [slabs][Mp][(n_q+2n_kv)*d], adds the biases
// (nullptr = none), normalises the q / k heads (q_norm, k_norm; nullptr = no), rotates q and k, writes q to
// q_out[M][n_q][d] and k / v to their cache rows.
int launch_qkv_finish(const float* partial, int n_slabs, size_t slab_stride, const void* bq, const void* bk,
                      const void* bv, const int32_t* pos, const int32_t* kv_len, void* q_out, void* k_cache,
                      void* v_cache, const void* q_norm, const void* k_norm, float eps,
                      const massv_attn_desc& a, float theta, hipStream_t st);
// bf16: y[m,:] = sum over slabs of partial[s][m,:]; r = base + (post ? rmsnorm(y, post) : y) with base = h_in (fp32
// rows) when given, else x; r is written to h_out (fp32) when given, else to x (bf16); if ln != nullptr also
// rmsnorm(r, ln) in operand order to xn_packed.
int launch_residual_finish(const float* partial, int n_slabs, size_t slab_stride, void* x, const float* h_in, float* h_out,
                           const void* post, const void* ln, void* xn_packed, int M, int H, float eps, hipStream_t st);
// fp32: x[m,:] += rmsnorm(y[m,:], g).
int launch_postnorm_residual(void* x, const void* y, const void* g, int M, int H, float eps, hipStream_t st);

// ---- projections (gemm.hip) ----
// One linear map Y = X W^T over M rows.  Up to three weight matrices that share
// X are applied in one launch; their outputs are laid side by side in Y
// ([M][n0+n1+n2]).
enum Epilogue {
    EPI_STORE = 0,      // f32 only: y = acc (+ bias)
    EPI_RESIDUAL = 1,   // f32 only: y = acc + residual (residual may alias y)
    EPI_GATED = 2,      // two matrices (gate, up) of equal size: y = act(gate) * up (bf16: y in operand order)
    EPI_LOGITS = 3,     // y = acc stored as float32 [M][N]
    EPI_PARTIAL = 4,    // bf16 only: fp32 partial sums y[slab][16*ceil(M/16)][N], one slab per K range;
                        // bias / residual are applied by the kernel that sums the slabs
    EPI_ARGMAX = 5,     // bf16 only: nothing is stored but, per row and workgroup, the largest output and its
                        // (lowest) column: y is RowPartial[M][gemm_row_pieces]
    EPI_LOGITS_STATS = 6 // bf16 only: EPI_LOGITS, and stats[M][gemm_row_pieces] receives per row and workgroup the largest
                        // output, its lowest column and the sum of exp((x - largest) / T) over the workgroup's columns
};
// Maximum, first arg-max and sum of exponentials of one piece of a logit row (pieces are merged by accept_decide_kernel).
struct RowPartial { float m; int arg; double s; };
struct GemmPlan { int nt, slabs, groups; };
// Greedy accept chain from per-piece row partials: part[row][C] for the B*(gamma+1) target rows (accept.hip).
int launch_accept_decide_greedy(const RowPartial* part, int C, const int32_t* draft_tokens, int B, int gamma, int V,
                                int32_t* n_accepted, int32_t* out_tokens, hipStream_t st);
// log2(e)/T split in two floats (d*hi + d*lo is d*log2(e)/T to about 1 ulp) and 1/T: how every kernel that forms
// exp((x - max)/T) scales its exponent.
struct TempScale { float hi, lo; double inv; };
TempScale temp_scale(float temperature);
// The accept rule at T > 0 with the target rows' statistics already formed by the vocabulary projection
// (part_t[B*(gamma+1)][C_t], written by an EPI_LOGITS_STATS launch).  Pass 1, over the draft rows only, goes out ahead of the
// projection with the norm of its rows (launch_norm_draft_stats: launch_rmsnorm_packed and pass 1 in one launch).
// ws: accept_prestats_bytes(B, gamma, V) bytes, the same for both.
int launch_norm_draft_stats(const void* x, const void* g, void* y, int M, int H, float eps, const float* draft_logits,
                            float temperature, int B, int gamma, int V, void* ws, hipStream_t st);
size_t accept_prestats_bytes(int B, int gamma, int V);
int launch_accept_prestats(const float* target_logits, const RowPartial* part_t, int C_t, const float* draft_logits,
                           const int32_t* draft_tokens, const float* uniforms, float temperature, int B, int gamma, int V,
                           int32_t* n_accepted, int32_t* out_tokens, void* ws, hipStream_t st);
struct GemmArgs {
    const void* x;            // f32: [M][K] row-major; bf16: operand order (packed_index), packed_elems(M,K) elements
    const void* w[3];         // [n_i][K]
    const void* bias[3];      // [n_i] or nullptr
    int n[3];                 // rows of each matrix (0 = unused)
    const void* residual;     // EPI_RESIDUAL: [M][n0]
    void* y;
    void* stats;              // EPI_LOGITS_STATS: RowPartial[M][gemm_row_pieces]
    float temperature;        // EPI_LOGITS_STATS: T > 0 of the exponentials
    const void* norm;         // f32 only: gains [K]; the rows of x are RMS-normalised first (nullptr: taken as they are)
    float norm_eps;
    int M, K;
    int epilogue, act, dtype;
    int kid;                  // massv_kernel_id bracketed by a pending trace request
};
int launch_gemm(const GemmArgs& g, hipStream_t st);

// ---- projections over the whole of K with what follows them (whole.hip); bf16 ----
// Rows that come as x * gains: their 1 / rms is applied to the projection's accumulators.  ss[parts][16 ceil(M/16)]: sums of
// squares of the rows' pieces, H the row's width; ss == nullptr: the rows are normalised already.
struct RowScale { const float* ss; int parts, H; float eps; };
// Each thread of T takes four rows of every (T / R4)-th piece; the first HOLD of them are asked for at once and stay on their way ...
template <int T, int MT>
struct RowScaleSums {
    static constexpr int R4 = 4 * MT;                              // threads a piece
    static constexpr int G = T / R4, HOLD = MT * 1024 / T;
    floatx4 v[HOLD];
    __device__ inline void load(const RowScale& r, int tid) {
        const int q = tid % R4;
#pragma unroll
        for (int i = 0; i < HOLD; ++i) {
            const int part = tid / R4 + i * G;
            v[i] = part < r.parts ? *reinterpret_cast<const floatx4*>(r.ss + (size_t)part * MT * 16 + q * 4) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
    }
// ... the threads of 16 lanes add theirs up and leave the share in s_ss[T / 16][16 MT] (a barrier later it may be read) ...
    __device__ inline void store(const RowScale& r, float* s_ss, int tid) {
        const int q = tid % R4;
        floatx4 s = v[0];
#pragma unroll
        for (int i = 1; i < HOLD; ++i) s += v[i];
        for (int part = tid / R4 + HOLD * G; part < r.parts; part += G)
            s += *reinterpret_cast<const floatx4*>(r.ss + (size_t)part * MT * 16 + q * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] += row_ror<8>(s[e]);
            if constexpr (R4 == 4) s[e] += row_ror<4>(s[e]);
        }
        const int l = tid % 16;
        if (l < R4) *reinterpret_cast<floatx4*>(s_ss + (tid / 16) * MT * 16 + l * 4) = s;
    }
};
// ... and a row's factor is formed from the T / 16 shares, by every thread for itself or, where the 16 threads of a row (c = 0 .. 15)
// all want it, together.
__device__ inline float row_rstd_of(const RowScale& r, float sum) { return 1.0f / sqrtf(sum / (float)r.H + r.eps); }
template <int T, int MT>
__device__ inline float row_rstd(const RowScale& r, const float* s_ss, int m) {
    float t = s_ss[m];
#pragma unroll
    for (int w = 1; w < T / 16; ++w) t += s_ss[w * MT * 16 + m];
    return row_rstd_of(r, t);
}
template <int T, int MT>
__device__ inline float row_rstd_by16(const RowScale& r, const float* s_ss, int m, int c) {
    float t = s_ss[c * MT * 16 + m];
#pragma unroll
    for (int w = 16; w < T / 16; w += 16) t += s_ss[(w + c) * MT * 16 + m];
    t += row_ror<8>(t); t += row_ror<4>(t); t += row_ror<2>(t); t += row_ror<1>(t);      // (the same sum in every lane)
    return row_rstd_of(r, t);
}

// Gated-MLP activations through the hardware exp2 and reciprocal (about 1e-6 relative error, the result is
// rounded to bf16): the library versions with exact division and tanhf made the projection's epilogue a few
// thousand instructions long, 3 us of a 46 us launch.  0.5 (1 + tanh(u)) is sigmoid(2u).
__device__ inline float fast_sigmoid(float x) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}
__device__ inline float gemm_act(float x, int act) {
    if (act == MASSV_ACT_SILU) return x * fast_sigmoid(x);
    const float c = 0.7978845608028654f;
    return x * fast_sigmoid(2.0f * c * (x + 0.044715f * x * x * x));
}

// Whether the projection (GemmArgs as for launch_gemm) is faster this way than as launch_gemm runs it.
bool whole_qkv_pays(const GemmArgs& g);
bool whole_residual_pays(const GemmArgs& g);
// launch_gemm + launch_qkv_finish in one launch (g.bias: nullptr = none); no head norms.  raw_x != nullptr: also the norm ahead of
// them, of the row-major rows raw_x with these gains (scale: H and eps; g.x is not read).
int launch_whole_qkv(const GemmArgs& g, const RowScale& scale, const void* raw_x, const void* gain, const int32_t* pos,
                     const int32_t* kv_len, void* q_out, void* k_cache, void* v_cache, const massv_attn_desc& a, float theta, hipStream_t st);
// launch_gemm + launch_residual_finish (without a post norm) in one launch, except that xn_packed receives rows * ln and
// ss[whole_residual_parts][16 ceil(M/16)] the sums of squares (both only when ln != nullptr).
int launch_whole_residual(const GemmArgs& g, const void* x_in, const float* h_in, void* x_out, float* h_out, const void* ln,
                          void* xn_packed, float* ss, hipStream_t st);
int whole_residual_parts(const GemmArgs& g);
// launch_gemm of an EPI_GATED projection, of rows * gains when scale.ss is set (at most 32 rows then).
int launch_gated(const GemmArgs& g, const RowScale& scale, hipStream_t st);
// f32: the q/k/v projections (g: matrices, biases, x and norm as for launch_gemm) with the rotation by pos and the append
// of k / v at cache rows kv_len[b] + i in the same launch; no head norms (those need a whole head: launch_rope_append).
int launch_qkv_rope_f32(const GemmArgs& g, const int32_t* pos, const int32_t* kv_len, void* q_out, void* k_cache, void* v_cache,
                        const massv_attn_desc& a, float theta, hipStream_t st);
// bf16: tile count per wave and number of K slabs launch_gemm will use; bytes of the EPI_PARTIAL output.
GemmPlan gemm_plan(const GemmArgs& g);
size_t gemm_partial_bytes(const GemmArgs& g);
// EPI_ARGMAX, EPI_LOGITS_STATS: records per row that the launch leaves (its workgroups).
int gemm_row_pieces(const GemmArgs& g);
// Whether launch_gemm can run this problem (host-side shape check only).
int gemm_supported(const GemmArgs& g);

// ---- attention (attention.hip) ----
size_t attention_workspace(const massv_attn_desc& a);
int check_attn_desc(const massv_attn_desc* a);
// out_packed (bf16 only): write out[B*Q][n_q*d] in operand order for the output projection.
int launch_attention(const massv_attn_desc& a, const void* q, const void* k_cache, const void* v_cache,
                     const int32_t* kv_len, void* out, void* ws, bool out_packed, hipStream_t st);

}  // namespace massv
