// Projections of a few rows whose workgroups own their output features over the whole of K, so that what follows a
// projection rides on it: bias, rotation and cache append behind q/k/v, the residual and the next norm behind O and down.
// (gemm_stream_kernel's K slabs leave both to a launch of their own that sums the slabs, 3.6 to 5 us each; an empty launch
// is 2.7.)  A layer of up to 16 rows is six launches instead of nine.
//
// The RMSNorm between two projections is split: the projection that closes a block stores row * gains as the next operand
// and, per workgroup and row, the sum of squares of its columns (of the fp32 row, ahead of any rounding); the projection that
// opens the next block sums those and multiplies its accumulators by 1 / rms.  Rounding row * gains to bf16 has the same
// relative size as rounding the normalised row.
//
// Bound by latency where the weights are few (an empty launch, one trip to memory, the sum over the waves), by L2 and HBM
// where they are many: a workgroup reads all of X for its 8, 16 or 32 features, which here comes at about
// 14 TB/s together and 60 GB/s a compute unit (L2 hits alone, with nothing else under way: 32 TB/s and 150 GB/s).  Hence 16 waves that take the 32-wide steps of K in turn with all loads of U steps in flight
// (a workgroup of 4 waves with fewer loads each took one more trip to memory), one round of workgroups, and the rules below on how many
// rows and features are worth it.  The operand rows past M are not fetched.
// us a layer in a stack, slabs and this, in turn on one card: 1.5B shape, 8 rows 48.3 -> 39.5, 16 rows 49.3 -> 45.8; 7B shape, 6 rows
// 107.5 -> 101.1; 12B shape (no extra norms), 6 rows 105.3 -> 94.8.  Launches of the 1.5B shape, 8 rows, before and now: q/k/v 4.4 + 3.9 -> 5.5,
// O 4.2 + 3.6 -> 4.4, gate / up 13.8 -> 12.9, down 7.3 -> 8.4 with 3.6 behind it before.
#include "gemm_stream.h"

#include <atomic>

namespace massv {

constexpr int kWholeWaves = 16, kWholeThreads = kWholeWaves * kWave;
constexpr int kWholeGroups = 256;               // workgroups of a launch: one a compute unit
constexpr int kFragPitch = 20;                  // 16 rows of 4 features, 20 apart: the sums are read without bank conflicts
constexpr int kFrag = 4 * kFragPitch * 4;       // floats of one 16 x 16 fragment

// Kernel arguments, no more of them than a kernel needs: every 64 bytes are a trip of their own at its head.
struct WholeQkv {
    const bf16_t* x;                // operand order; RAW: row-major, not normalised
    const bf16_t* w[3];
    const bf16_t* bias[3];
    const int32_t* pos;
    const int32_t* kv_len;
    bf16_t *q_out, *k_cache, *v_cache;
    int M, K, Q, n_q, n_kv, d, l_max;
    double log2_theta;
    RowScale scale;                 // RAW: H and eps alone
    const bf16_t* gain;             // RAW: of the norm
};
struct WholeRes {
    const bf16_t* x;
    const bf16_t* w;
    const bf16_t* x_in; const float* h_in;      // base rows: h_in when given, else x_in
    bf16_t* x_out; float* h_out;                // h_out when given, else x_out
    const bf16_t* ln; bf16_t* xn; float* ss_out;
    int M, K, N;
};
struct WholeGated {
    const bf16_t* x;
    const bf16_t* w[2];
    bf16_t* h;
    int M, K, share, rem, act;      // the first rem workgroups own share + 1 tiles, the others share
    RowScale scale;
};

// A wave's share of K, steps wave, wave + W, ... of n_steps, with U steps' loads in flight: load(slot, step), mul(slot).
// `early` runs once the first loads are on their way.
template <int U, int W, typename Load, typename Mul, typename Early>
__device__ inline void stream_steps(int wave, int n_steps, Load load, Mul mul, Early early) {
    const int cnt = wave < n_steps ? (n_steps - wave + W - 1) / W : 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < cnt) load(u, wave + u * W);
    early();
    int it = 0;
    for (; it + 2 * U <= cnt; it += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) { mul(u); load(u, wave + (it + U + u) * W); }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {                            // U to 2 U - 1 steps are left (fewer only where cnt < U)
        if (it + u < cnt) mul(u);
        if (it + U + u < cnt) load(u, wave + (it + U + u) * W);
    }
    it += U;
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
        if (it + u < cnt) mul(u);
}

// WHOLE_QKV8, WHOLE_QKV16: 8 or 16 rotary pairs (j, j + d/2) of one head a workgroup; 8 pairs are the 16 operand rows of one
//   tile, 16 pairs two tiles.  Angles and rotation in double, as qkv_finish_kernel forms them.
// WHOLE_RES16: 16 features.
// WHOLE_RES8: 8 features of up to 8 rows, K in steps of 64: the features at one 32 of K and the same features at the next 32
//   are the 16 operand rows, the rows of X at both the 16 operand columns; the two diagonal quarters of the product count.
//   Twice the workgroups where 16 features would leave compute units idle (1.5B shape, 8 rows: 43.9 -> 40.9 us a layer).
enum WholeKind { WHOLE_QKV8, WHOLE_QKV16, WHOLE_RES16, WHOLE_RES8 };
template <int KIND> struct WholeArgs { typedef WholeRes type; };
template <> struct WholeArgs<WHOLE_QKV8> { typedef WholeQkv type; };
template <> struct WholeArgs<WHOLE_QKV16> { typedef WholeQkv type; };
// RAW: the rows come as the layer's input does, row-major; the kernel multiplies them by the gains as it reads them and sums their
// squares along the way, which saves the launch that would normalise them first (4.6 us).
template <int MT, int U, int KIND, bool RAW>
__global__ __launch_bounds__(kWholeThreads)
void whole_proj_kernel(typename WholeArgs<KIND>::type g) {
    constexpr bool QKV = KIND <= WHOLE_QKV16, PAIR = KIND == WHOLE_RES8;
    constexpr bool SCALED = QKV && MT == 1 && !RAW;          // rows may come as row * gains (only small launches leave them so)
    constexpr int NT = KIND == WHOLE_QKV16 ? 2 : 1;
    constexpr int W = kWholeWaves, T = kWholeThreads, MP = MT * 16, ROWS = PAIR ? 8 : MP;
    constexpr int FW = PAIR ? 8 : 16, JP = KIND == WHOLE_QKV16 ? 16 : 8;
    static_assert(ROWS * 16 <= T && MP * JP <= T, "a value and an angle a thread");
    extern __shared__ __align__(16) float s_whole[];
    float* red = s_whole;                                    // [W][NT][MT][kFrag]
    float* s_ss = red + W * NT * MT * kFrag;                 // [T / 16][MP] (SCALED, RAW)
    float* s_ang = s_ss + (SCALED || RAW ? T * MT : 0);                  // [MP * JP] cosines, then sines, in double (QKV)
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lr = lane % 16, lc = lane / 16;
    const int tile_steps = g.K / 32, n_steps = PAIR ? g.K / 64 : tile_steps;

    // ---- what the epilogue needs besides the sums is asked for ahead of the weights ----
    // a thread finishes row m = tid / 16 and feature (or pair) c = tid % 16
    const int c = tid % 16, m = tid / 16;
    const bool live = m < g.M;
    const int fcol = blockIdx.x * FW + c % FW;
    int half = 0, seg = 0, hl = 0, jb = 0, feature = 0, cached = 0, pos = 0;
    float base = 0.f, gain = 0.f, bias = 0.f, bias2 = 0.f;
    if constexpr (QKV) {
        half = g.d / 2;
        const int per_head = half / JP, head = blockIdx.x / per_head;
        jb = (blockIdx.x % per_head) * JP;
        seg = head < g.n_q ? 0 : head < g.n_q + g.n_kv ? 1 : 2;
        hl = seg == 0 ? head : seg == 1 ? head - g.n_q : head - g.n_q - g.n_kv;
        feature = jb + (NT == 1 ? (c & 7) + (c < 8 ? 0 : half) : c);
        if (tid < MP * JP) pos = g.pos[tid / JP < g.M ? tid / JP : 0];
        if (live) cached = g.kv_len[m / g.Q];
        if (g.bias[seg]) {
            bias = (float)g.bias[seg][hl * g.d + feature];
            if (NT == 2) bias2 = (float)g.bias[seg][hl * g.d + feature + half];
        }
    } else {
        const size_t o = (size_t)(live ? m : 0) * g.N + fcol;
        base = g.h_in ? g.h_in[o] : (float)g.x_in[o];
        if (g.ln) gain = (float)g.ln[fcol];
    }
    RowScaleSums<T, 1> sums;
    if constexpr (SCALED) if (g.scale.ss) sums.load(g.scale, tid);

    // ---- the stream ----
    const bf16_t *wp[NT], *xp = g.x + (RAW ? (size_t)lr * g.K + lc * 8 : lane * 8);
    bool last_live = (MT - 1) * 16 + lr < g.M;
    if constexpr (KIND == WHOLE_QKV16) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) wp[nt] = g.w[seg] + (size_t)((hl * g.d + jb + nt * half) / 16) * tile_steps * 512 + lane * 8;
    } else if constexpr (KIND == WHOLE_QKV8) {
        const int row = hl * g.d + jb + (lr < 8 ? lr : half + lr - 8);
        wp[0] = g.w[seg] + (size_t)(row / 16) * tile_steps * 512 + (lc * 16 + row % 16) * 8;
    } else if constexpr (PAIR) {
        wp[0] = g.w + (size_t)(blockIdx.x / 2) * tile_steps * 512 + (lr < 8 ? 0 : 512) + (lc * 16 + (blockIdx.x & 1) * 8 + (lr & 7)) * 8;
        xp = g.x + (lr < 8 ? 0 : 512) + (lc * 16 + (lr & 7)) * 8;
        last_live = (lr & 7) < g.M;
    } else {
        wp[0] = g.w + (size_t)blockIdx.x * tile_steps * 512 + lane * 8;
    }
    constexpr int STEP = PAIR ? 1024 : 512;                  // elements of a step
    bf16x8 a[U][NT], xb[U][MT], gb[RAW ? U : 1];
    floatx4 acc[NT][MT];
    float ss[RAW ? MT : 1];
    if constexpr (RAW)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) ss[mt] = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) xb[u][MT - 1] = bf16x8{};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    stream_steps<U, W>(wave, n_steps,
        [&](int u, int s) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) a[u][nt] = ldg_stream(reinterpret_cast<const bf16x8*>(wp[nt] + (size_t)s * STEP));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (mt < MT - 1 || last_live)
                    xb[u][mt] = *reinterpret_cast<const bf16x8*>(RAW ? xp + (size_t)mt * 16 * g.K + s * 32 : xp + ((size_t)s * MT + mt) * STEP);
            if constexpr (RAW) gb[u] = *reinterpret_cast<const bf16x8*>(g.gain + s * 32 + lc * 8);
        },
        [&](int u) {
            if constexpr (RAW)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float v = (float)xb[u][mt][e];
                        ss[mt] += v * v;
                        xb[u][mt][e] = (bf16_t)(v * (float)gb[u][e]);
                    }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][nt], xb[u][mt], acc[nt][mt], 0, 0, 0);
        },
        [&]() {                                              // one (row, pair) angle a thread, while the first weights travel
            if constexpr (QKV) {
                if (seg < 2 && tid < MP * JP) {
                    double sn, cs;
                    sincos((double)pos * exp2(-2.0 * (double)(jb + tid % JP) / (double)g.d * g.log2_theta), &sn, &cs);
                    reinterpret_cast<double*>(s_ang)[tid] = cs;
                    reinterpret_cast<double*>(s_ang)[MP * JP + tid] = sn;
                }
            }
            if constexpr (SCALED) if (g.scale.ss) sums.store(g.scale, s_ss, tid);
        });

    // ---- the waves' sums, in wave order ----
    if constexpr (RAW)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) s_ss[(wave * 4 + lc) * MP + mt * 16 + lr] = ss[mt];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<floatx4*>(red + ((wave * NT + nt) * MT + mt) * kFrag + (lc * kFragPitch + lr) * 4) = acc[nt][mt];
    __syncthreads();
    if (m >= ROWS) return;                                   // whole waves
    const float* r = red + (m / 16) * kFrag + ((c / 4) * kFragPitch + m % 16 + (PAIR && c >= 8 ? 8 : 0)) * 4 + c % 4;
    float s = r[0], s2 = NT == 2 ? r[MT * kFrag] : 0.f;
#pragma unroll
    for (int w = 1; w < W; ++w) {
        s += r[w * NT * MT * kFrag];
        if (NT == 2) s2 += r[(w * NT + 1) * MT * kFrag];
    }
    if constexpr (QKV) {
        if constexpr (SCALED || RAW)
            if (RAW || g.scale.ss) { const float f = row_rstd_by16<T, MT>(g.scale, s_ss, m, c); s *= f; s2 *= f; }
        s += bias;
        s2 = NT == 2 ? s2 + bias2 : row_ror<8>(s);           // the pair's other feature
        if (!live) return;
        const int b = m / g.Q;
        const unsigned row = (unsigned)(cached < 0 ? 0 : cached) + (unsigned)(m % g.Q);      // (cannot overflow)
        if (seg < 2) {
            const double cs = reinterpret_cast<double*>(s_ang)[m * JP + c % JP], sn = reinterpret_cast<double*>(s_ang)[MP * JP + m * JP + c % JP];
            const double x1 = s, x2 = s2;
            s = NT == 2 || c < 8 ? (float)(x1 * cs - x2 * sn) : (float)(x1 * cs + x2 * sn);
            if (NT == 2) s2 = (float)(x2 * cs + x1 * sn);
        }
        if (seg == 0) {
            bf16_t* dst = g.q_out + ((size_t)m * g.n_q + hl) * g.d + feature;
            dst[0] = (bf16_t)s;
            if (NT == 2) dst[half] = (bf16_t)s2;
        } else if (row < (unsigned)g.l_max) {
            const size_t bg = (size_t)b * g.n_kv + hl;
            bf16_t* cache = seg == 1 ? g.k_cache : g.v_cache;
            auto at = [&](int f) { return seg == 1 ? k_cache_index(bg, g.l_max, g.d, (int)row, f) : v_cache_index(bg, g.l_max, g.d, (int)row, f); };
            cache[at(feature)] = (bf16_t)s;
            if (NT == 2) cache[at(feature + half)] = (bf16_t)s2;
        }
    } else {
        if constexpr (PAIR) s += row_ror<8>(s);              // both quarters; lanes c and c + 8 hold the same
        const float h = base + s;
        if (live && (!PAIR || c < 8)) {
            if (g.h_out) g.h_out[(size_t)m * g.N + fcol] = h;
            else g.x_out[(size_t)m * g.N + fcol] = (bf16_t)h;
            if (g.ln) g.xn[packed_index(m, fcol, MT)] = (bf16_t)(h * gain);
        }
        if (g.ln) {
            float q = h * h;
            if constexpr (!PAIR) q += row_ror<8>(q);
            q += row_ror<4>(q); q += row_ror<2>(q); q += row_ror<1>(q);
            if (c == 0) g.ss_out[(size_t)blockIdx.x * MP + m] = live ? q : 0.f;
        }
    }
}

// Gate and up projections of up to 16 rows, act(gate) * up in operand order.  The 16 operand rows of a tile are 8 features of the
// gate matrix and the same 8 of the up matrix, so a workgroup's share is even to 8 features: 1.5B shape, 4 or 5 such tiles
// a workgroup where gemm_stream_kernel has 2 or 3 pairs of whole tiles; and 8 waves have U steps of NT tiles in flight, all of K
// at 1536.  41.0 -> 39.4 us a layer at 8 rows, 96.9 -> 95.5 for the 12B shape.
constexpr int kGatedWaves = 8, kGatedThreads = kGatedWaves * kWave;
template <int NT, int U>
__global__ __launch_bounds__(kGatedThreads)
void whole_gated_kernel(WholeGated g) {
    constexpr int W = kGatedWaves, T = kGatedThreads;
    extern __shared__ __align__(16) float s_whole[];
    float* red = s_whole;                                    // [W][NT][kFrag]
    float* s_ss = red + W * NT * kFrag;                      // [T / 16][16]
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lr = lane % 16, lc = lane / 16;
    const int n_steps = g.K / 32, bx = blockIdx.x;
    const int unit0 = bx * g.share + (bx < g.rem ? bx : g.rem), owned = g.share + (bx < g.rem ? 1 : 0);      // NT or NT - 1
    RowScaleSums<T, 1> sums;
    if (g.scale.ss) sums.load(g.scale, tid);
    const bf16_t* wp[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int f = (unit0 + (nt < owned ? nt : 0)) * 8;
        wp[nt] = g.w[lr < 8 ? 0 : 1] + (size_t)(f / 16) * n_steps * 512 + (lc * 16 + f % 16 + (lr & 7)) * 8;
    }
    const bf16_t* xp = g.x + lane * 8;
    const bool live = lr < g.M;
    bf16x8 a[U][NT], xb[U];
    floatx4 acc[NT];
#pragma unroll
    for (int u = 0; u < U; ++u) xb[u] = bf16x8{};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    stream_steps<U, W>(wave, n_steps,
        [&](int u, int s) {
            if (live) xb[u] = *reinterpret_cast<const bf16x8*>(xp + (size_t)s * 512);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (nt < NT - 1 || nt < owned) a[u][nt] = ldg_stream(reinterpret_cast<const bf16x8*>(wp[nt] + (size_t)s * 512));
        },
        [&](int u) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (nt < NT - 1 || nt < owned) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][nt], xb[u], acc[nt], 0, 0, 0);
        },
        [&]() { if (g.scale.ss) sums.store(g.scale, s_ss, tid); });
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        *reinterpret_cast<floatx4*>(red + (wave * NT + nt) * kFrag + (lc * kFragPitch + lr) * 4) = acc[nt];
    __syncthreads();
    const int c = tid % 16;
    for (int v = tid / 16; v < owned * 16; v += T / 16) {
        const int nt = v / 16, m = v % 16;
        if (m >= g.M) continue;                              // (all 16 lanes of a row)
        const float* r = red + nt * kFrag + ((c / 4) * kFragPitch + m) * 4 + c % 4;
        float s = r[0];
#pragma unroll
        for (int w = 1; w < W; ++w) s += r[w * NT * kFrag];
        if (g.scale.ss) s *= row_rstd_by16<T, 1>(g.scale, s_ss, m, c);
        const float up = row_ror<8>(s);
        if (c < 8) g.h[packed_index(m, (unit0 + nt) * 8 + c, 1)] = (bf16_t)(gemm_act(s, g.act) * up);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <auto Kernel, typename Args>
static int launch_whole_kernel(const Args& d, int groups, int threads, size_t lds, int kid, hipStream_t st) {
    if (lds > 48 * 1024) {                       // more dynamic LDS than a kernel may use by default
        static std::atomic<bool> ready[64];       // zero-initialised; calls may come from several threads
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MASSV_ELAUNCH;
        if (!ready[dev].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return MASSV_ELAUNCH;
            ready[dev].store(true, std::memory_order_release);
        }
    }
    launch_traced(kid, Kernel, dim3(groups), dim3(threads), lds, st, d);
    return launch_status();
}

template <int MT, int U, int KIND, bool RAW = false>
static int launch_whole(const typename WholeArgs<KIND>::type& d, int groups, int kid, hipStream_t st) {
    constexpr bool qkv = KIND <= WHOLE_QKV16;
    constexpr int NT = KIND == WHOLE_QKV16 ? 2 : 1;
    const size_t lds = (size_t)kWholeWaves * NT * MT * kFrag * 4 + (RAW || (qkv && MT == 1) ? kWholeThreads * MT * 4 : 0) + (qkv ? MT * 16 * NT * 8 * 16 : 0);
    return launch_whole_kernel<&whole_proj_kernel<MT, U, KIND, RAW>>(d, groups, kWholeThreads, lds, kid, st);
}

static int n_total(const GemmArgs& g) { return g.n[0] + g.n[1] + g.n[2]; }

// q/k/v up to 48 rows, as 8 pairs a workgroup where that is one round of workgroups, else as 16.  us a layer, slabs and this:
// 1.5B shape (128 workgroups of 8 pairs), 8 / 24 / 48 / 64 rows 48.3 -> 45.8, 52.2 -> 50.2, 60.1 -> 57.9, 67.1 -> 65.2; 7B (144 of 16),
// 6 / 24 / 48 / 64 rows 107.7 -> 104.9, 115.0 -> 113.3, 124.6 -> 122.8, 150.7 -> 156.4 (8 pairs, 288 workgroups: 106.4, 115.4, 129.1 at
// 6, 24, 48 rows); 12B (256 of 16), 24 / 48 / 64 rows 117.7 -> 112.5, 136.2 -> 131.2, 151.4 -> 155.3.  Few workgroups are no reason against it
// either: 17 widths (hidden 256 to 5120, 16 to 224 workgroups), 1 to 48 rows, each of the three rules switched off against all on, a layer of
// a stack: q/k/v 1.01 to 1.24 times as fast by this kernel, gate / up 0.99 to 1.07 (the shape with 10 tiles does not take it), O and down
// 1.03 to 1.24 up to 8 rows, 1.00 to 1.08 at 17 to 32, and 0.98 to 1.25 at 9 to 16, where hidden 1152 to 2048 with an mlp of 7000 to 11000
// (72 to 128 workgroups) gain nothing from it.  Against slabs throughout, no layer of 18 widths and 1 to 64 rows is slower beyond the
// spread (0.99 to 1.48 times as fast).
bool whole_qkv_pays(const GemmArgs& g) {
    return g.dtype == MASSV_BF16 && g.M <= 48 && n_total(g) / 32 <= kWholeGroups && gemm_supported(g) == MASSV_OK;
}

// O up to 32 rows (1.5B, 24 / 40 rows 52.2 -> 50.8, 58.7 -> 57.7; 7B 115.0 -> 113.7, 128.5 -> 128.8; 12B 117.7 -> 115.6, 142.5 -> 142.3),
// down up to 16 (24 rows, K = 8960 to 18944: 0.4 to 1 us slower, X is re-read for every 16 features).
bool whole_residual_pays(const GemmArgs& g) {
    const int rows = g.kid == MASSV_K_DOWN ? 16 : 32;
    return g.dtype == MASSV_BF16 && g.M <= rows && g.n[0] / 16 <= kWholeGroups && gemm_supported(g) == MASSV_OK;
}
static bool whole_eights(const GemmArgs& g) { return g.M <= 8 && g.K % 64 == 0 && g.n[0] / 8 <= kWholeGroups; }
int whole_residual_parts(const GemmArgs& g) { return g.n[0] / (whole_eights(g) ? 8 : 16); }

// Gate / up of rows * gains where the kernel above does not pay: gemm_stream_kernel with the scale.
template <int MT, int NT>
static int launch_stream_scaled(const GemmScaledDev& d, const GemmPlan& p, int kid, hipStream_t st) {
    return launch_whole_kernel<&gemm_stream_kernel<MT, NT, EPI_GATED_SCALED>>(d, p.groups, kGemmWaves * kWave,
        (size_t)kGemmWaves * ReduceGroup<MT, NT>::value * MT * kWave * sizeof(floatx4), kid, st);
}
static int launch_gated_stream(const GemmArgs& g, const RowScale& scale, hipStream_t st) {
    const GemmPlan p = gemm_plan(g);
    GemmScaledDev d;
    const int rc = fill_gemm_dev(d, g, p);
    if (rc != MASSV_OK) return rc;
    d.scale = scale;
    switch ((g.M > 16 ? 100 : 0) + p.nt) {
        case 4: return launch_stream_scaled<1, 4>(d, p, g.kid, st);
        case 8: return launch_stream_scaled<1, 8>(d, p, g.kid, st);
        case 10: return launch_stream_scaled<1, 10>(d, p, g.kid, st);
        case 104: return launch_stream_scaled<2, 4>(d, p, g.kid, st);
        case 108: return launch_stream_scaled<2, 8>(d, p, g.kid, st);
        case 110: return launch_stream_scaled<2, 10>(d, p, g.kid, st);
    }
    return MASSV_EUNSUPPORTED;
}

// Gate / up up to 16 rows and 8 tiles a workgroup: with 10 (7B shape) no more than 4 steps fit the registers, 106.7 -> 109.4 us a layer.
static int gated_tiles(const GemmArgs& g) { return (g.n[0] / 8 + kWholeGroups - 1) / kWholeGroups; }
static bool whole_gated_pays(const GemmArgs& g) { return g.M <= 16 && gated_tiles(g) <= 8; }

int launch_whole_qkv(const GemmArgs& g, const RowScale& scale, const void* raw_x, const void* gain, const int32_t* pos,
                     const int32_t* kv_len, void* q_out, void* k_cache, void* v_cache, const massv_attn_desc& a, float theta, hipStream_t st) {
    WholeQkv d = {};
    d.x = (const bf16_t*)(raw_x ? raw_x : g.x); d.M = g.M; d.K = g.K; d.scale = scale; d.gain = (const bf16_t*)gain;
    for (int s = 0; s < 3; ++s) { d.w[s] = (const bf16_t*)g.w[s]; d.bias[s] = (const bf16_t*)g.bias[s]; }
    d.pos = pos; d.kv_len = kv_len; d.q_out = (bf16_t*)q_out; d.k_cache = (bf16_t*)k_cache; d.v_cache = (bf16_t*)v_cache;
    d.Q = a.n_query; d.n_q = a.n_q_heads; d.n_kv = a.n_kv_heads; d.d = a.head_dim; d.l_max = a.l_max;
    d.log2_theta = log2((double)theta);
    const int groups = n_total(g) / 16;
    if (raw_x && g.M > 16) return MASSV_EINVAL;
    if (raw_x)
        return groups <= kWholeGroups ? launch_whole<1, 4, WHOLE_QKV8, true>(d, groups, g.kid, st) : launch_whole<1, 4, WHOLE_QKV16, true>(d, groups / 2, g.kid, st);
    if (groups <= kWholeGroups) {
        if (g.M <= 16) return launch_whole<1, 4, WHOLE_QKV8>(d, groups, g.kid, st);
        if (g.M <= 32) return launch_whole<2, 4, WHOLE_QKV8>(d, groups, g.kid, st);
        return launch_whole<3, 4, WHOLE_QKV8>(d, groups, g.kid, st);
    }
    if (g.M <= 16) return launch_whole<1, 4, WHOLE_QKV16>(d, groups / 2, g.kid, st);
    if (g.M <= 32) return launch_whole<2, 4, WHOLE_QKV16>(d, groups / 2, g.kid, st);
    return launch_whole<3, 3, WHOLE_QKV16>(d, groups / 2, g.kid, st);
}

int launch_whole_residual(const GemmArgs& g, const void* x_in, const float* h_in, void* x_out, float* h_out, const void* ln,
                          void* xn_packed, float* ss, hipStream_t st) {
    WholeRes d = {};
    d.x = (const bf16_t*)g.x; d.w = (const bf16_t*)g.w[0]; d.M = g.M; d.K = g.K; d.N = g.n[0];
    d.x_in = (const bf16_t*)x_in; d.h_in = h_in; d.x_out = (bf16_t*)x_out; d.h_out = h_out;
    d.ln = (const bf16_t*)ln; d.xn = (bf16_t*)xn_packed; d.ss_out = ss;
    // (four slots where no wave has more than four steps: a small launch mostly waits for its instructions, O of the 1.5B shape, 8 rows,
    // 5.2 -> 4.4 us; for 9 to 16 rows an instance with four slots gained 0.2 to 0.5 % of a layer, within its spread, and is left out)
    if (whole_eights(g) && g.K <= 64 * kWholeWaves * 4) return launch_whole<1, 4, WHOLE_RES8>(d, g.n[0] / 8, g.kid, st);
    if (whole_eights(g)) return launch_whole<1, 10, WHOLE_RES8>(d, g.n[0] / 8, g.kid, st);
    if (g.M <= 16) return launch_whole<1, 8, WHOLE_RES16>(d, g.n[0] / 16, g.kid, st);
    return launch_whole<2, 4, WHOLE_RES16>(d, g.n[0] / 16, g.kid, st);
}

template <int NT, int U>
static int launch_gated_as(const WholeGated& d, int groups, int kid, hipStream_t st) {
    return launch_whole_kernel<&whole_gated_kernel<NT, U>>(d, groups, kGatedThreads, (size_t)(kGatedWaves * NT * kFrag + kGatedThreads) * 4, kid, st);
}

int launch_gated(const GemmArgs& g, const RowScale& scale, hipStream_t st) {
    const int rc = gemm_supported(g);
    if (rc != MASSV_OK) return rc;
    if (scale.ss && g.M > 32) return MASSV_EINVAL;
    if (!whole_gated_pays(g)) return scale.ss ? launch_gated_stream(g, scale, st) : launch_gemm(g, st);
    WholeGated d = {};
    d.x = (const bf16_t*)g.x; d.w[0] = (const bf16_t*)g.w[0]; d.w[1] = (const bf16_t*)g.w[1]; d.M = g.M; d.K = g.K;
    const int units = g.n[0] / 8, groups = units < kWholeGroups ? units : kWholeGroups;
    d.share = units / groups; d.rem = units % groups;
    d.scale = scale; d.act = g.act; d.h = (bf16_t*)g.y;
    switch (gated_tiles(g)) {
        case 1: return launch_gated_as<1, 14>(d, groups, g.kid, st);
        case 2: return launch_gated_as<2, 12>(d, groups, g.kid, st);
        case 3: return launch_gated_as<3, 8>(d, groups, g.kid, st);
        case 4: return launch_gated_as<4, 6>(d, groups, g.kid, st);
        case 5: return launch_gated_as<5, 6>(d, groups, g.kid, st);
        case 6: return launch_gated_as<6, 5>(d, groups, g.kid, st);
        case 7: return launch_gated_as<7, 4>(d, groups, g.kid, st);
        case 8: return launch_gated_as<8, 4>(d, groups, g.kid, st);
    }
    return MASSV_EUNSUPPORTED;
}

}  // namespace massv
