// Projections of the verify forward: Y[M][N] = X[M][K] W[N][K]^T with M = B*(gamma+1)
// rows (1 .. 64; the ones of few rows that carry what follows them are in whole.hip).  At these row counts every weight byte is used for only M
// multiply-adds, far below the machine balance, so the kernels are weight
// STREAMERS: the job is to pull W through HBM once at full bandwidth; the
// matrix cores only have to keep up.
//
// bf16 kernel (gemm_stream_kernel, in gemm_stream.h), shaped by measurements on MI355X:
//   * v_mfma_f32_16x16x32_bf16 with W as the A operand (16 output features x
//     32 k) and X as the B operand (32 k x 16 rows): every lane's W operand is
//     one 16-byte global load.  W is kept in the library's streaming layout
//     (massv_weight_pack): per 16-feature tile, the operands of consecutive
//     k-steps lie back to back, so a wave's load is a contiguous 1 KB of whole
//     cache lines and a tile is one sequential stream.  That allows the
//     non-temporal hint; measured against row-major W (64-byte pieces of 16
//     rows per load) the same kernel went from 4.4 to 5.2 TB/s on the gate/up
//     shape.
//   * X comes from L2, and those reads -- not HBM -- were the first limiter.
//     Two remedies: X is kept in operand order (packed_index) so a wave reads it
//     as contiguous 1 KB blocks, and a wave owns NT = 4..10 feature tiles per
//     chunk so that each X block it loads is used NT times.
//   * Each of the wave's NT tiles has its own register slot: right after the
//     matrix instructions of tile t for chunk c have been issued, the loads of
//     tile t for the wave's next chunk go out.  This keeps about NT-1 tile
//     loads (4 KB each) in flight per wave with ONE set of W registers; X is
//     double-buffered.
//   * A workgroup is 4 waves that split its K range in interleaved chunks of
//     four 32-element steps (so the workgroup reads contiguous 16 KB runs of
//     a tile; giving each wave one contiguous quarter instead measured 1%
//     slower on the whole step) with the ragged last round dealt evenly, and
//     are summed through LDS in wave order (deterministic).
//   * The grid is sized to at most one workgroup per CU (256) wherever
//     possible: with a register-heavy streaming kernel a second partial round
//     of workgroups costs as much as a full one.  Wide outputs (gate/up,
//     lm_head) choose NT for that; narrow outputs (q/k/v, O, down) split K
//     over gridDim.y slabs, write fp32 partial sums and leave the slab sum to
//     the row-wise kernel that follows anyway (bias + rotary + cache append,
//     residual + RMSNorm).
//   * Epilogues: fp32 partial sums, act(gate)*up for interleaved gate/up tiles
//     (written in operand order for the down projection), fp32 logits.
// f32 kernels: one wave per output feature, plain FMAs, for the small fp32
// configuration.
#include "gemm_stream.h"

#include <limits.h>
#include <atomic>
#include <type_traits>

namespace massv {

// 2^(d * log2(e)/T) for d <= 0 (a logit minus a running maximum; -inf and NaN from -inf - -inf give 0).
__device__ inline float exp2_scaled(float d, float hi, float lo) {
    d = fmaxf(d, -3.0e38f);
    return __builtin_amdgcn_exp2f(fmaf(d, lo, d * hi));
}

// ---------------------------------------------------------------------------
// Vocabulary projection: the same stream, with epilogues that store fp32 logits and / or keep row statistics.
// A workgroup of the vocabulary projection works off its shares one after the other: the loads that open the next
// share go out behind the matrix instructions that close this one, so HBM stays busy through the reduction and the
// epilogue (a workgroup per share, four rounds of them, had every compute unit start each share with an empty pipe:
// 48 rows, 3584 -> 152064, whole calls: logits and accept at T > 0 250 -> 232 us, T = 0 196 -> 175, logits alone 202 ->
// 197; 64 rows, 1536 wide, 197 -> 143 at T > 0).  Neighbouring workgroups hold neighbouring shares at any time: with a
// workgroup's shares side by side instead the logits took 203 us.
// What the shares' ends cost at 48 rows, 3584 -> 152064, T = 0.7 (whole call): logits stored into L2, which gives them back when the launch ends,
// 230.9 us, written through 211.4 (non-temporal 211.1; not stored at all 200), and with the statistics' rare part (a new maximum)
// behind a branch 205.0; 24 rows, 3840 -> 262144, 365 -> 340; T = 0, where nothing is stored, 182.1 -> 178.6 by the branch.
// EPI_ARGMAX and EPI_LOGITS_STATS carry a lane's maximum (and sum) across the workgroup's shares: one record per row and
// workgroup.
// MANY: more than one share a workgroup (with the loop over shares compiled in, single ones took up to 9 % longer: 16 rows, 1024
// -> 50000 21.2 us, 19.3 without).  Plain logits of one share a workgroup and more workgroups than CUs are gemm_stream_kernel's
// (32 rows, 1024 -> 45056 19.6 us, 21.7 here; 1024 -> 8192 7.6 there and 7.5 here).
// ---------------------------------------------------------------------------
template <int MT, int NT, int EPI, bool MANY>
__global__ __launch_bounds__(kGemmWaves * kWave)
void gemm_vocab_kernel(GemmDev g) {
    constexpr int WK = kGemmWaves;
    const int shares = MANY ? g.rounds : 1;
    extern __shared__ floatx4 red[];                 // [WK][GRP*MT][64]
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int lr = lane % 16, lc = lane / 16;
    const int K = g.K;

    // ---- the NT feature tiles of this workgroup's (next) share ----
    const bf16_t* wrow[NT];
    bool nvalid[NT];
    int unit0 = 0, n_units = 0;                       // first tile and tiles of the share; shares hold NT tiles or one fewer
    auto take_share = [&](int s) {                    // tiles of share s; wrow: where their weights begin
        unit0 = s * g.unit_base + (s < g.unit_rem ? s : g.unit_rem);
        n_units = g.unit_base + (s < g.unit_rem ? 1 : 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            nvalid[nt] = nt < n_units && unit0 + nt < g.tiles[0];
            wrow[nt] = g.w[0] + (size_t)(nvalid[nt] ? unit0 + nt : 0) * (K / 32) * 512 + lane * 8;      // streaming layout
        }
    };
    take_share(blockIdx.x);
    // X in operand order: the B operand of (k-step ks, row tile mt) is the 1 KB block ((ks*MT + mt)*64 + lane)*8
    const bf16_t* xlane = g.x + (size_t)lane * 8;

    floatx4 acc[NT][MT];

    // K is dealt to the waves in 32-element MFMA steps, as in gemm_stream_kernel
    const int n_steps = K / 32, rounds = n_steps / (4 * WK);
    const int tail = n_steps - rounds * 4 * WK;
    const int tb = tail / WK, tr = tail % WK;
    const int t_len = tb + (wave < tr ? 1 : 0);                              // 0..4 steps
    const int t_k0 = rounds * 4 * WK + wave * tb + (wave < tr ? wave : tr);
    const int n_it = rounds + (t_len > 0 ? 1 : 0);
    auto k0_of = [&](int it) { return it < rounds ? (it * WK + wave) * 4 : t_k0; };
    auto cnt_of = [&](int it) { return it < rounds ? 4 : t_len; };

    bf16x8 a[NT][4];
    bf16x8 xb[2][MT][4];
    auto wload = [&](int nt, int k0, int cnt) {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[nt][j] = ld8_stream(wrow[nt] + (size_t)(k0 + j) * 512, nvalid[nt] && j < cnt);
    };
    auto xload = [&](int buf, int k0, int cnt) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                xb[buf][mt][j] = ld8(xlane + (size_t)((k0 + j) * MT + mt) * 512, j < cnt);
    };
    if (n_it > 0) {
        xload(0, k0_of(0), cnt_of(0));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wload(nt, k0_of(0), cnt_of(0));
    }
    // EPI_ARGMAX, EPI_LOGITS_STATS: largest summed output (and its lowest column) seen by this lane for row
    // 16 mt + lr; EPI_LOGITS_STATS: also the sum of exp((x - largest)/T) over what the lane has seen (rescaled
    // whenever the largest moves): four terms at a time in fp32, the rest in double, over all of the workgroup's shares.
    constexpr bool STATS = (EPI == EPI_LOGITS_STATS);
    float best_v[MT];
    double sum_e[MT];
    int best_i[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) { best_v[mt] = -INFINITY; best_i[mt] = INT_MAX; sum_e[mt] = 0.0; }

    // Logits of more than 16 rows are written through L2 (store_through); fewer rows stay there for the accept rule, which reads them next (6 rows of
    // 152064 191 us either way, one row 88.4 and 89.3 us a call).  The line is drawn by rows, not by bytes, as few logits lose nothing: 4096 to 32000 of 17 to 64
    // rows (512 to 5120 wide, 500 calls) are 0.96 to 1.07 times as fast written through as cached, medians 1.00 to 1.02, 65536 1.01 to 1.03, 152064 1.03.  Plain
    // logits of 17 to 32 rows, one share a workgroup, stay in L2: written through, 12000 to 40000 of them were 0.976 to 0.99 times as fast in the medians (4096 1.007).
    auto put_logits = [&](int m, int col, floatx4 v) {
        floatx4* dst = reinterpret_cast<floatx4*>((float*)g.y + (size_t)m * g.ldy + col);
        if constexpr (MT > 2 || (MT > 1 && (MANY || STATS))) store_through(dst, v);
        else *dst = v;
    };
    // Barrier for what travels through LDS; loads on their way into registers stay on their way.
    auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    int par = 0;
    for (int round = 0; round < shares; ++round) {
        const int first = unit0, owned = n_units < g.tiles[0] - unit0 ? n_units : g.tiles[0] - unit0;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int it = 0; it < n_it; ++it, par ^= 1) {
            bool more = it + 1 < n_it;
            int nx = k0_of(it + 1), ncnt = cnt_of(it + 1);
            if (MANY && !more && round + 1 < shares) {
                take_share((round + 1) * gridDim.x + blockIdx.x);
                more = true; nx = k0_of(0); ncnt = cnt_of(0);
            }
            if (more) { if (par) xload(0, nx, ncnt); else xload(1, nx, ncnt); }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[nt][j], par ? xb[1][mt][j] : xb[0][mt][j],
                                                                             acc[nt][mt], 0, 0, 0);
                if (more) wload(nt, nx, ncnt);            // refill this tile's slot for the wave's next four steps
            }
        }
        if (MANY && n_it == 0 && round + 1 < shares) take_share((round + 1) * gridDim.x + blockIdx.x);      // a wave without a step (tiny K)

        // ---- sum the waves through LDS in wave order, GRP tiles per round ----
        constexpr int GRP = ReduceGroup<MT, NT>::value;
        for (int g0 = 0; g0 < NT; g0 += GRP) {
            if (g0 || (MANY && round)) lds_barrier();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (nt >= g0 && nt < g0 + GRP)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        red[(wave * GRP * MT + (nt - g0) * MT + mt) * kWave + lane] = acc[nt][mt];
            lds_barrier();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (nt < g0 || nt >= g0 + GRP) continue;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int f = (nt - g0) * MT + mt;
                    if (f % WK != wave || nt >= owned) continue;     // fragments are dealt round-robin to the waves
                    floatx4 s = red[f * kWave + lane];
                    for (int w = 1; w < WK; ++w) s += red[(w * GRP * MT + f) * kWave + lane];
                    const int m = mt * 16 + lr;
                    const int col = (first + nt) * 16 + lc * 4;      // 4 consecutive output features
                    if (EPI == EPI_ARGMAX || STATS) {
                        // (a lane's columns ascend: a tie keeps the lower one; a row of -inf alone gets its first column)
                        const float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
                        if (mx > best_v[mt] || (mx == best_v[mt] && best_i[mt] == INT_MAX)) {
                            if constexpr (STATS)
                                if (mx > best_v[mt]) sum_e[mt] *= (double)exp2_scaled(best_v[mt] - mx, g.ts_hi, g.ts_lo);
                            best_v[mt] = mx;
                            best_i[mt] = col + (s[0] == mx ? 0 : s[1] == mx ? 1 : s[2] == mx ? 2 : 3);
                        }
                        if constexpr (STATS) {
                            float four = 0.f;
#pragma unroll
                            for (int i = 0; i < 4; ++i) four += exp2_scaled(s[i] - best_v[mt], g.ts_hi, g.ts_lo);
                            sum_e[mt] += (double)four;
                        }
                        if (STATS && m < g.M) put_logits(m, col, s);
                    } else if (m < g.M) {
                        put_logits(m, col, s);
                    }
                }
            }
        }
    }
    if constexpr (EPI == EPI_ARGMAX || STATS) {
        // lanes of the four column groups of a row, then the four waves, then one record per row and workgroup
        lds_barrier();                                           // the reduction buffer is free
        float* bv = reinterpret_cast<float*>(red);               // [WK][MT*16]
        int* bi = reinterpret_cast<int*>(bv + WK * MT * 16);
        double* bs = reinterpret_cast<double*>(bi + WK * MT * 16);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float v = best_v[mt]; double se = sum_e[mt]; int i = best_i[mt];
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(v, o, kWave);
                const int oi = __shfl_xor(i, o, kWave);
                if constexpr (STATS) {
                    const double os = __shfl_xor(se, o, kWave);
                    const float mn = fmaxf(v, ov);
                    se = (mn == -INFINITY) ? 0.0 : se * (double)exp2_scaled(v - mn, g.ts_hi, g.ts_lo) + os * (double)exp2_scaled(ov - mn, g.ts_hi, g.ts_lo);
                }
                if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
            }
            if (lc == 0) { bv[wave * MT * 16 + mt * 16 + lr] = v; bi[wave * MT * 16 + mt * 16 + lr] = i; bs[wave * MT * 16 + mt * 16 + lr] = se; }
        }
        lds_barrier();
        if (tid < MT * 16 && tid < g.M) {
            float v = bv[tid]; int i = bi[tid];
            for (int w = 1; w < WK; ++w) {
                const float ov = bv[w * MT * 16 + tid]; const int oi = bi[w * MT * 16 + tid];
                if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
            }
            RowPartial r; r.m = v; r.arg = i; r.s = 0.0;
            if constexpr (STATS) {                               // wave order, in double
                for (int w = 0; w < WK; ++w)
                    if (bv[w * MT * 16 + tid] > -INFINITY)
                        r.s += bs[w * MT * 16 + tid] * (double)exp2_scaled(bv[w * MT * 16 + tid] - v, g.ts_hi, g.ts_lo);
            }
            reinterpret_cast<RowPartial*>(STATS ? g.stats : g.y)[(size_t)tid * gridDim.x + blockIdx.x] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// f32 kernels, for the small fp32 configuration: a few hundred features and rows, so a launch is its own latency (2.7 us
// empty) plus one trip to memory, and what counts is how many launches and how many dependent trips a layer makes.
// grid (outputs, ceil(M / 8)), one wave per output feature (or pair of features) and 8 rows; the lanes share K, 16 bytes
// a lane and load, four steps of loads in flight.  What precedes and follows a projection is done by the same wave: the
// RMSNorm of its rows (it reads them whole anyway), and the activation of a gate / up pair or the rotation and append of
// a (j, j + d/2) pair, each computed as two features of one wave.  2 x 6 rows of the 256-wide configuration: 13 launches
// and 110 us a layer before (3 + 2 projection launches, two norms, activation, rotation), see layer.hip for the rest.  A launch this
// short also waits for its own instructions: with the row sums formed eight at a time (wave_sum8), 100 instructions fewer, q/k/v
// takes 4.9 us instead of 7.1, gate / up 4.1 instead of 6.5, O and down 3.7 instead of 4.6.
// ---------------------------------------------------------------------------
constexpr int kF32Rows = 8;

template <int VEC> struct FVec { typedef floatx4_any type; };
template <> struct FVec<1> { typedef float type; };
__device__ inline float dot_step(float a, float b, float c) { return fmaf(a, b, c); }
__device__ inline float dot_step(floatx4_any a, floatx4_any b, float c) { return fmaf(a[3], b[3], fmaf(a[2], b[2], fmaf(a[1], b[1], fmaf(a[0], b[0], c)))); }
template <typename V> __device__ inline V scale_by(V a, V b) { return a * b; }

// acc[i][r] = sum_k w[i][k] g[k] x[m0 + r][k] / rms(x[m0 + r]) (NORM), or without g and rms.  Eight rows: lane l gets
// the sums of row l % 8, in acc[i][0]; fewer: every lane gets all of them.
// Rows past M repeat the last one.  K % VEC == 0.
template <int VEC, int NW, bool NORM, int R>
__device__ inline void rows_dot(const float* __restrict__ x, const float* const (&w)[NW], const float* __restrict__ g, float eps,
                                int m0, int M, int K, float (&acc)[NW][R]) {
    typedef typename FVec<VEC>::type V;
    const int lane = threadIdx.x, kv = K / VEC;
    const V* xr[R];
    float ss[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        xr[r] = reinterpret_cast<const V*>(x + (size_t)(m0 + r < M ? m0 + r : M - 1) * K);
        ss[r] = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[i][r] = 0.f;
    }
    // S steps of kWave groups with all their loads in flight: four at a time, then what is left (four
    // every time, zeros past K: 48 x 64 -> 4096 51 us, 15 without them)
    auto steps = [&](int k0, auto count) {
        constexpr int S = decltype(count)::value;
        V xv[S][R], wv[S][NW], gv[S];
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int k = k0 + u * kWave + lane;
            const bool ok = k < kv;
#pragma unroll
            for (int i = 0; i < NW; ++i) wv[u][i] = ok ? reinterpret_cast<const V*>(w[i])[k] : V{};
            if constexpr (NORM) gv[u] = ok ? reinterpret_cast<const V*>(g)[k] : V{};
#pragma unroll
            for (int r = 0; r < R; ++r) xv[u][r] = ok ? xr[r][k] : V{};
        }
#pragma unroll
        for (int u = 0; u < S; ++u) {
            if constexpr (NORM) {
#pragma unroll
                for (int i = 0; i < NW; ++i) wv[u][i] = scale_by(wv[u][i], gv[u]);
#pragma unroll
                for (int r = 0; r < R; ++r) ss[r] = dot_step(xv[u][r], xv[u][r], ss[r]);
            }
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int r = 0; r < R; ++r) acc[i][r] = dot_step(wv[u][i], xv[u][r], acc[i][r]);
        }
    };
    int k0 = 0;
    for (; k0 + 3 * kWave < kv; k0 += 4 * kWave) steps(k0, std::integral_constant<int, 4>{});
    if (k0 + 2 * kWave < kv) steps(k0, std::integral_constant<int, 3>{});
    else if (k0 + kWave < kv) steps(k0, std::integral_constant<int, 2>{});
    else if (k0 < kv) steps(k0, std::integral_constant<int, 1>{});
    if constexpr (R == kF32Rows) {                           // lane l: row l % 8
        float rstd = 1.f;
        if constexpr (NORM) rstd = 1.0f / sqrtf(wave_sum8(ss) / (float)K + eps);
#pragma unroll
        for (int i = 0; i < NW; ++i) acc[i][0] = wave_sum8(acc[i]) * rstd;
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float rstd = 1.f;
            if constexpr (NORM) rstd = 1.0f / sqrtf(wave_sum(ss[r]) / (float)K + eps);
#pragma unroll
            for (int i = 0; i < NW; ++i) acc[i][r] = wave_sum(acc[i][r]) * rstd;
        }
    }
}

// One feature per wave and R rows: y = x w^T (+ bias) (+ residual); up to three matrices side by side.
struct F32Mats { const float* w[3]; const float* bias[3]; int n[3]; };
template <int VEC, bool NORM, int R>
__global__ __launch_bounds__(kWave)
void gemm_f32_kernel(const float* __restrict__ x, const float* __restrict__ g, float eps, F32Mats mats, const float* residual,
                     float* y, int M, int K, int ldy) {
    const int n = blockIdx.x, m0 = blockIdx.y * R, lane = threadIdx.x;
    int seg = 0, local = n;
    if (local >= mats.n[0]) { local -= mats.n[0]; seg = 1; if (local >= mats.n[1]) { local -= mats.n[1]; seg = 2; } }
    const float* const w[1] = {mats.w[seg] + (size_t)local * K};
    float acc[1][R];
    rows_dot<VEC, 1, NORM, R>(x, w, g, eps, m0, M, K, acc);
    const float b = mats.bias[seg] ? mats.bias[seg][local] : 0.f;
    if constexpr (R == kF32Rows) {
        if (lane < R && m0 + lane < M) {
            const size_t o = (size_t)(m0 + lane) * ldy + n;
            y[o] = acc[0][0] + b + (residual ? residual[o] : 0.f);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (lane == r && m0 + r < M) {
                const size_t o = (size_t)(m0 + r) * ldy + n;
                y[o] = acc[0][r] + b + (residual ? residual[o] : 0.f);
            }
    }
}

// act(gate) * up: feature f of both matrices.
template <int VEC, bool NORM>
__global__ __launch_bounds__(kWave)
void gated_f32_kernel(const float* __restrict__ x, const float* __restrict__ g, float eps, const float* __restrict__ wg,
                      const float* __restrict__ wu, float* __restrict__ h, int M, int K, int F, int act) {
    const int f = blockIdx.x, m0 = blockIdx.y * kF32Rows, lane = threadIdx.x;
    const float* const w[2] = {wg + (size_t)f * K, wu + (size_t)f * K};
    float acc[2][kF32Rows];
    rows_dot<VEC, 2, NORM, kF32Rows>(x, w, g, eps, m0, M, K, acc);
    const float gv = acc[0][0], uv = acc[1][0];
    if (lane >= kF32Rows || m0 + lane >= M) return;
    float a;
    if (act == MASSV_ACT_SILU) a = gv / (1.0f + expf(-gv));
    else a = 0.5f * gv * (1.0f + tanhf(0.7978845608028654f * (gv + 0.044715f * gv * gv * gv)));
    h[(size_t)(m0 + lane) * F + f] = a * uv;
}

// Query, key and value projections with the rotation and the cache append: features j and j + d/2 of one head.
// grid (heads * d / 2, ceil(M / 8)); angles and rotation in double, as rope_append_kernel does them.
template <int VEC>
__global__ __launch_bounds__(kWave)
void qkv_rope_f32_kernel(const float* __restrict__ x, const float* __restrict__ g, float eps, F32Mats mats,
                         const int32_t* __restrict__ pos, const int32_t* __restrict__ kv_len, float* __restrict__ q_out,
                         float* __restrict__ k_cache, float* __restrict__ v_cache, int M, int K, int Q, int n_q, int n_kv,
                         int d, int l_max, double log2_theta) {
    const int half = d / 2, head = blockIdx.x / half, j = blockIdx.x % half;
    const int m0 = blockIdx.y * kF32Rows, lane = threadIdx.x;
    const int seg = head < n_q ? 0 : head < n_q + n_kv ? 1 : 2;
    const int hl = seg == 0 ? head : seg == 1 ? head - n_q : head - n_q - n_kv;
    const size_t row0 = (size_t)hl * d + j;
    const float* const w[2] = {mats.w[seg] + row0 * K, mats.w[seg] + (row0 + half) * K};
    // what the lane's row needs besides the products does not wait for them
    const int m = m0 + lane;
    const bool live = lane < kF32Rows && m < M;
    const int b = live ? m / Q : 0, i = live ? m % Q : 0;
    const int cached = kv_len[b];
    const float b1 = mats.bias[seg] ? mats.bias[seg][row0] : 0.f, b2 = mats.bias[seg] ? mats.bias[seg][row0 + half] : 0.f;
    double sn = 0.0, cs = 1.0;
    if (seg < 2) {
        const double ang = (double)pos[live ? m : 0] * exp2(-2.0 * (double)j / (double)d * log2_theta);
        sincos(ang, &sn, &cs);
    }
    float acc[2][kF32Rows];
    rows_dot<VEC, 2, true, kF32Rows>(x, w, g, eps, m0, M, K, acc);
    if (!live) return;
    const float x1 = acc[0][0] + b1, x2 = acc[1][0] + b2;
    const int row = cached_rows(cached, l_max) + i;
    if (seg < 2) {
        const float y1 = (float)((double)x1 * cs - (double)x2 * sn);
        const float y2 = (float)((double)x2 * cs + (double)x1 * sn);
        if (seg == 0) {
            float* dst = q_out + ((size_t)m * n_q + hl) * d;
            dst[j] = y1; dst[j + half] = y2;
        } else if (row < l_max) {
            float* dst = k_cache + (((size_t)b * n_kv + hl) * l_max + row) * d;
            dst[j] = y1; dst[j + half] = y2;
        }
    } else if (row < l_max) {
        const size_t blk = ((size_t)b * n_kv + hl) * (l_max / MASSV_V_BLOCK) + row / MASSV_V_BLOCK;
        float* dst = v_cache + blk * d * MASSV_V_BLOCK + row % MASSV_V_BLOCK;
        dst[(size_t)j * MASSV_V_BLOCK] = x1; dst[(size_t)(j + half) * MASSV_V_BLOCK] = x2;
    }
}

// 16-byte loads need K in whole groups of four (rows may start at any float: which loads are used, and with them the order of
// the sums, depends on K alone).  Under 256 values a row they leave lanes without work: 64 -> 4096 at 64 rows 18 us with single
// values, 29 with 16 bytes; 128 -> 152064 at 8 rows 71 and 133.
static bool f32_wide(int K) { return K % 4 == 0 && K >= 4 * kWave; }

int launch_qkv_rope_f32(const GemmArgs& g, const int32_t* pos, const int32_t* kv_len, void* q_out, void* k_cache, void* v_cache,
                        const massv_attn_desc& a, float theta, hipStream_t st) {
    F32Mats mats;
    for (int s = 0; s < 3; ++s) { mats.w[s] = (const float*)g.w[s]; mats.bias[s] = (const float*)g.bias[s]; mats.n[s] = g.n[s]; }
    const dim3 grid((a.n_q_heads + 2 * a.n_kv_heads) * (a.head_dim / 2), (g.M + kF32Rows - 1) / kF32Rows);
    const auto kernel = f32_wide(g.K) ? qkv_rope_f32_kernel<4> : qkv_rope_f32_kernel<1>;
    hipLaunchKernelGGL(kernel, grid, dim3(kWave), 0, st, (const float*)g.x, (const float*)g.norm, g.norm_eps, mats, pos, kv_len,
                  (float*)q_out, (float*)k_cache, (float*)v_cache, g.M, g.K, a.n_query, a.n_q_heads, a.n_kv_heads, a.head_dim,
                  a.l_max, log2((double)theta));
    return launch_status();
}

template <int R>
static auto gemm_f32_pick(bool norm, bool wide) {
    return norm ? (wide ? gemm_f32_kernel<4, true, R> : gemm_f32_kernel<1, true, R>) : (wide ? gemm_f32_kernel<4, false, R> : gemm_f32_kernel<1, false, R>);
}

static int launch_gemm_f32(const GemmArgs& g, hipStream_t st) {
    F32Mats mats;
    for (int s = 0; s < 3; ++s) { mats.w[s] = (const float*)g.w[s]; mats.bias[s] = (const float*)g.bias[s]; mats.n[s] = g.n[s]; }
    const bool wide = f32_wide(g.K);
    const unsigned row_groups = (g.M + kF32Rows - 1) / kF32Rows;
    const float *x = (const float*)g.x, *gain = (const float*)g.norm;
    if (g.epilogue == EPI_GATED) {
        const auto kernel = gain ? (wide ? gated_f32_kernel<4, true> : gated_f32_kernel<1, true>)
                                 : (wide ? gated_f32_kernel<4, false> : gated_f32_kernel<1, false>);
        hipLaunchKernelGGL(kernel, dim3(g.n[0], row_groups), dim3(kWave), 0, st, x, gain, g.norm_eps, mats.w[0], mats.w[1],
                      (float*)g.y, g.M, g.K, g.n[0], g.act);
        return launch_status();
    }
    const int N = g.n[0] + g.n[1] + g.n[2];
    const float* res = g.epilogue == EPI_RESIDUAL ? (const float*)g.residual : nullptr;
    // few rows: a wave does not multiply rows that are not there (1 x 256 -> 152064 34 us, 81 as one of 8 rows)
    const auto kernel = g.M == 1 ? gemm_f32_pick<1>(gain, wide) : g.M == 2 ? gemm_f32_pick<2>(gain, wide) : g.M <= 4 ? gemm_f32_pick<4>(gain, wide) : gemm_f32_pick<8>(gain, wide);
    hipLaunchKernelGGL(kernel, dim3(N, row_groups), dim3(kWave), 0, st, x, gain, g.norm_eps, mats, res, (float*)g.y, g.M, g.K, N);
    return launch_status();
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int n_total(const GemmArgs& g) { return g.n[0] + g.n[1] + g.n[2]; }

int gemm_supported(const GemmArgs& g) {
    if (g.M < 1 || g.K < 1 || g.n[0] < 1) return MASSV_EINVAL;
    if (g.epilogue == EPI_GATED && (g.n[1] != g.n[0] || g.n[2] != 0)) return MASSV_EINVAL;
    if (g.dtype == MASSV_F32)
        return (g.epilogue == EPI_PARTIAL || g.epilogue == EPI_ARGMAX || g.epilogue == EPI_LOGITS_STATS) ? MASSV_EINVAL : MASSV_OK;
    if (g.epilogue == EPI_LOGITS_STATS && (!g.stats || !(g.temperature > 0.f))) return MASSV_EINVAL;
    if (g.epilogue == EPI_STORE || g.epilogue == EPI_RESIDUAL) return MASSV_EINVAL;   // bf16 goes through partial sums
    if (g.M > MASSV_MAX_ROWS) return MASSV_EUNSUPPORTED;
    if (g.K % 32) return MASSV_EUNSUPPORTED;
    for (int s = 0; s < 3; ++s)
        if (g.n[s] % 16) return MASSV_EUNSUPPORTED;
    return MASSV_OK;
}

// Narrow outputs (fewer than 256 workgroups at full K): K is cut into slabs and the slab sums are left to the
// row-wise kernel that follows.  Tiles per wave and slabs are chosen by an estimate of the launch plus its share of
// that kernel, in microseconds, fitted to sweeps of the three split projections of the 7B-shaped layer (M = 48):
//   weights at 6.5 TB/s, stretched when fewer than 256 workgroups pull them;
//   X, re-read from L2 once per workgroup column: (T / nt) * K/32 * MT KB, at 14 TB/s;
//   0.8 us per MB of partial sums (written here, read back by the next kernel).  Of more than 16 rows they are written through L2
//   (store_through): 48-row layer 126.0 -> 125.3 us (128.2 -> 126.0 on another card), 28 rows of a drafter 1538 -> 1528; of 6 and 10 rows 100.1 and 110.5 us cached,
//   100.2 and 110.9 through.  Whole layers of 17 to 64 rows, 256 to 5120 wide, 300 calls: 0.98 to 1.02 times as fast as with cached sums, medians by width and rows 0.99
//   (256 wide, 64 rows) to 1.015; narrow ones, whose few hundred KB are read back at once, lose nothing either.
// Measured against the earlier rule "as many slabs as fill 256 workgroups, largest tile count": q/k/v (8 tiles, 7
// slabs) -> (4, 3) -1.9 us, output projection (7, 7) -> (4, 4) -1.0 us, down projection (7, 8) unchanged.
static GemmPlan plan_split(const GemmArgs& g, int mt, int T) {
    GemmPlan best = {0, 1, 0};
    const int n_steps = g.K / 32;
    int max_slabs = n_steps / kGemmWaves; if (max_slabs < 1) max_slabs = 1; if (max_slabs > 32) max_slabs = 32;   // a step per wave at least
    const double w_us = (double)n_total(g) * g.K * 2.0 / 6.5e6;
    const double slab_us = (double)(mt * 16) * n_total(g) * 4.0 / 1e6 * 0.8;
    static const int cand[] = {8, 7, 4};
    double best_t = 1e30;
    for (int nt : cand) {
        if (mt == 4 && nt > 4) continue;                       // register budget of four row tiles
        const int groups = (T + nt - 1) / nt;
        if (groups >= kCUs) continue;
        const double x_us = (double)groups * n_steps * mt * 1024.0 / 1e6 * 0.07;
        for (int slabs = 1; slabs <= max_slabs && groups * slabs <= kCUs; ++slabs) {
            const double t = w_us * (1.0 + 0.44 * ((double)kCUs / (groups * slabs) - 1.0)) + x_us + slabs * slab_us;
            if (t < best_t) { best_t = t; best.nt = nt; best.slabs = slabs; best.groups = groups; }
        }
    }
    return best;
}

// Tiles per wave and K slabs for one launch.  T: 16-feature tiles to produce.
//   wide output  (>= 256 groups): slabs = 1, NT chosen so that the last round of workgroups is as full as possible;
//   narrow output with the partial-sum epilogue: plan_split; the kernel deals the K/32 steps evenly over the slabs.
GemmPlan gemm_plan(const GemmArgs& g) {
    GemmPlan best = {0, 1, 0};
    if (g.dtype != MASSV_BF16) return best;
    const int mt = (g.M + 15) / 16;
    const int T = (g.epilogue == EPI_GATED) ? 2 * (g.n[0] / 16) : n_total(g) / 16;
    if (g.epilogue == EPI_PARTIAL && (T + 3) / 4 < kCUs) return plan_split(g, mt, T);
    // wide output (or a partial-sum output wide enough for 256 workgroups at full K): one slab
    static const int cand_partial[] = {8, 7, 4}, cand_gated[] = {10, 8, 4}, cand_logits[] = {10, 8, 4};
    const int* cand = g.epilogue == EPI_GATED ? cand_gated : (g.epilogue == EPI_LOGITS || g.epilogue == EPI_ARGMAX || g.epilogue == EPI_LOGITS_STATS) ? cand_logits : cand_partial;
    double best_score = -1.0;
    for (int i = 0; i < 3; ++i) {
        int nt = cand[i];
        if (mt == 4 && nt > 4) continue;                       // register budget of four row tiles
        const int ut = (g.epilogue == EPI_GATED) ? 2 : 1;      // tiles per unit
        int groups = (T + nt - 1) / nt;
        if (groups < kCUs) {                                    // one round: spread the units over as many CUs as there are
            const int units = T / ut;                           // (never a partial-sum launch: those went to plan_split)
            groups = units < kCUs ? units : kCUs;
        }
        const int rounds = (groups + kCUs - 1) / kCUs;
        if (rounds > 1 && rounds * kCUs <= T / ut) groups = rounds * kCUs;     // full rounds: the units are dealt evenly over them
        const double eff = (double)T / ((double)nt * rounds * kCUs);
        const double score = eff + 0.004 * nt;                 // near ties go to the larger tile count (less X traffic)
        if (score > best_score) { best_score = score; best.nt = nt; best.slabs = 1; best.groups = groups; }
    }
    return best;
}

constexpr bool is_vocab(int epi) { return epi == EPI_LOGITS || epi == EPI_ARGMAX || epi == EPI_LOGITS_STATS; }

// Shares that one workgroup of the vocabulary projection works off: all rounds of one workgroup per CU, where they are
// full.  Plain logits of few rows stay a workgroup per share where two such workgroups fit a CU and cover each other (16 rows
// and 8 tile slots, 32 and 4), or where the shares leave slots empty and so have less to cover.  Measured, a workgroup per
// share and one per CU: 16 rows, 8 slots, 1024 -> 45056 17.0 and 18.3 us, 2048 -> 65536 43.2 and 43.9, 640 -> 262144 63.1 and
// 63.6; 10 slots, 8.1 tiles, 1536 -> 100000 52.2 and 53.7, 8.5 tiles, 1536 -> 70000 39.0 and 37.5, 9.3, 1536 -> 152064 83.0 and
// 79.6; 32 rows, 4 slots, 2048 -> 49152 37.3 and 39.3, 8.1 of 10 tiles, 5120 -> 100352 181 and 184, 6.1 of 8, 1024 -> 50000
// 24.7 and 22.2, 7.5 of 8, 2048 -> 92544 72.4 and 68.3; from 33 rows on one per CU gains 3 to 33 %.
static int gemm_rounds(const GemmPlan& p, const GemmArgs& g) {
    if (!is_vocab(g.epilogue)) return 1;
    if (p.groups <= kCUs || p.groups % kCUs) return 1;
    if (g.epilogue == EPI_LOGITS && g.M <= 32) {
        const bool filled = g.n[0] / 16 >= 0.84 * p.groups * p.nt;
        if (g.M <= 16 ? !(p.nt == 10 && filled) : p.nt == 4 || !(filled || g.K <= 1024)) return 1;
    }
    return p.groups / kCUs;
}

int gemm_row_pieces(const GemmArgs& g) {
    const GemmPlan p = gemm_plan(g);
    return p.groups / gemm_rounds(p, g);
}

size_t gemm_partial_bytes(const GemmArgs& g) {
    if (g.dtype != MASSV_BF16 || g.epilogue != EPI_PARTIAL) return 0;
    const GemmPlan p = gemm_plan(g);
    return (size_t)p.slabs * ((g.M + 15) / 16 * 16) * n_total(g) * sizeof(float);
}

enum StreamKind { STREAM, VOCAB_ONE, VOCAB_MANY };
template <int MT, int NT, int EPI, int KIND>
static constexpr auto stream_kernel() {
    if constexpr (KIND == STREAM) return &gemm_stream_kernel<MT, NT, EPI>;
    else return &gemm_vocab_kernel<MT, NT, EPI, KIND == VOCAB_MANY>;
}

template <int MT, int NT, int EPI, int KIND>
static int launch_stream_as(const GemmDev& d, const GemmPlan& p, int kid, hipStream_t st) {
    constexpr int GRP = ReduceGroup<MT, NT>::value;
    const size_t lds = (size_t)kGemmWaves * GRP * MT * kWave * sizeof(floatx4);
    if (lds > 48 * 1024) {                       // more dynamic LDS than a kernel may use by default
        static std::atomic<bool> ready[64];       // zero-initialised; calls may come from several threads
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MASSV_ELAUNCH;
        if (!ready[dev].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute((const void*)stream_kernel<MT, NT, EPI, KIND>(), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds) != hipSuccess) return MASSV_ELAUNCH;
            ready[dev].store(true, std::memory_order_release);
        }
    }
    const dim3 grid = (EPI == EPI_PARTIAL) ? dim3(p.slabs, p.groups) : dim3(p.groups / d.rounds, p.slabs);
    launch_traced(kid, stream_kernel<MT, NT, EPI, KIND>(), grid, dim3(kGemmWaves * kWave), lds, st, d);
    return MASSV_OK;
}

template <int MT, int NT, int EPI>
static int launch_stream(const GemmDev& d, const GemmPlan& p, int kid, hipStream_t st) {
    if constexpr (is_vocab(EPI)) {
        if (d.rounds > 1) return launch_stream_as<MT, NT, EPI, VOCAB_MANY>(d, p, kid, st);
        if (EPI != EPI_LOGITS || p.groups <= kCUs) return launch_stream_as<MT, NT, EPI, VOCAB_ONE>(d, p, kid, st);
    }
    if constexpr (!is_vocab(EPI) || EPI == EPI_LOGITS) return launch_stream_as<MT, NT, EPI, STREAM>(d, p, kid, st);
    return MASSV_EUNSUPPORTED;                    // (not reached)
}

template <int MT, int EPI>
static int launch_stream_nt(const GemmDev& d, const GemmPlan& p, int kid, hipStream_t st) {
    switch (p.nt) {
        case 4: return launch_stream<MT, 4, EPI>(d, p, kid, st);
        case 7: if constexpr (EPI == EPI_PARTIAL && MT <= 3) return launch_stream<MT, 7, EPI>(d, p, kid, st); break;
        case 8: if constexpr (MT <= 3) return launch_stream<MT, 8, EPI>(d, p, kid, st); break;
        case 10: if constexpr (EPI != EPI_PARTIAL && MT <= 3) return launch_stream<MT, 10, EPI>(d, p, kid, st); break;
    }
    return MASSV_EUNSUPPORTED;
}

template <int EPI>
static int launch_stream_epi(const GemmDev& d, int M, const GemmPlan& p, int kid, hipStream_t st) {
    switch ((M + 15) / 16) {
        case 1: return launch_stream_nt<1, EPI>(d, p, kid, st);
        case 2: return launch_stream_nt<2, EPI>(d, p, kid, st);
        case 3: return launch_stream_nt<3, EPI>(d, p, kid, st);
        case 4: return launch_stream_nt<4, EPI>(d, p, kid, st);
    }
    return MASSV_EUNSUPPORTED;
}

int fill_gemm_dev(GemmDev& d, const GemmArgs& g, const GemmPlan& p) {
    const int N = n_total(g);
    d.x = (const bf16_t*)g.x;
    for (int s = 0; s < 3; ++s) { d.w[s] = (const bf16_t*)g.w[s]; d.tiles[s] = g.n[s] / 16; }
    d.y = g.y;
    d.stats = g.stats;
    d.ts_hi = 1.f; d.ts_lo = 0.f;
    if (g.epilogue == EPI_LOGITS_STATS) { const TempScale ts = temp_scale(g.temperature); d.ts_hi = ts.hi; d.ts_lo = ts.lo; }
    d.M = g.M; d.K = g.K;
    d.ldy = (g.epilogue == EPI_GATED) ? g.n[0] : N;
    d.act = g.act;
    const int ut = (g.epilogue == EPI_GATED) ? 2 : 1;
    const int units = ((g.epilogue == EPI_GATED) ? 2 * d.tiles[0] : N / 16) / ut;
    d.rounds = gemm_rounds(p, g);
    d.unit_base = units / p.groups;
    d.unit_rem = units % p.groups;
    d.slab_stride = (size_t)((g.M + 15) / 16 * 16) * N;
    return (d.unit_base + (d.unit_rem ? 1 : 0)) * ut > p.nt ? MASSV_EUNSUPPORTED : MASSV_OK;      // (always fits with gemm_plan's groups)
}

int launch_gemm(const GemmArgs& g, hipStream_t st) {
    const int rc = gemm_supported(g);
    if (rc != MASSV_OK) return rc;
    if (g.dtype == MASSV_F32) return launch_gemm_f32(g, st);
    const GemmPlan p = gemm_plan(g);
    GemmDev d;
    int rc2 = fill_gemm_dev(d, g, p);
    if (rc2 != MASSV_OK) return rc2;
    rc2 = MASSV_EUNSUPPORTED;
    switch (g.epilogue) {
        case EPI_PARTIAL: rc2 = launch_stream_epi<EPI_PARTIAL>(d, g.M, p, g.kid, st); break;
        case EPI_GATED: rc2 = launch_stream_epi<EPI_GATED>(d, g.M, p, g.kid, st); break;
        case EPI_LOGITS: rc2 = launch_stream_epi<EPI_LOGITS>(d, g.M, p, g.kid, st); break;
        case EPI_ARGMAX: rc2 = launch_stream_epi<EPI_ARGMAX>(d, g.M, p, g.kid, st); break;
        case EPI_LOGITS_STATS: rc2 = launch_stream_epi<EPI_LOGITS_STATS>(d, g.M, p, g.kid, st); break;
    }
    if (rc2 != MASSV_OK) return rc2;
    return launch_status();
}

}  // namespace massv
