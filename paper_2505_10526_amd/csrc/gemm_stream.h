// gemm_stream_kernel, the bf16 weight stream of gemm.hip (which describes it), as a template that two code objects instantiate: its
// plain epilogues in gemm.hip, EPI_GATED_SCALED in whole.hip (with both in one object the plain kernels moved and the 12B shape's
// q/k/v launch took 15.1 us instead of 14.75).
#pragma once

#include "kernels.h"

namespace massv {

constexpr int kGemmWaves = 4;            // waves per workgroup (K split)
constexpr int kCUs = 256;

struct GemmDev {
    const bf16_t* x;
    const bf16_t* w[3];
    int tiles[3];            // 16-feature tiles per matrix
    void* y;
    void* stats;             // EPI_LOGITS_STATS: RowPartial[M][gridDim.x]
    float ts_hi, ts_lo;      // EPI_LOGITS_STATS: log2(e)/T in two floats
    int M, K, ldy;           // ldy: elements per output row
    int act;
    int unit_base, unit_rem; // balanced split of the tile units over gridDim.x * rounds shares: the first unit_rem own unit_base+1
    int rounds;              // vocabulary projection: shares a workgroup works off one after the other
    size_t slab_stride;      // elements between the partial sums of consecutive K slabs
};
int fill_gemm_dev(GemmDev& d, const GemmArgs& g, const GemmPlan& p);

// EPI_GATED of rows that come as row * gains (at most 32 rows, see whole_residual_pays).  Its fields stay out of GemmDev: with them the
// grid's size, which lies behind the kernel arguments, moves into a third line of 64 bytes.
constexpr int EPI_GATED_SCALED = 7;
struct GemmScaledDev : GemmDev { RowScale scale; };
template <int EPI> struct GemmDevOf { typedef GemmDev type; };
template <> struct GemmDevOf<EPI_GATED_SCALED> { typedef GemmScaledDev type; };

__device__ inline bf16x8 ld8(const bf16_t* p, bool ok) {
    bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    return ok ? *reinterpret_cast<const bf16x8*>(p) : z;
}
__device__ inline bf16x8 ld8_stream(const bf16_t* p, bool ok) {      // weights: read once, whole lines
    bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    return ok ? ldg_stream(reinterpret_cast<const bf16x8*>(p)) : z;
}


// Tiles of LDS reduced per round: at most 128 KB of fp32 fragments at a time -- one round for every shape built
// (10 tiles x 3 row tiles x 4 waves = 120 KB); rounds of 48 KB cost two more barrier pairs per launch.
template <int MT, int NT>
struct ReduceGroup {
    static constexpr int kMax = 128 / (MT * kGemmWaves);
    static constexpr int raw = (NT < kMax) ? NT : kMax;
    static constexpr int value = (raw >= 2) ? (raw / 2) * 2 : 1;     // even, so gate/up pairs stay together
};

template <int MT, int NT, int EPI>
__global__ __launch_bounds__(kGemmWaves * kWave)
void gemm_stream_kernel(typename GemmDevOf<EPI>::type g) {
    constexpr int WK = kGemmWaves;
    constexpr bool SCALED = (EPI == EPI_GATED_SCALED), gated = (EPI == EPI_GATED) || SCALED;
    extern __shared__ floatx4 red[];                 // [WK][GRP*MT][64]
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int lr = lane % 16, lc = lane / 16;
    const int K = g.K;

    // ---- the NT feature tiles of this workgroup ----
    const bf16_t* wrow[NT];
    bool nvalid[NT];
    int ocol[NT];
    // a unit is one tile (a gate/up tile pair for the gated epilogue); units are dealt to the workgroups
    // as evenly as possible, so a workgroup may own fewer than its NT tile slots
    constexpr int UT = gated ? 2 : 1;
    // split-K launches: the slab is the fast grid index, so that the workgroups of one slab -- which read the same
    // piece of X -- have linear indices that are congruent modulo the slab count and fall on the same XCDs
    constexpr bool SLAB_FAST = (EPI == EPI_PARTIAL);
    const int bx = SLAB_FAST ? blockIdx.y : blockIdx.x;
    const int n_slabs = SLAB_FAST ? gridDim.x : gridDim.y;
    const int unit0 = bx * g.unit_base + (bx < g.unit_rem ? bx : g.unit_rem);
    const int n_units = g.unit_base + (bx < g.unit_rem ? 1 : 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int t = unit0 * UT + nt;
        const bool owned = nt < n_units * UT;
        int seg, local;
        if (gated) {                                  // tiles alternate gate, up of one 16-feature group
            seg = t & 1; local = t >> 1;
            nvalid[nt] = owned && local < g.tiles[0];
            ocol[nt] = local * 16;
        } else {
            if (t < g.tiles[0]) { seg = 0; local = t; }
            else if (t < g.tiles[0] + g.tiles[1]) { seg = 1; local = t - g.tiles[0]; }
            else { seg = 2; local = t - g.tiles[0] - g.tiles[1]; }
            nvalid[nt] = owned && t < g.tiles[0] + g.tiles[1] + g.tiles[2];
            ocol[nt] = t * 16;
        }
        if (!nvalid[nt]) { seg = 0; local = 0; }
        wrow[nt] = g.w[seg] + (size_t)local * (K / 32) * 512 + lane * 8;      // tile `local` of the streaming layout
    }
    // X in operand order: the B operand of (k-step ks, row tile mt) is the 1 KB block ((ks*MT + mt)*64 + lane)*8
    const bf16_t* xlane = g.x + (size_t)lane * 8;

    floatx4 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

    // K is dealt in 32-element MFMA steps.  The steps of the launch are split evenly over the gridDim.y slabs.  Inside
    // a slab the waves take chunks of four steps in turn (so the workgroup reads contiguous 16 KB runs of a tile), and
    // the last, incomplete round of 16 steps is split evenly: no wave does more than one step above the average.
    const int n_steps = K / 32;
    const int sb = n_steps / n_slabs, sr = n_steps % n_slabs;
    const int by = SLAB_FAST ? blockIdx.x : blockIdx.y;
    const int s_begin = by * sb + (by < sr ? by : sr);
    const int s_count = sb + (by < sr ? 1 : 0);
    const int rounds = s_count / (4 * WK);
    const int tail = s_count - rounds * 4 * WK;
    const int tb = tail / WK, tr = tail % WK;
    const int t_len = tb + (wave < tr ? 1 : 0);                              // 0..4 steps
    const int t_k0 = s_begin + rounds * 4 * WK + wave * tb + (wave < tr ? wave : tr);
    const int n_it = rounds + (t_len > 0 ? 1 : 0);
    auto k0_of = [&](int it) { return it < rounds ? s_begin + (it * WK + wave) * 4 : t_k0; };
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
    __shared__ __align__(16) float s_ss[SCALED ? WK * kWave * MT : 4];
    RowScaleSums<WK * kWave, SCALED ? MT : 1> sums;
    if constexpr (SCALED) sums.load(g.scale, tid);      // asked for ahead of the weights
    if (n_it > 0) {
        xload(0, k0_of(0), cnt_of(0));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wload(nt, k0_of(0), cnt_of(0));
    }
    if constexpr (SCALED) sums.store(g.scale, s_ss, tid);
    int par = 0;
    for (int it = 0; it < n_it; ++it, par ^= 1) {
        const bool more = it + 1 < n_it;
        const int nx = k0_of(it + 1), ncnt = cnt_of(it + 1);
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

    // ---- sum the waves through LDS in wave order, GRP tiles per round ----
    constexpr int GRP = ReduceGroup<MT, NT>::value;
    float rstd[MT];
    for (int g0 = 0; g0 < NT; g0 += GRP) {
        if (g0) __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (nt >= g0 && nt < g0 + GRP)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    red[(wave * GRP * MT + (nt - g0) * MT + mt) * kWave + lane] = acc[nt][mt];
        __syncthreads();
        if constexpr (SCALED)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) rstd[mt] = row_rstd<WK * kWave, MT>(g.scale, s_ss, mt * 16 + lr);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt < g0 || nt >= g0 + GRP) continue;
            if (gated && (nt & 1)) continue;                    // the up tile is consumed with its gate tile
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int item = gated ? ((nt - g0) / 2) * MT + mt : (nt - g0) * MT + mt;
                if (item % WK != wave || !nvalid[nt]) continue;  // items are dealt round-robin to the waves
                const int f = (nt - g0) * MT + mt;
                floatx4 s = red[f * kWave + lane];
                for (int w = 1; w < WK; ++w) s += red[(w * GRP * MT + f) * kWave + lane];
                const int m = mt * 16 + lr;
                const int col = ocol[nt] + lc * 4;               // 4 consecutive output features
                if (gated) {
                    constexpr int UP = (NT > 1) ? MT : 0;        // fragment of the paired up tile
                    floatx4 u = red[(f + UP) * kWave + lane];
                    for (int w = 1; w < WK; ++w) u += red[(w * GRP * MT + f + UP) * kWave + lane];
                    if (m < g.M) {
                        bf16x4 o;
                        if (SCALED) { s *= rstd[mt]; u *= rstd[mt]; }
#pragma unroll
                        for (int i = 0; i < 4; ++i) o[i] = (bf16_t)(gemm_act(s[i], g.act) * u[i]);
                        *reinterpret_cast<bf16x4*>((bf16_t*)g.y + packed_index(m, col, MT)) = o;
                    }
                } else if (m < g.M) {
                    float* dst = (float*)g.y + (size_t)by * g.slab_stride + (size_t)m * g.ldy + col;
                    // (more than 16 rows past L2: see plan_split for partial sums; plain logits of 17 to 32 rows whose shares are too many for one round of the
                    // chip, 50000 of them for instance, come this way too and are 0.97 to 1.05 times as fast so)
                    if constexpr (MT > 1) store_through(reinterpret_cast<floatx4*>(dst), s);
                    else *reinterpret_cast<floatx4*>(dst) = s;
                }
            }
        }
    }
}

}  // namespace massv
