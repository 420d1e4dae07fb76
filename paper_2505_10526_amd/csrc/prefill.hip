// prefill_attention: attention of the prompt pass that fills the cache (paper Section 2.2: the projected image
// features enter the sequence ahead of the text tokens, and the language model conditions on all of them).  Same
// definition as verify_attention -- the query at cache row r sees rows 0 .. r -- but with hundreds to thousands
// of new positions per sequence instead of gamma+1, so the work is a dense contraction and the matrix cores are
// the roof, not HBM.
//
// bf16, three kernels: prefill_attention_kernel (d <= 128), prefill_attention_lds_kernel (d <= 128, launches that do not fill the
// chip) and prefill_attention_rows16_kernel (d = 256), the latter two described where they stand.  The first:
//   * The caches are read in the library's blocked layouts; a wave's operands of both products are 16-byte loads per
//     lane straight into registers, no LDS staging and no transposes.
//   * The G query heads that share a KV head are stacked with the positions into rows (row = position * G + head),
//     so every key / value tile fetched serves all G heads.
//   * A wave owns two tiles of 32 stacked rows for the whole key range: Q stays in registers as the B operand of
//     v_mfma_f32_32x32x16_bf16, scores are formed transposed
//     (S^T = K Q^T) so that the probabilities already sit in the operand layout of O^T += V^T P^T, and the streaming
//     softmax keeps (reference, sum, O) in registers.  Nothing is merged between waves; each writes its own rows.
//   * The four waves of a workgroup take neighbouring row ranges, so they walk the same key blocks at nearly
//     the same time and share them through the CU's vector cache; workgroups of one (sequence, KV head) pair
//     have linear ids congruent modulo the pair count, which (8 dies, round-robin dispatch) puts them on one
//     die whenever the pair count is a multiple of 8, so the pair's keys and values are fetched into one L2.
//   * Only blocks that cross some row's first or last visible key pay for masks.
// Measured and dropped at 8 x 2048 positions, d = 128 (the shipped kernel: 285-304 us):
//   the 16x16x32 instruction with 4 tiles of 16 rows, 336-376 us (a lone wave issues one of those only every ~31
//   cycles, and twice as many are needed); two key / value register sets with Q re-read from LDS, 489 us; 32 rows
//   per wave with two waves per SIMD and operands loaded per wave, 343-378 us (the vector cache cannot feed twice
//   the operand traffic); eight waves of 32 rows with the blocks staged once per workgroup in LDS by direct
//   global->LDS loads (ring of 4 stages of 2 blocks, one barrier per stage), 283-313 us and no better on four
//   other shapes: the barrier re-aligns the two waves of a SIMD, which then want the same unit at the same time; the
//   same with the two waves held in opposite phases by two barriers per stage (one multiplies while the other forms
//   exponentials), 299-309 us: a phase of exponentials takes 2200 cycles, one of matrix instructions 1600.
// fp32: the plain one-workgroup-per-(position, head) kernel below, for the small configuration.
#include "kernels.h"

#include <atomic>
#include <type_traits>

namespace massv {

constexpr int kPfWaves = 4;
constexpr int kPfThreads = kPfWaves * kWave;
constexpr int kPfBlk = MASSV_V_BLOCK;

struct PrefillParams {
    const bf16_t* q; const bf16_t* kc; const bf16_t* vc;
    const int32_t* kv_len; const int32_t* n_new; const int32_t* n_bidir;     // n_bidir may be null
    bf16_t* out;
    int Lq, n_q, n_kv, l_max, window, n_tiles;
    float scale_log2;            // scale * log2(e)
};

// One past the last row visible to the query at cache row r: r + 1, or the end of the leading block of m rows
// that attends within itself when r lies inside it (never beyond the rows that exist, `total`).
__host__ __device__ inline int pf_hi(int r, int m, int total) {
    if (r < m) { const int e = m < total ? m : total; return e > r + 1 ? e : r + 1; }
    return r + 1;
}
__host__ __device__ inline int pf_lo(int r, int W) { return (W > 0 && r + 1 > W) ? r + 1 - W : 0; }

// max(a, b, c) in one instruction.  (fmaxf nests compile to a canonicalising self-maximum per operand plus the
// maximum itself: 11 instructions for 8 scores instead of 4; operands here are never NaN -- masked scores are -inf.)
__device__ inline float pf_max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// ---------------------------------------------------------------------------
// A lone wave per SIMD gets a 32x32x16 matrix instruction out every ~40 cycles (against ~31 for the 16x16x32 form
// that does half the work).  A wave owns two tiles of 32 stacked rows.
//   S^T tile (32 key slots x 32 rows): lane l holds row l % 32 and the slots 8 (v / 4) + 4 (l / 32) + v % 4, v = 0..15.
//   Key slot rho of a block carries key 16 (g / 2) + 8 h + 4 (g % 2) + r (rho = 8 g + 4 h + r), so that the lane's
//   values v = 8 t .. 8 t + 7 are the keys 16 t + 8 (l / 32) + (0..7): as they stand they are the B operand of step t
//   of O^T += V^T P^T, whose A operand is then one 16-byte load of 8 consecutive keys of one dim.
// ---------------------------------------------------------------------------
__device__ inline float pf_xor32_max(float v) { return fmaxf(v, __shfl_xor(v, 32, kWave)); }

template <int D>
__global__ __launch_bounds__(kPfThreads)
void prefill_attention_kernel(PrefillParams p) {
    constexpr int RT = 2;               // row tiles of a wave
    constexpr int KS = D / 16;          // 16-wide k-steps of the score product
    constexpr int NT = D / 32;          // 32-dim tiles of the output
    constexpr int RW = RT * 32;         // stacked rows per wave
    const int pair = blockIdx.x, b = pair / p.n_kv, g = pair % p.n_kv;
    const int tile = p.n_tiles - 1 - (int)blockIdx.y;                 // the longest key ranges are started first
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lr = lane % 32, hh = lane / 32;
    const int G = p.n_q / p.n_kv;
    const int L = cached_rows(p.kv_len[b], p.l_max);
    int n = p.n_new[b]; n = n < 0 ? 0 : (n > p.Lq ? p.Lq : n);
    if (L + n > p.l_max) n = p.l_max - L > 0 ? p.l_max - L : 0;
    const int rows = n * G;
    const int r0 = (tile * kPfWaves + wave) * RW;                     // first stacked row of this wave
    if (r0 >= rows) return;                                            // (no barriers below: waves are independent)
    const int total = L + n;
    const int m_bidir = p.n_bidir ? p.n_bidir[b] : 0;
    const int W = p.window;
    const size_t bg = (size_t)b * p.n_kv + g;

    // ---- rows of this wave: position, visible key range; Q operand in registers ----
    bf16x8 qreg[RT][KS];
    int hi_row[RT], lo_row[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        int r = r0 + rt * 32 + lr;
        if (r >= rows) r = rows - 1;                                   // padding rows repeat the last one; never stored
        const int i = r / G, qh = r % G;
        hi_row[rt] = pf_hi(L + i, m_bidir, total);
        lo_row[rt] = pf_lo(L + i, W);
        const bf16_t* qr = p.q + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[rt][ks] = *reinterpret_cast<const bf16x8*>(qr + ks * 16 + hh * 8);
    }
    const int i_first = r0 / G;
    const int r_last = (r0 + RW - 1 < rows - 1) ? r0 + RW - 1 : rows - 1;
    const int i_last = r_last / G;
    const int min_hi = pf_hi(L + i_first, m_bidir, total), max_hi = pf_hi(L + i_last, m_bidir, total);
    const int min_lo = pf_lo(L + i_first, W), max_lo = pf_lo(L + i_last, W);
    const int blk_begin = min_lo / kPfBlk, blk_end = (max_hi + kPfBlk - 1) / kPfBlk;

    floatx16 acc[RT][NT];
    float m_run[RT], l_run[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = -INFINITY; l_run[rt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[rt][nt][e] = 0.f;
    }

    // key slot lr = 8 g + 4 h + r of a block -> key 16 (g / 2) + 8 h + 4 (g % 2) + r, which the blocked key cache
    // keeps in its half g % 2 (bit 2 of the key) at place 4 (2 (g / 2) + h) + r; the lane's 8 dims are chunk
    // 2 ks + hh of that half
    const int sg = lr / 8, sh = (lr / 4) % 2, sr = lr % 4;
    const bf16_t* kbase = p.kc + bg * (size_t)p.l_max * D + (size_t)(sg % 2) * (D * 16) + hh * 128 + ((2 * (sg / 2) + sh) * 4 + sr) * 8;
    const bf16_t* vbase = p.vc + bg * (size_t)p.l_max * D + (size_t)lr * kPfBlk + hh * 8;
    auto load_k = [&](int blk, bf16x8 (&kreg)[KS]) {
        const bf16_t* kb = kbase + (size_t)blk * kPfBlk * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kreg[ks] = *reinterpret_cast<const bf16x8*>(kb + ks * 256);
    };
    // value operand (nt, t): dim 32 nt + lr, keys 16 t + 8 hh + (0..7) of the block
    auto load_v = [&](int blk, bf16x8 (&vreg)[NT][2]) {
        const bf16_t* vb = vbase + (size_t)blk * D * kPfBlk;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                vreg[nt][t] = *reinterpret_cast<const bf16x8*>(vb + (size_t)(nt * 32) * kPfBlk + t * 16);
    };

    constexpr float kLazy = 8.0f;       // a row's reference exponent is raised only when exceeded by 2^8
    // ---- pieces of one block for one row tile ----
    // S^T tile: KS matrix instructions
    auto s_tile = [&](bf16x8 (&kr)[KS], int rt, floatx16& sc) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[ks], qreg[rt][ks], sc, 0, 0, 0);
    };
    // O^T += V^T P^T: 2 NT matrix instructions
    auto pv_tile = [&](int rt, bf16x8 (&vr)[NT][2], bf16x8 (&pv)[2]) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[rt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[nt][t], pv[t], acc[rt][nt], 0, 0, 0);
    };
    // values of rows past the valid length may hold anything: zero them (last block only)
    auto v_clean = [&](int blk, bf16x8 (&vr)[NT][2]) {
        const int key0 = blk * kPfBlk + hh * 8;
        if ((blk + 1) * kPfBlk > total) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (key0 + 16 * t + e >= total) vr[nt][t][e] = (bf16_t)0.f;
        }
    };
    // first half of the streaming softmax: masks, the lane's maximum, and (rarely) a raised reference with the
    // accumulators rescaled.  Value v of the lane is key key0 + 16 (v / 8) + v % 8.
    auto soft_max = [&](int rt, int blk, floatx16& sc) {
        const int key0 = blk * kPfBlk + hh * 8;
        const bool masked = (blk + 1) * kPfBlk > min_hi || blk * kPfBlk < max_lo;
        if (masked) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = key0 + 16 * (v / 8) + v % 8;
                if (key >= hi_row[rt] || key < lo_row[rt]) sc[v] = -INFINITY;
            }
        }
        float mx = pf_max3(pf_max3(pf_max3(sc[0], sc[1], sc[2]), pf_max3(sc[3], sc[4], sc[5]), pf_max3(sc[6], sc[7], sc[8])),
                           pf_max3(pf_max3(sc[9], sc[10], sc[11]), pf_max3(sc[12], sc[13], sc[14]), sc[15]), sc[15]);
        mx *= p.scale_log2;
        if (__any(mx > m_run[rt] + kLazy)) {
            mx = pf_xor32_max(mx);
            if (mx > m_run[rt] + kLazy) {
                const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - mx);     // m_run = -inf gives 0
                l_run[rt] *= alpha;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    // keeps the copies out of the accumulation registers inside this rare branch
                    asm volatile("" : "+a"(acc[rt][nt]));
                    acc[rt][nt] *= alpha;
                }
                m_run[rt] = mx;
            }
        }
    };
    // second half: probabilities relative to the reference, their sum, and the bf16 operand of the second product
    auto soft_exp = [&](int rt, const floatx16& sc, bf16x8 (&pv)[2]) {
        const float neg_m = (m_run[rt] == -INFINITY) ? 0.f : -m_run[rt];
        float ps = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float pe = __builtin_amdgcn_exp2f(fmaf(sc[v], p.scale_log2, neg_m));
            ps += pe;
            pv[v / 8][v % 8] = (bf16_t)pe;
        }
        l_run[rt] += ps;
    };

    {
        // Two row tiles A and B leapfrog, so that the vector arithmetic of one tile's softmax is issued between the
        // matrix instructions of the other tile (one wave per SIMD: a matrix instruction holds the wave's issue for
        // about 18 of the 40 cycles it needs, the rest is free for independent vector instructions -- but only if
        // the instruction stream alternates, since a wave issues in order):
        //   step 1 of block i:  exponentials of (B, i)      between   O_A += V_i P_A,i   and   S_A,i+1 = K_i+1 Q_A
        //   step 2 of block i:  exponentials of (A, i + 1)  between   O_B += V_i P_B,i   and   S_B,i+1 = K_i+1 Q_B
        // Keys are held two blocks ahead and values one block ahead, in two register sets each.
        // A step is two halves of 8 score values each: the first next to the KS matrix instructions of the other
        // tile's next scores, the second next to the 2 NT matrix instructions of the other tile's second product.
        // One key set and one value set: the keys of block i + 2 are requested as soon as the scores of block i + 1
        // are formed (middle of step 2), the values of block i + 1 at the end of step 2; each has the other half of
        // the work before it is needed.
        auto exps = [&](int rv, const floatx16& sv, bf16x8& po, int v0, float neg_m, float& ps) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(sv[v0 + e], p.scale_log2, neg_m));
                ps += pe;
                po[e] = (bf16_t)pe;
            }
        };
        auto order = [&](auto n_mfma) {            // the order asked of the scheduler for one half
            constexpr int N = decltype(n_mfma)::value, VP = 8 / N;
#pragma unroll
            for (int m = 0; m < N; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2 * VP, 0);
                __builtin_amdgcn_sched_group_barrier(0x400, VP, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2 * VP, 0);
            }
        };
        // first half: tile rv's values 0..7, tile rm's scores of the block whose keys kq holds
        auto half_s = [&](int rv, const floatx16& sv, bf16x8 (&pvo)[2], float neg_m, float& ps, int rm, bf16x8 (&kq)[KS], floatx16& sm) {
            __builtin_amdgcn_sched_barrier(0);
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                sm = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kq[ks], qreg[rm][ks], ks == 0 ? zero : sm, 0, 0, 0);
            exps(rv, sv, pvo[0], 0, neg_m, ps);
            order(std::integral_constant<int, KS>{});
            // (the probabilities are first needed a step later; without a use here the compiler moves their
            // arithmetic down to that step, away from the matrix instructions it is meant to sit between)
            asm volatile("" : "+v"(pvo[0]), "+v"(ps));
            __builtin_amdgcn_sched_barrier(0);
        };
        // second half: tile rv's values 8..15, tile rm's second product with the values vq holds
        auto half_pv = [&](int rv, const floatx16& sv, bf16x8 (&pvo)[2], float neg_m, float& ps, int rm, bf16x8 (&pm)[2], bf16x8 (&vq)[NT][2]) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[rm][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vq[nt][t], pm[t], acc[rm][nt], 0, 0, 0);
            exps(rv, sv, pvo[1], 8, neg_m, ps);
            order(std::integral_constant<int, 2 * NT>{});
            asm volatile("" : "+v"(pvo[1]), "+v"(ps));
            __builtin_amdgcn_sched_barrier(0);
        };
        const int nb = blk_end - blk_begin;
        bf16x8 kq[KS], vq[NT][2];
        floatx16 sA, sB;
        bf16x8 pA[2], pB[2];
        if (nb > 0) {
            load_k(blk_begin, kq);
            s_tile(kq, 0, sA);
            s_tile(kq, 1, sB);
            if (nb > 1) load_k(blk_begin + 1, kq);
            load_v(blk_begin, vq);                     // keys before values, the order the loop requests them in
            soft_max(0, blk_begin, sA);
            soft_exp(0, sA, pA);
        }
        // entering block i: kq holds the keys of block i + 1, vq the values of block i, pA tile A's probabilities
        // and sB tile B's scores of block i
        for (int i = 0; i + 1 < nb; ++i) {
            const int blk = blk_begin + i;
            v_clean(blk, vq);
            soft_max(1, blk, sB);
            {
                const float neg_m = (m_run[1] == -INFINITY) ? 0.f : -m_run[1];
                float ps = 0.f;
                half_s(1, sB, pB, neg_m, ps, 0, kq, sA);
                half_pv(1, sB, pB, neg_m, ps, 0, pA, vq);
                l_run[1] += ps;
            }
            soft_max(0, blk + 1, sA);
            {
                const float neg_m = (m_run[0] == -INFINITY) ? 0.f : -m_run[0];
                float ps = 0.f;
                half_s(0, sA, pA, neg_m, ps, 1, kq, sB);
                if (i + 2 < nb) load_k(blk + 2, kq);
                half_pv(0, sA, pA, neg_m, ps, 1, pB, vq);
                load_v(blk + 1, vq);
                l_run[0] += ps;
            }
        }
        if (nb > 0) {                                  // the last block: nothing follows tile A's second product
            const int blk = blk_end - 1;
            v_clean(blk, vq);
            soft_max(1, blk, sB);
            const float neg_m = (m_run[1] == -INFINITY) ? 0.f : -m_run[1];
            float ps = 0.f;
            exps(1, sB, pB[0], 0, neg_m, ps);
            half_pv(1, sB, pB, neg_m, ps, 0, pA, vq);
            l_run[1] += ps;
            pv_tile(1, vq, pB);
        }
    }

    // ---- write this wave's rows: lane holds dims 32 nt + 8 (v / 4) + 4 hh + v % 4 of row 32 rt + lr ----
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const float l = l_run[rt] + __shfl_xor(l_run[rt], 32, kWave);
        const int r = r0 + rt * 32 + lr;
        if (r >= rows) continue;
        const float inv = 1.0f / l;                        // every row sees at least its own key
        const int i = r / G, qh = r % G;
        bf16_t* dst = p.out + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D + hh * 4;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const floatx16& v = acc[rt][nt];
                bf16x4 o = {(bf16_t)(v[4 * q4] * inv), (bf16_t)(v[4 * q4 + 1] * inv), (bf16_t)(v[4 * q4 + 2] * inv), (bf16_t)(v[4 * q4 + 3] * inv)};
                *reinterpret_cast<bf16x4*>(dst + nt * 32 + q4 * 8) = o;
            }
    }
}

// ---------------------------------------------------------------------------
// One tile of 32 rows per wave, blocks staged in LDS: for launches of d <= 128 that are too small to fill the chip (see the
// dispatch below).  The blocks travel into LDS once per workgroup (global_load_lds, a ring of
// four, two to three blocks ahead, one barrier per block) and the waves take their fragments from there; the
// exponentials of block i sit between the matrix instructions of block i + 1's scores, which are formed in two chains.
// A value block's pieces (8 keys of a dim) lie in LDS at place c ^ (dim / 4) % 4 of the dim's four: the 32 dims of a
// fragment are 64 bytes apart, which as they lie in the cache is four lanes to a bank.
// Waves without rows only bring their share of the blocks in (multiplying the last row along made calls of up to 32
// rows 4 to 12 % slower).
// HALVES = 2: a second group of four waves takes the later half of the key blocks, through a ring of its own, and the two sums are put together in
// LDS at the end.  What bounds these launches is the length of one wave's chain of blocks, with nothing else on its SIMD: now it is
// half as long and every SIMD has two.  All in vector registers (211 at d = 128; with the sums in accumulation registers, 128 and
// 126, the moves between them ate the gain: 1000 rows on 6000 93 us).  28 / 4 heads of 128, one half and two: 1 x 1111 rows 30.3 and 26.9 us,
// 1 x 800 24.2 and 21.2, 1000 on 6000 108.4 and 85.8, 16 on 8000 133.7 and 101.9; 14 / 2 heads of 64, 1 x 1111 22.1 and 17.2, 1000 on 6000
// 79.7 and 52.9.  Under pf_cut_blocks blocks the first group does it alone: setting up the second ring and putting the sums together takes 1 to 2 us (28 / 4
// heads of 128, 292 rows on 35, 11 blocks: in one piece 14.4 us, cut 15.8).  Cut against one piece over 1300 calls that fit the chip, medians by blocks of keys: d = 128 10 to
// 13 blocks 0.95 to 0.97 times as fast, 16 and 17 1.01, 18 1.03, 24 1.08; d = 64 10 to 13 blocks 0.98 to 1.01, 14 1.05, 24 1.13.  As it is, none of 1300 calls of 8 to 26
// blocks is slower than by four waves alone (0.99 to 1.36).
// ---------------------------------------------------------------------------
constexpr int kPfRing = 4;
constexpr int pf_cut_blocks(int D) { return D == 64 ? 10 : 18; }
constexpr size_t pf_lds_bytes(int D) { return (size_t)kPfRing * 2 * kPfBlk * D * sizeof(bf16_t); }      // 64 KB at d = 128

template <int D, bool DIRECT, int HALVES>
__global__ __launch_bounds__(kPfThreads * HALVES)
void prefill_attention_lds_kernel(PrefillParams p) {
    constexpr int KS = D / 16, NT = D / 32, BP = D * 4;      // BP: 16-byte pieces of a block's keys (or values)
    constexpr int NL = BP / kPfThreads;                               // requests a lane makes for a block's keys (and values)
    const int pair = blockIdx.x, b = pair / p.n_kv, g = pair % p.n_kv;
    const int tile = p.n_tiles - 1 - (int)blockIdx.y;                 // the longest key ranges are started first
    const int tid = threadIdx.x % kPfThreads, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), half = HALVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kPfThreads);
    const int lr = lane % 32, hh = lane / 32;
    const int G = p.n_q / p.n_kv;
    const int L = cached_rows(p.kv_len[b], p.l_max);
    int n = p.n_new[b]; n = n < 0 ? 0 : (n > p.Lq ? p.Lq : n);
    if (L + n > p.l_max) n = p.l_max - L > 0 ? p.l_max - L : 0;
    const int rows = n * G;
    const int w0 = tile * kPfWaves * 32;                              // first stacked row of the workgroup
    if (w0 >= rows) return;                                           // uniform over the workgroup
    const int total = L + n;
    const int m_bidir = p.n_bidir ? p.n_bidir[b] : 0;
    const int W = p.window;
    const size_t bg = (size_t)b * p.n_kv + g;

    // rows of this wave (one past the last row repeats it and is not stored) and the keys they see
    const int r0 = w0 + wave * 32;
    auto pos_of = [&](int r) { return (r < rows ? r : rows - 1) / G; };
    const int min_hi = pf_hi(L + pos_of(r0), m_bidir, total), max_hi = pf_hi(L + pos_of(r0 + 31), m_bidir, total);
    const int min_lo = pf_lo(L + pos_of(r0), W), max_lo = pf_lo(L + pos_of(r0 + 31), W);
    // blocks of the workgroup (visibility moves up with the row), of this half of it (few are not worth a second one), and of this wave
    const int all_begin = pf_lo(L + pos_of(w0), W) / kPfBlk;
    const int all_end = (pf_hi(L + pos_of(w0 + kPfWaves * 32 - 1), m_bidir, total) + kPfBlk - 1) / kPfBlk;
    const int cut = HALVES == 1 || all_end - all_begin < pf_cut_blocks(D) ? all_end : (all_begin + all_end + 1) / 2;
    const int blk_begin = half ? cut : all_begin, blk_end = half ? all_end : cut;
    int blk_first = min_lo / kPfBlk, blk_last = (max_hi - 1) / kPfBlk;
    const bool whole = HALVES == 1 || cut == all_end;
    if (HALVES == 2) {
        if (half && whole) return;                                    // (a barrier waits for the waves that are still there)
        blk_first = blk_first > blk_begin ? blk_first : blk_begin;
        blk_last = blk_last < blk_end - 1 ? blk_last : blk_end - 1;
    }

    extern __shared__ bf16x8 pf_lds_all[];                            // [HALVES][kPfRing][keys | values][BP]
    bf16x8* const pf_lds = pf_lds_all + half * (kPfRing * 2 * BP);
    // DIRECT: caches that start at a multiple of 16 bytes.  Others travel through registers (a load to LDS takes 16 bytes
    // from a multiple of 16 only; an ordinary load takes them from anywhere).
    const bf16_t* const kc = p.kc + bg * (size_t)p.l_max * D + tid * 8;
    const bf16_t* const vc = p.vc + bg * (size_t)p.l_max * D + (tid ^ ((tid / 16) % 4)) * 8;
    auto bring = [&](const bf16_t* src, bf16x8* dst) {
        if constexpr (DIRECT)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
        else
            dst[lane] = *reinterpret_cast<const bf16x8_any*>(src);
    };
    auto request = [&](int blk) {
        bf16x8* dst = pf_lds + (size_t)(blk % kPfRing) * 2 * BP + wave * kWave;
#pragma unroll
        for (int u = 0; u < NL; ++u) bring(kc + ((size_t)blk * BP + u * kPfThreads) * 8, dst + u * kPfThreads);
#pragma unroll
        for (int u = 0; u < NL; ++u) bring(vc + ((size_t)blk * BP + u * kPfThreads) * 8, dst + BP + u * kPfThreads);
    };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // Opens block blk: block blk + 1 has landed for every wave (a wave's requests complete in order; those of blk + 2 may
    // still be on their way), everybody is done with block blk - 1, and its place takes block blk + 3.
    // (the last block needs none of it: it landed when the one before was opened, or at the start)
    auto open = [&](int blk) {
        if (blk + 1 >= blk_end) return;
        if (!DIRECT) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        else if (blk + 2 < blk_end) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        barrier();
        if (blk + 3 < blk_end) request(blk + 3);
    };
    // the first block and Q have to be there to start with
    auto start = [&]() {
        if (!DIRECT) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        else if (blk_begin + 2 < blk_end) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        barrier();
    };
    auto request_first = [&]() {
        request(blk_begin);
        if (blk_begin + 1 < blk_end) request(blk_begin + 1);
        if (blk_begin + 2 < blk_end) request(blk_begin + 2);
    };
    const bool idle = r0 >= rows || blk_first > blk_last;     // such a wave only brings its share of the blocks in
    request_first();
    if (idle) {
        start();
        for (int blk = blk_begin; blk < blk_end; ++blk) open(blk);
    }
    if (idle && whole) return;

    floatx16 acc[NT];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[nt][e] = 0.f;
    if (!idle) {
        bf16x8 qreg[KS];
        int hi_row, lo_row;
        {
            const int r = r0 + lr < rows ? r0 + lr : rows - 1;
            const int i = r / G, qh = r % G;
            hi_row = pf_hi(L + i, m_bidir, total);
            lo_row = pf_lo(L + i, W);
            const bf16_t* qr = p.q + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qr + ks * 16 + hh * 8);
        }

        // fragments: key slot lr of a block lies in half (lr / 8) % 2 at place 4 (2 (lr / 16) + (lr / 4) % 2) + lr % 4
        const bf16x8* const kfrag = pf_lds + ((lr / 8) % 2) * (BP / 2) + hh * 16 + 4 * (2 * (lr / 16) + (lr / 4) % 2) + lr % 4;
        const bf16x8* const vfrag = pf_lds + BP + lr * 4;
        const int vx = (lr / 4) % 4;
        bf16x8 k0[KS], v0[NT][2];
        auto load_k = [&](int blk) {
            const bf16x8* kp = kfrag + (blk % kPfRing) * 2 * BP;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) k0[ks] = kp[ks * 32];
        };
        auto load_v = [&](int blk) {
            const bf16x8* vp = vfrag + (blk % kPfRing) * 2 * BP;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) v0[nt][t] = vp[nt * 128 + ((2 * t + hh) ^ vx)];
        };

        floatx16 sc, sn, so;
        bf16x8 pv[2];
        auto chains = [&]() {                          // S^T of the block whose keys k0 holds: even k-steps in sn, odd in so
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ks += 2) {
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[ks], qreg[ks], ks == 0 ? zero : sn, 0, 0, 0);
                so = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[ks + 1], qreg[ks + 1], ks == 0 ? zero : so, 0, 0, 0);
            }
        };
        constexpr float kLazy = 8.0f;                  // a row's reference exponent is raised only when exceeded by 2^8
        auto soft_max = [&](int blk) {                 // value v of the lane is key key0 + 16 (v / 8) + v % 8
            const int key0 = blk * kPfBlk + hh * 8;
            if ((blk + 1) * kPfBlk > min_hi || blk * kPfBlk < max_lo) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = key0 + 16 * (v / 8) + v % 8;
                    if (key >= hi_row || key < lo_row) sc[v] = -INFINITY;
                }
            }
            float mx = pf_max3(pf_max3(pf_max3(sc[0], sc[1], sc[2]), pf_max3(sc[3], sc[4], sc[5]), pf_max3(sc[6], sc[7], sc[8])),
                               pf_max3(pf_max3(sc[9], sc[10], sc[11]), pf_max3(sc[12], sc[13], sc[14]), sc[15]), sc[15]);
            mx *= p.scale_log2;
            if (__any(mx > m_run + kLazy)) {
                mx = pf_xor32_max(mx);
                if (mx > m_run + kLazy) {
                    const float alpha = __builtin_amdgcn_exp2f(m_run - mx);     // m_run = -inf gives 0
                    l_run *= alpha;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        // keeps the copies out of the accumulation registers inside this rare branch
                        if constexpr (HALVES == 1) asm volatile("" : "+a"(acc[nt]));
                        else asm volatile("" : "+v"(acc[nt]));
                        acc[nt] *= alpha;
                    }
                    m_run = mx;
                }
            }
        };
        auto soft_exp = [&](float neg_m) {
            float ps = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(sc[v], p.scale_log2, neg_m));
                ps += pe;
                pv[v / 8][v % 8] = (bf16_t)pe;
            }
            return ps;
        };
        auto product = [&]() {                         // O^T += V^T P^T
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v0[nt][t], pv[t], acc[nt], 0, 0, 0);
        };

        start();
        int blk = blk_begin;
        for (; blk < blk_first; ++blk) open(blk);      // blocks that only the rows of other waves see
        load_k(blk);
        chains();
        sc = sn + so;
        for (; blk < blk_last; ++blk) {
            open(blk);
            load_k(blk + 1);
            load_v(blk);
            soft_max(blk);
            const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
            __builtin_amdgcn_sched_barrier(0);
            chains();
            float ps = soft_exp(neg_m);
#pragma unroll
            for (int m = 0; m < KS; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 32 / KS, 0);
                __builtin_amdgcn_sched_group_barrier(0x400, 16 / KS, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 32 / KS, 0);
            }
            // (without a use here the compiler moves the exponentials down to the second product, their first use)
            asm volatile("" : "+v"(pv[0]), "+v"(pv[1]), "+v"(ps));
            __builtin_amdgcn_sched_barrier(0);
            l_run += ps;
            product();
            sc = sn + so;
        }
        open(blk);
        load_v(blk);
        if ((blk + 1) * kPfBlk > total) {              // values of rows past the valid ones may hold anything
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (blk * kPfBlk + hh * 8 + 16 * t + e >= total) v0[nt][t][e] = (bf16_t)0.f;
        }
        soft_max(blk);
        l_run += soft_exp((m_run == -INFINITY) ? 0.f : -m_run);
        product();
        for (++blk; blk < blk_end; ++blk) open(blk);
    }

    // The halves' sums: each wave hands its partner the dims that the partner finishes and takes those of its own.
    if (!whole) {
        constexpr int NH = NT / 2;
        if (all_end - cut < cut - all_begin && half) barrier();       // (one a block: as many in either half)
        floatx4* const mine = reinterpret_cast<floatx4*>(pf_lds_all) + (half * kPfWaves + wave) * (NH * 4 + 1) * kWave + lane;
        const floatx4* const other = reinterpret_cast<const floatx4*>(pf_lds_all) + ((1 - half) * kPfWaves + wave) * (NH * 4 + 1) * kWave + lane;
        __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NH; ++nt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const floatx16& v = half ? acc[nt] : acc[NH + nt];
                mine[(nt * 4 + q4) * kWave] = floatx4{v[4 * q4], v[4 * q4 + 1], v[4 * q4 + 2], v[4 * q4 + 3]};
            }
        mine[NH * 4 * kWave] = floatx4{m_run, l_run, 0.f, 0.f};
        __syncthreads();
        const floatx4 ml = other[NH * 4 * kWave];
        const float m = fmaxf(m_run, ml[0]);
        const float a = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m), c = ml[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[0] - m);
        l_run = l_run * a + ml[1] * c;
#pragma unroll
        for (int nt = 0; nt < NH; ++nt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const floatx4 o = other[(nt * 4 + q4) * kWave];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = half ? acc[NH + nt][4 * q4 + e] : acc[nt][4 * q4 + e];
                    acc[nt][4 * q4 + e] = x * a + o[e] * c;
                }
            }
        if (r0 >= rows) return;
    }

    // ---- write this wave's rows: lane holds dims 32 nt + 8 (v / 4) + 4 hh + v % 4 of row lr ----
    const float l = l_run + __shfl_xor(l_run, 32, kWave);
    const int r = r0 + lr;
    if (r >= rows) return;
    const float inv = 1.0f / l;                    // every row sees at least its own key
    const int i = r / G, qh = r % G;
    bf16_t* dst = p.out + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D + half * (D / 2) + hh * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (HALVES == 2 && nt >= NT / 2 && !whole) break;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const floatx16& v = acc[nt];
            bf16x4 o = {(bf16_t)(v[4 * q4] * inv), (bf16_t)(v[4 * q4 + 1] * inv), (bf16_t)(v[4 * q4 + 2] * inv), (bf16_t)(v[4 * q4 + 3] * inv)};
            *reinterpret_cast<bf16x4*>(dst + nt * 32 + q4 * 8) = o;
        }
    }
}

// ---------------------------------------------------------------------------
// d = 256: 16 rows per wave, eight waves, two a SIMD.  With 32 rows a wave is alone on its SIMD (accumulators and Q take 192
// registers) and its scores, softmax and second product follow one another; with 16 one wave's softmax, which goes first
// (s_setprio), runs beside the other's matrix instructions, for twice the LDS reads, at 256 bytes a cycle.  What bounds it: both
// waves of a SIMD wait for the same fragments behind a barrier.  Blocks are taken in pairs, one barrier a pair; half of a block's
// keys are read ahead, behind the second product of the block before.
// The blocks travel through a ring of five (all 160 KB): a wave asks for one as it opens a pair and for the next between the
// two blocks.  With a ring of two pairs and both asked for at once, a request held its wave as long as the memory took to accept it, and
// all waves stood still together: caches of 1200 rows and more that are not in the last-level cache, tiles of 128 rows, were 3 to 9 %
// slower than by 32 rows a wave (1 x 64 positions on 6000 211 us; ring of five, both at once 218, 32 rows a wave 197).
// Key fragments lie as in the cache, 1 KB each.  Piece c (8 keys) of dim v lies at place c ^ (-(v / 4)) % 4 of the dim's four:
// a fragment's 16 dims x 4 pieces then are free of bank conflicts (c ^ (v / 4) % 4, right for 32 dims x 2 pieces, cost two cycles
// a read).  The even and odd steps of a score are chains of their own; their sum also keeps the maximum, which is
// assembly, from reading a matrix result directly (the compiler does not wait for one there).
// The places of the ring rotate through five registers: as blk % 5, or counted and wrapped, they were work on the path from the barrier
// to the first keys (1 x 64 on 6000 184 us, 188 and now 174).
// 16 / 8 heads, caches not in the last-level cache, us by 32 rows a wave, ring of two pairs and now, in turn on one card: second pieces
// of 4 prompts of up to 1500 positions on up to 600 cached, window 1024, image block 149, 136 and 131; 4 x 2000 171, 159, 154; 8 x 1500
// on 1000, window 1024 304, 274, 264; 1 x 2048 on 6000 268, 279, 250; 1 x 64 on 6000 197, 211, 174; 1 x 1000 39.8, 36.9, 35.3; 300 on
// 1500 63.9, 61.0, 56.7; 100 rows 10.6, 9.3, 9.3; one row on 3000 cached ones 87, 73, 71, 16 of them 97, 98, 87.  Over 6600 calls (1 to
// 4096 rows, caches to 8000, windows, in and out of the last-level cache) none is slower than by 32 rows a wave.  Tried: two waves that
// share 32 rows and exchange halves of the scores, a barrier a block (4 to 12 % slower than 32 rows a wave); four waves and half the
// ring, two workgroups a compute unit (25 to 60 % slower); one load a thread that brings the pair after the next as far as L2 (up to
// 25 % slower); all of a block's keys ahead (spills).
// ---------------------------------------------------------------------------
constexpr int kPf16Waves = 8, kPf16Threads = kPf16Waves * kWave, kPf16Ring = 5;
template <int D>
constexpr size_t pf16_lds_bytes() { return (size_t)kPf16Ring * 2 * kPfBlk * D * sizeof(bf16_t); }

template <int D, bool DIRECT>
__global__ __launch_bounds__(kPf16Threads)
void prefill_attention_rows16_kernel(PrefillParams p) {
    constexpr int KS = D / 32, NT = D / 16, BP = D * 4;      // BP: 16-byte pieces of a block's keys (or values)
    constexpr int NL = BP / kPf16Threads;                               // requests a lane makes for a block's keys (and values)
    constexpr int WROWS = 16 * kPf16Waves;
    const int pair = blockIdx.x, b = pair / p.n_kv, g = pair % p.n_kv;
    const int tile = p.n_tiles - 1 - (int)blockIdx.y;                 // the longest key ranges are started first
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lr = lane % 16, lc = lane / 16;
    const int G = p.n_q / p.n_kv;
    const int L = cached_rows(p.kv_len[b], p.l_max);
    int n = p.n_new[b]; n = n < 0 ? 0 : (n > p.Lq ? p.Lq : n);
    if (L + n > p.l_max) n = p.l_max - L > 0 ? p.l_max - L : 0;
    const int rows = n * G;
    const int w0 = tile * WROWS;                                      // first stacked row of the workgroup
    if (w0 >= rows) return;                                           // uniform over the workgroup
    const int total = L + n;
    const int m_bidir = p.n_bidir ? p.n_bidir[b] : 0;
    const int W = p.window;
    const size_t bg = (size_t)b * p.n_kv + g;

    // rows of this wave (one past the last row repeats it and is not stored) and the keys they see
    const int r0 = w0 + wave * 16;
    auto pos_of = [&](int r) { return (r < rows ? r : rows - 1) / G; };
    const int min_hi = pf_hi(L + pos_of(r0), m_bidir, total), max_hi = pf_hi(L + pos_of(r0 + 15), m_bidir, total);
    const int min_lo = pf_lo(L + pos_of(r0), W), max_lo = pf_lo(L + pos_of(r0 + 15), W);
    // blocks of this wave, none where it has no row (it brings its share of the workgroup's blocks in all the same)
    const int blk_first = min_lo / kPfBlk, blk_last = r0 < rows ? (max_hi - 1) / kPfBlk : -1;
    // blocks of the workgroup (visibility moves up with the row)
    const int blk_begin = pf_lo(L + pos_of(w0), W) / kPfBlk;
    const int blk_end = (pf_hi(L + pos_of(w0 + WROWS - 1), m_bidir, total) + kPfBlk - 1) / kPfBlk;

    extern __shared__ bf16x8 pf_lds[];                                // [kPf16Ring][keys | values][BP]
    const bf16_t* const kc = p.kc + bg * (size_t)p.l_max * D + tid * 8;
    const bf16_t* const vc = p.vc + bg * (size_t)p.l_max * D + (tid ^ ((-(tid / 16)) & 3)) * 8;
    auto bring = [&](const bf16_t* src, bf16x8* dst) {
        if constexpr (DIRECT)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
        else
            dst[lane] = *reinterpret_cast<const bf16x8_any*>(src);
    };
    int ring[kPf16Ring] = {0, 2 * BP, 4 * BP, 6 * BP, 8 * BP};       // places of blocks blk0, blk0 + 1, ... in pf_lds
    auto request = [&](int blk, int place) {
        bf16x8* dst = pf_lds + place + wave * kWave;
#pragma unroll
        for (int u = 0; u < NL; ++u) bring(kc + ((size_t)blk * BP + u * kPf16Threads) * 8, dst + u * kPf16Threads);
#pragma unroll
        for (int u = 0; u < NL; ++u) bring(vc + ((size_t)blk * BP + u * kPf16Threads) * 8, dst + BP + u * kPf16Threads);
    };
    request(blk_begin, ring[0]);
    if (blk_begin + 1 < blk_end) request(blk_begin + 1, ring[1]);

    bf16x8 qreg[KS];
    int hi_row, lo_row;
    {
        const int r = r0 + lr < rows ? r0 + lr : rows - 1;
        const int i = r / G, qh = r % G;
        hi_row = pf_hi(L + i, m_bidir, total);
        lo_row = pf_lo(L + i, W);
        const bf16_t* qr = p.q + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qr + ks * 32 + lc * 8);
    }
    const bf16x8* const kfrag = pf_lds + lane;                        // operand (t, ks) of a block: 64 pieces in lane order
    const bf16x8* const vfrag = pf_lds + BP + lr * 4 + (lc ^ ((-(lr / 4)) & 3));

    floatx4 acc[NT];
    bf16x8 ka[KS / 2][2];                          // the first half of the next block's keys
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr float kLazy = 8.0f;                  // a row's reference exponent is raised only when exceeded by 2^8

    auto turn = [&]() {
        const int a = ring[0], b = ring[1];
        ring[0] = ring[2]; ring[1] = ring[3]; ring[2] = ring[4]; ring[3] = a; ring[4] = b;
    };
    for (int blk0 = blk_begin; blk0 < blk_end; blk0 += 2, turn()) {
        // these two blocks have landed for every wave (a wave's requests complete in order; the block behind them may still be on
        // its way) and everybody is done with the two before, whose places take the next
        if constexpr (DIRECT) {
            if (blk0 > blk_begin && blk0 + 2 < blk_end) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * NL) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const int first = blk0 > blk_first ? blk0 : blk_first, last = blk0 + 1 < blk_last ? blk0 + 1 : blk_last;
        if (blk0 == blk_begin && blk0 + 2 < blk_end) request(blk0 + 2, ring[2]);
        if (blk0 + 3 < blk_end) request(blk0 + 3, ring[3]);
        if (first >= last && blk0 + 4 < blk_end) request(blk0 + 4, ring[4]);
        if (first > last) continue;
        {
            const bf16x8* kp = kfrag + (first == blk0 ? ring[0] : ring[1]);
#pragma unroll
            for (int ks = 0; ks < KS / 2; ++ks) { ka[ks][0] = kp[ks * 64]; ka[ks][1] = kp[(KS + ks) * 64]; }
        }
        for (int blk = first; blk <= last; ++blk) {
            const bf16x8* kp = kfrag + (blk == blk0 ? ring[0] : ring[1]);
            const bf16x8* vp = vfrag + (blk == blk0 ? ring[0] : ring[1]);
            bf16x8 kb[KS / 2][2];
            floatx4 s[2][2];                       // [keys 8 lc + 4 t + (0..3)][even, odd steps] of row lr
#pragma unroll
            for (int ks = 0; ks < KS / 2; ++ks) { kb[ks][0] = kp[(KS / 2 + ks) * 64]; kb[ks][1] = kp[(KS + KS / 2 + ks) * 64]; }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    s[t][ks % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ks < KS / 2 ? ka[ks % (KS / 2)][t] : kb[ks % (KS / 2)][t], qreg[ks],
                                                                         ks < 2 ? floatx4{0.f, 0.f, 0.f, 0.f} : s[t][ks % 2], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 v0[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) v0[nt] = vp[nt * 64];
            __builtin_amdgcn_s_setprio(1);
            const floatx4 a0 = s[0][0] + s[0][1], a1 = s[1][0] + s[1][1];
            float sv[8] = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
            if ((blk + 1) * kPfBlk > min_hi || blk * kPfBlk < max_lo) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int key = blk * kPfBlk + lc * 8 + e;
                    if (key >= hi_row || key < lo_row) sv[e] = -INFINITY;
                }
                if ((blk + 1) * kPfBlk > total) {  // values of rows past the valid ones may hold anything
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (blk * kPfBlk + lc * 8 + e >= total) v0[nt][e] = (bf16_t)0.f;
                }
            }
            float mx = pf_max3(pf_max3(sv[0], sv[1], sv[2]), pf_max3(sv[3], sv[4], sv[5]), pf_max3(sv[6], sv[7], sv[7]));
            mx *= p.scale_log2;
            if (__any(mx > m_run + kLazy)) {
                mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
                mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
                if (mx > m_run + kLazy) {
                    const float alpha = __builtin_amdgcn_exp2f(m_run - mx);     // m_run = -inf gives 0
                    l_run *= alpha;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[nt] *= alpha;
                    m_run = mx;
                }
            }
            const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
            bf16x8 pv;
            float ps = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(sv[e], p.scale_log2, neg_m));
                ps += pe;
                pv[e] = (bf16_t)pe;
            }
            l_run += ps;
            __builtin_amdgcn_s_setprio(0);
            if (blk < last) {
                if (blk0 + 4 < blk_end) request(blk0 + 4, ring[4]);
                const bf16x8* kn = kfrag + ring[1];
#pragma unroll
                for (int ks = 0; ks < KS / 2; ++ks) { ka[ks][0] = kn[ks * 64]; ka[ks][1] = kn[(KS + ks) * 64]; }
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v0[nt], pv, acc[nt], 0, 0, 0);
            }
        }
    }

    // ---- write this wave's rows: lane holds dims 16 nt + 4 lc + (0..3) of row lr ----
    float l = l_run + __shfl_xor(l_run, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    const int r = r0 + lr;
    if (r >= rows) return;
    const float inv = 1.0f / l;                    // every row sees at least its own key
    const int i = r / G, qh = r % G;
    bf16_t* dst = p.out + (((size_t)b * p.Lq + i) * p.n_q + g * G + qh) * D + lc * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const bf16x4 o = {(bf16_t)(acc[nt][0] * inv), (bf16_t)(acc[nt][1] * inv), (bf16_t)(acc[nt][2] * inv), (bf16_t)(acc[nt][3] * inv)};
        *reinterpret_cast<bf16x4*>(dst + nt * 16) = o;
    }
}

// ---------------------------------------------------------------------------
// fp32: grid (L_q, n_q, B), 256 threads; keys 256 at a time (thread t scores key t, thread c accumulates column c).
// Row-major fp32 keys, blocked values.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256)
void prefill_generic_kernel(const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
                            const int32_t* __restrict__ kv_len, const int32_t* __restrict__ n_new,
                            const int32_t* __restrict__ n_bidir, float* __restrict__ out,
                            int Lq, int n_q, int n_kv, int d, int l_max, float scale, int window) {
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int G = n_q / n_kv, g = h / G;
    const size_t bg = (size_t)b * n_kv + g;
    const int L = cached_rows(kv_len[b], l_max);
    int n = n_new[b]; n = n < 0 ? 0 : (n > Lq ? Lq : n);
    if (L + n > l_max) n = l_max - L > 0 ? l_max - L : 0;
    if (i >= n) return;                                    // uniform over the workgroup
    const int hi = pf_hi(L + i, n_bidir ? n_bidir[b] : 0, L + n), lo = pf_lo(L + i, window);
    __shared__ float qs[256];
    __shared__ float w[256];
    __shared__ float red[4];
    const float* qr = q + (((size_t)b * Lq + i) * n_q + h) * d;
    if (tid < d) qs[tid] = qr[tid];
    __syncthreads();
    float m_run = -INFINITY, l_run = 0.f, acc = 0.f;
    for (int j0 = lo; j0 < hi; j0 += 256) {
        const int j = j0 + tid;
        float s = -INFINITY;
        if (j < hi) {
            const float* kr = kc + (bg * l_max + j) * d;
            float dot = 0.f;
            for (int c = 0; c < d; ++c) dot += qs[c] * kr[c];
            s = dot * scale;
        }
        float mx = wave_max(s);
        if ((tid & 63) == 0) red[tid >> 6] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        const float m_new = fmaxf(m_run, mx);              // finite: key j0 is visible
        const float pe = (j < hi) ? expf(s - m_new) : 0.f;
        w[tid] = pe;
        float ps = wave_sum(pe);
        __syncthreads();
        if ((tid & 63) == 0) red[tid >> 6] = ps;
        __syncthreads();
        ps = red[0] + red[1] + red[2] + red[3];
        const float alpha = expf(m_run - m_new);
        l_run = l_run * alpha + ps;
        acc *= alpha;
        if (tid < d) {
            const int cnt = (hi - j0) < 256 ? (hi - j0) : 256;
            for (int t = 0; t < cnt; ++t) {
                const int jj = j0 + t;
                acc += w[t] * vc[((bg * (size_t)(l_max / kPfBlk) + (size_t)(jj / kPfBlk)) * d + tid) * kPfBlk + (jj % kPfBlk)];
            }
        }
        m_run = m_new;
        __syncthreads();
    }
    if (tid < d) out[(((size_t)b * Lq + i) * n_q + h) * d + tid] = acc / l_run;
}

template <int D>
static int launch_prefill(const massv_attn_desc& a, PrefillParams p, hipStream_t st) {
    const int rows_max = a.n_query * (a.n_q_heads / a.n_kv_heads);
    const int per_wg = kPfWaves * 64;
    p.n_tiles = (rows_max + per_wg - 1) / per_wg;
    if (p.n_tiles > 65535) return MASSV_EUNSUPPORTED;
    launch_traced(MASSV_K_PREFILL_ATTENTION, prefill_attention_kernel<D>, dim3(a.batch * a.n_kv_heads, p.n_tiles),
                  dim3(kPfThreads), 0, st, p);
    return launch_status();
}

template <int D, bool DIRECT, int HALVES>
static int launch_prefill_lds(const massv_attn_desc& a, PrefillParams p, hipStream_t st) {
    // more LDS than a kernel gets by default: the limit is raised once per device
    static std::atomic<bool> ready[64];           // zero-initialised; calls may come from several threads
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MASSV_ELAUNCH;
    if (!ready[dev].load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute((const void*)prefill_attention_lds_kernel<D, DIRECT, HALVES>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                HALVES * (int)pf_lds_bytes(D)) != hipSuccess) return MASSV_ELAUNCH;
        ready[dev].store(true, std::memory_order_release);
    }
    const int rows_max = a.n_query * (a.n_q_heads / a.n_kv_heads);
    const int per_wg = kPfWaves * 32;
    p.n_tiles = (rows_max + per_wg - 1) / per_wg;
    if (p.n_tiles > 65535) return MASSV_EUNSUPPORTED;
    launch_traced(MASSV_K_PREFILL_ATTENTION, prefill_attention_lds_kernel<D, DIRECT, HALVES>, dim3(a.batch * a.n_kv_heads, p.n_tiles),
                  dim3(kPfThreads * HALVES), HALVES * pf_lds_bytes(D), st, p);
    return launch_status();
}
template <int D>
static int launch_prefill_lds(const massv_attn_desc& a, const PrefillParams& p, bool halves, hipStream_t st) {
    const bool direct = ((uintptr_t)p.kc | (uintptr_t)p.vc) % 16 == 0;
    if (D == 128 || halves) return direct ? launch_prefill_lds<D, true, 2>(a, p, st) : launch_prefill_lds<D, false, 2>(a, p, st);
    if constexpr (D == 64) return direct ? launch_prefill_lds<D, true, 1>(a, p, st) : launch_prefill_lds<D, false, 1>(a, p, st);
    return MASSV_EUNSUPPORTED;
}

template <int D, bool DIRECT>
static int launch_prefill16(const massv_attn_desc& a, PrefillParams p, hipStream_t st) {
    constexpr size_t lds = pf16_lds_bytes<D>();
    static std::atomic<bool> ready[64];           // zero-initialised; calls may come from several threads
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MASSV_ELAUNCH;
    if (!ready[dev].load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute((const void*)prefill_attention_rows16_kernel<D, DIRECT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return MASSV_ELAUNCH;
        ready[dev].store(true, std::memory_order_release);
    }
    const int rows_max = a.n_query * (a.n_q_heads / a.n_kv_heads), per_wg = kPf16Waves * 16;
    p.n_tiles = (rows_max + per_wg - 1) / per_wg;
    if (p.n_tiles > 65535) return MASSV_EUNSUPPORTED;
    launch_traced(MASSV_K_PREFILL_ATTENTION, prefill_attention_rows16_kernel<D, DIRECT>, dim3(a.batch * a.n_kv_heads, p.n_tiles),
                  dim3(kPf16Threads), lds, st, p);
    return launch_status();
}
template <int D>
static int launch_prefill16(const massv_attn_desc& a, const PrefillParams& p, hipStream_t st) {
    const bool direct = ((uintptr_t)p.kc | (uintptr_t)p.vc) % 16 == 0;
    return direct ? launch_prefill16<D, true>(a, p, st) : launch_prefill16<D, false>(a, p, st);
}

}  // namespace massv

using namespace massv;

extern "C" int massv_prefill_attention(const massv_attn_desc* desc, const void* q, const void* k_cache,
                                       const void* v_cache, const int32_t* kv_len, const int32_t* n_new,
                                       const int32_t* n_bidir, void* out, void* stream) {
    if (!desc) return MASSV_EINVAL;
    // the descriptor rules of verify_attention, except that the row count per KV head is not limited
    massv_attn_desc one = *desc;
    one.n_query = 1;
    const int rc = check_attn_desc(&one);
    if (rc != MASSV_OK) return rc;
    if (desc->n_query < 1 || desc->n_query > desc->l_max) return MASSV_EINVAL;
    if (!q || !k_cache || !v_cache || !kv_len || !n_new || !out) return MASSV_EINVAL;
    if ((int64_t)desc->batch * desc->n_kv_heads > 0x7fffffff) return MASSV_EUNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    const massv_attn_desc& a = *desc;
    const float scale = a.scale > 0.f ? a.scale : 1.0f / sqrtf((float)a.head_dim);
    if (a.dtype == MASSV_F32) {
        if (a.n_query > 65535) return MASSV_EUNSUPPORTED;
        hipLaunchKernelGGL(prefill_generic_kernel, dim3(a.n_query, a.n_q_heads, a.batch), dim3(256), 0, st,
                           (const float*)q, (const float*)k_cache, (const float*)v_cache, kv_len, n_new, n_bidir,
                           (float*)out, a.n_query, a.n_q_heads, a.n_kv_heads, a.head_dim, a.l_max, scale, a.window);
        return launch_status();
    }
    PrefillParams p;
    p.q = (const bf16_t*)q; p.kc = (const bf16_t*)k_cache; p.vc = (const bf16_t*)v_cache;
    p.kv_len = kv_len; p.n_new = n_new; p.n_bidir = n_bidir;
    p.out = (bf16_t*)out;
    p.Lq = a.n_query; p.n_q = a.n_q_heads; p.n_kv = a.n_kv_heads; p.l_max = a.l_max; p.window = a.window;
    p.n_tiles = 0;
    p.scale_log2 = scale * 1.4426950408889634f;
    // d <= 128: a launch of 32 rows per wave that fits the chip (256 workgroups of 128 rows, their key ranges in two halves) is the faster one,
    // by 1.0 to 1.6: the length of one wave's loop counts there.  Larger ones take 64 rows per wave, with two exceptions.
    // At d = 64 the smaller kernel, in one piece, stays ahead (1.05 to 1.5; its blocks are half as long) while workgroups of 256 rows would
    // fit the chip, unless a window makes them all alike (0.96 to 1.3) or rows are few before a long cache (100 rows on
    // 6000: 0.95).  At d = 128 it does so, in halves, for fresh prompts of up to 512 workgroups, whose many short key ranges fill up
    // what the long ones leave (64 rows a wave and halves: 28 / 4 heads, 4 x 300 20.0 and 14.8 us, 1 x 1500 39.6 and 34.1, 2 x 1000 32.3 and
    // 30.9, 544 workgroups 22.6 and 24.2; 16 / 8 heads, 2 x 2000 61.4 and 47.9, 752 workgroups 89.0 and 95.5; with a cache as long as the
    // prompt or longer 47.2 and 48.9, 62.8 and 70.3).  Over 700 such calls (1 to 8 heads a KV head, 100 to 4000 rows) it is 1.16 times as fast in the median, but
    // with 3 or 4 tiles a pair there are no long ranges to fill up behind: where their workgroups of 256 rows just fit the chip, those took 0.88 to 1.03 of
    // the time (16 heads, 8 x 341 on 82 cached 21.7 and 24.7 us), with 192 of them 1.01 to 1.20.
    const int64_t pairs = (int64_t)a.batch * a.n_kv_heads, rows = (int64_t)a.n_query * (a.n_q_heads / a.n_kv_heads);
    const int64_t wide = pairs * ((rows + kPfWaves * 64 - 1) / (kPfWaves * 64)), tiles = (rows + kPfWaves * 32 - 1) / (kPfWaves * 32);
    const bool banded = a.window > 0 && a.window < a.l_max;
    bool halves = pairs * tiles <= 256;
    if (a.head_dim == 128)
        halves = halves || (!banded && !n_bidir && pairs * tiles <= 512 && (tiles > 4 || wide <= 224) && (a.n_query >= 256 || tiles >= 24) &&
                             (int64_t)a.l_max * 4 <= (int64_t)a.n_query * 5 + 128);
    const bool few = halves || (a.head_dim == 64 && !banded && wide <= 256 && a.l_max / 8 <= a.n_query);
    switch (a.head_dim) {
        case 64: return few ? launch_prefill_lds<64>(a, p, halves, st) : launch_prefill<64>(a, p, st);
        case 128: return few ? launch_prefill_lds<128>(a, p, halves, st) : launch_prefill<128>(a, p, st);
        case 256: return launch_prefill16<256>(a, p, st);
    }
    return MASSV_EUNSUPPORTED;
}
