// Matrix-core scoring sweeps for bf16 storage (gfx950, v_mfma_f32_32x32x16_bf16).
//
// The post-vision window Q' K^T of Alg. 1 is the one dense contraction of the path: per KV head a
// (g * tau) x d x m product.  Following the two-sweep schedule of the paper's App. A.3, neither
// the logits nor the attention matrix reach HBM:
//   sweep 1 (row statistics) computes S^T = K Q'^T tile by tile, so that the 16 values a lane holds
//           belong to ONE query row: running max and sum stay in the lane, with one rescale per
//           32-key tile instead of one per element;
//   sweep 2 (column sums + ThresholdFilter counts) first merges sweep 1's per-split statistics for its own rows,
//           then computes S = Q' K^T, so that a lane holds 16
//           query rows of ONE key: the sum over the window rows of Sec. 3.2 is in-lane too, and the
//           Eq. 1 test is one compare on the exponent argument.
// Q' fragments of a block's rows live in registers for the whole sweep; K streams through LDS in
// chunks of 32 to 128 keys (global -> registers -> LDS, the next chunk in flight while the current one is
// multiplied).  Sweep 1 packs the window rows of the group's heads into 32-row blocks one after the other (a lane
// owns a row whatever block it is in, so the statistics have the same bits).  In sweep 2 each head's tau rows are padded to a
// multiple of 32 so that every 32-row block belongs to one query head, and its sums keep their order; padded rows carry a
// +inf offset and vanish from every sum, and groups of eight rows that are all padding are left out where that pays (SKIP; the
// exponentials are what costs power here, and power bounds both sweeps).  256 KV groups of 131072 keys, 4 heads of 50 rows (7 blocks instead of
// 8, 7 of 8 row groups): both sweeps 5990 -> 5600 us; 8 ragged requests of up to 100 rows 1325 -> 1270.
// In a ragged batch the blocks are those of the request's own window length, dealt to the waves from the first on (and
// round-robin where a wave takes two), so a shorter window costs the blocks it holds: the waves beyond it only
// help to stage K; in large batches whose longest window takes the 16-block forms, requests of up to 8 blocks get a launch
// of their own.
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "score_tiles.h"

namespace vlc {
namespace {

using namespace tiles;

struct MfmaArgs {
    const bf16_t* q_win;
    const bf16_t* k;
    const float* sm_scale;
    float2* part;            // [group][split][RP] partial (max, sum), exponent domain (log2)
    const float* row_max;    // natural-log domain, [B,L,Hq,tau]
    const float2* part_in;   // sweep 2: partials of sweep 1 to merge in the prologue, or null (statistics given)
    float* row_max_out;      // sweep 2 with part_in: where the merged statistics go ([B,L,Hq,tau]; either may be null)
    float* row_sum_out;
    const float* row_sum;
    float* scores;           // may be null
    unsigned long long* nnz; // may be null
    const int32_t* lens;     // per-request (m_b, tau_b), or null
    float log2p;
    int L, Hq, Hkv, g, m, tau, RP, keys_per_split, nsplit;     // RP: padded window rows of a KV group, for the longest window
    int rb0;                 // first 32-row block of this launch (a launch covers at most 16 of them)
    int rb_above, rb_upto;   // requests of this launch: those with more than rb_above row blocks from rb0 on, and at most rb_upto
    int accumulate;          // sweep 2: add to scores instead of overwriting (row groups after the first)
};

// Whether a launch takes the requests with so many 32-row blocks per KV group (block-uniform).
__device__ __forceinline__ bool in_class(const MfmaArgs& a, int row_blocks) {
    const int nrb = row_blocks - a.rb0;
    return nrb > a.rb_above && nrb <= a.rb_upto;
}

// ------------------------------------------------------------------------------------------------
// Sweep 1: partial row statistics of one key range of one KV group.
// CHUNK: keys staged at once.  Small chunks start a block sooner, and their registers (16 for 128 keys) make room for a third
// 8-wave block per CU.  Chunks of 128 / 64 / 32 keys, profiled: 4 waves (256 KV groups of 2944 keys, 128 rows) 41 / 38 / 35 us,
// 8 waves (1024 groups of 10368, 256 rows) 934 / 905 / 818, (256 of 131072, 200 rows) 2512 / 2450 / 2350.  Two LDS buffers and
// one barrier per chunk instead: 37.3, 853, 2389.  64 keys in two places, 64 / 32 keys: up
// to three row blocks in several rounds whose last one six blocks per CU leave the emptier of the two (1024 groups of 10368 keys, 2048
// blocks, one row block 451 / 485, three 482 / 527; 1920 of 10000, 3840 blocks, 838 / 847, 868 / 877; but 768 of 20000, 1536
// blocks, 716 / 638, and four row blocks 931 / 893); and two row blocks per wave over more than 8192 keys (256 groups of 100000,
// 512 rows 3680 / 3770, 64 of 100000 923 / 944).
// Two row blocks per wave: a K fragment is used for both as it arrives, instead of all eight fragments of a tile being held
// while one block's chain of products runs and then the other's.  That fits the registers of two blocks per CU: (1920 groups
// of 10368 keys, 448 rows) 2943 -> 2720 us, (ragged, up to 400 rows) 485 -> 377; within the old registers 3250 and 503.
// For up to 8 row blocks one per wave stays the better: 830 against 930, 2460 against 2550 with two in blocks of 4 waves.
template <int WAVES, int RB, int CHUNK>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 3 : RB == 1 ? 6 : 4) void rowstats_mfma_kernel(MfmaArgs a) {   // 4-wave blocks: registers for 3 blocks per CU, accumulators stay out of the AGPRs
    constexpr int THREADS = WAVES * 64;
    __shared__ __align__(16) bf16_t sK[CHUNK * kPitch];
    const int group = blockIdx.x, split = blockIdx.y;       // group-major: see the launch
    const int hkv = group % a.Hkv, bl = group / a.Hkv, l = bl % a.L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;     // wave index in a scalar register
    const float scale = a.sm_scale ? a.sm_scale[l] : rsqrtf((float)kD), c = exp_scale(scale);
    const bf16_t* kg = a.k + (size_t)group * a.m * kD;
    const ReqLen rl = request_len(a.lens, bl / a.L, a.m, a.tau);
    const int mb = rl.m, tb = rl.tau;                       // this request's prompt and window length
    const int R = a.g * tb;                                 // window rows of its KV groups, head after head
    const int k_begin = split * a.keys_per_split;
    const int k_end = min(mb, k_begin + a.keys_per_split);

    if (a.nnz && split == 0 && a.rb0 == 0 && (int)threadIdx.x < a.g)
        a.nnz[(size_t)bl * a.Hq + (size_t)hkv * a.g + threadIdx.x] = 0;      // sweep 2 adds into these
    if (!in_class(a, (R + 31) / 32)) return;                // this request's window is another launch's work
    uint4 qf[RB][kKSteps];
    load_q_frags<RB, WAVES>(a, bl, hkv, a.rb0 + wave, lane, tb, tb, qf);        // row blocks rb0 + wave + WAVES * rb
    // this lane's query row per row block, and the last key it may see (causal mask of Alg. 1)
    int jlim[RB];
    float m_run[RB], z_run[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = (a.rb0 + wave + WAVES * rb) * 32 + (lane & 31);
        jlim[rb] = mb - tb + (r % tb);
        m_run[rb] = -INFINITY;
        z_run[rb] = 0.f;
    }

    KStage<THREADS, CHUNK> st;
    if (k_begin < k_end) st.load(kg, k_begin, mb);
    sign_q_frags(qf, scale);
    for (int kc = k_begin; kc < k_end; kc += CHUNK) {
        __syncthreads();                                   // previous chunk fully consumed
        st.store(sK);
        __syncthreads();
        if (kc + CHUNK < k_end) st.load(kg, kc + CHUNK, mb);
        const bool masked = kc + CHUNK > mb - tb + 1;     // chunk reaches past the first window key
#pragma unroll 1
        for (int t = 0; t < CHUNK / 32; ++t) {
            if (kc + t * 32 >= k_end) break;
            uint4 kf[kKSteps];
            f32x16_t accs[RB];
            if constexpr (RB == 1) {
                load_k_frags(sK, t, lane, kf);
            } else {
                const bf16_t* row = sK + (t * 32 + (lane & 31)) * kPitch + (lane >> 5) * 8;
                auto products = [&](auto countc) {              // of this wave's first row blocks
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks) {
                        const uint4 k1 = *reinterpret_cast<const uint4*>(row + ks * 16);
#pragma unroll
                        for (int rb = 0; rb < decltype(countc)::value; ++rb)
                            accs[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(k1), as_frag(qf[rb][ks]), accs[rb], 0, 0, 0);
                    }
                };
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) accs[rb] = f32x16_t{0};
                if ((a.rb0 + wave + WAVES * (RB - 1)) * 32 < R) products(std::integral_constant<int, RB>{});     // wave-uniform
                else if ((a.rb0 + wave) * 32 < R) products(std::integral_constant<int, 1>{});
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if ((a.rb0 + wave + WAVES * rb) * 32 >= R) continue;        // wave-uniform: no rows here
                f32x16_t acc = {0};
                if constexpr (RB > 1) acc = accs[rb];
                else
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(kf[ks]), as_frag(qf[rb][ks]), acc, 0, 0, 0);
                // acc[i] = <k_key, q_row>, key = kc + 32 t + acc_row(i), row = this lane's
                float v[16];
                if (masked) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = (kc + t * 32 + acc_row(i, lane) <= jlim[rb]) ? acc[i] : -INFINITY;
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = acc[i];
                }
                float tmax = v[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, v[i]);
                const float m_new = fmaxf(m_run[rb], tmax * c);
                if (m_new > -INFINITY) {
                    float zs = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) zs += exp2_fast(fmaf(v[i], c, -m_new));
                    z_run[rb] = z_run[rb] * exp2_fast(m_run[rb] - m_new) + zs;
                    m_run[rb] = m_new;
                }
            }
        }
    }
    // the two lane halves hold disjoint keys of the same query row
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float mo = __shfl_xor(m_run[rb], 32, 64), zo = __shfl_xor(z_run[rb], 32, 64);
        const float mm = fmaxf(m_run[rb], mo);
        float z = 0.f;
        if (m_run[rb] > -INFINITY) z += z_run[rb] * exp2_fast(m_run[rb] - mm);
        if (mo > -INFINITY) z += zo * exp2_fast(mo - mm);
        const int r = (a.rb0 + wave + WAVES * rb) * 32 + (lane & 31);
        if (lane < 32 && r < R) a.part[((size_t)group * a.nsplit + split) * a.RP + r] = make_float2(mm, z);
    }
}

// ------------------------------------------------------------------------------------------------
// Sweep 2: column sums of the softmax over all window rows of the KV group, and per-head counts.
// CHUNK as above, but every chunk ends in a sum over the waves: for 128 / 64 / 32 keys 8 waves 933 / 970 / 995, 2795 / 3060 / 3300
// us, 16 waves 3100 / 3180 for 128 / 64.  4 waves: three blocks of 128 keys or four of 64 fit a CU, and the
// launch of several rounds takes the form whose rounds are the fuller; in one round short splits gain by the earlier start of 64
// keys (256 groups of 2944 keys, 1024 per split, 36.3 / 35.8 / 36.9 us, four row blocks 46.3 / 44.4 / 46.8).  In brackets, blocks; one row block: 352 groups of 38432 keys (1056) 758 / 882 / 947,
// 768 of 20000 (1536) 795 / 878 / 930, 256 of 100000 (768) 1307 / 1296 / 1364, 1920 of 10000 (3840) 985 / 999 / 1047, 1024 of 10368 (2048)
// 535 / 528 / 557, 512 of 4096 (1024) 120 / 104 / 108, 2048 of 1000 (2048) 118 / 109 / 114; of four row blocks 834 / 904 / 993,
// 833 / 852 / 962, 1375 / 1428 / 1536, 1057 / 1044 / 1096, 582 / 575 / 607, 153 / 122 / 124, 147 / 130 / 130.
// SKIP: row groups of padding are left out.  16 waves with / without: 352 groups of 38432 keys, 8 heads of 64 rows 2610 / 2546 us, 1920
// of 10000, 7 heads of 64 rows 3072 / 3030, 256 of 10368, 8 heads of 50 rows 416 / 410, of 40 rows 399 / 391; but 8 ragged requests of up to
// 100 rows, where whole windows are short, a compression 1534 / 1541.
template <int WAVES, int RB, int CHUNK, bool SKIP>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 3 : 4) void colsweep_mfma_kernel(MfmaArgs a) {   // waves per SIMD: 2 blocks of 8 waves, or 3 of 4
    constexpr int THREADS = WAVES * 64;
    __shared__ __align__(16) bf16_t sK[CHUNK * kPitch];
    __shared__ float sCol[WAVES][CHUNK];
    const int group = blockIdx.x, split = blockIdx.y;       // group-major: see the launch
    const int hkv = group % a.Hkv, bl = group / a.Hkv, l = bl % a.L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;     // wave index in a scalar register
    const float scale = a.sm_scale ? a.sm_scale[l] : rsqrtf((float)kD), c = exp_scale(scale);
    const bf16_t* kg = a.k + (size_t)group * a.m * kD;
    const ReqLen rl = request_len(a.lens, bl / a.L, a.m, a.tau);
    const int mb = rl.m, tb = rl.tau;                       // this request's prompt and window length
    const int tauP = padded_rows(tb), RP = a.g * tauP;      // and its padded rows, the launch's (a.RP) or fewer
    if (!in_class(a, RP / 32)) return;                      // this request's window is another launch's work
    const int k_begin = split * a.keys_per_split;
    const int k_end = min(mb, k_begin + a.keys_per_split);

    // Order of the first requests: the few bytes of sweep 1's partial statistics go out first (every block of the
    // launch starts at once, and behind 32 KB of K per block they would wait for the whole burst), then the first
    // K chunk, then the Q' fragments; the merge of the statistics and its barrier run while K is on its way.
    constexpr int kSplitRegs = 4;               // splits whose partials a thread holds at once (more are merged in rounds)
    float2 pin[kSplitRegs];
    const int r_mine = a.rb0 * 32 + (int)threadIdx.x;       // the row whose statistics this thread merges (first round)
    const bool mine = a.part_in && (int)threadIdx.x < WAVES * RB * 32 && r_mine < RP && r_mine % tauP < tb;
    if (mine) {
        const int at = r_mine / tauP * tb + r_mine % tauP;  // sweep 1 packs the heads' rows
#pragma unroll
        for (int sp = 0; sp < kSplitRegs; ++sp)
            pin[sp] = sp < a.nsplit ? a.part_in[((size_t)group * a.nsplit + sp) * a.RP + at] : make_float2(-INFINITY, 0.f);
    }
    KStage<THREADS, CHUNK> st;
    if (k_begin < k_end) st.load(kg, k_begin, mb);
    uint4 qf[RB][kKSteps];
    load_q_frags<RB, WAVES>(a, bl, hkv, a.rb0 + wave, lane, tb, tauP, qf);      // row blocks rb0 + wave + WAVES * rb
    sign_q_frags(qf, scale);
    // per accumulator slot: exponent offset (+inf for padded rows) and 1 / row sum
    float mc[RB][16], iz[RB][16];
    uint32_t cnt[RB];
    __shared__ __align__(16) float2 sStat[WAVES * RB * 32];
    if (a.part_in) {
        // the partial statistics of sweep 1's key splits are merged here, one thread per row of the block; the
        // block of the first split also writes the row maximum and sum the caller asked for
        for (int t = threadIdx.x; t < WAVES * RB * 32; t += THREADS) {
            const int r = a.rb0 * 32 + t;
            float2 st = make_float2(INFINITY, 0.f);
            const int hl = r / tauP, iw = r % tauP;
            if (r < RP && hl < a.g && iw < tb) {
                float M = -INFINITY, Z = 0.f;
                for (int sp0 = 0; sp0 < a.nsplit; sp0 += kSplitRegs) {
                    if (sp0 > 0 || t != (int)threadIdx.x) {          // beyond what was requested at the start
#pragma unroll
                        for (int sp = 0; sp < kSplitRegs; ++sp)
                            pin[sp] = sp0 + sp < a.nsplit ? a.part_in[((size_t)group * a.nsplit + sp0 + sp) * a.RP + hl * tb + iw] : make_float2(-INFINITY, 0.f);
                    }
                    float Mn = M;
#pragma unroll
                    for (int sp = 0; sp < kSplitRegs; ++sp) Mn = fmaxf(Mn, pin[sp].x);
                    if (Mn > -INFINITY) {
                        Z *= exp2_fast(M - Mn);                       // 0 on the first round (M = -inf)
#pragma unroll
                        for (int sp = 0; sp < kSplitRegs; ++sp)
                            if (pin[sp].x > -INFINITY) Z += pin[sp].y * exp2_fast(pin[sp].x - Mn);
                        M = Mn;
                    }
                }
                st = make_float2(M, 1.f / Z);
                if (split == 0) {                  // either output may be absent (a count-only sweep keeps no row sums)
                    const size_t o = ((size_t)bl * a.Hq + (size_t)hkv * a.g + hl) * a.tau + iw;
                    if (a.row_max_out) a.row_max_out[o] = M * kLn2;
                    if (a.row_sum_out) a.row_sum_out[o] = Z;
                }
            }
            sStat[t] = st;
        }
        __syncthreads();
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        cnt[rb] = 0;
        if (a.part_in) {
            const float2* sp = sStat + (wave + WAVES * rb) * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 lo = *reinterpret_cast<const float4*>(sp + 8 * q);
                const float4 hi = *reinterpret_cast<const float4*>(sp + 8 * q + 2);
                mc[rb][4 * q] = lo.x; iz[rb][4 * q] = lo.y; mc[rb][4 * q + 1] = lo.z; iz[rb][4 * q + 1] = lo.w;
                mc[rb][4 * q + 2] = hi.x; iz[rb][4 * q + 2] = hi.y; mc[rb][4 * q + 3] = hi.z; iz[rb][4 * q + 3] = hi.w;
            }
            continue;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = (a.rb0 + wave + WAVES * rb) * 32 + acc_row(i, lane);
            const int hl = r / tauP, iw = r % tauP;
            const bool ok = hl < a.g && iw < tb;
            const size_t o = ((size_t)bl * a.Hq + (size_t)hkv * a.g + (ok ? hl : 0)) * a.tau + (ok ? iw : 0);
            mc[rb][i] = ok ? a.row_max[o] * kLog2e : INFINITY;
            iz[rb][i] = (ok && a.row_sum) ? 1.f / a.row_sum[o] : 0.f;
        }
    }

    for (int kc = k_begin; kc < k_end; kc += CHUNK) {
        // no barrier in front of the store: the one that follows the tiles of the previous chunk (below) already
        // orders every wave's reads of sK before it, and the readers of sCol pass the barrier after the store
        // before any wave writes sCol again
        st.store(sK);
        __syncthreads();
        if (kc + CHUNK < k_end) st.load(kg, kc + CHUNK, mb);
        const bool masked = kc + CHUNK > mb - tb + 1;
#pragma unroll 1
        for (int t = 0; t < CHUNK / 32; ++t) {
            uint4 kf[kKSteps];
            load_k_frags(sK, t, lane, kf);
            const int key = kc + t * 32 + (lane & 31);          // this lane's key (column of the tile)
            float col = 0.f;
            auto add = [&](float product, int rb, int i) {
                const float ea = fmaf(product, c, -mc[rb][i]);
                col = fmaf(exp2_fast(ea), iz[rb][i], col);
                cnt[rb] += (uint32_t)__popcll(__ballot(ea >= a.log2p));   // wave-wide count on the scalar unit
            };
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int base = (a.rb0 + wave + WAVES * rb) * 32;
                if (base >= RP) continue;
                const int rows = tb - base % tauP;          // of the block that exist: the rest adds nothing, eight rows at a time
                f32x16_t acc = {0};
#pragma unroll
                for (int ks = 0; ks < kKSteps; ++ks)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(qf[rb][ks]), as_frag(kf[ks]), acc, 0, 0, 0);
                // acc[i] = <q_row, k_key>, row = row block base + acc_row(i), key = this lane's
                if (masked) {
                    const int last = mb - tb + base % tauP;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const bool valid = key <= last + acc_row(i, lane);
                        const float ea = fmaf(acc[i], c, -mc[rb][i]);
                        const float e = valid ? exp2_fast(ea) : 0.f;
                        col = fmaf(e, iz[rb][i], col);
                        cnt[rb] += (uint32_t)__popcll(__ballot(valid && ea >= a.log2p));
                    }
                } else if (!SKIP || rows > 24) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) add(acc[i], rb, i);
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (8 * q < rows) {                 // wave-uniform
#pragma unroll
                            for (int i = 4 * q; i < 4 * q + 4; ++i) add(acc[i], rb, i);
                        }
                }
            }
            {   // the lane halves hold different rows of the same key: lane l + lane l ^ 32, with the lane-swap
                // instruction rather than a shuffle through the LDS queue
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(col), __float_as_uint(col), false, false);
                col = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
            if (lane < 32) sCol[wave][t * 32 + lane] = col;
        }
        __syncthreads();
        if (a.scores && threadIdx.x < CHUNK && kc + threadIdx.x < k_end) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += sCol[w][threadIdx.x];
            float* dst = a.scores + (size_t)group * a.m + kc + threadIdx.x;
            *dst = a.accumulate ? *dst + s : s;
        }
    }
    // keys of the padded prompt beyond this request's own length score zero
    if (a.scores && a.lens) {
        const int z_end = min(a.m, k_begin + a.keys_per_split);
        for (int j = max(k_begin, mb) + (int)threadIdx.x; j < z_end; j += THREADS) a.scores[(size_t)group * a.m + j] = 0.f;
    }
    if (a.nnz) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int rbase = (a.rb0 + wave + WAVES * rb) * 32;
            if (rbase >= RP) continue;
            const uint32_t tot = cnt[rb];                        // already a wave-wide count
            const int hl = rbase / tauP;
            if (lane == 0 && tot && hl < a.g)
                atomicAdd(a.nnz + (size_t)bl * a.Hq + (size_t)hkv * a.g + hl, (unsigned long long)tot);
        }
    }
}

struct Plan { int RP, nsplit, keys_per_split; };

constexpr int kMaxRowBlocksPerLaunch = 16;      // 512 padded window rows per KV head and launch

Plan make_plan(const vlc_shape& s) {
    Plan p;
    const int g = s.Hq / s.Hkv;
    p.RP = g * ((s.tau + 31) / 32 * 32);
    const int groups = s.B * s.L * s.Hkv;
    const int chunks = (s.m + kChunk - 1) / kChunk;
    // Splits of the key range per KV group.  Measured on the 7B and 34B shapes: about one resident
    // round of blocks (768 four-wave blocks fit the chip) beats finer splits, whose per-block
    // prologue (Q' fragments, row statistics) is not hidden; with a thousand or more groups two
    // splits even out the last round.
    int ns = (768 + groups - 1) / groups;
    if (ns == 1 && chunks >= 16) ns = 2;
    if (ns > chunks) ns = chunks;
    if (ns < 1) ns = 1;
    const int cps = (chunks + ns - 1) / ns;
    p.keys_per_split = cps * kChunk;
    p.nsplit = (s.m + p.keys_per_split - 1) / p.keys_per_split;
    return p;
}

MfmaArgs make_args(const ScoreArgs& a, const Plan& p) {
    MfmaArgs m;
    const vlc_shape& s = a.s;
    m.q_win = (const bf16_t*)a.q_win; m.k = (const bf16_t*)a.k; m.sm_scale = a.sm_scale;
    m.part = (float2*)a.workspace;
    m.row_max = a.row_max; m.row_sum = a.row_sum;
    m.part_in = nullptr; m.row_max_out = a.row_max; m.row_sum_out = a.row_sum;
    m.scores = a.scores; m.nnz = (unsigned long long*)a.nnz;
    m.log2p = log2f(a.p);
    m.lens = s.lens;
    m.L = s.L; m.Hq = s.Hq; m.Hkv = s.Hkv; m.g = s.Hq / s.Hkv; m.m = s.m; m.tau = s.tau;
    m.RP = p.RP; m.keys_per_split = p.keys_per_split; m.nsplit = p.nsplit;
    m.rb0 = 0; m.accumulate = 0; m.rb_above = 0; m.rb_upto = INT32_MAX;
    return m;
}

size_t part_bytes(const vlc_shape& s, const Plan& p) {
    return ((size_t)s.B * s.L * s.Hkv * p.nsplit * p.RP * sizeof(float2) + 255) / 256 * 256;
}

}  // namespace

bool score_mfma_supported(const vlc_shape& s) {
    return s.dtype == VLC_BF16 && s.d == kD;
}

size_t score_mfma_workspace_bytes(const vlc_shape& s) {
    if (!score_mfma_supported(s)) return 0;
    return part_bytes(s, make_plan(s));
}

// How full a launch's rounds of resident blocks are, with so many of them per CU.
constexpr int kCUs = 256;
double round_fill(int64_t blocks, int per_cu) {
    const int64_t round = (int64_t)per_cu * kCUs;
    return (double)blocks / (double)((blocks + round - 1) / round * round);
}

// A launch covers up to 16 row blocks (32 padded window rows each) of every KV group; longer windows
// take several launches over consecutive row-block ranges.  Block shape by row blocks in the launch:
// up to 4 -> 4 waves, up to 8 -> 8 waves, else 8 waves x 2 row blocks (sweep 1) or 16 waves (sweep 2).
// A request with a shorter window than the longest computes its own row blocks only.  Where the longest window of a ragged
// batch takes the last forms, requests of up to 8 row blocks may also have a launch of the 8-wave form for themselves (the
// blocks of the other class leave at once): in 16-wave blocks half of the waves would idle.  The windows lie on the
// device, so a launch may turn out empty, and two launches one after the other need enough blocks each to fill the chip.
// Both sweeps, 7B heads, 100 window rows, one launch -> two: 2048 KV groups of 4099 keys, all windows long 2650 -> 2662 us,
// every other a third 2270 -> 2181, all but one 1738 -> 1524; 1024 groups of 2100 keys 761 -> 766, 684 -> 681, 537 -> 478;
// 512 of 1000 204 -> 207, 197 -> 202, 157 -> 154; 256 of 4099 343 -> 357, 303 -> 337, 232 -> 281; 8 of 300 22 -> 27, 22 -> 27,
// 22 -> 37.  And where prompts are short, blocks that leave at once cost as much as what they leave: 2048 groups of 300
// keys 363 -> 375, 301 -> 304, 211 -> 184; of 1000 744 -> 743, 634 -> 627, 488 -> 424.  So from 1024 groups and 1000 keys on.
bool launch_per_class(const vlc_shape& s) { return s.lens && s.B * s.L * s.Hkv >= 1024 && s.m >= 1000; }

hipError_t launch_rowstats_mfma(const ScoreArgs& a) {
    const vlc_shape& s = a.s;
    const Plan p = make_plan(s);
    MfmaArgs m = make_args(a, p);
    const int groups = s.B * s.L * s.Hkv;
    // Group-major grid: blocks go to the 8 XCDs round-robin by linear index, so with a multiple of 8 KV groups the key
    // splits of a group run on one XCD and share its Q' rows in that XCD's L2 (cfg1: 44.7 -> 42.3 us, sweep 2
    // 49.5 -> 45.5 us; no change for shapes whose splits are dispatched rounds apart).
    dim3 grid(groups, p.nsplit);
    const int64_t blocks = (int64_t)groups * p.nsplit;
    const int total_rb = (m.g * s.tau + 31) / 32;           // the heads' rows are packed
    for (int rb0 = 0; rb0 < total_rb; rb0 += kMaxRowBlocksPerLaunch) {
        const int nrb = total_rb - rb0 < kMaxRowBlocksPerLaunch ? total_rb - rb0 : kMaxRowBlocksPerLaunch;
        m.rb0 = rb0; m.rb_above = 0;
        if (nrb <= 3 && blocks > 6 * kCUs && round_fill(blocks, 5) > round_fill(blocks, 6)) rowstats_mfma_kernel<4, 1, 64><<<grid, 256, 0, a.stream>>>(m);
        else if (nrb <= 4) rowstats_mfma_kernel<4, 1, 32><<<grid, 256, 0, a.stream>>>(m);
        else if (nrb <= 8) rowstats_mfma_kernel<8, 1, 32><<<grid, 512, 0, a.stream>>>(m);
        else {
            if (launch_per_class(s)) {          // the requests with short windows in the form for them
                m.rb_upto = 8;
                rowstats_mfma_kernel<8, 1, 32><<<grid, 512, 0, a.stream>>>(m);
                m.rb_above = 8; m.rb_upto = INT32_MAX;
            }
            // two row blocks per wave: measured faster than 16 x 1 for this sweep
            if (p.keys_per_split > 8192) rowstats_mfma_kernel<8, 2, 64><<<grid, 512, 0, a.stream>>>(m);
            else rowstats_mfma_kernel<8, 2, 32><<<grid, 512, 0, a.stream>>>(m);
        }
    }
    return hipGetLastError();
}

hipError_t launch_colsweep_mfma(const ScoreArgs& a, bool merge_partials) {
    const vlc_shape& s = a.s;
    const Plan p = make_plan(s);
    MfmaArgs m = make_args(a, p);
    if (merge_partials) m.part_in = m.part;          // sweep 1 ran just before on the same workspace
    dim3 grid(s.B * s.L * s.Hkv, p.nsplit);       // group-major, as in sweep 1
    const int64_t blocks = (int64_t)s.B * s.L * s.Hkv * p.nsplit;
    const bool small_chunks = blocks <= 3 * kCUs ? p.keys_per_split <= 2048 : round_fill(blocks, 4) > round_fill(blocks, 3);
    const int total_rb = p.RP / 32;
    for (int rb0 = 0; rb0 < total_rb; rb0 += kMaxRowBlocksPerLaunch) {
        const int nrb = total_rb - rb0 < kMaxRowBlocksPerLaunch ? total_rb - rb0 : kMaxRowBlocksPerLaunch;
        m.rb0 = rb0; m.rb_above = 0;
        m.accumulate = rb0 > 0;                 // launches of one stream run in order: the column sums add up deterministically
        if (nrb <= 4 && small_chunks) colsweep_mfma_kernel<4, 1, 64, true><<<grid, 256, 0, a.stream>>>(m);
        else if (nrb <= 4) colsweep_mfma_kernel<4, 1, kChunk, true><<<grid, 256, 0, a.stream>>>(m);
        else if (nrb <= 8) colsweep_mfma_kernel<8, 1, kChunk, true><<<grid, 512, 0, a.stream>>>(m);
        else {
            if (launch_per_class(s)) {
                m.rb_upto = 8;
                colsweep_mfma_kernel<8, 1, kChunk, true><<<grid, 512, 0, a.stream>>>(m);
                m.rb_above = 8; m.rb_upto = INT32_MAX;
            }
            if (s.lens) colsweep_mfma_kernel<16, 1, kChunk, true><<<grid, 1024, 0, a.stream>>>(m);
            else colsweep_mfma_kernel<16, 1, kChunk, false><<<grid, 1024, 0, a.stream>>>(m);
        }
    }
    return hipGetLastError();
}

}  // namespace vlc
