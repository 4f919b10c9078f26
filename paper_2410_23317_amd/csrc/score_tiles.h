// Tiles of the matrix-core sweeps over the post-vision window (gfx950, v_mfma_f32_32x32x16_bf16):
// operand fragments, K chunk staging through LDS and the accumulator layout, shared by the scoring
// sweeps and the window attention kernel.
#pragma once

#include "common.h"

namespace vlc {
namespace tiles {

constexpr int kD = 128;                 // head dimension of this path
constexpr int kChunk = 128;             // keys per LDS chunk
constexpr int kPitch = kD + 8;          // bf16 elements per LDS row (272 bytes: conflict-free 16-byte reads)
constexpr int kKSteps = kD / 16;        // MFMA k-steps per tile

// Fragment of one operand: lane (l % 32) owns a row (or column) index, lane half l / 32 the
// 8 consecutive k-values [16 ks + 8 half, +8).
__device__ __forceinline__ bf16x8_t as_frag(const uint4& v) { return __builtin_bit_cast(bf16x8_t, v); }

// The 32-row blocks rb0 + STRIDE * rb (rb < RB) of this wave: rows of the KV group's window, a head every tauP of them (tb: packed).
template <int RB, int STRIDE, typename Args>
__device__ __forceinline__ void load_q_frags(const Args& a, int bl, int hkv, int rb0, int lane, int tb, int tauP, uint4 (&qf)[RB][kKSteps]) {
    const int half = lane >> 5;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = (rb0 + STRIDE * rb) * 32 + (lane & 31);
        const int hl = r / tauP, iw = r % tauP;
        const bool ok = hl < a.g && iw < tb;
        const bf16_t* row = a.q_win + (((size_t)bl * a.Hq + (size_t)hkv * a.g + (ok ? hl : 0)) * a.tau + (ok ? iw : 0)) * kD;
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks)
            qf[rb][ks] = ok ? *reinterpret_cast<const uint4*>(row + ks * 16 + half * 8) : make_uint4(0, 0, 0, 0);
    }
}

// A logit is the product times the layer's scale.  The kernels mask (-inf) and take maxima of the products, which stand for
// the logits only where the scale is positive: so Q' takes the scale's sign (exact), and is zero for a scale of zero, where
// every logit is 0.  To be called after a block's first requests are out: the scale is looked at here.
template <int RB>
__device__ __forceinline__ void sign_q_frags(uint4 (&qf)[RB][kKSteps], float scale) {
    uint32_t bits = __float_as_uint(scale);
    asm volatile("" : "+v"(bits) : : "memory");
    bits = __builtin_amdgcn_readfirstlane(bits);
    if ((int)bits > 0) return;                              // block-uniform
    const uint32_t flip = (bits >> 31) * 0x80008000u, keep = bits << 1 ? 0xffffffffu : 0u;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) {
            uint4& q = qf[rb][ks];
            q = make_uint4((q.x ^ flip) & keep, (q.y ^ flip) & keep, (q.z ^ flip) & keep, (q.w ^ flip) & keep);
        }
}
// Scale of the products in the exponent domain, with Q' signed as above.
__device__ __forceinline__ float exp_scale(float scale) { return (scale == 0.f ? 1.f : fabsf(scale)) * kLog2e; }

// Window rows of one head padded to whole 32-row blocks.
__device__ __forceinline__ int padded_rows(int tb) { return (tb + 31) & ~31; }

// K chunk staging: global -> registers -> LDS.  Keys at or beyond m are zero-filled.
template <int THREADS, int CHUNK = kChunk>
struct KStage {
    static constexpr int N = CHUNK * (kD / 8) / THREADS;      // 16-byte pieces per thread
    uint4 r[N];
    __device__ __forceinline__ void load(const bf16_t* kg, int key0, int m) {
        if (key0 + CHUNK <= m) {               // block-uniform: a whole chunk needs no per-row test
            const uint4* src = reinterpret_cast<const uint4*>(kg + (size_t)key0 * kD) + threadIdx.x;
#pragma unroll
            for (int u = 0; u < N; ++u) r[u] = src[THREADS * u];
            return;
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int x = threadIdx.x + THREADS * u;
            const int row = x >> 4, piece = x & 15;
            const int key = key0 + row;
            r[u] = (key < m) ? *reinterpret_cast<const uint4*>(kg + (size_t)key * kD + piece * 8) : make_uint4(0, 0, 0, 0);
        }
    }
    // The same in PARTS instalments (part P fetches pieces [P N / PARTS, (P + 1) N / PARTS)), for callers
    // that spread the requests of a chunk over their compute phases.
    template <int P, int PARTS>
    __device__ __forceinline__ void load_part(const bf16_t* kg, int key0, int m) {
        static_assert(N % PARTS == 0, "pieces per thread must divide evenly");
        const bool whole = key0 + CHUNK <= m;
#pragma unroll
        for (int u = P * (N / PARTS); u < (P + 1) * (N / PARTS); ++u) {
            const int x = threadIdx.x + THREADS * u;
            const int row = x >> 4, piece = x & 15;
            const int key = key0 + row;
            if (whole) r[u] = *reinterpret_cast<const uint4*>(kg + (size_t)key * kD + piece * 8);
            else r[u] = (key < m) ? *reinterpret_cast<const uint4*>(kg + (size_t)key * kD + piece * 8) : make_uint4(0, 0, 0, 0);
        }
    }
    template <int PITCH = kPitch>
    __device__ __forceinline__ void store(bf16_t* sK) const {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int x = threadIdx.x + THREADS * u;
            const int row = x >> 4, piece = x & 15;
            *reinterpret_cast<uint4*>(sK + row * PITCH + piece * 8) = r[u];
        }
    }
};

__device__ __forceinline__ void load_k_frags(const bf16_t* sK, int tile, int lane, uint4 (&kf)[kKSteps]) {
    const bf16_t* row = sK + (tile * 32 + (lane & 31)) * kPitch + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) kf[ks] = *reinterpret_cast<const uint4*>(row + ks * 16);
}

// Row index (0..31) of accumulator element i of a 32x32 MFMA tile in lane `lane`.
__device__ __forceinline__ int acc_row(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

}  // namespace tiles
}  // namespace vlc
