// Scoring sweeps on the matrix cores for bf16 storage with d = 64 and for fp32 storage (gfx950;
// v_mfma_f32_32x32x16_bf16, v_mfma_f32_32x32x2_f32).  bf16 with d = 128 has kernels of its own (score_mfma.hip).
//
// The same two sweeps (App. A.3) with another division of the work: the block's Q' rows are put into LDS once (they
// are few and serve the whole sweep), and every wave walks 32-key tiles of its own, K fragments straight from memory
// into registers, each tile multiplied with all 32-row blocks of the window.  The loop over the keys holds no barrier,
// so the waves of a SIMD drift apart and one's products run under another's exponentials; the next tile's K is
// requested into the same registers as soon as the last row block's products are issued.
// In both sweeps a tile is S^T = K Q'^T: the 16 values a lane holds belong to ONE query row, whose constants are then
// one value per lane.  Sweep 1 keeps each row block's running max and sum in registers, with one rescale per tile.
// Sweep 2 adds into one accumulator per key slot over all row blocks and sums across lanes once per key tile.
// Each head's window rows are padded to a multiple of 32 so that every 32-row block belongs to one query head; the
// blocks of a request are those of its own window length, so a short window in a ragged batch costs what it holds.
// Windows of up to 16 rows (one row where the cache's hit rate is asked for) share a block between heads instead, each
// head padded to a power of two; a row then counts its own entries of Eq. 1.  64 KV groups of 4 heads, 4096 keys, one row,
// both sweeps and sweep 2 alone: the plain ALU 70.5 and 17.5 us, a block per head 85.5 and 42.0, shared 34.8 and 17.5 (fp32,
// d = 64); 121 and 32, 147 and 74.5, 55.1 and 27.1 (fp32, d = 128); 50.3 and 11.8, 25.2 and 12.4, 16.1 and 7.3 (bf16).
//
// What bounds them: at d = 64 in bf16 the vector unit (about 330 issue cycles per tile beside 128 of matrix work), in
// fp32 the matrix cores (64 cycles per instruction and 2 contraction indexes), and for the smallest problems the
// chain of launch, first loads and merge.  Profiled against one thread per key on the plain ALU: bf16, 2 x 24 layers of 16
// (4 KV) heads of 64 over 4096 keys with 50 window rows, 717 + 9 + 417 us -> 56 + 61 us; fp32, 2 layers of 4 (2 KV) heads
// of 64 over 512 keys with 32 rows, 30 + 4 + 31 us -> 11.0 + 7.1 us.  Errors against 64-bit arithmetic are those of the
// plain-ALU sweeps or smaller (logits up to 20: scores 0.8-3e-7 relative, row maxima 0.5-2e-7, row sums 2-8e-7).
#include "common.h"
#include "internal.h"
#include "score_tiles.h"     // acc_row, as_frag

namespace vlc {
namespace {

using tiles::acc_row;

struct SweepArgs {
    const char* q_win;
    const char* k;
    const float* sm_scale;
    float2* part;            // [group][split][g * tau] partial (maximum M of the products, sum relative to 2^offset(M))
    const float* row_max;    // natural-log domain, [B,L,Hq,tau]
    const float* row_sum;    // null: count only
    const float2* part_in;   // sweep 2: partials of sweep 1 to merge in the prologue, or null (statistics given)
    float* row_max_out;      // sweep 2 with part_in: where the merged statistics go ([B,L,Hq,tau]; either may be null)
    float* row_sum_out;
    float* scores;           // may be null
    unsigned long long* nnz; // may be null
    const int32_t* lens;     // per-request (m_b, tau_b), or null
    float log2p, default_scale;
    int L, Hq, Hkv, g, m, tau, keys_per_split, nsplit;
    int head_shift;          // shared blocks: log2 of the rows a head is padded to
    int rb0;                 // first 32-row block of this launch
    int accumulate;          // sweep 2: add to scores instead of overwriting (row groups after the first)
};

// RBYTES: bytes of a Q' or K row.  NRB: most 32-row blocks of a launch.  W: waves per block.  Registers for four waves
// per SIMD: two 8-wave blocks per CU, or one of 16 waves where the Q' rows fill the LDS.  A K tile of 512-byte rows
// takes 64 registers (spills at four waves per SIMD): one 8-wave block per CU, whose matrix instructions (4096
// cycles per tile) need no other wave's help to keep the matrix cores busy.
// SHARED: heads share 32-row blocks (windows of up to 16 rows).
template <bool F32_, int RBYTES_, int NRB_, int W_, bool SHARED_>
struct Form {
    static constexpr bool F32 = F32_, SHARED = SHARED_;
    static constexpr int RBYTES = RBYTES_, NRB = NRB_, W = W_;
    static constexpr int THREADS = W * 64;
    static constexpr int WAVES_PER_SIMD = RBYTES == 512 ? 2 : 4;
    static constexpr int KS = RBYTES / 32;              // 16-byte fragments per lane and row
    static constexpr int PITCH = RBYTES + 16;           // LDS row of Q': 16-byte fragment reads free of bank conflicts
    static constexpr int ROWS = NRB * 32;
    static constexpr int CPR = RBYTES / 16;             // 16-byte pieces of a row
    static constexpr int NQ = ROWS * CPR / THREADS;     // pieces of Q' per thread
    static_assert(ROWS * CPR % THREADS == 0 && ROWS <= THREADS, "staging and statistics in whole passes");
};

// A layer's logit scale, its magnitude (1 if it is zero), and that in the exponent domain.
struct LogitScale { float given, mag, c; };
__device__ __forceinline__ LogitScale logit_scale(const SweepArgs& a, int l) {
    LogitScale s;
    s.given = a.sm_scale ? a.sm_scale[l] : a.default_scale;
    s.mag = s.given == 0.f ? 1.f : fabsf(s.given);
    s.c = s.mag * kLog2e;
    return s;
}

// PACKED (sweep 1): the heads' rows follow each other, a block may hold rows of several heads.  A parameter of the code, not of the launch:
// looked at there, it cost every launch of a window that takes several 0.5 to 1 us (8 KV groups of 500 keys, 7 heads of 40 rows in
// fp32, d = 128: four launches, 112.2 -> 118.5).
// What the blocks of one (request, layer, KV head) share.
struct Where {
    int hkv, bl, l, mb, tb, nb, nrb;        // nb: 32-row blocks per head, nrb: row blocks of this launch
    int k_begin, k_end, nt;                 // key range of the split, its 32-key tiles
    LogitScale ls;
};
template <typename F, bool PACKED>
__device__ __forceinline__ Where locate(const SweepArgs& a, int group, int split) {
    Where w;
    w.hkv = group % a.Hkv; w.bl = group / a.Hkv; w.l = w.bl % a.L;
    const ReqLen rl = request_len(a.lens, w.bl / a.L, a.m, a.tau);
    w.mb = rl.m; w.tb = rl.tau;                             // this request's prompt and window length
    w.nb = (w.tb + 31) >> 5;
    w.nrb = F::SHARED ? ((a.g << a.head_shift) + 31) >> 5 : PACKED ? (a.g * w.tb + 31) >> 5 : min(a.g * w.nb - a.rb0, F::NRB);
    w.k_begin = split * a.keys_per_split;
    w.k_end = min(w.mb, w.k_begin + a.keys_per_split);
    w.nt = w.k_end > w.k_begin ? (w.k_end - w.k_begin + 31) >> 5 : 0;
    w.ls = logit_scale(a, w.l);
    return w;
}

// Exponent offset of a row whose largest product is m: rounded by itself, so that the same maximum gives the same number
// everywhere (fused into a subtraction it would be another).
__device__ __forceinline__ float exp_offset(float m, float c) {
    float o = m * c;
    asm("" : "+v"(o));
    return o;
}
// Row statistics as the caller sees them.  A row's maximum is a rounded number, and exponents are measured from another
// rounded number, its offset; at logits of a few hundred the two differ by 1e-5.  So the row sum that is handed out belongs to the
// maximum that is handed out, and what rounding the offset of a given maximum leaves over goes into its row's factor: fp32, d = 128,
// logits up to 123, scores from vlc_score's own statistics 8.1e-7 off -> 3.3e-7, as its scores are.
__device__ __forceinline__ double exponent_per_logit(const LogitScale& s) {      // c as rounded over the scale's magnitude
    return (double)kLog2e + (double)(fmaf(-s.mag, kLog2e, s.c) / s.mag);
}
__device__ __forceinline__ float exp2_rest(float a, double b) { return fabsf(a) < INFINITY ? exp2_fast((float)((double)a - b)) : 1.f; }

// Row r of the launch's row blocks: its head, its window row, and whether it exists.
struct Row { int hl, iw; bool real; };
template <typename F, bool PACKED>
__device__ __forceinline__ Row window_row(const SweepArgs& a, const Where& w, int r) {
    Row o;
    if (F::SHARED) {
        o.hl = r >> a.head_shift;
        o.iw = r - (o.hl << a.head_shift);
        o.real = o.hl < a.g && o.iw < w.tb;
        return o;
    }
    if (PACKED) {
        o.hl = r / w.tb;
        o.iw = r - o.hl * w.tb;
        o.real = o.hl < a.g;
        return o;
    }
    const int rb = a.rb0 + (r >> 5);
    o.hl = rb / w.nb;
    o.iw = (rb - o.hl * w.nb) * 32 + (r & 31);
    o.real = (r >> 5) < w.nrb && o.iw < w.tb;
    return o;
}
// Window row of this lane's row in block `rb` (counted from its head's first, where the head has blocks of its own).
template <typename F>
__device__ __forceinline__ int lane_row(const SweepArgs& a, int rb, int lane) {
    return F::SHARED ? lane & ((1 << a.head_shift) - 1) : rb * 32 + (lane & 31);
}

// K fragments of the 32-key tile that starts at key0: lane l % 32 owns a key, lane half l / 32 the 16-byte pieces
// 2 s + half.  Keys beyond the prompt read its last row (the causal mask drops them), so nothing past it is touched.
template <int KS, int RBYTES>
__device__ __forceinline__ void load_keys(const char* kg, int key0, int mb, int lane, uint4 (&kf)[KS]) {
    const char* base = kg + (size_t)key0 * RBYTES;          // wave-uniform
    const uint32_t off = (uint32_t)min(lane & 31, mb - 1 - key0) * RBYTES + (lane >> 5) * 16;
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = *reinterpret_cast<const uint4*>(base + off + s * 32);
}

// The block's Q' rows into LDS.  A row that does not exist takes the values of a row that does, its head's last one (which sees every
// key) or, with packed rows, one of the last head's, whose statistics nobody keeps:
// its products are then the numbers of a row that exists, and drop out by an exponent of -inf (zeros would not: times a
// key's infinite entry they are NaN).  All requests of a thread are in flight together.
template <typename F, bool PACKED>
__device__ __forceinline__ void stage_q(const SweepArgs& a, const Where& w, char* sQ) {
    uint4 q[F::NQ];
#pragma unroll
    for (int u = 0; u < F::NQ; ++u) {
        const int x = threadIdx.x + F::THREADS * u, r = x / F::CPR;
        const Row o = window_row<F, PACKED>(a, w, r);
        const char* src = a.q_win + (((size_t)w.bl * a.Hq + (size_t)w.hkv * a.g + min(o.hl, a.g - 1)) * a.tau + min(o.iw, w.tb - 1)) * F::RBYTES;
        q[u] = *reinterpret_cast<const uint4*>(src + (x % F::CPR) * 16);
    }
    // A logit is the product times the layer's scale.  The sweeps mask (-inf) and take maxima of the products, which
    // stand for the logits only where the scale is positive: so Q' takes the scale's sign (exact), and is zero for a
    // scale of zero, where every logit is 0.  (The scale is first looked at here: a wait for it in front of the
    // requests above costs a small sweep 0.4 us of 9.)
    uint32_t scale = __float_as_uint(w.ls.given);
    asm volatile("" : "+s"(scale) : : "memory");
    const uint32_t flip = (scale >> 31) * (F::F32 ? 0x80000000u : 0x80008000u), keep = scale << 1 ? 0xffffffffu : 0u;
#pragma unroll
    for (int u = 0; u < F::NQ; ++u) {
        const int x = threadIdx.x + F::THREADS * u;
        *reinterpret_cast<uint4*>(sQ + (x / F::CPR) * F::PITCH + (x % F::CPR) * 16) =
            make_uint4((q[u].x ^ flip) & keep, (q[u].y ^ flip) & keep, (q[u].z ^ flip) & keep, (q[u].w ^ flip) & keep);
    }
}

// acc[i] = <key, row>: key acc_row(i, lane) of the tile, window row lane % 32 of row block rb.
template <typename F>
__device__ __forceinline__ f32x16_t tile_product(const char* sQ, int rb, int lane, const uint4 (&kf)[F::KS]) {
    const char* row = sQ + (rb * 32 + (lane & 31)) * F::PITCH + (lane >> 5) * 16;
    f32x16_t acc = {0};
#pragma unroll
    for (int s = 0; s < F::KS; ++s) {
        const uint4 q = *reinterpret_cast<const uint4*>(row + s * 32);
        if constexpr (F::F32) {
            // a lane half supplies one of the two contraction indexes of an instruction: element e of its 16-byte piece
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf[s].x), __uint_as_float(q.x), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf[s].y), __uint_as_float(q.y), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf[s].z), __uint_as_float(q.z), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(kf[s].w), __uint_as_float(q.w), acc, 0, 0, 0);
        } else {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tiles::as_frag(kf[s]), tiles::as_frag(q), acc, 0, 0, 0);
        }
    }
    return acc;
}

// ------------------------------------------------------------------------------------------------
// Sweep 1: partial row statistics of one key range of one KV group.
template <typename F, bool PACKED>
__global__ __launch_bounds__(F::THREADS, F::WAVES_PER_SIMD) void rowstats_wave_kernel(SweepArgs a) {
    constexpr int RBYTES = F::RBYTES, NRB = F::NRB, W = F::W, KS = F::KS;
    constexpr int QBYTES = F::ROWS * F::PITCH, MBYTES = W * F::ROWS * (int)sizeof(float2);
    __shared__ __align__(16) char smem[QBYTES > MBYTES ? QBYTES : MBYTES];      // Q' rows; after the sweep the waves' statistics
    const int group = blockIdx.x, split = blockIdx.y;       // group-major: see the launch
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;     // wave index in a scalar register
    const Where w = locate<F, PACKED>(a, group, split);
    if (a.nnz && split == 0 && a.rb0 == 0 && (int)threadIdx.x < a.g)
        a.nnz[(size_t)w.bl * a.Hq + (size_t)w.hkv * a.g + threadIdx.x] = 0;      // sweep 2 adds into these
    if (w.nrb <= 0) return;                                 // a shorter window than the longest of the batch
    const char* kg = a.k + (size_t)group * a.m * RBYTES;
    uint4 kf[KS];
    if (wave < w.nt) load_keys<KS, RBYTES>(kg, w.k_begin + wave * 32, w.mb, lane, kf);
    stage_q<F, PACKED>(a, w, smem);
    __syncthreads();
    float m_run[NRB], z_run[NRB];                           // this lane's row of each row block, over the keys its half holds
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) { m_run[rb] = -INFINITY; z_run[rb] = 0.f; }
#pragma unroll 1
    for (int t = wave; t < w.nt; t += W) {
        const int key0 = w.k_begin + t * 32;
        const bool masked = key0 + 32 > w.mb - w.tb + 1;    // the tile reaches past the first window key
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            if (rb < w.nrb) {                               // wave-uniform
                const f32x16_t acc = tile_product<F>(smem, rb, lane, kf);
                if (rb == w.nrb - 1 && t + W < w.nt) load_keys<KS, RBYTES>(kg, key0 + W * 32, w.mb, lane, kf);
                float v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = acc[i];
                if (masked) {                               // last key this lane's row may see (causal mask of Alg. 1)
                    int rbg = a.rb0 + rb;
                    asm volatile("" : "+s"(rbg));           // computed here: hoisted, the limits of all row blocks would take registers
                    const int iw = PACKED ? (rbg * 32 + (lane & 31)) % w.tb : lane_row<F>(a, rbg % w.nb, lane);
                    const int jlim = min(w.mb - w.tb + iw, w.mb - 1) - key0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = acc_row(i, lane) <= jlim ? v[i] : -INFINITY;
                }
                float tmax = v[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, v[i]);
                const float m_new = fmaxf(m_run[rb], tmax);
                const float m_use = m_new > -INFINITY ? exp_offset(m_new, w.ls.c) : 0.f;     // a row that has seen no key yet: every term is 0
                float zs = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) zs += exp2_fast(fmaf(v[i], w.ls.c, -m_use));
                z_run[rb] = z_run[rb] * exp2_fast(exp_offset(m_run[rb], w.ls.c) - m_use) + zs;
                m_run[rb] = m_new;
            }
        }
    }
    // the two lane halves hold disjoint keys of the same rows, the waves disjoint tiles
    __syncthreads();                                        // Q' is no longer read
    float2* sStat = reinterpret_cast<float2*>(smem);        // [W][ROWS]
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        const float mo = __shfl_xor(m_run[rb], 32, 64), zo = __shfl_xor(z_run[rb], 32, 64);
        const float mm = fmaxf(m_run[rb], mo), om = exp_offset(mm, w.ls.c);
        float z = 0.f;
        if (m_run[rb] > -INFINITY) z += z_run[rb] * exp2_fast(exp_offset(m_run[rb], w.ls.c) - om);
        if (mo > -INFINITY) z += zo * exp2_fast(exp_offset(mo, w.ls.c) - om);
        if (lane < 32) sStat[wave * F::ROWS + rb * 32 + lane] = make_float2(mm, z);
    }
    __syncthreads();
    const int r = threadIdx.x;
    const Row o = window_row<F, PACKED>(a, w, r);
    if (r < F::ROWS && o.real) {
        float M = -INFINITY, Z = 0.f;
#pragma unroll
        for (int v = 0; v < W; ++v) M = fmaxf(M, sStat[v * F::ROWS + r].x);
#pragma unroll
        for (int v = 0; v < W; ++v) {
            const float2 s = sStat[v * F::ROWS + r];
            if (s.x > -INFINITY) Z += s.y * exp2_fast(exp_offset(s.x, w.ls.c) - exp_offset(M, w.ls.c));
        }
        a.part[((size_t)group * a.nsplit + split) * a.g * a.tau + o.hl * a.tau + o.iw] = make_float2(M, Z);
    }
}

// Merge of sweep 1's key splits where they are too many for sweep 2's prologue: a wave per window row, a split per lane.
__global__ __launch_bounds__(256) void merge_splits_kernel(SweepArgs a, int rows) {
    const int x = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (x >= rows) return;                                  // wave-uniform; no barrier below
    const int per_group = a.g * a.tau, group = x / per_group, r = x % per_group;
    const int hkv = group % a.Hkv, bl = group / a.Hkv, hl = r / a.tau, iw = r % a.tau;
    if (iw >= request_len(a.lens, bl / a.L, a.m, a.tau).tau) return;
    const LogitScale ls = logit_scale(a, bl % a.L);
    const float2* p = a.part + (size_t)group * a.nsplit * per_group + r;
    float M = -INFINITY;
    for (int sp = lane; sp < a.nsplit; sp += 64) M = fmaxf(M, p[(size_t)sp * per_group].x);
    M = wave_allreduce_max(M);
    const float off = exp_offset(M, ls.c);
    float Z = 0.f;
    for (int sp = lane; sp < a.nsplit; sp += 64) {
        const float2 s = p[(size_t)sp * per_group];
        if (s.x > -INFINITY) Z += s.y * exp2_fast(exp_offset(s.x, ls.c) - off);
    }
    Z = wave_allreduce_sum(Z);
    if (lane == 0) {
        const size_t o = ((size_t)bl * a.Hq + (size_t)hkv * a.g + hl) * a.tau + iw;
        const float row_max = M * ls.mag;
        a.row_max_out[o] = row_max;
        a.row_sum_out[o] = Z * exp2_rest(off, (double)row_max * exponent_per_logit(ls));
    }
}

// ------------------------------------------------------------------------------------------------
// Sweep 2: column sums of the softmax over all window rows of the KV group, and per-head counts.
template <typename F>
__global__ __launch_bounds__(F::THREADS, F::WAVES_PER_SIMD) void colsweep_wave_kernel(SweepArgs a) {
    constexpr int RBYTES = F::RBYTES, W = F::W, KS = F::KS;
    __shared__ __align__(16) char sQ[F::ROWS * F::PITCH];
    __shared__ float2 sConst[F::ROWS];                      // per row: exponent offset (+inf for rows that do not exist), 1 / row sum
    __shared__ uint32_t sCnt[8];                            // Eq. 1 entries per query head of the group
    __shared__ uint32_t sRow[F::SHARED ? F::ROWS : 1];      // shared blocks: per row
    const int group = blockIdx.x, split = blockIdx.y;       // group-major: see the launch
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;     // wave index in a scalar register
    const Where w = locate<F, false>(a, group, split);
    if (w.nrb <= 0) return;
    const char* kg = a.k + (size_t)group * a.m * RBYTES;
    // Order of the first requests: the few bytes of the statistics go out first (every block of the launch starts at
    // once, and behind the K bursts they would wait), then the first K tile, then Q'.
    const Row o = window_row<F, false>(a, w, (int)threadIdx.x);
    const bool mine = (int)threadIdx.x < F::ROWS && o.real;
    constexpr int kSplitRegs = 4;                           // splits whose partials a thread holds at once (more are merged in rounds)
    float2 pin[kSplitRegs];
    const float2* pp = a.part_in + (size_t)group * a.nsplit * a.g * a.tau + o.hl * a.tau + o.iw;
    const size_t split_stride = (size_t)a.g * a.tau;
    if (mine && a.part_in) {
#pragma unroll
        for (int sp = 0; sp < kSplitRegs; ++sp) pin[sp] = sp < a.nsplit ? pp[sp * split_stride] : make_float2(-INFINITY, 0.f);
    }
    uint4 kf[KS];
    if (wave < w.nt) load_keys<KS, RBYTES>(kg, w.k_begin + wave * 32, w.mb, lane, kf);
    stage_q<F, false>(a, w, sQ);
    if (threadIdx.x < 8) sCnt[threadIdx.x] = 0;
    if (F::SHARED && (int)threadIdx.x < F::ROWS) sRow[threadIdx.x] = 0;
    if ((int)threadIdx.x < F::ROWS) {
        float2 st = make_float2(INFINITY, 0.f);
        const size_t x = ((size_t)w.bl * a.Hq + (size_t)w.hkv * a.g + o.hl) * a.tau + o.iw;
        if (mine && a.part_in) {
            // merge of the key splits of sweep 1; the block of the first split also writes the row maximum and sum
            // the caller asked for (either may be absent: a count-only sweep keeps no row sums)
            float M = -INFINITY, Z = 0.f;
            for (int sp0 = 0; sp0 < a.nsplit; sp0 += kSplitRegs) {
                if (sp0 > 0) {
#pragma unroll
                    for (int sp = 0; sp < kSplitRegs; ++sp) pin[sp] = sp0 + sp < a.nsplit ? pp[(sp0 + sp) * split_stride] : make_float2(-INFINITY, 0.f);
                }
                float Mn = M;
#pragma unroll
                for (int sp = 0; sp < kSplitRegs; ++sp) Mn = fmaxf(Mn, pin[sp].x);
                if (Mn > -INFINITY) {
                    const float on = exp_offset(Mn, w.ls.c);
                    Z *= exp2_fast(exp_offset(M, w.ls.c) - on);            // 0 on the first round (M = -inf)
#pragma unroll
                    for (int sp = 0; sp < kSplitRegs; ++sp)
                        if (pin[sp].x > -INFINITY) Z += pin[sp].y * exp2_fast(exp_offset(pin[sp].x, w.ls.c) - on);
                    M = Mn;
                }
            }
            const float off = exp_offset(M, w.ls.c);
            st = make_float2(off, 1.f / Z);
            if (split == 0) {
                const float row_max = M * w.ls.mag;
                if (a.row_max_out) a.row_max_out[x] = row_max;
                if (a.row_sum_out) a.row_sum_out[x] = Z * exp2_rest(off, (double)row_max * exponent_per_logit(w.ls));
            }
        } else if (mine) {
            const double offset = (double)a.row_max[x] * exponent_per_logit(w.ls);
            st = make_float2((float)offset, a.row_sum ? exp2_rest((float)offset, offset) / a.row_sum[x] : 0.f);
        }
        sConst[threadIdx.x] = st;
    }
    __syncthreads();
    const int j_first = a.rb0 % w.nb, h_first = a.rb0 / w.nb;
#pragma unroll 1
    for (int t = wave; t < w.nt; t += W) {
        const int key0 = w.k_begin + t * 32;
        const bool masked = key0 + 32 > w.mb - w.tb + 1;    // the tile reaches past the first window key
        float col[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) col[i] = 0.f;
        uint32_t cnt = 0;                                   // wave-wide, on the scalar unit (shared blocks: per lane)
        int j = j_first, hl = h_first;                      // block within its head, head
#pragma unroll 1
        for (int rb = 0; rb < w.nrb; ++rb) {
            const float2 rc = sConst[rb * 32 + (lane & 31)];
            const f32x16_t acc = tile_product<F>(sQ, rb, lane, kf);
            if (rb == w.nrb - 1 && t + W < w.nt) load_keys<KS, RBYTES>(kg, key0 + W * 32, w.mb, lane, kf);
            float ea[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) ea[i] = fmaf(acc[i], w.ls.c, -rc.x);
            if (masked) {
                const int jlim = min(w.mb - w.tb + lane_row<F>(a, j, lane), w.mb - 1) - key0;
#pragma unroll
                for (int i = 0; i < 16; ++i) ea[i] = acc_row(i, lane) <= jlim ? ea[i] : -INFINITY;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                col[i] = fmaf(exp2_fast(ea[i]), rc.y, col[i]);
                if (F::SHARED) cnt += ea[i] >= a.log2p ? 1u : 0u;         // this lane's row
                else cnt += (uint32_t)__popcll(__ballot(ea[i] >= a.log2p));
            }
            if (F::SHARED) {
                if (a.nnz && cnt) atomicAdd(&sRow[rb * 32 + (lane & 31)], cnt);
                cnt = 0;
            } else if (++j == w.nb || rb == w.nrb - 1) {           // last block of its head here
                if (a.nnz && lane == 0 && cnt) atomicAdd(&sCnt[hl], cnt);
                cnt = 0; j = 0; ++hl;
            }
        }
        if (!a.scores) continue;
        // Sum over the 32 rows each lane half holds: v_permlane16_swap halves 16 slots to 8 (lane row 0 of a half keeps
        // slots 0..7, row 1 slots 8..15), the row reduce-scatter leaves one slot per lane pair.
        float h8[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const auto s2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(col[i]), __float_as_uint(col[i + 8]), false, false);
            h8[i] = __uint_as_float(s2[0]) + __uint_as_float(s2[1]);
        }
        const float tot = row16_reduce_scatter8<8>(h8, lane & 15);
        const int slot = ((lane >> 1) & 1) + ((lane >> 2) & 1) * 2 + ((lane >> 3) & 1) * 4 + ((lane >> 4) & 1) * 8;
        const int key = key0 + acc_row(slot, lane);
        if ((lane & 1) == 0 && key < w.k_end) {
            float* dst = a.scores + (size_t)group * a.m + key;
            *dst = a.accumulate ? *dst + tot : tot;
        }
    }
    // keys of the padded prompt beyond this request's own length score zero
    if (a.scores && a.lens && !a.accumulate) {
        const int z_end = min(a.m, w.k_begin + a.keys_per_split);
        for (int x = max(w.k_begin, w.mb) + (int)threadIdx.x; x < z_end; x += F::THREADS) a.scores[(size_t)group * a.m + x] = 0.f;
    }
    if (a.nnz) {
        __syncthreads();
        if (F::SHARED) {
            if (mine && sRow[threadIdx.x]) atomicAdd(&sCnt[o.hl], sRow[threadIdx.x]);
            __syncthreads();
        }
        if ((int)threadIdx.x < a.g && sCnt[threadIdx.x])
            atomicAdd(a.nnz + (size_t)w.bl * a.Hq + (size_t)w.hkv * a.g + threadIdx.x, (unsigned long long)sCnt[threadIdx.x]);
    }
}

int row_bytes(const vlc_shape& s) { return s.d * (s.dtype == VLC_F32 ? 4 : 2); }
int max_row_blocks(const vlc_shape& s) { return row_bytes(s) == 512 ? 8 : 16; }       // per launch: what fits the LDS

struct Plan {
    int nrb, nsplit, keys_per_split;        // splits of sweep 1, whose partial statistics sweep 2 merges
    int keys_per_split2;    // of sweep 2
    int head_shift;         // < 0: every head has row blocks of its own
    bool merge_apart;       // sweep 1's splits are merged by a kernel of their own, not in sweep 2's prologue
};

Plan make_plan(const vlc_shape& s) {
    Plan p;
    const int g = s.Hq / s.Hkv;
    p.head_shift = s.tau <= 16 ? 0 : -1;
    if (s.tau <= 16) {
        while (1 << p.head_shift < s.tau) ++p.head_shift;
        p.nrb = ((g << p.head_shift) + 31) / 32;
    } else {
        p.nrb = g * ((s.tau + 31) / 32);
    }
    const int64_t groups = (int64_t)s.B * s.L * s.Hkv;
    const int tiles = s.m / 32 + (s.m % 32 != 0);
    const int nrb = p.nrb < max_row_blocks(s) ? p.nrb : max_row_blocks(s);
    const bool wide = row_bytes(s) == 256 && nrb > 8;                      // see launch_sweep
    const int W = wide ? 16 : 8, resident = wide || row_bytes(s) == 512 ? 256 : 512;      // blocks that 256 CUs hold at once
    // Splits of the key range per KV group: the number with the least modelled time, in units of one key tile per
    // wave -- rounds of resident blocks, each as long as its fullest wave plus a prologue (Q' into LDS, statistics:
    // about 3 us, where a tile costs a wave about 1 us per row block).  At most one split per 256 keys and 32 in all:
    // the partial statistics then never need more than those of the plain-ALU sweep of the same shape (one per 256 keys).
    const double prologue = 3.0 / nrb;
    double best = 0.0;
    int ns = 1;
    const int top256 = s.m / 256 + (s.m % 256 != 0), top = top256 < 32 ? top256 : 32;
    for (int n = 1; n <= top; ++n) {
        const int tps = (tiles + n - 1) / n;
        const double cost = (double)((groups * n + resident - 1) / resident) * ((tps + W - 1) / W + prologue);
        if (n == 1 || cost < best * 0.999) { best = cost; ns = n; }
    }
    // Fewer than 8 KV groups leave CUs idle at 32 splits: then as many as give every CU a block, and where that is more than
    // a prologue should merge, a kernel merges them.  Plain-ALU sweeps, 32 splits, now, both sweeps and sweep 2 alone: one
    // group of 8 heads, 65536 keys, 50 rows, fp32 d = 64 394 and 171 us, 547 and 274, 93 and 42; d = 128 685 and 317, 1033
    // and 525, 167 and 78; bf16 383 and 161, 134 and 75, 37 and 15.  4 heads, 16384 keys, 32 rows, fp32 d = 64 106 and 54, 49 and
    // 23, 28 and 9.  (7 groups of 20000 keys still take 32: 63 and 30.)
    p.merge_apart = false;
    if (groups < 8) {
        const int n = top256 < 256 / (int)groups ? top256 : 256 / (int)groups;
        if (n > 32) { ns = n; p.merge_apart = true; }
    }
    const int tps = (tiles + ns - 1) / ns;
    p.keys_per_split = tps * 32;
    p.nsplit = (tiles + tps - 1) / tps;
    // Sweep 2 leaves no partials: while CUs are idle its splits may be as short as 4 tiles, one per SIMD (fp32, 4 groups of
    // 2 heads of 64 over 512 keys, 32 rows: 9.0 -> 6.3 us; 16 of 2 heads of 128 over 2048 keys, 33 rows: 22.5 -> 13.6).
    p.keys_per_split2 = p.keys_per_split;
    const int n2 = groups < 256 ? 256 / (int)groups : 1, tps2 = (tiles + n2 - 1) / n2 > 4 ? (tiles + n2 - 1) / n2 : 4;
    if (tps2 < tps) p.keys_per_split2 = tps2 * 32;
    return p;
}

SweepArgs make_args(const ScoreArgs& a, const Plan& p) {
    SweepArgs m;
    const vlc_shape& s = a.s;
    m.q_win = (const char*)a.q_win; m.k = (const char*)a.k; m.sm_scale = a.sm_scale;
    m.part = (float2*)a.workspace;
    m.row_max = a.row_max; m.row_sum = a.row_sum;
    m.part_in = nullptr; m.row_max_out = a.row_max; m.row_sum_out = a.row_sum;
    m.scores = a.scores; m.nnz = (unsigned long long*)a.nnz;
    m.log2p = log2f(a.p); m.default_scale = 1.0f / sqrtf((float)s.d);
    m.lens = s.lens;
    m.L = s.L; m.Hq = s.Hq; m.Hkv = s.Hkv; m.g = s.Hq / s.Hkv; m.m = s.m; m.tau = s.tau;
    m.keys_per_split = p.keys_per_split; m.nsplit = p.nsplit;
    m.head_shift = p.head_shift;
    m.rb0 = 0; m.accumulate = 0;
    return m;
}

template <bool SWEEP1, bool F32, int RBYTES, int NRB, int W, bool SHARED = false>
void launch_form(const SweepArgs& m, bool packed, dim3 grid, hipStream_t st) {
    using F = Form<F32, RBYTES, NRB, W, SHARED>;
    if (!SWEEP1) colsweep_wave_kernel<F><<<grid, F::THREADS, 0, st>>>(m);
    else if (!SHARED && packed) rowstats_wave_kernel<F, !SHARED><<<grid, F::THREADS, 0, st>>>(m);
    else rowstats_wave_kernel<F, false><<<grid, F::THREADS, 0, st>>>(m);
}

// Windows of more row blocks than a launch holds take several launches over consecutive row-block ranges.  Group-major
// grid: blocks go to the 8 XCDs round-robin by linear index, so with a multiple of 8 KV groups the key splits of a
// group run on one XCD and share its Q' rows in that XCD's L2.
template <bool SWEEP1>
hipError_t launch_sweep(SweepArgs m, const Plan& p, const vlc_shape& s, hipStream_t st) {
    m.keys_per_split = SWEEP1 ? p.keys_per_split : p.keys_per_split2;
    const dim3 grid(s.B * s.L * s.Hkv, s.m / m.keys_per_split + (s.m % m.keys_per_split != 0));
    const int step = max_row_blocks(s);
    // Sweep 1 of a window that one launch holds: a lane owns a row whatever block it is in, so the heads' rows may follow each
    // other (with the form, and with it each row's order of additions, chosen as for blocks of one head).  192 KV groups of 4096
    // keys, 4 heads of 50 rows of 64 in bf16, 7 blocks instead of 8: a
    // whole compression 152.1 -> 146.5 us.
    const bool packed = SWEEP1 && p.head_shift < 0 && p.nrb <= step;
    for (int rb0 = 0; rb0 < p.nrb; rb0 += step) {
        const int nrb = p.nrb - rb0 < step ? p.nrb - rb0 : step;
        m.rb0 = rb0;
        m.accumulate = rb0 > 0;                 // launches of one stream run in order: the column sums add up deterministically
        if (p.head_shift >= 0) {                // at most 8 heads of 16 rows
            if (s.dtype == VLC_F32 && s.d == 128) launch_form<SWEEP1, true, 512, 4, 8, true>(m, packed, grid, st);
            else if (s.dtype == VLC_F32) launch_form<SWEEP1, true, 256, 4, 8, true>(m, packed, grid, st);
            else launch_form<SWEEP1, false, 128, 4, 8, true>(m, packed, grid, st);
        } else if (s.dtype == VLC_F32 && s.d == 128) {
            if (nrb <= 4) launch_form<SWEEP1, true, 512, 4, 8>(m, packed, grid, st);
            else launch_form<SWEEP1, true, 512, 8, 8>(m, packed, grid, st);
        } else if (s.dtype == VLC_F32) {
            if (nrb <= 4) launch_form<SWEEP1, true, 256, 4, 8>(m, packed, grid, st);
            else if (nrb <= 8) launch_form<SWEEP1, true, 256, 8, 8>(m, packed, grid, st);
            else launch_form<SWEEP1, true, 256, 16, 16>(m, packed, grid, st);
        } else {
            if (nrb <= 4) launch_form<SWEEP1, false, 128, 4, 8>(m, packed, grid, st);
            else if (nrb <= 8) launch_form<SWEEP1, false, 128, 8, 8>(m, packed, grid, st);
            else launch_form<SWEEP1, false, 128, 16, 8>(m, packed, grid, st);
        }
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rowstats_wave(const ScoreArgs& a) {
    const Plan p = make_plan(a.s);
    const SweepArgs m = make_args(a, p);
    const hipError_t e = launch_sweep<true>(m, p, a.s, a.stream);
    if (e != hipSuccess || !p.merge_apart) return e;
    const int rows = a.s.B * a.s.L * a.s.Hq * a.s.tau;
    merge_splits_kernel<<<(rows + 3) / 4, 256, 0, a.stream>>>(m, rows);
    return hipGetLastError();
}

hipError_t launch_colsweep_wave(const ScoreArgs& a, bool merge_partials) {
    const Plan p = make_plan(a.s);
    SweepArgs m = make_args(a, p);
    if (merge_partials && !p.merge_apart) m.part_in = m.part;          // sweep 1 ran just before on the same workspace
    return launch_sweep<false>(m, p, a.s, a.stream);
}

}  // namespace vlc
