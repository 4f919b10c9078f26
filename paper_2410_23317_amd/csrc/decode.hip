// GQA decode attention over the compressed, ragged per-layer cache (paper Sec. 2.1, decoding
// phase: the new key/value is appended, then softmax(q K^T / sqrt d) V over every cached slot).
//
// Bandwidth-bound: every K and V row is read once and serves all g query heads of its KV group.
// Rows are ragged (layer budgets differ by 25x), so the work is cut into block-units of 128 to 2048
// slots listed in device-side work lists that vlc_topk_compact builds; a call launches one block per
// unit of the slice of a list that belongs to its layer range.  Inside a block-unit the tiles of 32 slots
// are dealt round-robin to the 4 waves, both products of a tile run on the matrix cores (bf16 and FP8 caches; the
// vector unit for fp32 storage, see the tiles below) and the 4 waves merge through LDS.  A row that spans several
// block-units leaves unnormalised partials in scratch; the unit that finishes last (device-scope counter) merges
// them.  The partials and the counter are only ever touched with device-scope accesses, which are coherent across
// the XCDs' L2 caches by themselves, so no cache-wide release/acquire fence is needed (those cost tens of
// microseconds here).
// What bounds a launch: large ones the memory (about 5 TB/s); a launch over one layer is a chain of dependent steps, timed
// with shader-clock stamps on the 7B shape (rows of 50 to 700 slots, 5.7 us per launch): 1.2 us between two launches, 0.5
// until the unit's record is there, 0.6 to 1 to request a tile (a CU takes 64 bytes per clock of a load), 1 until it is
// multiplied, 0.6 merge of the waves, 0.9 partial acknowledged and counted, 1.0 merge of the row.
//
// Nothing that changes from step to step is a launch parameter: the number of appends a layer has
// received is read from the cache (dev.appended), and the launch that appends leaves count + 1 behind.
// Every block takes a ticket (dev.readers) once each of its waves has read the count (a barrier stands between the reads and
// the ticket, which one thread takes); the block that holds the last ticket of the launch knows that every wave of every
// block that holds a unit has read the count and writes the new one.
// A HIP graph that holds one decode step can therefore be replayed step after step.
#include <float.h>
#include <stddef.h>
#include <stdlib.h>

#include <type_traits>

#include "common.h"
#include "internal.h"

namespace vlc {
namespace {

struct DecodeParams {
    const void* q;
    const void* k_new;
    const void* v_new;
    void* out;
    const float* sm_scale;   // [L], or null: default_scale for every layer
    const WorkItem* heads;   // launches over one layer: copies of its first records (of kHeadUnits), else null
    WorkList wl;             // the work list this launch walks
    // of the cache, as in CacheDev
    const int32_t* kept;
    const int64_t* slot_off;
    int32_t* appended;
    char* kv;
    int32_t* readers;
    int32_t* counters;
    float* partials;
    int32_t* idx;
    float* scales;
    int32_t* status;
    int ub_shift, us_shift;  // log2 of the list's unit sizes
    int part_shift;          // log2 of the slots that a row has a partial for
    int B, L, Hq, Hkv, m;
    int layer_begin, n_layers, T_max;
    int append_mode;         // 0: attend only; 1: k_new / v_new are appended by this kernel
    int merge_mode;          // 1: last unit of a row merges in-kernel; 2: separate merge kernel
    int zigzag;              // 1 off; 2: tile order within a unit alternates between steps; 3: also the walk over the whole units
    int kv_fp8;              // the cache rows are E4M3 codes with per-row scales
    float default_scale;
};

constexpr int pad_pow2(int g) { return g <= 1 ? 1 : (g <= 2 ? 2 : (g <= 4 ? 4 : 8)); }

__device__ __forceinline__ void store_agent(int32_t* p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// two neighbouring floats (8-byte aligned) as one device-scope store
__device__ __forceinline__ void store_agent2(float* p, float a, float b) {
    const unsigned long long v = ((unsigned long long)__float_as_uint(b) << 32) | __float_as_uint(a);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// two neighbouring output elements as one store
__device__ __forceinline__ void store_pair(float* p, float a, float b) { *reinterpret_cast<float2*>(p) = make_float2(a, b); }
__device__ __forceinline__ void store_pair(bf16_t* p, float a, float b) {
    *reinterpret_cast<uint32_t*>(p) = (uint32_t)f32_to_bf16_bits(a) | ((uint32_t)f32_to_bf16_bits(b) << 16);
}
__device__ __forceinline__ int32_t add_agent(int32_t* p, int32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Place of a row's first partial result: a row owns a partial for every 1 << shift slots of its slab, and one more.
// (Rows follow each other in the slot order, so the ranges of two rows never meet, whatever the unit sizes.)
__device__ __forceinline__ int64_t first_partial(int64_t idx_base, int row_abs, int shift) { return (idx_base >> shift) + row_abs; }

// 1 / l and o / l as the outputs of type T want them: to the last bit where they keep 32, and by v_rcp_f32, which is within an
// ulp of that, where they are rounded to bf16.
template <typename T> struct Quotient;
template <> struct Quotient<float> {
    float l;
    __device__ __forceinline__ explicit Quotient(float sum) : l(sum) {}
    __device__ __forceinline__ float operator()(float o) const { return o / l; }
};
template <> struct Quotient<bf16_t> {
    float inv;
    __device__ __forceinline__ explicit Quotient(float sum) : inv(__builtin_amdgcn_rcpf(sum)) {}
    __device__ __forceinline__ float operator()(float o) const { return o * inv; }
};

// Merge the nu partials of one row, one element per thread.
template <typename T, int D, int G, int THREADS>
__device__ __forceinline__ void merge_partials(const float* part, T* outp, int nu, int tid) {
    for (int x = tid; x < G * D; x += THREADS) {
        const float* p = part;
        const int ml = G * D + (x / D) * 2;
        float mt = -INFINITY, o = 0.f, lt = 0.f;
        for (int u = 0; u < nu; ++u, p += partial_floats(G, D)) {
            const float mn = fmaxf(mt, p[ml]);
            const float wo = (mt > -INFINITY) ? exp2_fast(mt - mn) : 0.f;
            const float wn = (p[ml] > -INFINITY) ? exp2_fast(p[ml] - mn) : 0.f;
            o = o * wo + p[x] * wn;
            lt = lt * wo + p[ml + 1] * wn;
            mt = mn;
        }
        Elem<T>::store(outp + x, o / lt);
    }
}

// A row's slots in memory as a buffer resource: a load beyond the last of them returns zeros, so a tile's loads need no
// tests and no second form for the row's end.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slots_buffer(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t b, int off) {
    return __builtin_bit_cast(uint4, (u32x4_t)__builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}
__device__ __forceinline__ uint2 buffer_load8(__amdgpu_buffer_rsrc_t b, int off) {
    return __builtin_bit_cast(uint2, (u32x2_t)__builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
}
__device__ __forceinline__ float buffer_load4(__amdgpu_buffer_rsrc_t b, int off) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0));
}
// the same with device scope (the cache-policy bit that a device-scope atomic load sets)
constexpr int kDeviceScope = 16;
__device__ __forceinline__ float4 buffer_load16_agent(__amdgpu_buffer_rsrc_t b, int off) {
    return __builtin_bit_cast(float4, (u32x4_t)__builtin_amdgcn_raw_buffer_load_b128(b, off, 0, kDeviceScope));
}
__device__ __forceinline__ float2 buffer_load8_agent(__amdgpu_buffer_rsrc_t b, int off) {
    return __builtin_bit_cast(float2, (u32x2_t)__builtin_amdgcn_raw_buffer_load_b64(b, off, 0, kDeviceScope));
}

// Sum of G values over the 16 lanes of a DPP row, scattered: lane c ends up with the total of
// head (c >> 2) & 3 (for G <= 4) -- 11 operations instead of 16 for four separate all-reduces.
template <int G>
__device__ __forceinline__ float row16_reduce_scatter(const float (&v)[G], int c) {
    static_assert(G <= 4, "scatter form covers up to four heads");
    const bool hi8 = (c & 8) != 0, hi4 = (c & 4) != 0;
    // distance 8: lanes with bit 3 clear keep heads {0,1}, the others heads {2,3}
    const float v0 = v[0], v1 = G > 1 ? v[1] : 0.f, v2 = G > 2 ? v[2] : 0.f, v3 = G > 3 ? v[3] : 0.f;
    const float keepA = hi8 ? v2 : v0, sendA = hi8 ? v0 : v2;
    const float keepB = hi8 ? v3 : v1, sendB = hi8 ? v1 : v3;
    const float a = keepA + dpp_mov<kDppRowRor(8)>(sendA);
    const float b = keepB + dpp_mov<kDppRowRor(8)>(sendB);
    // bit 2 picks between the two heads still held; the half-row mirror pairs lane c with c^7
    const float keep = hi4 ? b : a, send = hi4 ? a : b;
    float r = keep + dpp_mov<kDppRowHalfMirror>(send);  // partner c^7: other value of bit 2, same bit 3
    // the two quads of a half-row now hold complementary lanes: finish with sums inside the quad
    r += dpp_mov<kDppQuadPerm(2, 3, 0, 1)>(r);
    r += dpp_mov<kDppQuadPerm(1, 0, 3, 2)>(r);
    return r;                                           // total of head 2*bit3 + bit2
}

__device__ __forceinline__ float lane_value(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <typename T> struct IsBf16 { static constexpr bool value = false; };
template <> struct IsBf16<bf16_t> { static constexpr bool value = true; };

// Running maxima start at the lowest finite number: slots whose logits are all -inf (keys masked by infinite entries, or
// products that overflow) then weigh nothing in the tiles as in the merges; from -inf they would give -inf - -inf.
constexpr float kNoMax = -FLT_MAX;

// ---- tiles ------------------------------------------------------------------------------------------
// What a unit's waves know of its row.
template <typename T>
struct RowRefs {
    const char *K, *V;          // slot 0 of the row's K and V in the cache
    const float *Ksc, *Vsc;     // FP8 caches: their scales
    const T *q, *knew, *vnew;   // the group's query rows; the row being appended
    int len;                    // slots of the row, the one being appended included
    int held;                   // slots that the cache holds: without it
    int new_slot;               // the slot being appended, or -1
    float scale2;               // logit scale in the exponent domain
};

// A tile of 32 slots of a bf16 or FP8 cache, on the matrix cores (v_mfma_f32_16x16x32_bf16), both products:
//   logits   S^T[slot][head] = K Q^T: two instructions' worth of 16 slots, the query heads in the 16 columns;
//   outputs  O^T[d][head] += V^T P^T over the 32 slots, 16 of the D values per instruction.
// The operands come from memory in the order the instructions want, without a trip through LDS or across lanes: slot
// 8 g + j of the tile is "lane group g = lane / 16, place j".  A lane fetches the K pieces of the slot whose logits come
// out for its own column and group, holds 8 logits of ONE head (lane % 16) after the first product, their probabilities
// are then the second product's operand as they are, and the V operand is a transpose inside the lane (one
// v_perm_b32 per register) of the rows 8 g + j it has fetched.  Lanes of columns beyond G repeat the last head; their
// results are never read.  A tile costs about 75 vector instructions and 16 matrix instructions whatever G (packed
// dot products on the vector unit took 540 for G = 4), and the accumulators D / 4 registers whatever G: launches over one
// layer of the 7B shape 7.7 -> 5.9 us, of its batch of four 13.9 -> 10.6; over all layers 14.4 -> 12.0 (45 MB), FP8 rows of a
// 32768-token prompt 49 -> 40; the 34B shape's, seven heads, 204 -> 189.
// K of the next tile is requested as soon as the logits are formed, V as soon as the outputs are: the same registers.
// FP8 codes are expanded to bf16 (exactly) where they are consumed.
template <int D, int G, bool Q8>
struct TileMfma {
    static constexpr int TK = 32;               // slots per tile
    static constexpr int KST = D / 32;          // k-steps of the logits
    static constexpr int KLD = Q8 ? KST / 2 : KST;      // 16-byte K pieces of a lane per slot
    static constexpr int EV = D / 16;           // V elements of a lane per slot
    static constexpr int VW = Q8 ? EV / 4 : EV / 2;     // and their registers
    static constexpr int RB = Q8 ? D : 2 * D;   // bytes of a cached row
    uint4 qf[KST];
    uint4 kf[2][KLD];
    uint32_t vw[8][VW];
    float ksc[Q8 ? 8 : 1], vsc[Q8 ? 8 : 1];
    float x[8];                                 // logits of slots 8 (lane / 16) + j for head lane % 16
    f32x4_t acc[EV];                            // acc[e][i]: d = EV (4 (lane / 16) + i) + e of head lane % 16
    float m_run, l_run;                         // this head's running max; the sum over this lane's slots

    // first of the 8 elements that lane group g multiplies in k-step s: a 16-byte piece of K holds 8 bf16 values, or the
    // 16 codes of two k-steps
    static __device__ __forceinline__ int k_elem(int s, int g) { return Q8 ? 64 * (s >> 1) + 16 * g + 8 * (s & 1) : 32 * s + 8 * g; }
    // slot (of 0..31) whose K a lane fetches for instruction t of the logits
    static __device__ __forceinline__ int k_slot(int t, int lane) { return 8 * ((lane >> 2) & 3) + 4 * t + (lane & 3); }

    __device__ __forceinline__ void begin(const RowRefs<bf16_t>& r, int lane) {
        const bf16_t* row = r.q + (size_t)min(lane & 15, G - 1) * D;
#pragma unroll
        for (int s = 0; s < KST; ++s) qf[s] = *reinterpret_cast<const uint4*>(row + k_elem(s, lane >> 4));
        m_run = kNoMax; l_run = 0.f;
#pragma unroll
        for (int e = 0; e < EV; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    // The tile that starts at slot t0.  Slots that memory does not hold read as zeros, without an access.
    __device__ __forceinline__ void request_k(const RowRefs<bf16_t>& r, int t0, int lane) {
        const int rows = uniform(max(min(r.held - t0, TK), 0));
        const auto kr = slots_buffer(r.K + (int64_t)t0 * RB, rows * RB);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KLD; ++s) kf[t][s] = buffer_load16(kr, k_slot(t, lane) * RB + (lane >> 4) * 16 + s * 64);
        if constexpr (Q8) {
            const auto ks = slots_buffer(r.Ksc + t0, rows * 4);
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const uint4 a = buffer_load16(ks, (lane >> 4) * 32 + 16 * y);
                ksc[4 * y] = __uint_as_float(a.x); ksc[4 * y + 1] = __uint_as_float(a.y); ksc[4 * y + 2] = __uint_as_float(a.z); ksc[4 * y + 3] = __uint_as_float(a.w);
            }
        }
    }
    __device__ __forceinline__ void request_v(const RowRefs<bf16_t>& r, int t0, int lane) {
        const int rows = uniform(max(min(r.held - t0, TK), 0));
        const auto vr = slots_buffer(r.V + (int64_t)t0 * RB, rows * RB);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int at = (8 * (lane >> 4) + j) * RB + (lane & 15) * (RB / 16);
            if constexpr (VW == 4) {
                const uint4 v = buffer_load16(vr, at);
                vw[j][0] = v.x; vw[j][1] = v.y; vw[j][2] = v.z; vw[j][3] = v.w;
            } else if constexpr (VW == 2) {
                const uint2 v = buffer_load8(vr, at);
                vw[j][0] = v.x; vw[j][1] = v.y;
            } else {
                vw[j][0] = __float_as_uint(buffer_load4(vr, at));
            }
        }
        if constexpr (Q8) {
            const auto vs = slots_buffer(r.Vsc + t0, rows * 4);
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const uint4 a = buffer_load16(vs, (lane >> 4) * 32 + 16 * y);
                vsc[4 * y] = __uint_as_float(a.x); vsc[4 * y + 1] = __uint_as_float(a.y); vsc[4 * y + 2] = __uint_as_float(a.z); vsc[4 * y + 3] = __uint_as_float(a.w);
            }
        }
    }
    static __device__ __forceinline__ float max_over_groups(float v) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    }
    static __device__ __forceinline__ float sum_over_groups(float v) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(b[0]) + __uint_as_float(b[1]);
    }
    __device__ __forceinline__ void logits(const RowRefs<bf16_t>& r, int t0, int lane) {
        f32x4_t s[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            s[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KST; ++k) {
                uint4 piece;
                if constexpr (Q8) piece = e4m3x8_to_bf16x8(k & 1 ? make_uint2(kf[t][k / 2].z, kf[t][k / 2].w) : make_uint2(kf[t][k / 2].x, kf[t][k / 2].y));
                else piece = kf[t][k];
                s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, piece), __builtin_bit_cast(bf16x8_t, qf[k]), s[t], 0, 0, 0);
            }
        }
        const int live = r.held - t0 - 8 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = s[j >> 2][j & 3] * (Q8 ? r.scale2 * ksc[j] : r.scale2);
            x[j] = j < live ? x[j] : -INFINITY;
        }
    }
    // Running max, accumulators and sum brought to the new maximum over the logits held by all lanes of a head.
    __device__ __forceinline__ void raise_max(float mt) {
        const float m_new = fmaxf(m_run, max_over_groups(mt));
        if (__ballot(m_new > m_run)) {
            const float corr = exp2_fast(m_run - m_new);
            l_run *= corr;
#pragma unroll
            for (int e = 0; e < EV; ++e) acc[e] *= corr;
            m_run = m_new;
        }
    }
    // acc += V^T P^T; v[j]: the bf16 pairs of slot j, pb: the probabilities
    __device__ __forceinline__ void add_outputs(const uint32_t (&v)[8][EV / 2], const bf16x8_t& pb) {
#pragma unroll
        for (int e = 0; e < EV; ++e) {
            u32x4_t vt;
#pragma unroll
            for (int w = 0; w < 4; ++w) vt[w] = __builtin_amdgcn_perm(v[2 * w + 1][e / 2], v[2 * w][e / 2], e & 1 ? 0x07060302u : 0x05040100u);
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, vt), pb, acc[e], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void outputs(const RowRefs<bf16_t>&, int) {
        float mt = x[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) mt = fmaxf(mt, x[j]);
        raise_max(mt);
        bf16x8_t pb;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float p = exp2_fast(x[j] - m_run);
            l_run += p;
            pb[j] = (__bf16)(Q8 ? p * vsc[j] : p);      // FP8: the V scale rides on the probability
        }
        uint32_t v[8][EV / 2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if constexpr (!Q8) {
#pragma unroll
                for (int w = 0; w < EV / 2; ++w) v[j][w] = vw[j][w];
            } else {
                const uint4 b = e4m3x8_to_bf16x8(make_uint2(vw[j][0], VW == 2 ? vw[j][VW - 1] : 0u));
                v[j][0] = b.x; v[j][1] = b.y;
                if constexpr (VW == 2) { v[j][2] = b.z; v[j][3] = b.w; }
            }
        }
        add_outputs(v, pb);
    }
    // The row being appended, attended over by one wave beside its tiles: it comes from the caller's tensors, so the
    // tiles make no exception for its slot.  Lane group g holds K's pieces of its k-steps (nk), lane c of every 16 V's elements
    // EV c .. EV c + EV - 1 (nv); FP8: already quantised and expanded again, with its scales.
    __device__ __forceinline__ void add_new(const RowRefs<bf16_t>& r, const uint4 (&nk)[KST], const uint32_t (&nv)[EV / 2], float ks, float vs, int lane) {
        f32x4_t s = {0.f, 0.f, 0.f, 0.f};       // every row of the operand is the new row
#pragma unroll
        for (int k = 0; k < KST; ++k)
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, nk[k]), __builtin_bit_cast(bf16x8_t, qf[k]), s, 0, 0, 0);
        const float xn = s[0] * (Q8 ? r.scale2 * ks : r.scale2);
        raise_max(xn);
        const bool first = lane < 16;           // the row counts once: place 0 of lane group 0
        const float p = first ? exp2_fast(xn - m_run) : 0.f;
        l_run += p;
        bf16x8_t pb = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
        pb[0] = (__bf16)(Q8 ? p * vs : p);
        uint32_t v[8][EV / 2];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int w = 0; w < EV / 2; ++w) v[j][w] = j == 0 && first ? nv[w] : 0u;
        add_outputs(v, pb);
    }
    // The wave's share (outputs, max, sum) of the unit into its LDS rows [G][D + 4].
    __device__ __forceinline__ void leave(float (*rows)[D + 4], int lane) {
        const float l = sum_over_groups(l_run);
        if ((lane & 15) < G) {
            float* row = rows[lane & 15];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < EV; e += 4)
                    *reinterpret_cast<float4*>(row + EV * (4 * (lane >> 4) + i) + e) = make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
            if (lane < 16) *reinterpret_cast<float2*>(row + D) = make_float2(m_run, l);
        }
    }
};

// A tile of 32 slots of fp32 storage, on the vector unit (the matrix cores' fp32 products would need V transposed and
// run at a sixteenth of the bf16 rate):
//   1. K and V rows are loaded 16 bytes per lane (LPR lanes per row, fully coalesced);
//   2. logits: FMAs against the g query rows held in registers, summed over the LPR lanes of a row, parked in LDS;
//   3. softmax bookkeeping with one 16-lane row per head (DPP row reductions only), the probabilities parked in LDS;
//   4. P.V with the K lane mapping; the 64 / LPR row groups of a wave are summed once per unit.
template <int D, int G>
struct TileF32 {
    static constexpr int TK = 32;
    static constexpr int LPR = D / 4;           // lanes per K/V row
    static constexpr int KPI = 64 / LPR;        // rows per wave load
    static constexpr int NIT = TK / KPI;        // loads per tile and operand
    static constexpr int GP = pad_pow2(G);
    static constexpr int HR = (GP + 3) / 4;     // heads per 16-lane row in the softmax step
    static constexpr int KK = TK / 16;          // slots per lane in the softmax step
    static constexpr int RB = 4 * D;            // bytes of a row
    static_assert(G <= LPR, "one lane per head needed when parking logits");
    float4 qv[G], kb[NIT], vb[NIT], xk, xv;
    float m_run[HR], l_run[HR], acc[G][4];      // 16-lane row r owns heads r*HR .. r*HR + HR - 1
    float (*sL)[GP];                            // [TK] this wave's logits, then its probabilities

    __device__ __forceinline__ void begin(const RowRefs<float>& r, int lane) {
#pragma unroll
        for (int h = 0; h < G; ++h) qv[h] = *reinterpret_cast<const float4*>(r.q + (size_t)h * D + (lane % LPR) * 4);
#pragma unroll
        for (int hh = 0; hh < HR; ++hh) { m_run[hh] = kNoMax; l_run[hh] = 0.f; }
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[h][e] = 0.f;
    }
    // The tile that starts at slot t0 (at least one slot of it is there).  Slots that memory does not hold read as zeros; the
    // row being appended is requested beside them (x) and put in its place when the tile is used.  (Fetched in its place, by a
    // second form of these loads with a pointer for each lane, it held them up one after the other: over one layer of 16 prompts
    // of 4096 tokens at 2 %, 2 / 3 / 4 heads per KV head, d = 128, 14.7 / 15.4 / 17.7 us instead of 12.1 / 13.0 / 14.6.)
    __device__ __forceinline__ void request(const char* rows_at, const float* fresh, float4 (&to)[NIT], float4& x, const RowRefs<float>& r, int t0, int lane) {
        const int rows = uniform(max(min(r.held - t0, TK), 0));     // said to be uniform: the compiler looped over the lanes' buffers
        const auto b = slots_buffer(rows_at + (int64_t)t0 * RB, rows * RB);
#pragma unroll
        for (int i = 0; i < NIT; ++i) to[i] = __builtin_bit_cast(float4, buffer_load16(b, (i * KPI + lane / LPR) * RB + (lane % LPR) * 16));
        if (has_new(r, t0)) x = reinterpret_cast<const float4*>(fresh)[lane % LPR];         // wave-uniform
    }
    static __device__ __forceinline__ bool has_new(const RowRefs<float>& r, int t0) { return r.new_slot >= t0 && r.new_slot < t0 + TK; }
    static __device__ __forceinline__ void put_new(float4 (&to)[NIT], const float4& x, const RowRefs<float>& r, int t0, int lane) {
        const int rel = r.new_slot - t0;
        const bool mine = lane / LPR == rel % KPI;
#pragma unroll
        for (int i = 0; i < NIT; ++i)
            if (rel / KPI == i && mine) to[i] = x;
    }
    __device__ __forceinline__ void request_k(const RowRefs<float>& r, int t0, int lane) { request(r.K, r.knew, kb, xk, r, t0, lane); }
    __device__ __forceinline__ void request_v(const RowRefs<float>& r, int t0, int lane) { request(r.V, r.vnew, vb, xv, r, t0, lane); }
    __device__ __forceinline__ void logits(const RowRefs<float>& r, int t0, int lane) {
        if (has_new(r, t0)) put_new(kb, xk, r, t0, lane);
        const int sub = lane / LPR, c = lane % LPR;
        const int live_rows = r.len - t0;
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const bool live = i * KPI + sub < live_rows;
            float part[G];
#pragma unroll
            for (int h = 0; h < G; ++h)
                part[h] = fmaf(kb[i].w, qv[h].w, fmaf(kb[i].z, qv[h].z, fmaf(kb[i].y, qv[h].y, kb[i].x * qv[h].x)));
            if constexpr (LPR == 16 && G <= 4) {
                const float tot = row16_reduce_scatter<G>(part, c);
                const int hh = ((c >> 3) << 1) | ((c >> 2) & 1);
                if ((c & 3) == 0 && hh < G) sL[i * KPI + sub][hh] = live ? tot * r.scale2 : -INFINITY;
            } else if constexpr (LPR == 16) {
                const float tot = row16_reduce_scatter8<G>(part, c);
                const int hh = ((c >> 3) << 2) | (((c >> 2) & 1) << 1) | ((c >> 1) & 1);
                if ((c & 1) == 0 && hh < G) sL[i * KPI + sub][hh] = live ? tot * r.scale2 : -INFINITY;
            } else {
                float mine = 0.f;
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    const float tot = group_allreduce_sum<LPR>(part[h]);
                    mine = (c == h) ? tot : mine;
                }
                if (c < G) sL[i * KPI + sub][c] = live ? mine * r.scale2 : -INFINITY;
            }
        }
    }
    __device__ __forceinline__ void outputs(const RowRefs<float>& r, int t0) {
        const int lane = threadIdx.x & 63, sub = lane / LPR, srow = lane >> 4, scol = lane & 15;
        __builtin_amdgcn_wave_barrier();
        // softmax bookkeeping: 16-lane row r handles heads r*HR.., lane column j slots j, j+16
        float corr_row[HR];
#pragma unroll
        for (int hh = 0; hh < HR; ++hh) {
            const int h = srow * HR + hh;
            float x[KK], mt = -INFINITY;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                x[kk] = (h < G) ? sL[scol + 16 * kk][h % GP] : -INFINITY;
                mt = fmaxf(mt, x[kk]);
            }
            mt = fmaxf(mt, dpp_mov<kDppRowRor(8)>(mt));
            mt = fmaxf(mt, dpp_mov<kDppRowRor(4)>(mt));
            mt = fmaxf(mt, dpp_mov<kDppRowRor(2)>(mt));
            mt = fmaxf(mt, dpp_mov<kDppRowRor(1)>(mt));
            const float m_new = fmaxf(m_run[hh], mt);
            float ps = 0.f;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const float pr = exp2_fast(x[kk] - m_new);
                ps += pr;
                if (h < G) sL[scol + 16 * kk][h % GP] = pr;
            }
            ps = group_allreduce_sum<16>(ps);
            corr_row[hh] = exp2_fast(m_run[hh] - m_new);
            l_run[hh] = l_run[hh] * corr_row[hh] + ps;
            m_run[hh] = m_new;
        }
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const float ch = lane_value(corr_row[h % HR], 16 * (h / HR));
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[h][e] *= ch;
        }
        if (has_new(r, t0)) put_new(vb, xv, r, t0, lane);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const float* pp = sL[i * KPI + sub];
#pragma unroll
            for (int h = 0; h < G; ++h) {
                const float ph = pp[h];
                acc[h][0] = fmaf(ph, vb[i].x, acc[h][0]);
                acc[h][1] = fmaf(ph, vb[i].y, acc[h][1]);
                acc[h][2] = fmaf(ph, vb[i].z, acc[h][2]);
                acc[h][3] = fmaf(ph, vb[i].w, acc[h][3]);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ void leave(float (*rows)[D + 4], int lane) {
        const int sub = lane / LPR, c = lane % LPR, srow = lane >> 4;
        if constexpr (LPR == 16) {
            // Four row groups = the four 16-lane rows of the wave.  Reduce-scatter with the lane-swap instructions
            // (v_permlane16_swap, v_permlane32_swap: vector-unit moves, no trip through the LDS queue): of four
            // accumulators x0..x3, row r ends up with the total of x_r.
            // swap16(a, b) = ([a.r0, b.r0, a.r2, b.r2], [a.r1, b.r1, a.r3, b.r3]), swap32(a, b) = ([a.lo, b.lo], [a.hi, b.hi]).
            auto pair_sum16 = [](float a, float b) {
                const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
                return __uint_as_float(x[0]) + __uint_as_float(x[1]);       // [a.r0 + a.r1, b.r0 + b.r1, a.r2 + a.r3, b.r2 + b.r3]
            };
            auto pair_sum32 = [](float a, float b) {
                const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
                return __uint_as_float(x[0]) + __uint_as_float(x[1]);
            };
#pragma unroll
            for (int h = 0; h < G; ++h)
                rows[h][c * 4 + sub] = pair_sum32(pair_sum16(acc[h][0], acc[h][1]), pair_sum16(acc[h][2], acc[h][3]));   // row `sub` holds the total of element `sub`
        } else {
#pragma unroll
            for (int h = 0; h < G; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[h][e] += __shfl_xor(acc[h][e], 32, 64);
            if (sub == 0) {
#pragma unroll
                for (int h = 0; h < G; ++h)
                    *reinterpret_cast<float4*>(&rows[h][c * 4]) = make_float4(acc[h][0], acc[h][1], acc[h][2], acc[h][3]);
            }
        }
        if ((lane & 15) == 0) {
#pragma unroll
            for (int hh = 0; hh < HR; ++hh)
                if (srow * HR + hh < G) *reinterpret_cast<float2*>(&rows[srow * HR + hh][D]) = make_float2(m_run[hh], l_run[hh]);
        }
    }
};

// ---- the kernel -------------------------------------------------------------------------------------
// Q8: the cache rows are E4M3 codes with one fp32 scale per row; codes are expanded to bf16 (exactly) where they are
// consumed, the K scale multiplies the finished logit, the V scale the probability before it is rounded to bf16.  The row
// being appended is quantised by the wave that attends over it, which stores it too.
// Blocks of four waves, several per CU: the blocks of a CU overlap each other's start-up and merge phases.  One wide block
// per row (12 waves, no merge across blocks) measured no faster: the row's loads then queue at a single CU's address path.
// WALK: the grid is smaller than the slice may be (launches over a layer range, see launch_decode), a block takes further
// units with the grid as stride.
template <typename T, int D, int G, bool Q8, bool WALK>
__global__ __launch_bounds__(256, (IsBf16<T>::value ? (D == 64 && !Q8 ? 4 : 3) : G <= 4 && D == 64 ? 3 : 2)) void decode_kernel(DecodeParams P) {
    constexpr int NW = 4;                       // waves per block
    constexpr int THREADS = NW * 64;
    constexpr bool BF = IsBf16<T>::value;
    static_assert(!Q8 || BF, "FP8 caches hold bf16 models");
    typedef typename std::conditional<BF, TileMfma<D, G, Q8>, TileF32<D, G>>::type Tile;
    constexpr int TK = Tile::TK;
    constexpr int RB = Tile::RB;                // bytes of a cached row
    constexpr int PS = partial_floats(G, D);
    constexpr int DL = D + 4;                   // LDS row of the wave merge: D outputs, max, sum; a multiple of 16 bytes

    __shared__ __align__(16) float sMerge[NW][G][DL];
    __shared__ __align__(16) float sL[BF ? 1 : NW][TK][pad_pow2(G)];      // fp32 storage: the waves' logits and probabilities
    __shared__ int sLast;

    const int tid = threadIdx.x;
    // The work list and its layer index, budgets and slab offsets were written by the compaction, in an earlier launch:
    // they are constant while this kernel runs and are read as such, which puts their (block-uniform) loads on the scalar unit.
    typedef const __attribute__((address_space(4))) int32_t* IndexPtr;
    typedef const __attribute__((address_space(4))) float* ScalePtr;
    // ---- what the whole launch shares: the slice of the list, and the append count of its layers
    const IndexPtr layer_start = (IndexPtr)P.wl.layer_start;
    const int begin = P.layer_begin ? layer_start[P.layer_begin] : 0;
    const int end = layer_start[P.layer_begin + P.n_layers];
    const int appended = P.appended[P.layer_begin];
    // ---- the unit of this block.  One block-unit per block while the grid covers the slice: the hardware dispatcher balances
    // the ragged units.  The grid is a host-side upper bound on the units of the layer range, or a cap below it, and blocks
    // beyond the slice leave at once.
    // The record is read word by word.  A layer's first records (launches over one layer) are requested together with the
    // values above, the others, whose place depends on them, a round trip later.
    static_assert(offsetof(WorkItem, row_abs) == 0 && offsetof(WorkItem, key0) == 4 && offsetof(WorkItem, kept) == 8 &&
                  offsetof(WorkItem, unit) == 12 && offsetof(WorkItem, kbase) == 16 && offsetof(WorkItem, idx_base) == 24 &&
                  offsetof(WorkItem, b) == 32 && offsetof(WorkItem, l) == 36 &&
                  offsetof(WorkItem, ucap) == 44 && offsetof(WorkItem, hkv) == 48 && offsetof(WorkItem, layer_units) == 52,
                  "the record is read as 16 words");
    int rec[14];
    auto read = [&](const WorkItem* item) {
#pragma unroll
        for (int i = 0; i < 14; ++i) rec[i] = ((IndexPtr)item)[i];
    };
    int w = blockIdx.x;
    bool listed = true;
    if (P.heads && w < kHeadUnits) {
        read(P.heads + w);
        w += begin;
    } else {
        const bool odd = ((appended + (P.append_mode && appended < P.T_max ? 1 : 0)) & 1) != 0;
        if (P.wl.by_size && P.zigzag > 2 && odd) {  // size-class order, odd step: the whole units are walked backwards, so that
            const int nf = min(layer_start[P.L + 1], (int)gridDim.x);   // what the memory-side cache kept of the last step comes first
            const int nf8 = nf & ~7;            // whole groups of 8 change places, so a unit stays on its XCD (and its L2)
            if (w < nf8) w = nf8 - 8 - (w & ~7) + (w & 7);
        }
        w += begin;
        listed = w < P.wl.cap;
        if (listed) read(P.wl.items + w);
    }
    int mode = P.append_mode;
    // more steps than slots were reserved (only a replayed graph gets here): attend over what the cache holds,
    // append nothing, count nothing, and report it (after the block's first unit: a store in front of the unit
    // record's load would keep that load off the scalar unit)
    const bool over = mode && appended >= P.T_max;
    if (over) mode = 0;
    const bool appending = mode == 1;
    const int step = appended + (mode ? 1 : 0); // appends the cache holds once this launch is done
    auto process_unit = [&](const auto& A, int tid) {
        const int lane = tid & 63, wave = uniform(tid >> 6);
        // The block that holds the last ticket of its layer, and then of the launch, publishes the new count.
        auto finish = [&](int ticket, int il, int n_layer) {
            if (ticket != n_layer - 1) return;
            store_agent(A.readers + il * kReaderStride, 0);
            if (A.n_layers > 1) {
                if (add_agent(A.readers + A.L * kReaderStride, 1) != A.n_layers - 1) return;
                store_agent(A.readers + A.L * kReaderStride, 0);
            }
            for (int l = A.layer_begin; l < A.layer_begin + A.n_layers; ++l) store_agent(A.appended + l, step);
        };
        if (!listed) return;
        const int row_abs = rec[0], key0 = rec[1], kept = rec[2], unit = rec[3];
        const int64_t kbase = (int64_t)(((uint64_t)(uint32_t)rec[5] << 32) | (uint32_t)rec[4]);
        const int64_t idx_base = (int64_t)(((uint64_t)(uint32_t)rec[7] << 32) | (uint32_t)rec[6]);
        const int ib = rec[8], il = rec[9], ucap = rec[11], hkv = rec[12], n_layer = rec[13];
        if (w >= end) return;
        const int nbig = kept >> A.ub_shift;    // units of this row that hold slots now: the whole ones, and the small ones up to len
        const int nu = nbig + ((kept + step - (nbig << A.ub_shift) + (1 << A.us_shift) - 1) >> A.us_shift);
        const int lr = il - A.layer_begin;
        // The ticket: taken at once by a unit that has nothing to read, else behind the loads of the unit's first
        // tile (returns come back in issue order: in front of them it would hold up the first tile).  A block takes it only
        // after all of its waves have read the append count, or a wave could still meet the new one: each wave's read is consumed
        // in front of the barrier, and the operand of the atomic add is produced behind it.  (The bare barrier: it waits for no
        // memory request.  The waves come here together, right behind the record.)
        int one = 1;
        if (A.append_mode) {
            asm volatile("" : : "s"(appended));
            __builtin_amdgcn_s_barrier();
            asm volatile("" : "+s"(one));
        }
        auto take_ticket = [&]() { return (mode && tid == 0) ? add_agent(A.readers + il * kReaderStride, one) : -1; };
        T* outp = reinterpret_cast<T*>(A.out) + ((size_t)(lr * A.B + ib) * A.Hq + (size_t)hkv * G) * D;
        const int len = kept + step;
        if (__builtin_expect(kept == 0 || key0 >= len, 0)) {    // a request rejected at compaction (defined output, no reads), or a unit reserved for later appends
            if (kept == 0)
                for (int x = tid; x < G * D; x += THREADS) Elem<T>::store(outp + x, 0.f);
            const int ticket = take_ticket();
            if (mode && tid == 0) finish(ticket, il, n_layer);
            return;
        }
        const int cap = kept + A.T_max;
        const int new_slot = appending ? len - 1 : -1;
        const int held = BF && appending ? len - 1 : len;                       // slots the tiles cover
        const int lim = min(held, key0 + ucap);                                 // end of the unit's slots
        RowRefs<T> row;
        row.K = A.kv + kbase * (Q8 ? 1 : (int)sizeof(T));
        row.V = row.K + (int64_t)A.Hkv * cap * RB;
        row.Ksc = A.scales + kbase / D;
        row.Vsc = row.Ksc + (int64_t)A.Hkv * cap;
        row.q = reinterpret_cast<const T*>(A.q) + ((size_t)(lr * A.B + ib) * A.Hq + (size_t)hkv * G) * D;
        row.knew = reinterpret_cast<const T*>(A.k_new) + ((size_t)(lr * A.B + ib) * A.Hkv + hkv) * D;
        row.vnew = reinterpret_cast<const T*>(A.v_new) + ((size_t)(lr * A.B + ib) * A.Hkv + hkv) * D;
        row.len = len;
        row.held = appending ? len - 1 : len;
        row.new_slot = new_slot;
        row.scale2 = (A.sm_scale ? ((ScalePtr)A.sm_scale)[il] : A.default_scale) * kLog2e;
        Tile tile;
        if constexpr (!BF) {
            tile.sL = sL[wave];
        }
        tile.begin(row, lane);

        // tiles of the unit are dealt round-robin to the 4 waves, so a partly filled unit keeps all of them busy.
        // A wave walks its tiles forwards on even steps and backwards on odd ones: a cache that is a little
        // larger than an L2 then finds the tiles it touched last in the previous step first in this one.
        const int tw0 = key0 + wave * TK;
        const int nt_w = tw0 < lim ? (lim - tw0 + NW * TK - 1) / (NW * TK) : 0;    // tiles of this wave that hold slots
        const bool rev = A.zigzag > 1 && (step & 1);
        int t0 = tw0 + (rev && nt_w > 0 ? nt_w - 1 : 0) * NW * TK;
        const int stride = rev ? -NW * TK : NW * TK;
        // the last wave of the unit that holds the new slot (it has the fewest rows) also attends over and stores the new row
        const bool fresh = BF && appending && wave == NW - 1 && new_slot >= key0 && new_slot < key0 + ucap;       // wave-uniform
        auto request = [&](int at) { tile.request_k(row, at, lane); tile.request_v(row, at, lane); };
        int ticket = -1;                        // taken when the first tile's rows are on their way
        if constexpr (!BF) {
#pragma unroll 1
            for (int i = nt_w; i > 0; --i, t0 += stride) {      // a tile ahead does not fit the registers
                request(t0);
                if (i == nt_w) ticket = take_ticket();          // (wave 0 of a unit that holds slots has a tile)
                tile.logits(row, t0, lane);
                tile.outputs(row, t0);
            }
        } else if (nt_w > 0 || fresh) {
            // The new row is requested in front of the first tile, multiplied and stored while that is on its way.  A wave that
            // attends over the new row alone requests a tile of no bytes: with a test around the request, the compiler would wait
            // for the new row as if no tile had been requested, which is until the tile is there.  (That and K stored with one
            // instruction instead of four, us per launch over all layers, rows of 102 to 121 slots: 4096 of them 47.4 -> 38.3,
            // 16384 206.6 -> 192.2, with one query head 201.5 -> 185.0; launches over one layer of the 7B shape 5.8 -> 5.7.)
            uint4 nk[D / 32];
            uint32_t nv[D / 32];
            uint4 raw_k = make_uint4(0, 0, 0, 0), raw_v = raw_k;
            if (fresh) {
                if constexpr (Q8) {             // lane c of every D / 8: elements 8 c .. 8 c + 7, to be quantised
                    raw_k = *reinterpret_cast<const uint4*>(row.knew + (lane % (D / 8)) * 8);
                    raw_v = *reinterpret_cast<const uint4*>(row.vnew + (lane % (D / 8)) * 8);
                } else {
#pragma unroll
                    for (int k = 0; k < D / 32; ++k) nk[k] = *reinterpret_cast<const uint4*>(row.knew + Tile::k_elem(k, lane >> 4));
                    const uint32_t* src = reinterpret_cast<const uint32_t*>(row.vnew) + (lane & 15) * (D / 32);
#pragma unroll
                    for (int w = 0; w < D / 32; ++w) nv[w] = src[w];
                }
            }
            request(t0);
            ticket = take_ticket();
            if (fresh) {
                float sk = 0.f, sv = 0.f;
                char* kdst = const_cast<char*>(row.K) + (int64_t)new_slot * RB;
                char* vdst = const_cast<char*>(row.V) + (int64_t)new_slot * RB;
                if constexpr (Q8) {
                    constexpr int LPR = D / 8;
                    const uint2 qk = quantize_row_e4m3<LPR>(raw_k, sk), qv = quantize_row_e4m3<LPR>(raw_v, sv);
                    if (lane < LPR) {
                        reinterpret_cast<uint2*>(kdst)[lane] = qk;
                        reinterpret_cast<uint2*>(vdst)[lane] = qv;
                        if (lane == 0) {
                            const_cast<float*>(row.Ksc)[new_slot] = sk;
                            const_cast<float*>(row.Vsc)[new_slot] = sv;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < D / 32; ++k) {
                        const int from = Tile::k_elem(k, lane >> 4) / 8;
                        nk[k] = e4m3x8_to_bf16x8(make_uint2((uint32_t)__shfl((int)qk.x, from, 64), (uint32_t)__shfl((int)qk.y, from, 64)));
                    }
                    const uint4 b = e4m3x8_to_bf16x8(qv);
                    if constexpr (D == 128) {
                        nv[0] = b.x; nv[1] = b.y; nv[2] = b.z; nv[3] = b.w;
                    } else {                    // 4 elements per lane: half of what a quantising lane holds
                        const int from = (lane & 15) >> 1;
                        const uint32_t w0 = (uint32_t)__shfl((int)b.x, from, 64), w1 = (uint32_t)__shfl((int)b.y, from, 64);
                        const uint32_t w2 = (uint32_t)__shfl((int)b.z, from, 64), w3 = (uint32_t)__shfl((int)b.w, from, 64);
                        nv[0] = lane & 1 ? w2 : w0; nv[1] = lane & 1 ? w3 : w1;
                    }
                } else {
                    // lane c of every 16 stores the piece of k-step c that its group holds: the whole row in one instruction
                    uint4 piece = nk[0];
#pragma unroll
                    for (int k = 1; k < D / 32; ++k) if ((lane & 15) == k) piece = nk[k];
                    if ((lane & 15) < D / 32) *reinterpret_cast<uint4*>(kdst + 2 * Tile::k_elem(lane & 15, lane >> 4)) = piece;
                    if (lane < 16) {
#pragma unroll
                        for (int w = 0; w < D / 32; ++w) reinterpret_cast<uint32_t*>(vdst)[lane * (D / 32) + w] = nv[w];
                    }
                }
                if (lane == 0) A.idx[idx_base + new_slot] = A.m + appended;
                tile.add_new(row, nk, nv, sk, sv, lane);
            }
            // The last tile stands behind the loop, so that the requests in the loop have no test and every wait is for what it
            // needs: the logits for K, the outputs for V.  Launches over several layers wait for V in front of the logits all
            // the same, which keeps K of the next tile behind it: batch of four of 10368 tokens, all layers, 103.5 us, without
            // that wait 107.2 (launches over one layer of it 10.0, with it 10.2; of one FP8 prompt of 32768 tokens 8.0 and 8.3).
#pragma unroll 1
            for (int i = nt_w; i > 1; --i, t0 += stride) {
                if (!A.heads) __builtin_amdgcn_s_waitcnt(0x0f70);       // vmcnt(0)
                tile.logits(row, t0, lane);
                tile.request_k(row, t0 + stride, lane);
                tile.outputs(row, t0);
                tile.request_v(row, t0 + stride, lane);
            }
            if (nt_w > 0) {
                tile.logits(row, t0, lane);
                tile.outputs(row, t0);
            }
        } else {
            ticket = take_ticket();
        }

        // fp32 storage: the unit that holds the new slot also stores the new row into the cache
        if (!BF && appending && new_slot >= key0 && new_slot < key0 + ucap && tid < RB / 16) {
            reinterpret_cast<uint4*>(const_cast<char*>(row.K) + (int64_t)new_slot * RB)[tid] = reinterpret_cast<const uint4*>(row.knew)[tid];
            reinterpret_cast<uint4*>(const_cast<char*>(row.V) + (int64_t)new_slot * RB)[tid] = reinterpret_cast<const uint4*>(row.vnew)[tid];
            if (tid == 0) A.idx[idx_base + new_slot] = A.m + appended;
        }

        // ---- merge the 4 waves through LDS
        tile.leave(sMerge[wave], lane);
        __syncthreads();
        // every thread merges two neighbouring output elements of one head over the waves' shares in sMerge: one weight
        // per wave, one store; into the output, or into the unit's partial
        float* part = A.partials + (first_partial(idx_base, row_abs, A.part_shift) + unit) * PS;
        auto merge_waves = [&](bool whole) {
            for (int x = tid; x < G * D / 2; x += THREADS) {
                const int h = x / (D / 2), e = (x % (D / 2)) * 2;
                float2 ml[NW];
                float mt = -INFINITY;
#pragma unroll
                for (int wv = 0; wv < NW; ++wv) {
                    ml[wv] = *reinterpret_cast<const float2*>(&sMerge[wv][h][D]);
                    mt = fmaxf(mt, ml[wv].x);
                }
                float o0 = 0.f, o1 = 0.f, lt = 0.f;
#pragma unroll
                for (int wv = 0; wv < NW; ++wv) {
                    const float wgt = (ml[wv].x > -INFINITY) ? exp2_fast(ml[wv].x - mt) : 0.f;
                    const float2 ov = *reinterpret_cast<const float2*>(&sMerge[wv][h][e]);
                    o0 = fmaf(ov.x, wgt, o0);
                    o1 = fmaf(ov.y, wgt, o1);
                    lt = fmaf(ml[wv].y, wgt, lt);
                }
                if (whole) {
                    const Quotient<T> by_sum(lt);
                    store_pair(outp + h * D + e, by_sum(o0), by_sum(o1));
                } else {                                            // device-scope stores: see below
                    store_agent2(part + h * D + e, o0, o1);
                    if (e == 0) store_agent2(part + G * D + h * 2, mt, lt);
                }
            }
        };
        merge_waves(nu == 1);
        if (nu > 1 && A.merge_mode == 1) {
            // Publication of the partials.  They were written with device-scope stores, which go through to the
            // memory side of the XCDs' L2 caches.  Every thread first waits until its own stores have been
            // acknowledged (a workgroup barrier alone does not drain another wave's outstanding stores), then
            // the barrier orders all four waves before thread 0, and only then does thread 0 add to the row's
            // counter.  The unit that counts nu - 1 predecessors therefore finds every partial of the row in
            // memory; it reads them with device-scope loads, which do not hit a stale line of its own L2.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            int32_t* counter = A.counters + row_abs;
            if (tid == 0) sLast = (add_agent(counter, 1) == nu - 1) ? 1 : 0;
            __syncthreads();
            // The last unit merges.  Few partials: a thread merges two neighbouring outputs over all of them, without a word to
            // the other threads.  (Launches over one layer of the 7B shape 6.15 -> 6.0 us, over all 12.1 -> 11.7; the line at 2, 4 or
            // 8 partials: 5.83, 5.75 and 5.70 us, 10.39, 10.33 and 10.27 for the batch of four; for every number of them 10.43,
            // because a load of 8 bytes per lane keeps the CU's address path as long as one of 16.)
            constexpr int kFew = 8;
            if (sLast && tid == 0) store_agent(counter, 0);
            if (sLast && nu <= kFew) {
                const auto pr = slots_buffer(part - unit * PS, nu * (PS * 4));
                for (int x = tid * 2; x < G * D; x += THREADS * 2) {
                    float2 ml[kFew], ov[kFew];
#pragma unroll
                    for (int j = 0; j < kFew; ++j) {
                        ml[j] = make_float2(-INFINITY, 0.f); ov[j] = make_float2(0.f, 0.f);
                        if (j < nu) {                           // wave-uniform
                            ml[j] = buffer_load8_agent(pr, j * (PS * 4) + (G * D + x / D * 2) * 4);
                            ov[j] = buffer_load8_agent(pr, j * (PS * 4) + x * 4);
                        }
                    }
                    float mt = ml[0].x, o0 = 0.f, o1 = 0.f, lt = 0.f;
#pragma unroll
                    for (int j = 1; j < kFew; ++j) mt = fmaxf(mt, ml[j].x);
#pragma unroll
                    for (int j = 0; j < kFew; ++j) {
                        const float wgt = (ml[j].x > -INFINITY) ? exp2_fast(ml[j].x - mt) : 0.f;
                        o0 = fmaf(ov[j].x, wgt, o0); o1 = fmaf(ov[j].y, wgt, o1); lt = fmaf(ml[j].y, wgt, lt);
                    }
                    const Quotient<T> by_sum(lt);
                    store_pair(outp + x, by_sum(o0), by_sum(o1));
                }
            } else if (sLast) {
                // More: they are dealt to the waves; a lane holds NP times four neighbouring outputs and the weight
                // of their head.  The loads of NB partials are in flight together, so a row of up to 4 NB units costs one
                // round trip to memory; 16 bytes per lane and load, because the CU takes 16 cycles per load instruction
                // whatever its width.  Then the waves merge through LDS like the shares of a unit.
                constexpr int NB = 4, NP = (G * D + 255) / 256;
                const auto pr = slots_buffer(part - unit * PS, nu * (PS * 4));
                float m2[NP], l2[NP];
                float4 o2[NP];
#pragma unroll
                for (int k = 0; k < NP; ++k) { m2[k] = -INFINITY; l2[k] = 0.f; o2[k] = make_float4(0.f, 0.f, 0.f, 0.f); }
#pragma unroll 1
                for (int u0 = wave; u0 < nu; u0 += NW * NB) {
                    float2 ml[NB][NP];
                    float4 ov[NB][NP];
#pragma unroll
                    for (int j = 0; j < NB; ++j)
#pragma unroll
                        for (int k = 0; k < NP; ++k) {
                            ml[j][k] = make_float2(-INFINITY, 0.f);
                            ov[j][k] = make_float4(0.f, 0.f, 0.f, 0.f);
                            const int x = (k * 64 + lane) * 4;
                            if (u0 + j * NW < nu && x < G * D) {
                                const int at = (u0 + j * NW) * (PS * 4);
                                ml[j][k] = buffer_load8_agent(pr, at + (G * D + x / D * 2) * 4);
                                ov[j][k] = buffer_load16_agent(pr, at + x * 4);
                            }
                        }
#pragma unroll
                    for (int k = 0; k < NP; ++k) {
                        float mn = m2[k];
#pragma unroll
                        for (int j = 0; j < NB; ++j) mn = fmaxf(mn, ml[j][k].x);
                        const float wo = m2[k] > -INFINITY ? exp2_fast(m2[k] - mn) : 0.f;
                        l2[k] *= wo;
                        o2[k].x *= wo; o2[k].y *= wo; o2[k].z *= wo; o2[k].w *= wo;
#pragma unroll
                        for (int j = 0; j < NB; ++j) {
                            const float wn = ml[j][k].x > -INFINITY ? exp2_fast(ml[j][k].x - mn) : 0.f;
                            l2[k] = fmaf(ml[j][k].y, wn, l2[k]);
                            o2[k].x = fmaf(ov[j][k].x, wn, o2[k].x); o2[k].y = fmaf(ov[j][k].y, wn, o2[k].y);
                            o2[k].z = fmaf(ov[j][k].z, wn, o2[k].z); o2[k].w = fmaf(ov[j][k].w, wn, o2[k].w);
                        }
                        m2[k] = mn;
                    }
                }
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const int x = (k * 64 + lane) * 4;
                    if (x < G * D) {
                        *reinterpret_cast<float4*>(&sMerge[wave][x / D][x % D]) = o2[k];
                        if (x % D == 0) *reinterpret_cast<float2*>(&sMerge[wave][x / D][D]) = make_float2(m2[k], l2[k]);
                    }
                }
                __syncthreads();
                merge_waves(true);
            }
        }
        if (mode && tid == 0) finish(ticket, il, n_layer);
    };
    if constexpr (!WALK) {
        process_unit(P, tid);
    } else {
        // Loop invariants would be held in registers, and spill: the thread's index and the parameters are read anew for
        // each unit, the latter through a pointer to the kernel's arguments that the compiler cannot see through.
        typedef const __attribute__((address_space(4))) DecodeParams* ParamsPtr;
#pragma unroll 1
        for (;;) {
            ParamsPtr Q = (ParamsPtr)__builtin_amdgcn_kernarg_segment_ptr();
            int t = threadIdx.x;
            asm volatile("" : "+s"(Q), "+v"(t));
            process_unit(*Q, t);
            w += (int)gridDim.x;                // the list of a layer range is in its own order
            if (w >= end) break;
            __syncthreads();                    // the previous unit's merge buffers are free again
            read(P.wl.items + w);
        }
    }
    if (over && blockIdx.x == 0 && tid == 0) set_sticky(P.status, VLC_ERR_CAPACITY, -3, P.layer_begin, appended);
}

// Second kernel of merge mode 2: one block per (layer, request, KV head) row.  It runs after the attention
// kernel of the same call, so the append count it reads already includes this call's step.
template <typename T, int D, int G>
__global__ __launch_bounds__(256) void decode_merge_kernel(DecodeParams P) {
    const int row = blockIdx.x;
    const int hkv = row % P.Hkv;
    const int b = (row / P.Hkv) % P.B;
    const int lr = row / (P.Hkv * P.B);
    const int bl = b * P.L + P.layer_begin + lr;
    const int kept = P.kept[bl];
    if (kept == 0) return;
    const int len = kept + P.appended[P.layer_begin];
    const int nbig = kept >> P.ub_shift;
    const int nu = nbig + ((len - (nbig << P.ub_shift) + (1 << P.us_shift) - 1) >> P.us_shift);
    if (nu == 1) return;
    T* outp = reinterpret_cast<T*>(P.out) + ((size_t)(lr * P.B + b) * P.Hq + (size_t)hkv * G) * D;
    const int64_t idx_base = P.slot_off[bl] * P.Hkv + (int64_t)hkv * (kept + P.T_max);
    merge_partials<T, D, G, 256>(P.partials + first_partial(idx_base, bl * P.Hkv + hkv, P.part_shift) * partial_floats(G, D), outp, nu, threadIdx.x);
}

template <typename T, int D, int G>
hipError_t launch_one(const DecodeParams& P, int grid, bool walk, int rows, hipStream_t st) {
    bool done = false;
    if constexpr (IsBf16<T>::value) {
        if (P.kv_fp8) {
            if (walk) decode_kernel<T, D, G, true, true><<<grid, 256, 0, st>>>(P);
            else decode_kernel<T, D, G, true, false><<<grid, 256, 0, st>>>(P);
            done = true;
        }
    }
    if (!done && walk) decode_kernel<T, D, G, false, true><<<grid, 256, 0, st>>>(P);
    else if (!done) decode_kernel<T, D, G, false, false><<<grid, 256, 0, st>>>(P);
    if (P.merge_mode == 2) decode_merge_kernel<T, D, G><<<rows, 256, 0, st>>>(P);
    return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_g(const DecodeParams& P, int g, int grid, bool walk, int rows, hipStream_t st) {
    switch (g) {
        case 1: return launch_one<T, D, 1>(P, grid, walk, rows, st);
        case 2: return launch_one<T, D, 2>(P, grid, walk, rows, st);
        case 3: return launch_one<T, D, 3>(P, grid, walk, rows, st);
        case 4: return launch_one<T, D, 4>(P, grid, walk, rows, st);
        case 5: return launch_one<T, D, 5>(P, grid, walk, rows, st);
        case 6: return launch_one<T, D, 6>(P, grid, walk, rows, st);
        case 7: return launch_one<T, D, 7>(P, grid, walk, rows, st);
        case 8: return launch_one<T, D, 8>(P, grid, walk, rows, st);
    }
    return hipErrorInvalidValue;
}

int log2i(int v) {
    int s = 0;
    while ((1 << s) < v) ++s;
    return s;
}

}  // namespace

hipError_t launch_decode(const DecodeArgs& a) {
    const vlc_cache& c = *a.c;
    const vlc_shape& s = c.shape;
    DecodeParams P;
    P.q = a.q; P.k_new = a.k_new; P.v_new = a.v_new; P.out = a.out; P.sm_scale = a.sm_scale;
    P.kept = c.dev.kept; P.slot_off = c.dev.slot_off; P.appended = c.dev.appended; P.kv = c.dev.kv; P.readers = c.dev.readers;
    P.counters = c.dev.counters; P.partials = c.dev.partials; P.idx = c.dev.idx; P.scales = c.dev.scales; P.status = c.dev.status;
    // A launch over all layers walks list 1 (coarser units; by size class once the cache has more units than
    // fit the chip at once, so that the blocks dispatched last are short), a launch over a layer range list 0
    // (fine units in layer order, so that one layer of the batch still fills the chip).
    const bool all_layers = a.layer_begin == 0 && a.n_layers == s.L;
    P.wl = c.dev.list[all_layers ? 1 : 0];
    P.heads = !all_layers && a.n_layers == 1 ? c.dev.heads + (size_t)a.layer_begin * kHeadUnits : nullptr;
    P.ub_shift = log2i(P.wl.u_big); P.us_shift = log2i(P.wl.u_small);
    P.part_shift = log2i(c.dev.partial_slots);
    P.B = s.B; P.L = s.L; P.Hq = s.Hq; P.Hkv = s.Hkv; P.m = s.m;
    P.layer_begin = a.layer_begin; P.n_layers = a.n_layers; P.T_max = c.T_max;
    P.append_mode = a.k_new ? 1 : 0;
    P.default_scale = 1.0f / sqrtf((float)s.d);
    P.merge_mode = c.opt.decode_merge;
    P.zigzag = c.opt.decode_zigzag;
    P.kv_fp8 = c.kv_fp8 ? 1 : 0;
    const int rows = a.n_layers * s.B * s.Hkv;
    // One block per unit.  The budgets, and with them the true number of units, are known on the device only: the grid is
    // the upper bound, every row at the full prompt length and never more than the whole work list, and blocks beyond the
    // slice leave at once.  A launch over a layer range gets one resident round of blocks (three per CU) that walk the units instead
    // where the blocks to leave are more than eight rounds and cannot hide behind the reads: about 2000 of them come and go
    // per us, and half of the time that the rows take (5 MB per us) covers them.  us per launch, covering grid / walk, 7B shape: one
    // layer of 32 prompts of 4096 tokens at 1 % (8448 blocks for 512 units, 5 MB) 8.7 / 6.3, 64 of 2944 at 1 % (12288 for 1024, 8 MB)
    // 13.9 / 8.3, 128 of 1024 at 1 % (9216 for 2048, 5 MB) 13.6 / 9.9, at 10 % (52 MB) 23.6 / 24.6; two layers of one prompt of 131072
    // (8208 for 832, 107 MB) 32.1 / 35.2, eight (32832, 430 MB) 97 / 115; 16 layers of 16 prompts of 2944 (49152, 308 MB) 83 / 88.
    int64_t grid = (int64_t)rows * (((int64_t)s.m + c.T_max) / P.wl.u_small + 1);
    if (grid > P.wl.cap) grid = P.wl.cap;
    const int64_t round = 3 * (int64_t)c.num_cus, mean_row = c.sum_k_max / s.L;
    const int64_t leave = grid - rows * ((mean_row + c.T_max) / P.wl.u_small + 1);
    const int64_t bytes = rows * mean_row * 2 * s.d * (c.kv_fp8 ? 1 : s.dtype == VLC_F32 ? 4 : 2);
    const bool walk = !all_layers && leave > 8 * round && leave > bytes / 5000;
    if (walk) grid = round;
    if (grid < 1) grid = 1;
    const int g = s.Hq / s.Hkv;
    if (s.dtype == VLC_F32)
        return s.d == 64 ? launch_g<float, 64>(P, g, (int)grid, walk, rows, a.stream) : launch_g<float, 128>(P, g, (int)grid, walk, rows, a.stream);
    return s.d == 64 ? launch_g<bf16_t, 64>(P, g, (int)grid, walk, rows, a.stream) : launch_g<bf16_t, 128>(P, g, (int)grid, walk, rows, a.stream);
}

}  // namespace vlc
