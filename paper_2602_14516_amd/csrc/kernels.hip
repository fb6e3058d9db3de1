// HIP kernels for gfx950 (CDNA4, wave64): paged KV append, attention over paged K/V
// (wide = prefill tiles, narrow = decode-style split-KV items, fused in one launch) and the
// split-KV combine.
//
// Operation (paper Section 3: prefill with history l_hist = C and incremental length
// l_incr = L; decode = one token per request): query i of a row sits at position C + i
// and attends keys 0..C+i; query head hq reads KV head hq / G.
//
// Matrix-core formulation.  Everything is computed transposed so that all softmax state is
// per lane:
//   S^T[key][q]  = K[key][:] . Q[q][:]          v_mfma_f32_32x32x16_bf16, A = K rows, B = Q^T
//   O^T[d][q]   += V^T[d][key] . P^T[key][q]    A = V^T (LDS transpose read), B = P^T
// In the 32x32 accumulator layout lane l owns column q = l % 32 and rows
// (i/4)*8 + (l/32)*4 + i%4 for register i, so a lane's 16 registers of S^T are 16 keys of
// ONE query row: row max / row sum are in-lane reductions plus one exchange with lane l^32,
// and the bf16 P^T operand of the second product is built from the same registers without
// leaving the register file.  The V^T operand needs 4 consecutive keys per lane for a
// fixed d; ds_read_b64_tr_b16 delivers exactly that from [key][d] data in LDS.
// Narrow items of at most 16 query rows (a decode row's grouped heads) use the same formulation on
// v_mfma_f32_16x16x32_bf16 tiles (lane l owns column q = l % 16 and keys 4 (l/16) + i, 16 + 4 (l/16) + i):
// half the matrix and softmax work per key of the 32-row tiles, most of which would be padding there.
//
// LDS tile layout ("groups"): keys are stored in groups of KPW = 64 / (d/8) keys (4 for
// d = 128), one group = exactly the 1 KB that one wave-wide 16-byte-per-lane load delivers.
// Inside a group, 64-byte quads of chunks stay together and the keys interleave:
//   addr(key, chunk) = (key / KPW) * GS + (chunk / 4) * (KPW * 64) + (key % KPW) * 64 + (chunk % 4) * 16,
//   GS = 1024 + 16.
// With this order (a) a wave's direct global->LDS load (lane i -> LDS slot i) fills a group
// while every 4 consecutive lanes fetch 64 contiguous bytes of one key row, (b) the 16 lanes
// that read one chunk of 16 consecutive keys for the first product hit 64 distinct banks
// (4 keys 64 B apart per group, groups shifted by the 16-byte pad), the 32 lanes of a
// transpose read for the second product touch 256 contiguous bytes, and (c) every operand
// address is a per-lane base plus a compile-time constant.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace ampd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(uintptr_t)(p))
typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef const __attribute__((address_space(1))) u32x4* GlobalChunk;

constexpr int WG = 256;                 // append / combine kernels
constexpr int AWG = 64 * ATTN_WAVES;    // attention kernel: 8 waves, one workgroup per CU
constexpr int KT = 128;                 // keys per LDS stage of a wide item (one barrier per stage)
constexpr int NSTAGE = 2;               // LDS ring of K/V stages for wide items
constexpr float NEG_INF = -__builtin_inff();

template <int D>
struct Geo {
    static constexpr int CPK = D / 8;                  // 16-byte (8-element) chunks per key row
    static constexpr int KPW = 64 / CPK;               // keys per group (one wave-wide load)
    static constexpr int GS = 1024 + 16;               // LDS bytes per group
    static constexpr int B32 = (32 / KPW) * GS;        // bytes of a 32-key block (K or V)
    static constexpr int KTILE = (KT / 32) * B32;      // bytes of KT keys (K or V)
    static constexpr int WIDE_STAGE = 2 * KTILE;       // KT keys of K, then KT keys of V
    static constexpr int MERGE = ATTN_WAVES * 32 * (D + 4) * 4 + ATTN_WAVES * 32 * 2 * 4;   // narrow items: waves x (O, m, l)
    static constexpr int NARROW = ATTN_WAVES * 2 * B32;                // one private 32-key K+V block per wave
    static constexpr int SMEM0 = NSTAGE * WIDE_STAGE > MERGE ? NSTAGE * WIDE_STAGE : MERGE;
    static constexpr int SMEM = SMEM0 > NARROW ? SMEM0 : NARROW;
    static constexpr int NDB = D / 32;                 // 32-row blocks of O^T
    static constexpr int NKK = D / 16;                 // MFMA k-steps of the first product
};

// ---------------------------------------------------------------------------------------------
// small helpers

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exchange with lane^32 folded into the reduction: v_permlane32_swap(x, x) returns
// r0 = {x[0..31], x[0..31]} and r1 = {x[32..63], x[32..63]} (by destination lane halves), so
// op(r0, r1) is op(x[l], x[l^32]) in every lane.
__device__ __forceinline__ float max_xor32(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor32(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// A wave-uniform global address in scalar registers.
__device__ __forceinline__ GlobalBytes scalar_base(const char* p) {
    const uint64_t a = (uint64_t)p;
    return (GlobalBytes)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a));
}

// 8 stored elements -> 8 bf16 (as a 16-byte vector) for LDS.
template <int KVT>
struct RawChunk;
template <>
struct RawChunk<KV_BF16> {
    u32x4 v;
    static constexpr int ES = 2;                      // bytes per stored element
    __device__ __forceinline__ void zero() { v = u32x4{0, 0, 0, 0}; }
    __device__ __forceinline__ void load(const char* base, uint32_t lane_off) {
        v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + lane_off));   // streamed: see BlockLoader
    }
    __device__ __forceinline__ u32x4 widen(float) const { return v; }
};
template <>
struct RawChunk<KV_FP8> {
    u32x4 v;                                          // 16 codes: two neighbouring chunks of one key row
    static constexpr int ES = 1;
    __device__ __forceinline__ void zero() { v = u32x4{0, 0, 0, 0}; }
    __device__ __forceinline__ void load(const char* base, uint32_t lane_off) {
        v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + lane_off));
    }
    // decode(code) * scale is exact in bf16: 4 significant bits times a power of two.  The page scales are
    // powers of two (the append kernel writes no others), so the hardware's scaled conversion, which applies
    // the exponent of `scale` only, is that product: one instruction per two elements.
    __device__ __forceinline__ static u32x4 widen8(uint32_t lo, uint32_t hi, float scale) {
        const bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false);
        const bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true);
        const bf16x2 c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, false);
        const bf16x2 d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, true);
        return u32x4{__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, c),
                     __builtin_bit_cast(uint32_t, d)};
    }
    __device__ __forceinline__ u32x4 widen_first(float scale) const { return widen8(v.x, v.y, scale); }
    __device__ __forceinline__ u32x4 widen_second(float scale) const { return widen8(v.z, v.w, scale); }
};

struct ItemCtx {
    int req, kvh, g0, gn, q0, nq, kv_begin, kv_end, part_off;
    int C, row_off;
    int c_rows;                // keys from this position on are read from the packed new rows (k_new / v_new), not from
                               // the pages: C when the page writes of this call ride in the same launch, else "never"
    const int32_t* bt_row;     // block-table row of the request
    bool rounded;              // a prefill row (more than 32 query rows per KV head): its sums are taken over the rounded probabilities, in
                               // a block as in a tile; decode rows and short chunks, narrow in every launch, sum the fp32 ones
};
constexpr int NEVER = 0x3fffffff;

template <int KVT>
__device__ __forceinline__ ItemCtx item_ctx(const AttnParams& p, const Item& it) {
    ItemCtx c;
    c.req = it.req;
    c.kvh = it.heads & 0xff;
    c.g0 = (it.heads >> 8) & 0xff;
    c.gn = (it.heads >> 16) & 0xff;
    c.q0 = it.q0;
    c.nq = it.nq;
    c.kv_begin = it.kv_begin;
    c.kv_end = it.kv_end;
    c.part_off = it.part_off;
    c.C = it.C;
    c.row_off = it.row_off;
    c.c_rows = KVT == KV_BF16 && p.k_new ? it.C : NEVER;
    c.bt_row = p.block_table + (int64_t)it.req * p.max_pages;
    c.rounded = it.row_L * c.gn > 32;
    return c;
}

// Per-lane state of one wave: 32 query rows (lane % 32), O^T as D/32 accumulator blocks.
// m is a *reference* maximum in the log2 domain (scale * log2(e) folded in), not the exact
// running maximum: it is raised (and O, l rescaled) only when probabilities against it would grow too large:
// narrow items raise it when a block maximum exceeds it by more than RESCALE_SLACK (probabilities stay below
// 2^RESCALE_SLACK); wide items when a lane's 16 probabilities of a block sum to more than PSUM_LIMIT.
// (m, l, O) remain a consistent triple, which is all the final normalisation and the split-KV
// merge need.
template <int D>
struct WaveAcc {
    f32x16 O[Geo<D>::NDB];
    float m;
    float l;      // this lane's share of the running sum (lanes l and l^32 hold halves)
};
constexpr float RESCALE_SLACK = 8.0f;
constexpr float PSUM_LIMIT = 4096.0f;

// ---------------------------------------------------------------------------------------------
// the steps of one 32-key block

// S^T = K Q^T for the 32 keys whose LDS tile starts at kl.
template <int D>
__device__ __forceinline__ void qk32(uint32_t kl, const bf16x8 (&Q)[Geo<D>::NKK], f32x16& S, int lane) {
    using G_ = Geo<D>;
    const int r = lane & 31, g = lane >> 5;
    // chunk 2*kk + g of key r
    const uint32_t ka = kl + (r / G_::KPW) * G_::GS + (r % G_::KPW) * 64 + g * 16;
    S = f32x16{0};
#pragma unroll
    for (int kk = 0; kk < G_::NKK; ++kk) {
        const u32x4 raw = *LDS_PTR(const u32x4, ka + (kk >> 1) * (G_::KPW * 64) + (kk & 1) * 32);
        S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw), Q[kk], S, 0, 0, 0);
    }
}

// rel: per lane, (last visible key of this lane's query) - (first key of the block) - 4*(lane/32)
__device__ __forceinline__ void mask32(f32x16& S, int rel) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int koff = (i >> 2) * 8 + (i & 3);
        S[i] = koff <= rel ? S[i] : NEG_INF;
    }
}

__device__ __forceinline__ float rowmax32(const f32x16& S) {
    float mx = S[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[i]);
    return max_xor32(mx);
}

// Raise the reference maximum to cover mx (log2 domain) and rescale O and l.
template <int D>
__device__ __forceinline__ void raise_reference(WaveAcc<D>& st, float mx) {
    const float m_new = fmaxf(st.m, mx);
    const float alpha = fast_exp2(st.m - (m_new == NEG_INF ? 0.0f : m_new));
    st.l *= alpha;
#pragma unroll
    for (int db = 0; db < Geo<D>::NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.O[db][i] *= alpha;
    st.m = m_new;
}

// p = 2^(S*c - m); returns psum + this lane's sum over the ROUNDED probabilities, two per instruction (dot product of a bf16 pair with
// (1, 1) accumulated in fp32), which is also what the second product adds up; P = bf16(p) as the two B operands.  The rule of prefill rows:
// tiles, and blocks that take a tile's place (see ItemCtx::rounded).
__device__ __forceinline__ float exp32_dot(const f32x16& S, float c, float m_use, bf16x8 (&P)[2], float psum) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        const bf16x2 pr = {(__bf16)fast_exp2(__builtin_fmaf(S[i], c, -m_use)), (__bf16)fast_exp2(__builtin_fmaf(S[i + 1], c, -m_use))};
        psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, psum, false);
        P[i >> 3][i & 7] = pr[0];
        P[i >> 3][(i + 1) & 7] = pr[1];
    }
    return psum;
}

// The same for a lane of a narrow item with its N logits in S: the sum is taken over the rounded probabilities where `rounded`
// (uniform) says so, over the fp32 ones otherwise.  Both sums are taken: a branch would keep the reads of V from moving up past it.
template <int N, class Logit, class Prob>
__device__ __forceinline__ float exp_sum(float c, float m_use, bool rounded, Logit&& S, Prob&& P) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float sum = 0.0f, rounded_sum = 0.0f;
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        const float p0 = fast_exp2(__builtin_fmaf(S(i), c, -m_use)), p1 = fast_exp2(__builtin_fmaf(S(i + 1), c, -m_use));
        const bf16x2 pr = {(__bf16)p0, (__bf16)p1};
        sum += p0;
        sum += p1;
        rounded_sum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rounded_sum, false);
        P(i, pr[0]);
        P(i + 1, pr[1]);
    }
    return rounded ? rounded_sum : sum;
}

// O^T += V^T P^T for the 32 keys whose LDS tile starts at vl.
// k-slot s of MFMA cc is key 16*cc + 8*(s/4) + 4*(lane/32) + s%4 of the block.
template <int D>
__device__ __forceinline__ void pv32(uint32_t vl, const bf16x8 (&P)[2], WaveAcc<D>& st, int lane) {
    using G_ = Geo<D>;
    const int g = lane >> 5, hi = (lane >> 4) & 1, i16 = lane & 15;
    // the 16 lanes of a transpose read address 4 keys (4*g + i16/4 ..) x 16 consecutive d
    const int key = 4 * g + (i16 >> 2);
    // inside the 64-byte quad of d block db: bytes hi*32 + (i16&3)*8
    const uint32_t va = vl + (key / G_::KPW) * G_::GS + (key % G_::KPW) * 64 + hi * 32 + (i16 & 3) * 8;
    constexpr int K8 = (8 / G_::KPW) * G_::GS + (8 % G_::KPW) * 64;      // +8 keys
    constexpr int K16 = (16 / G_::KPW) * G_::GS;                        // +16 keys
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
        for (int db = 0; db < G_::NDB; ++db) {
            const uint32_t a0 = va + cc * K16 + db * (G_::KPW * 64);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0));
            const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0 + K8));
            const s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi4[0], hi4[1], hi4[2], hi4[3]};
            st.O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), P[cc], st.O[db], 0, 0, 0);
        }
    }
}

// One 32-key block, straight: used by narrow items (bandwidth-bound, no pipelining needed).
template <int D>
__device__ __forceinline__ void block32(uint32_t kl, uint32_t vl, const bf16x8 (&Q)[Geo<D>::NKK], WaveAcc<D>& st,
                                        float c, int rel, bool masked, bool rounded, int lane) {
    f32x16 S;
    bf16x8 P[2];
    qk32<D>(kl, Q, S, lane);
    if (masked) mask32(S, rel);                          // wave-uniform
    const float mx = rowmax32(S) * c;
    if (__any(mx > st.m + RESCALE_SLACK)) raise_reference<D>(st, mx);
    st.l += exp_sum<16>(c, st.m == NEG_INF ? 0.0f : st.m, rounded, [&](int i) { return S[i]; }, [&](int i, __bf16 v) { P[i >> 3][i & 7] = v; });
    pv32<D>(vl, P, st, lane);
}

// ---------------------------------------------------------------------------------------------
// The same steps for a wave of at most 16 query rows (a decode row's grouped heads), with v_mfma_f32_16x16x32_bf16:
// half the matrix and softmax work of the 32-row steps per key.  A lane owns query column lane % 16; with g = lane / 16
// it holds S^T for keys 4 k + i and 16 + 4 k + i (i < 4; k = key_group16(g)) of the block, which are also its eight k-slots
// of the second product, so P^T is again built in registers; O^T tile dt holds d = 16 dt + 4 g + i.

__device__ __forceinline__ float max_xor16(float x) {      // as max_xor32, for lane ^ 16
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor16(float x) {
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Which group of 4 keys (of the 16 keys of a tile) the lanes 16 g .. 16 g + 15 hold: 0, 2, 1, 3.  With this order the 32 lanes
// that one pass of a transpose read serves (g = 0, 1 or g = 2, 3) touch 256 contiguous bytes of the padded key groups
// (keys 0-3 and 8-11, or 4-7 and 12-15: LDS groups 16 bytes apart modulo 256) for d = 128; measured, the bank-conflict
// cycles of a decode launch are half of those with the order 0, 1, 2, 3.
__device__ __forceinline__ int key_group16(int g) { return ((g & 1) << 1) | ((g >> 1) & 1); }

template <int D>
struct WaveAcc16 {
    f32x4 O[D / 16];
    float m;
    float l;      // this lane's share of the running sum (the four lanes of a column hold quarters)
};

template <int D>
__device__ __forceinline__ void qk16(uint32_t kl, const bf16x8 (&Q)[D / 32], f32x4 (&S)[2], int lane) {
    using G_ = Geo<D>;
    // matrix row rho = lane % 16 carries key 4 * key_group16(rho / 4) + rho % 4 of the tile, so that lane group g ends up
    // with the keys of group key_group16(g)
    const int r = key_group16((lane & 15) >> 2) * 4 + (lane & 3), g = lane >> 4;
    // chunk 4*kk + g of key 16*t + r
    const uint32_t ka = kl + (r / G_::KPW) * G_::GS + (r % G_::KPW) * 64 + g * 16;
    constexpr int K16 = (16 / G_::KPW) * G_::GS;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        S[t] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) {
            const u32x4 raw = *LDS_PTR(const u32x4, ka + t * K16 + kk * (G_::KPW * 64));
            S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw), Q[kk], S[t], 0, 0, 0);
        }
    }
}

// rel: per lane, (last visible key of this lane's query) - (first key of the block) - 4*key_group16(lane/16)
__device__ __forceinline__ void mask16(f32x4 (&S)[2], int rel) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) S[t][i] = 16 * t + i <= rel ? S[t][i] : NEG_INF;
}

template <int D>
__device__ __forceinline__ void raise_reference16(WaveAcc16<D>& st, float mx) {
    const float m_new = fmaxf(st.m, mx);
    const float alpha = fast_exp2(st.m - (m_new == NEG_INF ? 0.0f : m_new));
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) st.O[dt] *= alpha;
    st.m = m_new;
}

template <int D>
__device__ __forceinline__ void pv16(uint32_t vl, const bf16x8& P, WaveAcc16<D>& st, int lane) {
    using G_ = Geo<D>;
    const int g = lane >> 4, i16 = lane & 15;
    // the 16 lanes of a transpose read address 4 keys x 16 consecutive d and receive 4 keys of one d each
    const int key = 4 * key_group16(g) + (i16 >> 2);
    const uint32_t va = vl + (key / G_::KPW) * G_::GS + (key % G_::KPW) * 64 + (i16 & 3) * 8;
    constexpr int K16 = (16 / G_::KPW) * G_::GS;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) {
        const uint32_t a0 = va + (dt >> 1) * (G_::KPW * 64) + (dt & 1) * 32;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0));
        const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0 + K16));
        const s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi4[0], hi4[1], hi4[2], hi4[3]};
        st.O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), P, st.O[dt], 0, 0, 0);
    }
}

// S^T and its softmax; P = the operand of the second product
template <int D>
__device__ __forceinline__ bf16x8 softmax16(uint32_t kl, const bf16x8 (&Q)[D / 32], WaveAcc16<D>& st, float c, int rel, bool masked, bool rounded, int lane) {
    f32x4 S[2];
    qk16<D>(kl, Q, S, lane);
    if (masked) mask16(S, rel);                          // wave-uniform
    float mx = fmaxf(fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3])), fmaxf(fmaxf(S[1][0], S[1][1]), fmaxf(S[1][2], S[1][3])));
    mx = max_xor32(max_xor16(mx)) * c;
    if (__any(mx > st.m + RESCALE_SLACK)) raise_reference16<D>(st, mx);
    bf16x8 P;
    st.l += exp_sum<8>(c, st.m == NEG_INF ? 0.0f : st.m, rounded, [&](int i) { return S[i >> 2][i & 3]; }, [&](int i, __bf16 v) { P[i] = v; });
    return P;
}

// ---------------------------------------------------------------------------------------------
// Software-pipelined processing of one LDS stage by one wave, at 32-key granularity.
//
// On this device the vector instructions of the softmax hide behind matrix instructions mostly when both come
// from the SAME wave, finely interleaved in program order (a SIMD running the products of one wave and the vector
// work of another needs the products' time plus two thirds of the vector work's time; interleaved in one wave, one
// quarter).  One pipeline iteration therefore carries, step by step,
//     one product of S^T(b+1) = K(b+1) Q^T,   the exponentials of a slice of block b,   one product of O^T += V(b-1)^T P(b-1)^T
// for three consecutive 32-key blocks, with the LDS fragment reads three steps ahead; scheduling fences keep the steps
// in this order.  The pipeline is filled and drained inside every stage (6 iterations for 4 blocks), because the next
// stage's K rows are only known to have landed after the barrier that ends this one.
//
// The exponentials of a block are taken against the reference the row already has; the block's own maximum is only
// looked at when that turned out too low (some probability above 2^12: the lane's sum says so) or when the row has
// no reference yet.  That check sits at the end of the iteration, where S^T(b) is still in registers and O holds the
// blocks up to b-1: the reference is raised, O and l are rescaled, and P(b) is redone in place.

// f(integral_constant<int, I>) for I = I0 .. N-1, unrolled at compile time (a runtime loop, even one marked for
// unrolling, leaves the fragment arrays below indexed at run time, i.e. in scratch memory)
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}


template <int D>
struct PipeState {
    f32x16 S[2];            // logits of two consecutive blocks (block b lives in S[b & 1])
    bf16x8 P[2][2];         // probabilities of two consecutive blocks
};

// All blocks of one stage (NB = KT / 32 blocks; K rows at kst, V rows at vst), for one wave: NB + 2 iterations of NS
// steps, written as one flat sequence of steps so that the fragment reads also run ahead across the iterations'
// ends (only the first PF steps of a stage wait for their LDS reads).  In iteration i, block i is multiplied
// (QK, i < NB), block i-1 exponentiated (SM), block i-2 multiplied into O (PV).
//   rel0: (last visible key of the lane's row) - (first key of the stage) - 4 * (lane / 32) (read when MASK).
template <int D, bool MASK>
__device__ __forceinline__ void stage_pipelined(uint32_t kst, uint32_t vst, const bf16x8 (&Q)[Geo<D>::NKK], WaveAcc<D>& st,
                                                PipeState<D>& ps, float c, int rel0, int lane) {
    using G_ = Geo<D>;
    constexpr int NB = KT / 32;
    constexpr int NS = G_::NKK;                      // steps per iteration: one K fragment and one V fragment per step
    constexpr int LPS = 16 / NS;                     // logits per lane and step
    constexpr int PF = 3;                            // fragment reads run this many steps ahead (2 to 4 measure alike, 5 and 6 slower)
    constexpr int NSTEP = (NB + 2) * NS;
    static_assert(2 * G_::NDB == NS && LPS % 2 == 0, "steps per block");
    const int g = lane >> 5, r = lane & 31, hi = (lane >> 4) & 1, i16 = lane & 15;
    const uint32_t ka = kst + (r / G_::KPW) * G_::GS + (r % G_::KPW) * 64 + g * 16;
    const int key = 4 * g + (i16 >> 2);
    const uint32_t va = vst + (key / G_::KPW) * G_::GS + (key % G_::KPW) * 64 + hi * 32 + (i16 & 3) * 8;
    constexpr int K8 = (8 / G_::KPW) * G_::GS + (8 % G_::KPW) * 64;      // +8 keys
    constexpr int K16 = (16 / G_::KPW) * G_::GS;                        // +16 keys
    // the fragments step t needs: K fragment t % NS of block t / NS (t < NB * NS), V fragment of block t / NS - 2
    u32x4 kf[NSTEP];
    s16x8 vf[NSTEP];
    auto fetch = [&](int t) {
        const int i = t / NS, j = t % NS;
        if (i < NB) kf[t] = *LDS_PTR(const u32x4, ka + i * G_::B32 + (j >> 1) * (G_::KPW * 64) + (j & 1) * 32);
        if (i >= 2) {                                // fragment j = cc * NDB + db
            const uint32_t a0 = va + (i - 2) * G_::B32 + (j / G_::NDB) * K16 + (j % G_::NDB) * (G_::KPW * 64);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0));
            const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a0 + K8));
            vf[t] = s16x8{lo[0], lo[1], lo[2], lo[3], h4[0], h4[1], h4[2], h4[3]};
        }
    };
    static_for<0, PF>([&](auto tc) { fetch(decltype(tc)::value); });
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float m_use = 0.0f, psum = 0.0f;
    static_for<0, NSTEP>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int i = t / NS, j = t % NS;
        constexpr bool QK = i < NB, SM = i >= 1 && i <= NB, PV = i >= 2;
        f32x16& S_out = ps.S[i & 1];
        f32x16& S_in = ps.S[(i + 1) & 1];            // block i - 1
        bf16x8 (&P_out)[2] = ps.P[(i + 1) & 1];
        const bf16x8 (&P_prev)[2] = ps.P[i & 1];     // block i - 2
        if constexpr (t + PF < NSTEP) fetch(t + PF);
        if constexpr (SM && j == 0) {
            if (MASK) mask32(S_in, rel0 - 32 * (i - 1));
            m_use = st.m == NEG_INF ? 0.0f : st.m;
            psum = 0.0f;
        }
        if constexpr (QK)
            S_out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[t]), Q[j], j == 0 ? f32x16{0} : S_out, 0, 0, 0);
        // the slice's exponentials go half before and half behind the second product, so that each half runs in the
        // shadow of one matrix instruction of this wave
        float p_even[LPS / 2];
        if constexpr (SM) {
#pragma unroll
            for (int h = 0; h < LPS / 2; ++h) p_even[h] = fast_exp2(__builtin_fmaf(S_in[j * LPS + 2 * h], c, -m_use));
        }
        if constexpr (SM && PV) __builtin_amdgcn_sched_barrier(0);
        if constexpr (PV)
            st.O[j % G_::NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[t]), P_prev[j / G_::NDB],
                                                                        st.O[j % G_::NDB], 0, 0, 0);
        if constexpr (SM) {
#pragma unroll
            for (int h = 0; h < LPS / 2; ++h) {
                const int e = j * LPS + 2 * h;
                const bf16x2 pr = {(__bf16)p_even[h], (__bf16)fast_exp2(__builtin_fmaf(S_in[e + 1], c, -m_use))};
                psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, psum, false);
                P_out[e >> 3][e & 7] = pr[0];
                P_out[e >> 3][(e + 1) & 7] = pr[1];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SM && j == NS - 1) {
            if (__any(st.m == NEG_INF || !(psum <= PSUM_LIMIT))) {                    // rare
                raise_reference<D>(st, rowmax32(S_in) * c);
                psum = exp32_dot(S_in, c, st.m == NEG_INF ? 0.0f : st.m, P_out, 0.0f);
            }
            st.l += psum;
        }
    });
}

// Load the B operand (Q^T) of one wave: lane holds row lane%32, d = kk*16 + (lane/32)*8 .. +8.
template <int D>
__device__ __forceinline__ void load_q(const AttnParams& p, const ItemCtx& ic, int tok, int head_in_group,
                                       bool valid, int lane, bf16x8 (&Q)[Geo<D>::NKK]) {
    const int g = lane >> 5;
    if (valid) {
        const int hq = ic.kvh * (p.Hq / p.Hkv) + ic.g0 + head_in_group;
        const char* src = static_cast<const char*>(p.q) + (((int64_t)(ic.row_off + tok) * p.Hq + hq) * D + g * 8) * 2;
#pragma unroll
        for (int kk = 0; kk < Geo<D>::NKK; ++kk)
            Q[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + kk * 32));
    } else {
#pragma unroll
        for (int kk = 0; kk < Geo<D>::NKK; ++kk) Q[kk] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    }
}

// The same for a wave of 16 rows: lane holds row lane%16, d = kk*32 + (lane/16)*8 .. +8.
template <int D>
__device__ __forceinline__ void load_q16(const AttnParams& p, const ItemCtx& ic, int tok, int head_in_group,
                                         bool valid, int lane, bf16x8 (&Q)[D / 32]) {
    const int g = lane >> 4;
    if (valid) {
        const int hq = ic.kvh * (p.Hq / p.Hkv) + ic.g0 + head_in_group;
        const char* src = static_cast<const char*>(p.q) + (((int64_t)(ic.row_off + tok) * p.Hq + hq) * D + g * 8) * 2;
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk)
            Q[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + kk * 64));
    } else {
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) Q[kk] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    }
}

// One wave-wide direct global -> LDS load: lane i moves the 16 bytes at gbase + voff_i to LDS
// byte lds + 16 i (gbase and lds wave-uniform; the LDS base travels in M0).  Written as inline
// assembly so that the compiler does not track it: its own LDS reads of the *other* pipeline
// stage would otherwise wait for these loads.  dma_wait() must precede the barrier that
// publishes the data.  Compiler-issued vmcnt waits stay correct: vector-memory loads retire in
// order, so extra loads in flight only make them stricter.  M0 is named as clobbered so that the compiler never
// assumes a value of its own survives the statement (it is a reserved register, which the compiler reports with a
// warning that is silenced here: nothing has to be preserved, M0 is rewritten before every use).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const char* gbase, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(gbase)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------------------------
// K/V tile loader.  NTHR threads move NKEYS consecutive keys (K and V rows) from the paged
// pools into LDS, one group (KPW keys, 1 KB) per wave and pass.  Page ids are fetched one
// tile earlier than the rows they address, so that the dependent block-table -> pool load
// chain is never on the critical path; a group never straddles a page, so the page id is
// wave-uniform: it is moved to a scalar register and the 64-bit address arithmetic runs on
// the scalar unit.  Lane i fetches the chunk that belongs in LDS slot i of its group.
//   DMA = true  (bf16 cache): global -> LDS directly (global_load_lds_dwordx4), no staging
//                 registers; the data is in LDS once the vector-memory counter has drained,
//                 which the barrier that ends a pipeline step waits for.
//   DMA = false: global -> registers (fetch_kv) -> LDS (commit), widening 8-bit codes.
template <int D, int KVT, int NTHR, int NKEYS>
struct Loader {
    using G_ = Geo<D>;
    static constexpr int KPW = G_::KPW;
    static constexpr int NGRP = NKEYS / KPW;          // groups per tile
    static constexpr int NW = NTHR / 64;              // cooperating waves
    // 8-bit cache: a wave moves two consecutive groups per pass, 16 codes per lane (lanes 0-31 the first group, 32-63 the
    // second; a lane fills two neighbouring LDS slots): half as many loads and address computations per byte as with
    // one 8-byte chunk per lane.  Two groups are 8 or 16 keys from a multiple of that, so they share a page too.
    static constexpr int GPP = KVT == KV_FP8 ? 2 : 1; // groups per wave and pass
    static constexpr int KPP = GPP * KPW;             // keys per wave and pass
    static constexpr int NPASS = NGRP / (NW * GPP);
    static_assert(NPASS >= 1 && NPASS * NW * GPP == NGRP, "tile, waves and passes");
    static constexpr int ES = RawChunk<KVT>::ES;
    int pg[NPASS];
    RawChunk<KVT> k[NPASS], v[NPASS];
    float ks[NPASS], vs[NPASS];                       // 8-bit cache: the page scales of the passes

    // t: thread index inside the group of NTHR threads.  The block table is read through the
    // scalar cache (it is constant for the duration of the kernel): scalar loads do not count
    // as vector-memory loads, so waiting for a page id never waits for K/V data in flight.
    // (They do share a counter with LDS reads: the register-staged paths and the first stage
    // of a wide item use this variant, the direct-load pipeline uses fetch_pages_v below.)
    __device__ __forceinline__ void fetch_pages(const AttnParams& p, const ItemCtx& ic, int kbase, int t) {
        const auto* bt = reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(
            reinterpret_cast<uintptr_t>(ic.bt_row));
        const int w = __builtin_amdgcn_readfirstlane(t >> 6);
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) {
            const int key0 = kbase + (ps * NW + w) * KPP;
            pg[ps] = key0 < ic.kv_end ? bt[key0 >> p.logP] : 0;
        }
    }
    // The same page ids through the vector memory path, for the direct-load pipeline of wide items: lane ps of a
    // wave fetches the id of the wave's pass ps with one load, and take_pages() moves the ids into scalar registers
    // once the load has landed.  Scalar loads share their counter with LDS reads and return out of order, so a wave
    // with page ids in flight has to drain that counter completely at its next fragment read; vector loads retire
    // in order behind the direct loads of the same step, and the wait that ends the step covers them.
    int pgv;
    __device__ __forceinline__ void fetch_pages_v(const AttnParams& p, const ItemCtx& ic, int kbase, int t) {
        const int key0 = kbase + (((t & 63) % NPASS) * NW + (t >> 6)) * KPP;
        pgv = key0 < ic.kv_end ? ic.bt_row[key0 >> p.logP] : 0;
    }
    __device__ __forceinline__ void take_pages() {
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) pg[ps] = __builtin_amdgcn_readlane(pgv, ps);
    }

    // The lane's first LDS slot inside its group, and which of the pass's groups that is.  Slot l = (quad, key, chunk in
    // quad); with two groups per pass a lane owns slots l and l + 1 (l even: neighbouring chunks of one key row).
    __device__ __forceinline__ static int lane_slot(int t) { return GPP == 1 ? (t & 63) : 2 * (t & 31); }
    __device__ __forceinline__ static int lane_group(int t) { return GPP == 1 ? 0 : (t & 63) >> 5; }
    __device__ __forceinline__ static int lane_key(int t) { return lane_group(t) * KPW + (lane_slot(t) >> 2) % KPW; }   // within the pass
    __device__ __forceinline__ static uint32_t lane_off(int t) {
        const int l = lane_slot(t);
        return (uint32_t)((lane_key(t) * D + ((l / (4 * KPW)) * 4 + (l & 3)) * 8) * ES);
    }

    struct Row {
        const char *kb, *vb;
        int key0, page;
    };
    __device__ __forceinline__ Row row_of(const AttnParams& p, const ItemCtx& ic, int kbase, int t, int ps) const {
        Row r;
        r.key0 = __builtin_amdgcn_readfirstlane(kbase + (ps * NW + (t >> 6)) * KPP);
        r.page = __builtin_amdgcn_readfirstlane(pg[ps]);
        const int64_t row = ((((int64_t)r.page * p.Hkv + ic.kvh) << p.logP) + (r.key0 & (p.P - 1))) * D * ES;
        r.kb = static_cast<const char*>(p.k_pool) + row;
        r.vb = static_cast<const char*>(p.v_pool) + row;
        return r;
    }
    // The same group when its keys are new tokens of this call: packed rows [token][Hkv][D] of k_new / v_new (bf16
    // cache only).  The base is the row of the group's first key (for a group that straddles C it lies before the
    // request's first row and is only ever used by lanes whose key is >= C); consecutive keys are Hkv rows apart.
    __device__ __forceinline__ Row new_row_of(const AttnParams& p, const ItemCtx& ic, const Row& r) const {
        Row n = r;
        const int64_t off = (((int64_t)ic.row_off + (r.key0 - ic.C)) * p.Hkv + ic.kvh) * (D * 2);
        n.kb = reinterpret_cast<const char*>(reinterpret_cast<intptr_t>(p.k_new) + off);
        n.vb = reinterpret_cast<const char*>(reinterpret_cast<intptr_t>(p.v_new) + off);
        return n;
    }
    __device__ __forceinline__ static uint32_t new_lane_off(const AttnParams& p, int t) {
        const int l = t & 63;
        return (uint32_t)(((l >> 2) % KPW) * p.Hkv * D * 2 + ((l / (4 * KPW)) * 4 + (l & 3)) * 16);
    }

    // ---- register-staged path
    // FULL: the whole tile lies inside the key range and in the pages
    template <bool FULL>
    __device__ __forceinline__ void fetch_kv_impl(const AttnParams& p, const ItemCtx& ic, int kbase, int t) {
        const uint32_t lo = lane_off(t);
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) {
            const Row r = row_of(p, ic, kbase, t, ps);
            ks[ps] = vs[ps] = 1.0f;
            if (KVT == KV_FP8 && (FULL || r.key0 < ic.kv_end)) {      // (a group past the key range has no page)
                ks[ps] = p.k_scale[(int64_t)r.page * p.Hkv + ic.kvh];
                vs[ps] = p.v_scale[(int64_t)r.page * p.Hkv + ic.kvh];
            }
            const int key = r.key0 + lane_key(t);
            if (FULL || (key < ic.kv_end && key < ic.c_rows)) {
                k[ps].load(r.kb, lo);
                v[ps].load(r.vb, lo);
            } else if (KVT == KV_BF16 && key < ic.kv_end) {      // a new token of this call: read its packed row
                const Row n = new_row_of(p, ic, r);
                const uint32_t nlo = new_lane_off(p, t);
                k[ps].load(n.kb, nlo);
                v[ps].load(n.vb, nlo);
            } else {
                k[ps].zero();                                    // keys past the item's end: zeros, so
                v[ps].zero();                                    // that 0-weights never meet NaN garbage
            }
        }
    }
    __device__ __forceinline__ void fetch_kv(const AttnParams& p, const ItemCtx& ic, int kbase, int t) {
        if (kbase + NKEYS <= min(ic.kv_end, ic.c_rows))          // uniform: whole tile inside the key range, in pages
            fetch_kv_impl<true>(p, ic, kbase, t);
        else
            fetch_kv_impl<false>(p, ic, kbase, t);
    }
    // kl / vl: LDS byte addresses of this tile's K and V
    __device__ __forceinline__ void commit(uint32_t kl, uint32_t vl, int t) const {
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) {
            put(k[ps], ks[ps], kl + slot_of(ps, t));
            put(v[ps], vs[ps], vl + slot_of(ps, t));
        }
    }
    __device__ __forceinline__ static uint32_t slot_of(int ps, int t) {
        return ((ps * NW + (t >> 6)) * GPP + lane_group(t)) * G_::GS + lane_slot(t) * 16;
    }
    __device__ __forceinline__ static void put(const RawChunk<KVT>& c, float scale, uint32_t at) {
        if constexpr (KVT == KV_FP8) {
            *LDS_PTR(u32x4, at) = c.widen_first(scale);
            *LDS_PTR(u32x4, at + 16) = c.widen_second(scale);
        } else {
            *LDS_PTR(u32x4, at) = c.widen(scale);
        }
    }

    // ---- direct path (bf16 only)
    template <bool FULL>
    __device__ __forceinline__ void dma_impl(const AttnParams& p, const ItemCtx& ic, int kbase, int t, uint32_t kl,
                                             uint32_t vl) const {
        const uint32_t lo = lane_off(t);
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) {
            const Row r = row_of(p, ic, kbase, t, ps);
            // wave-uniform LDS offset of the group
            const uint32_t go = __builtin_amdgcn_readfirstlane((ps * NW + (t >> 6)) * G_::GS);
            const int key = r.key0 + lane_key(t);
            if (FULL || (key < ic.kv_end && key < ic.c_rows)) {
                dma16(r.kb, lo, __builtin_amdgcn_readfirstlane(kl) + go);
                dma16(r.vb, lo, __builtin_amdgcn_readfirstlane(vl) + go);
            } else if (key < ic.kv_end) {                        // a new token of this call: its packed row
                const Row n = new_row_of(p, ic, r);
                const uint32_t nlo = new_lane_off(p, t);
                dma16(n.kb, nlo, __builtin_amdgcn_readfirstlane(kl) + go);
                dma16(n.vb, nlo, __builtin_amdgcn_readfirstlane(vl) + go);
            } else {
                *LDS_PTR(u32x4, kl + go + (t & 63) * 16) = u32x4{0, 0, 0, 0};
                *LDS_PTR(u32x4, vl + go + (t & 63) * 16) = u32x4{0, 0, 0, 0};
            }
        }
    }
    __device__ __forceinline__ void dma(const AttnParams& p, const ItemCtx& ic, int kbase, int t, uint32_t kl,
                                        uint32_t vl) const {
        if (kbase + NKEYS <= min(ic.kv_end, ic.c_rows))
            dma_impl<true>(p, ic, kbase, t, kl, vl);
        else
            dma_impl<false>(p, ic, kbase, t, kl, vl);
    }
};

// Final write of one wave's O^T of a tile: either bf16 output rows or fp32 partials.  A lane holds scattered quads of one row,
// so the wave turns its rows around in LDS (16-byte chunks, exclusive-or swizzled by the row: no bank is hit more than twice)
// and stores 16 consecutive bytes per lane, whole rows per instruction: written straight from the accumulators, every store
// instruction touched 32 rows 16 or 32 bytes at a time (per call, before -> now: one prefill of 509 tokens over 4 099 in 256
// pieces 59.0 -> 56.7 us, 24 decode rows next to a prefill of 701 over an 8-bit cache 114.0 -> 110.5, 16 prefills -1 %).
//   wbase: 32 * D * 4 bytes of LDS of this wave's own (the stages are free by then); wave_row0: the wave's first row in the item
template <int D>
__device__ __forceinline__ void store_tile(const AttnParams& p, const ItemCtx& ic, WaveAcc<D>& st, uint32_t wbase, int wave_tok0,
                                           int tqw, int lane) {
    using G_ = Geo<D>;
    const int g = lane >> 5, row = lane & 31;
    const float ltot = sum_xor32(st.l);
    const int nrows = min(tqw, ic.nq - wave_tok0) * ic.gn;          // rows of this wave (<= 0: none)
    if (ic.part_off < 0) {
        constexpr int CPR = D / 8;                                  // 16-byte chunks per output row
        const float inv = 1.0f / ltot;
#pragma unroll
        for (int db = 0; db < G_::NDB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const bf16x4 o = {(__bf16)(st.O[db][i4 * 4] * inv), (__bf16)(st.O[db][i4 * 4 + 1] * inv),
                                  (__bf16)(st.O[db][i4 * 4 + 2] * inv), (__bf16)(st.O[db][i4 * 4 + 3] * inv)};
                *LDS_PTR(u32x2, wbase + row * (CPR * 16) + (((db * 4 + i4) ^ (row & (CPR - 1))) * 16) + g * 8) = __builtin_bit_cast(u32x2, o);
            }
        const int magic = (65536 + ic.gn - 1) / ic.gn;              // r / gn = r * magic >> 16 for r < 32
        char* out = static_cast<char*>(p.out) +
                    (((int64_t)(ic.row_off + ic.q0 + wave_tok0) * p.Hq + ic.kvh * (p.Hq / p.Hkv) + ic.g0) * D) * 2;
#pragma unroll
        for (int k = 0; k < 32 * CPR / 64; ++k) {
            const int r = k * (64 / CPR) + lane / CPR, c = lane % CPR;
            const u32x4 v = *LDS_PTR(const u32x4, wbase + r * (CPR * 16) + (c ^ (r & (CPR - 1))) * 16);
            const int tl = (r * magic) >> 16, hg = r - tl * ic.gn;
            if (r < nrows) *reinterpret_cast<u32x4*>(out + ((int64_t)tl * p.Hq + hg) * (D * 2) + c * 16) = v;
        }
    } else {
        constexpr int CPR = D / 4;                                  // 16-byte chunks per partial row
#pragma unroll
        for (int db = 0; db < G_::NDB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 o = {st.O[db][i4 * 4], st.O[db][i4 * 4 + 1], st.O[db][i4 * 4 + 2], st.O[db][i4 * 4 + 3]};
                *LDS_PTR(f32x4, wbase + row * (CPR * 16) + (((db * 8 + i4 * 2 + g) ^ (row & (CPR - 1))) * 16)) = o;
            }
        const int rows = ic.nq * ic.gn, row0 = wave_tok0 * ic.gn;
        float* po = p.partial + ic.part_off + (int64_t)row0 * D;
#pragma unroll
        for (int k = 0; k < 32 * CPR / 64; ++k) {
            const int r = k * (64 / CPR) + lane / CPR, c = lane % CPR;
            const f32x4 v = *LDS_PTR(const f32x4, wbase + r * (CPR * 16) + (c ^ (r & (CPR - 1))) * 16);
            if (r < nrows) *reinterpret_cast<f32x4*>(po + r * D + c * 4) = v;
        }
        if (g == 0 && row < nrows) {
            float* ml = p.partial + ic.part_off + (int64_t)rows * D + (row0 + row) * 2;
            ml[0] = st.m;
            ml[1] = ltot;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// wide body: 8 waves x 32 query rows share 128-key K/V stages (two in LDS: one consumed, one being filled).
// bf16 cache: stages travel global -> LDS directly, issued by one wave of every SIMD; one barrier per stage.
// 8-bit cache: register-staged and widened on the way into LDS, by all waves.

template <int D, int KVT>
__device__ __forceinline__ void wide_body(const AttnParams& p, const ItemCtx& ic, uint32_t smem, int tid) {
    using G_ = Geo<D>;
    constexpr bool DMA = KVT == KV_BF16;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tqw = 32 / ic.gn;                            // tokens per wave
    const int row = lane & 31;
    const int tl = row / ic.gn, hg = row - tl * ic.gn;
    const int tok_local = wave * tqw + tl;                 // token index inside the item
    const bool valid = tl < tqw && tok_local < ic.nq;
    const int tok = ic.q0 + tok_local;
    // wave-level causal bounds (last visible key = C + token)
    const int w_last = ic.C + ic.q0 + min(wave * tqw + tqw, ic.nq) - 1;
    const bool wave_active = wave * tqw < ic.nq;
    const int lim = valid ? ic.C + tok : 0x3fffffff;

    bf16x8 Q[G_::NKK];
    load_q<D>(p, ic, tok, hg, valid, lane, Q);
    WaveAcc<D> st;
#pragma unroll
    for (int db = 0; db < G_::NDB; ++db) st.O[db] = f32x16{0};
    st.m = NEG_INF;
    st.l = 0.0f;

    const int k_lo = ic.kv_begin;                          // multiple of 64
    const int ntiles = (ic.kv_end - k_lo + KT - 1) / KT;
    const int nfull = (ic.kv_end - k_lo) / KT;             // tiles 0..nfull-1 lie entirely inside the key range
    // Tiles whose last key is visible to every row of the workgroup need no causal select;
    // the remaining (at most a few) tiles around the diagonal take the masked variant.
    const int wg_first = ic.C + ic.q0;                     // smallest last-visible key in the workgroup
    const int t_diag = min(min(ntiles, nfull), max(0, (wg_first + 1 - k_lo) / KT));   // (a ragged last stage is masked too)
    Loader<D, KVT, AWG, KT> ld;
    PipeState<D> ps;
    // keys from kv_end on (the ragged tail of the last stage) count as masked
    const int lim_eff = min(lim, ic.kv_end - 1);
    // a wave without rows, or one whose rows all end before this stage, skips it
    auto computes = [&](int t) { return wave_active && k_lo + t * KT <= w_last; };
    auto compute = [&](int t, uint32_t stage, auto masked) {
        const int kbase = k_lo + t * KT;
        if (computes(t))
            stage_pipelined<D, decltype(masked)::value>(stage, stage + G_::KTILE, Q, st, ps, p.c_log2,
                                                        lim_eff - kbase - 4 * (lane >> 5), lane);
    };
    if (DMA) {
        // Who issues the direct loads.  The CU's memory pipeline takes one 1 KB direct load every ~23 cycles, and a
        // wave whose load finds the queue full is blocked (instructions issue in order) and computes nothing: when all
        // eight waves issued their share at the start of a stage, the matrix pipes of all four SIMDs stood still for
        // the ~1 500 cycles the 64 loads of a stage need, in every stage.  So only one wave of every SIMD loads (waves
        // w and w + 4 share a SIMD): the four loading waves issue the whole next stage at the start of a stage while
        // their SIMD partners already compute, and catch up afterwards.  A tile with rows for at most four waves lets
        // its idle half do the loading.
        static_assert(NSTAGE == 2, "tile t + 1 is loaded during stage t; the page ids of tile t + 2 travel behind it");
        constexpr int LW = ATTN_WAVES / 2;
        using LD = Loader<D, KVT, 64 * LW, KT>;
        LD ldh;
        const int n_active = (ic.nq + tqw - 1) / tqw;      // waves that have rows
        const int lbase = n_active <= LW ? LW : 0;
        const bool loader = wave >= lbase && wave < lbase + LW;
        const int lt = tid - lbase * 64;                   // thread index among the loading waves
        if (loader) {
            ldh.fetch_pages(p, ic, k_lo, lt);
            ldh.dma(p, ic, k_lo, lt, smem, smem + G_::KTILE);
            if (ntiles > 1) ldh.fetch_pages_v(p, ic, k_lo + KT, lt);
        }
        dma_wait();
        __syncthreads();
        auto step = [&](int t, auto masked) {
            if (loader && t + 1 < ntiles) {
                const uint32_t sg = smem + ((t + 1) % NSTAGE) * G_::WIDE_STAGE;
                ldh.take_pages();                          // (their load was waited for at the end of the previous step)
                ldh.dma(p, ic, k_lo + (t + 1) * KT, lt, sg, sg + G_::KTILE);
                if (t + 2 < ntiles) ldh.fetch_pages_v(p, ic, k_lo + (t + 2) * KT, lt);
            }
            compute(t, smem + (t % NSTAGE) * G_::WIDE_STAGE, masked);
            dma_wait();                                    // tile t+1 and the page ids of tile t+2 have landed
            __syncthreads();
        };
        for (int t = 0; t < t_diag; ++t) step(t, std::false_type{});
        for (int t = t_diag; t < ntiles; ++t) step(t, std::true_type{});
    } else {
        static_assert(NSTAGE >= 2, "two stages for the register-staged path");
        ld.fetch_pages(p, ic, k_lo, tid);
        ld.fetch_kv(p, ic, k_lo, tid);
        if (ntiles > 1) ld.fetch_pages(p, ic, k_lo + KT, tid);
        ld.commit(smem, smem + G_::KTILE, tid);
        __syncthreads();
        auto step = [&](int t, auto masked) {
            const uint32_t cur = smem + (t & 1) * G_::WIDE_STAGE;
            const uint32_t nxt = smem + ((t + 1) & 1) * G_::WIDE_STAGE;
            const bool more = t + 1 < ntiles;
            if (more) {
                ld.fetch_kv(p, ic, k_lo + (t + 1) * KT, tid);
                if (t + 2 < ntiles) ld.fetch_pages(p, ic, k_lo + (t + 2) * KT, tid);
            }
            compute(t, cur, masked);
            if (more) ld.commit(nxt, nxt + G_::KTILE, tid);
            __syncthreads();
        };
        for (int t = 0; t < t_diag; ++t) step(t, std::false_type{});
        for (int t = t_diag; t < ntiles; ++t) step(t, std::true_type{});
    }
    store_tile<D>(p, ic, st, smem + wave * (32 * D * 4), wave * tqw, tqw, lane);
}

// ---------------------------------------------------------------------------------------------
// quantising new tokens into an 8-bit cache: the steps, and the two forms in which a decode row's item appends its own

__device__ __forceinline__ int exponent_for(float amax) {
    // smallest e with amax <= 448 * 2^e  (448 = 1.75 * 2^8), clamped to [-40, 119]
    const uint32_t u = __float_as_uint(amax);
    const int ex = (int)(u >> 23) - 127;
    const uint32_t man = u & 0x7fffffu;
    int e = (man <= 0x600000u) ? ex - 8 : ex - 7;
    if ((u >> 23) == 0) e = -40;                              // zero / subnormal
    return min(119, max(-40, e));
}

__device__ __forceinline__ uint32_t encode4(float a, float b, float c, float d) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    return (uint32_t)w;
}

// The three passes over one (page, KV head) of K or V that an append into an 8-bit cache takes, by nthr threads (this one: t).
// src: packed row of the first new token of this page and head (consecutive tokens row_bytes apart); n: new tokens of the page.
__device__ __forceinline__ u32x4 new_chunk(const char* src, int64_t row_bytes, int u, int cph) {
    return *reinterpret_cast<const u32x4*>(src + (u / cph) * row_bytes + (u % cph) * 16);
}
__device__ __forceinline__ float chunk_amax(const u32x4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    float amax = 0.0f;
#pragma unroll
    for (int x = 0; x < 4; ++x) amax = fmaxf(amax, fmaxf(fabsf(__uint_as_float(w[x] << 16)), fabsf(__uint_as_float(w[x] & 0xffff0000u))));
    return amax;
}
__device__ __forceinline__ u32x2 encode_chunk(const u32x4& v, float inv) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    float f[8];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        f[2 * x] = __uint_as_float(w[x] << 16) * inv;
        f[2 * x + 1] = __uint_as_float(w[x] & 0xffff0000u) * inv;
    }
    return u32x2{encode4(f[0], f[1], f[2], f[3]), encode4(f[4], f[5], f[6], f[7])};
}
// this thread's largest magnitude
__device__ __forceinline__ float page_amax(const char* src, int64_t row_bytes, int n, int cph, int t, int nthr) {
    float amax = 0.0f;
    for (int u = t; u < n * cph; u += nthr) amax = fmaxf(amax, chunk_amax(new_chunk(src, row_bytes, u, cph)));
    return amax;
}
// the page's first n_old slots held codes of exponent e_old: re-encode them for e > e_old
__device__ __forceinline__ void page_reencode(uint8_t* pg, int n_old, int D, int e_old, int e, int t, int nthr) {
    const float f = __uint_as_float((uint32_t)(e_old - e + 127) << 23);     // 2^(e_old - e)
    for (int u = t; u < n_old * (D / 4); u += nthr) {
        uint32_t* q4 = reinterpret_cast<uint32_t*>(pg) + u;
        const uint32_t w = *q4;
        const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(w, false);
        const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
        *q4 = encode4(lo.x * f, lo.y * f, hi.x * f, hi.y * f);
    }
}
// encode the new tokens into the slots from dst on: x * 2^-e, |.| <= 448 by construction
__device__ __forceinline__ void page_encode(uint8_t* dst, const char* src, int64_t row_bytes, int n, int D, int e, int t, int nthr) {
    const int cph = D / 8;
    const float inv = __uint_as_float((uint32_t)(127 - e) << 23);
    for (int u = t; u < n * cph; u += nthr)
        *reinterpret_cast<u32x2*>(dst + (u / cph) * D + (u % cph) * 8) = encode_chunk(new_chunk(src, row_bytes, u, cph), inv);
}

// The append of an item's own new tokens into an 8-bit cache (launches of decode rows alone: one item holds all pages of its
// KV head that new tokens fall into, or shares them with a neighbour page by page, since pieces start at multiples of 64 keys).
// A wave takes one (page, K or V) at a time.
template <int D, int NW>
__device__ __forceinline__ void append_item_pages(const AttnParams& p, const ItemCtx& ic, int tid) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = max(ic.C, ic.kv_begin);
    const int lp0 = first >> p.logP, npages = ((ic.kv_end - 1) >> p.logP) - lp0 + 1;
    const int64_t row_bytes = (int64_t)p.Hkv * D * 2;
    for (int w = wave; w < 2 * npages; w += NW) {
        const int lp = lp0 + (w >> 1), is_v = w & 1;
        const int t0 = max(first, lp << p.logP), t1 = min(ic.kv_end, (lp + 1) << p.logP);
        const int n_old = max(0, ic.C - (lp << p.logP));
        const int page = ic.bt_row[lp];
        const char* src = static_cast<const char*>(is_v ? p.v_new : p.k_new) +
                          ((int64_t)(ic.row_off + t0 - ic.C) * p.Hkv + ic.kvh) * D * 2;
        float* scl = const_cast<float*>(is_v ? p.v_scale : p.k_scale) + (int64_t)page * p.Hkv + ic.kvh;
        uint8_t* pg = static_cast<uint8_t*>(const_cast<void*>(is_v ? p.v_pool : p.k_pool)) +
                      (((int64_t)page * p.Hkv + ic.kvh) << p.logP) * D;
        const float s_old = n_old > 0 ? *scl : 0.0f;
        float amax = page_amax(src, row_bytes, t1 - t0, D / 8, lane, 64);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        int e = exponent_for(amax);
        if (n_old > 0) {
            const int e_old = (int)(__float_as_uint(s_old) >> 23) - 127;
            if (e > e_old)
                page_reencode(pg, n_old, D, e_old, e, lane, 64);
            else
                e = e_old;
        }
        page_encode(pg + (int64_t)(t0 & (p.P - 1)) * D, src, row_bytes, t1 - t0, D, e, lane, 64);
        if (lane == 0) *scl = __uint_as_float((uint32_t)(e + 127) << 23);
    }
}

// The same for a row with one new token (a decode step) whose page's cached tokens all lie in the row's last block (see
// page_in_last_block: finish() may re-encode every one of them, and no other wave may be reading them), by the one wave that
// streams that block, without holding up the others: start() issues the loads before the wave streams its first block, finish()
// encodes and stores when the wave is about to fetch the last block.  Lanes 0 .. D/8 - 1 carry K, as many after them V.  (Done by the whole workgroup in front of its stream instead, the append cost a launch of 608 items 6 us.)
template <int D>
struct NewToken {
    static constexpr int CPK = D / 8;
    u32x4 row;
    float s_old;
    int page;
    __device__ __forceinline__ static bool carries(int lane) { return lane < 2 * CPK; }
    __device__ __forceinline__ static bool is_v(int lane) { return lane >= CPK; }
    __device__ __forceinline__ static float* scale(const AttnParams& p, const ItemCtx& ic, int page, int lane) {
        return const_cast<float*>(is_v(lane) ? p.v_scale : p.k_scale) + (int64_t)page * p.Hkv + ic.kvh;
    }
    __device__ __forceinline__ void start(const AttnParams& p, const ItemCtx& ic, int lane) {
        page = ic.bt_row[ic.C >> p.logP];
        if (carries(lane))
            row = *reinterpret_cast<const u32x4*>(static_cast<const char*>(is_v(lane) ? p.v_new : p.k_new) +
                                                  (((int64_t)ic.row_off * p.Hkv + ic.kvh) * D + (lane % CPK) * 8) * 2);
    }
    __device__ __forceinline__ void start_scale(const AttnParams& p, const ItemCtx& ic, int lane) {
        if (carries(lane)) s_old = *scale(p, ic, page, lane);
    }
    __device__ __forceinline__ void finish(const AttnParams& p, const ItemCtx& ic, int lane) {
        const uint32_t w[4] = {row.x, row.y, row.z, row.w};
        float f[8], amax = 0.0f;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            f[2 * x] = __uint_as_float(w[x] << 16);
            f[2 * x + 1] = __uint_as_float(w[x] & 0xffff0000u);
            amax = fmaxf(amax, fmaxf(fabsf(f[2 * x]), fabsf(f[2 * x + 1])));
        }
#pragma unroll
        for (int o = CPK / 2; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        const int slot = ic.C & (p.P - 1);                    // = tokens the page already holds
        int e = exponent_for(amax);
        const int e_old = slot > 0 ? (int)(__float_as_uint(s_old) >> 23) - 127 : e;
        const int64_t tile = (((int64_t)page * p.Hkv + ic.kvh) << p.logP) * D;
        if (__any(carries(lane) && e > e_old)) {              // rare: the page's exponent rises
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int ne = __builtin_amdgcn_readlane(e, v * CPK), oe = __builtin_amdgcn_readlane(e_old, v * CPK);
                if (ne > oe)
                    page_reencode(static_cast<uint8_t*>(const_cast<void*>(v ? p.v_pool : p.k_pool)) + tile, slot, D, oe, ne, lane, 64);
            }
        }
        e = max(e, e_old);
        if (carries(lane)) {
            const float inv = __uint_as_float((uint32_t)(127 - e) << 23);
            const u32x2 o = {encode4(f[0] * inv, f[1] * inv, f[2] * inv, f[3] * inv), encode4(f[4] * inv, f[5] * inv, f[6] * inv, f[7] * inv)};
            uint8_t* pg = static_cast<uint8_t*>(const_cast<void*>(is_v(lane) ? p.v_pool : p.k_pool)) + tile;
            *reinterpret_cast<u32x2*>(pg + slot * D + (lane % CPK) * 8) = o;
            if (lane % CPK == 0) *scale(p, ic, page, lane) = __uint_as_float((uint32_t)(e + 127) << 23);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave's own stores and loads stay in order
    }
};

// ---------------------------------------------------------------------------------------------
// narrow body: <= 32 query rows; the 32-key blocks of the key range belong round-robin to 8 softmax states, which are
// merged through LDS at the end.  A workgroup of 8 waves keeps one state per wave, one of 4 waves two per wave (the same
// blocks in the same order per state, so the result is the same bit for bit); a wave stages its blocks through an LDS
// region of its own.

// K/V loader of one wave of a narrow item: 32-key blocks (from a multiple of 32), global -> registers -> the wave's LDS region.
// A wave alone issues an instruction every four cycles or more, and the block loop used to be bound by that: page ids, branches and
// 64-bit addresses for every 1 KB load were a quarter of its instructions.  A block touches at most two pages (page size >= 16), so it
// takes one address per half block, the loads of a half differ in their immediate offset only, and one vector load fetches
// the page ids of the wave's next 8 blocks (scalar loads share their counter with LDS reads and return out of order: the first
// fragment read of every block waited for the next block's page ids).  bf16 d = 128: 240 instructions a block instead of 330.
// Four rows over 36-70 k keys 26.6 -> 25.9 us; 90 drawn batches: decode at d = 128 0.98 of its time before, at d = 64 (a block always
// was two or four loads a side) 1.00, mixed 0.99, small prefill 0.98.
// Loads are non-temporal: a decode row's keys are read once and should not displace L2 lines (plain loads: more than 128 rows of up to
// 2 k tokens 1.06 in 8 bits, 1.2 in bf16).  The eight blocks of a prefill row that share keys on a die find most of them in its L2 all the same
// (256 tokens over 2 048: 85 % hits; 102 such launches with plain loads 1.00, the worst 1.05, the best 0.98).
template <int D, int KVT>
struct BlockLoader {
    using G_ = Geo<D>;
    using T = Loader<D, KVT, 64, 32>;                 // the lane's place in a load and in LDS
    static constexpr int ES = RawChunk<KVT>::ES;
    static constexpr int KPL = 1024 / (D * ES);       // keys per load
    static constexpr int LPH = 16 / KPL;              // loads per half block
    static constexpr int NL = 2 * LPH;
    static_assert(KPL == T::KPP && LPH >= 1 && 1024 * LPH <= 4096, "a half block is addressed by immediate offsets");
    RawChunk<KVT> k[NL], v[NL];
    static constexpr int IDS = 8;                     // blocks whose page ids one load fetches
    int ids;                                          // lane 2 n + h: page of half h of the wave's block j / IDS * IDS + n
    int page[2];                                      // of the block that is fetched next
    int64_t off[2];                                   // byte offset of the fetched block's halves in the pools
    float scale[4];                                   // 8-bit cache: [h]: K's scale of half h's page, [2 + h]: V's
    float sc[4];                                      // the same of the block that is being committed

    // page ids of the wave's blocks j .. j + IDS - 1 (j a multiple of IDS); past the key range: the last key's page
    __device__ __forceinline__ void fetch_ids(const AttnParams& p, const ItemCtx& ic, int first_key, int step, int j, int lane) {
        const int key = first_key + (j + (lane >> 1) % IDS) * step + (lane & 1) * 16;
        ids = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(ic.bt_row) + (uint32_t)(min(key, ic.kv_end - 1) >> p.logP) * 4u);
    }
    __device__ __forceinline__ void take_pages(int j) {
        page[0] = __builtin_amdgcn_readlane(ids, 2 * (j % IDS));
        page[1] = __builtin_amdgcn_readlane(ids, 2 * (j % IDS) + 1);
    }
    __device__ __forceinline__ void locate(const AttnParams& p, const ItemCtx& ic, int kbase) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            off[h] = ((((int64_t)page[h] * p.Hkv + ic.kvh) << p.logP) + ((kbase + 16 * h) & (p.P - 1))) * (D * ES);
    }
    __device__ __forceinline__ void fetch_scales(const AttnParams& p, const ItemCtx& ic) {
        // through the vector memory path: this workgroup may have written one itself, see append_item_pages, and the scalar
        // cache would not see the store.  Four loads of one address each: one of four addresses with the scales read out of its
        // lanes costs 1.5 % at d = 64, 40 drawn decode batches.
        if constexpr (KVT == KV_FP8) {
#pragma unroll
            for (int l = 0; l < 4; ++l)
                scale[l] = __hip_atomic_load((l & 2 ? p.v_scale : p.k_scale) + ic.kvh + (int64_t)page[l & 1] * p.Hkv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    // Every block issues the same number of loads (so that waiting for the older of two operands never waits for the younger one as
    // well): a slot past the key range is the last key's once more, and zeroed by commit_v.
    template <bool DO_K, bool DO_V, bool SPACED>
    __device__ __forceinline__ void fetch_kv(const AttnParams& p, const ItemCtx& ic, int kbase, int lane) {
        uint32_t lo = T::lane_off(lane);
        const bool plain = kbase + 32 <= min(ic.kv_end, ic.c_rows);     // uniform: all keys in pages (8-bit: or anything there)
        if (plain) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const GlobalBytes ka = scalar_base(static_cast<const char*>(p.k_pool) + off[h]), va = scalar_base(static_cast<const char*>(p.v_pool) + off[h]);
                asm("" : "+v"(lo));                                  // (with the scalar bases: 32-bit lane offsets, not 64-bit addresses per lane)
#pragma unroll
                for (int i = 0; i < LPH; ++i) {
                    if (DO_K) k[h * LPH + i].v = __builtin_nontemporal_load((GlobalChunk)(ka + i * 1024 + lo));
                    if (DO_V) v[h * LPH + i].v = __builtin_nontemporal_load((GlobalChunk)(va + i * 1024 + lo));
                    if (SPACED) __builtin_amdgcn_s_sleep(0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            const int64_t row0 = ((int64_t)ic.row_off * p.Hkv + ic.kvh) * (D * ES);    // packed rows [token][Hkv][D]
            const uint32_t chunk = lo - T::lane_key(lane) * (D * ES);
#pragma unroll
            for (int n = 0; n < NL; ++n) {
                const int key = min(n * KPL + T::lane_key(lane), ic.kv_end - 1 - kbase);    // within the block
                const bool is_new = KVT == KV_BF16 && kbase + key >= ic.c_rows;             // a new token of this call: its packed row
                const int64_t at = is_new ? row0 + (int64_t)(kbase + key - ic.C) * (p.Hkv * D * ES) + chunk
                                          : (key < 16 ? off[0] : off[1]) + (key & 15) * (D * ES) + chunk;
                if (DO_K) k[n].load(static_cast<const char*>(is_new ? p.k_new : p.k_pool) + at, 0);
                if (DO_V) v[n].load(static_cast<const char*>(is_new ? p.v_new : p.v_pool) + at, 0);
                __builtin_amdgcn_sched_barrier(0);                   // (one address per lane at a time: registers)
            }
        }
    }
    __device__ __forceinline__ void commit_k(uint32_t kl, int lane) {
#pragma unroll
        for (int l = 0; l < 4; ++l) sc[l] = KVT == KV_FP8 ? scale[l] : 1.0f;
        // (a K row past the key range may hold anything: its logits are replaced by the causal select)
#pragma unroll
        for (int n = 0; n < NL; ++n) T::put(k[n], sc[n / LPH], kl + T::slot_of(0, lane) + n * (T::GPP * G_::GS));
    }
    // V rows past the key range: zeros, so that 0-weights never meet NaN garbage
    __device__ __forceinline__ void commit_v(const ItemCtx& ic, int kbase, uint32_t vl, int lane) {
        if (kbase + 32 > ic.kv_end) {                         // uniform
#pragma unroll
            for (int n = 0; n < NL; ++n)
                if (kbase + n * KPL + T::lane_key(lane) >= ic.kv_end) v[n].zero();
        }
#pragma unroll
        for (int n = 0; n < NL; ++n) T::put(v[n], sc[2 + n / LPH], vl + T::slot_of(0, lane) + n * (T::GPP * G_::GS));
    }
};

constexpr int LEAN_ROWS = 8;
// ROWS: query rows a wave carries (32, or 16 for items of at most 16 rows: half the matrix and softmax work per key)
// NW: waves of the workgroup.  QUANT: the item appends its own new tokens (8-bit cache) before it reads its pages.
// LEAN: K and V of a block take turns in one LDS region per wave, and the merge holds the item's rows only (at most 8).
// rounded: see ItemCtx.  SPACED: see decode_rows_kernel.
template <int D, int KVT, int ROWS, int NW, bool QUANT = false, bool LEAN = false, bool SPACED = false>
__device__ __forceinline__ void narrow_body(const AttnParams& p, const ItemCtx& ic, uint32_t smem, int tid, bool rounded) {
    using G_ = Geo<D>;
    constexpr bool R16 = ROWS == 16;
    constexpr int NACC = ATTN_WAVES / NW;
    constexpr bool ONE_TOKEN = QUANT && R16 && !LEAN;     // (the lean form has no registers left for it)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & (ROWS - 1);
    const int tl = row / ic.gn, hg = row - tl * ic.gn;
    const bool valid = tl < ic.nq;
    const int tok = ic.q0 + tl;
    const int lim = valid ? ic.C + tok : 0x3fffffff;
    const int first_lim = ic.C + ic.q0;                  // smallest last-visible key among the rows

    const int nblocks = (ic.kv_end - ic.kv_begin + 31) >> 5;
    constexpr int STEP = 32 * NW;                         // the wave's block j: block wave + j * NW, keys key0 + j * STEP ..
    const int key0 = ic.kv_begin + wave * 32;
    const int nj = (nblocks - wave + NW - 1) / NW;        // the wave's blocks (<= 0: none)
    // page ids before Q: loads return in order, and Q comes from HBM
    BlockLoader<D, KVT> ld;
    if (nj > 0) ld.fetch_ids(p, ic, key0, STEP, 0, lane);
    bf16x8 Q[R16 ? D / 32 : G_::NKK];
    std::conditional_t<R16, WaveAcc16<D>, WaveAcc<D>> acc[NACC];
    if constexpr (R16) {
        load_q16<D>(p, ic, tok, hg, valid, lane, Q);
    } else {
        load_q<D>(p, ic, tok, hg, valid, lane, Q);
    }
#pragma unroll
    for (auto& st : acc) {
        if constexpr (R16) {
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) st.O[dt] = f32x4{0, 0, 0, 0};
        } else {
#pragma unroll
            for (int db = 0; db < G_::NDB; ++db) st.O[db] = f32x16{0};
        }
        st.m = NEG_INF;
        st.l = 0.0f;
    }

    const uint32_t kl = smem + wave * ((LEAN ? 1 : 2) * G_::B32);
    const uint32_t vl = LEAN ? kl : kl + G_::B32;
    NewToken<D> nt;
    bool pending = false;                                 // this wave has a token to encode before it fetches the last block
    // block j, K and V or (LEAN) K alone: its pages are known; with every eighth block, the page ids of the next eight
    auto fetch = [&](int j) {
        if constexpr (ONE_TOKEN) {
            if (pending && j == nj - 1) nt.finish(p, ic, lane);
        }
        ld.locate(p, ic, key0 + j * STEP);
        if ((j + 1) % ld.IDS == 0) ld.fetch_ids(p, ic, key0, STEP, j + 1, lane);
        ld.fetch_scales(p, ic);
        ld.template fetch_kv<true, !LEAN, SPACED>(p, ic, key0 + j * STEP, lane);
    };
    auto first_block = [&]() {
        ld.take_pages(0);
        fetch(0);
        if constexpr (LEAN) {
            ld.template fetch_kv<false, true, SPACED>(p, ic, key0, lane);
            ld.take_pages(1);
        }
    };
    if (QUANT && p.k_new && ic.kv_end > ic.C) {           // uniform
        if (ONE_TOKEN && ic.nq == 1 && page_in_last_block(ic.C, p.P)) {
            pending = nj > 0 && wave + (nj - 1) * NW == nblocks - 1;
            if (pending) nt.start(p, ic, lane);
            if (pending && nj == 1) nt.start_scale(p, ic, lane);
            if (nj > 0) first_block();
            if (pending && nj > 1) nt.start_scale(p, ic, lane);
        } else {
            // blocks from nold on hold pages that get new tokens; the first blocks before them travel while the append runs
            const int nold = ((max(ic.C, ic.kv_begin) & ~(p.P - 1)) - ic.kv_begin) >> 5;
            if (wave < nold) first_block();
            append_item_pages<D, NW>(p, ic, tid);
            __syncthreads();
            if (wave >= nold && nj > 0) first_block();
        }
    } else if (nj > 0) {
        first_block();
    }
    for (int j0 = 0; j0 < nj; j0 += NACC) {
        static_for<0, NACC>([&](auto ac) {
            auto& st = acc[decltype(ac)::value];
            const int j = j0 + decltype(ac)::value;
            if (j >= nj) return;
            const int kbase = key0 + j * STEP;
            const bool more = j + 1 < nj;
            const int rel = lim - kbase - 4 * (R16 ? key_group16(lane >> 4) : lane >> 5);
            const bool masked = kbase + 31 > first_lim;
            ld.commit_k(kl, lane);
            if constexpr (LEAN) {
                if (more) fetch(j + 1);
                const bf16x8 P = softmax16<D>(kl, Q, st, p.c_log2, rel, masked, rounded, lane);
                ld.commit_v(ic, kbase, vl, lane);
                if (more) {
                    ld.take_pages(j + 2);
                    ld.template fetch_kv<false, true, SPACED>(p, ic, kbase + STEP, lane);
                }
                pv16<D>(vl, P, st, lane);
                return;
            }
            ld.commit_v(ic, kbase, vl, lane);
            if (more) {
                ld.take_pages(j + 1);
                fetch(j + 1);
            }
            if constexpr (R16) {
                const bf16x8 P = softmax16<D>(kl, Q, st, p.c_log2, rel, masked, rounded, lane);
                pv16<D>(vl, P, st, lane);
            } else {
                block32<D>(kl, vl, Q, st, p.c_log2, rel, masked, rounded, lane);
            }
        });
    }
    // merge the waves' states: LDS holds O as [state][row][D + 4] fp32 and (m, l) as [state][row][2]
    __syncthreads();                                      // every wave is done with its K/V region
    constexpr int OSTR = D + 4;
    const uint32_t obase = smem;
    const int mrows = LEAN ? LEAN_ROWS : ROWS;            // rows of a state in LDS
    const uint32_t mlbase = smem + ATTN_WAVES * mrows * OSTR * 4;
    static_for<0, NACC>([&](auto ac) {
        const auto& st = acc[decltype(ac)::value];
        const int g = lane / ROWS;
        const int slot = (wave + decltype(ac)::value * NW) * mrows + row;
        const uint32_t orow = obase + slot * OSTR * 4;
        const float ltot = R16 ? sum_xor32(sum_xor16(st.l)) : sum_xor32(st.l);
        if (LEAN && row >= LEAN_ROWS) return;
        if constexpr (R16) {
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) *LDS_PTR(f32x4, orow + (dt * 16 + g * 4) * 4) = st.O[dt];
        } else {
#pragma unroll
            for (int db = 0; db < G_::NDB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int d0 = db * 32 + i4 * 8 + g * 4;
                    f32x4 o = {st.O[db][i4 * 4], st.O[db][i4 * 4 + 1], st.O[db][i4 * 4 + 2], st.O[db][i4 * 4 + 3]};
                    *LDS_PTR(f32x4, orow + d0 * 4) = o;
                }
        }
        if (g == 0) {
            *LDS_PTR(float, mlbase + slot * 8) = st.m;
            *LDS_PTR(float, mlbase + slot * 8 + 4) = ltot;
        }
    });
    __syncthreads();
    // thread -> (row r, DPT consecutive d): 16 threads per row
    constexpr int DPT = D / 16, NS = ATTN_WAVES;
    const int dc = (tid & 15) * DPT;
    const int rows = ic.nq * ic.gn;
    for (int r = tid >> 4; r < rows; r += 4 * NW) {
        float mw[NS], lw[NS];
        float mall = NEG_INF;
#pragma unroll
        for (int w = 0; w < NS; ++w) {
            mw[w] = *LDS_PTR(float, mlbase + ((w * mrows + r) * 2) * 4);
            lw[w] = *LDS_PTR(float, mlbase + ((w * mrows + r) * 2 + 1) * 4);
            mall = fmaxf(mall, mw[w]);
        }
        const float muse = mall == NEG_INF ? 0.0f : mall;
        float lsum = 0.0f, wgt[NS];
#pragma unroll
        for (int w = 0; w < NS; ++w) {
            wgt[w] = fast_exp2(mw[w] - muse);
            lsum += lw[w] * wgt[w];
        }
        float acc[DPT];
#pragma unroll
        for (int x = 0; x < DPT; ++x) acc[x] = 0.0f;
#pragma unroll
        for (int w = 0; w < NS; ++w) {
            const uint32_t src = obase + ((w * mrows + r) * OSTR + dc) * 4;
#pragma unroll
            for (int x = 0; x < DPT; x += 4) {
                const f32x4 o = *LDS_PTR(f32x4, src + x * 4);
                acc[x] += o[0] * wgt[w];
                acc[x + 1] += o[1] * wgt[w];
                acc[x + 2] += o[2] * wgt[w];
                acc[x + 3] += o[3] * wgt[w];
            }
        }
        const int rtl = r / ic.gn, rhg = r - rtl * ic.gn;
        if (ic.part_off < 0) {
            const float inv = 1.0f / lsum;
            const int hq = ic.kvh * (p.Hq / p.Hkv) + ic.g0 + rhg;
            char* dst = static_cast<char*>(p.out) + (((int64_t)(ic.row_off + ic.q0 + rtl) * p.Hq + hq) * D + dc) * 2;
#pragma unroll
            for (int x = 0; x < DPT; x += 4) {
                bf16x4 o = {(__bf16)(acc[x] * inv), (__bf16)(acc[x + 1] * inv), (__bf16)(acc[x + 2] * inv),
                            (__bf16)(acc[x + 3] * inv)};
                *reinterpret_cast<u32x2*>(dst + x * 2) = __builtin_bit_cast(u32x2, o);
            }
        } else {
            float* po = p.partial + ic.part_off + (int64_t)r * D + dc;
#pragma unroll
            for (int x = 0; x < DPT; x += 4) {
                f32x4 o = {acc[x], acc[x + 1], acc[x + 2], acc[x + 3]};
                *reinterpret_cast<f32x4*>(po + x) = o;
            }
            if ((tid & 15) == 0) {
                float* ml = p.partial + ic.part_off + (int64_t)rows * D + r * 2;
                ml[0] = mall;
                ml[1] = lsum;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// append item (bf16 cache): the page writes of the call, riding in the attention launch.  One item moves nq
// consecutive packed rows of k_new / v_new, starting with new token q0 of request req and running on into the
// following requests, to their pages: a bit-exact copy, 16 bytes per thread and step.  The attention items of
// the same launch never read these page slots (they take new tokens from the packed rows), so the two kinds
// need no order among themselves.

// total 16-byte chunks of k_new and v_new to the pages; where(u, src, dst): element offsets of chunk u (u rises from call to
// call).  Four chunks of each in flight per thread: one at a time, an item of 64 rows over 8 heads was a chain of 16 round
// trips to memory, 14 us; now 12.7 us, which is what one CU moves.
template <int NTHR, class F>
__device__ __forceinline__ void copy_new_rows(const AttnParams& p, int total, int tid, F&& where) {
    constexpr int UN = 4;
    for (int u0 = tid; u0 < total; u0 += UN * NTHR) {
        u32x4 kx[UN], vx[UN];
        int64_t dst[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            int64_t src;
            where(min(u0 + i * NTHR, total - 1), src, dst[i]);      // (past the end: the last chunk once more, not stored)
            kx[i] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(p.k_new) + src * 2);
            vx[i] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(p.v_new) + src * 2);
        }
#pragma unroll
        for (int i = 0; i < UN; ++i)
            if (u0 + i * NTHR < total) {
                *reinterpret_cast<u32x4*>(static_cast<char*>(const_cast<void*>(p.k_pool)) + dst[i] * 2) = kx[i];
                *reinterpret_cast<u32x4*>(static_cast<char*>(const_cast<void*>(p.v_pool)) + dst[i] * 2) = vx[i];
            }
    }
}

// rows [first_row, first_row + nrows) of the packed rows; req_of(r): the r-th row of the batch, r: one at or before first_row's
template <class F>
__device__ __forceinline__ void append_body(const AttnParams& p, int first_row, int nrows, int r, F&& req_of, int D, int tid) {
    const int cpt = p.Hkv * D / 8;                           // 16-byte chunks per packed row (one of K or V)
    const int cph = D / 8;
    ReqInfo ri = req_of(r);                                  // request of the row this thread is at: rows only move forward
    copy_new_rows<AWG>(p, nrows * cpt, tid, [&](int u, int64_t& src, int64_t& dst) {
        const int row = first_row + u / cpt, rem = u % cpt;
        while (row >= ri.row_off + ri.L) ri = req_of(++r);   // (requests with L = 0 are stepped over)
        const int h = rem / cph, ch = rem % cph;
        const int t = ri.C + (row - ri.row_off);
        const int page = p.block_table[(int64_t)ri.req * p.max_pages + (t >> p.logP)];
        src = ((int64_t)row * p.Hkv + h) * D + ch * 8;
        dst = ((((int64_t)page * p.Hkv + h) << p.logP) + (t & (p.P - 1))) * D + ch * 8;
    });
}

// ---------------------------------------------------------------------------------------------
// the fused attention launch: one workgroup per work item, wide and narrow items in one grid

// Next item of die queue q (items q, q + NUM_QUEUES, ...), or -1 when the queue is used up.
__device__ __forceinline__ int take_item(const AttnParams& p, int q) {
    const int pos = __hip_atomic_fetch_add(p.queue_heads + q, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int idx = q + NUM_QUEUES * pos;
    return idx < p.nitems ? idx : -1;
}
// An item of the queue with the most items left, or -1 when every queue is used up.  Called by the whole first wave: lanes
// 0 .. NUM_QUEUES - 1 read one queue head each (one round trip for the scan), lane 0 takes the item.  Bounded: an attempt
// fails only when another workgroup took the last item of the chosen queue in between, and that workgroup runs it.
__device__ __forceinline__ int steal_item(const AttnParams& p, int lane) {
    for (int attempt = 0; attempt < 4 * NUM_QUEUES; ++attempt) {
        int left = 0;
        if (lane < NUM_QUEUES) {
            const int pos = __hip_atomic_load(p.queue_heads + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            left = (p.nitems - lane + NUM_QUEUES - 1) / NUM_QUEUES - pos;
        }
        int best = -1, best_left = 0;
#pragma unroll
        for (int q = 0; q < NUM_QUEUES; ++q) {
            const int l = __builtin_amdgcn_readlane(left, q);
            if (l > best_left) {
                best_left = l;
                best = q;
            }
        }
        if (best < 0) return -1;
        int idx = -1;
        if (lane == 0) idx = take_item(p, best);
        idx = __builtin_amdgcn_readfirstlane(idx);
        if (idx >= 0) return idx;
    }
    return -1;
}

template <int D, int KVT>
__device__ __forceinline__ void run_item(const AttnParams& p, int idx, uint32_t smem, int tid) {
    const int kind = (p.items[idx].heads >> 24) & 0xff;
    if (kind == KIND_NULL) return;                         // a filler that keeps the following items on their XCD
    const ItemCtx ic = item_ctx<KVT>(p, p.items[idx]);
    if (kind == KIND_WIDE)
        wide_body<D, KVT>(p, ic, smem, tid);
    else if (kind == KIND_NARROW) {                        // (next to tiles: rows of at most 32 query rows alone)
        if (ic.nq * ic.gn <= 16)
            narrow_body<D, KVT, 16, ATTN_WAVES>(p, ic, smem, tid, false);
        else
            narrow_body<D, KVT, 32, ATTN_WAVES>(p, ic, smem, tid, false);
    }
    else if (KVT == KV_BF16)
        append_body(p, ic.row_off + ic.q0, ic.nq, ic.req, [&](int r) { return p.reqs[r]; }, D, tid);
}

// One workgroup per work item when the items fit one round on the CUs (gridDim.x = number of items).  Otherwise
// gridDim.x persistent workgroups: workgroup i runs item i, then items of the queue of its die (workgroup i of a launch
// is dispatched to die i % NUM_QUEUES, and so were the items of queue i % NUM_QUEUES meant to be: their K/V streams share
// that die's L2), and when that queue is used up it helps out on the queue with the most items left, so that the dies
// finish together.
// No workgroup ever waits for another: every loop ends when the queues are used up.
template <int D, int KVT>
__global__ __launch_bounds__(AWG, 1) void attn_kernel(const AttnParams p) {
    __shared__ __attribute__((aligned(16))) char smem_raw[Geo<D>::SMEM];
    __shared__ int s_next;
    const uint32_t smem = (uint32_t)(uintptr_t)LDS_PTR(char, smem_raw);
    if (blockIdx.x == 0 && threadIdx.x == 0 && p.slot_flag)   // releases the host's staging slot (see AttnParams)
        __hip_atomic_store(p.slot_flag, p.slot_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const bool persistent = p.nitems > (int)gridDim.x;
    const int home = blockIdx.x % NUM_QUEUES;
    int idx = blockIdx.x;
    for (;;) {
        // The thread index is made opaque in every iteration: otherwise everything the three kinds of item derive from it
        // is hoisted out of the loop and live at once, which does not fit the register file (spills to scratch memory).
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        run_item<D, KVT>(p, idx, smem, tid);
        if (!persistent) return;
        __syncthreads();                                   // every wave is done with this item's LDS
        if (tid < 64) {
            // The next item is taken when this one is done, not before (measured: a reservation at the start of the item
            // +5 % on long tiles, one during its last stage +1 %): the queues are ordered longest first, and an item
            // reserved early goes to a workgroup by its position in the launch instead of to the one that is free first.
            int next = -1;
            if (tid == 0) next = take_item(p, home);
            next = __builtin_amdgcn_readfirstlane(next);
            if (next < 0) next = steal_item(p, tid);
            if (tid == 0) s_next = next;
        }
        __syncthreads();
        idx = __builtin_amdgcn_readfirstlane(s_next);      // uniform: the item is then read through the scalar unit
        __syncthreads();                                   // (s_next is written again at the end of the next item)
        if (idx < 0) return;
    }
}

template <int D, int NW, bool LEAN>
constexpr int rows_smem() {
    constexpr int kv = NW * (LEAN ? 1 : 2) * Geo<D>::B32;
    constexpr int merge = ATTN_WAVES * (LEAN ? LEAN_ROWS : NW == ATTN_WAVES ? 32 : 16) * ((D + 4) * 4 + 8);
    return kv > merge ? kv : merge;
}

// A launch without tiles whose list lies in the workspace: blocks of prefill rows next to short rows, or more short rows than the
// row table holds.  One workgroup per item.  (Apart from attn_kernel for the sums of both kinds of row, see ItemCtx::rounded: taken side
// by side, next to tiles the 8-bit decode rows, which are bound by their instructions, lose by it: 24 of them next to a prefill 87.0 -> 87.5 us.)
template <int D, int KVT>
__global__ __launch_bounds__(AWG, D == 64 ? 4 : 1) void narrow_kernel(const AttnParams p) {
    __shared__ __attribute__((aligned(16))) char smem_raw[rows_smem<D, ATTN_WAVES, false>()];
    const uint32_t smem = (uint32_t)(uintptr_t)LDS_PTR(char, smem_raw);
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid == 0 && p.slot_flag)           // releases the host's staging slot (see AttnParams)
        __hip_atomic_store(p.slot_flag, p.slot_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const Item& it = p.items[blockIdx.x];
    const int kind = (it.heads >> 24) & 0xff;
    if (kind == KIND_NULL) return;
    const ItemCtx ic = item_ctx<KVT>(p, it);
    if (kind == KIND_NARROW) {
        if (ic.nq * ic.gn <= 16)
            narrow_body<D, KVT, 16, ATTN_WAVES>(p, ic, smem, tid, ic.rounded);
        else
            narrow_body<D, KVT, 32, ATTN_WAVES>(p, ic, smem, tid, ic.rounded);
    }
    else if (KVT == KV_BF16)
        append_body(p, ic.row_off + ic.q0, ic.nq, ic.req, [&](int r) { return p.reqs[r]; }, D, tid);
}

// A small launch of tiles alone over a bf16 cache, whose list travels in the arguments (see TileTable): one workgroup per tile or
// piece, then the append items.  KIND_NARROW: blocks of at most 32 query rows instead of tiles of 256 (see take_blocks for where).  Bound there:
// the chain item -> page ids -> keys, whose latency eight waves with a block of 32 keys each pass once per 256 keys, where a tile's
// stage of 128 waits for its own loads (one row of 32 tokens over 256, d = 64: 7.9 -> 6.8 us; of 64 over 1 024, 8 KV heads of 128: 22.6 -> 14.6).
// SHORT_ROWS: rows of at most 32 query rows are among them, whose sums differ (a kernel of its own without them: taking both sums costs the
// smallest launch 6.1 -> 6.2 us, and a second pair of bodies behind a branch, whose instructions have to be fetched, 6.5).
template <int D, int KIND, bool SHORT_ROWS>
__global__ __launch_bounds__(AWG, KIND == KIND_NARROW && D == 64 ? 4 : 1) void attn_tiles_kernel(const AttnParams p, const TileTable t) {
    __shared__ __attribute__((aligned(16))) char smem_raw[KIND == KIND_NARROW ? rows_smem<D, ATTN_WAVES, false>() : Geo<D>::SMEM];
    const uint32_t smem = (uint32_t)(uintptr_t)LDS_PTR(char, smem_raw);
    const int idx = blockIdx.x, tid = threadIdx.x;
    if (idx >= t.n_items) {
        const int first_row = (idx - t.n_items) * t.append_rows;
        append_body(p, first_row, min(t.append_rows, t.sum_L - first_row), 0, [&](int r) { return t.rows[r]; }, D, tid);
        return;
    }
    const uint32_t code = t.items[idx];
    if (code == TILE_NULL) return;                           // a filler that keeps the following items on their XCD
    const ItemCtx ic = item_ctx<KV_BF16>(p, tile_item(t, code));
    const bool rounded = SHORT_ROWS ? ic.rounded : true;
    if constexpr (KIND == KIND_WIDE)
        wide_body<D, KV_BF16>(p, ic, smem, tid);
    else if (ic.nq * ic.gn <= 16)
        narrow_body<D, KV_BF16, 16, ATTN_WAVES>(p, ic, smem, tid, rounded);
    else
        narrow_body<D, KV_BF16, 32, ATTN_WAVES>(p, ic, smem, tid, rounded);
}

// The launch of a batch of decode rows alone whose work list travels in the arguments (see RowTable): one workgroup of NW
// waves per item, then (bf16 cache) the append items.  Bound: HBM, and around an item's stream its latencies (item, page
// ids, first block before the first key; merge behind the last), which only other items can hide.
//   8 waves: one workgroup fills a CU (137 KB of LDS; 57 GB/s when it streams alone, over an 8-bit cache 41).  Few items,
//     or whole rows that keep HBM busy by themselves.
//   4 waves: two (bf16 cache: 232 -> 212 registers, 69 KB) or three workgroups per CU (8-bit cache: K and V of a block take
//     turns in one LDS region and the merge holds 8 rows, 34 KB and 166 registers), so that an item's latencies pass under
//     its neighbours' streams.
// No list in memory means no upload launch in front; over an 8-bit cache the item that reads the pages of a row's new tokens
// quantises them itself, so the append launch is gone too (25 rows of 0.7-7 k tokens over 8 KV heads: append 5.1 us + gap
// 4 + attention 43.9 -> 40.5 us; four bf16 rows of 36-70 k tokens 30.3 -> 27.8 us per call, one row of 1.5 k 16.7 -> 13.5).

// Page writes of packed rows [first_row, first_row + APPEND_ITEM_ROWS): which request and position a row belongs to is
// written to LDS by the table's entries first.
template <int D, int NTHR>
__device__ __forceinline__ void append_table_rows(const AttnParams& p, const RowTable& t, int first_row, uint32_t smem, int tid) {
    if (tid < t.n) {
        const RowEntry e = t.e[tid];
        const int L = e.req_L >> 24;
        for (int i = 0; i < L; ++i) {
            const int row = e.row_off + i - first_row;
            if (row >= 0 && row < APPEND_ITEM_ROWS) *LDS_PTR(u32x2, smem + row * 8) = u32x2{(uint32_t)e.req_L & 0xffffff, (uint32_t)(e.C + i)};
        }
    }
    __syncthreads();
    const int nrows = min(APPEND_ITEM_ROWS, t.sum_L - first_row);
    const int cpt = p.Hkv * (D / 8);                         // 16-byte chunks per packed row (one of K or V)
    copy_new_rows<NTHR>(p, nrows * cpt, tid, [&](int u, int64_t& src, int64_t& dst) {
        const int row = u / cpt, rem = u % cpt, h = rem / (D / 8), ch = rem % (D / 8);
        const u32x2 at = *LDS_PTR(const u32x2, smem + row * 8);
        const int pos = (int)at.y;
        const int page = p.block_table[(int64_t)at.x * p.max_pages + (pos >> p.logP)];
        src = (int64_t)(first_row + row) * p.Hkv * D + rem * 8;
        dst = ((((int64_t)page * p.Hkv + h) << p.logP) + (pos & (p.P - 1))) * D + ch * 8;
    });
}

template <int D, int KVT, int NW>
__global__ __launch_bounds__(64 * NW, D == 64 ? 4 : NW < ATTN_WAVES && KVT == KV_FP8 ? 3 : 2) void decode_rows_kernel(const AttnParams p, const RowTable t) {
    constexpr bool LEAN = NW < ATTN_WAVES && KVT == KV_FP8;
    // An empty sleep between the pairs of loads of a block: where several items per CU saturate HBM it serves the loads better so than in one
    // burst (96 rows of 2-16 k tokens over 8 KV heads 544 us without it, 541.6 with it; rows of 4-16 k 0.995), and it costs the others little
    // (0.995 to 1.01 from 512 to 2 k tokens, 1.00 below; s_nop 7 and s_sleep 1 measure alike, s_sleep 4 costs rows of 64 tokens 3 %).
    // Only there a block is enough loads to matter: 8-bit decode batches of d = 64 lose 0.3 % by it, d = 128 0.2 %.
    constexpr bool SPACED = D == 128 && KVT == KV_BF16 && NW == ATTN_WAVES;
    __shared__ __attribute__((aligned(16))) char smem_raw[rows_smem<D, NW, LEAN>()];
    const uint32_t smem = (uint32_t)(uintptr_t)LDS_PTR(char, smem_raw);
    const int idx = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (idx >= t.n_items) {
        if constexpr (KVT == KV_BF16) append_table_rows<D, 64 * NW>(p, t, (idx - t.n_items) * APPEND_ITEM_ROWS, smem, tid);
        return;
    }
    int row;
    if (idx < t.n_whole) {                                   // the last row whose whole pieces start at or before idx
        const bool a = lane < t.n && t.e[min(lane, t.n - 1)].first <= idx;
        const bool b = lane + 64 < t.n && t.e[min(lane + 64, t.n - 1)].first <= idx;
        row = __popcll(__ballot(a)) + __popcll(__ballot(b)) - 1;
    } else {
        row = (idx - t.n_whole) / t.Hkv;
    }
    const ItemCtx ic = item_ctx<KVT>(p, table_item(t, t.e[__builtin_amdgcn_readfirstlane(row)], idx));
    if (NW < ATTN_WAVES || ic.nq * ic.gn <= 16)
        narrow_body<D, KVT, 16, NW, KVT == KV_FP8, LEAN, SPACED>(p, ic, smem, tid, false);   // (rows of at most 32 query rows)
    else
        narrow_body<D, KVT, 32, NW, KVT == KV_FP8, false, SPACED>(p, ic, smem, tid, false);
}

// ---------------------------------------------------------------------------------------------
// combine: merge the split-KV partials of one query tile
//   m = max_s m_s;  l = sum_s l_s 2^(m_s - m);  O = sum_s O_s 2^(m_s - m) / l

constexpr int COMB_ROWS = 16;          // query rows per combine workgroup when a tile has few splits
constexpr int COMB_ROWS_SLICED = 2;    // ... and when it has many: the workgroup's threads then share the splits

// One output quad (4 consecutive d of one row) merged over the splits s_begin, s_begin + s_step, ... < nsplit, UN splits
// at a time: all loads of a group are issued before any is used, so a thread pays one memory latency per UN splits,
// and the maximum is carried along (acc and l are rescaled when a group raises it) instead of being taken in a pass
// of its own.  Returns the running maximum (-inf when the thread had no split).
template <int D, int UN>
__device__ __forceinline__ float combine_quad(const float* part0, int nsplit, int s_begin, int s_step, int64_t stride,
                                              int64_t ml_off, int64_t o_off, f32x4& acc, float& lsum) {
    float m_run = NEG_INF;
    lsum = 0.0f;
    acc = f32x4{0, 0, 0, 0};
    for (int s0 = s_begin; s0 < nsplit; s0 += UN * s_step) {
        float mv[UN], lv[UN];
        f32x4 ov[UN];
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            const int sp = min(s0 + j * s_step, nsplit - 1);         // the tail re-reads the last split and drops it below
            const float* base = part0 + (int64_t)sp * stride;
            mv[j] = base[ml_off];
            lv[j] = base[ml_off + 1];
            ov[j] = *reinterpret_cast<const f32x4*>(base + o_off);
        }
        float mg = m_run;
#pragma unroll
        for (int j = 0; j < UN; ++j) mg = fmaxf(mg, mv[j]);          // (a duplicate of the last split changes nothing)
        const float muse = mg == NEG_INF ? 0.0f : mg;
        const float back = fast_exp2(m_run - muse);                  // 0 on the first group
        lsum *= back;
        acc *= back;
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            if (s0 + j * s_step < nsplit) {
                const float w = fast_exp2(mv[j] - muse);
                lsum += lv[j] * w;
                acc += ov[j] * w;
            }
        }
        m_run = mg;
    }
    return m_run;
}

// CR query rows per workgroup.  CR * D / 4 output quads; when that is less than the workgroup, its WG / (CR * D / 4)
// thread slices each take every NSL-th split of a quad and slice 0 merges their results through LDS: a tile with a
// hundred splits and few rows (a decode row over a long context) is then a chain of one or two memory latencies per
// thread instead of eight, on NSL times as many workgroups.
template <int D, int CR>
__device__ __forceinline__ void combine_tile(const AttnParams& p, const CombItem& ci, int row_off) {
    constexpr int QPR = D / 4;                         // float4 groups per row
    constexpr int NSL = CR * QPR >= WG ? 1 : WG / (CR * QPR);
    constexpr int PER = CR * QPR < WG ? CR * QPR : WG; // (row, quad) pairs in flight per pass
    __shared__ float red[NSL > 1 ? (NSL - 1) * PER * 6 : 1];
    const int kvh = ci.heads & 0xff, g0 = (ci.heads >> 8) & 0xff, gn = (ci.heads >> 16) & 0xff;
    const int rows = ci.nq * gn;
    const int r0 = blockIdx.y * CR;                    // grid.y covers the tallest tile
    if (r0 >= rows) return;
    const int nr = min(CR, rows - r0);
    const int slice = threadIdx.x / PER, u0 = threadIdx.x % PER;
    const float* part0 = p.partial + ci.part_off;
    auto finish = [&](int r, int dq, const f32x4& acc, float lsum) {
        const float inv = 1.0f / lsum;
        const int tl = r / gn, hg = r - tl * gn;
        const int hq = kvh * (p.Hq / p.Hkv) + g0 + hg;
        char* dst = static_cast<char*>(p.out) + (((int64_t)(row_off + ci.q0 + tl) * p.Hq + hq) * D + dq) * 2;
        bf16x4 o = {(__bf16)(acc[0] * inv), (__bf16)(acc[1] * inv), (__bf16)(acc[2] * inv), (__bf16)(acc[3] * inv)};
        *reinterpret_cast<u32x2*>(dst) = __builtin_bit_cast(u32x2, o);
    };
    if constexpr (NSL == 1) {
        for (int u = u0; u < nr * QPR; u += PER) {
            const int r = r0 + u / QPR, dq = (u % QPR) * 4;
            const int64_t ml_off = (int64_t)rows * D + r * 2;
            float lsum;
            f32x4 acc;
            if (ci.nsplit > 8)
                combine_quad<D, 16>(part0, ci.nsplit, 0, 1, ci.part_stride, ml_off, (int64_t)r * D + dq, acc, lsum);
            else
                combine_quad<D, 4>(part0, ci.nsplit, 0, 1, ci.part_stride, ml_off, (int64_t)r * D + dq, acc, lsum);
            finish(r, dq, acc, lsum);
        }
    } else {
        const bool active = u0 < nr * QPR;             // one pass: nr * QPR <= PER
        const int r = r0 + u0 / QPR, dq = (u0 % QPR) * 4;
        float lsum = 0.0f, m = NEG_INF;
        f32x4 acc = {0, 0, 0, 0};
        if (active)
            m = combine_quad<D, 16>(part0, ci.nsplit, slice, NSL, ci.part_stride, (int64_t)rows * D + r * 2,
                                    (int64_t)r * D + dq, acc, lsum);
        if (active && slice > 0) {
            float* w = red + ((slice - 1) * PER + u0) * 6;
            w[0] = m; w[1] = lsum; w[2] = acc[0]; w[3] = acc[1]; w[4] = acc[2]; w[5] = acc[3];
        }
        __syncthreads();
        if (!active || slice > 0) return;
        float mall = m;
#pragma unroll
        for (int s = 1; s < NSL; ++s) mall = fmaxf(mall, red[((s - 1) * PER + u0) * 6]);
        const float muse = mall == NEG_INF ? 0.0f : mall;
        const float w0 = fast_exp2(m - muse);
        lsum *= w0;
        acc *= w0;
#pragma unroll
        for (int s = 1; s < NSL; ++s) {
            const float* rd = red + ((s - 1) * PER + u0) * 6;
            const float w = fast_exp2(rd[0] - muse);
            lsum += rd[1] * w;
            acc += f32x4{rd[2], rd[3], rd[4], rd[5]} * w;
        }
        finish(r, dq, acc, lsum);
    }
}

template <int D, int CR>
__global__ __launch_bounds__(WG) void combine_kernel(const AttnParams p) {
    const CombItem ci = p.combs[blockIdx.x];
    combine_tile<D, CR>(p, ci, p.reqs[ci.req].row_off);
}
// the same for a launch by table: one grid column per (row, KV head)
template <int D, int CR>
__global__ __launch_bounds__(WG) void combine_rows_kernel(const AttnParams p, const RowTable t) {
    const RowEntry e = t.e[blockIdx.x / t.Hkv];
    if (e.part_off >= 0) combine_tile<D, CR>(p, table_comb(t, e, blockIdx.x % t.Hkv), e.row_off);
}
template <int D, int CR>
__global__ __launch_bounds__(WG) void combine_tiles_kernel(const AttnParams p, const TileTable t) {
    combine_tile<D, CR>(p, tile_comb(t, blockIdx.x), t.rows[t.combs[blockIdx.x].code & 15].row_off);
}

// ---------------------------------------------------------------------------------------------
// KV append / pack / unpack, as launches of their own.  Bound: HBM, and for small calls the chain row -> page id -> data.
// One workgroup column per page that new tokens fall into, the rows' pages laid end to end: with a grid of (most pages of a
// row) x (rows) instead, a prefill row of 45 pages next to 24 decode rows was 19 125 workgroups, 1 100 of them with work (8-bit append
// 6.8 -> 3.9 us).

// The workgroups in front of the pages' carry the work list of the attention launch that follows from pinned host memory into
// the workspace (saves a launch per call).
__device__ __forceinline__ void upload_rider(const AppendParams& p) {
    const u32x4* src = static_cast<const u32x4*>(p.up_src);
    u32x4* dst = static_cast<u32x4*>(p.up_dst);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < p.up_n16; i += p.up_blocks * blockDim.x) dst[i] = src[i];
}

struct PageJob {
    int page;                  // physical page
    int C, t0, t1;             // cached tokens of the row; positions [t0, t1) of it are this page's new tokens
    int row;                   // packed row of token t0
};
// Every lane loads a row or two, and the row of this workgroup's page is then picked from the lanes: one trip to the arguments.
__device__ __forceinline__ PageJob page_job(const AppendParams& p) {
    const int idx = p.pg0 + (int)blockIdx.x - p.up_blocks, lane = threadIdx.x & 63;
    static_assert(APPEND_MAX_REQS == 128, "two rows per lane");
    const AppendRow lo = p.rows[lane];
    AppendRow hi = {0, 0, 0, 0};
    if (p.n > 64) hi = p.rows[lane + 64];
    // the last row whose pages start at or before idx (rows without new tokens share their successor's start)
    const int r = __popcll(__ballot(lane < p.n && lo.pg_off <= idx)) + __popcll(__ballot(lane + 64 < p.n && hi.pg_off <= idx)) - 1;
    const AppendRow s = r < 64 ? lo : hi;
    const int C = __builtin_amdgcn_readlane(s.C, r & 63), L = __builtin_amdgcn_readlane(s.L, r & 63);
    const int lp = (C >> p.logP) + idx - __builtin_amdgcn_readlane(s.pg_off, r & 63);
    PageJob j;
    j.C = C;
    j.t0 = max(C, lp << p.logP);
    j.t1 = min(C + L, (lp + 1) << p.logP);
    j.row = __builtin_amdgcn_readlane(s.row_off, r & 63) + j.t0 - C;
    j.page = p.block_table[(int64_t)(p.req0 + r) * p.max_pages + lp];
    return j;
}

// bf16 cache: bit-exact copies.  grid = (pages, 2 {K, V})
// PACK = false: packed rows [tokens][hn][D] -> pages (append, or unpack of a received head share);
// PACK = true:  pages -> packed rows (the send buffer of a KV transfer).
// Chunks are numbered in page order (head, token, chunk), and four are in flight per thread: 8 700 tokens, 4 of 8 heads of 128,
// pack and unpack together 18.6 -> 14.3 us, of which the non-temporal stores 2.4 (with non-temporal loads too 17).  The stores pay
// with a decode step right behind a merge, too, which reads the pages back: append + step, plain -> non-temporal stores: 16 rows of 64 to
// 1 024 new tokens 86.0 -> 71.3 us, four of 4 096 over 32 k (one head) 27.2 -> 24.7, 4 of 25 rows with 600 82.0 -> 77.2, one of 509 15.7 ->
// 15.1; only long initial prefills lose, one of 4 096 18.1 -> 18.7, 16 of them 142 -> 149.
template <bool PACK>
__global__ __launch_bounds__(WG) void kv_move_bf16_kernel(const AppendParams p) {
    if ((int)blockIdx.x < p.up_blocks) {
        if (blockIdx.y == 0) upload_rider(p);
        return;
    }
    const PageJob j = page_job(p);
    const int lc = p.D == 128 ? 4 : 3;                       // log2 of the 16-byte chunks per row and head
    const int s0 = j.t0 & (p.P - 1), ns = j.t1 - j.t0, total = (p.hn * ns) << lc;
    char* rows = static_cast<char*>(const_cast<void*>(blockIdx.y ? p.v_new : p.k_new)) + (int64_t)j.row * p.hn * p.D * 2;
    char* pool = static_cast<char*>(blockIdx.y ? p.v_pool : p.k_pool) + ((((int64_t)j.page * p.Hkv + p.h0) << p.logP) + s0) * p.D * 2;
    const float inv_ns = __builtin_amdgcn_rcpf((float)ns);   // y / ns = (y + 0.5) * inv_ns rounded down: y < 2^14, ns <= 64
    constexpr int UN = 4;
    for (int u0 = threadIdx.x; u0 < total; u0 += UN * WG) {
        u32x4 x[UN];
        uint32_t dst[UN];                                    // (offsets inside a page or its packed rows: below 2^23)
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int u = u0 + i * WG, y = u >> lc;
            const int h = (int)(((float)y + 0.5f) * inv_ns), tok = y - h * ns, ch = u & ((1 << lc) - 1);
            const uint32_t ro = ((uint32_t)(tok * p.hn + h) << (lc + 4)) + ch * 16, po = ((uint32_t)((h << p.logP) + tok) << (lc + 4)) + ch * 16;
            dst[i] = PACK ? ro : po;
            if (u < total) x[i] = *reinterpret_cast<const u32x4*>(PACK ? pool + po : rows + ro);
        }
#pragma unroll
        for (int i = 0; i < UN; ++i)
            if (u0 + i * WG < total) __builtin_nontemporal_store(x[i], reinterpret_cast<u32x4*>((PACK ? rows : pool) + dst[i]));
    }
}

// 8-bit cache.  grid = (pages, K and V of the KV heads over the workgroup's waves): WPU waves take one (page, head, K or V)
// with all its new tokens in registers: amax -> exponent -> (re-encode old slots) -> encode, one trip to memory in front and
// one behind.  Many units: a wave each (a workgroup each, which read the tokens twice, and a grid padded to the longest row:
// 8 700 tokens over 8 heads of 128 15.2 -> 11.6 us, 8.2 at the rate of a copy).  Few: up to four waves share one, since a page of 64
// tokens of 128 is 16 chunks per lane of one wave, all in a row.
template <int D, int P, int WPU>
__global__ __launch_bounds__(WG) void append_fp8_kernel(const AppendParams p) {
    constexpr int CPH = D / 8, NCH = P * CPH / (64 * WPU);   // 8-token-element chunks per token; chunks per lane
    static_assert(NCH >= 1, "every wave of a unit has a chunk per lane");
    __shared__ float shared_amax[WG / 64], shared_scale[WG / 64];
    if ((int)blockIdx.x < p.up_blocks) {
        if (blockIdx.y == 0) upload_rider(p);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int unit = (int)(blockIdx.y * ((blockDim.x >> 6) / WPU)) + wave / WPU, t = (wave % WPU) * 64 + lane;
    if (WPU == 1 && unit >= 2 * p.Hkv) return;               // (WPU > 1: the units fill their workgroups, see launch_append)
    const PageJob j = page_job(p);
    const int is_v = unit & 1, h = unit >> 1, n = j.t1 - j.t0, s0 = j.t0 & (P - 1);
    const int64_t row_bytes = (int64_t)p.Hkv * D * 2;
    const char* src = static_cast<const char*>(is_v ? p.v_new : p.k_new) + ((int64_t)j.row * p.Hkv + h) * D * 2;
    uint8_t* pg = static_cast<uint8_t*>(is_v ? p.v_pool : p.k_pool) + ((int64_t)j.page * p.Hkv + h) * (P * D);
    float* scl = (is_v ? p.v_scale : p.k_scale) + (int64_t)j.page * p.Hkv + h;
    const int n_old = max(0, j.C - (j.t0 & ~(P - 1)));       // slots that already hold tokens
    float s_old = n_old > 0 && t < 64 ? *scl : 0.0f;
    u32x4 x[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const int u = t + 64 * WPU * k;
        x[k] = u32x4{0, 0, 0, 0};
        if (u / CPH < n) x[k] = new_chunk(src, row_bytes, u, CPH);
    }
    float amax = 0.0f;
#pragma unroll
    for (int k = 0; k < NCH; ++k) amax = fmaxf(amax, chunk_amax(x[k]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
    if constexpr (WPU > 1) {                                 // the unit's first wave has read the scale it will overwrite
        const int w0 = wave / WPU * WPU;
        if (lane == 0) {
            shared_amax[wave] = amax;
            shared_scale[wave] = s_old;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WPU; ++w) amax = fmaxf(amax, shared_amax[w0 + w]);
        s_old = shared_scale[w0];
    }
    int e = exponent_for(amax);
    if (n_old > 0) {
        const int e_old = (int)(__float_as_uint(s_old) >> 23) - 127;
        if (e > e_old)
            page_reencode(pg, n_old, D, e_old, e, t, 64 * WPU);
        else
            e = e_old;
    }
    const float inv = __uint_as_float((uint32_t)(127 - e) << 23);
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const int u = t + 64 * WPU * k;
        if (u / CPH < n) *reinterpret_cast<u32x2*>(pg + (s0 + u / CPH) * D + (u % CPH) * 8) = encode_chunk(x[k], inv);
    }
    if (t == 0) *scl = __uint_as_float((uint32_t)(e + 127) << 23);
}

// Work-list upload: the workgroups read the host-built plan straight out of pinned host memory
// and write it to the workspace (cheaper than a runtime copy command for ~100 KB).
__global__ __launch_bounds__(WG) void upload_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int n16) {
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}

// ---------------------------------------------------------------------------------------------
// launchers

hipError_t launch_upload(const void* h_src, void* d_dst, size_t bytes, hipStream_t st) {
    const int n16 = (int)((bytes + 15) / 16);
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(upload_kernel, dim3((n16 + WG - 1) / WG), dim3(WG), 0, st,
                       static_cast<const u32x4*>(h_src), static_cast<u32x4*>(d_dst), n16);
    return hipGetLastError();
}

hipError_t launch_attn(const AttnParams& p, int D, int kvt, bool tiles, int grid, hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    if ((D != 64 && D != 128) || (kvt != KV_BF16 && kvt != KV_FP8)) return hipErrorInvalidValue;
    auto kern = tiles ? (D == 128 ? (kvt == KV_BF16 ? attn_kernel<128, KV_BF16> : attn_kernel<128, KV_FP8>)
                                  : (kvt == KV_BF16 ? attn_kernel<64, KV_BF16> : attn_kernel<64, KV_FP8>))
                      : (D == 128 ? (kvt == KV_BF16 ? narrow_kernel<128, KV_BF16> : narrow_kernel<128, KV_FP8>)
                                  : (kvt == KV_BF16 ? narrow_kernel<64, KV_BF16> : narrow_kernel<64, KV_FP8>));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(AWG), 0, st, p);
    return hipGetLastError();
}

template <int D, int KVT>
static hipError_t launch_rows_t(const AttnParams& p, const RowTable& t, int grid, hipStream_t st) {
    // d = 64: two workgroups of 8 waves fit a CU as they are.
    if constexpr (D == 128) {
        if (t.small && t.max_rows <= (KVT == KV_FP8 ? LEAN_ROWS : 16)) {
            hipLaunchKernelGGL((decode_rows_kernel<D, KVT, 4>), dim3(grid), dim3(256), 0, st, p, t);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((decode_rows_kernel<D, KVT, 8>), dim3(grid), dim3(512), 0, st, p, t);
    return hipGetLastError();
}


hipError_t launch_rows(const AttnParams& p, const RowTable& t, int kvt, int grid, hipStream_t st) {
    if (t.D == 128 && kvt == KV_BF16) return launch_rows_t<128, KV_BF16>(p, t, grid, st);
    if (t.D == 64 && kvt == KV_BF16) return launch_rows_t<64, KV_BF16>(p, t, grid, st);
    if (t.D == 128 && kvt == KV_FP8) return launch_rows_t<128, KV_FP8>(p, t, grid, st);
    if (t.D == 64 && kvt == KV_FP8) return launch_rows_t<64, KV_FP8>(p, t, grid, st);
    return hipErrorInvalidValue;
}

hipError_t launch_tiles(const AttnParams& p, const TileTable& t, int grid, hipStream_t st) {
    bool short_rows = false;
    for (int i = 0; i < t.n_rows; ++i) short_rows |= t.rows[i].L * t.G <= 32;
    auto kern = t.kind == KIND_WIDE ? (t.D == 128 ? attn_tiles_kernel<128, KIND_WIDE, false> : attn_tiles_kernel<64, KIND_WIDE, false>)
                : short_rows        ? (t.D == 128 ? attn_tiles_kernel<128, KIND_NARROW, true> : attn_tiles_kernel<64, KIND_NARROW, true>)
                                    : (t.D == 128 ? attn_tiles_kernel<128, KIND_NARROW, false> : attn_tiles_kernel<64, KIND_NARROW, false>);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(AWG), 0, st, p, t);
    return hipGetLastError();
}

// max_rows: rows of the tallest tile; max_splits: splits of the most finely split one
// t, tt: the launch went by this table (ncombs: split tiles in it), or null
template <int D, int CR>
static void launch_combine_t(const AttnParams& p, const RowTable* t, const TileTable* tt, int ncombs, int max_rows, hipStream_t st) {
    const int ny = (max_rows + CR - 1) / CR;
    if (t)
        hipLaunchKernelGGL((combine_rows_kernel<D, CR>), dim3(t->n * t->Hkv, ny), dim3(WG), 0, st, p, *t);
    else if (tt)
        hipLaunchKernelGGL((combine_tiles_kernel<D, CR>), dim3(ncombs, ny), dim3(WG), 0, st, p, *tt);
    else
        hipLaunchKernelGGL((combine_kernel<D, CR>), dim3(ncombs, ny), dim3(WG), 0, st, p);
}

hipError_t launch_combine(const AttnParams& p, const RowTable* t, const TileTable* tt, int D, int ncombs, int max_rows, int max_splits,
                          hipStream_t st) {
    if (ncombs <= 0) return hipSuccess;
    // many splits and a launch that would otherwise leave most of the chip idle: let thread slices share the splits
    const bool sliced = max_splits > 16 && (int64_t)ncombs * ((max_rows + COMB_ROWS - 1) / COMB_ROWS) < 512;
    if (D == 128) {
        if (sliced) launch_combine_t<128, COMB_ROWS_SLICED>(p, t, tt, ncombs, max_rows, st);
        else launch_combine_t<128, COMB_ROWS>(p, t, tt, ncombs, max_rows, st);
    } else {
        if (sliced) launch_combine_t<64, COMB_ROWS_SLICED>(p, t, tt, ncombs, max_rows, st);
        else launch_combine_t<64, COMB_ROWS>(p, t, tt, ncombs, max_rows, st);
    }
    return hipGetLastError();
}

// f(workgroup columns): one launch per MAX_PAGES pages (a grid holds fewer than 2^32 threads)
template <class F>
static hipError_t for_pages(AppendParams& p, int64_t pages, F&& f) {
    constexpr int64_t MAX_PAGES = 1 << 22;
    for (int64_t at = 0; at < pages; at += MAX_PAGES) {
        p.pg0 = (int32_t)at;
        p.up_blocks = at == 0 ? std::min((p.up_n16 + WG - 1) / WG, 64) : 0;
        f((unsigned)(std::min(MAX_PAGES, pages - at) + p.up_blocks));
    }
    return hipGetLastError();
}

// Waves share units as long as there is no more than one unit per SIMD (4 x 256).  us a launch, one wave a unit -> shared, at 4-127,
// 256-511, 1 024-2 047 and 2 048-4 095 units, d = 128: pages of 64 tokens 4.5 -> 3.4, 5.2 -> 4.2, 7.2 -> 6.8, 12.2 -> 13.0; of 32
// 3.7 -> 3.1, 4.0 -> 3.4, 5.0 -> 4.9, 6.9 -> 8.0; of 16 3.4 -> 3.0, 3.6 -> 3.2, 4.2 -> 4.5, 6.1 -> 7.4.
template <int D, int P>
static hipError_t launch_append_fp8(AppendParams& p, int64_t pages, hipStream_t st) {
    constexpr int SHARE = std::min(WG / 64, P * D / 512);    // waves that share a unit in small launches: a chunk per lane at least
    const int units = 2 * p.Hkv;
    if (pages * units <= 4 * 256)
        return for_pages(p, pages, [&](unsigned nx) {
            hipLaunchKernelGGL((append_fp8_kernel<D, P, SHARE>), dim3(nx, units * SHARE / 4), dim3(WG), 0, st, p);
        });
    const int waves = std::min(WG / 64, units);
    return for_pages(p, pages, [&](unsigned nx) {
        hipLaunchKernelGGL((append_fp8_kernel<D, P, 1>), dim3(nx, (units + waves - 1) / waves), dim3(64 * waves), 0, st, p);
    });
}

hipError_t launch_append(AppendParams& p, int kvt, int64_t pages, hipStream_t st) {
    if (kvt == KV_BF16)
        return for_pages(p, pages, [&](unsigned nx) { hipLaunchKernelGGL(kv_move_bf16_kernel<false>, dim3(nx, 2), dim3(WG), 0, st, p); });
    if (p.D == 128)
        return p.P == 16 ? launch_append_fp8<128, 16>(p, pages, st) : p.P == 32 ? launch_append_fp8<128, 32>(p, pages, st) : launch_append_fp8<128, 64>(p, pages, st);
    return p.P == 16 ? launch_append_fp8<64, 16>(p, pages, st) : p.P == 32 ? launch_append_fp8<64, 32>(p, pages, st) : launch_append_fp8<64, 64>(p, pages, st);
}

hipError_t launch_kv_move(AppendParams& p, bool pack, int64_t pages, hipStream_t st) {
    auto kern = pack ? kv_move_bf16_kernel<true> : kv_move_bf16_kernel<false>;
    return for_pages(p, pages, [&](unsigned nx) { hipLaunchKernelGGL(kern, dim3(nx, 2), dim3(WG), 0, st, p); });
}

}  // namespace ampd
