// Chunked conjugate gradients + read-out in fp32 accuracy on the bf16 matrix cores, for
// d_k = 64 and chunk C = 64 (MESA_PREC_F32, and the backward's fp32 solve).
//
// An fp32 number has 24 significant bits, three bf16 numbers 8 each: every fp32 operand of a
// product is carried exactly as x = h + m + l (h = bf16(x), m = bf16(x - h), l = x - h - m)
// between 2^-98 and 2^127 (below, l falls under the smallest bf16 number; at the top, h rounds
// to infinity; see lift_by), and a product a b as the six terms
//
//   h_a h_b + (h_a m_b + m_a h_b) + (h_a l_b + l_a h_b + m_a m_b),
//
// smallest first, with fp32 accumulation.  What is left out, m_a l_b + l_a m_b + l_a l_b, is
// below 2^-26 of the term, a quarter of an fp32 rounding.  Six v_mfma_f32_16x16x32_bf16 take
// 96 cycles for a 32-long contraction of a 16x16 tile; the eight v_mfma_f32_16x16x4f32 of the
// same contraction take 256.
//
// Work split: as in the other single-wave-per-sub-chunk kernels, wave w owns the tokens
// j = 16w .. 16w+15 and runs their CG without synchronising, with the state entering them,
//
//   B_w = zeta_{16w-1} H_c + sum_{i < 16w} beta_i zeta_{16w-1,i} k_i k_i^T,
//
// in registers (three planes, 96 of them).  It is put together from the sub-chunks' own sums
// E_v = sum_{i in v} beta_i zeta_{end of v,i} k_i k_i^T (48 products by the wave that owns v,
// exchanged through LDS once), so that every weight is a decay (at most one) and nothing is
// divided by one.  A product is then
//
//   (H_t + Lambda) p_j = zs_j (B_w p_j) + sum_{16w <= i <= j} beta_i Z[i][j] k_i (k_i^T p_j) + Lambda p_j,
//
// zs_j the decay from token 16w-1 (wave 0: from the chunk's entering state) to j: 72 matrix
// products per wave and iteration, against up to 192 of four times the length in fp32 form
// (whose causal sum runs over all earlier tokens of the chunk).  Contractions over the 16
// tokens of a sub-chunk fill a 32-long one with two of the six terms side by side.
//
// Bound by the vector work of the splits and the serial chain of an iteration; the keys' parts
// stay in LDS so that two workgroups share a compute unit (in registers: 305 of them, one
// workgroup, 141 us where this takes 100).  Solve, 15 iterations, in fp32 form and here: B4 H8
// T2048 217 and 100 us, B1 H2 T256 (eight workgroups) 52 and 27 us; error against 64 bits
// 2.9e-7 and 2.6e-7.
#include "mesa_device.hpp"
#include "mesa_kernels.hpp"
#include "mesa_mfma.hpp"

namespace mesa {
namespace {

constexpr int kC = 64;
constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int DK = 64;
constexpr int MT = DK / 16;  // 16-row tiles of a per-token vector
constexpr int KS = DK / 32;  // 32-long contraction steps over features

// Three bf16 parts of two fp32 values, each pair packed as a | b << 16.  The empty asm keeps
// the packed word the only source of the widened parts (the compiler would otherwise convert
// the first value of the pair once more).
__device__ __forceinline__ void split3x2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = pack_bf16x2(a, b);
    asm("" : "+v"(h));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = pack_bf16x2(a, b);
    asm("" : "+v"(m));
    l = pack_bf16x2(a - __uint_as_float(m << 16), b - __uint_as_float(m & 0xffff0000u));
}

struct Half3 {  // three parts of four values: half of an 8-wide operand each
    uint2 h, m, l;
};
__device__ __forceinline__ Half3 split3(const f32x4& v)
{
    Half3 r;
    split3x2(v[0], v[1], r.h.x, r.m.x, r.l.x);
    split3x2(v[2], v[3], r.h.y, r.m.y, r.l.y);
    return r;
}
__device__ __forceinline__ bf16x8 halves(const uint2& a, const uint2& b)
{
    return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
}

struct Op3 {  // three parts of an 8-wide operand
    bf16x8 h, m, l;
};
__device__ __forceinline__ Op3 op3(const f32x4& lo, const f32x4& hi)
{
    const Half3 a = split3(lo), b = split3(hi);
    return Op3{halves(a.h, b.h), halves(a.m, b.m), halves(a.l, b.l)};
}
// acc + a b
__device__ __forceinline__ f32x4 mfma6(const Op3& a, const Op3& b, f32x4 acc)
{
    acc = mfma16(a.l, b.h, acc);
    acc = mfma16(a.h, b.l, acc);
    acc = mfma16(a.m, b.m, acc);
    acc = mfma16(a.m, b.h, acc);
    acc = mfma16(a.h, b.m, acc);
    return mfma16(a.h, b.h, acc);
}

// The same for a 16-long contraction, two terms per 32-long one: the left operand as (h, h),
// (m, m), (h, l), the right one as (h, m), (l, h).
struct Left16 {
    bf16x8 hh, mm, hl;
};
struct Right16 {
    bf16x8 hm, lh;
};
__device__ __forceinline__ Left16 left16(const Half3& a) { return Left16{halves(a.h, a.h), halves(a.m, a.m), halves(a.h, a.l)}; }
__device__ __forceinline__ Right16 right16(const Half3& a) { return Right16{halves(a.h, a.m), halves(a.l, a.h)}; }
__device__ __forceinline__ f32x4 mfma6(const Left16& a, const Right16& b, f32x4 acc)
{
    acc = mfma16(a.hl, b.lh, acc);
    acc = mfma16(a.mm, b.hm, acc);
    return mfma16(a.hh, b.hm, acc);
}

// The values four packed parts stand for.
__device__ __forceinline__ f32x4 join3(const Half3& a)
{
    const uint32_t h[2] = {a.h.x, a.h.y}, m[2] = {a.m.x, a.m.y}, l[2] = {a.l.x, a.l.y};
    f32x4 r;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        r[2 * q] = __uint_as_float(h[q] << 16) + (__uint_as_float(m[q] << 16) + __uint_as_float(l[q] << 16));
        r[2 * q + 1] = __uint_as_float(h[q] & 0xffff0000u) + (__uint_as_float(m[q] & 0xffff0000u) + __uint_as_float(l[q] & 0xffff0000u));
    }
    return r;
}

// Operands that lie at an end of fp32 are brought into the range that splits exactly by a power of
// two, which the result gives back: reach 0 stands for numbers all below 2^-60, 2 for some from
// 2^127 on, 1 for others (the same for every lane of a wave).  The keys are split as they are (the
// parts of one of 2^-110 still hold 23 bits of it; its square is long gone from H).
__device__ __forceinline__ float lift_by(int reach) { return reach == 0 ? 0x1p60f : reach == 2 ? 0x1p-60f : 1.0f; }
__device__ __forceinline__ int reach_of(float largest)
{
    return __any(largest >= 0x1p127f) ? 2 : __any(largest >= 0x1p-60f) ? 1 : 0;
}
__device__ __forceinline__ float largest4(float m, const f32x4& v)
{
    return fmaxf(fmaxf(m, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
}
template <int N>
__device__ __forceinline__ int reach_of(const f32x4 (&v)[N])
{
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) t = largest4(t, v[i]);
    return reach_of(t);
}
template <int N>
__device__ __forceinline__ void scale(f32x4 (&v)[N], float by)
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] *= by;
}

constexpr int kSwizzle = 8;  // of the token-major tiles: also spreads reads of one feature group of 16 tokens

// Operand with rows = tokens 16 i + n, contraction = features 32 s ..: two 8-byte reads at a
// lane offset that is formed once (bytes; the piece index is its bits above 16 bytes, rows
// are a power of two long).
template <int D>
__device__ __forceinline__ uint32_t row_frag_offset(int i, int g, int n)
{
    return (16 * i + n) * D * 2 + ((g / 2) ^ (n % 8)) * 16 + 8 * (g % 2);
}
__device__ __forceinline__ bf16x8 row_frag_at(const uint16_t* tile, uint32_t off, int s)
{
    const char* base = reinterpret_cast<const char*>(tile);
    return halves(*reinterpret_cast<const uint2*>(base + (off ^ (4 * s * 16))),
                  *reinterpret_cast<const uint2*>(base + (off ^ ((4 * s + 2) * 16))));
}

// beta_i prod_{s=i+1..j} gamma_s for the tokens i = i4 .. i4+3 (zero for i > j): lgj = lg[j], zlj = zl[j].
__device__ __forceinline__ f32x4 decay_weights4(const float* lg, const float* beta, float lgj, int zlj, int i4, int j)
{
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (i4 + e <= j && zlj <= i4 + e) ? beta[i4 + e] * expf(lgj - lg[i4 + e]) : 0.0f;
    return r;
}

template <typename Tin, int DV>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void chunk_cg_f32_split_kernel(CgArgs a)
{
    constexpr int MTV = DV / 16;
    const ForwardShape s = a.s;
    const int n_chunk = blockIdx.x % s.n_chunks;
    const int64_t bh = blockIdx.x / s.n_chunks;
    const int64_t t0 = int64_t(n_chunk) * kC;
    const int valid = int(min<int64_t>(kC, s.seq_len - t0));
    const int64_t tok0 = bh * s.seq_len + t0;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave, g = lane / 16, n = lane % 16;
    const int j = 16 * wave + n;  // this lane's token

    __shared__ __attribute__((aligned(16))) uint16_t sK[3][kC * DK];   // keys, three parts, token-major
    // the sub-chunk sums E_0 .. E_2 (16 tiles of 64 lanes x 4), then, during CG, every wave's
    // key columns as left operands, and at the read-out the values' three parts
    constexpr int kEBytes = (kWaves - 1) * MT * MT * kWave * 16, kVBytes = 3 * kC * DV * 2;
    __shared__ __attribute__((aligned(16))) unsigned char sEV[kEBytes > kVBytes ? kEBytes : kVBytes];
    static_assert(kWaves * MT * 3 * kWave * 16 <= kEBytes, "the key operands run past the sums");
    __shared__ __attribute__((aligned(16))) float sLam[DK];
    __shared__ float sDiag[kWaves][DK];
    __shared__ float sLg[kC], sBeta[kC];
    __shared__ __attribute__((aligned(16))) float sWe[kC];  // beta_i x decay from i to its sub-chunk's last token
    __shared__ int sZl[kC];
    __shared__ int sReach[kWaves];
    f32x4* sE = reinterpret_cast<f32x4*>(sEV);
    bf16x8* sKL = reinterpret_cast<bf16x8*>(sEV);
    uint16_t* sV = reinterpret_cast<uint16_t*>(sEV);

    const Tin* kp = static_cast<const Tin*>(a.k) + tok0 * DK;
    const Tin* vp = static_cast<const Tin*>(a.v) + tok0 * DV;
    const f32x4 zero4 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- staging: gates, lambda, the keys' parts; right-hand side and H_c to registers.  The
    // gates are loaded first: loads return in order, and their scan is the longest way to the
    // barrier.
    const float gl = wave == 0 && lane < valid ? a.gamma[tok0 + lane] : 1.0f;
    const float bl = lane < valid ? a.beta[tok0 + lane] : 0.0f;
    const float laml = a.lambda[(bh % s.heads) * DK + lane];
    constexpr int kPer = kC * DK / 8 / kThreads;  // 8-feature pieces per thread
    f32x4 kv[kPer][2];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int piece = tid + u * kThreads, tok = piece / (DK / 8), c = piece % (DK / 8);
        const Tin* src = kp + int64_t(min(tok, valid - 1)) * DK + 8 * c;
        kv[u][0] = load_vec4(src);
        kv[u][1] = load_vec4(src + 4);
    }
    // A operand tile (mt, ks), half hh: H[16 mt + n][32 ks + 16 hh + 4 g ..] (H symmetric)
    const float* Hc = static_cast<const float*>(a.Hs) + (bh * s.n_chunks + n_chunk) * int64_t(DK) * DK;
    f32x4 hacc[MT][KS][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                hacc[mt][ks][hh] = *reinterpret_cast<const f32x4*>(Hc + (16 * mt + n) * DK + 32 * ks + 16 * hh + 4 * g);
    f32x4 qv[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int64_t off = (tok0 + min(j, valid - 1)) * DK + 16 * t + 4 * g;
        const f32x4 v = a.rhs ? load_vec4(a.rhs + off) : load_vec4(static_cast<const Tin*>(a.q) + off);
        qv[t] = j < valid ? v : zero4;
    }
    if (wave == 0) {  // gate log-cumsums; a zero gate resets memory through zl instead of log 0
        sLg[lane] = wave_scan_add(gl > 0.0f ? logf(gl) : 0.0f);
        sZl[lane] = wave_scan_max((lane < valid && !(gl > 0.0f)) ? lane : -1);
    }
    if (wave == 1) sBeta[lane] = bl;
    if (wave == 2) sLam[lane] = laml;
    static_assert(DK == kWave, "one lane per feature of lambda");
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int piece = tid + u * kThreads, tok = piece / (DK / 8), c = piece % (DK / 8);
        if (tok >= valid) kv[u][0] = kv[u][1] = zero4;
        const Op3 k3 = op3(kv[u][0], kv[u][1]);
        *reinterpret_cast<bf16x8*>(tile_piece<DK, kSwizzle>(sK[0], tok, c)) = k3.h;
        *reinterpret_cast<bf16x8*>(tile_piece<DK, kSwizzle>(sK[1], tok, c)) = k3.m;
        *reinterpret_cast<bf16x8*>(tile_piece<DK, kSwizzle>(sK[2], tok, c)) = k3.l;
    }
    __syncthreads();

    // ---- this sub-chunk's keys as operands: columns of W (features x the 16 tokens) and rows of S
    const float lgj = sLg[j];
    const int zlj = sZl[j];
    const int jb = 16 * wave - 1, je = 16 * wave + 15;  // the sub-chunk's entering and last token
    // decay from the sub-chunk's entering state to token j
    const float zs = wave == 0 ? decay_from_start(sLg, sZl, j) : decay_between(sLg, sZl, jb, j);
    const f32x4 zw = decay_weights4(sLg, sBeta, lgj, zlj, 16 * wave + 4 * g, j);
    Half3 kh[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
        kh[t] = Half3{tile_col_half<DK, kSwizzle>(sK[0], t, wave, g, n), tile_col_half<DK, kSwizzle>(sK[1], t, wave, g, n),
                      tile_col_half<DK, kSwizzle>(sK[2], t, wave, g, n)};

    // ---- E_w (the last wave's is not needed), then B_w, and its parts as operands.  Tile
    // (rt, ct) of E holds rows 16 rt + 4 g .., column 16 ct + n: the layout of hacc[ct][rt / 2][rt % 2].
    const f32x4 we = decay_weights4(sLg, sBeta, sLg[je], sZl[je], 16 * wave + 4 * g, je);
    if (n == 0) *reinterpret_cast<f32x4*>(sWe + 16 * wave + 4 * g) = we;
    if (wave + 1 < kWaves) {
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            const Right16 wk = right16(split3(join3(kh[ct]) * we));
#pragma unroll
            for (int rt = 0; rt < MT; ++rt) sE[((wave * MT + ct) * MT + rt) * kWave + lane] = mfma6(left16(kh[rt]), wk, zero4);
        }
    }
    __syncthreads();
    // decays to the sub-chunk's entering token: of E_v
    float zv[kWaves - 1];
#pragma unroll
    for (int v = 0; v < kWaves - 1; ++v) zv[v] = v < wave ? decay_between(sLg, sZl, 16 * v + 15, jb) : 0.0f;
    Op3 hf[MT][KS];
    float zh;  // zs, and what takes the lift of hf back
    {
        const float z0 = wave == 0 ? 1.0f : decay_from_start(sLg, sZl, jb);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) hacc[mt][ks][hh] *= z0;
#pragma unroll
        for (int v = 0; v < kWaves - 1; ++v)
            if (v < wave) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int hh = 0; hh < 2; ++hh)
                            hacc[mt][ks][hh] += zv[v] * sE[((v * MT + mt) * MT + 2 * ks + hh) * kWave + lane];
            }
        // diagonal: row 16 mt + n of row tile mt sits at 4 g + e = n.  B_w is positive semidefinite, so no
        // element is larger than the largest of it.
        float top = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f32x4 d = hacc[mt][mt / 2][mt % 2];
            const int e = n - 4 * g;
            if (e >= 0 && e < 4) {
                const float de = e == 0 ? d[0] : e == 1 ? d[1] : e == 2 ? d[2] : d[3];
                sDiag[wave][16 * mt + n] = de;
                top = fmaxf(top, de);
            }
        }
        const int reach_h = reach_of(top);
        zh = zs * lift_by(2 - reach_h);
        if (reach_h != 1) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) scale(hacc[mt][ks], lift_by(reach_h));
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) hf[mt][ks] = op3(hacc[mt][ks][0], hacc[mt][ks][1]);
    }

    __syncthreads();  // every wave is done with the sums
    // The key columns are operands of every product; in LDS (read back each time) they leave
    // the registers to two workgroups per compute unit, whose products and vector work overlap.
    const int kl0 = wave * MT * 3 * kWave + lane;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const Left16 kl = left16(kh[t]);
        sKL[kl0 + (3 * t + 0) * kWave] = kl.hh;
        sKL[kl0 + (3 * t + 1) * kWave] = kl.mm;
        sKL[kl0 + (3 * t + 2) * kWave] = kl.hl;
    }
    const uint32_t kf0 = row_frag_offset<DK>(wave, g, n);

    auto col_dot = [&](const f32x4 (&u)[MT], const f32x4 (&v)[MT]) __attribute__((always_inline)) -> float {
        f32x4 acc = u[0] * v[0];
#pragma unroll
        for (int t = 1; t < MT; ++t) acc += u[t] * v[t];
        return row_pair_sums((acc[0] + acc[1]) + (acc[2] + acc[3]));
    };
    // w = A_j vec
    auto matvec = [&](const f32x4 (&vec)[MT], f32x4 (&w)[MT]) __attribute__((always_inline)) {
        uint32_t kfo = kf0;
        int klo = kl0;
        asm volatile("" : "+v"(kfo), "+v"(klo));  // the operands are read each time, not kept
        f32x4 sacc = zero4;
        Op3 kf[KS], v[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            kf[ks] = Op3{row_frag_at(sK[0], kfo, ks), row_frag_at(sK[1], kfo, ks), row_frag_at(sK[2], kfo, ks)};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) v[ks] = op3(vec[2 * ks], vec[2 * ks + 1]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            sacc = mfma6(kf[ks], v[ks], sacc);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) w[mt] = mfma6(hf[mt][ks], v[ks], ks == 0 ? zero4 : w[mt]);
        }
        const Right16 sb = right16(split3(sacc * zw));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f32x4 lam = *reinterpret_cast<const f32x4*>(sLam + 16 * mt + 4 * g);
            const Left16 kl = Left16{sKL[klo + 3 * mt * kWave], sKL[klo + (3 * mt + 1) * kWave], sKL[klo + (3 * mt + 2) * kWave]};
            w[mt] = mfma6(kl, sb, zh * w[mt] + lam * vec[mt]);
        }
    };

    // ---- each column solves for q scaled by a power of two that brings |q|^2 into [1/2, 2);
    // Jacobi start with diag(H_t + Lambda) = zs_j diag(B_w) + sum_i beta_i Z[i][j] k_i^2 + lambda
    const int qsh = cg_scale_shift(col_dot(qv, qv));
    f32x4 x[MT], r[MT], p[MT], w[MT];
    {
        const float qs = __builtin_ldexpf(1.0f, -qsh);
        const Right16 zb = right16(split3(zw));
        f32x4 d[MT];
        float least = INFINITY, top = 0.0f;
#pragma unroll
        for (int t = 0; t < MT; ++t) top = largest4(top, join3(kh[t]));
        // squares of keys below 2^-30 or from 2^63 on lie at an end of fp32
        const float kup = !__any(top >= 0x1p-30f) ? 0x1p30f : __any(top >= 0x1p63f) ? 0x1p-30f : 1.0f, kback = 1.0f / (kup * kup);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const f32x4 k = kup * join3(kh[t]);
            const f32x4 acc = mfma6(left16(split3(k * k)), zb, zero4);
            qv[t] *= qs;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int f = 16 * t + 4 * g + e;
                d[t][e] = zs * sDiag[wave][f] + kback * acc[e] + sLam[f];
                least = fminf(least, d[t][e]);
            }
        }
        // a large system has a small x, a tiny one a large x; CG's other directions are residuals
        // of a unit q
        const bool large = !__any(least < 0x1p60f), tiny = __any(least < 0x1p-100f);
        const float up = large ? 0x1p60f : tiny ? 0x1p-60f : 1.0f, down = large ? 0x1p-60f : tiny ? 0x1p60f : 1.0f;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[t][e] = up * qv[t][e] / d[t][e];
            x[t] = down * p[t];
        }
        matvec(p, w);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            r[t] = qv[t] - down * w[t];
            p[t] = r[t];
        }
    }
    float delta = col_dot(r, r);
    const float thr = a.eps2 * delta;  // Alg. 1: the column stops once |r|^2 <= eps^2 |r_0|^2
    bool active = delta >= kMinNormal;
    int steps = 0;

    // ---- CG (App. C, Alg. 1), branch-free over the columns: a stopped column takes alpha = 0
    // and keeps x.  It stops after its x update when the new squared residual meets the
    // relative test or falls below the smallest normal number, and without an update when
    // p^T A p is not a positive normal number.
    for (int it = 0; it < a.n_cg; ++it) {
        if (!__any(active)) break;
        matvec(p, w);
        const float pw = col_dot(p, w);
        const bool act1 = active && pw >= kMinNormal;
        steps += act1 ? 1 : 0;
        const float alpha = act1 ? delta / pw : 0.0f;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            r[t] -= alpha * w[t];
            x[t] += alpha * p[t];
        }
        const float dn = col_dot(r, r);
        const bool act2 = act1 && dn >= kMinNormal && dn > thr;
        const float bcg = act2 ? dn / delta : 0.0f;
#pragma unroll
        for (int t = 0; t < MT; ++t) p[t] = r[t] + bcg * p[t];
        delta = act2 ? dn : delta;
        active = act2;
    }
    {
        const float us = __builtin_ldexpf(1.0f, qsh);
#pragma unroll
        for (int t = 0; t < MT; ++t) x[t] *= us;
    }
    if (a.steps && g == 0 && j < valid) a.steps[tok0 + j] = steps;
    if (a.qstar && j < valid) {
#pragma unroll
        for (int t = 0; t < MT; ++t) *reinterpret_cast<f32x4*>(a.qstar + (tok0 + j) * DK + 16 * t + 4 * g) = x[t];
    }
    if (!a.out) return;  // solve only (uniform across the workgroup)

    // ---- read-out o_j = zeta_j G_c x_j + sum_{i<=j} beta_i zeta_{j,i} v_i (k_i . x_j)
    constexpr int kPerV = kC * DV / 8 / kThreads;
    auto load_v = [&](f32x4 (&vv)[2 * kPerV], int id) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kPerV; ++u) {
            const int piece = id + u * kThreads, tok = piece / (DV / 8), c = piece % (DV / 8);
            const Tin* src = vp + int64_t(min(tok, valid - 1)) * DV + 8 * c;
            vv[2 * u] = load_vec4(src);
            vv[2 * u + 1] = load_vec4(src + 4);
            if (tok >= valid) vv[2 * u] = vv[2 * u + 1] = zero4;
        }
    };
    auto stage_v = [&](const f32x4 (&vv)[2 * kPerV], int id) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kPerV; ++u) {
            const int piece = id + u * kThreads, tok = piece / (DV / 8), c = piece % (DV / 8);
            const Op3 v3 = op3(vv[2 * u], vv[2 * u + 1]);
            *reinterpret_cast<bf16x8*>(tile_piece<DV, kSwizzle>(sV, tok, c)) = v3.h;
            *reinterpret_cast<bf16x8*>(tile_piece<DV, kSwizzle>(sV + kC * DV, tok, c)) = v3.m;
            *reinterpret_cast<bf16x8*>(tile_piece<DV, kSwizzle>(sV + 2 * kC * DV, tok, c)) = v3.l;
        }
    };
    f32x4 vv[2 * kPerV];
    load_v(vv, tid);
    // G_c's rows as operand halves, all on their way before the products that come first
    const float* Gc = static_cast<const float*>(a.Gs) + (bh * s.n_chunks + n_chunk) * int64_t(DV) * DK;
    constexpr int kAhead = 4;  // row tiles in flight (64 registers)
    auto load_g = [&](f32x4 (&gv)[2 * KS], int mt) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) gv[2 * ks + hh] = load_vec4(Gc + (16 * mt + n) * DK + 32 * ks + 16 * hh + 4 * g);
    };
    auto times_x = [&](const f32x4 (&gv)[2 * KS], const Op3 (&xv)[KS]) __attribute__((always_inline)) -> f32x4 {
        f32x4 o = zero4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) o = mfma6(op3(gv[2 * ks], gv[2 * ks + 1]), xv[ks], o);
        return o;
    };
    f32x4 gv[kAhead][2 * KS];
#pragma unroll
    for (int mt = 0; mt < kAhead; ++mt) load_g(gv[mt], mt);
    const int reach_x = reach_of(x);
    const float back = lift_by(2 - reach_x);
    if (reach_x != 1) scale(x, lift_by(reach_x));
    Op3 xv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xv[ks] = op3(x[2 * ks], x[2 * ks + 1]);
    int jr = j, nr = n;
    asm volatile("" : "+v"(jr), "+v"(nr));  // decays and addresses are formed again, not kept through CG
    const float zeta = decay_from_start(sLg, sZl, jr), zr = wave == 0 ? zeta : decay_between(sLg, sZl, jb, jr);
    // S' over the token tiles, as right operands of two 32-token steps.  Every wave forms all
    // four tiles (the last wave needs them, and the others wait for it) and drops the ones past
    // its own; the weight of an earlier sub-chunk's token is the product of three decays.
    f32x4 sp[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        sp[it] = zero4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint32_t off = row_frag_offset<DK>(it, g, n);
            sp[it] = mfma6(Op3{row_frag_at(sK[0], off, ks), row_frag_at(sK[1], off, ks), row_frag_at(sK[2], off, ks)}, xv[ks], sp[it]);
        }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const f32x4 wt = it == wave ? zw : zr * (zv[it < kWaves - 1 ? it : 0] * *reinterpret_cast<const f32x4*>(sWe + 16 * it + 4 * g));
#pragma unroll
        for (int e = 0; e < 4; ++e) sp[it][e] = 16 * it + 4 * g + e <= j ? sp[it][e] * wt[e] : 0.0f;
    }
    Op3 so[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) so[u] = op3(sp[2 * u], sp[2 * u + 1]);
    // o + the staged values' part of row tile mt
    auto add_values = [&](f32x4 o, int mt) __attribute__((always_inline)) -> f32x4 {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (2 * u > wave) continue;
            // a later sub-chunk's values are masked out, not multiplied by zero: an infinity or a
            // NaN among them must not reach this sub-chunk's tokens
            const uint32_t keep = 2 * u + 1 <= wave ? ~0u : 0u;
            auto pair = [&](uint16_t* tv) __attribute__((always_inline)) -> bf16x8 {
                const uint2 later = tile_col_half<DV, kSwizzle>(tv, mt, 2 * u + 1, g, nr);
                return halves(tile_col_half<DV, kSwizzle>(tv, mt, 2 * u, g, nr), make_uint2(later.x & keep, later.y & keep));
            };
            o = mfma6(Op3{pair(sV), pair(sV + kC * DV), pair(sV + 2 * kC * DV)}, so[u], o);
        }
        return o;
    };
    __syncthreads();  // every wave is done with its key operands
    stage_v(vv, tid);
    __syncthreads();
    float sum = 0.0f;  // of this lane's |outputs|
#pragma unroll
    for (int mt = 0; mt < MTV; ++mt) {
        f32x4 o = times_x(gv[mt % kAhead], xv);
        if (mt + kAhead < MTV) load_g(gv[mt % kAhead], mt + kAhead);
        o = add_values(o * zeta, mt) * back;
        sum += (fabsf(o[0]) + fabsf(o[1])) + (fabsf(o[2]) + fabsf(o[3]));
        if (j < valid) *reinterpret_cast<f32x4*>(a.out + (tok0 + j) * DV + 16 * mt + 4 * g) = o;
    }
    // A sub-chunk whose outputs are all tiny or not all finite may owe it to values or a state at an
    // end of fp32: its read-out is done again with those lifted, row tile by row tile.  (Lifting
    // them in the loop above: B1 H2 T256 34.1 us; this way 32.9.)
    const bool again = 16 * wave < valid && (!__any(j < valid && sum >= 0x1p-60f) || __any(j < valid && !(sum < INFINITY)));
    if (lane == 0) sReach[wave] = again;
    __syncthreads();
    if (!(sReach[0] | sReach[1] | sReach[2] | sReach[3])) return;
    int id = tid;
    asm volatile("" : "+v"(id));  // addresses are formed again, not kept
    load_v(vv, id);
    const int rv = reach_of(vv);
    __syncthreads();  // every wave has read the flags
    if (lane == 0) sReach[wave] = rv;
    __syncthreads();
    const int reach_v = max(max(sReach[0], sReach[1]), max(sReach[2], sReach[3]));
    scale(vv, lift_by(reach_v));
    stage_v(vv, id);
    __syncthreads();
    if (!again) return;
#pragma unroll 1
    for (int mt = 0; mt < MTV; ++mt) {
        load_g(gv[0], mt);
        const int reach_g = reach_of(gv[0]);
        scale(gv[0], lift_by(reach_g));
        const f32x4 o = times_x(gv[0], xv) * (zeta * lift_by(2 - reach_g) * back) + add_values(zero4, mt) * (lift_by(2 - reach_v) * back);
        if (j < valid) *reinterpret_cast<f32x4*>(a.out + (tok0 + j) * DV + 16 * mt + 4 * g) = o;
    }
}

template <typename Tin>
hipError_t launch_tin(const CgArgs& a, hipStream_t stream)
{
    const unsigned blocks = unsigned(a.s.batch * a.s.heads * a.s.n_chunks);
    if (a.s.d_v == 64)
        hipLaunchKernelGGL((chunk_cg_f32_split_kernel<Tin, 64>), dim3(blocks), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((chunk_cg_f32_split_kernel<Tin, 128>), dim3(blocks), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_chunk_cg_f32_split(const CgArgs& a, hipStream_t stream)
{
    if (a.s.d_k != DK || a.s.chunk != kC || (a.s.d_v != 64 && a.s.d_v != 128)) return hipErrorInvalidValue;
    return a.s.bf16 ? launch_tin<bf16_t>(a, stream) : launch_tin<float>(a, stream);
}

}  // namespace mesa
