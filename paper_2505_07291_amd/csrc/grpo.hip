// libgrpo: token-level GRPO objective with two-sided clipping (INTELLECT-2 paper,
// section 3.4, objective with the bound delta; token-level mean of section 4.1),
// forward and fused backward, hand-written for gfx950 (MI355X).
//
// The path is a streaming reduction over rows of 152k logits: it is bound by HBM
// bandwidth, not by arithmetic, so there is no MFMA here.  The design keeps one
// whole row resident in the vector registers of one workgroup (304 KB of the CU's
// 512 KB register file for a 152064-wide bf16 row: 512 lanes with 256 registers each,
// 152 of them the row), so that the row is
// read from HBM once, reduced twice (max, sum of exponentials) out of registers,
// and the gradient is produced from the same registers: 1 read + 1 write of HBM
// traffic per row instead of 2 reads + 1 write.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>

#include "grpo.h"

// The row kernels' instantiations take most of the compiler's time: build.py compiles this file once for each element type
// with and without the auxiliary terms (GRPO_ROWS_OF: the arguments of launch_rows) and once for everything else
// (GRPO_ROWS_APART), at the same time.  With neither defined it is the whole library.  The parts find each other's names, and
// nothing outside the library does: two builds of it in one process would otherwise call each other's.
namespace __attribute__((visibility("hidden"))) grpo_impl {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr unsigned kNegInfF32 = 0xff800000u;
constexpr unsigned kNegInfBf16x2 = 0xff80ff80u;

constexpr int kFlagClipHigh = 1, kFlagClipLow = 2, kFlagDelta = 4, kFlagOutOfBand = 8;

// First 256 bytes of the caller's workspace.
struct WsHeader {
    double D;      // denominator of the token-level mean
    double inv_D;  // 1 / D, or 0 when D == 0
    long long M;   // rows with mask != 0
    int error;     // sticky data-error word (bit 0: token id out of range)
    unsigned fin_ticket;  // blocks of grpo_finalize that have delivered their partial sums
};
// The row queue: up to kQueueParts counters, each on a 128-byte line of its own, follow
// the 256-byte header.  With P counters in use, counter q hands out the rows q, q + P,
// q + 2P, ...  One counter for the whole GPU sustains only some 15-25 million increments
// a second under contention (measured): enough for 300 KB rows (8 million rows a second),
// not for 64 KB rows.  Narrow rows therefore use eight interleaved partitions, each
// started on by an eighth of the workgroups and then stolen from in turn, which keeps
// single-row granularity; wide rows use one counter, which measured 4-6 % faster there.
constexpr int kOrderRows = 4096;    // rows one workgroup of grpo_prepare orders: four per lane
constexpr int kFinSegment = 16384;  // rows one workgroup of grpo_finalize takes: sixteen per lane
constexpr int kQueueParts = 8;
constexpr long long kOrderMinRowBytes = 32768;  // narrower rows are handed out several at a time, in index order
constexpr int kQueueStride = 16;  // in unsigned long long: 128 bytes
constexpr size_t kHeaderBytes = 256 + (size_t)kQueueParts * kQueueStride * 8;
__device__ __forceinline__ unsigned long long *queue_counters(WsHeader *hdr)
{
    return (unsigned long long *)((char *)hdr + 256);
}
constexpr long long kMaxVocab = 1ll << 28;  // byte offsets inside a row stay below 2^32

struct RowParams {
    const void *logits;
    void *grad;  // may alias logits: deliberately no __restrict__ anywhere
    const long long *tokens;
    const float *old_lp;
    const float *adv;
    const unsigned char *mask;
    float *logprobs_out;
    float *J_ws;
    unsigned char *flags_ws;
    WsHeader *hdr;
    long long n_tokens, vocab, row_stride;
    float k;      // log2(e) / T: exponents are kept in base 2 for v_exp_f32
    float inv_T;  // 1 / T
    float lo, hi, delta, grad_scale;
    int bwd;  // 0: log-probs only (grpo_logprobs_fwd), 1: objective + gradient
    const int *order;  // optional: the rows in the order they are handed out (grpo_prepare, row_of), else 0, 1, 2, ...
    int queued;       // rows come from the queue in the workspace (0: strided over the grid)
    int queue_chunk;  // rows taken from the queue per increment
    int queue_parts;  // counters in use (1 or kQueueParts)
    int queue_more;   // log-probs only: how many at once while a counter has not passed more_until
    long long more_until;
    // auxiliary terms (kernels instantiated with AUX only)
    const float *ref_lp;  // reference-policy log-probs, or NULL (no KL term)
    const float *token_w; // per-token weights omega_t, or NULL (all ones); 0 = masked row
    float *KL_ws, *H_ws;  // per-row KL estimate and entropy
    float *entropy_out;   // optional copy of the per-row entropy for the caller
    float kl_coef, ent_coef;
    // small batches of narrow rows: the row kernel counts the rows that take part itself (kCountRows)
    int count_here;
    double denom;  // the caller's denominator, or <= 0: that count
    // where gradient rows start inside a 128-byte line, in 16-byte vectors: row r at (shift0 + r shift_step) mod 8
    // (both 0: rows are processed from their first vector on, see row_shift)
    unsigned shift0, shift_step;
};

// How many vectors in front of row r its first 128-byte line of gradients begins: rows are taken from there on, so that every
// store of a wavefront covers whole lines.  A store that begins inside a line leaves its first and its last line to be
// written in two parts, by two wavefronts, and the memory writes each part by itself: 4096 x 152064 bf16, a third of the
// rows masked, 359 us a step at a pitch of 152064 and 409 at 152072, where it now takes 367; 4096 x 50257 fp32 257 at 50304
// and 283 at 50260, now 261 (loads do not care: the log-probs pass takes the same time at either pitch).
__device__ __forceinline__ unsigned row_shift(const RowParams &p, long long r)
{
    return (p.shift0 + (unsigned)r * p.shift_step) & 7u;
}

template <grpo_dtype DT>
struct Elem;
template <>
struct Elem<GRPO_BF16> {
    static constexpr int EPV = 8, BYTES = 2;
};
template <>
struct Elem<GRPO_F32> {
    static constexpr int EPV = 4, BYTES = 4;
};

// Tunables, with the settings measured best on MI355X (5 GB to 20 GB of logits):
//  - non-temporal loads and stores for the two row streams: every byte is touched
//    once, so nothing is gained by keeping it in L2 / Infinity Cache
//    (log-probs pass 5.5 -> 6.3 TB/s, mixed batches about 4% faster).
#ifndef GRPO_NT_LOAD
#define GRPO_NT_LOAD 1
#endif
#ifndef GRPO_NT_STORE
#define GRPO_NT_STORE 1
#endif
// 16-byte global accesses of the row streams.
__device__ __forceinline__ u32x4 ld16(const char *p)
{
#if GRPO_NT_LOAD
    return __builtin_nontemporal_load((const u32x4 *)p);
#else
    return *(const u32x4 *)p;
#endif
}
__device__ __forceinline__ void st16(char *p, const u32x4 &v)
{
#if GRPO_NT_STORE
    __builtin_nontemporal_store(v, (u32x4 *)p);
#else
    *(u32x4 *)p = v;
#endif
}

__device__ __forceinline__ float as_f32(unsigned u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ unsigned as_u32(float f) { return __builtin_bit_cast(unsigned, f); }

// 16-byte vector -> EPV floats.  A bf16 is the upper half of a binary32.
template <grpo_dtype DT>
__device__ __forceinline__ void unpack(const u32x4 &v, float (&f)[Elem<DT>::EPV])
{
    if constexpr (DT == GRPO_BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = as_f32(v[i] << 16);
            f[2 * i + 1] = as_f32(v[i] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = as_f32(v[i]);
    }
}

// EPV floats -> 16-byte vector; bf16 rounds to nearest even (v_cvt_pk_bf16_f32).
template <grpo_dtype DT>
__device__ __forceinline__ u32x4 pack(const float (&f)[Elem<DT>::EPV])
{
    u32x4 v;
    if constexpr (DT == GRPO_BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f32x2 p = {f[2 * i], f[2 * i + 1]};
            v[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = as_u32(f[i]);
    }
    return v;
}

template <grpo_dtype DT>
__device__ __forceinline__ float load_elem(const char *row, long long j)
{
    if constexpr (DT == GRPO_BF16)
        return as_f32((unsigned)((const unsigned short *)row)[j] << 16);
    else
        return ((const float *)row)[j];
}

template <grpo_dtype DT>
__device__ __forceinline__ void store_elem(char *row, long long j, float x)
{
    if constexpr (DT == GRPO_BF16) {
        f32x2 p = {x, 0.f};
        unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2));
        ((unsigned short *)row)[j] = (unsigned short)(u & 0xffffu);
    } else {
        ((float *)row)[j] = x;
    }
}

template <grpo_dtype DT>
__device__ __forceinline__ u32x4 neg_inf_vec()
{
    unsigned w = (DT == GRPO_BF16) ? kNegInfBf16x2 : kNegInfF32;
    u32x4 v = {w, w, w, w};
    return v;
}

template <grpo_dtype DT, int BLOCK>
__device__ __forceinline__ void zero_row(char *row, int nvec_full, int tail, int tid)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    const int s = (int)(((unsigned long long)row >> 4) & 7u);  // whole lines, as in row_shift
    if (tid >= s && tid - s < nvec_full) st16(row + (unsigned)(tid - s) * 16u, z);
    for (int v = BLOCK + tid - s; v < nvec_full; v += BLOCK) st16(row + (unsigned)v * 16u, z);
    if (tail && tid < tail) store_elem<DT>(row, (long long)nvec_full * Elem<DT>::EPV + tid, 0.f);
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every
// outstanding global load and store of the wavefront, which would drain the gradient
// stores of the previous row and the prefetch of the next one at each of the three
// barriers a row needs.  Nothing in the row kernels passes data between lanes through
// global memory, so LDS ordering is all the barrier has to provide.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- reductions: data-parallel-primitive (DPP) steps inside the 64-lane wavefront, LDS
// across waves, always in the same order, so results are bitwise reproducible ----
// A DPP step costs a few cycles; the same reduction through ds_bpermute took six round
// trips to LDS of about a hundred cycles each, in front of a workgroup barrier every time.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move(float identity, float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity),
                                                                   __builtin_bit_cast(int, v), CTRL, ROW_MASK,
                                                                   0xf, false));
}
// Quad swaps, mirror inside 8, mirror inside 16: every lane of a row of 16 holds the row's
// result; then lane 15 of a row is added into the next row (rows 1 and 3), lane 31 into
// rows 2 and 3, and lane 63, which has seen everything, is read out for all.
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_move<0xB1, 0xf>(v, v));
    v = fmaxf(v, dpp_move<0x4E, 0xf>(v, v));
    v = fmaxf(v, dpp_move<0x141, 0xf>(v, v));
    v = fmaxf(v, dpp_move<0x140, 0xf>(v, v));
    v = fmaxf(v, dpp_move<0x142, 0xa>(-INFINITY, v));
    v = fmaxf(v, dpp_move<0x143, 0xc>(-INFINITY, v));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_move<0xB1, 0xf>(0.f, v);
    v += dpp_move<0x4E, 0xf>(0.f, v);
    v += dpp_move<0x141, 0xf>(0.f, v);
    v += dpp_move<0x140, 0xf>(0.f, v);
    v += dpp_move<0x142, 0xa>(0.f, v);
    v += dpp_move<0x143, 0xc>(0.f, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_move(int identity, int v)
{
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_sum(int v)
{
    v += dpp_move<0xB1, 0xf>(0, v);
    v += dpp_move<0x4E, 0xf>(0, v);
    v += dpp_move<0x141, 0xf>(0, v);
    v += dpp_move<0x140, 0xf>(0, v);
    v += dpp_move<0x142, 0xa>(0, v);
    v += dpp_move<0x143, 0xc>(0, v);
    return __builtin_amdgcn_readlane(v, 63);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v)  // 0 where the row mask leaves a lane out
{
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)dpp_move<CTRL, ROW_MASK>(0, (int)b);
    const unsigned hi = (unsigned)dpp_move<CTRL, ROW_MASK>(0, (int)(b >> 32));
    return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum_dpp(double v)
{
    v += dpp_move<0xB1, 0xf>(v);
    v += dpp_move<0x4E, 0xf>(v);
    v += dpp_move<0x141, 0xf>(v);
    v += dpp_move<0x140, 0xf>(v);
    v += dpp_move<0x142, 0xa>(v);
    v += dpp_move<0x143, 0xc>(v);
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ long long wave_sum(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The caller guarantees a __syncthreads() between the reads of one call and the
// writes of the next call on the same LDS array (the other reduction sits between).
template <int BLOCK>
__device__ __forceinline__ float block_max(float v, float *lds)
{
    constexpr int NW = BLOCK / 64;
    v = wave_max(v);
    if constexpr (NW == 1) return v;
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    lds_barrier();
    float r = lds[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r = fmaxf(r, lds[i]);
    return r;
}
template <int BLOCK>
__device__ __forceinline__ float block_sum(float v, float *lds)
{
    constexpr int NW = BLOCK / 64;
    v = wave_sum(v);
    if constexpr (NW == 1) return v;
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    lds_barrier();
    float r = lds[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r += lds[i];
    return r;
}

// Exponents (log2 units) are kept above this floor where they are multiplied by their
// probability: an element at -inf has probability 0 and must contribute 0 to
// sum p log p, not 0 * inf = NaN.  The probability itself is taken from the exponent as it is:
// the floor (fmaxf) would turn a NaN into a probability of 0 and hide it.
constexpr float kExpFloor = -1.0e30f;

// Two sums behind one barrier.
template <int BLOCK>
__device__ __forceinline__ void block_sum2(float &a, float &b, float *lds_a, float *lds_b)
{
    constexpr int NW = BLOCK / 64;
    a = wave_sum(a);
    b = wave_sum(b);
    if constexpr (NW == 1) return;
    if ((threadIdx.x & 63) == 0) {
        lds_a[threadIdx.x >> 6] = a;
        lds_b[threadIdx.x >> 6] = b;
    }
    lds_barrier();
    a = lds_a[0];
    b = lds_b[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        a += lds_a[i];
        b += lds_b[i];
    }
}

// Reads what no kernel of this call writes while it runs, through the scalar cache where the address is uniform.  A vector
// load's wait is a wait for everything older in the memory queue too, the gradient stores of the row before among it.
template <typename T>
__device__ __forceinline__ T fixed_load(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(unsigned long long)p;
}
// A byte of an array of n: the four bytes around it where they are all inside the array.
__device__ __forceinline__ bool fixed_byte_set(const unsigned char *a, long long i, long long n)
{
    const unsigned long long at = (unsigned long long)(a + i), word = at & ~3ull;
    if (word >= (unsigned long long)a && word + 4 <= (unsigned long long)(a + n))
        return (fixed_load((const unsigned *)word) >> (8 * (unsigned)(at & 3))) & 0xffu;
    return a[i] != 0;
}

// Per-row scalars once the row statistics are known.
//   mk     = (max_j z_j) * k                      (k = log2 e / T)
//   s_excl = sum_{j != y} exp2(z_j k - mk)        (the sampled token is left out so that
//            1 - p_y = s_excl / s keeps its precision on near-one-hot rows, where
//            1 - p_y cancels to nothing in fp32)
// Produces l = log pi(y), the bracketed surrogate term J of section 3.4, its
// indicator bits, and c = grad_scale * dloss/dl.
struct RowScalars {
    float logp, J, c, shift, s, s_excl;
    int flags;
    // auxiliary terms: b = weight of -H in the gradient, q2 and bq the two constants of
    // the fused gradient g_j = p_j (q2 + bq a'_j), gy_ent the entropy part of g_y
    float b, q2, bq, gy_ent, mx, log2s;
};

// Scalar transcendental functions of the once-per-row arithmetic, built on the
// hardware's base-2 exponential and logarithm (1 ulp each).  The library versions are
// exact to the last bit but need dozens of registers at the one point of the kernel
// where the whole row is resident; the per-row quantities need 1e-6, not 1e-8.
__device__ __forceinline__ float hw_exp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
__device__ __forceinline__ float hw_log(float x) { return __builtin_amdgcn_logf(x) * kLn2; }
// ln(1 + x), x >= 0: the series below 1/32 (next term x^7/7 < 5e-12), else the logarithm
__device__ __forceinline__ float hw_log1p(float x)
{
    const float series = x * (1.f + x * (-0.5f + x * (1.f / 3 + x * (-0.25f + x * (0.2f - x * (1.f / 6))))));
    return x < 0.03125f ? series : hw_log(1.f + x);
}
// exp(d) - 1: the series below |d| = 0.1 (next term d^8/40320), else the exponential
__device__ __forceinline__ float hw_expm1(float d)
{
    const float series = d * (1.f + d * (0.5f + d * (1.f / 6 + d * (1.f / 24 + d * (1.f / 120 +
                         d * (1.f / 720 + d * (1.f / 5040)))))));
    return fabsf(d) < 0.1f ? series : hw_exp(d) - 1.f;
}

// J, dJ/dl and the indicator bits of the bracketed surrogate term of section 3.4.
__device__ __forceinline__ void surrogate(const RowParams &p, float r, float A, float &J, float &dJ,
                                          int &fl)
{
    // J = min( min(r, delta) A , clip(r, 1 - eps_low, 1 + eps_high) A )
    const float s1 = fminf(r, p.delta) * A;
    const float s2 = fminf(fmaxf(r, p.lo), p.hi) * A;
    const bool first = s1 <= s2;
    J = first ? s1 : s2;
    // dJ/dl = r dJ/dr; a ratio exactly on a boundary counts as not clipped
    const bool open = first ? (r <= p.delta) : (r >= p.lo && r <= p.hi);
    dJ = open ? A * r : 0.f;
    if (r != r || A != A) {  // fminf/fmaxf drop NaNs: put them back
        J = NAN;
        dJ = NAN;
    }
    fl = 0;
    if (A > 0.f && r > p.hi) fl |= kFlagClipHigh;
    if (A < 0.f && r < p.lo) fl |= kFlagClipLow;
    if (A < 0.f && r > p.delta) fl |= kFlagDelta;
    if (r < p.lo || r > p.hi) fl |= kFlagOutOfBand;
}

// inv_D: 1 / D as the header holds it, or a workgroup's own (not looked at without the gradient)
__device__ __forceinline__ RowScalars row_scalars(const RowParams &p, long long row, float zy,
                                                  float mk, float s_excl, const float *inv_D = nullptr)
{
    RowScalars o = {};
    const float ay = fmaf(zy, p.k, -mk);
    // A sum that is not finite has no logarithm: NaN, so that the row is poisoned whatever way
    // a +inf logit came in (with +inf as the row's maximum inf - inf has already made it NaN).
    const float s0 = s_excl + __builtin_amdgcn_exp2f(ay);
    const float s = s0 < INFINITY ? s0 : NAN;
    const float log2s = __builtin_amdgcn_logf(s);
    o.s = s;
    o.s_excl = s_excl;
    o.shift = mk + log2s;
    o.logp = (ay - log2s) * kLn2;
    if (!p.bwd) return o;

    float dJ;
    surrogate(p, hw_exp(o.logp - fixed_load(p.old_lp + row)), fixed_load(p.adv + row), o.J, dJ, o.flags);
    o.c = -(p.grad_scale * dJ) * (inv_D ? *inv_D : (float)fixed_load(&p.hdr->inv_D));
    return o;
}

// The same with the auxiliary terms (sampled-token KL estimator against a reference
// policy, entropy bonus).  w_excl = sum_{j != y} e_j a_j with a_j = z_j k - mk (log2
// units), a_j = (z_j - max) k here, and e_j = exp2(a_j).
//   H = ln s - ln2 * (sum_j e_j a_j) / s            entropy of softmax(z / T)
//   kl = exp(d) - d - 1, d = l_ref - l              dkl/dl = 1 - exp(d)
//   total gradient: g_j = (c/T)(1[j=y] - p_j) + (b/T) p_j (ln p_j + H)
// where ln p_j + H = ln2 (a_j - Abar), Abar = (sum e a)/s: the normaliser cancels, so
// the entropy part needs no difference of nearly equal numbers even when p_max -> 1.
__device__ __forceinline__ RowScalars row_scalars_aux(const RowParams &p, long long row, float zy,
                                                      float mx, float s_excl, float w_excl,
                                                      float &kl_out, float &H_out, const float *inv_D = nullptr)
{
    RowScalars o = {};
    const float ay = (zy - mx) * p.k;
    const float e_y = __builtin_amdgcn_exp2f(ay);
    const float s = s_excl + e_y;
    float ln_s;
    if (e_y > s_excl) {  // the sampled token dominates: ln(1 + x) form keeps l accurate
        const float t = hw_log1p(s_excl / e_y);
        ln_s = fmaf(ay, kLn2, t);
        o.logp = -t;
    } else {
        ln_s = hw_log(s);
        o.logp = fmaf(ay, kLn2, -ln_s);
    }
    const float log2s = ln_s * kLog2e;
    o.s = s;
    o.s_excl = s_excl;
    o.mx = mx;
    o.log2s = log2s;
    const float ay_f = fmaxf(ay, kExpFloor);
    const float abar = fmaf(e_y, ay_f, w_excl) / s;
    const float H = fmaf(-kLn2, abar, ln_s);

    float dJ;
    surrogate(p, hw_exp(o.logp - p.old_lp[row]), p.adv[row], o.J, dJ, o.flags);
    float kl = 0.f, dkl = 0.f;
    if (p.ref_lp) {
        const float d = p.ref_lp[row] - o.logp;
        const float em1 = hw_expm1(d);
        dkl = -em1;
        // exp(d) - d - 1: below |d| = 0.1 the difference cancels, the series does not
        const float series = d * d * (0.5f + d * (1.f / 6 + d * (1.f / 24 + d * (1.f / 120 +
                             d * (1.f / 720 + d * (1.f / 5040))))));
        kl = fabsf(d) < 0.1f ? series : em1 - d;
    }
    // omega_t / D: the weight of this row in all three sums
    const float wD = (p.token_w ? p.token_w[row] : 1.f) * (inv_D ? *inv_D : (float)p.hdr->inv_D);
    o.c = (p.grad_scale * (-dJ + p.kl_coef * dkl)) * wD;
    o.b = (p.grad_scale * p.ent_coef) * wD;
    o.bq = o.b * p.inv_T * kLn2;
    o.q2 = fmaf(o.bq, log2s - abar, -o.c * p.inv_T);
    o.gy_ent = o.bq * ((e_y / s) * (ay_f - abar));
    // A coefficient that is no finite number: p_j q2 is infinite, or NaN, and NaN where p_j is 0, which the product of
    // grad_vec_aux hides.  Against a maximum of -inf a logit of -inf is NaN and every other one +inf, and so are the
    // exponent, the probability and, with bq of the sign of q2, the product.
    if (!(fabsf(o.q2) < INFINITY)) {
        o.mx = -INFINITY;
        o.bq = copysignf(1.f, o.q2);
    }
    if (p.token_w) {  // the reductions sum omega_t J_t, omega_t kl_t, omega_t H_t
        const float w = p.token_w[row];
        o.J *= w;
        kl *= w;
    }
    kl_out = kl;
    H_out = H;
    return o;
}

// Overwrites element e of a resident vector with -inf.
template <grpo_dtype DT>
__device__ __forceinline__ void set_neg_inf(u32x4 &v, int e)
{
    if constexpr (DT == GRPO_BF16) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            if (d == (e >> 1))
                v[d] = (e & 1) ? ((v[d] & 0x0000ffffu) | 0xff800000u) : ((v[d] & 0xffff0000u) | 0x0000ff80u);
        }
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (d == e) v[d] = kNegInfF32;
    }
}

// max(a, b, c) as one v_max3_f32.  fmaxf() costs more than it looks: the compiler must first
// quiet a possible signalling NaN in every operand it knows nothing about (one v_max_f32 x, x, x
// each), which doubled the instructions of the maximum pass.  The instruction itself skips quiet
// NaNs like fmaxf and turns a signalling NaN into a quiet NaN result; both are fine here, a
// NaN logit poisons its row in the sum pass in any case.  The operands are never results of
// transcendental instructions (those need a wait state the compiler does not insert for
// inline assembly).
__device__ __forceinline__ float max3_f32(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The running maximum m joined with the elements of one vector: one v_max3_f32 per 32-bit word
// (two bf16, each widened exactly: the upper one by masking, the lower one by a shift), or per
// two fp32 values.  The maximum is exact, which the entropy gradient of a near-one-hot row needs
// (a difference a_max - Abar of order 1e-8 survives in fp32 only if a_max is exactly zero).
template <grpo_dtype DT>
__device__ __forceinline__ float vec_max_into(float m, const u32x4 &z)
{
    if constexpr (DT == GRPO_BF16) {
#pragma unroll
        for (int d = 0; d < 4; ++d) m = max3_f32(m, as_f32(z[d] & 0xffff0000u), as_f32(z[d] << 16));
    } else {
        m = max3_f32(m, as_f32(z[0]), as_f32(z[1]));
        m = max3_f32(m, as_f32(z[2]), as_f32(z[3]));
    }
    return m;
}

// sum_e exp2(z_e k - mk) over one vector.
template <grpo_dtype DT>
__device__ __forceinline__ float exp_sum_vec(const u32x4 &z, float k, float mk)
{
    constexpr int EPV = Elem<DT>::EPV;
    float f[EPV];
    unpack<DT>(z, f);
    float part = 0.f;
#pragma unroll
    for (int e = 0; e < EPV; ++e) part += __builtin_amdgcn_exp2f(fmaf(f[e], k, -mk));
    return part;
}

// Keeps the instruction scheduler from interleaving the work of different vectors of
// the unrolled row loops: with 76 registers per lane holding the row, there is room
// for the temporaries of one vector at a time, not of several.
#define VECTOR_FENCE() __builtin_amdgcn_sched_barrier(0)

// Makes the compiler forget what it knows about a resident vector.  Without this the
// bf16 -> fp32 widening done in one pass over the row is kept alive for the next pass
// (common-subexpression elimination), which turns 4 registers per vector into 12 and
// spills the row to scratch memory.  Emits no instruction.
__device__ __forceinline__ void forget(u32x4 &v) { asm volatile("" : "+v"(v)); }

// Inside a branch on a uniform condition: keeps it a branch.  The compiler would otherwise compute the few
// cheap instructions of either side for every row and select.  Emits no instruction.
__device__ __forceinline__ void keep_branch(float &x) { asm volatile("" : "+v"(x)); }

// One 32-bit word of a resident vector -> its elements (2 bf16 or 1 f32).
template <grpo_dtype DT>
__device__ __forceinline__ void unpack_word(unsigned w, float (&f)[Elem<DT>::EPV / 4])
{
    if constexpr (DT == GRPO_BF16) {
        f[0] = as_f32(w << 16);
        f[1] = as_f32(w & 0xffff0000u);
    } else {
        f[0] = as_f32(w);
    }
}

// The same, also accumulating sum_e e_e a_e (a = exponent in log2 units, floored so
// that an element at -inf contributes 0).  Word by word, with a scheduling fence between words: the auxiliary
// variants need more temporaries per element and the row leaves room for few.
template <grpo_dtype DT>
__device__ __forceinline__ float exp_sum_vec_aux(u32x4 &z, float k, float mx, float &w)
{
    constexpr int EPW = Elem<DT>::EPV / 4;
    float part = 0.f, partw = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        float f[EPW];
        forget(z);  // the widening of word d may not start before this point
        unpack_word<DT>(z[d], f);
#pragma unroll
        for (int e = 0; e < EPW; ++e) {
            // (z - max) k rather than fma(z, k, -max k): exactly 0 at the maximum, which the
            // entropy of a near-one-hot row needs (its sum e a is all cancellation otherwise)
            // (only the factor of the weighted sum is floored: fmaxf drops a NaN, which must reach the sum)
            const float a = (f[e] - mx) * k;
            const float ex = __builtin_amdgcn_exp2f(a);
            part += ex;
            partw = fmaf(ex, fmaxf(a, kExpFloor), partw);
        }
        // the running sums must exist here: left alone, the additions drift to the end
        // of the row pass and every product waits for them in a register of its own
        asm volatile("" : "+v"(part), "+v"(partw));
        VECTOR_FENCE();
    }
    w += partw;
    asm volatile("" : "+v"(w));
    return part;
}

// a b, but 0 wherever a or b is 0: what an element of probability 0 (a logit of -inf) contributes, whatever its logarithm.
// v_mul_legacy_f32 has no builtin.  a may come from the exponential, whose result must not be used by the very next instruction.
__device__ __forceinline__ float mul_zero(float a, float b)
{
    float r;
    asm("s_nop 0\n\tv_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Gradient of one vector with the entropy term fused in: g_j = p_j (q2 + bq a'_j),
// a'_j = (z_j - max) k - log2 s = log2 p_j.  Returns the packed vector; the sampled token's element is
// put in by the caller (put_elem), in one slot of one lane: selected at every element it cost one instruction in
// ten of the gradient pass (8192 x 128256 packed step 630 -> 618 us).  Word by word as above (two and four
// words between the fences, where the registers hold them: 630 and 641 us).  The exponent is not floored as in the
// sums: the product takes care of a probability of 0, one instruction of seven (8192 x 128256 bf16 634 -> 614 us, 4096 x 152064
// 383 -> 375).
template <grpo_dtype DT>
__device__ __forceinline__ u32x4 grad_vec_aux(u32x4 &z, float k, float mx, float log2s, float q2, float bq)
{
    constexpr int EPW = Elem<DT>::EPV / 4;
    u32x4 out;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        float f[EPW], g[EPW];
        forget(z);
        unpack_word<DT>(z[d], f);
#pragma unroll
        for (int e = 0; e < EPW; ++e) {
            const float a = fmaf(f[e] - mx, k, -log2s);
            g[e] = mul_zero(__builtin_amdgcn_exp2f(a), fmaf(bq, a, q2));
        }
        if constexpr (DT == GRPO_BF16) {
            f32x2 pr = {g[0], g[1]};
            out[d] = __builtin_bit_cast(unsigned, __builtin_convertvector(pr, bf16x2));
        } else {
            out[d] = as_u32(g[0]);
        }
        VECTOR_FENCE();
    }
    return out;
}

// Element e of a packed vector becomes x (rounded as the others are).
template <grpo_dtype DT>
__device__ __forceinline__ void put_elem(u32x4 &v, int e, float x)
{
    asm volatile("" : "+v"(x));  // keeps this behind a branch: it is for one lane of one slot
    if constexpr (DT == GRPO_BF16) {
        f32x2 pr = {x, x};
        const unsigned xx = __builtin_bit_cast(unsigned, __builtin_convertvector(pr, bf16x2));
        const unsigned keep = (e & 1) ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (d == (e >> 1)) v[d] = (v[d] & keep) | (xx & ~keep);
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (d == e) v[d] = as_u32(x);
    }
}

// Gradient of one vector: g_j = -(c/T) p_j with p_j = exp2(z_j k - shift), and at
// the sampled token g_y = (c/T) (1 - p_y) = (c/T) s_excl / s.
template <grpo_dtype DT>
__device__ __forceinline__ void grad_vec(const u32x4 &z, float k, float shift, float q, bool has_y,
                                         int ey, float gy, float (&g)[Elem<DT>::EPV])
{
    constexpr int EPV = Elem<DT>::EPV;
    float f[EPV];
    unpack<DT>(z, f);
#pragma unroll
    for (int i = 0; i < EPV; ++i) g[i] = __builtin_amdgcn_exp2f(fmaf(f[i], k, -shift)) * q;
    if (has_y) {
#pragma unroll
        for (int i = 0; i < EPV; ++i)
            if (i == ey) g[i] = gy;
    }
}

__device__ __forceinline__ void write_row_outputs(const RowParams &p, long long row, float logp,
                                                  float J, int flags)
{
    if (p.logprobs_out) p.logprobs_out[row] = logp;
    if (p.bwd) {
        p.J_ws[row] = J;
        p.flags_ws[row] = (unsigned char)flags;
    }
}
__device__ __forceinline__ void write_row_aux(const RowParams &p, long long row, float kl, float H)
{
    if (p.KL_ws) p.KL_ws[row] = kl;
    if (p.H_ws) p.H_ws[row] = p.token_w ? H * p.token_w[row] : H;
    if (p.entropy_out) p.entropy_out[row] = H;
}

// Decides whether a row takes part; handles the rows that do not (masked, or with a
// token id outside the vocabulary).  Returns true when the row must be processed.
// COUNT: the header's error word is not the rows' business (see grpo_rows_cached).
template <grpo_dtype DT, int BLOCK, bool COUNT = false, bool FIXED = false>
__device__ __forceinline__ bool row_is_live(const RowParams &p, long long row, int nvec_full,
                                            int tail, long long &y)
{
    bool live = p.mask ? (FIXED ? fixed_byte_set(p.mask, row, p.n_tokens) : p.mask[row] != 0) : true;
    if (live && p.token_w) live = p.token_w[row] != 0.f;
    bool bad = false;
    y = 0;
    if (live) {
        y = FIXED ? fixed_load(p.tokens + row) : p.tokens[row];
        if (y < 0 || y >= p.vocab) {
            live = false;
            bad = true;
        }
    }
    if (live) return true;
    if (threadIdx.x == 0) {
        // log-probs-only mode has no error word: a bad token id shows up as NaN
        write_row_outputs(p, row, (bad && !p.bwd) ? NAN : 0.f, 0.f, 0);
        write_row_aux(p, row, 0.f, 0.f);
        if (!COUNT && bad && p.bwd) atomicOr(&p.hdr->error, 1);
    }
    if (p.bwd)
        zero_row<DT, BLOCK>((char *)p.grad + row * p.row_stride * Elem<DT>::BYTES, nvec_full, tail,
                            threadIdx.x);
    return false;
}

// A value every lane holds alike, moved to scalar registers: what is derived from it
// (row base addresses, loop conditions) then stays scalar too.
__device__ __forceinline__ long long uniform(long long v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// Pins program order: whatever is computed from `off` afterwards (the address of the
// next row's load into a slot) cannot be moved above the point where `x` (the last
// value computed from the slot's current contents) exists.  Otherwise the compiler
// starts those loads early into fresh registers and the row no longer fits.  Emits no
// instruction.
template <typename X>
__device__ __forceinline__ void order_after(unsigned &off, X &x)
{
    asm volatile("" : "+v"(off), "+v"(x));
}


// One vector of an online softmax pass: running maximum m (in logit units), sum s of the
// exponentials relative to it and, for the entropy, w = sum e a with a the exponent in log2
// units.  The sampled token's element (has_y, ey) takes part in the maximum only.  As long as a lane
// has seen no maximum (all -inf, or NaN, which the maximum skips) its exponents are taken relative
// to 0: -inf adds nothing, NaN poisons s.
template <grpo_dtype DT, bool AUX>
__device__ __forceinline__ void online_vec(const u32x4 &z, bool has_y, int ey, float k, float &m, float &s,
                                           float &w)
{
    constexpr int EPV = Elem<DT>::EPV;
    float f[EPV];
    unpack<DT>(z, f);
    float vm = f[0];
#pragma unroll
    for (int e = 1; e + 1 < EPV; e += 2) vm = max3_f32(vm, f[e], f[e + 1]);
    vm = max3_f32(vm, f[EPV - 1], f[EPV - 1]);  // EPV is even: the last element is still to come
    if (vm > m) {
        // new reference: every exponent so far moves by dlt, every term by 2^dlt
        const float dlt = (m - vm) * k;  // -inf the first time: s and w are 0 (s: or NaN) and stay so
        const float sc_ = __builtin_amdgcn_exp2f(dlt);
        if constexpr (AUX) w = (s > 0.f) ? sc_ * fmaf(dlt, s, w) : 0.f;
        s *= sc_;
        m = vm;
    }
    const float ref = m > -INFINITY ? m : 0.f, mk_t = ref * k;
    float part = 0.f, partw = 0.f;
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        const float a = AUX ? (f[e] - ref) * k : fmaf(f[e], k, -mk_t);
        float ex = __builtin_amdgcn_exp2f(a);
        if (has_y && e == ey) ex = 0.f;
        part += ex;
        if constexpr (AUX) partw = fmaf(ex, fmaxf(a, kExpFloor), partw);
    }
    s += part;
    if constexpr (AUX) w += partw;
}

// The online partials (m, s, w) of one lane moved to the row's reference maximum mx.
template <bool AUX>
__device__ __forceinline__ void online_rescale(float m, float s, float w, float mx, float k, float &scaled,
                                               float &scaledw)
{
    const float dlt = (m - mx) * k;
    const float sc_ = __builtin_amdgcn_exp2f(dlt);
    scaled = (m > -INFINITY) ? s * sc_ : s;  // no maximum seen: s is 0, or NaN
    scaledw = (AUX && m > -INFINITY && s > 0.f) ? sc_ * fmaf(dlt, s, w) : 0.f;
}

// Workgroups that share a CU, by instantiation.
constexpr int row_blocks_per_cu(int block, int nv)
{
    // more than 19 slots: the instantiations with 256 registers per lane, 512 lanes per CU
    return block == 1024 ? 1 : nv > 19 ? 512 / block : block == 512 ? 2 : nv >= 16 ? 4 : 8;
}
// How many gradient slots of a row wait before they are stored (see the kernel).  In LDS: as
// many as an equal share of 144 KB of the CU's LDS holds for each workgroup on the CU (a slot
// is 16 bytes per lane), at most all of them.  In registers: only the instantiations with 256
// registers per lane; in the benchmark's (512 lanes x 38 slots, the row takes 152 registers)
// 16 slots is the most the compiler fits without spilling, the others state their number.
#ifndef GRPO_ROW_STASH_KB
#define GRPO_ROW_STASH_KB 144
#endif
#ifndef GRPO_ROW_RSTASH
#define GRPO_ROW_RSTASH 16
#endif
constexpr int row_reg_stash_slots(int block, int nv) { return nv > 19 ? GRPO_ROW_RSTASH : 0; }
// Rows wider than 44 slots of 512 lanes keep 50 slots in registers and up to 18 (8 KB each) in
// LDS, 544 KB together.
#ifndef GRPO_WIDE_NV
#define GRPO_WIDE_NV 50
#endif
#ifndef GRPO_WIDE_RST
#define GRPO_WIDE_RST 0
#endif
constexpr int kWideRegSlots = GRPO_WIDE_NV;
// 1: the lane's number is opaque at every use also where the row fits the registers (the per-slot
// in-range masks are then recomputed instead of kept in scalar registers and spilled to lanes)
#ifndef GRPO_OPAQUE_LANE
#define GRPO_OPAQUE_LANE 1
#endif
#ifndef GRPO_REM_NV
#define GRPO_REM_NV 48
#endif
constexpr int kRemRegSlots = GRPO_REM_NV;  // with a streamed remainder: its loop needs registers too
constexpr int row_stash_slots(int block, int nv, int nl = 0)
{
    const int fit = GRPO_ROW_STASH_KB * 1024 / row_blocks_per_cu(block, nv) / (block * 16) - nl;
    return fit < 0 ? 0 : fit < nv ? fit : nv;
}

// Position in the hand-out order -> row.  late: a masked row of which a workgroup with a live row in hand fills one only.
__device__ __forceinline__ long long row_of(int entry, bool &late)
{
    late = entry < 0;
    return late ? ~entry : entry;
}

// ---------------------------------------------------------------------------
// Register-resident row kernel: requires ceil(vocab / EPV) <= BLOCK * (NV + NL).
// One workgroup per row at a time, rows strided over a persistent grid.
// NL > 0: the row is wider than the registers hold and its last NL slots live in LDS, which
// the loads fill directly (buffer loads with LDS as their target).
// RST >= 0: the number of gradient slots that wait in registers, for the instantiations with
// 256 registers beside the benchmark's width; what LDS the row leaves free holds waiting slots too.
// (Skipping the empty slots of a narrower row with a branch per slot was tried instead of
// several widths: the wait counters are then reset to zero at every join and the gradient
// pass ran 1.5 times as long.)
// REM: the row may be wider still; what lies beyond slot NV + NL is streamed from memory, once
// for an online (max, sum) pass that is merged into the resident part's statistics and once
// more for the gradient: 2 reads + 1 write for that remainder only.
// SHIFT: gradient rows begin inside a 128-byte line (row_shift).  An instantiation of its own: on rows that begin with a
// line the conditions it adds per slot cost 1 to 2 % of a step and 5 to 8 % of a log-probs pass (4096 x 128256 bf16 297 -> 304
// us, 129 -> 139), where rows that do not gain 7 to 14 % (128264 apart 339 -> 305, 16384 x 32001 bf16 361 -> 322, 8192 x 50304
// at a pitch of 50312 267 -> 247, 32768 x 8001 204 -> 174).
// FEW: a batch of few rows, see few_rounds.
// COUNT: a small batch of narrow rows.  Every workgroup counts the rows that take part (up to four bytes a
// lane, on their way while the first row is looked up), and the first one writes the header, error word
// included, for grpo_finalize: no grpo_prepare in front, which is one of four launches of a step on 512 fp32 rows
// of 1024 (figures at kCountRows).
// ---------------------------------------------------------------------------
template <grpo_dtype DT, int BLOCK, int NV, bool AUX, bool TAIL, int NL = 0, int RST = -1, bool REM = false, bool COUNT = false, bool SHIFT = false, bool FEW = false>
// 4 wavefronts per SIMD and 128 registers each; the widest instantiations 2 and 256
__global__ void __launch_bounds__(BLOCK, NV > 19 ? 2 : 4) grpo_rows_cached(RowParams p)
{
    constexpr int EPV = Elem<DT>::EPV;
    constexpr int BYTES = Elem<DT>::BYTES;
    constexpr unsigned SLAB = BLOCK * 16u;  // bytes one pass of the workgroup covers
    static_assert(NL == 0 || !TAIL, "LDS-resident slots come without the ragged-tail slot");
    static_assert(!REM || !TAIL, "the streamed remainder comes without the ragged-tail slot");
    static_assert(!SHIFT || NL == 0, "rows are held further back in registers only");
    constexpr int RU = AUX ? 2 : 4;  // vectors per lane in flight in the remainder loops (what the registers leave)
    // Gradient vectors of the first STASH slots wait in LDS (each lane its own 16 bytes per
    // slot, no sharing), those of the next RSTASH slots in registers, and all of them are
    // stored after the loop over the slots, so that the next row's loads stand in front of
    // them in the memory queue.  Loads and stores retire in issue order: with a store in
    // front of every load the last load returns when everything is done, and the row
    // statistics that follow run with nothing in flight; with the stores behind the loads
    // they drain during that arithmetic (what a row whose gradient is zero gets for free: it
    // issues all loads, then all stores).
    constexpr int STASH = row_stash_slots(BLOCK, NV, NL);
    // further slots that wait in registers
    constexpr int RSTASH = RST < 0 ? row_reg_stash_slots(BLOCK, NV) : RST < NV - STASH ? RST : NV - STASH;
    static_assert(STASH + RSTASH <= NV, "more waiting slots than register slots");
    // The next row is asked for before the passes over this one; not where the registers are short (256 lanes of 26 and 32
    // slots: 8192 x 32000 fp32 step 304 us, 312 with it; the auxiliary terms -1 to +2 %), and not in batches of few rows.
    constexpr bool AHEAD = !FEW && !AUX && !REM && !(BLOCK == 256 && NV > 19);
    constexpr bool ORDERED = BLOCK * NV * 16ll >= kOrderMinRowBytes;  // serves rows that come in an order
    extern __shared__ __attribute__((aligned(16))) char row_stash[];
    char *const grad_stash = row_stash + (size_t)NL * SLAB;  // behind the LDS-resident part of the row
    __shared__ float lds_max[BLOCK / 64];
    __shared__ float lds_sum[BLOCK / 64];
    __shared__ float lds_sumw[BLOCK / 64];
    __shared__ float lds_turn[SHIFT && AUX ? 2 : 1][SHIFT ? BLOCK : 1];
    __shared__ long long lds_row[2];
    __shared__ int lds_count[COUNT ? BLOCK / 64 : 1], lds_bad[COUNT ? BLOCK / 64 : 1];
    __shared__ float lds_inv_D;
    const int tid = threadIdx.x;
    const unsigned toff = (unsigned)tid * 16u;
    int rows_on = 0, rows_bad = 0;  // COUNT: this lane's share of the rows that take part, and of those with a bad token id
    if constexpr (COUNT) {
#pragma unroll 4
        for (int i = tid; i < (int)p.n_tokens; i += BLOCK) {
            const bool on = (!p.mask || p.mask[i] != 0) && (!p.token_w || p.token_w[i] != 0.f);
            rows_on += on ? 1 : 0;
            if (blockIdx.x == 0 && on && (p.tokens[i] < 0 || p.tokens[i] >= p.vocab)) rows_bad = 1;
        }
    }
    const int nvec_full = (int)(p.vocab / EPV);
    const int tail = (int)(p.vocab % EPV);
    // The ragged last vector (vocab not a multiple of EPV): lane i < tail holds its entry i, one
    // register (tz; the other lanes' are -inf) and one exponential more per pass, against the four of
    // a slot of its own.  Rows without a ragged end never enter those branches.
    const bool ragged = TAIL && tail != 0;

    // ---- which row next ----
    // With a workspace (objective + gradient) rows are handed out through a counter in
    // it, one at a time, to whichever workgroup is free: masked rows cost a third of a
    // live row, and a fixed assignment leaves some workgroups with all the live ones.
    // Without a workspace (log-probs only), and in small batches (launch_cached), rows are
    // strided over the grid, the workgroups turned by 5/8 of the grid from round to round: response lengths
    // that divide the grid would otherwise give one workgroup the same, masked, position of every
    // response (log-probs of 3000 bf16 rows of 262144, responses of up to 256: 257 us, turned 206).  Not turned
    // are batches of any length, i.e. without a workspace, where several workgroups share a CU: those with
    // live rows take over what the others leave, and turning only costs (65536 fp32 rows of 1024, responses of
    // up to 1024: 92 us turned, 73 not; 16384 bf16 rows of 4000 37 and 32).
    const bool queued = p.queued != 0;
    constexpr bool ALONE = row_blocks_per_cu(BLOCK, NV) == 1;
    const unsigned turn_step = p.hdr ? gridDim.x / 8 * 5 : 0;
    long long strided_base = 0;
    unsigned turn = blockIdx.x, grabs = 0;
    // very narrow rows are also handed out several at a time
    long long chunk = p.queue_chunk;
    long long chunk_next = 0, chunk_end = 0;  // positions inside the current partition
    // consecutive workgroups sit on different XCDs; dividing by 8 first spreads every
    // partition over all XCDs (tying a partition to one XCD measured 4 % slower)
    const int nparts = p.queue_parts;
    int part = (int)((blockIdx.x / 8) % nparts), parts_done = 0;
    // The counter is asked before the passes over a row (ask) and its answer shared with one of their barriers (tell).  Asked
    // when it was needed, counter, mask, order and token were four loads in a chain between two rows, and each wait was for
    // everything in flight (the next three now go through the scalar cache).  Log-probs of 8192 x 128256 bf16
    // 251 -> 238 us, of 4096 x 50304 fp32 98 -> 94; steps on rows of several workgroups to a CU 340 -> 308 (30000 x 16384 bf16)
    // and 333 -> 322 (16384 x 32000), on wider ones, which HBM bounds, as before.
    bool asked = false;
    unsigned long long answer = 0;
    auto ask = [&]() __attribute__((always_inline)) {
        asked = AHEAD && queued && chunk_next >= chunk_end && parts_done < nparts;
        if (!AUX && !REM && !p.bwd) chunk = chunk_end < p.more_until ? p.queue_more : p.queue_chunk;
        if (asked && tid == 0) answer = atomicAdd(queue_counters(p.hdr) + part * kQueueStride, (unsigned long long)chunk);
    };
    auto tell = [&]() __attribute__((always_inline)) {
        if (asked && tid == 0) lds_row[grabs & 1u] = (long long)answer;
    };
    auto grab = [&]() -> long long {
        if (!queued) {
            const long long r = strided_base + turn;
            strided_base += gridDim.x;
            turn += ALONE ? gridDim.x / 8 * 5 : turn_step;
            if (turn >= gridDim.x) turn -= gridDim.x;
            return r;  // only the last round has positions past the batch: they end the workgroup's work
        }
        for (;;) {
            if (chunk_next < chunk_end) {
                const long long r = part + (long long)nparts * chunk_next++;
                if (r < p.n_tokens) return r;
                chunk_next = chunk_end;  // ran off the end of this partition
            }
            if (parts_done == nparts) return p.n_tokens;
            // two LDS slots used alternately: the barrier of grab k+1 separates the reads
            // of grab k from the write of grab k+2 into the same slot
            const unsigned slot = grabs++ & 1u;
            if (!asked) {
                if (!AUX && !REM && !p.bwd) chunk = chunk_end < p.more_until ? p.queue_more : p.queue_chunk;
                if (tid == 0)
                    lds_row[slot] = (long long)atomicAdd(queue_counters(p.hdr) + part * kQueueStride,
                                                         (unsigned long long)chunk);
                lds_barrier();
            }
            asked = false;
            const long long base = uniform(lds_row[slot]);
            if (part + (long long)nparts * base >= p.n_tokens) {
                part = (part + 1) % nparts;  // this partition is exhausted: help with the next
                ++parts_done;
                continue;
            }
            chunk_next = base;
            chunk_end = base + chunk;
        }
    };
    // next row that needs the full treatment; rows that do not (masked, bad token id) are finished on the way.  With a live row
    // in hand (`holding`) and live rows handed out first, of masked rows that are marked as late only one is: LateRule.
    bool rows_left = false;
    auto acquire = [&](long long &y, bool holding) -> long long {
        for (;;) {
            long long r = grab();
            if (r >= p.n_tokens) return p.n_tokens;
            bool late = false;
            if (p.order) r = row_of(uniform(AHEAD ? fixed_load(p.order + r) : p.order[r]), late);
            if (row_is_live<DT, BLOCK, COUNT, AHEAD>(p, r, nvec_full, tail, y)) return r;
            if (ORDERED && !REM && holding && late) {
                rows_left = true;
                return p.n_tokens;
            }
        }
    };

    // slot i of lane tid holds vector i * BLOCK + tid of the resident row: consecutive
    // lanes hold consecutive 16-byte pieces; slots past the end of the row stay -inf
    u32x4 buf[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) buf[i] = neg_inf_vec<DT>();
    float zy = 0.f, tz = -INFINITY;
    // The streamed remainder of the next row, up to 128 KB of it, is brought into L2 with the row's other
    // loads, one lane to a 128-byte line; its two reads, each a few loads at a time behind everything that is
    // in flight, then come from there (2048 x 152064 fp32 step, 67 KB of remainder a row: 397 -> 378 us).
    constexpr int REM_PF = REM ? 2 : 1;
    unsigned pf[REM_PF] = {};

    // The lane's number and byte offset as the slot loops use them.  In the instantiations with
    // LDS-resident slots they are made opaque at every use: otherwise the compiler keeps the
    // vector number, the store offset and the in-range mask of each of the 60 to 68 slots in
    // registers of their own across the whole row loop, and the row spills.
    auto lane = [&]() __attribute__((always_inline)) {
        int t = tid;
        if constexpr (NL > 0 || GRPO_OPAQUE_LANE) asm volatile("" : "+v"(t));
        return t;
    };
    unsigned noff = toff;  // byte offset of this lane inside a slab, as used by the refills
    auto lane_off = [&]() __attribute__((always_inline)) {
        unsigned o = SHIFT ? noff : toff;  // (held apart they would cost the row a register)
        if constexpr (NL > 0 || GRPO_OPAQUE_LANE) asm volatile("" : "+v"(o));
        return o;
    };
    // A row that begins s vectors into a line of its gradient is held s vectors further back (row_shift): vector v of the
    // row sits at position v + s, position q in slot q / BLOCK of lane q % BLOCK.  Slot addresses are relative to
    // position 0 (rows' addresses less 16 s); the first s lanes have nothing in slot 0.
    auto shift_of = [&](long long r) __attribute__((always_inline)) -> int { return SHIFT ? (int)row_shift(p, r) : 0; };
    auto fetch_slot = [&](const char *zpos, int i, int s) __attribute__((always_inline)) {
        if (i * BLOCK + lane() < nvec_full + s && (!SHIFT || i > 0 || lane() >= s)) buf[i] = ld16(zpos + (size_t)i * SLAB + noff);
    };
    // LDS-resident slot j (slot NV + j of the row): lane tid owns the 16 bytes at j * SLAB + toff,
    // which is also where the load puts them (wavefront base in M0, 16 bytes per lane).  Lanes
    // past the end of the row load nothing and read their piece as -inf.
    const int wave_lds = __builtin_amdgcn_readfirstlane(tid >> 6) * 1024;
    auto fetch_lds_slot = [&](const char *zrow, int j) __attribute__((always_inline)) {
        if constexpr (NL > 0) {
            if ((NV + j) * BLOCK + lane() < nvec_full) {
                const __amdgpu_buffer_rsrc_t rsrc =
                    __builtin_amdgcn_make_buffer_rsrc((void *)zrow, 0, -1, 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rsrc, (__attribute__((address_space(3))) void *)(row_stash + (size_t)j * SLAB + wave_lds), 16,
                    (int)((unsigned)(NV + j) * SLAB + noff), 0, 0, GRPO_NT_LOAD ? 2 : 0);
            }
        }
    };
    auto lds_slot = [&](int j, int vy_, int ey_) __attribute__((always_inline)) -> u32x4 {
        // each pass reads the slot anew: with an address the compiler can recognise it keeps the
        // first pass's values of all slots in registers for the later passes, and the row spills
        unsigned off = toff;
        asm volatile("" : "+v"(off));
        u32x4 z = *(const u32x4 *)(row_stash + (size_t)j * SLAB + off);
        const int v = (NV + j) * BLOCK + lane();
        if (v >= nvec_full) z = neg_inf_vec<DT>();
        if (v == vy_) set_neg_inf<DT>(z, ey_);  // the sampled token's logit stays out of the sums
        return z;
    };
    // Every load has landed (they retire in order, those bound for LDS last).  Also in front of the loads of a whole row: nothing,
    // or nothing but stores that have had two passes' time, is in flight there, but the compiler reckons with what an earlier row
    // may have asked for, in a register that it takes for an address, and then waits for everything in front of every slot's
    // load.  Log-probs of 120 fp32 rows of 78144 25.8 us, 13.6 with this; steps on 700 fp32 rows of 50304, a third of them
    // masked and many clipped, 68 and 56.
    auto nothing_in_flight = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
    };
    // (always inlined: as a function of its own it would take the row out of the registers)
    auto fetch_all = [&](const char *zpos, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NV; ++i) fetch_slot(zpos, i, s);
#pragma unroll
        for (int j = 0; j < NL; ++j) fetch_lds_slot(zpos, j);
    };
    auto fetch_rest = [&](const char *zrow, long long y) {
        if (ragged && tid < tail) tz = load_elem<DT>(zrow, (long long)nvec_full * EPV + tid);
        zy = load_elem<DT>(zrow, y);
        if constexpr (REM) {
#pragma unroll
            for (int i = 0; i < REM_PF; ++i) {
                const unsigned off = (unsigned)(NV + NL) * SLAB + (unsigned)(i * BLOCK + tid) * 128u;
                pf[i] = off < (unsigned)nvec_full * 16u ? *(const unsigned *)(zrow + off) : 0u;
            }
        }
    };

    long long y = 0, y_next = 0, row;
    int sh;
rows_from_none:
    row = acquire(y, false);
    sh = shift_of(row);
    if (row < p.n_tokens) {
        const char *zrow = (const char *)p.logits + row * p.row_stride * BYTES;
        nothing_in_flight();
        fetch_all(zrow - sh * 16, sh);
        fetch_rest(zrow, y);
    }
    if constexpr (COUNT) {
        rows_on = wave_sum(rows_on);
        rows_bad = __any(rows_bad) ? 1 : 0;
        if ((tid & 63) == 0) {
            lds_count[tid >> 6] = rows_on;
            lds_bad[tid >> 6] = rows_bad;
        }
        lds_barrier();
        if (tid == 0) {
            long long M = 0;
            int bad = 0;
#pragma unroll
            for (int w = 0; w < BLOCK / 64; ++w) M += lds_count[w], bad |= lds_bad[w];
            const double D = p.denom > 0.0 ? p.denom : (double)M, inv_D = D > 0.0 ? 1.0 / D : 0.0;
            lds_inv_D = (float)inv_D;  // read behind the barriers of a row's reductions
            if (blockIdx.x == 0) {
                p.hdr->D = D;
                p.hdr->inv_D = inv_D;
                p.hdr->M = M;
                p.hdr->error = bad;
                p.hdr->fin_ticket = 0u;
            }
        }
    }

    while (row < p.n_tokens) {
        // Take the following row: its loads are issued while this row's last pass
        // still computes, into the registers that pass has just finished with.
        long long next;
        bool has_next;
        const char *zrow_next, *zpos_next;
        int sh_next;
        auto take_next = [&]() __attribute__((always_inline)) {
            next = acquire(y_next, true);
            has_next = next < p.n_tokens;
            zrow_next = (const char *)p.logits + (has_next ? next : row) * p.row_stride * BYTES;
            sh_next = shift_of(next);
            zpos_next = zrow_next - sh_next * 16;
        };
        if constexpr (AHEAD)
            ask();
        else
            take_next();
        const int vy = (int)(y / EPV) + sh;  // the sampled token's position
        const int ey = (int)(y % EPV);
        const int npos = nvec_full + sh;
        if constexpr (SHIFT) {
            // Where this row has nothing, the one before it may have had something: in front of its first vector and up to
            // the last position any row has.
            if (tid < sh) buf[0] = neg_inf_vec<DT>();
            const int q = npos + ((tid - npos) & (BLOCK - 1));  // this lane's first position behind the row
            if (q < nvec_full + 7) {
#pragma unroll
                for (int i = 0; i < NV; ++i)
                    if (i == q / BLOCK) buf[i] = neg_inf_vec<DT>();
            }
        }
        // The sampled token's logit is taken out of the resident row (replaced by -inf):
        // the sum below is then s_excl = sum_{j != y}, which keeps 1 - p_y = s_excl / s
        // accurate on near-one-hot rows where it would cancel to 0 in fp32.  One lane
        // of one wavefront does this once per row.
        if (tid == (vy & (BLOCK - 1)) && vy < npos) {
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (i == vy / BLOCK) set_neg_inf<DT>(buf[i], ey);
        }
        if (ragged) {
            keep_branch(tz);
            if (vy == npos && tid == ey) tz = -INFINITY;
        }

        // reference maximum over j != y, then joined with z_y
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            forget(buf[i]);
            mx = vec_max_into<DT>(mx, buf[i]);
            VECTOR_FENCE();
        }
        if constexpr (NL > 0) {
            nothing_in_flight();
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                    const u32x4 z = lds_slot(j, vy, ey);
                mx = vec_max_into<DT>(mx, z);
                asm volatile("" : "+v"(mx));  // done with this slot before the next one is read
                VECTOR_FENCE();
            }
        }
        if (ragged) {
            keep_branch(tz);
            mx = fmaxf(mx, tz);
        }
        // the part of the row that is not resident: online statistics, first read (kept in the caches)
        const char *zrow_cur = (const char *)p.logits + row * p.row_stride * BYTES;
        float rem_m = -INFINITY, rem_s = 0.f, rem_w = 0.f;
        if constexpr (REM) {
#pragma unroll
            for (int i = 0; i < REM_PF; ++i) asm volatile("" ::"v"(pf[i]));  // landed with the row; its value is not needed
            for (int base = (NV + NL) * BLOCK; base < nvec_full; base += RU * BLOCK) {
                u32x4 z[RU];
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    const int v = base + u * BLOCK + tid;
                    z[u] = neg_inf_vec<DT>();
                    if (v < nvec_full) z[u] = *(const u32x4 *)(zrow_cur + (size_t)v * 16);
                }
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    online_vec<DT, AUX>(z[u], base + u * BLOCK + tid == vy, ey, p.k, rem_m, rem_s, rem_w);
                    VECTOR_FENCE();
                }
            }
            mx = fmaxf(mx, rem_m);
        }
        if constexpr (AHEAD) tell();
        mx = fmaxf(block_max<BLOCK>(mx, lds_max), zy);
        const float mk = mx * p.k;

        if constexpr (AHEAD) take_next();

        // sum of exponentials over j != y; in log-probs-only mode this is the last use
        // of the row, so the next row is fetched slot by slot behind it
        float acc = 0.f, accw = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            forget(buf[i]);
            if constexpr (AUX)
                acc += exp_sum_vec_aux<DT>(buf[i], p.k, mx, accw);
            else
                acc += exp_sum_vec<DT>(buf[i], p.k, mk);
            if (!p.bwd && has_next) {
                order_after(noff, acc);
                fetch_slot(zpos_next, i, sh_next);
            }
            VECTOR_FENCE();
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            u32x4 z = lds_slot(j, vy, ey);
            if constexpr (AUX)
                acc += exp_sum_vec_aux<DT>(z, p.k, mx, accw);
            else
                acc += exp_sum_vec<DT>(z, p.k, mk);
            asm volatile("" : "+v"(acc));  // done with this slot before the next one is read
            if (!p.bwd && has_next) {
                order_after(noff, acc);  // the slot has been read: its refill may start
                fetch_lds_slot(zpos_next, j);
            }
            VECTOR_FENCE();
        }
        if (SHIFT && sh != 0) {  // the lanes' sums to the lanes that have them for a row that begins with a line: the same order of summation
            const int at = (tid - sh) & (BLOCK - 1);
            lds_turn[0][SHIFT ? at : 0] = acc;
            if constexpr (AUX) lds_turn[SHIFT ? 1 : 0][SHIFT ? at : 0] = accw;
            lds_barrier();
            acc = lds_turn[0][SHIFT ? tid : 0];
            if constexpr (AUX) accw = lds_turn[SHIFT ? 1 : 0][SHIFT ? tid : 0];
        }
        if (ragged) {
            keep_branch(tz);
            const float a = AUX ? (tz - mx) * p.k : fmaf(tz, p.k, -mk);
            const float ex = __builtin_amdgcn_exp2f(a);
            if (tid < tail) {  // (the other lanes' -inf is no number against a maximum of -inf)
                acc += ex;
                if constexpr (AUX) accw = fmaf(ex, fmaxf(a, kExpFloor), accw);
            }
        }
        if constexpr (REM) {
            float scaled, scaledw;
            online_rescale<AUX>(rem_m, rem_s, rem_w, mx, p.k, scaled, scaledw);
            acc += scaled;
            accw += scaledw;
        }
        const float zy_row = zy;
        if (!p.bwd && has_next) fetch_rest(zrow_next, y_next);
        RowScalars sc;
        if constexpr (AUX) {
            block_sum2<BLOCK>(acc, accw, lds_sum, lds_sumw);
            float kl, H;
            sc = row_scalars_aux(p, row, zy_row, mx, acc, accw, kl, H, COUNT ? &lds_inv_D : nullptr);
            if (tid == 0) write_row_aux(p, row, kl, H);
        } else {
            const float s_excl = block_sum<BLOCK>(acc, lds_sum);
            sc = row_scalars(p, row, zy_row, mk, s_excl, COUNT ? &lds_inv_D : nullptr);
        }
        if (tid == 0) write_row_outputs(p, row, sc.logp, sc.J, sc.flags);

        if (p.bwd) {
            char *grow = (char *)p.grad + row * p.row_stride * BYTES;
            if (sc.c == 0.f && (!AUX || sc.b == 0.f)) {
                // the gradient of this row is cut: fetch the next row, then zero-fill
                if (has_next) {
                    nothing_in_flight();
                    fetch_all(zpos_next, sh_next);
                    fetch_rest(zrow_next, y_next);
                }
                zero_row<DT, BLOCK>(grow, nvec_full, tail, tid);
            } else {
                const float q = -sc.c * p.inv_T;
                const float gy = (sc.c * p.inv_T) * (sc.s_excl / sc.s) + (AUX ? sc.gy_ent : 0.f);
                if constexpr (REM) {
                    // second read of the remainder, before the resident slots: behind their
                    // refills these loads would wait for the whole next row
                    for (int base = (NV + NL) * BLOCK; base < nvec_full; base += RU * BLOCK) {
                        u32x4 z[RU];
#pragma unroll
                        for (int u = 0; u < RU; ++u) {
                            const int v = base + u * BLOCK + tid;
                            z[u] = neg_inf_vec<DT>();
                            if (v < nvec_full) z[u] = ld16(zrow_cur + (size_t)v * 16);
                        }
#pragma unroll
                        for (int u = 0; u < RU; ++u) {
                            const int v = base + u * BLOCK + tid;
                            u32x4 packed;
                            if constexpr (AUX) {
                                packed = grad_vec_aux<DT>(z[u], p.k, sc.mx, sc.log2s, sc.q2, sc.bq);
                                if (v == vy) put_elem<DT>(packed, ey, gy);
                            } else {
                                float g[EPV];
                                grad_vec<DT>(z[u], p.k, sc.shift, q, v == vy, ey, gy, g);
                                packed = pack<DT>(g);
                            }
                            if (v < nvec_full) st16(grow + (size_t)v * 16, packed);
                            VECTOR_FENCE();
                        }
                    }
                }
                char *const gpos = grow - sh * 16;
                u32x4 rstash[RSTASH > 0 ? RSTASH : 1];
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                            const int v = i * BLOCK + lane();
                    forget(buf[i]);
                    u32x4 packed;
                    if constexpr (AUX) {
                        packed = grad_vec_aux<DT>(buf[i], p.k, sc.mx, sc.log2s, sc.q2, sc.bq);
                        if (i == vy / BLOCK && v == vy) put_elem<DT>(packed, ey, gy);
                    } else {
                        float g[EPV];
                        grad_vec<DT>(buf[i], p.k, sc.shift, q, v == vy, ey, gy, g);
                        packed = pack<DT>(g);
                    }
                    order_after(noff, packed);
                    // the slot's gradient waits (LDS, then registers) or, for the last slots, is
                    // stored at once, but in every case behind the next row's load into the slot
                    if (i < STASH) *(u32x4 *)(grad_stash + (size_t)i * SLAB + lane_off()) = packed;
                    if (has_next) fetch_slot(zpos_next, i, sh_next);
                    if (i >= STASH && i < STASH + RSTASH) rstash[i - STASH < 0 ? 0 : i - STASH] = packed;
                    if (i >= STASH + RSTASH && v < npos && (!SHIFT || i > 0 || lane() >= sh)) st16(gpos + (size_t)i * SLAB + lane_off(), packed);
                    VECTOR_FENCE();
                }
#pragma unroll
                for (int j = 0; j < NL; ++j) {
                            const int v = (NV + j) * BLOCK + lane();
                    u32x4 z = lds_slot(j, -1, 0);
                    u32x4 packed;
                    if constexpr (AUX) {
                        packed = grad_vec_aux<DT>(z, p.k, sc.mx, sc.log2s, sc.q2, sc.bq);
                        if (NV + j == vy / BLOCK && v == vy) put_elem<DT>(packed, ey, gy);
                    } else {
                        float g[EPV];
                        grad_vec<DT>(z, p.k, sc.shift, q, v == vy, ey, gy, g);
                        packed = pack<DT>(g);
                    }
                    order_after(noff, packed);  // the slot has been read: its refill may start
                    if (has_next) fetch_lds_slot(zpos_next, j);
                    if (v < npos) st16(gpos + (size_t)(NV + j) * SLAB + lane_off(), packed);
                    VECTOR_FENCE();
                }
                if (ragged && tid < tail) {
                    keep_branch(tz);
                    float g;
                    if constexpr (AUX) {
                        const float a = fmaxf(fmaf(tz - sc.mx, p.k, -sc.log2s), kExpFloor);
                        g = __builtin_amdgcn_exp2f(a) * fmaf(sc.bq, a, sc.q2);
                    } else {
                        g = __builtin_amdgcn_exp2f(fmaf(tz, p.k, -sc.shift)) * q;
                    }
                    if (vy == npos && tid == ey) g = gy;
                    store_elem<DT>(grow, (long long)nvec_full * EPV + tid, g);
                }
                if (has_next) fetch_rest(zrow_next, y_next);
#pragma unroll
                for (int i = 0; i < STASH; ++i) {
                    const u32x4 packed = *(const u32x4 *)(grad_stash + (size_t)i * SLAB + lane_off());
                    if (i * BLOCK + lane() < npos && (!SHIFT || i > 0 || lane() >= sh)) st16(gpos + (size_t)i * SLAB + lane_off(), packed);
                }
#pragma unroll
                for (int i = STASH; i < STASH + RSTASH; ++i)
                    if (i * BLOCK + lane() < npos && (!SHIFT || i > 0 || lane() >= sh)) st16(gpos + (size_t)i * SLAB + lane_off(), rstash[i - STASH]);
            }
        }
        row = next;
        y = y_next;
        sh = sh_next;
    }
    if (rows_left) {
        rows_left = false;
        goto rows_from_none;
    }
}

// One batch of vectors joined into a lane's online statistics: running maximum m (in logit units),
// sum s of the exponentials relative to it, and for the entropy w = sum e a.  One comparison with
// the running maximum for the whole batch; a lane without a maximum as in online_vec.
template <grpo_dtype DT, bool AUX, int U>
__device__ __forceinline__ void online_batch(u32x4 (&z)[U], float k, float &m, float &s, float &w)
{
    constexpr int EPW = Elem<DT>::EPV / 4;
    float vm = m;
#pragma unroll
    for (int u = 0; u < U; ++u) vm = vec_max_into<DT>(vm, z[u]);
    if (vm > m) {
        // new reference: every exponent so far moves by dlt, every term by 2^dlt
        const float dlt = (m - vm) * k;  // -inf the first time: s and w are 0 (s: or NaN) and stay so
        const float sc_ = __builtin_amdgcn_exp2f(dlt);
        if constexpr (AUX) w = (s > 0.f) ? sc_ * fmaf(dlt, s, w) : 0.f;
        s *= sc_;
        m = vm;
    }
    const float ref = m > -INFINITY ? m : 0.f, mk_t = ref * k;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        forget(z[u]);  // see the register-resident kernel: the widening is done anew
        float part = 0.f, partw = 0.f;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            float f[EPW];
            unpack_word<DT>(z[u][d], f);
#pragma unroll
            for (int e = 0; e < EPW; ++e) {
                const float a = AUX ? (f[e] - ref) * k : fmaf(f[e], k, -mk_t);
                const float ex = __builtin_amdgcn_exp2f(a);
                part += ex;
                if constexpr (AUX) partw = fmaf(ex, fmaxf(a, kExpFloor), partw);
            }
        }
        s += part;
        if constexpr (AUX) w += partw;
        VECTOR_FENCE();
    }
}

// ---------------------------------------------------------------------------
// Streaming row kernel for rows the register-resident kernel cannot hold: an online (max, sum)
// pass and a gradient pass, each reading the row.
//
// Bound: HBM, if enough loads are in flight and the second read does not go there.  Two workgroups
// of 512 lanes share a CU.  A lane works in batches of four vectors through two register buffers, even
// batches in A, odd ones in B: while one is reduced the other's loads are in flight, up to 128 KB
// per CU.  The gradient pass walks the batches backwards: the last two are still in the buffers and
// are not read again, the ones before them are the most recent in the caches, and the buffers it
// frees last take the first two batches of the next row.  The loads are ordinary ones: 512 rows of
// 300 KB in flight fit the memory-side cache, non-temporal reads pass it by (312 us instead of 270,
// 519 instead of 466 on the two batches below).  Loads stand in front of the stores of the same step.
// Rows come from the queue, live ones first, like the resident kernel's.
// Whole step in turn on one card, against one vector in flight per lane and rows strided over the grid (which
// gave some workgroups the live head of every response and others its masked tail): 2048 x 100003 fp32
// 317 -> 270 us, 4096 x 152069 bf16 550 -> 466 us.  Batches of five and six: 270 and 286, 473 and 486.
// Rows whose gradient begins inside a line are stored in whole lines by lanes turned by that much (4096 x 152069 bf16 step
// 462 -> 412 us, what it takes at a pitch of whole lines; 2048 x 100003 fp32 333 -> 301).  Two more batches of a row
// held in LDS between the passes saved 1 %: the second reads are served by the caches.
// ---------------------------------------------------------------------------
constexpr int kStreamBlock = 512, kStreamPerCu = 2, kStreamBatch = 4;
template <grpo_dtype DT, bool AUX, bool SHIFT>
__global__ void __launch_bounds__(kStreamBlock, 4) grpo_rows_streamed(RowParams p)
{
    constexpr int EPV = Elem<DT>::EPV, BYTES = Elem<DT>::BYTES, BLOCK = kStreamBlock, U = kStreamBatch;
    constexpr unsigned SLAB = BLOCK * 16u;  // bytes one slot of the workgroup covers
    __shared__ float lds_max[BLOCK / 64];
    __shared__ float lds_sum[BLOCK / 64];
    __shared__ float lds_sumw[BLOCK / 64];
    __shared__ float lds_turn[SHIFT && AUX ? 2 : 1][SHIFT ? BLOCK : 1];
    __shared__ long long lds_row[2];
    const int tid = threadIdx.x;
    const int nvec_full = (int)(p.vocab / EPV);
    const int tail = (int)(p.vocab % EPV);
    const int nb = (nvec_full + U * BLOCK - 1) / (U * BLOCK);  // batches; at least 2 (the plan's widths)
    const bool queued = p.queued != 0;
    long long strided_next = blockIdx.x;
    unsigned grabs = 0;
    bool rows_left = false;  // as in the resident kernel
    auto acquire = [&](long long &y, bool holding) -> long long {
        for (;;) {
            long long r;
            if (queued) {
                const unsigned slot = grabs++ & 1u;  // alternating, as in the resident kernel
                if (tid == 0) lds_row[slot] = (long long)atomicAdd(queue_counters(p.hdr), 1ull);
                lds_barrier();
                r = uniform(lds_row[slot]);
            } else {
                r = strided_next;
                strided_next += gridDim.x;
            }
            if (r >= p.n_tokens) return p.n_tokens;
            bool late = false;
            if (p.order) r = row_of(uniform(p.order[r]), late);
            if (row_is_live<DT, BLOCK>(p, r, nvec_full, tail, y)) return r;
            if (holding && late) {
                rows_left = true;
                return p.n_tokens;
            }
        }
    };
    u32x4 A[U], B[U];
    float zy = 0.f, tz = -INFINITY;  // the sampled token's logit; lane i < tail: entry i of the ragged last vector
    // Lanes are turned by as many vectors as the row's gradient begins inside a line (row_shift): lane t has the vectors
    // (t - s) mod BLOCK of every slot, so that a wavefront's stores are whole lines but for the one at a slot's border.  The
    // lane's byte offset in a slot is opaque at every use (see the resident kernel: kept for every
    // slot of every batch it would fill the registers).
    unsigned noff = (unsigned)tid * 16u;
    auto offset = [&](int s) __attribute__((always_inline)) -> unsigned {
        unsigned o = noff;
        asm volatile("" : "+v"(o));
        return SHIFT ? (o - 16u * (unsigned)s) & (SLAB - 1u) : o;
    };
    auto first_vector = [&](int s) __attribute__((always_inline)) -> int { return (int)(offset(s) >> 4); };
    // how far into slot `slot` the row's vectors reach, in bytes
    auto reach = [&](int slot) __attribute__((always_inline)) -> int { return (nvec_full - slot * BLOCK) * 16; };
    auto load_slot = [&](u32x4 &z, const char *zrow, int s, int slot) __attribute__((always_inline)) {
        z = neg_inf_vec<DT>();
        const unsigned o = offset(s);
        if ((int)o < reach(slot)) z = *(const u32x4 *)(zrow + (size_t)slot * SLAB + o);
    };
    auto load_batch = [&](u32x4 (&buf)[U], const char *zrow, int s, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_slot(buf[u], zrow, s, b * U + u);
    };
    auto load_last = [&](const char *zrow, int s, long long y) __attribute__((always_inline)) {
        zy = load_elem<DT>(zrow, y);
        const int l = first_vector(s);
        if (l < tail) tz = load_elem<DT>(zrow, (long long)nvec_full * EPV + l);
    };
    auto load_first = [&](const char *zrow, int s, long long y) __attribute__((always_inline)) {
        load_batch(A, zrow, s, 0);
        load_batch(B, zrow, s, 1);
        load_last(zrow, s, y);
    };

    long long y = 0, y_next = 0, row;
    int sh;
rows_from_none:
    row = acquire(y, false);
    sh = (SHIFT ? (int)row_shift(p, row) : 0);
    if (row < p.n_tokens) load_first((const char *)p.logits + row * p.row_stride * BYTES, sh, y);

    while (row < p.n_tokens) {
        const char *zrow = (const char *)p.logits + row * p.row_stride * BYTES;
        const long long next = acquire(y_next, true);
        const bool has_next = next < p.n_tokens;
        const char *zrow_next = (const char *)p.logits + (has_next ? next : row) * p.row_stride * BYTES;
        const int sh_next = (SHIFT ? (int)row_shift(p, next) : 0);
        const int vy = (int)(y / EPV);
        const int ey = (int)(y % EPV);

        float m = -INFINITY, s = 0.f, w = 0.f;
        auto stat_step = [&](u32x4 (&buf)[U], int b) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < U; ++u)  // the sampled token's logit stays out of the sums
                if ((b * U + u) == vy / BLOCK && offset(sh) == (unsigned)(vy % BLOCK) * 16u && vy < nvec_full) set_neg_inf<DT>(buf[u], ey);
            online_batch<DT, AUX, U>(buf, p.k, m, s, w);
            if (b + 2 < nb) load_batch(buf, zrow, sh, b + 2);
        };
        for (int b = 0; b < nb; b += 2) {
            stat_step(A, b);
            if (b + 1 < nb) stat_step(B, b + 1);
        }
        // the ragged last vector, one entry per lane: its word (the rest of the lane's vector is -inf)
        unsigned tword = kNegInfF32;
        if (DT == GRPO_BF16) tword = kNegInfBf16x2;
        if (tail) {
            const int l = first_vector(sh);
            if (l < tail && !(vy == nvec_full && l == ey))
                tword = DT == GRPO_BF16 ? (kNegInfF32 | (as_u32(tz) >> 16)) : as_u32(tz);
            u32x4 tv[1] = {neg_inf_vec<DT>()};
            tv[0][0] = tword;
            online_batch<DT, AUX, 1>(tv, p.k, m, s, w);
        }
        const float mx = fmaxf(block_max<BLOCK>(m, lds_max), zy);
        const float mk = mx * p.k;
        float scaled, scaledw;
        online_rescale<AUX>(m, s, w, mx, p.k, scaled, scaledw);
        if (SHIFT && sh != 0) {  // the lanes' sums in the order of an unturned row
            const int l = first_vector(sh);
            lds_turn[0][SHIFT ? l : 0] = scaled;
            if constexpr (AUX) lds_turn[SHIFT && AUX ? 1 : 0][SHIFT ? l : 0] = scaledw;
            lds_barrier();
            scaled = lds_turn[0][SHIFT ? tid : 0];
            if constexpr (AUX) scaledw = lds_turn[SHIFT && AUX ? 1 : 0][SHIFT ? tid : 0];
        }
        RowScalars sc;
        if constexpr (AUX) {
            block_sum2<BLOCK>(scaled, scaledw, lds_sum, lds_sumw);
            if (!(mx > -INFINITY)) scaled = NAN;  // a row of -inf (or NaN) has no softmax
            float kl, H;
            sc = row_scalars_aux(p, row, zy, mx, scaled, scaledw, kl, H);
            if (tid == 0) write_row_aux(p, row, kl, H);
        } else {
            float s_excl = block_sum<BLOCK>(scaled, lds_sum);
            if (!(mx > -INFINITY)) s_excl = NAN;
            sc = row_scalars(p, row, zy, mk, s_excl);
        }
        if (tid == 0) write_row_outputs(p, row, sc.logp, sc.J, sc.flags);
        lds_barrier();  // this row's reads of the LDS arrays, the next one's writes

        char *grow = (char *)p.grad + row * p.row_stride * BYTES;
        if (!p.bwd || (sc.c == 0.f && (!AUX || sc.b == 0.f))) {
            if (has_next) load_first(zrow_next, sh_next, y_next);
            if (p.bwd) zero_row<DT, BLOCK>(grow, nvec_full, tail, tid);
        } else {
            const float q = -sc.c * p.inv_T;
            const float gy = (sc.c * p.inv_T) * (sc.s_excl / sc.s) + (AUX ? sc.gy_ent : 0.f);
            auto grad_of = [&](u32x4 &z, bool has_y, int e) __attribute__((always_inline)) {
                if constexpr (AUX) {
                    z = grad_vec_aux<DT>(z, p.k, sc.mx, sc.log2s, sc.q2, sc.bq);
                    if (has_y) put_elem<DT>(z, e, gy);
                } else {
                    float g[EPV];
                    grad_vec<DT>(z, p.k, sc.shift, q, has_y, e, gy, g);
                    z = pack<DT>(g);
                }
            };
            auto grad_step = [&](u32x4 (&buf)[U], int b) __attribute__((always_inline)) {
                u32x4 out[U];
                const bool more = b >= 2 || has_next;  // A is done with batch 0, B with batch 1: the next row's
                const char *from = b >= 2 ? zrow : zrow_next;
                const int b_load = b >= 2 ? b - 2 : b, s_load = b >= 2 ? sh : sh_next;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    forget(buf[u]);
                    out[u] = buf[u];
                    grad_of(out[u], (int)offset(sh) == (vy - (b * U + u) * BLOCK) * 16, ey);
                    order_after(noff, out[u]);
                    if (more) load_slot(buf[u], from, s_load, b_load * U + u);
                    VECTOR_FENCE();
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const unsigned o = offset(sh);
                    if ((int)o < reach(b * U + u)) st16(grow + (size_t)(b * U + u) * SLAB + o, out[u]);
                }
            };
            for (int b = (nb - 1) | 1; b > 0; b -= 2) {
                if (b < nb) grad_step(B, b);
                grad_step(A, b - 1);
            }
            if (tail) {
                const int l = first_vector(sh);
                u32x4 tv = neg_inf_vec<DT>();
                tv[0] = tword;
                grad_of(tv, vy == nvec_full && l == ey, 0);
                if (l < tail) {
                    if constexpr (DT == GRPO_BF16)
                        ((unsigned short *)grow)[(long long)nvec_full * EPV + l] = (unsigned short)(tv[0] & 0xffffu);
                    else
                        ((unsigned *)grow)[(long long)nvec_full * EPV + l] = tv[0];
                }
            }
            if (has_next) load_last(zrow_next, sh_next, y_next);
        }
        row = next;
        y = y_next;
        sh = sh_next;
    }
    if (rows_left) {
        rows_left = false;
        goto rows_from_none;
    }
}

// ---------------------------------------------------------------------------
// Small kernels around the row kernel
// ---------------------------------------------------------------------------

// How many of the rows [r0, r1) take part (mask not 0, weight not 0): this lane's share of them.
__device__ __forceinline__ int count_live(const unsigned char *mask, const float *token_w, long long r0, long long r1)
{
    int cnt = 0;
    if (mask && !token_w) {
        // the mask alone: 16 bytes per lane and step between the first and the last 16-byte
        // boundary inside it, single bytes before and after (the counts are integers: any order)
        const unsigned char *m = mask + r0;
        const long long n = r1 - r0;
        const long long head = ((16 - (long long)((unsigned long long)m & 15u)) & 15);
        const long long lead = head < n ? head : n;
        const long long nvec = (n - lead) / 16;
        for (long long i = threadIdx.x; i < lead; i += 1024) cnt += m[i] ? 1 : 0;
        for (long long v = threadIdx.x; v < nvec; v += 1024) {
            const u32x4 w = *(const u32x4 *)(m + lead + 16 * v);
#pragma unroll
            for (int d = 0; d < 4; ++d)  // bit 7 of every byte that is not zero, then count them
                cnt += __builtin_popcount((w[d] | ((w[d] & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u);
        }
        for (long long i = lead + 16 * nvec + threadIdx.x; i < n; i += 1024) cnt += m[i] ? 1 : 0;
    } else if (mask || token_w) {
        for (long long i = r0 + threadIdx.x; i < r1; i += 1024)
            cnt += ((!mask || mask[i]) && (!token_w || token_w[i] != 0.f)) ? 1 : 0;
    }
    return cnt;
}

// The rows of each segment of 4096 that take part, for batches too long for every workgroup of
// grpo_prepare to count them all itself.
static __global__ void __launch_bounds__(1024) grpo_count_rows(const unsigned char *mask, const float *token_w, long long n,
                                                        int *live_of)
{
    __shared__ int lds[16];
    const long long r0 = (long long)blockIdx.x * kOrderRows, r1 = r0 + kOrderRows < n ? r0 + kOrderRows : n;
    const int cnt = wave_sum(count_live(mask, token_w, r0, r1));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) total += lds[i];
        live_of[blockIdx.x] = total;
    }
}

// When a workgroup with a live row in hand, whose loads are under way, fills only one of the masked rows that it comes to, then takes
// its row and fills the others behind it (late), and when it fills them first until none is left.  Late, a workgroup's last
// live row is not kept waiting for the end of the batch, but the workgroup asks the queue once more when that row's gradient is
// stored.  That pays where each has several masked rows (1000 x 152064 bf16, 900 masked, 80 -> 71 us, 3000 of which 1125 277 -> 275;
// with the auxiliary terms, whose passes are longer, 1400 of which 525 163 -> 159 and, sharing CUs, 4096 x 16384 of which
// 1536 80 -> 74; 1400 x 32000, 1260 masked, 38 -> 36), or
// where it has one live row at most and shares its CU (1400 x 32000, 525 masked, with the auxiliary terms 52 -> 46), without the auxiliary
// terms and four to a CU up to five rows on four of them (1741 x 17470, 564 masked, 44.5 -> 42.8, 461 masked 45.3 -> 44.7, 2600 of which
// 1423 are 48.7 -> 47.9, 1500 x 32000, 272 masked, 48.4 -> 46.4; at thirteen on ten even, from there on it loses up to 8 %).  Fewer masked
// rows are filled by workgroups that are out of live rows while others have one more (700 x 152064, 263 masked, with the auxiliary
// terms 82 us, late 91; 1400 x 65536, 525 masked, 71 and 76; 400 x 81920, 150 masked, 41 and 45).  Streamed rows, of which
// none is held, have them late in all long batches (4096 x 152069, 1452 masked, 423 -> 421, 2500 of which 334 are 306 -> 305; 1100 of which
// 417 are 132 and 134).
struct LateRule {
    long long grid;   // the row kernel's workgroups; 0: never
    int few;          // masked rows to a workgroup up to which they are filled first
    long long up_to;  // late up to so many live rows
    long long from;   // and with more than so many
    __host__ __device__ bool late(long long n, long long live) const
    {
        const long long masked = n - live;
        return grid > 0 && (masked > few * grid || (masked > grid && masked > 4 * live) || live <= up_to || live > from);
    }
};

// Counts the unmasked rows, fixes the denominator and resets the queue before any row is processed;
// with `order`, also writes the order in which the row kernels hand out the rows of a batch with
// masked rows: first the rows that take part (mask 1 and weight not 0), then the masked ones, which
// only need zeros.  Handed out in index order, masked rows between live ones cost more than their
// bytes: the same rows with the masked ones at the end ran 5 to 8 % faster at V = 152064 (the zero fill
// of a masked row and the read-compute-write cycle of a live row share the memory system badly).
// One workgroup per 4096 rows: an ordered compaction inside the workgroup, behind the rows counted
// before its own.  Every workgroup counts the whole mask itself, at 16 bytes a lane: for the 16 KB of
// 16384 rows that is one step, against a launch of its own for the counting (2 to 5 us) and two
// atomics on the way.  That work grows with the square of the batch: in longer batches (prepare_counts_itself)
// grpo_count_rows has counted each segment (live_of) and only those numbers are added up here.
// order[0 .. M) are the live rows in increasing order, order[M .. n) the masked ones (written from the end), by their complements
// where the rule says that they are late.
static __global__ void __launch_bounds__(1024) grpo_prepare(const unsigned char *mask, const float *token_w, long long n,
                                                     double denom, WsHeader *hdr, int *order, const int *live_of, LateRule rule)
{
    __shared__ long long lds_before[16], lds_rest[16];
    __shared__ int wave_l[16], wave_m[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const long long seg0 = (long long)blockIdx.x * kOrderRows < n ? (long long)blockIdx.x * kOrderRows : n;
    int cb = 0, cr = 0;
    if (live_of) {
        for (unsigned i = tid; i < gridDim.x; i += 1024) (i < blockIdx.x ? cb : cr) += live_of[i];
    } else {
        cb = count_live(mask, token_w, 0, seg0);
        cr = count_live(mask, token_w, seg0, n);
    }
    cb = wave_sum(cb);
    cr = wave_sum(cr);
    if (lane == 0) {
        lds_before[wv] = cb;
        lds_rest[wv] = cr;
    }
    if (blockIdx.x == 0 && tid < kQueueParts) queue_counters(hdr)[tid * kQueueStride] = 0ull;
    const long long r0 = seg0 + tid * 4ll;  // four consecutive rows per lane
    bool live[4], valid[4];
    int cl = 0, cm = 0, il = 0, im = 0;
    if (order) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const long long r = r0 + e;
            valid[e] = r < n && r < seg0 + kOrderRows;
            live[e] = valid[e] && (!mask || mask[r] != 0) && (!token_w || token_w[r] != 0.f);
            cl += live[e] ? 1 : 0;
            cm += (valid[e] && !live[e]) ? 1 : 0;
        }
        il = cl, im = cm;  // inclusive scans inside the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int ul = __shfl_up(il, o, 64), um = __shfl_up(im, o, 64);
            if (lane >= o) {
                il += ul;
                im += um;
            }
        }
        if (lane == 63) {
            wave_l[wv] = il;
            wave_m[wv] = im;
        }
    }
    __syncthreads();
    long long before = 0, rest = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        before += lds_before[i];
        rest += lds_rest[i];
    }
    if (blockIdx.x == 0 && tid == 0) {
        const long long M = (!mask && !token_w) ? n : before + rest;
        const double D = denom > 0.0 ? denom : (double)M;
        hdr->D = D;
        hdr->inv_D = D > 0.0 ? 1.0 / D : 0.0;
        hdr->M = M;
        hdr->error = 0;
        hdr->fin_ticket = 0u;
    }
    if (!order) return;
    int before_l = 0, before_m = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < wv) {
            before_l += wave_l[w];
            before_m += wave_m[w];
        }
    }
    const int mark = rule.late(n, before + rest) ? -1 : 0;
    long long pl = before + before_l + (il - cl);
    long long pm = (seg0 - before) + before_m + (im - cm);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (live[e])
            order[pl++] = (int)(r0 + e);
        else if (valid[e])
            order[n - 1 - pm++] = (int)(r0 + e) ^ mark;
    }
}

// Log-probs-only calls that bring a workspace use it for the row queue alone.
static __global__ void grpo_reset_queue(WsHeader *hdr)
{
    if (threadIdx.x < kQueueParts) queue_counters(hdr)[threadIdx.x * kQueueStride] = 0ull;
    if (threadIdx.x == 0) {
        hdr->error = 0;
    }
}

// loss = -(1/D) sum_t J_t in fp64 and a fixed order; indicator counts.  With the
// auxiliary arrays (KL_ws, H_ws non-NULL) loss_out has four entries:
// total = policy + kl_coef * mean kl - ent_coef * mean H, policy, mean kl, mean H.
//
// One workgroup per segment of kFinSegment rows: it sums its rows (a fixed assignment of rows to
// lanes, wavefronts combined in a fixed order), and unless it is the only one leaves the partial sums
// in the workspace and draws a ticket; the workgroup that draws the last ticket adds the partials in
// segment order and writes the results.  Which workgroup that is varies from run to run, what it
// computes does not: the sums are bitwise reproducible.
// Bound by latency, so what counts is how few dependent steps there are: all of a lane's loads are
// issued at once, sums across lanes are DPP steps on 32-bit halves, the four counters of a workgroup
// travel as 16-bit fields of two words (at most 16384 each), and up to 16384 rows need no ticket (with
// segments of 4096 rows, seven shuffled sums and a walk over 16 wavefronts: 6.8 us for 512 rows, 17 us for 16384;
// now 3.6 and 4.6 us).
struct FinPartial {
    double s[3];
    long long c[4];
    long long pad;
};
static_assert(sizeof(FinPartial) == 64, "one partial per 64 bytes");
static_assert(kFinSegment < 65536, "counters of a segment fit 16 bits");
// One partial per 4096 rows, more than the segments need: what a workspace must hold is part of the interface and
// stays; grpo_count_rows leaves a count per 4096 rows in the same place.
constexpr size_t fin_partials_bytes(long long n)
{
    return (((size_t)((n + 4095) / 4096) * sizeof(FinPartial)) + 255) / 256 * 256;
}

struct FinParams {
    const float *J_ws, *KL_ws, *H_ws;
    const unsigned char *flags_ws;
    long long n;
    WsHeader *hdr;
    FinPartial *partials;
    float kl_coef, ent_coef;
    float *loss_out;
    long long *counts_out;
    int *error_out;
};
// What workgroup `block` of the segments' does; 1024 lanes.
__device__ __forceinline__ void finalize_segment(const FinParams &f, unsigned block)
{
    const float *J_ws = f.J_ws, *KL_ws = f.KL_ws, *H_ws = f.H_ws;
    const unsigned char *flags_ws = f.flags_ws;
    const long long n = f.n;
    WsHeader *hdr = f.hdr;
    FinPartial *partials = f.partials;
    const float kl_coef = f.kl_coef, ent_coef = f.ent_coef;
    float *loss_out = f.loss_out;
    long long *counts_out = f.counts_out;
    int *error_out = f.error_out;
    __shared__ double lds_s[3][16];
    __shared__ int lds_c[2][16];
    __shared__ long long lds_c4[4][16];
    __shared__ unsigned lds_ticket;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const bool aux = KL_ws != nullptr;
    const long long nseg = (n + kFinSegment - 1) / kFinSegment;  // 0 for an empty batch: one block, no rows
    // this block's segment, four consecutive rows per lane and step (the arrays start on 256-byte
    // boundaries and a segment is a multiple of four rows), the batch's last n % 4 rows one by one
    const long long seg0 = (long long)block * kFinSegment;
    const long long seg1 = seg0 + kFinSegment < n ? seg0 + kFinSegment : n;
    constexpr int STEPS = kFinSegment / 4096;
    f32x4 j[STEPS], kl[STEPS], h[STEPS];
    unsigned fl[STEPS];
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
        const long long i = seg0 + q * 4096ll + tid * 4ll;
        j[q] = kl[q] = h[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        fl[q] = 0u;
        if (i + 3 < seg1) {
            j[q] = *(const f32x4 *)(J_ws + i);
            fl[q] = *(const unsigned *)(flags_ws + i);
            if (aux) {
                kl[q] = *(const f32x4 *)(KL_ws + i);
                h[q] = *(const f32x4 *)(H_ws + i);
            }
        } else if (i < seg1) {  // at most three rows, in one lane of the last segment
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                if (e >= (int)(seg1 - i)) break;
                j[q][e] = J_ws[i + e];
                fl[q] |= (unsigned)flags_ws[i + e] << (8 * e);
                if (aux) {
                    kl[q][e] = KL_ws[i + e];
                    h[q][e] = H_ws[i + e];
                }
            }
        }
    }
    double s[3] = {0.0, 0.0, 0.0};
    int c01 = 0, c23 = 0;  // two counters each, 16 bits
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[0] += (double)j[q][e];
            if (aux) {
                s[1] += (double)kl[q][e];
                s[2] += (double)h[q][e];
            }
        }
        static_assert(kFlagClipHigh == 1 && kFlagClipLow == 2 && kFlagDelta == 4 && kFlagOutOfBand == 8, "bit positions");
        c01 += __builtin_popcount(fl[q] & 0x01010101u) + (__builtin_popcount(fl[q] & 0x02020202u) << 16);
        c23 += __builtin_popcount(fl[q] & 0x04040404u) + (__builtin_popcount(fl[q] & 0x08080808u) << 16);
    }
    // totals of the workgroup, in every lane of its first wavefront
    auto block_totals = [&]() {
        s[0] = wave_sum_dpp(s[0]);
        if (aux) {
            s[1] = wave_sum_dpp(s[1]);
            s[2] = wave_sum_dpp(s[2]);
        }
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) lds_s[q][wv] = s[q];
        }
    };
    auto first_wave_sums = [&]() {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (q == 0 || aux) s[q] = wave_sum_dpp(lane < 16 ? lds_s[q][lane & 15] : 0.0);
    };
    block_totals();
    c01 = wave_sum(c01);
    c23 = wave_sum(c23);
    if (lane == 0) {
        lds_c[0][wv] = c01;
        lds_c[1][wv] = c23;
    }
    __syncthreads();
    long long c[4] = {0, 0, 0, 0};
    if (wv == 0) {
        first_wave_sums();
        c01 = wave_sum(lane < 16 ? lds_c[0][lane & 15] : 0);
        c23 = wave_sum(lane < 16 ? lds_c[1][lane & 15] : 0);
        c[0] = c01 & 0xffff, c[1] = (unsigned)c01 >> 16;
        c[2] = c23 & 0xffff, c[3] = (unsigned)c23 >> 16;
    }
    if (nseg > 1) {
        if (tid == 0) {
            FinPartial pt;
#pragma unroll
            for (int q = 0; q < 3; ++q) pt.s[q] = s[q];
#pragma unroll
            for (int q = 0; q < 4; ++q) pt.c[q] = c[q];
            pt.pad = 0;
            partials[block] = pt;
            __threadfence();  // the partial is visible before the ticket is
            lds_ticket = atomicAdd(&hdr->fin_ticket, 1u);
        }
        __syncthreads();
        if (lds_ticket != (unsigned)(nseg - 1)) return;  // whole workgroup alike
        __threadfence();  // the last ticket: every partial has been delivered; read them afresh
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q] = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = 0;
        for (long long sgm = tid; sgm < nseg; sgm += 1024) {  // lane l: segments l, l + 1024, ...
            const volatile FinPartial *pp = partials + sgm;
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] += pp->s[q];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] += pp->c[q];
        }
        block_totals();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = wave_sum(c[q]);
            if (lane == 0) lds_c4[q][wv] = c[q];
        }
        __syncthreads();
        if (wv == 0) {
            first_wave_sums();
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = wave_sum(lane < 16 ? lds_c4[q][lane & 15] : 0ll);
        }
    }
    if (tid == 0) {
        const double policy = 0.0 - s[0] * hdr->inv_D;
        if (aux) {
            const double klm = s[1] * hdr->inv_D, hm = s[2] * hdr->inv_D;
            loss_out[0] = (float)(policy + (double)kl_coef * klm - (double)ent_coef * hm);
            loss_out[1] = (float)policy;
            loss_out[2] = (float)klm;
            loss_out[3] = (float)hm;
        } else {
            loss_out[0] = (float)policy;
        }
        if (error_out) *error_out = hdr->error;  // every row kernel has finished: the word is final
        if (counts_out) {
            counts_out[GRPO_COUNT_TOKENS] = hdr->M;
            counts_out[GRPO_COUNT_CLIP_HIGH] = c[0];
            counts_out[GRPO_COUNT_CLIP_LOW] = c[1];
            counts_out[GRPO_COUNT_DELTA] = c[2];
            counts_out[GRPO_COUNT_OUT_OF_BAND] = c[3];
        }
    }
}

static __global__ void __launch_bounds__(1024) grpo_finalize(FinParams f) { finalize_segment(f, blockIdx.x); }

// One wavefront per group: mean, then spread around the mean, both in fp64.
static __global__ void __launch_bounds__(64) grpo_group_adv(const float *rewards, long long n_rollouts,
                                                     const int *offsets, long long n_groups,
                                                     long long group_size, double eps_std, int ddof,
                                                     float *adv_out)
{
    const int lane = threadIdx.x;
    for (long long g = blockIdx.x; g < n_groups; g += gridDim.x) {
        long long b = offsets ? (long long)offsets[g] : g * group_size;
        long long e = offsets ? (long long)offsets[g + 1] : (g + 1) * group_size;
        b = b < 0 ? 0 : (b > n_rollouts ? n_rollouts : b);
        e = e < b ? b : (e > n_rollouts ? n_rollouts : e);
        const long long G = e - b;
        if (G == 0) continue;
        double sum = 0.0;
        for (long long i = b + lane; i < e; i += 64) sum += (double)rewards[i];
        const double mu = wave_sum(sum) / (double)G;
        double ss = 0.0;
        for (long long i = b + lane; i < e; i += 64) {
            const double d = (double)rewards[i] - mu;
            ss += d * d;
        }
        ss = wave_sum(ss);
        const double sigma = (G - ddof > 0) ? sqrt(ss / (double)(G - ddof)) : 0.0;
        const double den = sigma + eps_std;
        for (long long i = b + lane; i < e; i += 64)
            adv_out[i] = den > 0.0 ? (float)(((double)rewards[i] - mu) / den) : 0.f;
    }
}

static __global__ void __launch_bounds__(256) grpo_adv_to_tokens(const float *adv, long long n_rollouts,
                                                          const int *rollout_of_token,
                                                          long long n_tokens, float *adv_tok)
{
    for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < n_tokens;
         t += (long long)gridDim.x * 256) {
        const int r = rollout_of_token[t];
        adv_tok[t] = (r >= 0 && r < n_rollouts) ? adv[r] : NAN;
    }
}

// Both in one launch, for a batch of few groups of one size: every workgroup computes all advantages
// (16 lanes to a group of up to 16 rollouts, 64 to a larger one; the sums run over the lanes in the
// same order as above) and looks its tokens up in LDS; the first one also writes adv_out.  Two launches
// of 2 to 5 us each became one of the same length.  Up to 1024 rollouts and four rounds of groups: beyond
// them the repeated work costs more than the launch.  Neither output may overlap the rewards: a workgroup may
// still be reading them when another one writes (in place, the two launches above are taken).
constexpr int kAdvRollouts = 1024, kAdvTokens = 4096;
static __global__ void __launch_bounds__(1024) grpo_adv_fused(const float *rewards, int n_rollouts, int n_groups, int group_size,
                                                       double eps_std, int ddof, float *adv_out,
                                                       const int *rollout_of_token, long long n_tokens, float *adv_tok)
{
    __shared__ float adv[kAdvRollouts];
    const int W = group_size <= 16 ? 16 : 64;  // lanes to a group
    const int l = threadIdx.x & (W - 1);
    int tok[kAdvTokens / 1024];
#pragma unroll
    for (int q = 0; q < kAdvTokens / 1024; ++q) {
        const long long t = (long long)blockIdx.x * kAdvTokens + q * 1024 + threadIdx.x;
        tok[q] = t < n_tokens ? rollout_of_token[t] : -1;
    }
    for (int g0 = 0; g0 < n_groups; g0 += 1024 / W) {
        const int g = g0 + (int)threadIdx.x / W;
        const int b = g * group_size, e = g < n_groups ? b + group_size : b;
        auto sum_lanes = [&](double v) {
            if (W == 64) {
                v += __shfl_xor(v, 32, 64);
                v += __shfl_xor(v, 16, 64);
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            return v;
        };
        double sum = 0.0;
        for (int i = b + l; i < e; i += W) sum += (double)rewards[i];
        const double mu = sum_lanes(sum) / (double)group_size;
        double ss = 0.0;
        for (int i = b + l; i < e; i += W) {
            const double d = (double)rewards[i] - mu;
            ss += d * d;
        }
        ss = sum_lanes(ss);
        const double sigma = (group_size - ddof > 0) ? sqrt(ss / (double)(group_size - ddof)) : 0.0;
        const double den = sigma + eps_std;
        for (int i = b + l; i < e; i += W) {
            const float A = den > 0.0 ? (float)(((double)rewards[i] - mu) / den) : 0.f;
            adv[i] = A;
            if (blockIdx.x == 0) adv_out[i] = A;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kAdvTokens / 1024; ++q) {
        const long long t = (long long)blockIdx.x * kAdvTokens + q * 1024 + threadIdx.x;
        if (t < n_tokens) adv_tok[t] = (tok[q] >= 0 && tok[q] < n_rollouts) ? adv[tok[q]] : NAN;
    }
}

// r_total = r_task - alpha |l_target - l_y| (section 3.1).  The length difference is formed
// in integers, so it is exact.
static __global__ void __launch_bounds__(256) grpo_total_rewards_k(const float *task, const int *len,
                                                            const int *target, long long n,
                                                            float alpha, float *out)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        const long long d = (long long)target[i] - (long long)len[i];
        out[i] = task[i] - alpha * (float)(d < 0 ? -d : d);
    }
}

// Online filter (section 3.3): flags the groups whose rewards are not all equal.  One
// wavefront per group.
static __global__ void __launch_bounds__(64) grpo_filter_flag(const float *rewards, long long n_rollouts,
                                                       const int *offsets, long long n_groups,
                                                       long long group_size, unsigned char *keep,
                                                       unsigned char *rollout_keep)
{
    const int lane = threadIdx.x;
    for (long long g = blockIdx.x; g < n_groups; g += gridDim.x) {
        long long b = offsets ? (long long)offsets[g] : g * group_size;
        long long e = offsets ? (long long)offsets[g + 1] : (g + 1) * group_size;
        b = b < 0 ? 0 : (b > n_rollouts ? n_rollouts : b);
        e = e < b ? b : (e > n_rollouts ? n_rollouts : e);
        int differs = 0;
        if (e > b) {
            const float first = rewards[b];
            for (long long i = b + lane; i < e; i += 64) differs |= rewards[i] != first ? 1 : 0;
        }
        differs = __any(differs) ? 1 : 0;
        if (lane == 0) keep[g] = (unsigned char)differs;
        if (rollout_keep)
            for (long long i = b + lane; i < e; i += 64) rollout_keep[i] = (unsigned char)differs;
    }
}

// Flags and compaction in one launch for up to 1024 groups of one size of up to 64, 16384 rollouts in all: a
// lane to a group (its rewards lie next to one another), the kept ones counted ahead of each lane.  One
// workgroup reads everything, its lanes a group's length apart, so the number of rollouts decides (whole
// call; the two kernels around this one take 13 us at any of these sizes): 1024 groups of 16 10 us, of 24 13,
// of 32 19, of 48 26, of 64 36; 64, 128 and 256 groups of 64 10, 10 and 12.
constexpr int kFilterGroups = 1024, kFilterSize = 64, kFilterRollouts = 16384;
static __global__ void __launch_bounds__(kFilterGroups) grpo_filter_fused(const float *rewards, int n_groups, int group_size,
                                                                   unsigned char *keep, unsigned char *rollout_keep,
                                                                   int *kept_groups, int *n_kept)
{
    __shared__ int wave_tot[kFilterGroups / 64];
    const int g = threadIdx.x, lane = g & 63, wv = g >> 6;
    const int b = g * group_size;
    bool differs = false;
    if (g < n_groups) {
        const float first = rewards[b];
        for (int i = 0; i < group_size; ++i) differs |= rewards[b + i] != first;
        keep[g] = differs ? 1 : 0;
        if (rollout_keep)
            for (int i = 0; i < group_size; ++i) rollout_keep[b + i] = differs ? 1 : 0;
    }
    const unsigned long long kept = __ballot(differs);
    const int ahead = __popcll(kept & ((1ull << lane) - 1ull));
    if (lane == 0) wave_tot[wv] = __popcll(kept);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kFilterGroups / 64; ++w) {
        if (w < wv) before += wave_tot[w];
        total += wave_tot[w];
    }
    if (differs) kept_groups[before + ahead] = g;
    if (g >= total && g < n_groups) kept_groups[g] = -1;
    if (g == 0) *n_kept = total;
}

// Ordered compaction of the kept group indices: one workgroup walks the flags in chunks
// of 1024 with a running offset, so the output order is the input order.
static __global__ void __launch_bounds__(1024) grpo_filter_compact(const unsigned char *keep, long long n_groups,
                                                            int *kept_groups, int *n_kept)
{
    __shared__ int wave_tot[16];
    __shared__ int base;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) base = 0;
    __syncthreads();
    for (long long g0 = 0; g0 < n_groups; g0 += 1024) {
        const long long g = g0 + tid;
        const int k = (g < n_groups && keep[g]) ? 1 : 0;
        int incl = k;  // inclusive scan inside the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane == 63) wave_tot[wv] = incl;
        __syncthreads();
        int before = base;
        for (int w2 = 0; w2 < wv; ++w2) before += wave_tot[w2];
        if (k) kept_groups[before + incl - 1] = (int)g;
        __syncthreads();
        if (tid == 0) {
            int tot = 0;
            for (int w2 = 0; w2 < 16; ++w2) tot += wave_tot[w2];
            base += tot;
        }
        __syncthreads();
    }
    const int total = base;
    for (long long g = total + tid; g < n_groups; g += 1024) kept_groups[g] = -1;
    if (tid == 0) *n_kept = total;
}

// Packed (variable-length) batches: rollout i owns rows [cu[i], cu[i+1]).  A wavefront takes 256
// consecutive rows: it finds the rollouts of its first and of its last row together, 64 lanes
// probing at once (two rounds for 4096 rollouts), and each lane then searches between those two.
// How many of the R + 1 entries of cu are <= t (they do not decrease; if they do, the result is
// some number in range).
__device__ __forceinline__ long long count_le(const long long *cu, long long R, long long t)
{
    long long lo = 0, len = R + 1;
    for (;;) {
        const long long step = (len + 63) / 64;
        const long long at = lo + (long long)((threadIdx.x & 63) + 1) * step - 1;  // last entry of this lane's piece
        const int cnt = __popcll(__ballot(at < lo + len && cu[at < lo + len ? at : lo] <= t));
        lo += cnt * step;
        len -= cnt * step;
        if (step == 1 || len <= 0) return lo;
        if (len > step) len = step;
    }
}
static __global__ void __launch_bounds__(256) grpo_packed_rows(const long long *cu, long long n_rollouts, long long n_tokens,
                                                        int sample_level, float *weights, int *rollout_of_token)
{
    const int lane = threadIdx.x & 63;
    for (long long t0 = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 256; t0 < n_tokens; t0 += (long long)gridDim.x * 1024) {
        const long long t1 = (t0 + 256 < n_tokens ? t0 + 256 : n_tokens) - 1;
        const long long c0 = n_rollouts > 0 ? count_le(cu, n_rollouts, t0) : 0;
        const long long c1 = n_rollouts > 0 ? count_le(cu, n_rollouts, t1) : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const long long t = t0 + q * 64 + lane;
            if (t > t1) break;
            long long lo = c0, hi = c1;  // entries <= t: between those of the first and of the last row
            while (lo < hi) {
                const long long mid = (lo + hi) >> 1;
                if (cu[mid] <= t)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            float w = 0.f;
            int r = -1;
            if (lo > 0 && lo <= n_rollouts) {
                long long b = cu[lo - 1], e = cu[lo];
                b = b < 0 ? 0 : (b > n_tokens ? n_tokens : b);
                e = e < b ? b : (e > n_tokens ? n_tokens : e);
                if (t >= b && t < e) {  // always, unless cu decreases: such a row is nobody's rather than of weight 1 / 0
                    r = (int)(lo - 1);
                    w = sample_level ? (float)(1.0 / (double)(e - b)) : 1.f;
                }
            }
            if (weights) weights[t] = w;
            if (rollout_of_token) rollout_of_token[t] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static int cu_count()
{
    static std::atomic<int> cached[64];          // zero-initialised; host threads may race here
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

template <grpo_dtype DT, int BLOCK, int NV, bool AUX, bool TAIL, int NL = 0, int RST = -1, bool REM = false, bool COUNT = false, bool SHIFT = false, bool FEW = false>
void launch_cached(const RowParams &p_in, int blocks_per_cu, hipStream_t st)
{
    RowParams p = p_in;
    long long grid = (long long)cu_count() * blocks_per_cu;
    // Batches of so few rows that the queue costs more than the balance it gives: with at most one
    // row for each workgroup there is nothing to balance; narrow rows, which are queued several at a
    // time, leave workgroups without any until there are several chunks for each, and a workgroup
    // that finds the queue empty has asked all its counters in turn.  A step on 512 fp32 rows of 1024
    // entries (64 chunks of 8, 512 workgroups): 29 us through the queue, 19 strided; on 16000 bf16 rows
    // of 4000 (eight rounds) 77 and 73.  With more rounds the narrowest rows still gain (40000 bf16 rows of 1000
    // 126 and 114) but wider ones lose (32000 of 4000 126 and 140, 10000 fp32 rows of 7001, ten rounds, 107 and 113).
    if (p.n_tokens <= grid || (p.queue_chunk > 1 && p.n_tokens <= 8 * grid)) p.queued = 0;
    if (grid > p.n_tokens) grid = p.n_tokens;
    // The log-probs pass asks for twice as many rows at once while two rounds of that are left, if there is a mask: a masked
    // row, which it only looks at, costs it the counter's answer all the same.  Responses padded at their end, a third of the rows
    // masked: 16384 x 152064 bf16 491 us one at a time, 464 two, 3000 x 128256 87 and 77, 8192 x 65536 124 and 121; four and eight gain
    // no more.  A mask without a zero costs the widest rows 1 % by it (16384 x 152064 751 and 760 us, 8192 x 128256 328 and 326), but
    // to ask for two only behind a masked row, by a flag or by counts, costs every batch 1 to 3 %.
    p.queue_more = p.queue_chunk * (p.mask ? 2 : 1);
    p.more_until = (p.n_tokens - 2 * grid * p.queue_more) / p.queue_parts;
    // dynamic LDS: the waiting gradient slots, or the LDS-resident part of the row
    constexpr unsigned lds_bytes = (unsigned)(NL + row_stash_slots(BLOCK, NV, NL)) * BLOCK * 16u;
    if constexpr (lds_bytes > 0) {
        static std::atomic<bool> attr_done[64];  // setting the attribute twice is harmless
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64 && !attr_done[dev].load()) {
            if (hipFuncSetAttribute((const void *)grpo_rows_cached<DT, BLOCK, NV, AUX, TAIL, NL, RST, REM, COUNT, SHIFT, FEW>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) == hipSuccess)
                attr_done[dev].store(true);
        }
    }
    hipLaunchKernelGGL((grpo_rows_cached<DT, BLOCK, NV, AUX, TAIL, NL, RST, REM, COUNT, SHIFT, FEW>), dim3((unsigned)grid), dim3(BLOCK),
                       lds_bytes, st, p);
}

#ifndef GRPO_QUEUE_CHUNK_BYTES
#define GRPO_QUEUE_CHUNK_BYTES 32768
#endif
// One line per instantiation of the register-resident row kernel:
//   X(id, BLOCK, NV, TAIL, NL, RST without / with the auxiliary terms, REM, workgroups per CU)
// RST: gradient slots that wait in registers (-1: the instantiation's own rule), what fits beside
// the row; the auxiliary terms need a few registers more.
#define GRPO_ROW_KERNELS(X)                                   \
    X(0, 256, 1, true, 0, -1, -1, false, 8)                   \
    X(1, 256, 4, true, 0, -1, -1, false, 8)                   \
    X(2, 256, 16, true, 0, -1, -1, false, 4)                  \
    X(3, 256, 26, false, 0, 8, 8, false, 2)                   \
    X(4, 256, 32, false, 0, 14, 14, false, 2)                 \
    X(5, 512, 16, true, 0, -1, -1, false, 2)                  \
    X(6, 512, 20, false, 0, 2, 2, false, 1)                   \
    X(7, 1024, 10, true, 0, -1, -1, false, 1)                 \
    X(8, 512, 26, false, 0, 8, 8, false, 1)                   \
    X(16, 512, 26, true, 0, 8, 8, false, 1)                   \
    X(17, 512, 32, true, 0, 14, 14, false, 1)                 \
    X(9, 512, 32, false, 0, 14, 14, false, 1)                 \
    X(10, 512, 38, false, 0, -1, -1, false, 1)                \
    X(11, 512, 44, false, 0, 10, 8, false, 1)                 \
    X(12, 512, kWideRegSlots, false, 4, GRPO_WIDE_RST, GRPO_WIDE_RST, false, 1)  \
    X(13, 512, kWideRegSlots, false, 10, GRPO_WIDE_RST, GRPO_WIDE_RST, false, 1) \
    X(14, 512, kWideRegSlots, false, 18, GRPO_WIDE_RST, GRPO_WIDE_RST, false, 1) \
    X(15, 512, kRemRegSlots, false, 18, 0, 0, true, 1)
constexpr int kRowStreaming = -1;  // the plan's id for grpo_rows_streamed

// Which kernel serves rows of nvec 16-byte vectors (the last one ragged or not).  Host logic only.
//
// Narrow rows take small workgroups, several per CU (each around 16 slots per lane): the
// phases of different rows then overlap inside a CU and the per-row bookkeeping
// (queue, three barriers, scalar arithmetic) is hidden.  Only rows too wide for that
// use one workgroup per CU: 512 lanes with twice the registers, the spare ones holding
// gradient vectors back behind the next row's loads (ragged rows of up to 10 slots of 1024 lanes
// take those).
static int plan_rows(long long nvec, bool ragged)
{
    if (nvec <= 256 * 1) return 0;
    if (nvec <= 256 * 4) return 1;
    if (nvec <= 256 * 16) return 2;
    // two workgroups of 256 lanes with 256 registers each, every gradient slot waiting behind
    // the loads, are 3 % ahead of two of 512 lanes with 128.  (The log-probs pass alone gains
    // nothing, but it takes the same instantiation: the two entry points then give the same
    // bits, and the ratio of an unchanged policy to itself is exactly 1.)
    if (nvec <= 256 * 26 && !ragged) return 3;
    if (nvec <= 256 * 32 && !ragged) return 4;
    if (nvec <= 512 * 16) return 5;
    if (nvec <= 512 * 20 && !ragged) return 6;  // all 20 gradient slots wait: 18 in LDS, 2 in registers
    if (nvec <= 1024 * 10) return 7;
    // 512 lanes with twice the registers, in several widths: the arithmetic of a pass runs over
    // every slot of the instantiation, used or not.  Ragged rows as well up to 32 slots (step on
    // 4096 x 50257 fp32: 290 us, streamed 326); wider ones are streamed.  With one workgroup to a CU against
    // two, the log-probs pass alone loses there on the few row counts that just begin another round (512 rows of
    // 50257 fp32 19 us, streamed 16; 257 of 107003 bf16 18 and 16; from 1000 rows on it gains a quarter and
    // more); one plan serves both calls, so that they give the same bits.
    if (nvec <= 512 * 26) return ragged ? 16 : 8;
    if (nvec <= 512 * 32) return ragged ? 17 : 9;
    if (ragged) return kRowStreaming;
    if (nvec <= 512 * 38) return 10;
    if (nvec <= 512 * 44) return 11;
    // wider than the registers: the last slots of the row live in LDS
    if (nvec <= 512 * (kWideRegSlots + 4)) return 12;
    if (nvec <= 512 * (kWideRegSlots + 10)) return 13;
    if (nvec <= 512 * (kWideRegSlots + 18)) return 14;
    // wider than registers and LDS together: the remainder is read twice, up to as much again
    if (nvec <= 512 * 2 * (kRemRegSlots + 18)) return 15;
    return kRowStreaming;
}

// Batches of which a workgroup that has its CU to itself takes a live row or two (of padded responses five eighths of the rows are
// live): the masked ones that a workgroup without a second live row fills it fills under its first one's loads, not behind
// its first pass (FEW).  600 x 152064 bf16, a third of them masked, 77 -> 73.5 us, 512 x 200064 97.5 -> 94.5, 420 x 107001 53 -> 50.  With one live row at most
// to each the other way is 1 to 3 % ahead (400 x 152064), from 1000 rows on both are even, then it is 1 to 2 %.
constexpr bool few_rounds(long long n, long long cus) { return 5 * n > 8 * cus && n <= 3 * cus; }

// Where rows held further back, whose stores are whole lines, pay (SHIFT): wide ones in batches of any length (256 x 107001 bf16
// 33.5 -> 30.3 us, 2048 x 32001 58 -> 53); not the narrow ones, whose time the additional conditions per slot are rather
// than the memory (16384 x 1619 bf16 55.9 us, 58.8 with, x 4001 72.5 and 78, with the auxiliary terms 100 and 118) up to where the
// memory is (16384 x 8001 109 and 103, 32768 x 4001 fp32 199 and 169), and with the auxiliary terms not where few rows
// of middling width go to a workgroup (1400 x 16001 38.3 and 40.3, 2048 x 8001 fp32 36.0 and 38.5; 9000 x 16001 137 with).
constexpr bool shift_pays(int vectors, bool aux, long long row_bytes, long long n, long long cus)
{
    if (vectors <= 1024) return row_bytes >= 12288;  // (not reached by rows of up to 256 vectors, or 1024 with the auxiliary terms)
    return !aux || vectors > 4096 || row_bytes >= 40960 || n > 8 * cus;
}

template <grpo_dtype DT, bool AUX>
void launch_rows(const RowParams &p_in, hipStream_t st)
{
    RowParams p = p_in;
    {   // rows per queue increment: 1 from 32 KB per row upwards, more for narrower rows
        const long long row_bytes = p.vocab * Elem<DT>::BYTES;
        long long c = (GRPO_QUEUE_CHUNK_BYTES + row_bytes - 1) / row_bytes;
        p.queue_chunk = (int)(c < 1 ? 1 : (c > 64 ? 64 : c));
        p.queue_parts = row_bytes < 200 * 1024 ? kQueueParts : 1;
    }
    p.queued = p.hdr != nullptr;
    const long long nvec = (p.vocab + Elem<DT>::EPV - 1) / Elem<DT>::EPV;
    if (p.count_here) {
        p.queued = 0;
        if (nvec <= 256 * 1)
            launch_cached<DT, 256, 1, AUX, true, 0, -1, false, true>(p, 8, st);
        else
            launch_cached<DT, 256, 4, AUX, true, 0, -1, false, true>(p, 8, st);
        return;
    }
    switch (plan_rows(nvec, p.vocab % Elem<DT>::EPV != 0)) {
#define GRPO_ROW_CASE(ID, BLOCK, NV, TAIL, NL, RSTP, RSTA, REM, PERCU)                              \
    case ID:                                                                                       \
        static_assert(PERCU == row_blocks_per_cu(BLOCK, NV), "workgroups per CU");                \
        /* gradient rows that begin inside a line, if the slots hold a row seven vectors further back */ \
        if constexpr (NL == 0 && BLOCK * NV > (AUX ? 1024 : 256)) {                                \
            /* 512 lanes of 26 and 32 slots: the kernel for ragged rows serves whole ones too */   \
            constexpr bool T = TAIL || (BLOCK == 512 && (NV == 26 || NV == 32));                   \
            if ((p.shift0 | p.shift_step) != 0 && p.vocab / Elem<DT>::EPV + 7 <= BLOCK * NV &&     \
                shift_pays(BLOCK * NV, AUX, p.vocab * Elem<DT>::BYTES, p.n_tokens, cu_count())) {  \
                launch_cached<DT, BLOCK, NV, AUX, T, 0, (AUX ? RSTA : RSTP), false, false, true>(p, PERCU, st); \
                break;                                                                             \
            }                                                                                      \
        }                                                                                          \
        if constexpr (!AUX && !REM && PERCU == 1) {                                                \
            if (p.order && few_rounds(p.n_tokens, cu_count())) {                                   \
                launch_cached<DT, BLOCK, NV, AUX, TAIL, NL, RSTP, false, false, false, true>(p, PERCU, st); \
                break;                                                                             \
            }                                                                                      \
        }                                                                                          \
        launch_cached<DT, BLOCK, NV, AUX, TAIL, NL, (AUX ? RSTA : RSTP), REM>(p, PERCU, st);      \
        break;
        GRPO_ROW_KERNELS(GRPO_ROW_CASE)
#undef GRPO_ROW_CASE
    default: {
        long long grid = (long long)cu_count() * kStreamPerCu;
        // turned lanes cost a row instructions (59 fp32 rows of 126615 35.2 and 36.8 us a step): not where each workgroup has
        // one row at most, whose time no memory bounds
        const bool shift = (p.shift0 | p.shift_step) != 0 && p.n_tokens > grid;
        if (p.n_tokens <= grid) {
            p.queued = 0;
            grid = p.n_tokens;
        }
        if (shift)
            hipLaunchKernelGGL((grpo_rows_streamed<DT, AUX, true>), dim3((unsigned)grid), dim3(kStreamBlock), 0, st, p);
        else
            hipLaunchKernelGGL((grpo_rows_streamed<DT, AUX, false>), dim3((unsigned)grid), dim3(kStreamBlock), 0, st, p);
    }
    }
}

#ifdef GRPO_ROWS_OF
template void launch_rows<GRPO_ROWS_OF>(const RowParams &, hipStream_t);
}  // namespace grpo_impl
#else
#ifdef GRPO_ROWS_APART
extern template void launch_rows<GRPO_BF16, false>(const RowParams &, hipStream_t);
extern template void launch_rows<GRPO_BF16, true>(const RowParams &, hipStream_t);
extern template void launch_rows<GRPO_F32, false>(const RowParams &, hipStream_t);
extern template void launch_rows<GRPO_F32, true>(const RowParams &, hipStream_t);
#endif

// The integer a C caller put into an enum parameter.  The C ABI passes enums as ints and a C caller
// may pass any int; in C++ merely reading an enum object that holds no enumerator's value is
// undefined, so the boundary reads the bytes instead and validates the integer.
template <typename E>
int raw_enum(const E &e)
{
    static_assert(sizeof(E) == sizeof(int), "enums of the C ABI are ints");
    int v;
    __builtin_memcpy(&v, &e, sizeof v);
    return v;
}

static grpo_status check_logits_args(const void *logits, int dtype, int64_t n_tokens, int64_t vocab,
                              int64_t row_stride, const int64_t *tokens, float temperature)
{
    if (dtype != GRPO_F32 && dtype != GRPO_BF16) return GRPO_ERR_DTYPE;
    if (n_tokens < 0 || vocab <= 0 || vocab > kMaxVocab || row_stride < vocab) return GRPO_ERR_SHAPE;
    if (!(temperature > 0.f) || !std::isfinite(temperature)) return GRPO_ERR_PARAM;
    if (n_tokens == 0) return GRPO_OK;
    if (!logits || !tokens) return GRPO_ERR_NULL;
    const int64_t bytes = dtype == GRPO_BF16 ? 2 : 4;
    if (((uintptr_t)logits & 15u) != 0 || ((row_stride * bytes) & 15) != 0) return GRPO_ERR_ALIGN;
    return GRPO_OK;
}

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static unsigned fin_blocks(int64_t n) { return (unsigned)(n > 0 ? (n + kFinSegment - 1) / kFinSegment : 1); }
// header | J, KL estimate, entropy per row (f32 each) | indicator bits per row (u8) | partial sums per
// segment | the order the rows are handed out in (i32 per row)
constexpr size_t loss_workspace_bytes(long long n)
{
    return kHeaderBytes + 4 * (((size_t)n * 4 + 255) / 256 * 256) + ((size_t)n + 255) / 256 * 256 + fin_partials_bytes(n);
}
// Up to how many rows, of at most how many vectors, the row kernel counts the rows itself and grpo_prepare is not
// launched.  Every workgroup then reads the whole mask, and the weights.  Step with and without grpo_prepare: 512 rows of
// 1000 fp32 21.4 and 18.1 us, 1024 rows of 8000 bf16 21.0 and 18.6, with weights and auxiliary terms 28.4 and 27.0
// (4000 bf16); 1500 rows 23.1 and 22.1, 30.2 and 30.3; 2048 rows 27.0 and 27.6, 34.2 and 36.0.  Wider rows take
// long enough, and from more rows than CUs on they want grpo_prepare's order.
constexpr long long kCountRows = 1024, kCountVectors = 1024;
// Up to how many rows every workgroup of grpo_prepare counts all of them itself.  Counting them first takes 9.5 us
// for both launches up to 524288 rows and 13 for 2097152; counted by every workgroup, a mask of 131072 rows
// takes 7.3 us, of 262144 10.3, of 2097152 51 and of 4194304 194; weights, read one by one, of 16384 rows 8.5,
// of 32768 13.7 and of 4194304 3300 (mask and weights 5200).
constexpr bool prepare_counts_itself(long long n, bool weights) { return n <= (weights ? 16384 : 131072); }

static grpo_status loss_impl(bool aux, const void *logits, int dtype, int64_t n_tokens, int64_t vocab,
                      int64_t row_stride, const int64_t *tokens, const float *old_logprobs,
                      const float *ref_logprobs, const float *advantages, const uint8_t *mask,
                      const float *token_weights, float eps_low, float eps_high, float delta,
                      float temperature, float kl_coef,
                      float entropy_coef, double denom, float grad_scale, float *loss_out,
                      float *logprobs_out, float *entropy_out, int64_t *counts_out,
                      void *grad_logits, void *workspace, size_t workspace_bytes, void *stream,
                      int32_t *error_out = nullptr)
{
    grpo_status rc = check_logits_args(logits, dtype, n_tokens, vocab, row_stride, tokens, temperature);
    if (rc != GRPO_OK) return rc;
    if (!(eps_low >= 0.f && eps_low <= 1.f) || !(eps_high >= 0.f) || !std::isfinite(eps_high) ||
        !(delta > 1.f + eps_high) || std::isnan(denom) || std::isnan(grad_scale) ||
        !std::isfinite(kl_coef) || !std::isfinite(entropy_coef))
        return GRPO_ERR_PARAM;
    if (!loss_out) return GRPO_ERR_NULL;
    if (n_tokens > 0 && (!old_logprobs || !advantages || !grad_logits)) return GRPO_ERR_NULL;
    if (n_tokens > 0 && kl_coef != 0.f && !ref_logprobs) return GRPO_ERR_NULL;
    if (n_tokens > 0 && ((uintptr_t)grad_logits & 15u) != 0) return GRPO_ERR_ALIGN;
    if (!workspace || ((uintptr_t)workspace & 255u) != 0 ||
        workspace_bytes < grpo_workspace_bytes(n_tokens))
        return GRPO_ERR_WORKSPACE;

    char *ws = (char *)workspace;
    const size_t col = align_up((size_t)n_tokens * 4, 256);
    WsHeader *hdr = (WsHeader *)ws;
    float *J_ws = (float *)(ws + kHeaderBytes);
    float *KL_ws = (float *)(ws + kHeaderBytes + col);
    float *H_ws = (float *)(ws + kHeaderBytes + 2 * col);
    unsigned char *flags_ws = (unsigned char *)(ws + kHeaderBytes + 3 * col);
    FinPartial *partials = (FinPartial *)(ws + kHeaderBytes + 3 * col + align_up((size_t)n_tokens, 256));
    int *order = (int *)((char *)partials + fin_partials_bytes(n_tokens));
    hipStream_t st = (hipStream_t)stream;

    // rows of 32 KB and more, some of them masked, more of them than CUs: the live rows first, then the masked ones
    if (!((mask || (aux && token_weights)) && n_tokens <= 0x7fffffffll && n_tokens > cu_count() &&
          vocab * (dtype == GRPO_BF16 ? 2 : 4) >= kOrderMinRowBytes))
        order = nullptr;
    LateRule rule = {};
    if (order) {
        grpo_row_plan plan;
        grpo_row_kernel_plan((grpo_dtype)dtype, vocab, &plan);
        const long long grid = (long long)cu_count() * plan.workgroups_per_cu;
        // (from the queue only; rows with a streamed remainder gain nothing)
        if (n_tokens > grid && !plan.streamed_remainder) {
            const bool shared = plan.workgroups_per_cu > 1;
            rule = {grid, !aux ? 4 : shared ? 1 : 2, !shared ? 0 : !aux && plan.workgroups_per_cu == 4 ? grid + grid / 4 : grid,
                    plan.streaming ? 4 * grid : n_tokens};
        }
    }
    const float *weights = aux ? token_weights : nullptr;
    const dim3 segments(order ? (unsigned)((n_tokens + kOrderRows - 1) / kOrderRows) : 1u);
    int *live_of = nullptr;
    if (order && !prepare_counts_itself(n_tokens, weights)) {
        live_of = (int *)partials;  // 64 bytes for each 4096 rows, free until grpo_finalize
        hipLaunchKernelGGL(grpo_count_rows, segments, dim3(1024), 0, st, mask, weights, (long long)n_tokens, live_of);
    }
    const long long epv = dtype == GRPO_BF16 ? 8 : 4;
    const bool count_here = n_tokens > 0 && n_tokens <= kCountRows && (vocab + epv - 1) / epv <= kCountVectors;
    if (!count_here)
        hipLaunchKernelGGL(grpo_prepare, segments, dim3(1024), 0, st, mask, weights, (long long)n_tokens, denom, hdr, order,
                           (const int *)live_of, rule);
    if (n_tokens > 0) {
        RowParams p = {};
        p.count_here = count_here ? 1 : 0;
        p.denom = denom;
        p.logits = logits;
        p.grad = grad_logits;
        p.tokens = (const long long *)tokens;
        p.old_lp = old_logprobs;
        p.adv = advantages;
        p.mask = mask;
        p.logprobs_out = logprobs_out;
        p.J_ws = J_ws;
        p.flags_ws = flags_ws;
        p.hdr = hdr;
        p.n_tokens = n_tokens;
        p.vocab = vocab;
        p.row_stride = row_stride;
        p.inv_T = 1.0f / temperature;
        p.k = (float)((double)kLog2e / (double)temperature);
        p.lo = 1.0f - eps_low;
        p.hi = 1.0f + eps_high;
        p.delta = delta;
        p.grad_scale = grad_scale;
        p.bwd = 1;
        p.shift0 = (unsigned)((uintptr_t)grad_logits >> 4) & 7u;
        p.shift_step = (unsigned)(row_stride * (dtype == GRPO_BF16 ? 2 : 4) >> 4) & 7u;
        p.order = order;
        if (aux) {
            p.ref_lp = kl_coef != 0.f ? ref_logprobs : nullptr;
            p.token_w = token_weights;
            p.KL_ws = KL_ws;
            p.H_ws = H_ws;
            p.entropy_out = entropy_out;
            p.kl_coef = kl_coef;
            p.ent_coef = entropy_coef;
            if (dtype == GRPO_BF16)
                launch_rows<GRPO_BF16, true>(p, st);
            else
                launch_rows<GRPO_F32, true>(p, st);
        } else {
            if (dtype == GRPO_BF16)
                launch_rows<GRPO_BF16, false>(p, st);
            else
                launch_rows<GRPO_F32, false>(p, st);
        }
    }
    const FinParams fin = {J_ws, aux ? KL_ws : nullptr, H_ws, flags_ws, (long long)n_tokens, hdr, partials, kl_coef,
                           entropy_coef, loss_out, (long long *)counts_out, (int *)error_out};
    hipLaunchKernelGGL(grpo_finalize, dim3(fin_blocks(n_tokens)), dim3(1024), 0, st, fin);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

// ---------------------------------------------------------------------------
// Built-in scratch for grpo_loss_fwd_bwd_noalloc: the workspace of grpo_loss_fwd_bwd for
// GRPO_NOALLOC_MAX_TOKENS rows as an array in the device image, so that callers that cannot
// allocate (graph capture, serving loops) need not bring one.  Every GPU that loads the
// library holds its own copy at its own address.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = loss_workspace_bytes(GRPO_NOALLOC_MAX_TOKENS);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// The device address of `scratch` on the current device.  In host code the array's name is
// only a handle for the runtime, not an address a kernel can use: the address comes from
// hipGetSymbolAddress, once per device, with that device current, and is kept per device.
static void *scratch_address()
{
    static std::atomic<void *> cached[64];  // zero-initialised; racing host threads store the same value
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    void *ptr = cached[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();  // leave no sticky error behind for the caller's next HIP call
            return nullptr;
        }
        cached[dev].store(ptr, std::memory_order_release);
    }
    return ptr;
}

}  // namespace grpo_impl
using namespace grpo_impl;

extern "C" {

const char *grpo_status_string(grpo_status status)
{
    switch (raw_enum(status)) {
        case GRPO_OK: return "ok";
        case GRPO_ERR_NULL: return "a required pointer is NULL";
        case GRPO_ERR_SHAPE: return "bad shape: negative size, vocab outside [1, 2^28] or row_stride < vocab";
        case GRPO_ERR_DTYPE: return "unknown dtype";
        case GRPO_ERR_ALIGN: return "logits/grad base pointer or row pitch is not 16-byte aligned";
        case GRPO_ERR_PARAM:
            return "bad parameter: need temperature > 0, 0 <= eps_low <= 1, eps_high >= 0, "
                   "delta > 1 + eps_high, eps_std >= 0, ddof in {0,1}";
        case GRPO_ERR_WORKSPACE: return "workspace is NULL, not 256-byte aligned or too small";
        case GRPO_ERR_HIP: return "HIP runtime error at kernel launch";
        case GRPO_ERR_CAPACITY:
            return "n_tokens exceeds GRPO_NOALLOC_MAX_TOKENS, the rows the library's built-in scratch array holds";
    }
    return "unknown status";
}

grpo_status grpo_row_kernel_plan(grpo_dtype dtype_arg, int64_t vocab, grpo_row_plan *plan_out)
{
    const int dtype = raw_enum(dtype_arg);
    if (dtype != GRPO_F32 && dtype != GRPO_BF16) return GRPO_ERR_DTYPE;
    if (vocab <= 0 || vocab > kMaxVocab) return GRPO_ERR_SHAPE;
    if (!plan_out) return GRPO_ERR_NULL;
    const int epv = dtype == GRPO_BF16 ? 8 : 4;
    grpo_row_plan r = {};
    r.vectors = (vocab + epv - 1) / epv;
    switch (plan_rows(r.vectors, vocab % epv != 0)) {
#define GRPO_ROW_CASE(ID, BLOCK, NV, TAIL, NL, RSTP, RSTA, REM, PERCU) \
    case ID:                                                          \
        r.lanes = BLOCK;                                              \
        r.register_slots = NV;                                        \
        r.lds_slots = NL;                                             \
        r.workgroups_per_cu = PERCU;                                  \
        r.ragged_tail_slot = TAIL ? 1 : 0;                            \
        r.streamed_remainder = REM ? 1 : 0;                           \
        break;
        GRPO_ROW_KERNELS(GRPO_ROW_CASE)
#undef GRPO_ROW_CASE
    default:
        r.streaming = 1;
        r.lanes = kStreamBlock;
        r.workgroups_per_cu = kStreamPerCu;
    }
    const int64_t capacity = (int64_t)r.lanes * (r.register_slots + r.lds_slots);
    r.resident_vectors = r.streaming ? 0 : (r.vectors < capacity ? r.vectors : capacity);
    *plan_out = r;
    return GRPO_OK;
}

size_t grpo_workspace_bytes(int64_t n_tokens)
{
    if (n_tokens < 0) return 0;
    return loss_workspace_bytes(n_tokens);
}

// Do [a, a + na) and [b, b + nb) share a byte?
static bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

grpo_status grpo_group_advantages(const float *rewards, int64_t n_rollouts,
                                  const int32_t *group_offsets, int64_t n_groups,
                                  int64_t group_size, float eps_std, int ddof, float *adv_out,
                                  const int32_t *rollout_of_token, int64_t n_tokens,
                                  float *adv_tok_out, void *stream)
{
    if (n_rollouts < 0 || n_groups < 0 || n_tokens < 0) return GRPO_ERR_SHAPE;
    if (!group_offsets && (group_size <= 0 || n_groups * group_size != n_rollouts) && n_groups > 0)
        return GRPO_ERR_SHAPE;
    if (!(eps_std >= 0.f) || !std::isfinite(eps_std) || (ddof != 0 && ddof != 1)) return GRPO_ERR_PARAM;
    if (n_groups > 0 && n_rollouts > 0 && (!rewards || !adv_out)) return GRPO_ERR_NULL;
    if (rollout_of_token && n_tokens > 0 && (!adv_tok_out || !adv_out)) return GRPO_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    const bool any_work = (n_groups > 0 && n_rollouts > 0) || (rollout_of_token && n_tokens > 0);
    if (!any_work) return GRPO_OK;
    if (!group_offsets && n_groups > 0 && n_rollouts > 0 && rollout_of_token && n_tokens > 0 &&
        n_rollouts <= kAdvRollouts && n_groups <= (group_size <= 16 ? 4 * 64 : 4 * 16) &&
        !overlap(rewards, (size_t)n_rollouts * 4, adv_out, (size_t)n_rollouts * 4) &&
        !overlap(rewards, (size_t)n_rollouts * 4, adv_tok_out, (size_t)n_tokens * 4)) {
        hipLaunchKernelGGL(grpo_adv_fused, dim3((unsigned)((n_tokens + kAdvTokens - 1) / kAdvTokens)), dim3(1024), 0, st,
                           rewards, (int)n_rollouts, (int)n_groups, (int)group_size, (double)eps_std, ddof, adv_out,
                           rollout_of_token, (long long)n_tokens, adv_tok_out);
        return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
    }
    if (n_groups > 0 && n_rollouts > 0) {
        const unsigned grid = (unsigned)(n_groups < 4096 ? n_groups : 4096);
        hipLaunchKernelGGL(grpo_group_adv, dim3(grid), dim3(64), 0, st, rewards, (long long)n_rollouts,
                           group_offsets, (long long)n_groups, (long long)group_size, (double)eps_std,
                           ddof, adv_out);
    }
    if (rollout_of_token && n_tokens > 0) {
        long long blocks = (n_tokens + 255) / 256;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(grpo_adv_to_tokens, dim3((unsigned)blocks), dim3(256), 0, st, adv_out,
                           (long long)n_rollouts, rollout_of_token, (long long)n_tokens, adv_tok_out);
    }
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

grpo_status grpo_total_rewards(const float *task_rewards, const int32_t *lengths,
                               const int32_t *target_lengths, int64_t n_rollouts, float alpha,
                               float *rewards_out, void *stream)
{
    if (n_rollouts < 0) return GRPO_ERR_SHAPE;
    if (!std::isfinite(alpha)) return GRPO_ERR_PARAM;
    if (n_rollouts == 0) return GRPO_OK;
    if (!task_rewards || !lengths || !target_lengths || !rewards_out) return GRPO_ERR_NULL;
    long long blocks = (n_rollouts + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(grpo_total_rewards_k, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       task_rewards, lengths, target_lengths, (long long)n_rollouts, alpha, rewards_out);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

grpo_status grpo_filter_groups(const float *rewards, int64_t n_rollouts, const int32_t *group_offsets,
                               int64_t n_groups, int64_t group_size, uint8_t *keep_out,
                               int32_t *kept_groups_out, int32_t *n_kept_out,
                               uint8_t *rollout_keep_out, void *stream)
{
    if (n_rollouts < 0 || n_groups < 0 || n_groups > 0x7fffffffll) return GRPO_ERR_SHAPE;
    if (!group_offsets && n_groups > 0 && (group_size <= 0 || n_groups * group_size != n_rollouts))
        return GRPO_ERR_SHAPE;
    if (!n_kept_out) return GRPO_ERR_NULL;
    if (n_groups > 0 && (!keep_out || !kept_groups_out)) return GRPO_ERR_NULL;
    if (n_groups > 0 && n_rollouts > 0 && !rewards) return GRPO_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    if (!group_offsets && n_groups > 0 && n_groups <= kFilterGroups && group_size <= kFilterSize &&
        n_rollouts <= kFilterRollouts) {
        hipLaunchKernelGGL(grpo_filter_fused, dim3(1), dim3(kFilterGroups), 0, st, rewards, (int)n_groups, (int)group_size,
                           keep_out, rollout_keep_out, kept_groups_out, n_kept_out);
        return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
    }
    if (n_groups > 0) {
        const unsigned grid = (unsigned)(n_groups < 4096 ? n_groups : 4096);
        hipLaunchKernelGGL(grpo_filter_flag, dim3(grid), dim3(64), 0, st, rewards, (long long)n_rollouts,
                           group_offsets, (long long)n_groups, (long long)group_size, keep_out,
                           rollout_keep_out);
    }
    hipLaunchKernelGGL(grpo_filter_compact, dim3(1), dim3(1024), 0, st, keep_out, (long long)n_groups,
                       kept_groups_out, n_kept_out);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

grpo_status grpo_packed_layout(const int64_t *cu_seqlens, int64_t n_rollouts, int64_t n_tokens,
                               int sample_level, float *weights_out, int32_t *rollout_of_token_out,
                               void *stream)
{
    if (n_rollouts < 0 || n_tokens < 0 || n_rollouts > 0x7fffffffll) return GRPO_ERR_SHAPE;
    if (n_rollouts > 0 && !cu_seqlens) return GRPO_ERR_NULL;
    if (!weights_out && !rollout_of_token_out) return GRPO_ERR_NULL;
    if (n_tokens == 0) return GRPO_OK;
    hipStream_t st = (hipStream_t)stream;
    long long blocks = (n_tokens + 1023) / 1024;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(grpo_packed_rows, dim3((unsigned)blocks), dim3(256), 0, st, (const long long *)cu_seqlens,
                       (long long)n_rollouts, (long long)n_tokens, sample_level ? 1 : 0, weights_out, rollout_of_token_out);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

grpo_status grpo_logprobs_fwd(const void *logits, grpo_dtype dtype_arg, int64_t n_tokens, int64_t vocab,
                              int64_t row_stride, const int64_t *tokens, const uint8_t *mask,
                              float temperature, float *logprobs_out, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    const int dtype = raw_enum(dtype_arg);
    grpo_status rc = check_logits_args(logits, dtype, n_tokens, vocab, row_stride, tokens, temperature);
    if (rc != GRPO_OK) return rc;
    if (workspace && (((uintptr_t)workspace & 255u) != 0 || workspace_bytes < kHeaderBytes))
        return GRPO_ERR_WORKSPACE;
    if (n_tokens == 0) return GRPO_OK;
    if (!logprobs_out) return GRPO_ERR_NULL;
    RowParams p = {};
    p.logits = logits;
    p.tokens = (const long long *)tokens;
    p.mask = mask;
    p.logprobs_out = logprobs_out;
    p.hdr = (WsHeader *)workspace;  // NULL: rows are strided over the grid instead of queued
    p.n_tokens = n_tokens;
    p.vocab = vocab;
    p.row_stride = row_stride;
    p.inv_T = 1.0f / temperature;
    p.k = (float)((double)kLog2e / (double)temperature);
    p.bwd = 0;
    hipStream_t st = (hipStream_t)stream;
    if (workspace) hipLaunchKernelGGL(grpo_reset_queue, dim3(1), dim3(64), 0, st, p.hdr);
    if (dtype == GRPO_BF16)
        launch_rows<GRPO_BF16, false>(p, st);
    else
        launch_rows<GRPO_F32, false>(p, st);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

grpo_status grpo_loss_fwd_bwd(const void *logits, grpo_dtype dtype_arg, int64_t n_tokens, int64_t vocab,
                              int64_t row_stride, const int64_t *tokens, const float *old_logprobs,
                              const float *advantages, const uint8_t *mask, float eps_low,
                              float eps_high, float delta, float temperature, double denom,
                              float grad_scale, float *loss_out, float *logprobs_out,
                              int64_t *counts_out, void *grad_logits, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    const int dtype = raw_enum(dtype_arg);
    return loss_impl(false, logits, dtype, n_tokens, vocab, row_stride, tokens, old_logprobs, nullptr,
                     advantages, mask, nullptr, eps_low, eps_high, delta, temperature, 0.f, 0.f, denom,
                     grad_scale, loss_out, logprobs_out, nullptr, counts_out, grad_logits, workspace,
                     workspace_bytes, stream);
}

grpo_status grpo_loss_fwd_bwd_noalloc(const void *logits, grpo_dtype dtype_arg, int64_t n_tokens,
                                      int64_t vocab, int64_t row_stride, const int64_t *tokens,
                                      const float *old_logprobs, const float *advantages,
                                      const uint8_t *mask, float eps_low, float eps_high,
                                      float delta, float temperature, double denom,
                                      float grad_scale, float *loss_out, float *logprobs_out,
                                      int64_t *counts_out, void *grad_logits, int32_t *error_out,
                                      void *stream)
{
    const int dtype = raw_enum(dtype_arg);
    // the size limit first: it needs no device, and nothing may be launched beyond it
    if (n_tokens > (int64_t)GRPO_NOALLOC_MAX_TOKENS) return GRPO_ERR_CAPACITY;
    static_assert(kScratchBytes % 256 == 0, "the scratch array is a whole number of 256-byte lines");
    // Validate everything else against a stand-in address before the device is asked for the
    // real one, so that argument errors are reported the same way with or without a GPU.
    // (loss_impl launches nothing when validation fails, and fails here only on arguments.)
    if (n_tokens >= 0 && grpo_workspace_bytes(n_tokens) > kScratchBytes) return GRPO_ERR_CAPACITY;
    {
        const grpo_status rc = check_logits_args(logits, dtype, n_tokens, vocab, row_stride, tokens, temperature);
        if (rc != GRPO_OK) return rc;
        if (!(eps_low >= 0.f && eps_low <= 1.f) || !(eps_high >= 0.f) || !std::isfinite(eps_high) ||
            !(delta > 1.f + eps_high) || std::isnan(denom) || std::isnan(grad_scale))
            return GRPO_ERR_PARAM;
        if (!loss_out) return GRPO_ERR_NULL;
        if (n_tokens > 0 && (!old_logprobs || !advantages || !grad_logits)) return GRPO_ERR_NULL;
        if (n_tokens > 0 && ((uintptr_t)grad_logits & 15u) != 0) return GRPO_ERR_ALIGN;
    }
    void *ws = scratch_address();
    if (!ws) return GRPO_ERR_HIP;
    return loss_impl(false, logits, dtype, n_tokens, vocab, row_stride, tokens, old_logprobs, nullptr,
                     advantages, mask, nullptr, eps_low, eps_high, delta, temperature, 0.f, 0.f, denom,
                     grad_scale, loss_out, logprobs_out, nullptr, counts_out, grad_logits, ws,
                     kScratchBytes, stream, error_out);
}

grpo_status grpo_loss_aux_fwd_bwd(const void *logits, grpo_dtype dtype_arg, int64_t n_tokens,
                                  int64_t vocab, int64_t row_stride, const int64_t *tokens,
                                  const float *old_logprobs, const float *ref_logprobs,
                                  const float *advantages, const uint8_t *mask,
                                  const float *token_weights, float eps_low, float eps_high,
                                  float delta, float temperature, float kl_coef,
                                  float entropy_coef, double denom, float grad_scale,
                                  float *loss_out, float *logprobs_out, float *entropy_out,
                                  int64_t *counts_out, void *grad_logits, void *workspace,
                                  size_t workspace_bytes, void *stream)
{
    const int dtype = raw_enum(dtype_arg);
    return loss_impl(true, logits, dtype, n_tokens, vocab, row_stride, tokens, old_logprobs,
                     ref_logprobs, advantages, mask, token_weights, eps_low, eps_high, delta,
                     temperature, kl_coef,
                     entropy_coef, denom, grad_scale, loss_out, logprobs_out, entropy_out, counts_out,
                     grad_logits, workspace, workspace_bytes, stream);
}

grpo_status grpo_workspace_error(const void *workspace, int32_t *flag_out, void *stream)
{
    if (!workspace || !flag_out) return GRPO_ERR_NULL;
    const WsHeader *hdr = (const WsHeader *)workspace;
    int v = 0;
    if (hipMemcpyAsync(&v, &hdr->error, sizeof(int), hipMemcpyDeviceToHost, (hipStream_t)stream) != hipSuccess)
        return GRPO_ERR_HIP;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return GRPO_ERR_HIP;
    *flag_out = v;
    return GRPO_OK;
}

}  // extern "C"

#include "lmhead.hpp"
#endif  // GRPO_ROWS_OF
