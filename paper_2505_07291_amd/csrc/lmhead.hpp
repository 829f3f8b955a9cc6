// Language-model head fused with the GRPO objective: the logits z = h W^T of the policy of
// section 3.4 are produced, reduced and differentiated here instead of being handed in.
// This file is the second half of grpo.hip's translation unit (it is included at its end
// and uses the row arithmetic, the workspace header and the small kernels defined there).
//
// Everything heavy is one bf16 MFMA kernel, lm_gemm_nt: C[M x N] = A[M x K] B[N x K]^T with
// fp32 accumulation.  An operand is either contiguous along K ([M][K], the plain case) or
// "K-major" ([K][M], read from LDS with the transposing reads of gfx950).  It runs three times:
//   logits   z  = H W^T        (K = d_model)  A = H, B = W, both plain
//                                             epilogue: per-row softmax partials in fp32
//                                             from the accumulators, z_y, optional fp32 z
//   dL/dH       = G W          (K = vocab)    A = G plain, B = W K-major; epilogue: bf16 store
//   dL/dW       = G^T H        (K = tokens)   A = G K-major, B = H^T plain; epilogue: fp32 store
//                                             or accumulate
// G = dL/dz is formed once, in bf16, by an elementwise kernel and serves both gradient
// products as it lies; W is never copied; H^T (the chunk's gradient rows, [d][rows]) is the
// one transposed copy, 1/30 of G's size.
//
// The backward works through the rows that take part in chunks of at most `cap` rows (a
// multiple of 256 chosen from the size of the caller's workspace): logits, G and H^T
// exist for one chunk at a time, dL/dH rows of different chunks are disjoint and dL/dW is
// accumulated in fp32 from chunk to chunk.  The workspace is therefore bounded by the
// chunk, not by the number of tokens.  The live rows are dealt evenly over the chunks
// that are needed (lm_chunk_range, computed on the device from the live count), so no
// chunk is a small remainder.
//
// Kernel shape (gfx950): 512 lanes = 8 wavefronts per workgroup (two per SIMD), one workgroup
// for each CU that walks through 256 x 256 tiles of C, K in steps of 64.  Each wavefront owns a 128 x 64 part
// as 8 x 4 blocks of v_mfma_f32_16x16x32_bf16 (128 accumulator registers per lane).  Eight
// wavefronts rather than four because one wavefront sustains only about one 16-byte-per-lane
// load every 170 cycles and one ds_read_b128 every 58 (measured, whatever is in flight):
// at four wavefronts the tile's operand loads take longer than its products.  Operand
// tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds, no register
// staging, no vector address arithmetic) through a ring of five 32 KB slots, all 160 KB of a
// CU, that runs on from one tile of C to the next.  Inside a tile row the eight 16-byte chunks are stored at
// chunk ^ ((row >> 1) & 7), applied on the global-address side, so that 16 consecutive rows of one logical chunk (a
// quarter of a ds_read_b128 fragment read) fall on 16 different groups of four banks.
// What bounds it is power: the chip lowers its clock until the products of random data fit.  In registers alone,
// 16 x 16 x 32 products of normally distributed values reach 2065 TFLOP/s and 32 x 32 x 16 ones 1780 (both about 2480 on
// zeros): half of the accumulator traffic per product.  Fragments from LDS bring that to 1670 (profiles/mfma_rates.txt).
// Log-probs of 2048 x 65536 x 4096 take 635 us (1730 TFLOP/s) on copies of this kernel whose operand tiles are loaded once
// and for all, 766 (1435) where every load finds its tile in the L2 cache, 813 (1350) as it is.  With the
// products in this form, their loads issued at the beginning of a half step and wavefronts in the middle of their products
// preferred over others (1.3 and 2.3 % of a call), the three products of about 2560 live rows with [152064, 5120]
// went from 3.11 / 2.72 / 2.72 ms (logits with their fp32 copy, dL/dH, dL/dW) to 2.75 / 2.36 / 2.66.  Because power
// bounds it, a wait costs little by itself: with workgroups started out of step, so that the bursts of stores between
// tiles meet others' products, that call took 2 % longer.  What the form costs: log-probs of d_model 64, whose second K step
// does not exist and is multiplied as zeros, take 3 to 9 % longer than before (32768 x 4096: 78 and 85 us; products
// left out behind the loop, 82, but those of d_model 5120 then took 1 % more).

#include <algorithm>
#include <type_traits>

#include "lm_plan.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int LM_THREADS = 512;                      // 8 wavefronts, two per SIMD
constexpr int LM_WM = 2, LM_WN = 4;                  // wavefront grid over the tile
constexpr int LM_FA = 8, LM_FB = 4;                  // 16 x 16 blocks per wavefront: 128 x 64
constexpr int LM_CPR = LM_BK / 8;                    // 16-byte chunks per tile row: 8
constexpr int LM_TILE_BYTES = LM_BM * LM_BK * 2;     // one operand tile: 32 KB
constexpr int LM_SLOTS = 5;                          // operand tiles resident in LDS: all 160 KB
constexpr int LM_LPT = LM_BM * LM_CPR / LM_THREADS;  // 16-byte loads per lane and operand tile: 4
constexpr int LM_LDS_BYTES = LM_SLOTS * LM_TILE_BYTES;

constexpr int LM_CHUNK_MAX = 1 << 20;  // rows of a chunk; keeps every per-chunk grid extent and 32-bit offset in range
constexpr int LM_LEAD_STEPS = 16;                     // contractions of up to so many K steps: see lm_gemm_nt

enum { LM_EPI_LSE = 0, LM_EPI_BF16 = 1, LM_EPI_F32 = 2 };
enum { LM_Z_NONE = 0, LM_Z_KEPT = 1, LM_Z_LARGE = 2 };  // the fp32 copy of the logits: none, stored, stored past the caches

struct GemmParams {
    const __bf16 *A;
    const __bf16 *B;
    long long lda, ldb;  // elements; rows 16-byte aligned
    int M, N, K;         // host-side sizes: M and K are upper bounds when the device values below are given
    const int *M_dev;    // optional: number of rows of A actually present (<= M)
    int chunk, chunk_cap;  // chunk_cap > 0: *M_dev counts the rows of ALL chunks and this launch works on chunk
                           // number `chunk` of them (lm_chunk_range): A, tokens32 and zy start at the
                           // chunk's first row, the partials and Z are the chunk's own
    const int *K_dev;    // optional: length of the contraction actually present, rounded up to LM_BK
                         // in the kernel (the padding must hold zeros); 0 gives a zero result
    int tiles_n;
    // LM_EPI_BF16 / LM_EPI_F32
    void *C;
    long long ldc;
    const int *c_rows;   // LM_EPI_BF16, optional: row i of the result goes to row c_rows[i] of C
    // LM_EPI_BF16, optional split of the contraction (split_items > 0): the tiles that do not fill
    // a whole round of the CUs are cut into parts along K (lm_plan, from the live row count);
    // part s of the t-th such tile goes as a 256 x 256 fp32 block to split_ws[t * parts + s] and
    // lm_split_reduce finishes.  split_items: how many such blocks split_ws holds.
    int split_items, n_cu;
    float *split_ws;
    int accumulate;      // LM_EPI_F32: C += result
    // LM_EPI_LSE
    const int *tokens32; // [M]: sampled token of each row of A
    float k;             // log2(e) / T
    float *part_m, *part_s;  // [tiles_n][part_stride]: max of z over the tile's columns and sum of exp2((z - max) k), y left out
    float *part_w;           // with the auxiliary terms: sum of exp2(a) a, a = (z - max) k, over the same columns
    long long part_stride;
    float *zy;               // [M]: the accumulator at the sampled token's column
    float *Z;                // optional fp32 copy of the logits: lm_z_part
    long long ldz;
    // K-major operands (AKM / BKM: stored [K][M] resp. [K][N], contiguous along M resp. N, lda / ldb between
    // k rows): how many elements of a k row exist (a multiple of 8; chunks past them re-read the last one)
    int a_cols, b_cols;
    // K-major B: how many k rows exist (K or fewer).  The rows past them read
    // as zeros: the buffer descriptor of the last K step ends with the last row that exists, and a load
    // past a descriptor's end puts zeros into LDS (measured on gfx950).
    int b_rows;
};

// A K-major operand tile in LDS is [64 k][256 m] bf16, 512 bytes per k row.  The 16-byte chunk at
// position pc of row k holds logical chunk pc ^ lm_km_swizzle(k) (applied on the global-address side):
// a transposing fragment read touches rows k .. k + 3 (and k + 8 .. k + 11 in the other half of the
// wavefront), 64 bytes of each, and with the swizzle those land on different banks.
__device__ __forceinline__ int lm_km_swizzle(int k) { return (4 * (k & 3)) ^ (2 * ((k >> 3) & 1)); }

// Which column of the tile lies in row r of B's operand tile in LDS.  For fp32 results the 64 columns of a wavefront
// are dealt so that a lane, which holds column lane % 16 of every block of 16 columns, has four neighbouring ones:
// its 16-byte stores and those of its neighbours make whole lines.
template <int EPI>
__device__ __forceinline__ int lm_column_of(int r)
{
    return EPI == LM_EPI_F32 ? (r & ~63) | ((r & 15) << 2) | ((r >> 4) & 3) : r;
}

// Where entry (row, col) of the fp32 logits of a chunk lies in Z (in floats, a multiple of 4; col a multiple of 4).  Z is kept
// the way the accumulators are: for each part of 128 rows x 64 columns, 8 x 4 blocks of 16 x 16, in a block 16 bytes per
// lane, lane = row % 16 + 16 (col % 16 / 4).  A wavefront stores 1 KB at a time, whole; written by rows, every lane's
// 16 bytes went to another line: 7 us of a CU's time for a tile, now 2.  The space is rows (a multiple of 128) x ldz.
__device__ __forceinline__ long long lm_z_part(int row, int col, long long ldz)
{
    return ((long long)(row >> 7) * (ldz >> 6) + (col >> 6)) * (128 * 64);
}
__device__ __forceinline__ int lm_z_in_part(int row, int col)
{
    return ((((row >> 4) & 7) * 4 + ((col >> 4) & 3)) * 64 + (row & 15) + 16 * ((col >> 2) & 3)) * 4;
}

template <int EPI, int Z, bool AUX = false, bool AKM = false, bool BKM = false, bool LEAD = false>
__global__ void __launch_bounds__(LM_THREADS) lm_gemm_nt(GemmParams p)
{
    extern __shared__ __attribute__((aligned(1024))) char lm_smem[];
    int M = p.M_dev ? min(*p.M_dev, p.M) : p.M;
    int chunk_base = 0;  // first row of this launch's chunk in A, tokens32 and zy
    if (p.chunk_cap > 0) {
        int count;
        lm_chunk_range(*p.M_dev, p.chunk_cap, p.chunk, chunk_base, count);
        M = min(count, p.M);
    }
    const int K = p.K_dev ? min((*p.K_dev + LM_BK - 1) / LM_BK * LM_BK, p.K) : p.K;
    if (EPI == LM_EPI_F32 && p.accumulate && K == 0) return;  // nothing to add (an empty chunk)
    const LmPlan pl = lm_plan(M, p.tiles_n, K / LM_BK, EPI == LM_EPI_BF16 && p.split_items > 0, p.split_items, p.n_cu);
    // The workgroups stay: the grid has one for each CU (all of its LDS), workgroup b takes the items b / 8,
    // b / 8 + grid / 8, ... of XCD b % 8's list - the order in which one workgroup per item would be
    // dispatched - and its loads run ahead into the next item (below).
    const int xcd = (int)(blockIdx.x & 7), per_xcd = (int)(gridDim.x >> 3), n_items = lm_items_per_xcd(pl);
    int idx = (int)(blockIdx.x >> 3);
    // Of short contractions a workgroup takes the half or thin tile at the end of its places first: workgroups that have one then
    // store their tiles while the others multiply.  In step, 256 of them store 64 MB at once, as long as 6 K steps, and multiply
    // with the memory idle (1024 x 50304 x 768 with the auxiliary terms 311 -> 295 us a call, 4096 x 32000 x 256 347 ->
    // 331, 1500 x 30000 x 640 258 -> 246).  Of long ones it is the operands that count, which neighbouring tiles share
    // while they are in step (log-probs of 2048 x 152064 x 5120 1682 us, 1704 with it); even the possibility costs the
    // logits' 0.5 %, so it is an instantiation of its own (LEAD).
    int lead = -1, idx_end = n_items;  // the place taken first, if any, and where the others end
    if (LEAD && K <= LM_LEAD_STEPS * LM_BK && idx < n_items) {
        const int last = idx + (n_items - 1 - idx) / per_xcd * per_xcd;
        if (last > idx && last >= (pl.full + 7) / 8) lead = last, idx_end = last;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // in a scalar register: LDS targets are uniform
    const int wm = wave / LM_WN, wn = wave % LM_WN;  // this wavefront's 128 x 64 part of the tile

    // The item being loaded: its tile, its part of the contraction (K steps [kt0, kt0 + KT)) and the addresses of its
    // loads.  Byte offsets of this lane's four 16-byte loads per operand tile, relative to the
    // tile's first row at k = 0.  Load i of a wavefront fills LDS chunks [i*512 + wave*64,
    // +64) of the tile; chunk c sits in tile row c / 8 at physical position c % 8 and holds
    // logical chunk (c % 8) ^ ((row >> 1) & 7).  Rows past the item's last re-read that
    // row (their results are never stored).
    LmItem item = {};
    int L = 0, L_end = 0, tm = 0, group_row0 = 0, group_rows = 1, step_m = 0, step_n = 0;  // its place among the whole tiles
    int kt0 = 0, KT = 0;
    unsigned a_off[LM_LPT], b_off[LM_LPT];
    const char *a_tile = nullptr, *b_tile = nullptr;
    const long long a_kstep = (long long)LM_BK * p.lda * 2, b_kstep = (long long)LM_BK * p.ldb * 2;  // K-major only
    // takes this workgroup's next item, from position idx on; false: none is left
    auto next_item = [&]() __attribute__((always_inline)) -> bool {
        if (L + per_xcd < L_end) {  // the next whole tile of the same group of tile rows: per_xcd further on, no division
            L += per_xcd;
            tm += step_m;
            item.tn += step_n;
            if (tm >= group_rows) {
                tm -= group_rows;
                ++item.tn;
            }
            item.row0 = (group_row0 + tm) * LM_BM;
            idx += per_xcd;
        } else if (item.pair) {
            item.pair = 0;
            ++item.tn;
        } else {
            LmItem it;
            int at;
            for (;; idx += per_xcd) {
                if (LEAD && lead >= 0) {
                    at = lead;
                    lead = -1;
                    idx -= per_xcd;  // the first place is still to come
                } else {
                    if (idx >= idx_end) {  // whole workgroup alike
                        KT = 0;  // the loads that still follow find no step and touch no memory
                        return false;
                    }
                    at = idx;
                }
                if (lm_map_item(xcd, at, p.tiles_n, pl, it)) break;
            }
            item = it;
            const int n1 = (pl.full + 7) / 8;
            L_end = 0;
            if (at < n1) {
                const int group_tiles = LM_GROUP_M * p.tiles_n;
                L = xcd * n1 + at;
                group_row0 = L / group_tiles * LM_GROUP_M;
                group_rows = min(LM_GROUP_M, pl.rows_w - group_row0);
                L_end = min(min(pl.full, (xcd + 1) * n1), (L / group_tiles + 1) * group_tiles);
                tm = it.row0 / LM_BM - group_row0;
                step_n = per_xcd / group_rows;
                step_m = per_xcd - step_n * group_rows;
            }
            idx += per_xcd;
        }
        const LmItem &it = item;
        const int row0 = it.row0, col0 = it.tn * LM_BN, row_end = min(M, row0 + it.height);
        int t = tid;  // opaque: what follows from it is computed again for each item, not kept in registers
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int i = 0; i < LM_LPT; ++i) {
            const int c = i * LM_THREADS + t;
            const int r = c / LM_CPR, pc = c % LM_CPR;
            const int lc = pc ^ ((r >> 1) & (LM_CPR - 1));
            const int ra = min(row0 + r, row_end - 1) - row0;
            const int rb = min(col0 + lm_column_of<EPI>(r), p.N - 1) - col0;
            // K-major operand: the tile is [64 k rows][256 m]; chunk c is k row c / 32 at position c % 32 and holds
            // logical chunk (c % 32) ^ lm_km_swizzle(k row); chunks past the item's last row or the end of the
            // operand's k row re-read the last chunk (they belong to rows or columns of C that are never stored)
            const int kk = c >> 5, lck = (c & 31) ^ lm_km_swizzle(kk);
            if constexpr (AKM) {
                const int ch = min((row0 >> 3) + lck, (min(row_end + 7, p.a_cols) >> 3) - 1) - (row0 >> 3);
                a_off[i] = (unsigned)((long long)kk * p.lda * 2 + ch * 16);
            } else {
                a_off[i] = (unsigned)(((long long)ra * p.lda + lc * 8) * 2);
            }
            if constexpr (BKM) {
                const int ch = min((col0 >> 3) + lck, (p.b_cols >> 3) - 1) - (col0 >> 3);
                b_off[i] = (unsigned)((long long)kk * p.ldb * 2 + ch * 16);
            } else {
                b_off[i] = (unsigned)(((long long)rb * p.ldb + lc * 8) * 2);
            }
        }
        // K / LM_BK < 2^17 where there are parts (at most 64): see lm_bwd_vocab_ok
        kt0 = it.parts > 1 ? (int)((unsigned)(K / LM_BK) * (unsigned)it.part / (unsigned)it.parts) : 0;
        KT = (it.parts > 1 ? (int)((unsigned)(K / LM_BK) * (unsigned)(it.part + 1) / (unsigned)it.parts) : K / LM_BK) - kt0;
        a_tile = AKM ? (const char *)p.A + ((long long)kt0 * LM_BK * p.lda + row0) * 2
                     : (const char *)p.A + ((long long)(chunk_base + row0) * p.lda + (long long)kt0 * LM_BK) * 2;
        b_tile = BKM ? (const char *)p.B + ((long long)kt0 * LM_BK * p.ldb + col0) * 2
                     : (const char *)p.B + ((long long)col0 * p.ldb + (long long)kt0 * LM_BK) * 2;
        return true;
    };
    if (!next_item()) return;  // before any barrier

    // LDS is a ring of five 32 KB slots that operand tiles pass through in the order
    // A(0), B(0), A(1), B(1), ..., from item to item without a break: behind the last K step of one item come the
    // first ones of the next.  Two slots hold the step being multiplied, two the next step, and the fifth
    // takes A of the step after that; its B goes where the current A was.  An item takes two steps at least
    // (steps that its contraction does not have read zeros), so that the loads never run further ahead than
    // the next item.  `slot` is where A of the current step lies.
    int slot = 0;
    auto slot_at = [&](int ahead) __attribute__((always_inline)) -> int {  // slot + ahead, ahead < 5
        int q = slot + ahead;
        if (q >= LM_SLOTS) q -= LM_SLOTS;
        return q * LM_TILE_BYTES;
    };
    // The loads are buffer loads with LDS as their target: the tile's first row at this
    // item's first K step is the buffer's base, the lane's offset inside the tile a
    // vector register, the K position a scalar one, the LDS address goes through M0 - no
    // vector arithmetic per load.  The range check of the buffer is left wide open (rows are
    // clamped above, so every address of a step that exists is inside the operand), shut for a step that does not
    // exist, and ends with the last row there is in a ragged last step of a K-major B.
    // A K-major operand moves by whole k rows from step to step, further than a 32-bit offset reaches:
    // its descriptor is made again for every step (scalar arithmetic).
    struct Source {
        const char *base;
        unsigned bytes;
        int k0;
    };
    auto source_of = [&](bool b_operand, int kt) __attribute__((always_inline)) -> Source {
        unsigned bytes = kt < KT ? 0xfffffff0u : 0u;  // (as -1 the select would become a vector instruction)
        if (b_operand && BKM) {
            const int left = kt < KT ? p.b_rows - (kt0 + kt) * LM_BK : 0;  // rows of B from this step on
            const unsigned edge = left > 0 ? (unsigned)(left - 1) * (unsigned)(p.ldb * 2) + (unsigned)(p.b_cols - item.tn * LM_BN) * 2u : 0u;
            bytes = left >= LM_BK ? 0xfffffff0u : edge;
        }
        const bool km = b_operand ? BKM : AKM;
        const char *base = (b_operand ? b_tile : a_tile) + (km ? kt * (b_operand ? b_kstep : a_kstep) : 0);
        return {base, bytes, km ? 0 : kt * (LM_BK * 2)};
    };
    auto issue_load = [&](const Source &src, bool b_operand, int at, int i) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)src.base, 0, (int)src.bytes, 0x00020000);
        const int k0 = src.k0;  // (given as a member, the compiler's host pass drops the kernel)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc, (__attribute__((address_space(3))) void *)(lm_smem + at + wave * 1024 + i * (LM_THREADS * 16)), 16,
            (int)(b_operand ? b_off[i] : a_off[i]), k0, 0, 0);
    };

    // Fragment addresses.  Lane (r = lane % 16, g = lane / 16) holds, for the 16 x 16 x 32 product, the 8 consecutive
    // k from 8 g on of row r of a 16-row block: logical chunk 4 ks + g of that tile row, for half ks of the step.
    const int fr = lane & 15, fg = lane >> 4;
    const unsigned frag0 = (unsigned)((fr * LM_CPR + (fg ^ ((fr >> 1) & (LM_CPR - 1)))) * 16);  // half 1: ^ 64
    // K-major tiles are read with the transposing 64-bit LDS read: lane i of a group of 16 lanes gives the
    // address of 4 consecutive m at k row i / 4 (piece i % 4 of 16 m) and receives the 4 k values of m = i.
    // Two such reads (k rows +0..3 and +4..7) make a lane's 8 consecutive k; group g of 16 lanes has the k rows from
    // 8 g on.  Block i is 32 i bytes further on inside a k row: bits that the swizzle of the chunks only flips.
    unsigned akm0, bkm0;
    {
        const int kkl = 8 * fg + (fr >> 2), sw = lm_km_swizzle(kkl);
        akm0 = (unsigned)(kkl * (LM_BM * 2) + (((wm * (LM_FA * 2) + ((fr & 3) >> 1)) ^ sw) * 16) + (fr & 1) * 8);
        bkm0 = (unsigned)(kkl * (LM_BN * 2) + (((wn * (LM_FB * 2) + ((fr & 3) >> 1)) ^ sw) * 16) + (fr & 1) * 8);
    }
    // Written as assembly: the compiler holds the builtin form of this read back behind every outstanding
    // load to LDS (s_waitcnt vmcnt(0) in front of each half's reads), which the pipeline below exists to
    // avoid.  The results arrive asynchronously; every use sits behind an explicit lgkmcnt(0).
    auto tr_frag = [&](unsigned at) __attribute__((always_inline)) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        s16x4 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:2048"
                     : "=&v"(lo), "=&v"(hi)
                     : "v"(at)
                     : "memory");
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    static_assert(4 * (LM_BM * 2) == 2048, "the second read's offset is written into the assembly");
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)lm_smem;

    f32x4 acc[LM_FA][LM_FB];

    // Fragments are double buffered in registers (F[0], F[1]) and read one half step ahead of the products that use
    // them: B's, then A's.  One barrier per step, in its middle: by then every wavefront holds the second half's
    // fragments in registers, so the step's two slots are free, and everybody's loads of the next step have landed.
    bf16x8 F[2][LM_FB + LM_FA];
    auto read_frag = [&](int f, int at_a, int at_b, int ks) __attribute__((always_inline)) -> bf16x8 {
        if (f < LM_FB) {
            if constexpr (BKM)
                return tr_frag((lds0 + at_b + ks * (32 * LM_BN * 2) + bkm0) ^ (f * 32));
            else
                return *(const bf16x8 *)(lm_smem + at_b + wn * (LM_FB * 16 * LM_BK * 2) + (frag0 ^ (ks * 64)) + f * (16 * LM_BK * 2));
        }
        if constexpr (AKM)
            return tr_frag((lds0 + at_a + ks * (32 * LM_BM * 2) + akm0) ^ ((f - LM_FB) * 32));
        else
            return *(const bf16x8 *)(lm_smem + at_a + wm * (LM_FA * 16 * LM_BK * 2) + (frag0 ^ (ks * 64)) +
                                     (f - LM_FB) * (16 * LM_BK * 2));
    };
    auto lds_landed = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) and nothing else
        __builtin_amdgcn_sched_barrier(0);
    };
    // One half step: the products of the fragments in `f`, the reads of the next half's into `nf` and the loads of one
    // operand tile dealt out between them.  A block row of A goes through the columns of B to and fro, so that
    // consecutive products share an operand.  Which operand comes first says what a lane holds of a 16 x 16 block of C:
    // A: column lane % 16, rows 4 (lane / 16) + v (fp32 results); B: row lane % 16, columns 4 (lane / 16) + v (the others).
    auto half_step = [&](const bf16x8 (&f)[LM_FB + LM_FA], bf16x8 (&nf)[LM_FB + LM_FA], int next_a, int next_b, int next_ks,
                         bool b_operand, int load_at, int load_kt) __attribute__((always_inline)) {
        const Source src = source_of(b_operand, load_kt);
#pragma unroll
        for (int i = 0; i < LM_FA; ++i) {
            if (2 * i < LM_FB + LM_FA) {
                nf[2 * i] = read_frag(2 * i, next_a, next_b, next_ks);
                nf[2 * i + 1] = read_frag(2 * i + 1, next_a, next_b, next_ks);
            }
            if (i < LM_LPT) issue_load(src, b_operand, load_at, i);
#pragma unroll
            for (int jj = 0; jj < LM_FB; ++jj) {
                if (jj == 0) __builtin_amdgcn_s_setprio(1);
                if (jj == LM_FB - 1) __builtin_amdgcn_s_setprio(0);
                const int j = i % 2 ? LM_FB - 1 - jj : jj;
                if constexpr (EPI == LM_EPI_F32)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[LM_FB + i], f[j], acc[i][j], 0, 0, 0);
                else
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j], f[LM_FB + i], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    static_assert(LM_BM == 256 && LM_BN == 256, "K-major tiles: 32 chunks per k row");
    static_assert(LM_BK == 64 && LM_SLOTS == 5 && LM_LPT == 4 && LM_FA == 8 && LM_FB == 4,
                  "the pipeline and its wait counts are written for two halves, 5 slots, 4 loads per operand tile");

    // Memory operations retire in order, so "at most n outstanding" means that everything older
    // than the n youngest is done.  The wait, the wait for the own LDS reads and the
    // workgroup barrier are one asm statement so that nothing is scheduled in between.
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const Source src = source_of(q & 1, q >> 1);
#pragma unroll
        for (int i = 0; i < LM_LPT; ++i) issue_load(src, q & 1, q * LM_TILE_BYTES, i);
    }
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // A(0), B(0)
#pragma unroll
    for (int f = 0; f < LM_FB + LM_FA; ++f) F[0][f] = read_frag(f, slot_at(0), slot_at(1), 0);
    lds_landed();
    bool landed = false;  // the next step's loads are known to have landed without a wait
    int load_kt = 2;      // K step of the item being loaded that is loaded next

    for (;;) {
        // the item being multiplied
        const int row0 = item.row0, col0 = item.tn * LM_BN, part = item.part, parts = item.parts, block = item.block;
        const int rows_here = min(item.height, M - row0);
        const int steps = max(KT, 2);
        const bool active = wm * (LM_FA * 16) < rows_here;  // else this wavefront's part has no row that exists
        const int wrow = wm * (LM_FA * 16), wcol = wn * (LM_FB * 16);
        int tok0 = 0, tok1 = 0;  // sampled tokens of rows `lane` and 64 + `lane` of the wavefront's part
        if constexpr (EPI == LM_EPI_LSE) {
            tok0 = p.tokens32[chunk_base + min(row0 + wrow + lane, M - 1)];
            tok1 = p.tokens32[chunk_base + min(row0 + wrow + 64 + lane, M - 1)];
        }
#pragma unroll
        for (int i = 0; i < LM_FA; ++i)
#pragma unroll
            for (int j = 0; j < LM_FB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        bool more = false;
        auto landed_barrier = [&]() __attribute__((always_inline)) {
            // outstanding, oldest first: ..., A and B of the next step, A of the one after: 4 left = the next step landed
            if (landed)
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else
                asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            landed = false;
        };
        if (active) {
            for (int kt = 0; kt < steps; ++kt) {
                if (kt == steps - 2) {  // from here on the loads are the next item's
                    more = next_item();
                    load_kt = 0;
                }
                half_step(F[0], F[1], slot_at(0), slot_at(1), 1, false, slot_at(4), load_kt);
                landed_barrier();
                lds_landed();  // (for the compiler, which does not look into the statement above)
                half_step(F[1], F[0], slot_at(2), slot_at(3), 0, true, slot_at(0), load_kt);
                lds_landed();
                ++load_kt;
                slot += 2;
                if (slot >= LM_SLOTS) slot -= LM_SLOTS;
            }
        } else {
            for (int kt = 0; kt < steps; ++kt) {
                if (kt == steps - 2) {
                    more = next_item();
                    load_kt = 0;
                }
                const Source a_src = source_of(false, load_kt), b_src = source_of(true, load_kt);
#pragma unroll
                for (int i = 0; i < LM_LPT; ++i) issue_load(a_src, false, slot_at(4), i);
                landed_barrier();
#pragma unroll
                for (int i = 0; i < LM_LPT; ++i) issue_load(b_src, true, slot_at(0), i);
                ++load_kt;
                slot += 2;
                if (slot >= LM_SLOTS) slot -= LM_SLOTS;
            }
#pragma unroll
            for (int f = 0; f < LM_FB + LM_FA; ++f) F[0][f] = read_frag(f, slot_at(0), slot_at(1), 0);
            lds_landed();
        }

        // The result is stored while the next item's first two steps are on their way: they have landed when no more
        // operations are outstanding than the stores issued since.
        auto loads_landed = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
        auto loads_landed_behind_stores = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(32)" ::: "memory"); };
        landed = true;
        int ln = lane;  // opaque, as above
        asm volatile("" : "+v"(ln));
        const int n = ln & 15, g = ln >> 4;  // this lane's place in a block, see half_step
        // the wavefront's part as the accumulators lie, 1 KB a store
        auto store_blocks = [&](float *base, auto nontemporal) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < LM_FA; ++i)
#pragma unroll
                for (int j = 0; j < LM_FB; ++j) {
                    f32x4 *at = (f32x4 *)(base + ((i * LM_FB + j) * 64 + ln) * 4);
                    if constexpr (decltype(nontemporal)::value)
                        __builtin_nontemporal_store(acc[i][j], at);
                    else
                        *at = acc[i][j];
                }
        };

        if constexpr (EPI == LM_EPI_F32) {
            if (!active || col0 + wcol >= p.N) {  // N is a multiple of 64: a part's columns are all inside or all outside
                loads_landed();
            } else {
                // this lane's columns 4 n .. 4 n + 3 (see lm_column_of), rows 16 i + 4 g + v
                float *cw = (float *)p.C + (long long)(row0 + wrow) * p.ldc + col0 + wcol;
                const int rows = min(rows_here - wrow, LM_FA * 16);
                const unsigned voff = (unsigned)((4 * g * p.ldc + 4 * n) * 4);
                if ((((unsigned long long)p.C | (unsigned long long)(p.ldc * 4)) & 15u) != 0 || p.ldc >= (1ll << 26)) {
                    // C itself not in whole 16-byte pieces: element by element
#pragma unroll
                    for (int i = 0; i < LM_FA; ++i)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int r = i * 16 + 4 * g + v;
                            if (r >= rows) continue;
                            float *at = cw + (long long)r * p.ldc + 4 * n;
#pragma unroll
                            for (int j = 0; j < LM_FB; ++j) at[j] = p.accumulate ? at[j] + acc[i][j][v] : acc[i][j][v];
                        }
                    loads_landed();
                } else if (p.accumulate) {
                    // C += result: all loads of two block rows first, then the sums and stores (a dependent load in
                    // front of every store made this epilogue take 2 ms longer than the plain store)
#pragma unroll
                    for (int i = 0; i < LM_FA; i += 2) {
                        f32x4 old[8];
                        char *at = (char *)(cw + (long long)i * 16 * p.ldc);
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            old[q] = (i + q / 4) * 16 + 4 * g + q % 4 < rows
                                         ? *(const f32x4 *)(at + ((q / 4) * 16 + q % 4) * (p.ldc * 4) + voff)
                                         : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
#pragma unroll
                            for (int j = 0; j < LM_FB; ++j) old[q][j] += acc[i + q / 4][j][q % 4];
                            if ((i + q / 4) * 16 + 4 * g + q % 4 < rows)
                                __builtin_nontemporal_store(old[q], (f32x4 *)(at + ((q / 4) * 16 + q % 4) * (p.ldc * 4) + voff));
                        }
                    }
                    loads_landed();
                } else {
#pragma unroll
                    for (int i = 0; i < LM_FA; ++i)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            if (rows < LM_FA * 16 && i * 16 + 4 * g + v >= rows) continue;
                            __builtin_nontemporal_store(f32x4{acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]},
                                                        (f32x4 *)((char *)cw + (i * 16 + v) * (p.ldc * 4) + voff));
                        }
                    if (rows == LM_FA * 16)
                        loads_landed_behind_stores();  // 32 of them
                    else
                        loads_landed();
                }
            }
        }
        if constexpr (EPI == LM_EPI_BF16) {
            if (!active || col0 + wcol >= p.N) {
                loads_landed();
            } else if (parts > 1) {
                // read only where rows and columns exist: stored whole
                store_blocks(p.split_ws + ((long long)block << 16) + wave * (LM_FA * LM_FB * 256), std::false_type{});
                loads_landed_behind_stores();
            } else {
                const bool quads = (((unsigned long long)p.C | (unsigned long long)(p.ldc * 2)) & 7u) == 0;
#pragma unroll
                for (int i = 0; i < LM_FA; ++i) {
                    const int r = wrow + i * 16 + n;
                    if (r >= rows_here) continue;
                    const long long orow = p.c_rows ? p.c_rows[row0 + r] : row0 + r;
                    __bf16 *at = (__bf16 *)p.C + orow * p.ldc + col0 + wcol + 4 * g;
#pragma unroll
                    for (int j = 0; j < LM_FB; ++j) {
                        const bf16x2 lo = __builtin_convertvector((f32x2){acc[i][j][0], acc[i][j][1]}, bf16x2);
                        const bf16x2 hi = __builtin_convertvector((f32x2){acc[i][j][2], acc[i][j][3]}, bf16x2);
                        if (quads) {
                            *(u32x2 *)(at + j * 16) = u32x2{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
                        } else {
                            at[j * 16] = lo[0];
                            at[j * 16 + 1] = lo[1];
                            at[j * 16 + 2] = hi[0];
                            at[j * 16 + 3] = hi[1];
                        }
                    }
                }
                loads_landed();
            }
        }
        if constexpr (EPI == LM_EPI_LSE) {
            // Softmax partials of this tile: for every row the maximum of z over the tile's
            // columns and the sum of exp2((z - max) k), the sampled token's column left out of both
            // (its accumulator goes to zy instead) so that 1 - p_y keeps its precision later.
            //
            // A lane holds 16 of a row's 64 columns in this wavefront's part, the four lanes n, n + 16, n + 32, n + 48 the
            // whole of them: two exchanges finish a row, and no accumulator passes through LDS.  Only the partials of
            // the four wavefronts that share a row meet there, in the one slot of the ring that is free between two items.
            float *red_m = (float *)(lm_smem + slot_at(4));  // [LM_WN][256]
            float *red_s = red_m + LM_WN * LM_BM;
            float *red_w = red_s + LM_WN * LM_BM;
            static_assert(3 * LM_WN * LM_BM * 4 <= LM_TILE_BYTES, "the partials fit the free slot");
            if (active) {
                const int ncols = max(0, min(LM_FB * 16, p.N - col0 - wcol));  // columns of this part inside the matrix
                // the columns of the sampled tokens inside this part: mostly nowhere
                const unsigned y0 = (unsigned)(tok0 - col0 - wcol), y1 = (unsigned)(tok1 - col0 - wcol);
                const bool y_here = __any(y0 < (unsigned)ncols || y1 < (unsigned)ncols);
                auto both = [](float a, auto op) __attribute__((always_inline)) {  // op over lanes n, n + 16, n + 32, n + 48
                    // (the bits go through scalars: of an element of a vector, __builtin_bit_cast takes the first one)
                    auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, a),
                                                              false, false);
                    unsigned u0 = q[0], u1 = q[1];
                    a = op(__builtin_bit_cast(float, u0), __builtin_bit_cast(float, u1));
                    q = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, a), false,
                                                         false);
                    u0 = q[0], u1 = q[1];
                    return op(__builtin_bit_cast(float, u0), __builtin_bit_cast(float, u1));
                };
                auto add = [](float a, float b) __attribute__((always_inline)) { return a + b; };
                auto larger = [](float a, float b) __attribute__((always_inline)) { return fmaxf(a, b); };
                float out_m[2] = {0.f, 0.f}, out_s[2] = {0.f, 0.f}, out_w[2] = {0.f, 0.f};
#pragma unroll
                for (int i = 0; i < LM_FA; ++i) {
                    float z[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) z[e] = acc[i][e >> 2][e & 3];
                    if (y_here) {
                        const int yc = (int)__shfl(i < 4 ? y0 : y1, 16 * (i & 3) + n, 64);
                        // the sampled token's place among this lane's 16 columns
                        const int at = (unsigned)yc < (unsigned)ncols && ((yc >> 2) & 3) == g ? 4 * (yc >> 4) + (yc & 3) : -1;
                        if (__any(at >= 0)) {
                            const int r = row0 + wrow + i * 16 + n;
                            float zy = 0.f;
#pragma unroll
                            for (int e = 0; e < 16; ++e) {
                                zy = e == at ? z[e] : zy;
                                z[e] = e == at ? -INFINITY : z[e];
                            }
                            if (at >= 0 && r < M) p.zy[chunk_base + r] = zy;
                        }
                    }
                    if (ncols < LM_FB * 16) {
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if (16 * (e >> 2) + (e & 3) >= ncols - 4 * g) z[e] = -INFINITY;
                    }
                    float mz = fmaxf(z[0], z[1]);
#pragma unroll
                    for (int e = 2; e < 16; e += 2) mz = fmaxf(fmaxf(mz, z[e]), z[e + 1]);
                    mz = both(mz, larger);
                    float s0 = 0.f, s1 = 0.f, w0 = 0.f, w1 = 0.f;
                    if constexpr (AUX) {
                        // exponents (z - max) k, exactly 0 at the maximum: the entropy gradient of a near-one-hot
                        // row depends on it (see row_scalars_aux); elements at -inf contribute 0, not 0 * inf
                        const float refz = mz == -INFINITY ? 0.f : mz;
#pragma unroll
                        for (int e = 0; e < 16; e += 2) {
                            const float a0 = (z[e] - refz) * p.k, a1 = (z[e + 1] - refz) * p.k;
                            const float e0 = __builtin_amdgcn_exp2f(a0), e1 = __builtin_amdgcn_exp2f(a1);
                            s0 += e0;
                            s1 += e1;
                            w0 = fmaf(e0, fmaxf(a0, kExpFloor), w0);
                            w1 = fmaf(e1, fmaxf(a1, kExpFloor), w1);
                        }
                        w0 = both(w0 + w1, add);
                    } else {
                        const float ref = mz == -INFINITY ? 0.f : mz * p.k;  // 0 for a row with nothing to sum
#pragma unroll
                        for (int e = 0; e < 16; e += 2) {
                            s0 += __builtin_amdgcn_exp2f(fmaf(z[e], p.k, -ref));
                            s1 += __builtin_amdgcn_exp2f(fmaf(z[e + 1], p.k, -ref));
                        }
                    }
                    s0 = both(s0 + s1, add);
                    if (g == (i & 3)) {  // lane 16 g + n keeps rows `lane` and 64 + `lane` of the part
                        out_m[i >> 2] = mz;  // in units of z
                        out_s[i >> 2] = s0;
                        out_w[i >> 2] = w0;
                    }
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    red_m[wn * LM_BM + wrow + q * 64 + ln] = out_m[q];
                    red_s[wn * LM_BM + wrow + q * 64 + ln] = out_s[q];
                    if constexpr (AUX) red_w[wn * LM_BM + wrow + q * 64 + ln] = out_w[q];
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (tid < rows_here) {  // at most 256
                const int row = row0 + tid;
                float m = -INFINITY;
#pragma unroll
                for (int w = 0; w < LM_WN; ++w) m = fmaxf(m, red_m[w * LM_BM + tid]);
                float s = 0.f, ws = 0.f;
#pragma unroll
                for (int w = 0; w < LM_WN; ++w) {
                    const float mw = red_m[w * LM_BM + tid], sw = red_s[w * LM_BM + tid];
                    if (mw != -INFINITY) {
                        const float d = (mw - m) * p.k;  // <= 0; exactly 0 for the part that holds the maximum
                        const float f = __builtin_amdgcn_exp2f(d);
                        s = fmaf(sw, f, s);
                        if constexpr (AUX) ws = fmaf(f, fmaf(d, sw, red_w[w * LM_BM + tid]), ws);
                    } else {
                        s += sw;  // a part without a number: 0, or NaN, which the maximum has skipped
                    }
                }
                p.part_m[(long long)(col0 / LM_BN) * p.part_stride + row] = m;
                p.part_s[(long long)(col0 / LM_BN) * p.part_stride + row] = s;
                if constexpr (AUX) p.part_w[(long long)(col0 / LM_BN) * p.part_stride + row] = ws;
            }
            // the slot is free again for the next item's loads when every wavefront has read its partials
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            loads_landed();
            // the fp32 copy of the logits, rows past the last one and the columns between N and the row pitch of Z with the
            // products of the clamped operand rows: never read
            if (Z != LM_Z_NONE && active && col0 + wcol < p.ldz) {  // ldz < 2^23: see lm_bwd_vocab_ok
                float *at = p.Z + lm_z_part(row0 + wrow, col0 + wcol, p.ldz);
                store_blocks(at, std::bool_constant<Z == LM_Z_LARGE>{});
            }
        }
        if (!more) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads behind the last item write zeros to LDS until they are done
}

// Per-row arrays the fused path keeps between its kernels.  Rows that take part (mask 1,
// token id inside the vocabulary) are compacted: "compact row i" is original row rows[i],
// i < *n_live.  Of those, the ones with a gradient (c != 0) are compacted once more for
// the backward, in order: bit i % 16 of gmask[i / 16] says whether row i of the chunk is one, gradient row j is original row
// orig2[j], j < *n_grad.
// The masked tail of every rollout and the clipped tokens then cost no matrix work at all.
struct LmRows {
    int *rows, *tokens32, *n_live;   // [n], [n] (by compact row), [1]
    int *orig2, *n_grad;             // [cap], [1]
    unsigned *gmask;                 // [cap / 16]
    int *gsum;                       // gradient rows of every LM_SUM_WORDS words of gmask, in chunks of more than LM_SUM_FROM rows
    float *zy;     // by compact row: logit of the sampled token (fp32 accumulator)
    float *shift;  // max k + log2(sum): p_j = exp2(z_j k - shift)
    float *q;      // c / T
    float *gy;     // gradient at the sampled token: q (1 - p_y), from the sum without y
    // with the auxiliary terms: g_j = p_j (q2 + bq a_j), a_j = (z_j - mx) k - log2s = log2 p_j
    float *mx, *log2s, *q2, *bq;
    float *part_m, *part_s, *part_w;  // [tiles_n][part_stride], by row inside the chunk
    long long part_stride;
    int tiles_n;
    int chunk, chunk_cap;  // the chunk of compact rows the per-chunk kernels work on (lm_chunk_range)
};

// Ordered compaction by one workgroup: keeps the indices i < n with keep(i), in order.
// `emit(pos, i)` stores entry number pos; returns the count (in every lane).
template <typename Keep, typename Emit>
__device__ __forceinline__ int lm_ordered_select(long long n, Keep keep, Emit emit)
{
    __shared__ int wave_tot[16];
    __shared__ int base;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) base = 0;
    __syncthreads();
    for (long long i0 = 0; i0 < n; i0 += 1024) {
        const long long i = i0 + tid;
        const int kp = (i < n && keep(i)) ? 1 : 0;
        int incl = kp;  // inclusive scan inside the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane == 63) wave_tot[wv] = incl;
        __syncthreads();
        int before = base;
        for (int w2 = 0; w2 < wv; ++w2) before += wave_tot[w2];
        if (kp) emit(before + incl - 1, i);
        __syncthreads();
        if (tid == 0) {
            int tot = 0;
            for (int w2 = 0; w2 < 16; ++w2) tot += wave_tot[w2];
            base += tot;
        }
        __syncthreads();
    }
    return base;
}

// Rows that take part -> rows[], tokens32[], *n_live; rows that do not get their defined
// outputs here (log-prob 0, or NaN for a bad token id in the log-probs-only call).
__global__ void __launch_bounds__(1024) lm_select_rows(RowParams p, LmRows w)
{
    const int total = lm_ordered_select(
        p.n_tokens,
        [&](long long r) {
            bool live = p.mask ? (p.mask[r] != 0) : true;
            if (live && p.token_w && p.token_w[r] == 0.f) live = false;  // a zero weight masks the row
            bool bad = false;
            if (live) {
                const long long y = p.tokens[r];
                if (y < 0 || y >= p.vocab) {
                    live = false;
                    bad = true;
                }
            }
            if (!live) {
                write_row_outputs(p, r, (bad && !p.bwd) ? NAN : 0.f, 0.f, 0);
                write_row_aux(p, r, 0.f, 0.f);
                if (bad && p.bwd) atomicOr(&p.hdr->error, 1);
            }
            return live;
        },
        [&](int pos, long long r) {
            w.rows[pos] = (int)r;
            w.tokens32[pos] = (int)p.tokens[r];
        });
    if (threadIdx.x == 0) *w.n_live = total;
}

// The same for up to LM_TAKE_MAX tokens, with everything else that happens per row before the first
// product: the hidden states of the rows that take part are copied side by side, and with the backward
// dL/dH is zeroed (rows without gradient keep that) and the header set as grpo_prepare sets it.  A
// workgroup takes 16 rows and counts the rows ahead of its own itself, 9 bytes a row from the caches: more
// reading than one workgroup walking through the batch, but no step waits for another (724 rows: four
// launches of 12 us together, now one of 6; 4096 rows of 5120 values: 53 us before).  Beyond the limit the repeated counting, which
// grows with the square of the batch, would cost more than the walk.
constexpr int LM_TAKE_ROWS = 16, LM_TAKE_THREADS = 512;
constexpr long long LM_TAKE_MAX = 32768;
__global__ void __launch_bounds__(LM_TAKE_THREADS) lm_take_rows(RowParams p, LmRows w, const __bf16 *hidden, long long ldh,
                                                                int d, __bf16 *out, unsigned short *grad_hidden,
                                                                long long ldgh, double denom, WsHeader *hdr)
{
    __shared__ int lds_live[LM_TAKE_THREADS / 64], lds_mask[LM_TAKE_THREADS / 64], lds_pos[LM_TAKE_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const long long r0 = (long long)blockIdx.x * LM_TAKE_ROWS;
    // bit 0: takes part; bit 1: counts towards M (a bad token id does, see grpo_loss_fwd_bwd)
    auto state_of = [&](long long r) -> int {
        const bool on = (!p.mask || p.mask[r] != 0) && (!p.token_w || p.token_w[r] != 0.f);
        if (!on) return 0;
        const long long y = p.tokens[r];
        return y >= 0 && y < p.vocab ? 3 : 2;
    };
    int live_before = 0, mask_before = 0;
#pragma unroll 4
    for (long long r = tid; r < r0; r += LM_TAKE_THREADS) {
        const int st = state_of(r);
        live_before += st & 1;
        mask_before += st >> 1;
    }
    live_before = wave_sum(live_before);
    mask_before = wave_sum(mask_before);
    if (lane == 0) {
        lds_live[wv] = live_before;
        lds_mask[wv] = mask_before;
    }
    const long long r = r0 + lane;
    const int st = (wv == 0 && lane < LM_TAKE_ROWS && r < p.n_tokens) ? state_of(r) : 0;
    __syncthreads();
    int before = 0, mask_all = 0;
#pragma unroll
    for (int i = 0; i < LM_TAKE_THREADS / 64; ++i) {
        before += lds_live[i];
        mask_all += lds_mask[i];
    }
    if (wv == 0) {
        const unsigned long long live = __ballot(st & 1), masked = __ballot(st >> 1);
        const int pos = before + __popcll(live & ((1ull << lane) - 1ull));
        if (lane < LM_TAKE_ROWS) lds_pos[lane] = (st & 1) ? pos : -1;
        if (st & 1) {
            w.rows[pos] = (int)r;
            w.tokens32[pos] = (int)p.tokens[r];
        } else if (lane < LM_TAKE_ROWS && r < p.n_tokens) {
            write_row_outputs(p, r, (st == 2 && !p.bwd) ? NAN : 0.f, 0.f, 0);
            write_row_aux(p, r, 0.f, 0.f);
        }
        if (lane == 0 && blockIdx.x == gridDim.x - 1) {
            const int n_live = before + __popcll(live);
            *w.n_live = n_live;
            if (hdr) {
                const long long M = mask_all + __popcll(masked);
                const double D = denom > 0.0 ? denom : (double)M;
                hdr->D = D;
                hdr->inv_D = D > 0.0 ? 1.0 / D : 0.0;
                hdr->M = M;
                hdr->error = M != n_live ? 1 : 0;  // some unmasked row has a bad token id
                hdr->fin_ticket = 0u;
            }
        }
    }
    __syncthreads();
    const int rows_here = (int)(p.n_tokens - r0 < LM_TAKE_ROWS ? p.n_tokens - r0 : LM_TAKE_ROWS);
    for (int i = wv; i < rows_here; i += LM_TAKE_THREADS / 64) {  // a wavefront to a row
        const int pos = __builtin_amdgcn_readfirstlane(lds_pos[i]);
        if (pos >= 0) {
            const u32x4 *src = (const u32x4 *)(hidden + (r0 + i) * ldh);
            u32x4 *dst = (u32x4 *)(out + (long long)pos * d);
#pragma unroll 4
            for (int c = lane; c < d / 8; c += 64) dst[c] = src[c];
        }
        if (grad_hidden) {
            unsigned short *row = grad_hidden + (r0 + i) * ldgh;
            const u32x4 z = {0u, 0u, 0u, 0u};
            if ((((unsigned long long)grad_hidden | (unsigned long long)(ldgh * 2)) & 15u) == 0) {  // d is a multiple of 64
                for (int c = lane; c < d / 8; c += 64) *(u32x4 *)(row + c * 8) = z;
            } else {
                for (int c = lane; c < d; c += 64) row[c] = 0;
            }
        }
    }
}

// out[i][:] = in[rowmap[i]][:] for i < *count: d bf16 values per row, 16 bytes per lane.
__global__ void __launch_bounds__(256) lm_gather_rows(const __bf16 *in, long long ldi, const int *rowmap,
                                                      const int *count, int d, __bf16 *out, long long ldo)
{
    const int n = *count;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const u32x4 *src = (const u32x4 *)(in + (long long)rowmap[i] * ldi);
        u32x4 *dst = (u32x4 *)(out + (long long)i * ldo);
        for (int c = threadIdx.x; c < d / 8; c += 256) dst[c] = src[c];
    }
}

// Merges the tile partials of each compact row, then the objective's once-per-row arithmetic.
// A workgroup takes 16 compact rows; LANES lanes share a row, lane l merging tiles l, l + LANES, ...,
// and their results meet in LDS in lane order (fixed order: the bits repeat from run to run).  What
// bounds it is latency - the partials of 1056 rows and 594 tiles are 5 MB - so every lane reads all
// of its partials into registers at once (LM_CMB_KEEP each; tiles beyond them are read twice) and the
// maximum and the sums are taken from there.  16 lanes where they hold all tiles (V <= 49152), 64
// for more: 16 lanes walking 594 tiles twice took 48 us on that batch, 64 lanes take 8; 64 lanes on the
// 11 tiles of V = 2711 made a whole 29 us call 1 us longer.
constexpr int LM_CMB_ROWS = 16, LM_CMB_KEEP = 12;
inline int lm_combine_lanes(int tiles_n) { return tiles_n <= 16 * LM_CMB_KEEP ? 16 : 64; }
template <bool AUX, int LM_CMB_LANES>
__global__ void __launch_bounds__(LM_CMB_ROWS * LM_CMB_LANES) lm_combine(RowParams p, LmRows w)
{
    __shared__ float sh_m[LM_CMB_LANES][LM_CMB_ROWS + 1], sh_s[LM_CMB_LANES][LM_CMB_ROWS + 1];
    __shared__ float sh_w[AUX ? LM_CMB_LANES : 1][LM_CMB_ROWS + 1];
    const int rl = threadIdx.x % LM_CMB_ROWS, tl = threadIdx.x / LM_CMB_ROWS;
    int base, count;
    lm_chunk_range(*w.n_live, w.chunk_cap, w.chunk, base, count);
    if ((long long)blockIdx.x * LM_CMB_ROWS >= count) return;  // whole workgroup alike
    const long long il = (long long)blockIdx.x * LM_CMB_ROWS + rl;  // row inside the chunk: the partials' index
    const long long i = base + il;                                  // compact row: the per-row arrays' index
    const bool live = il < count;
    float pm[LM_CMB_KEEP], ps[LM_CMB_KEEP], pw[AUX ? LM_CMB_KEEP : 1];
    const int tiles = live ? w.tiles_n : 0;
#pragma unroll
    for (int j = 0; j < LM_CMB_KEEP; ++j) {
        const int t = tl + j * LM_CMB_LANES;
        const long long at = (long long)t * w.part_stride + il;
        pm[j] = t < tiles ? w.part_m[at] : -INFINITY;
        ps[j] = t < tiles ? w.part_s[at] : 0.f;
        if constexpr (AUX) pw[j] = t < tiles ? w.part_w[at] : 0.f;
    }
    const float zy = live ? w.zy[i] : 0.f;
    float mz = -INFINITY;  // maximum over the tiles, in units of z
#pragma unroll
    for (int j = 0; j < LM_CMB_KEEP; ++j) mz = fmaxf(mz, pm[j]);
    for (int t = tl + LM_CMB_KEEP * LM_CMB_LANES; t < tiles; t += LM_CMB_LANES)
        mz = fmaxf(mz, w.part_m[(long long)t * w.part_stride + il]);
    sh_m[tl][rl] = mz;
    __syncthreads();
#pragma unroll 16
    for (int l = 0; l < LM_CMB_LANES; ++l) mz = fmaxf(mz, sh_m[l][rl]);
    const float mx = fmaxf(mz, zy);  // the sampled token may be the row's maximum
    const float mk = mx * p.k;
    float s = 0.f, ws = 0.f;
    auto add = [&](float mt, float st, float wt) __attribute__((always_inline)) {
        if (mt == -INFINITY) {
            s += st;  // no tile, or one without a number: 0, or NaN, which the maximum has skipped
        } else if constexpr (AUX) {
            const float d = (mt - mx) * p.k;
            const float f = __builtin_amdgcn_exp2f(d);
            s = fmaf(st, f, s);
            ws = fmaf(f, fmaf(d, st, wt), ws);
        } else {
            s = fmaf(st, __builtin_amdgcn_exp2f(fmaf(mt, p.k, -mk)), s);
        }
    };
#pragma unroll
    for (int j = 0; j < LM_CMB_KEEP; ++j) add(pm[j], ps[j], AUX ? pw[AUX ? j : 0] : 0.f);
    for (int t = tl + LM_CMB_KEEP * LM_CMB_LANES; t < tiles; t += LM_CMB_LANES) {
        const long long at = (long long)t * w.part_stride + il;
        add(w.part_m[at], w.part_s[at], AUX ? w.part_w[at] : 0.f);
    }
    sh_s[tl][rl] = s;
    if constexpr (AUX) sh_w[tl][rl] = ws;
    __syncthreads();
    if (tl != 0 || !live) return;
    float s_excl = 0.f, w_excl = 0.f;
#pragma unroll 16
    for (int l = 0; l < LM_CMB_LANES; ++l) {
        s_excl += sh_s[l][rl];
        if constexpr (AUX) w_excl += sh_w[l][rl];
    }
    const long long row = w.rows[i];
    bool has_grad = false;
    if constexpr (AUX) {
        float kl, H;
        const RowScalars o = row_scalars_aux(p, row, zy, mx, s_excl, w_excl, kl, H);
        write_row_aux(p, row, kl, H);
        write_row_outputs(p, row, o.logp, o.J, o.flags);
        const float q = o.c * p.inv_T;
        w.q[i] = q;
        w.gy[i] = q * (o.s_excl / o.s) + o.gy_ent;
        w.mx[i] = o.mx;
        w.log2s[i] = o.log2s;
        w.q2[i] = o.q2;
        w.bq[i] = o.bq;
        has_grad = q != 0.f || o.bq != 0.f;
    } else {
        const RowScalars o = row_scalars(p, row, zy, mk, s_excl);
        write_row_outputs(p, row, o.logp, o.J, o.flags);
        if (p.bwd) {
            const float q = o.c * p.inv_T;
            w.q[i] = q;
            w.gy[i] = q * (o.s_excl / o.s);
            w.shift[i] = o.shift;
            has_grad = q != 0.f;
        }
    }
    if (p.bwd) {  // the workgroup's 16 rows are lanes 0 .. 15, those that exist
        const unsigned grads = (unsigned)__ballot(has_grad) & 0xffffu;
        if (rl == 0) w.gmask[il / LM_CMB_ROWS] = grads;
    }
}

// The gradient rows of every LM_SUM_WORDS words of gmask.
constexpr int LM_SUM_WORDS = 256;
__global__ void __launch_bounds__(LM_SUM_WORDS) lm_count_grads(LmRows w)
{
    __shared__ int lds_n[LM_SUM_WORDS / 64];
    int base, count;
    lm_chunk_range(*w.n_live, w.chunk_cap, w.chunk, base, count);
    const int q = (int)(blockIdx.x * LM_SUM_WORDS + threadIdx.x);
    const int n = wave_sum(q * LM_CMB_ROWS < count ? __builtin_popcount(w.gmask[q]) : 0);
    if ((threadIdx.x & 63) == 0) lds_n[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) w.gsum[blockIdx.x] = lds_n[0] + lds_n[1] + lds_n[2] + lds_n[3];
}

// One 64 x 64 tile of out[c][r] = in[rowmap[r - r0]][c], r < R, c < C, at (r0, c0); the
// columns R .. of out are zero-filled.  Through LDS, four consecutive
// elements (8 bytes) per lane on both sides; C and ldo are multiples of 4 and both matrices
// 8-byte aligned (the operands of this path: d_model is a multiple of 64, rows 16-byte aligned).
__device__ __forceinline__ void lm_transpose_tile(int r0, int c0, const __bf16 *in, long long ldi, int R, const int *rowmap,
                                                  int C, __bf16 *out, long long ldo, unsigned short (*tile)[66])
{
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;  // 16 lanes x 4 elements across, 16 down
    const unsigned short *src = (const unsigned short *)in;
    unsigned short *dst = (unsigned short *)out;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int rl = ty + 16 * i, r = r0 + rl, c = c0 + tx * 4;
        unsigned lo = 0, hi = 0;
        if (r < R && c < C) {
            const unsigned *q = (const unsigned *)(src + (long long)rowmap[rl] * ldi + c);
            lo = q[0];
            hi = q[1];
        }
        tile[rl][tx * 4 + 0] = (unsigned short)lo;
        tile[rl][tx * 4 + 1] = (unsigned short)(lo >> 16);
        tile[rl][tx * 4 + 2] = (unsigned short)hi;
        tile[rl][tx * 4 + 3] = (unsigned short)(hi >> 16);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int cl2 = ty + 16 * i, c = c0 + cl2, r = r0 + tx * 4;  // a row of the output, four of its columns
        if (c < C && r < ldo) {
            unsigned *q = (unsigned *)(dst + (long long)c * ldo + r);
            q[0] = (unsigned)tile[tx * 4][cl2] | ((unsigned)tile[tx * 4 + 1][cl2] << 16);
            q[1] = (unsigned)tile[tx * 4 + 2][cl2] | ((unsigned)tile[tx * 4 + 3][cl2] << 16);
        }
    }
}

// G = dL/dz in bf16 for the chunk's gradient rows, row-major [n_grad][ldg], from the fp32 logits:
// g_j = -q p_j, g_y = q (1 - p_y).  A wavefront takes 16 rows of Z x 128 entries.  A lane reads 16 bytes, four entries of row
// lane % 16 (the rows' own values are read once), as Z lies: 1 KB a wavefront; the rows are turned round through
// LDS and leave 256 bytes at a time, each to its place among the gradient rows.  Padding is written as zeros: the
// columns V .. ldg (dL/dH runs over whole K steps of the vocabulary) and the rows n_grad .. the next
// multiple of 64 (dL/dW runs over whole K steps of rows).
// Reading Z in that order costs this kernel something (10066 rows of 152064: 648 us, 584 with Z row by row; 992 and 901 with
// the auxiliary terms) and saves the product in front 5 us of a CU's time per tile, 0.46 ms of those rows.
// Which rows have a gradient, and so where theirs go, every workgroup takes from gmask: a word for 16 rows, a load or three a
// lane while its logits are on their way.  The list in order, and their number, which the products read, come from here
// too (a kernel of one workgroup in front of this one made them: 4096 x 32000 x 256 332 -> 323 us a call, 100 x 3000 x 256
// 62.4 -> 60.3, 1024 x 50304 x 768 291.5 -> 290).
constexpr int LM_GL_COLS = 512, LM_GL_ROWS = 16;
static_assert(LM_GL_ROWS == LM_CMB_ROWS, "a word of gmask to a workgroup's rows");
static_assert(LM_SUM_WORDS == 256 && LM_CHUNK_MAX / LM_GL_ROWS / LM_SUM_WORDS <= 256, "a lane to every word of gsum");
// Every workgroup looking at all of the words costs chunks of many rows more and more of the launch (the rows of a default
// chunk are 640 words, a caller's workspace may hold 65536 of them): of chunks of more than LM_SUM_FROM rows lm_count_grads has
// counted the gradient rows of every 256 words (SUMS; an instantiation of its own: the choice inside cost 4096 x 32000 x 256
// 4 us), and only the words of a workgroup's own 4096 rows are looked at.  Call on one chunk of 1048576 x 256 x 64: 15100 us without,
// 13800 with, 65536 x 4000 x 512 1422 and 1382, 65536 x 1000 x 256 857 and 842, 20480 x 1000 x 256 287 and 289.
constexpr int LM_SUM_FROM = 32768;
template <bool AUX, bool SUMS>
__global__ void __launch_bounds__(256) lm_grad_logits(const float *Z, long long ldz, int V, LmRows w,
                                                      float k, __bf16 *G, long long ldg, int col_groups, unsigned gl_blocks,
                                                      const __bf16 *hidden, long long ldh, int d, __bf16 *Ht, long long ldht)
{
    constexpr int WAVE_COLS = LM_GL_COLS / 4, PITCH = WAVE_COLS * 2 + 16;  // bytes: 16-byte aligned rows, 4 banks apart
    __shared__ __attribute__((aligned(16))) char turn_all[4 * LM_GL_ROWS * PITCH];
    static_assert(sizeof(turn_all) >= 64 * 66 * 2, "the tile that is turned round for H^T fits");
    __shared__ int lds_n[2][4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
    int zbase, zcount;  // Z holds the current chunk's rows only
    lm_chunk_range(*w.n_live, w.chunk_cap, w.chunk, zbase, zcount);
    const int groups = (zcount + LM_GL_ROWS - 1) / LM_GL_ROWS;
    if (blockIdx.x >= gl_blocks) {  // H^T of the chunk's gradient rows, [d][ldht]: independent of G, in the same launch
        __shared__ int rowmap[64], lds_from[2], lds_to;
        const int t = (int)(blockIdx.x - gl_blocks), across = (int)(ldht / 64), first = t % across * 64;
        // what the lanes before this one have, added to `pos`, and what all of them have, added to `sum` (read before a barrier)
        auto scan = [&](int own, int &pos, int &sum) {
            int incl = own;  // inclusive scan inside the wavefront
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(incl, o, 64);
                if (lane >= o) incl += up;
            }
            if (lane == 63) lds_n[0][wv] = incl;
            __syncthreads();
            pos += incl - own;
            for (int i = 0; i < 4; ++i) {
                if (i < wv) pos += lds_n[0][i];
                sum += lds_n[0][i];
            }
        };
        int total = 0, n2 = 0, q_from = 0, q_to = groups;
        if constexpr (SUMS) {  // only the words that hold rows first .. first + 63
            const int own = (int)threadIdx.x * LM_SUM_WORDS < groups ? w.gsum[threadIdx.x] : 0;
            int pos = 0;
            scan(own, pos, n2);
            if (first >= n2) return;  // whole workgroup alike
            if (pos <= first && first < pos + own) lds_from[0] = (int)threadIdx.x * LM_SUM_WORDS, lds_from[1] = pos;
            const int last = min(first + 64, n2);
            if (pos < last && last <= pos + own) lds_to = min(((int)threadIdx.x + 1) * LM_SUM_WORDS, groups);
            __syncthreads();
            q_from = lds_from[0], total = lds_from[1], q_to = lds_to;
        }
        for (int q0 = q_from; q0 < q_to; q0 += 256) {  // whole workgroup alike
            const int q = q0 + (int)threadIdx.x;
            unsigned bits = q < groups ? w.gmask[q] : 0u;
            const int own = __builtin_popcount(bits);
            int pos = total - first;
            scan(own, pos, total);
            if (pos < 64 && pos + own > 0)
                for (; bits != 0u; bits &= bits - 1u, ++pos)
                    if (pos >= 0 && pos < 64) rowmap[pos] = w.rows[zbase + q * LM_GL_ROWS + __builtin_ctz(bits)];
            __syncthreads();
        }
        if constexpr (!SUMS) n2 = total;
        // columns past the rows that exist are read as zeros up to the next whole K step, and not at all beyond it
        if (first < (n2 + 63) / 64 * 64)
            lm_transpose_tile(first, t / across * 64, hidden, ldh, n2, rowmap, d, Ht, ldht, (unsigned short(*)[66])turn_all);
        return;
    }
    const int r0 = (int)(blockIdx.x / (unsigned)col_groups) * LM_GL_ROWS;
    // rows n_grad and up of the chunk, of which there are no more than it has: at most up to the next multiple of 64
    if (r0 >= (zcount + 63) / 64 * 64 && blockIdx.x != 0) return;
    const int c0 = (int)(blockIdx.x % (unsigned)col_groups) * LM_GL_COLS + wv * WAVE_COLS;  // this wavefront's columns
    char *turn = turn_all + wv * (LM_GL_ROWS * PITCH);
    const int ci = zbase + r0 + n;  // this lane's compact row
    // all of this lane's logits at once, whether the row has a gradient or not (Z is there up to whole parts); V <= ldz,
    // which is a multiple of 64.  They are read once: what the caches hold longer is G, which both products read
    // (non-temporal or not: 1024 x 50304 x 768 278 and 289 us a call, 3000 rows of it 759 and 785)
    f32x4 z[WAVE_COLS / 16];
#pragma unroll
    for (int it = 0; it < WAVE_COLS / 16; ++it) {
        const int c = c0 + it * 16 + 4 * g;
        z[it] = r0 < zcount && c < ldz
                    ? __builtin_nontemporal_load((const f32x4 *)(Z + lm_z_part(r0, c, ldz) + lm_z_in_part(r0 + n, c)))
                    : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int before = 0, n2 = 0;  // gradient rows ahead of this workgroup's, and in the chunk
    const int mine = r0 / LM_GL_ROWS;
    if constexpr (SUMS) {
        const int c = (int)threadIdx.x * LM_SUM_WORDS < groups ? w.gsum[threadIdx.x] : 0, q = mine / LM_SUM_WORDS * LM_SUM_WORDS + (int)threadIdx.x;
        n2 = c;
        before = ((int)threadIdx.x < mine / LM_SUM_WORDS ? c : 0) + (q < mine && q < groups ? __builtin_popcount(w.gmask[q]) : 0);
    } else {
        for (int q = threadIdx.x; q < groups; q += 256) {
            const int c = __builtin_popcount(w.gmask[q]);
            n2 += c;
            before += q < mine ? c : 0;
        }
    }
    before = wave_sum(before);
    n2 = wave_sum(n2);
    if (lane == 0) lds_n[0][wv] = before, lds_n[1][wv] = n2;
    __syncthreads();
    before = lds_n[0][0] + lds_n[0][1] + lds_n[0][2] + lds_n[0][3];
    n2 = lds_n[1][0] + lds_n[1][1] + lds_n[1][2] + lds_n[1][3];
    const int n2_pad = (n2 + 63) / 64 * 64;
    const unsigned grads = r0 < zcount ? w.gmask[mine] : 0u;
    const int pos = (grads >> n) & 1u ? before + __builtin_popcount(grads & ((1u << n) - 1u)) : -1;
    if (blockIdx.x == 0 && threadIdx.x == 0) *w.n_grad = n2;
    if (blockIdx.x % (unsigned)col_groups == 0 && threadIdx.x < LM_GL_ROWS && pos >= 0) w.orig2[pos] = w.rows[zbase + r0 + n];
    float q = 0.f, sh = 0.f, mxr = 0.f, l2s = 0.f, q2 = 0.f, bq = 0.f, gy = 0.f;
    int y = -1;
    if (r0 + n < zcount) {  // (of a row without a gradient nothing is stored)
        if constexpr (AUX) {
            mxr = w.mx[ci], l2s = w.log2s[ci], q2 = w.q2[ci], bq = w.bq[ci];
        } else {
            q = w.q[ci], sh = w.shift[ci];
        }
        gy = w.gy[ci];
        y = w.tokens32[ci];
    }
    const int yc = y - c0 - 4 * g, ncols = V - c0 - 4 * g;  // the sampled token and the end of the row, from this lane's first column
    const bool whole = c0 + WAVE_COLS <= V;
#pragma unroll
    for (int it = 0; it < WAVE_COLS / 16; ++it) {
        float gv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (AUX) {
                // g_j = p_j (q2 + bq log2 p_j): policy, KL and entropy parts in one (see grad_vec_aux)
                const float a = fmaxf(fmaf(z[it][e] - mxr, k, -l2s), kExpFloor);
                gv[e] = __builtin_amdgcn_exp2f(a) * fmaf(bq, a, q2);
            } else {
                gv[e] = -q * __builtin_amdgcn_exp2f(fmaf(z[it][e], k, -sh));
            }
            gv[e] = it * 16 + e == yc ? gy : gv[e];
        }
        if (!whole) {
#pragma unroll
            for (int e = 0; e < 4; ++e) gv[e] = it * 16 + e >= ncols ? 0.f : gv[e];
        }
        const bf16x2 lo = __builtin_convertvector((f32x2){gv[0], gv[1]}, bf16x2);
        const bf16x2 hi = __builtin_convertvector((f32x2){gv[2], gv[3]}, bf16x2);
        *(u32x2 *)(turn + n * PITCH + (it * 16 + 4 * g) * 2) = u32x2{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
    }
    // LDS serves a wavefront's accesses in order: no barrier.  16 lanes to a row, four rows a store
    const int c = c0 + n * 8;
#pragma unroll
    for (int i = 0; i < LM_GL_ROWS / 4; ++i) {
        const int r = 4 * i + g;
        const u32x4 out = *(const u32x4 *)(turn + r * PITCH + n * 16);
        const int to = __shfl(pos, r, 64);  // lane r < 16 holds row r's
        if (c < ldg) {                      // ldg is a multiple of 64: whole groups of eight
            if (to >= 0) *(u32x4 *)(G + (long long)to * ldg + c) = out;
            if (r0 + r >= n2 && r0 + r < n2_pad) *(u32x4 *)(G + (long long)(r0 + r) * ldg + c) = u32x4{0u, 0u, 0u, 0u};
        }
    }
}

// Sum of the parts of the tiles lm_gemm_nt has cut: C[c_rows[r]][:] = bf16(sum over s of the
// tile's partial blocks) for the rows present, parts in order.  Does nothing when no tile was cut.
// The workgroups behind its own are grpo_finalize's: neither waits for anything of the other, and a launch of its own costs
// the sums of a small call what they take (724 x 12331 x 1152 134 -> 130 us a call).
constexpr int LM_REDUCE_BLOCKS = 512;
__global__ void __launch_bounds__(1024) lm_split_reduce(const float *ws, const int *M_dev, int M, int N, int tiles_n,
                                                       int k_tiles, int max_items, int n_cu,
                                                       const int *c_rows, __bf16 *C, long long ldc, FinParams fin)
{
    if (blockIdx.x >= LM_REDUCE_BLOCKS) {  // whole workgroup alike
        finalize_segment(fin, blockIdx.x - LM_REDUCE_BLOCKS);
        return;
    }
    const int rows = M_dev ? min(*M_dev, M) : M;
    const LmPlan pl = lm_plan(rows, tiles_n, k_tiles, true, max_items, n_cu);
    if (pl.s2 == 1) return;
    // 16 bytes a lane, as lm_gemm_nt's wavefronts have stored them; whole tiles first, then thin ones (wavefronts 0 .. 3)
    constexpr int quads = LM_BM * LM_BN / 4;
    const long long rest = (long long)pl.rest * quads, total = rest + (long long)pl.thin * (quads / 2);
    for (long long e = (long long)blockIdx.x * 1024 + threadIdx.x; e < total; e += LM_REDUCE_BLOCKS * 1024ll) {
        int row, col, parts, q;
        const float *src;
        if (e < rest) {
            const int t = (int)(e / quads);
            q = (int)(e % quads);
            int tm, tn;
            lm_tile_of(pl.full + t, pl.rows_w, tiles_n, tm, tn);
            row = tm * LM_BM, col = tn * LM_BN, parts = pl.s2;
            src = ws + (((long long)t * pl.s2) << 16) + q * 4;
        } else {
            const long long e2 = e - rest;
            const int t = (int)(e2 / (quads / 2));
            q = (int)(e2 % (quads / 2));
            row = pl.rows_w * LM_BM, col = t * LM_BN, parts = pl.t2;
            src = ws + (((long long)pl.rest * pl.s2 + (long long)t * pl.t2) << 16) + q * 4;
        }
        const int wave = q / (LM_FA * LM_FB * 64), lane = q & 63;
        row += wave / LM_WN * (LM_FA * 16) + (q / (LM_FB * 64)) % LM_FA * 16 + (lane & 15);
        col += wave % LM_WN * (LM_FB * 16) + (q / 64) % LM_FB * 16 + 4 * (lane >> 4);
        if (row >= rows || col >= N || parts == 1) continue;  // N is a multiple of LM_BK: a quad is inside or outside
        f32x4 a = *(const f32x4 *)src;
#pragma unroll 8
        for (int s = 1; s < parts; ++s) a += *(const f32x4 *)(src + ((long long)s << 16));
        const bf16x2 lo = __builtin_convertvector((f32x2){a[0], a[1]}, bf16x2);
        const bf16x2 hi = __builtin_convertvector((f32x2){a[2], a[3]}, bf16x2);
        __bf16 *dst = C + (long long)(c_rows ? c_rows[row] : row) * ldc + col;
        if ((((unsigned long long)C | (unsigned long long)(ldc * 2)) & 7u) == 0) {
            *(u32x2 *)dst = u32x2{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
        } else {
            dst[0] = lo[0];
            dst[1] = lo[1];
            dst[2] = hi[0];
            dst[3] = hi[1];
        }
    }
}

// rows x cols zeros into a row-strided matrix (fill kernels rather than memsets, so that
// the call can be captured into a graph)
template <typename T>
__global__ void __launch_bounds__(256) lm_zero(T *out, long long rows, long long cols, long long ld)
{
    const long long total = rows * cols;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256)
        out[(i / cols) * ld + i % cols] = (T)0;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

template <int EPI, int Z, bool AUX = false, bool AKM = false, bool BKM = false, bool LEAD = false>
hipError_t lm_launch_gemm(GemmParams p, hipStream_t st)
{
    static std::atomic<bool> attr_done[64];      // setting the attribute twice is harmless
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && !attr_done[dev].load()) {
        e = hipFuncSetAttribute((const void *)lm_gemm_nt<EPI, Z, AUX, AKM, BKM, LEAD>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LM_LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done[dev].store(true);
    }
    p.tiles_n = (p.N + LM_BN - 1) / LM_BN;
    p.n_cu = cu_count();
    const unsigned grid = 8u * (unsigned)lm_workgroups_per_xcd(p.M, p.tiles_n, EPI == LM_EPI_BF16 && p.split_items > 0, p.n_cu);
    hipLaunchKernelGGL((lm_gemm_nt<EPI, Z, AUX, AKM, BKM, LEAD>), dim3(grid), dim3(LM_THREADS), LM_LDS_BYTES, st, p);
    return hipGetLastError();
}

struct LmLayout {
    size_t rows, tokens32, gmask, orig2, counts, zy, shift, q, gy, mx, log2s, q2, bq, part_m, part_s, part_w, Hc, Z, G, Ht,
        total;
    long long ldz, ldg, ldgt;  // vocab and chunk rows rounded up to whole K steps
    int tiles_n;
    int cap;  // rows per chunk: what the partials, Z, G and H^T are sized for
};

// Default limit of a chunk of the backward: 10240 rows keep the workspace at V = 152064 under
// 10 GB whatever the number of tokens (6 bytes per chunk row and vocabulary entry), and a chunk
// still fills the chip (40 tile rows: 23760 tiles of the logits product, 800 of dL/dH).  A caller
// that brings more gets larger chunks.
constexpr int64_t kLmChunkRows = 10240;
constexpr int64_t kLmChunkMax = LM_CHUNK_MAX;

int64_t lm_cap_limit(int64_t n) { return std::min<int64_t>(kLmChunkMax, std::max<int64_t>(256, (n + 255) / 256 * 256)); }

// cap: rows per chunk, a multiple of 256 in [256, lm_cap_limit(n)] (the forward alone is one chunk)
LmLayout lm_layout(int64_t n, int64_t V, int64_t d, bool bwd, int64_t cap)
{
    LmLayout L = {};
    L.cap = (int)cap;
    L.tiles_n = (int)((V + LM_BN - 1) / LM_BN);
    L.ldz = L.ldg = (long long)align_up((size_t)V, 64);  // whole K steps, 128-byte rows
    L.ldgt = (long long)align_up((size_t)cap, 64);
    size_t off = align_up(grpo_workspace_bytes(n), 256);
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes, 256);
        return at;
    };
    L.counts = take(256);
    L.rows = take((size_t)n * 4);
    L.tokens32 = take((size_t)n * 4);
    L.zy = take((size_t)n * 4);
    L.part_m = take((size_t)L.tiles_n * cap * 4);
    L.part_s = take((size_t)L.tiles_n * cap * 4);
    L.Hc = take((size_t)n * d * 2);
    if (bwd) {
        L.gmask = take((size_t)cap * 4);
        L.orig2 = take((size_t)cap * 4);
        L.shift = take((size_t)n * 4);
        L.q = take((size_t)n * 4);
        L.gy = take((size_t)n * 4);
        L.mx = take((size_t)n * 4);  // these four and part_w: only the call with the auxiliary terms
        L.log2s = take((size_t)n * 4);
        L.q2 = take((size_t)n * 4);
        L.bq = take((size_t)n * 4);
        L.part_w = take((size_t)L.tiles_n * cap * 4);
        L.Z = take((size_t)cap * L.ldz * 4);
        L.G = take((size_t)cap * L.ldg * 2);
        L.Ht = take((size_t)d * L.ldgt * 2);
    }
    L.total = off;
    return L;
}

// The largest chunk (multiple of 256 rows) whose workspace fits `bytes`; 0 if not even 256 rows do.
int64_t lm_cap_for_workspace(int64_t n, int64_t V, int64_t d, size_t bytes)
{
    int64_t lo = 0, hi = lm_cap_limit(n) / 256;  // in units of 256 rows; the size grows with the chunk
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (lm_layout(n, V, d, true, mid * 256).total <= bytes)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo * 256;
}

bool lm_sizes_ok(int64_t n_tokens, int64_t vocab, int64_t d_model)
{
    return n_tokens >= 0 && n_tokens <= 0x7fffff00ll && vocab > 0 && vocab <= kMaxVocab && d_model > 0 &&
           d_model <= (1 << 20) && d_model % LM_BK == 0;
}
// With the backward G is an operand whose rows are align64(vocab) elements long: the byte offset
// of row 255 of an operand tile must fit 32 bits.
bool lm_bwd_vocab_ok(int64_t vocab) { return (int64_t)align_up((size_t)vocab, 64) * 2 * LM_BM < (1ll << 32); }

grpo_status lm_check_common(const void *hidden, int64_t hidden_stride, const void *weight,
                            int64_t weight_stride, int64_t n_tokens, int64_t vocab, int64_t d_model,
                            const int64_t *tokens, float temperature, bool bwd)
{
    if (!lm_sizes_ok(n_tokens, vocab, d_model) || hidden_stride < d_model || weight_stride < d_model)
        return GRPO_ERR_SHAPE;
    if (bwd && !lm_bwd_vocab_ok(vocab)) return GRPO_ERR_SHAPE;
    if (!(temperature > 0.f) || !std::isfinite(temperature)) return GRPO_ERR_PARAM;
    if (n_tokens == 0) return GRPO_OK;
    if (!hidden || !weight || !tokens) return GRPO_ERR_NULL;
    if (((uintptr_t)hidden & 15u) || ((uintptr_t)weight & 15u) || ((hidden_stride * 2) & 15) ||
        ((weight_stride * 2) & 15))
        return GRPO_ERR_ALIGN;
    // byte offsets inside one 256-row operand tile must fit 32 bits
    if (weight_stride * 2 * LM_BN >= (1ll << 32)) return GRPO_ERR_SHAPE;
    return GRPO_OK;
}

grpo_status lm_impl(bool bwd, bool aux, const void *hidden, int64_t hidden_stride, const void *weight,
                    int64_t weight_stride, int64_t n_tokens, int64_t vocab, int64_t d_model,
                    const int64_t *tokens, const float *old_logprobs, const float *ref_logprobs,
                    const float *advantages, const uint8_t *mask, const float *token_weights, float eps_low,
                    float eps_high, float delta, float temperature, float kl_coef, float entropy_coef,
                    double denom, float grad_scale, float *loss_out, float *logprobs_out, float *entropy_out,
                    int64_t *counts_out, void *grad_hidden, int64_t grad_hidden_stride,
                    float *grad_weight, int64_t grad_weight_stride, int accumulate_grad_weight,
                    void *workspace, size_t workspace_bytes, void *stream)
{
    grpo_status rc = lm_check_common(hidden, hidden_stride, weight, weight_stride, n_tokens, vocab,
                                     d_model, tokens, temperature, bwd);
    if (rc != GRPO_OK) return rc;
    if (bwd) {
        if (!(eps_low >= 0.f && eps_low <= 1.f) || !(eps_high >= 0.f) || !std::isfinite(eps_high) ||
            !(delta > 1.f + eps_high) || std::isnan(denom) || std::isnan(grad_scale) ||
            !std::isfinite(kl_coef) || !std::isfinite(entropy_coef))
            return GRPO_ERR_PARAM;
        if (!loss_out) return GRPO_ERR_NULL;
        if (n_tokens > 0 && (!old_logprobs || !advantages || !grad_hidden)) return GRPO_ERR_NULL;
        if (n_tokens > 0 && kl_coef != 0.f && !ref_logprobs) return GRPO_ERR_NULL;
        if (!grad_weight) return GRPO_ERR_NULL;
        if (grad_hidden_stride < d_model || grad_weight_stride < d_model) return GRPO_ERR_SHAPE;
    } else {
        if (n_tokens == 0) return GRPO_OK;
        if (!logprobs_out) return GRPO_ERR_NULL;
    }
    if (!workspace || ((uintptr_t)workspace & 255u) != 0) return GRPO_ERR_WORKSPACE;
    // the forward alone keeps nothing per logit and takes the largest chunk there is (one chunk up
    // to 2^20 tokens); the backward takes the largest chunk the caller's workspace holds
    const int64_t cap = bwd ? lm_cap_for_workspace(n_tokens, vocab, d_model, workspace_bytes) : lm_cap_limit(n_tokens);
    if (cap == 0) return GRPO_ERR_WORKSPACE;
    const LmLayout L = lm_layout(n_tokens, vocab, d_model, bwd, cap);
    if (workspace_bytes < L.total) return GRPO_ERR_WORKSPACE;

    char *ws = (char *)workspace;
    hipStream_t st = (hipStream_t)stream;
    const size_t col = align_up((size_t)n_tokens * 4, 256);
    WsHeader *hdr = (WsHeader *)ws;
    float *J_ws = (float *)(ws + kHeaderBytes);
    float *KL_ws = (float *)(ws + kHeaderBytes + col);
    float *H_ws = (float *)(ws + kHeaderBytes + 2 * col);
    unsigned char *flags_ws = (unsigned char *)(ws + kHeaderBytes + 3 * col);
    FinPartial *partials = (FinPartial *)(ws + kHeaderBytes + 3 * col + align_up((size_t)n_tokens, 256));
    const FinParams fin = {J_ws, aux ? KL_ws : nullptr, H_ws, flags_ws, (long long)n_tokens, hdr, partials, kl_coef,
                           entropy_coef, loss_out, (long long *)counts_out, nullptr};
    bool finalized = false;

    const bool take = n_tokens > 0 && n_tokens <= LM_TAKE_MAX;
    if (bwd && !take)
        hipLaunchKernelGGL(grpo_prepare, dim3(1), dim3(1024), 0, st, mask, aux ? token_weights : (const float *)nullptr,
                           (long long)n_tokens, denom, hdr, (int *)nullptr, (const int *)nullptr, LateRule{});
    if (n_tokens > 0) {
        const int M = (int)n_tokens, V = (int)vocab, D = (int)d_model;
        const int Mc = (int)std::min<int64_t>(cap, n_tokens);  // most rows a chunk can have
        const int n_chunks = (int)((n_tokens + cap - 1) / cap);
        LmRows w = {};
        w.n_live = (int *)(ws + L.counts);
        w.n_grad = w.n_live + 1;
        w.rows = (int *)(ws + L.rows);
        w.tokens32 = (int *)(ws + L.tokens32);
        w.zy = (float *)(ws + L.zy);
        w.part_m = (float *)(ws + L.part_m);
        w.part_s = (float *)(ws + L.part_s);
        w.part_stride = cap;
        w.tiles_n = L.tiles_n;
        w.chunk_cap = (int)cap;
        if (aux) {
            w.part_w = (float *)(ws + L.part_w);
            w.mx = (float *)(ws + L.mx);
            w.log2s = (float *)(ws + L.log2s);
            w.q2 = (float *)(ws + L.q2);
            w.bq = (float *)(ws + L.bq);
        }
        if (bwd) {
            w.gmask = (unsigned *)(ws + L.gmask);
            w.orig2 = (int *)(ws + L.orig2);
            w.shift = (float *)(ws + L.shift);
            w.q = (float *)(ws + L.q);
            w.gy = (float *)(ws + L.gy);
        }
        const float k = (float)((double)kLog2e / (double)temperature);

        RowParams p = {};
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
        p.inv_T = 1.0f / temperature;
        p.k = k;
        p.lo = 1.0f - eps_low;
        p.hi = 1.0f + eps_high;
        p.delta = delta;
        p.grad_scale = grad_scale;
        p.bwd = bwd ? 1 : 0;
        if (aux) {
            p.ref_lp = kl_coef != 0.f ? ref_logprobs : nullptr;
            p.token_w = token_weights;
            p.KL_ws = KL_ws;
            p.H_ws = H_ws;
            p.entropy_out = entropy_out;
            p.kl_coef = kl_coef;
            p.ent_coef = entropy_coef;
        }

        // rows that take part, and their hidden states side by side; dL/dH zeroed (fill kernels rather than
        // memsets, so that the call can be captured into a graph)
        __bf16 *Hc = (__bf16 *)(ws + L.Hc);
        __bf16 *G = nullptr, *Ht = nullptr;
        const int n_cu = cu_count();
        if (bwd) G = (__bf16 *)(ws + L.G), Ht = (__bf16 *)(ws + L.Ht);
        if (take) {
            hipLaunchKernelGGL(lm_take_rows, dim3((unsigned)((M + LM_TAKE_ROWS - 1) / LM_TAKE_ROWS)), dim3(LM_TAKE_THREADS), 0, st,
                               p, w, (const __bf16 *)hidden, (long long)hidden_stride, D, Hc,
                               bwd ? (unsigned short *)grad_hidden : (unsigned short *)nullptr, (long long)grad_hidden_stride,
                               denom, bwd ? hdr : (WsHeader *)nullptr);
        } else {
            hipLaunchKernelGGL(lm_select_rows, dim3(1), dim3(1024), 0, st, p, w);
            hipLaunchKernelGGL(lm_gather_rows, dim3((unsigned)(M < 8192 ? M : 8192)), dim3(256), 0, st,
                               (const __bf16 *)hidden, (long long)hidden_stride, (const int *)w.rows,
                               (const int *)w.n_live, D, Hc, (long long)d_model);
            if (bwd)
                hipLaunchKernelGGL(lm_zero<unsigned short>, dim3(2048), dim3(256), 0, st, (unsigned short *)grad_hidden,
                                   (long long)n_tokens, (long long)d_model, (long long)grad_hidden_stride);
        }

        for (int c = 0; c < n_chunks; ++c) {
            w.chunk = c;
            GemmParams g = {};  // logits of the chunk's rows: softmax partials, z_y, fp32 copy for the backward
            g.A = Hc;
            g.lda = d_model;
            g.B = (const __bf16 *)weight;
            g.ldb = weight_stride;
            g.M = Mc;
            g.M_dev = w.n_live;
            g.chunk = c;
            g.chunk_cap = (int)cap;
            g.N = V;
            g.K = D;
            g.tokens32 = w.tokens32;
            g.k = k;
            g.part_m = w.part_m;
            g.part_s = w.part_s;
            g.part_w = w.part_w;
            g.part_stride = cap;
            g.zy = w.zy;
            g.Z = bwd ? (float *)(ws + L.Z) : nullptr;
            g.ldz = L.ldz;
            // Logits beyond what the 256 MB memory-side cache holds until lm_grad_logits reads them pass it by (as far as the
            // host knows their number): call on 6000 x 50304 x 512 tokens, five eighths of them live, 1029 us kept and
            // 1003 past it, 3000 x 50304 x 768 with auxiliary terms 759 and 744; on 1000 x 30000 x 512 153 and 157, on
            // 2000 x 20000 x 1024 264 and 268.
            const bool large = (long long)Mc * L.ldz > (256ll << 20) / 4;
            auto logits = [&](auto lead) {
                constexpr bool LD = decltype(lead)::value;
                return aux   ? large ? lm_launch_gemm<LM_EPI_LSE, LM_Z_LARGE, true, false, false, LD>(g, st)
                                     : lm_launch_gemm<LM_EPI_LSE, LM_Z_KEPT, true, false, false, LD>(g, st)
                       : !bwd ? lm_launch_gemm<LM_EPI_LSE, LM_Z_NONE, false, false, false, LD>(g, st)
                       : large ? lm_launch_gemm<LM_EPI_LSE, LM_Z_LARGE, false, false, false, LD>(g, st)
                               : lm_launch_gemm<LM_EPI_LSE, LM_Z_KEPT, false, false, false, LD>(g, st);
            };
            hipError_t e = D <= LM_LEAD_STEPS * LM_BK ? logits(std::true_type{}) : logits(std::false_type{});
            if (e != hipSuccess) return GRPO_ERR_HIP;

            const dim3 cmb_grid((unsigned)((Mc + LM_CMB_ROWS - 1) / LM_CMB_ROWS));
            const bool few = lm_combine_lanes(L.tiles_n) == 16;
            const dim3 cmb_block((unsigned)(LM_CMB_ROWS * lm_combine_lanes(L.tiles_n)));
            if (aux)
                hipLaunchKernelGGL((few ? lm_combine<true, 16> : lm_combine<true, 64>), cmb_grid, cmb_block, 0, st, p, w);
            else
                hipLaunchKernelGGL((few ? lm_combine<false, 16> : lm_combine<false, 64>), cmb_grid, cmb_block, 0, st, p, w);
            if (!bwd) continue;

            const bool sums = Mc > LM_SUM_FROM;
            if (sums) {
                w.gsum = (int *)(w.gmask + cap / LM_GL_ROWS);  // in the space behind the words
                hipLaunchKernelGGL(lm_count_grads, dim3((unsigned)((Mc + LM_GL_ROWS * LM_SUM_WORDS - 1) / (LM_GL_ROWS * LM_SUM_WORDS))),
                                   dim3(LM_SUM_WORDS), 0, st, w);
            }
            const int gl_cols = (int)((L.ldg + LM_GL_COLS - 1) / LM_GL_COLS);
            // rows up to the next multiple of 64: the padding rows are written too (G has cap >= 256 rows)
            const unsigned gl_blocks = (unsigned)((long long)gl_cols * ((Mc + 63) / 64 * (64 / LM_GL_ROWS)));
            const dim3 gl_grid(gl_blocks + (unsigned)((L.ldgt / 64) * ((D + 63) / 64)));  // then the tiles of H^T
            hipLaunchKernelGGL((aux ? sums ? lm_grad_logits<true, true> : lm_grad_logits<true, false>
                                    : sums ? lm_grad_logits<false, true> : lm_grad_logits<false, false>), gl_grid, dim3(256), 0, st,
                               (const float *)(ws + L.Z), L.ldz, V, w, k, G, L.ldg, gl_cols, gl_blocks,
                               (const __bf16 *)hidden, (long long)hidden_stride, D, Ht, L.ldgt);

            GemmParams gh = {};  // dL/dH [gradient rows][d] = G . W, scattered to the original rows; W is read as it
                                 // lies, [vocab][d]: K-major, its rows past the vocabulary read as zeros
            gh.A = G;
            gh.lda = L.ldg;
            gh.B = (const __bf16 *)weight;
            gh.ldb = weight_stride;
            gh.b_cols = D;
            gh.b_rows = V;
            gh.M = Mc;
            gh.M_dev = w.n_grad;
            gh.N = D;
            gh.K = (int)L.ldg;
            gh.C = grad_hidden;
            gh.ldc = grad_hidden_stride;
            gh.c_rows = w.orig2;
            // The fp32 logits are no longer needed: their space takes the partial results (blocks of
            // 256 x 256 fp32) of the tiles whose contraction over the vocabulary is cut into parts.
            const size_t z_blocks = (size_t)cap * (size_t)L.ldz * 4 / ((size_t)LM_BM * LM_BN * 4);
            gh.split_items = (int)(z_blocks < 0x7fffffffu ? z_blocks : 0x7fffffffu);
            gh.split_ws = (float *)(ws + L.Z);
            e = lm_launch_gemm<LM_EPI_BF16, LM_Z_NONE, false, false, true>(gh, st);
            if (e != hipSuccess) return GRPO_ERR_HIP;
            if (gh.split_items > 0) {
                const bool last = c == n_chunks - 1;  // every row's objective is there
                hipLaunchKernelGGL(lm_split_reduce, dim3(LM_REDUCE_BLOCKS + (last ? fin_blocks(n_tokens) : 0)), dim3(1024), 0, st,
                                   (const float *)gh.split_ws, (const int *)w.n_grad, Mc, D, (D + LM_BN - 1) / LM_BN,
                                   (int)(L.ldg / LM_BK), gh.split_items, n_cu, (const int *)w.orig2, (__bf16 *)grad_hidden,
                                   (long long)grad_hidden_stride, fin);
                finalized = last;
            }

            GemmParams gw = {};  // dL/dW [V][d] (+)= G^T . H over the chunk's gradient rows; G is read as it lies,
                                 // [rows][ldg]: K-major
            gw.A = G;
            gw.lda = L.ldg;
            gw.a_cols = (int)L.ldg;
            gw.B = Ht;
            gw.ldb = L.ldgt;
            gw.M = V;
            gw.N = D;
            gw.K = (int)L.ldgt;
            gw.K_dev = w.n_grad;
            gw.C = grad_weight;
            gw.ldc = grad_weight_stride;
            gw.accumulate = (accumulate_grad_weight || c > 0) ? 1 : 0;  // the first chunk starts the sum
            // (how many rows it contracts the host does not know; the possibility costs this product's long contractions
            // nothing: call on 4096 x 152064 x 5120 11084 us with it, 11122 without, 2048 x 152064 x 2048 2740 either way)
            e = lm_launch_gemm<LM_EPI_F32, LM_Z_NONE, false, true, false, true>(gw, st);
            if (e != hipSuccess) return GRPO_ERR_HIP;
        }
    } else if (bwd && !accumulate_grad_weight && vocab > 0) {
        // no tokens: the weight gradient is zero
        hipLaunchKernelGGL(lm_zero<float>, dim3(4096), dim3(256), 0, st, grad_weight, (long long)vocab,
                           (long long)d_model, (long long)grad_weight_stride);
    }
    if (bwd && !finalized) hipLaunchKernelGGL(grpo_finalize, dim3(fin_blocks(n_tokens)), dim3(1024), 0, st, fin);
    return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

}  // namespace

extern "C" {

size_t grpo_lmhead_workspace_bytes(int64_t n_tokens, int64_t vocab, int64_t d_model, int with_backward)
{
    if (!lm_sizes_ok(n_tokens, vocab, d_model) || (with_backward && !lm_bwd_vocab_ok(vocab))) return 0;
    const int64_t cap = with_backward ? std::min<int64_t>(lm_cap_limit(n_tokens), kLmChunkRows) : lm_cap_limit(n_tokens);
    return lm_layout(n_tokens, vocab, d_model, with_backward != 0, cap).total;
}

size_t grpo_lmhead_workspace_bytes_for_chunk(int64_t n_tokens, int64_t vocab, int64_t d_model, int64_t chunk_rows)
{
    if (!lm_sizes_ok(n_tokens, vocab, d_model) || !lm_bwd_vocab_ok(vocab) || chunk_rows <= 0) return 0;
    const int64_t cap = std::min<int64_t>(lm_cap_limit(n_tokens), (std::min<int64_t>(chunk_rows, kLmChunkMax) + 255) / 256 * 256);
    return lm_layout(n_tokens, vocab, d_model, true, cap).total;
}

grpo_status grpo_lmhead_logprobs_fwd(const void *hidden, int64_t hidden_stride, const void *weight,
                                     int64_t weight_stride, int64_t n_tokens, int64_t vocab,
                                     int64_t d_model, const int64_t *tokens, const uint8_t *mask,
                                     float temperature, float *logprobs_out, void *workspace,
                                     size_t workspace_bytes, void *stream)
{
    return lm_impl(false, false, hidden, hidden_stride, weight, weight_stride, n_tokens, vocab, d_model, tokens,
                   nullptr, nullptr, nullptr, mask, nullptr, 0.f, 0.f, 0.f, temperature, 0.f, 0.f, 0.0, 0.f, nullptr,
                   logprobs_out, nullptr, nullptr, nullptr, 0, nullptr, 0, 0, workspace, workspace_bytes, stream);
}

grpo_status grpo_lmhead_loss_fwd_bwd(const void *hidden, int64_t hidden_stride, const void *weight,
                                     int64_t weight_stride, int64_t n_tokens, int64_t vocab,
                                     int64_t d_model, const int64_t *tokens, const float *old_logprobs,
                                     const float *advantages, const uint8_t *mask, float eps_low,
                                     float eps_high, float delta, float temperature, double denom,
                                     float grad_scale, float *loss_out, float *logprobs_out,
                                     int64_t *counts_out, void *grad_hidden, int64_t grad_hidden_stride,
                                     float *grad_weight, int64_t grad_weight_stride,
                                     int accumulate_grad_weight, void *workspace, size_t workspace_bytes,
                                     void *stream)
{
    return lm_impl(true, false, hidden, hidden_stride, weight, weight_stride, n_tokens, vocab, d_model, tokens,
                   old_logprobs, nullptr, advantages, mask, nullptr, eps_low, eps_high, delta, temperature, 0.f, 0.f,
                   denom, grad_scale, loss_out, logprobs_out, nullptr, counts_out, grad_hidden, grad_hidden_stride,
                   grad_weight, grad_weight_stride, accumulate_grad_weight, workspace, workspace_bytes, stream);
}

grpo_status grpo_lmhead_loss_aux_fwd_bwd(const void *hidden, int64_t hidden_stride, const void *weight,
                                         int64_t weight_stride, int64_t n_tokens, int64_t vocab,
                                         int64_t d_model, const int64_t *tokens, const float *old_logprobs,
                                         const float *ref_logprobs, const float *advantages,
                                         const uint8_t *mask, const float *token_weights, float eps_low,
                                         float eps_high, float delta, float temperature, float kl_coef,
                                         float entropy_coef, double denom, float grad_scale, float *loss_out,
                                         float *logprobs_out, float *entropy_out, int64_t *counts_out,
                                         void *grad_hidden, int64_t grad_hidden_stride, float *grad_weight,
                                         int64_t grad_weight_stride, int accumulate_grad_weight,
                                         void *workspace, size_t workspace_bytes, void *stream)
{
    return lm_impl(true, true, hidden, hidden_stride, weight, weight_stride, n_tokens, vocab, d_model, tokens,
                   old_logprobs, ref_logprobs, advantages, mask, token_weights, eps_low, eps_high, delta,
                   temperature, kl_coef, entropy_coef, denom, grad_scale, loss_out, logprobs_out, entropy_out,
                   counts_out, grad_hidden, grad_hidden_stride, grad_weight, grad_weight_stride,
                   accumulate_grad_weight, workspace, workspace_bytes, stream);
}

}  // extern "C"
