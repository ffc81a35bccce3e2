// Device code of the adapter's training step (Section 3.1, "Training Loss", Eq. 3; AdamW per
// Section 4.1): the adapter runs over all T positions of a sequence at once, the cross entropy of
// its draft distribution against the frozen target's is differentiated by hand (chain rule written
// out: RMSNorm, rotary embedding, causal attention, projections), and AdamW updates fp32 master
// copies of the adapter's tensors.  All arithmetic is fp32; the dense contractions go through the
// bf16 MFMA with every fp32 number as the exact sum of three bf16 numbers, weights of the frozen LM head are read
// from their bf16 tiles as they are.  Included by kangaroo.hip after kernels.hip.h.
#pragma once


// ---------------------------------------------------------------------------------------------
// C[M][N] (+)= sum_k A(m, k) * B(k, n), fp32, any strides.
//   A(m, k) = A[m * sam + k * sak]
//   B(k, n) = b_mode 0: B[k * sbk + n * sbn]
//             b_mode 1: element (row n, col k) of a matrix stored as bf16 MFMA tiles (the layout of
//                       pack_w_bf16_kernel: tile (row/16, col/32), 16-byte unit (col%32/8)*16 + row%16)
//             b_mode 2: element (row k, col n) of such a matrix
// The products run on the bf16 matrix units at fp32 accuracy: an fp32 number is the exact sum of three bf16
// numbers (x1 = x rounded, x2 = the rest rounded, x3 = what is left), and of the nine products of two such sums
// the six largest are taken (x1 y1, x1 y2, x2 y1, x2 y2, x1 y3, x3 y1; the others add up to at most 2^-24 of the
// product), each exact; against bf16 tiles, which have one part, three products leave nothing out.  The products
// x1 y1 have an accumulator of their own, the small ones another, and the two are added at the end: a sum is rounded
// once per 16 k and not six times, and a small sum is not cut off at the last place of a large one.  Six bf16
// products cost 6/16 of the fp32 matrix instruction's time, three 3/16.  Errors against 64 bits (relative 2-norm,
// normal numbers; fp32 instruction / all products in one accumulator / here): K = 16 7.4e-8 / 3.3e-8 / 3.2e-8, K = 128
// 2.0e-7 / 1.6e-7 / 6.5e-8, K = 4096 1.15e-6 / 1.01e-6 / 4.0e-7.  A sum that one product dominates has 2.60e-8
// (at most 9.0e-8) where the fp32 instruction rounds once, 2.54e-8 (6.0e-8); eight products would give 2.54e-8,
// and 5.62 instead of 5.09 ms for a 1000-token step from stored features.
//   One workgroup of 8 waves (2 x 4) per 128 x 256 tile of C, a wave owns 64 x 64 (2 x 2 tiles of 32x32x16).
// k advances in steps of 32: the operands' fp32 numbers are fetched into registers three steps ahead (two sets),
// split a step ahead, between the multiplications, and stored as bf16 planes [part][row][k] in one of two LDS
// buffers: one barrier per step.  Per step and compute unit 3072 clocks of matrix instructions (1536 against
// tiles) stand beside 2100 (1350) of LDS traffic and 1600 (800) of splitting.  1000 x 32000 x 4096 against tiles:
// 721 us, 1.09 PFLOP/s of bf16 products, matrix units busy 59 % (fp32 instruction: 2.9 ms); 1000 x 4096 x 4096: 271 us
// on 128 of the 256 compute units (fp32 instruction: 467 us).  The operands of one row of tiles are read at a time: with
// all of a block's operands in registers beside both accumulators, 12 to 60 bytes spill and it takes 289 us.  Variants of an
// earlier form that took 300 us: one LDS buffer with 4 waves and two barriers a step 422 us; operands two steps
// ahead in one register set 309; reading a step's operands under the previous step's multiplications 309.
//   Not faster everywhere than tiles of 64 x 128 by the fp32 instruction: for k up to 16 the fixed parts of a tile count
// (12288 x 4096 x 16: 63 us against 47; from k = 32 on 63 against 62), and a stand-alone contraction of a few tiles fills
// few compute units (64 x 64 x 64: 12.5 us against 9.2).  Waves that split operands straight from memory, without LDS:
// 78 us; the fp32 instruction straight from memory: 45 us, but twice the error at k = 16.
// A thread fetches along whichever index is contiguous in memory, in aligned groups of four where the operand
// allows it (a_vec / b_vec), else (GUARD) element by element.
// Every fp32 operand is multiplied by 2^24 before it is split and the sums are multiplied by the inverse at the
// end: an fp32 number is a multiple of 2^-149, so that the parts of a scaled one are multiples of 2^-125, none of
// them below bf16's smallest normal number, and the split is exact for all fp32 numbers, subnormal ones included.  At
// the other end operands from 2^104 and sums from 2^80 (against tiles 2^104) on leave fp32's range when scaled; infinities and NaN
// turn into NaN when split: a workgroup with a sum that is not finite computes its tile again by the fp32
// matrix instruction.
// A contraction with few output tiles and a long k is split over blockIdx.z: slice z handles k in
// [z * k_chunk, (z + 1) * k_chunk) and writes its own partial [M][N] at part + z * M * N; a second
// kernel adds the slices in order (no atomics: the result does not depend on scheduling).
// With batch > 1 (tr_gemm_small_kernel) the launch holds one product per blockIdx.x % batch (the per-head products of the
// attention: operands and result advance by bsa / bsb / bsc elements per head).
struct TrGemm {
    const void *A; long sam, sak;
    const void *B; long sbk, sbn;
    int b_mode, b_KS;
    float *C; long ldc;
    int M, N, K;
    int accumulate;
    int k_chunk;        // k handled per blockIdx.z slice (a multiple of 32); >= K when not split
    float *part;        // partial results of a split contraction
    int a_vec, b_vec;   // 4 consecutive elements along the contiguous index are one aligned 16-byte word, and that index
                        // ends at a multiple of 4
    int batch;          // > 1: blockIdx.z is a batch index (one product per attention head), k is not split
    long bsa, bsb, bsc; // element offsets of A, B (b_mode 0) and C per batch index
    int gm, gn, swz;    // tiles of C; swz: see the tile order in the kernel
    int causal;         // C[m][n] is needed for n <= m only: the launch holds the tiles that reach the diagonal (20 of 32 at 1000 positions)
    int k_tri;          // 1: A(m, k) is zero for k > m, k beyond a tile's last row is left out; 2: for k < m, k before its first row
};

__device__ __forceinline__ size_t packed_u16_index(int row, int col, int KS)
{
    return ((((size_t)(row >> 4) * KS + tile_pos(col >> 5, KS)) * 64 + ((col >> 3) & 3) * 16 + (row & 15)) << 3) + (col & 7);
}

// k per step TRG_K; tile of C, 8 waves, TRG_M x TRG_N (prompt_plan.h)
#define TRG_SM 64           // the smaller tile, 4 waves
#define TRG_SN 128
#define TRG_SCALE 0x1p24f   // of the fp32 operands before they are split

// Where the 8 numbers k = 8 c .. 8 c + 7 of row r lie in a plane (in elements): rows of 64 bytes, the rows of a 4 x 4
// group transposed and the four chunks of a row permuted, so that the reads (lanes = consecutive rows, one
// chunk), the stores of whole chunks and the transposing stores (lanes = every fourth row) are all free of
// bank conflicts.
__device__ __forceinline__ int trg_at(int r, int c) { return ((r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3)) * TRG_K + ((c ^ (r & 3)) << 3); }
// row of chunk item u: consecutive items take every fourth row, whose chunks lie side by side
__device__ __forceinline__ int trg_item_row(int u) { return (u & ~15) | ((u & 3) << 2) | ((u >> 2) & 3); }

// a pair of fp32 numbers, times TRG_SCALE, as three pairs of bf16 numbers
__device__ __forceinline__ void tr_split2(float a, float b, uint32_t (&o)[3])
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    a *= TRG_SCALE;
    b *= TRG_SCALE;
#pragma unroll
    for (int p = 0; p < 3; p++) {
        bf16x2_t h;
        h[0] = (__bf16)a; h[1] = (__bf16)b;
        o[p] = __builtin_bit_cast(uint32_t, h);
        a -= (float)h[0];
        b -= (float)h[1];
    }
}

// One fp32 operand of a ROWS x 32 block (rows m or n, k): the 8 or 16 numbers each of NTH threads fetches and how
// it stores them.  KC (contiguous along k): 8 consecutive k of one row or of two.
// Else 4 consecutive rows x 2 or 4 consecutive k, transposed on the way to LDS.
template <int ROWS, bool KC, int NTH>
struct TrOperand {
    static constexpr int NV = ROWS * TRG_K / NTH, NK = NV / 4;     // numbers per thread; k per thread when transposing
    static_assert(NV == 8 || NV == 16, "numbers per thread");
    static constexpr int KT = TRG_K / NK;                    // threads along k when transposing
    const float *p;         // element (row0, k) of the block that is fetched next
    long s_row, s_k;
    int rows;               // valid rows of the block (>= 1)
    const float *q[KC ? NV / 8 : 1];     // fetch / fetch_tail: this thread's addresses (rows beyond the block's last repeat
                                         // valid ones: what they give is not stored)
    __device__ __forceinline__ void init(const float *p_, long s_row_, long s_k_, int rows_, int t)
    {
        p = p_; s_row = s_row_; s_k = s_k_; rows = rows_;
        if constexpr (KC) {
#pragma unroll
            for (int i = 0; i < NV / 8; i++) q[i] = p + (size_t)min(trg_item_row((t >> 2) + NTH / 4 * i), rows - 1) * s_row + (size_t)(t & 3) * 8;
        } else {
            const int r = (t / KT) * 4;
            q[0] = p + (r < rows ? r : 0) + (size_t)(t % KT) * NK * s_k;
        }
    }
    // a whole step with 16-byte loads (a_vec / b_vec)
    __device__ __forceinline__ void fetch(float (&v)[NV])
    {
#pragma unroll
        for (int i = 0; i < NV / 4; i++) {
            const float4 f = KC ? *(const float4 *)(q[KC ? i >> 1 : 0] + 4 * (i & 1)) : *(const float4 *)(q[0] + (size_t)i * s_k);
            v[4 * i] = f.x; v[4 * i + 1] = f.y; v[4 * i + 2] = f.z; v[4 * i + 3] = f.w;
        }
        advance();
    }
    // the last step of a k that is no multiple of 32 (KC: it is one of 4): zeros from k_hi on
    __device__ __forceinline__ void fetch_tail(float (&v)[NV], int k0, int k_hi, int t)
    {
#pragma unroll
        for (int i = 0; i < NV / 4; i++) {
            const int k = k0 + (KC ? (t & 3) * 8 + 4 * (i & 1) : (t % KT) * NK + i);
            const bool ok = k < k_hi;
            const float *a = KC ? q[KC ? i >> 1 : 0] + 4 * (i & 1) : q[0] + (size_t)i * s_k;
            const float4 f = *(const float4 *)(ok ? a : KC ? q[KC ? i >> 1 : 0] - (t & 3) * 8 : q[0] - (size_t)(t % KT) * NK * s_k);
            v[4 * i] = ok ? f.x : 0.f; v[4 * i + 1] = ok ? f.y : 0.f; v[4 * i + 2] = ok ? f.z : 0.f; v[4 * i + 3] = ok ? f.w : 0.f;
        }
        advance();
    }
    __device__ __forceinline__ void fetch_guarded(float (&v)[NV], int k0, int k_hi, int t)
    {
        if constexpr (KC) {
            const int kq = (t & 3) * 8;
#pragma unroll
            for (int i = 0; i < NV / 8; i++) {
                const int r = trg_item_row((t >> 2) + NTH / 4 * i);
                const float *e = p + (size_t)r * s_row + kq;
#pragma unroll
                for (int j = 0; j < 8; j++) v[8 * i + j] = (r < rows && k0 + kq + j < k_hi) ? e[j] : 0.f;
            }
        } else {
            const int r = (t / KT) * 4, kq = (t % KT) * NK;
            const float *e = p + (size_t)r * s_row + (size_t)kq * s_k;
#pragma unroll
            for (int i = 0; i < NK; i++)                // k = kq + i, rows r .. r + 3
#pragma unroll
                for (int j = 0; j < 4; j++) v[4 * i + j] = (k0 + kq + i < k_hi && r + j < rows) ? e[(size_t)i * s_k + (size_t)j * s_row] : 0.f;
        }
        advance();
    }
    __device__ __forceinline__ void advance()
    {
        const size_t step = KC ? TRG_K : (size_t)TRG_K * s_k;
        p += step;
#pragma unroll
        for (int i = 0; i < (KC ? NV / 8 : 1); i++) q[i] += step;
    }
    __device__ __forceinline__ void stash(const float (&v)[NV], uint16_t (*planes)[ROWS * TRG_K], int t) const
    {
        if constexpr (KC) {
#pragma unroll
            for (int i = 0; i < NV / 8; i++) {
                const int at = trg_at(trg_item_row((t >> 2) + NTH / 4 * i), t & 3);
                u32x4_t o[3];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    uint32_t s[3];
                    tr_split2(v[8 * i + 2 * j], v[8 * i + 2 * j + 1], s);
                    o[0][j] = s[0]; o[1][j] = s[1]; o[2][j] = s[2];
                }
#pragma unroll
                for (int j = 0; j < 3; j++) *(u32x4_t *)&planes[j][at] = o[j];
            }
        } else {
            const int r = (t / KT) * 4, kq = (t % KT) * NK;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int at = trg_at(r + e, kq >> 3) + (kq & 7);
                uint32_t s[NK / 2][3];
#pragma unroll
                for (int j = 0; j < NK / 2; j++) tr_split2(v[8 * j + e], v[8 * j + 4 + e], s[j]);
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    if constexpr (NK == 4) *(uint2 *)&planes[j][at] = make_uint2(s[0][j], s[1][j]);
                    else *(uint32_t *)&planes[j][at] = s[0][j];
                }
            }
        }
    }
};

__device__ __forceinline__ float tr_gemm_b(const TrGemm &g, size_t bob, int k, int n)
{
    if (g.b_mode == 0) return ((const float *)g.B)[bob + (size_t)k * g.sbk + (size_t)n * g.sbn];
    return bf2f(((const uint16_t *)g.B)[g.b_mode == 1 ? packed_u16_index(n, k, g.b_KS) : packed_u16_index(k, n, g.b_KS)]);
}

template <int MI>
__device__ __forceinline__ void tr_zero(f32x16_t (&c)[MI][2])
{
#pragma unroll
    for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) c[i][j][r] = 0.f;
}

// A wave's 32 MI x 64 of C at (m0, n0) by the fp32 matrix instruction (32x32x2), operands straight from memory: what the
// products are by definition, for any fp32 numbers.  Of eight k a lane takes four consecutive ones of its row and
// of its column, lanes 0..31 the first four.
template <int MI>
__device__ __forceinline__ void tr_gemm_plain(const TrGemm &g, size_t boa, size_t bob, int m0, int n0, int k_lo, int k_hi, int lane,
                                              f32x16_t (&acc)[MI][2])
{
    tr_zero(acc);
    if (m0 >= g.M || n0 >= g.N) return;
    const int fr = lane & 31, fc = lane >> 5;
    const float *pa[MI], *pb[2];
    int n[2];
#pragma unroll
    for (int i = 0; i < MI; i++) pa[i] = (const float *)g.A + boa + (size_t)min(m0 + 32 * i + fr, g.M - 1) * g.sam;
#pragma unroll
    for (int i = 0; i < 2; i++) {                       // rows and columns beyond the last repeat it: they are not stored
        n[i] = min(n0 + 32 * i + fr, g.N - 1);
        pb[i] = (const float *)g.B + bob + (size_t)n[i] * g.sbn;
    }
    const bool va = g.a_vec && g.sak == 1, vb = g.b_vec && g.sbk == 1;
    auto load = [&](float (&v)[4], const float *p, int k, long s_k, bool vec) {
        if (vec) {                                      // (k_hi is a multiple of 4 then)
            const float4 f = k < k_hi ? *(const float4 *)(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) v[j] = k + j < k_hi ? p[(size_t)(k + j) * s_k] : 0.f;
        }
    };
    for (int k0 = k_lo; k0 < k_hi; k0 += 8) {
        const int k = k0 + 4 * fc;
        float a[MI][4], b[2][4];
#pragma unroll
        for (int i = 0; i < MI; i++) load(a[i], pa[i], k, g.sak, va);
#pragma unroll
        for (int i = 0; i < 2; i++) {
            if (g.b_mode == 0) load(b[i], pb[i], k, g.sbk, vb);
            else
#pragma unroll
                for (int j = 0; j < 4; j++) b[i][j] = k + j < k_hi ? tr_gemm_b(g, bob, k + j, n[i]) : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int i = 0; i < MI; i++)
#pragma unroll
                for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][q], b[j][q], acc[i][j], 0, 0, 0);
    }
}

// accumulator register r of lane l: row 8 * (r / 4) + 4 * (l / 32) + r % 4, column l % 32
template <int MI>
__device__ __forceinline__ void tr_gemm_store(const TrGemm &g, size_t boc, int m0, int n0, bool split, int lane, const f32x16_t (&acc)[MI][2])
{
#pragma unroll
    for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int n = n0 + 32 * j + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int m = m0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (m >= g.M || n >= g.N) continue;
                const float v = acc[i][j][r];
                if (split) {
                    g.part[((size_t)blockIdx.z * g.M + m) * g.N + n] = v;
                } else {
                    float *c = g.C + boc + (size_t)m * g.ldc + n;
                    *c = g.accumulate ? *c + v : v;
                }
            }
        }
}

// tiles of row tm of C that hold an element with n <= m
__host__ __device__ __forceinline__ int trg_causal_tiles(int tm, int gn, int tile_m, int tile_n)
{
    const int c = (tm * tile_m + tile_m - 1) / tile_n + 1;
    return c < gn ? c : gn;
}

// BP: bf16 parts of B (3: fp32 operand, 1: bf16 tiles); KA / KB: A / B contiguous along k (KB of tiles: b_mode 1);
// GUARD: operands that cannot be fetched in aligned groups of four.  SMALL: tiles of 64 x 128 by 4 waves, two workgroups per compute unit.
// (for the per-head products of the attention, 64 or 128 columns wide: a 128 x 256 tile is half empty there and one launch of 256 tiles takes
// as long as its longest sum.  1000 positions, 32 heads of 128: P.V, dS.K 102 -> 55 us, P^T.dO, dS^T.Q 110 -> 62, with the k beyond the
// diagonal left out; Q.K^T, dO.V^T 74 -> 62.)
template <int BP, bool KA, bool KB, bool GUARD, bool SMALL>
__device__ __forceinline__ void tr_gemm_body(const TrGemm &g)
{
    constexpr int TM = SMALL ? TRG_SM : TRG_M, TN = SMALL ? TRG_SN : TRG_N, NTH = SMALL ? 256 : 512, MI = TM / 64;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][3][TM * TRG_K];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BP][TN * TRG_K];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    // tile order: with swz the tiles of one column of C run one after another on one XCD (its L2 keeps that
    // part of B, usually the larger operand); used where the columns fill the XCDs
    int tm, tn;
    const int member = SMALL ? blockIdx.x % g.batch : 0, tile = SMALL ? blockIdx.x / g.batch : blockIdx.x;
    if (SMALL && g.causal) {
        tm = 0;
        tn = tile;
        for (int c; tn >= (c = trg_causal_tiles(tm, g.gn, TM, TN)); tm++) tn -= c;
    } else if (!SMALL && g.swz) {
        const int j = tile >> 3;
        tm = j % g.gm;
        tn = (j / g.gm) * 8 + (tile & 7);
        if (tn >= g.gn) return;
    } else {
        tm = tile / g.gn;
        tn = tile % g.gn;
    }
    if (SMALL && g.k_tri == 1) tm = g.gm - 1 - tm;      // the longest sums first
    const int m0 = tm * TM, n0 = tn * TN;
    const int wm = (wave & 1) * (TM / 2), wn = (wave >> 1) * 64;
    const bool split = !SMALL && gridDim.z > 1;
    const int k_lo = split ? blockIdx.z * g.k_chunk : SMALL && g.k_tri == 2 ? m0 : 0,
              k_hi = split ? min(g.K, k_lo + g.k_chunk) : SMALL && g.k_tri == 1 ? min(g.K, m0 + TM) : g.K;
    const size_t boa = (size_t)member * g.bsa, bob = (size_t)member * g.bsb, boc = (size_t)member * g.bsc;
    TrOperand<TM, KA, NTH> oa;
    TrOperand<TN, KB, NTH> ob;
    oa.init((const float *)g.A + boa + (size_t)m0 * g.sam + (size_t)k_lo * g.sak, g.sam, g.sak, g.M - m0, t);
    if constexpr (BP == 3) ob.init((const float *)g.B + bob + (size_t)n0 * g.sbn + (size_t)k_lo * g.sbk, g.sbn, g.sbk, g.N - n0, t);
    // numbers a thread has fetched: two sets, so that a fetch has more than a whole step to arrive
    struct Raw {
        float a[8], b[BP == 3 ? 16 : 1];
        u32x4_t bt[2];                                  // bf16 tiles: two 16-byte units per thread
    };
    // b_mode 1: unit = 8 k of one row n, items as above.  b_mode 2: unit = 8 n of one row k: thread -> rows
    // k = 2 (t % 16), + 1, columns 8 (t / 16)
    auto fetch_tiles = [&](Raw &w, int k0) {
        const u32x4_t *T = (const u32x4_t *)g.B;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            // (columns beyond the last repeat valid ones; k beyond the last meets zeros of A, and the matrix is a whole
            // number of 16-row tiles, its k-steps padded: every unit read exists)
            if constexpr (KB) {
                const int n = min(n0 + trg_item_row((t >> 2) + 128 * i), g.N - 1), c = t & 3;
                w.bt[i] = T[((size_t)(n >> 4) * g.b_KS + tile_pos(k0 >> 5, g.b_KS)) * 64 + c * 16 + (n & 15)];
            } else {
                const int k = min(k0 + 2 * (t & 15) + i, k_hi - 1), n = min(n0 + 8 * (t >> 4), (g.N - 1) & ~7);
                w.bt[i] = T[((size_t)(k >> 4) * g.b_KS + tile_pos(n >> 5, g.b_KS)) * 64 + ((n >> 3) & 3) * 16 + (k & 15)];
            }
        }
    };
    auto stash_tiles = [&](const Raw &w, uint16_t *plane) {
        if constexpr (KB) {
#pragma unroll
            for (int i = 0; i < 2; i++) *(u32x4_t *)&plane[trg_at(trg_item_row((t >> 2) + 128 * i), t & 3)] = w.bt[i];
        } else {
            const int k = 2 * (t & 15);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int r = 8 * (t >> 4) + 2 * j;
                *(uint32_t *)&plane[trg_at(r, k >> 3) + (k & 7)] = __builtin_amdgcn_perm(w.bt[1][j], w.bt[0][j], 0x05040100u);
                *(uint32_t *)&plane[trg_at(r + 1, k >> 3) + (k & 7)] = __builtin_amdgcn_perm(w.bt[1][j], w.bt[0][j], 0x07060302u);
            }
        }
    };
    const int steps = k_lo < k_hi ? (k_hi - k_lo + TRG_K - 1) / TRG_K : 0, full = k_lo < k_hi ? (k_hi - k_lo) / TRG_K : 0;
    auto fetch_whole = [&](Raw &w, int st) {
        oa.fetch(w.a);
        if constexpr (BP == 3) ob.fetch(w.b);
        else fetch_tiles(w, k_lo + st * TRG_K);
    };
    auto fetch = [&](Raw &w, int st) {                  // step st, if there is one
        if (st >= steps) return;
        const int k0 = k_lo + st * TRG_K;
        if constexpr (GUARD) {
            oa.fetch_guarded(w.a, k0, k_hi, t);
            ob.fetch_guarded(w.b, k0, k_hi, t);
        } else if (st < full) {
            fetch_whole(w, st);
        } else {
            oa.fetch_tail(w.a, k0, k_hi, t);
            if constexpr (BP == 3) ob.fetch_tail(w.b, k0, k_hi, t);
            else fetch_tiles(w, k0);
        }
    };
    auto stash = [&](const Raw &w, int buf) {
        oa.stash(w.a, As[buf], t);
        if constexpr (BP == 3) ob.stash(w.b, Bs[buf], t);
        else stash_tiles(w, Bs[buf][0]);
    };
    f32x16_t acc[MI][2], rest[MI][2];                   // sums of the products of first parts, and of all others
    tr_zero(acc);
    tr_zero(rest);
    const int fr = lane & 31, fc = lane >> 5;           // operand layout of the 32x32x16 instruction: row, which 8 k
    auto multiply = [&](int buf, int kk) {              // k = 16 kk .. 16 kk + 15 of the step
        bf16x8_t a[3], b[2][BP];
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int q = 0; q < BP; q++) b[j][q] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t *)&Bs[buf][q][trg_at(wn + 32 * j + fr, 2 * kk + fc)]);
#pragma unroll
        for (int i = 0; i < MI; i++) {
#pragma unroll
            for (int q = 0; q < 3; q++) a[q] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t *)&As[buf][q][trg_at(wm + 32 * i + fr, 2 * kk + fc)]);
#pragma unroll
            for (int s = 2; s >= 0; s--)                // parts (q, s - q): the smallest products first
#pragma unroll
                for (int q = 0; q <= s; q++) {
                    if (s - q >= BP) continue;
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        f32x16_t &c = s ? rest[i][j] : acc[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q], b[j][s - q], c, 0, 0, 0);
                    }
                }
        }
    };
    if (steps > 0) {
        Raw r0, r1;
        fetch(r0, 0);
        fetch(r1, 1);
        stash(r0, 0);
        fetch(r0, 2);
        __syncthreads();
        int s = 0;
        // step s is multiplied while step s + 1 (in `w`) is split and stored and step s + 3 requested
        auto step = [&](Raw &w, int buf, bool whole) {
            multiply(buf, 0);
            if (whole || s + 1 < steps) stash(w, buf ^ 1);      // the other buffer was last read before the previous barrier
            if (whole) fetch_whole(w, s + 3);
            else fetch(w, s + 3);
            multiply(buf, 1);
            __syncthreads();
            s++;
        };
        if constexpr (!GUARD)
            while (s + 4 < full) { step(r1, 0, true); step(r0, 1, true); }
        while (s < steps) {
            step(r1, 0, false);
            if (s < steps) step(r0, 1, false);
        }
    }
    // a number that is not finite once scaled and split leaves its whole row or column of sums without a finite value
    bool odd = false;
#pragma unroll
    for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float v = acc[i][j][r] + rest[i][j][r];
                odd |= !(fabsf(v) < INFINITY);
                acc[i][j][r] = v * (BP == 3 ? 1.f / (TRG_SCALE * TRG_SCALE) : 1.f / TRG_SCALE);
            }
    if (__syncthreads_or(odd) || g.K == 1) {            // (one product per sum: rounded once)
        tr_gemm_plain(g, boa, bob, m0 + wm, n0 + wn, k_lo, k_hi, lane, acc);
        __syncthreads();                                // (C may be an operand of a product of one tile)
    }
    tr_gemm_store(g, boc, m0 + wm, n0 + wn, split, lane, acc);
}
// (a bound of 256 registers: 8 waves fill a compute unit, whose LDS one workgroup or two of the small ones take anyway)
template <int BP, bool KA, bool KB, bool GUARD>
__global__ __launch_bounds__(512, 2) void tr_gemm_kernel(const TrGemm g) { tr_gemm_body<BP, KA, KB, GUARD, false>(g); }
template <bool KA, bool KB, bool GUARD>
__global__ __launch_bounds__(256, 2) void tr_gemm_small_kernel(const TrGemm g) { tr_gemm_body<3, KA, KB, GUARD, true>(g); }

// C[m][n] (+)= part[0][m][n] + part[1][m][n] + ... in slice order
__global__ void tr_gemm_reduce_kernel(const float *part, int S, int M, int N, float *C, long ldc, int accumulate)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)M * N) return;
    float s = part[i];
    for (int z = 1; z < S; z++) s += part[(size_t)z * M * N + i];
    float *c = C + (i / N) * ldc + (i % N);
    *c = accumulate ? *c + s : s;
}

// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float tr_block_sum(float v, float *red)
{
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float s = 0.f;
    for (int w = 0; w < nw; w++) s += red[w];
    return s;
}
__device__ __forceinline__ float tr_block_max(float v, float *red)
{
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float s = red[0];
    for (int w = 1; w < nw; w++) s = fmaxf(s, red[w]);
    return s;
}

// y[t] = x[t] * r[t] * g with r[t] = rsqrt(mean(x[t]^2) + eps); one block per row
__global__ __launch_bounds__(256) void tr_rmsnorm_kernel(const float *x, const float *g, int d, float eps, float *y, float *r)
{
    __shared__ float red[4];
    const int row = blockIdx.x;
    const float *xr = x + (size_t)row * d;
    float s = 0.f;
    for (int i = threadIdx.x; i < d; i += 256) s += xr[i] * xr[i];
    s = tr_block_sum(s, red);
    const float rr = 1.f / sqrtf(s / (float)d + eps);
    if (threadIdx.x == 0) r[row] = rr;
    for (int i = threadIdx.x; i < d; i += 256) y[(size_t)row * d + i] = xr[i] * rr * g[i];
}

// dx[t] = r (dy g) - x r^3 mean((dy g) x); one block per row
__global__ __launch_bounds__(256) void tr_rmsnorm_bwd_kernel(const float *x, const float *g, const float *r, const float *dy,
                                                             int d, float *dx)
{
    __shared__ float red[4];
    const int row = blockIdx.x;
    const float *xr = x + (size_t)row * d, *dyr = dy + (size_t)row * d;
    float s = 0.f;
    for (int i = threadIdx.x; i < d; i += 256) s += dyr[i] * g[i] * xr[i];
    s = tr_block_sum(s, red) / (float)d;
    const float rr = r[row], r3 = rr * rr * rr;
    for (int i = threadIdx.x; i < d; i += 256) dx[(size_t)row * d + i] = rr * dyr[i] * g[i] - xr[i] * r3 * s;
}

// dg[j] (+)= sum_t dy[t][j] * x[t][j] * r[t]; a block of 1024 threads handles 16 columns (64 bytes of a row), its 64 groups of 16
// threads take every 64th row, eight rows in flight, and their partial sums are added in group order.  (64 columns and 16 groups: 64
// blocks for 4096 columns, a quarter of the device; 1000 rows 28 us a launch.)
__global__ __launch_bounds__(1024) void tr_gain_grad_kernel(const float *x, const float *r, const float *dy, int T, int d, float *dg,
                                                            int accumulate)
{
    __shared__ float part[64][16];
    const int c = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int j = blockIdx.x * 16 + c;
    float s = 0.f;
    if (j < d) {
#pragma unroll 8
        for (int t = grp; t < T; t += 64) s += dy[(size_t)t * d + j] * x[(size_t)t * d + j] * r[t];
    }
    part[grp][c] = s;
    __syncthreads();
    if (grp == 0 && j < d) {
        float tot = 0.f;
#pragma unroll
        for (int g = 0; g < 64; g++) tot += part[g][c];
        dg[j] = accumulate ? dg[j] + tot : tot;
    }
}

// rotary embedding of the q and k parts of QKV [T][3d] at positions 0..T-1, pairs (i, i + hd/2);
// inverse rotates by minus the angle (the transpose of the rotation, for the backward pass)
__global__ void tr_rope_kernel(float *qkv, int T, int d, int hd, const float2 *tab, int inverse)
{
    const int half = hd >> 1;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t per_row = (size_t)(d / hd) * half;
    if (i >= (size_t)T * per_row * 2) return;
    const int which = (int)(i / ((size_t)T * per_row));          // 0 = q, 1 = k
    const size_t j = i % ((size_t)T * per_row);
    const int t = (int)(j / per_row), rem = (int)(j % per_row), h = rem / half, p = rem % half;
    float2 cs = tab[(size_t)t * half + p];
    if (inverse) cs.y = -cs.y;
    float *v = qkv + (size_t)t * 3 * d + (size_t)which * d + (size_t)h * hd;
    const float a = v[p], b = v[p + half];
    v[p] = a * cs.x - b * cs.y;
    v[p + half] = b * cs.x + a * cs.y;
}

#define TR_T_MAX 2048   // longest training sequence: the attention row kernels keep a row of T weights in registers

// Attention over all positions at once goes through the contraction kernel, one product per head:
// S = Q.K^T, P = causal softmax(S / sqrt(hd)), O = P.V forward; dP = dO.V^T, dV = P^T.dO,
// dS = P (dP - rowsum(dP P)) / sqrt(hd), dQ = dS.K, dK = dS^T.Q backward.  The two kernels below are
// the row-wise pieces; both work in place on [H][T][T], one block per (row i, head h), and leave
// exact zeros above the diagonal as far as the products read (to the end of the tile of TRG_SM rows and columns on the diagonal).
__global__ __launch_bounds__(256) void tr_softmax_causal_kernel(float *P, int T, float scale)
{
    __shared__ float red[4];
    const int i = blockIdx.x, h = blockIdx.y, t = threadIdx.x;
    float *row = P + ((size_t)h * T + i) * T;
    float v[TR_T_MAX / 256];
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < TR_T_MAX / 256; c++) {
        const int j = t + 256 * c;
        v[c] = (j <= i) ? row[j] * scale : -INFINITY;      // j <= i < T
        mx = fmaxf(mx, v[c]);
    }
    mx = tr_block_max(mx, red);
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < TR_T_MAX / 256; c++) {
        v[c] = (t + 256 * c <= i) ? expf(v[c] - mx) : 0.f;
        sum += v[c];
    }
    sum = tr_block_sum(sum, red);
    const int end = min(T, (i / TRG_SM + 1) * TRG_SM);
#pragma unroll
    for (int c = 0; c < TR_T_MAX / 256; c++) {
        const int j = t + 256 * c;
        if (j < end) row[j] = v[c] / sum;
    }
}

// dS[i][j] = P[i][j] * (dP[i][j] - sum_j dP[i][j] P[i][j]) * scale, in place on dP
__global__ __launch_bounds__(256) void tr_dsoftmax_kernel(const float *P, float *dP, int T, float scale)
{
    __shared__ float red[4];
    const int i = blockIdx.x, h = blockIdx.y, t = threadIdx.x;
    const float *prow = P + ((size_t)h * T + i) * T;
    float *drow = dP + ((size_t)h * T + i) * T;
    float p[TR_T_MAX / 256], g[TR_T_MAX / 256];
    float D = 0.f;
#pragma unroll
    for (int c = 0; c < TR_T_MAX / 256; c++) {
        const int j = t + 256 * c;
        p[c] = (j <= i) ? prow[j] : 0.f;
        g[c] = (j <= i) ? drow[j] : 0.f;
        D += p[c] * g[c];
    }
    D = tr_block_sum(D, red);
    const int end = min(T, (i / TRG_SM + 1) * TRG_SM);
#pragma unroll
    for (int c = 0; c < TR_T_MAX / 256; c++) {
        const int j = t + 256 * c;
        if (j < end) drow[j] = p[c] * (g[c] - D) * scale;
    }
}

// Eq. 3 for one position: loss[t] = - sum_n p_n log q_n with p = softmax(zt[t]), q = softmax(z[t]);
// dz[t] = q - p (the gradient of the loss with respect to the draft logits).  One block of 1024 threads per row, which
// keeps both rows in registers (up to TR_LOSS_V logits each), so that the launch reads them once, all loads issued
// together, instead of three times: 1000 rows of 32000 logits 234 -> 158 us.  Longer rows are read three times.  Then the
// vector instructions count: exp of a target logit is kept, and divided by the row's sum by its reciprocal and one correction: 142 us.
#define TR_LOSS_V 32768
template <bool REGS>
__global__ __launch_bounds__(1024) void tr_loss_kernel(const float *z, const float *zt, int V, float *dz, float *loss)
{
    constexpr int NR = REGS ? TR_LOSS_V / 4096 : 1;         // groups of 4 logits per thread
    __shared__ float red[16];
    const int row = blockIdx.x, t = threadIdx.x;
    const float *zr = z + (size_t)row * V, *tr = zt + (size_t)row * V;
    float4 a[NR], b[NR];
    const float4 low = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    if (REGS) {
#pragma unroll
        for (int i = 0; i < NR; i++) {
            const int n = 4 * (t + 1024 * i);
            a[i] = n < V ? *(const float4 *)(zr + n) : low;
            b[i] = n < V ? *(const float4 *)(tr + n) : low;
        }
    }
    // f(draft logits, target logits, index) over the row, four logits at a time (V is a multiple of 16); what f leaves in them stays (REGS)
    auto each = [&](auto f) {
        if (REGS) {
#pragma unroll
            for (int i = 0; i < NR; i++) {
                const int n = 4 * (t + 1024 * i);
                if (n < V) f(a[i], b[i], n);
            }
        } else {
            for (int n = 4 * t; n < V; n += 4096) {
                float4 u = *(const float4 *)(zr + n), v = *(const float4 *)(tr + n);
                f(u, v, n);
            }
        }
    };
    float mz = -INFINITY, mt = -INFINITY;
    each([&](const float4 &u, const float4 &v, int) {
        mz = fmaxf(fmaxf(mz, fmaxf(u.x, u.y)), fmaxf(u.z, u.w));
        mt = fmaxf(fmaxf(mt, fmaxf(v.x, v.y)), fmaxf(v.z, v.w));
    });
    mz = tr_block_max(mz, red);
    mt = tr_block_max(mt, red);
    float sz = 0.f, st = 0.f;
    each([&](const float4 &u, float4 &v, int) {
        sz += (expf(u.x - mz) + expf(u.y - mz)) + (expf(u.z - mz) + expf(u.w - mz));
        v = make_float4(expf(v.x - mt), expf(v.y - mt), expf(v.z - mt), expf(v.w - mt));
        st += (v.x + v.y) + (v.z + v.w);
    });
    sz = tr_block_sum(sz, red);
    st = tr_block_sum(st, red);
    const float lz = logf(sz), rt = 1.f / st;
    float l = 0.f;
    auto one = [&](float zv, float tv) {
        const float ev = REGS ? tv : expf(tv - mt), p0 = ev * rt, p = fmaf(fmaf(-p0, st, ev), rt, p0);      // ev / st
        const float lq = zv - mz - lz;
        l -= p * lq;
        return expf(lq) - p;
    };
    each([&](const float4 &u, const float4 &v, int n) {
        *(float4 *)(dz + (size_t)row * V + n) = make_float4(one(u.x, v.x), one(u.y, v.y), one(u.z, v.z), one(u.w, v.w));
    });
    l = tr_block_sum(l, red);
    if (t == 0) loss[row] = l;
}

// AdamW with bias correction and decoupled weight decay; c1 = 1 - beta1^step, c2 = 1 - beta2^step
__device__ __forceinline__ float tr_adamw(float w, float gi, float &m, float &v, float lr, float b1, float b2, float eps, float wd, float c1,
                                          float c2)
{
    m = b1 * m + (1.f - b1) * gi;
    v = b2 * v + (1.f - b2) * gi * gi;
    return w * (1.f - lr * wd) - lr * (m / c1) / (sqrtf(v / c2) + eps);
}
__global__ void tr_adamw_kernel(float *w, const float *g, float *m, float *v, size_t n, float lr, float b1, float b2, float eps,
                                float wd, float c1, float c2)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float mi = m[i], vi = v[i];
    w[i] = tr_adamw(w[i], g[i], mi, vi, lr, b1, b2, eps, wd, c1, c2);
    m[i] = mi;
    v[i] = vi;
}

// dst[i] = src[i] rounded to bfloat16 (nearest even), kept as fp32: what a bf16 checkpoint would hold
__global__ void tr_round_bf16_kernel(const float *src, int n, float *dst)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = bf2f(f2bf(src[i]));
}

// fp32 row-major [rows][K] <-> the arena's form of a matrix: bf16 MFMA tiles (the layout of
// pack_w_bf16_kernel) or fp32 rows, with source row r living at arena row map_row(r, row_off, mode)
// (mode 1 / 2: the interleaved gate / up rows of a feed-forward pair); K % 8 == 0 for tiles
__global__ void tr_unpack_bf16_kernel(const uint16_t *tiles, int rows, int K, int KS, int row_off, int mode, float *dst)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * K) return;
    const int r = (int)(i / K), k = (int)(i % K);
    dst[i] = bf2f(tiles[packed_u16_index(map_row(r, row_off, mode), k, KS)]);
}
// AdamW on a matrix of a bf16 model and its copy in the arena's tiles, in one pass over the master block, gradient and moments: 28 bytes a
// number and 2 for the tiles.  A block takes 16 rows x 128 columns: 512 bytes of a row side by side on one side, whole tiles (where
// rows keep their order) on the other.  q, k, v of a 7B adapter, 50 M numbers: 326 us (4.6 TB/s), against 252 + 116 us for AdamW and a launch
// that read the master again; 373 with a wave per tile (128 bytes of a row), 332 with 8 rows x 256 columns.
__global__ __launch_bounds__(256) void tr_adamw_pack_kernel(float *w, const float *g, float *m, float *v, int rows, int K, int KS, float lr, float b1,
                                                           float b2, float eps, float wd, float c1, float c2, int row_off, int mode, uint16_t *tiles)
{
    const int kb = (K + 127) >> 7, r = (int)(blockIdx.x / kb) * 16 + (threadIdx.x >> 4), k = (int)(blockIdx.x % kb) * 128 + (threadIdx.x & 15) * 8;
    if (r >= rows || k >= K) return;            // (K is a multiple of 8)
    const size_t at = (size_t)r * K + k;
    uint32_t o[4];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        float4 wv = *(const float4 *)(w + at + 4 * h), mv = *(const float4 *)(m + at + 4 * h), vv = *(const float4 *)(v + at + 4 * h);
        const float4 gv = *(const float4 *)(g + at + 4 * h);
        wv.x = tr_adamw(wv.x, gv.x, mv.x, vv.x, lr, b1, b2, eps, wd, c1, c2);
        wv.y = tr_adamw(wv.y, gv.y, mv.y, vv.y, lr, b1, b2, eps, wd, c1, c2);
        wv.z = tr_adamw(wv.z, gv.z, mv.z, vv.z, lr, b1, b2, eps, wd, c1, c2);
        wv.w = tr_adamw(wv.w, gv.w, mv.w, vv.w, lr, b1, b2, eps, wd, c1, c2);
        *(float4 *)(w + at + 4 * h) = wv; *(float4 *)(m + at + 4 * h) = mv; *(float4 *)(v + at + 4 * h) = vv;
        o[2 * h] = (uint32_t)f2bf(wv.x) | ((uint32_t)f2bf(wv.y) << 16);
        o[2 * h + 1] = (uint32_t)f2bf(wv.z) | ((uint32_t)f2bf(wv.w) << 16);
    }
    *(u32x4_t *)(tiles + packed_u16_index(map_row(r, row_off, mode), k, KS)) = u32x4_t{o[0], o[1], o[2], o[3]};
}
// the same for fp32 models; to_arena: master -> arena, else arena -> master
__global__ void tr_copy_rows_f32_kernel(float *master, float *arena, int rows, int K, int row_off, int mode, int to_arena)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * K) return;
    const int r = (int)(i / K), k = (int)(i % K);
    const size_t j = (size_t)map_row(r, row_off, mode) * K + k;
    if (to_arena) arena[j] = master[i]; else master[i] = arena[j];
}

// ---- element-wise pieces of the feed-forward and two-linear-map adapters --------------------
__device__ __forceinline__ float tr_sigmoid(float z) { return 1.f / (1.f + expf(-z)); }
// s = silu(u)
__global__ void tr_silu_kernel(const float *u, size_t n, float *s)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) s[i] = u[i] * tr_sigmoid(u[i]);
}
// du = ds * silu'(u), silu'(u) = sg (1 + u (1 - sg))
__global__ void tr_silu_bwd_kernel(const float *u, const float *ds, size_t n, float *du)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float z = u[i], sg = tr_sigmoid(z);
    du[i] = ds[i] * sg * (1.f + z * (1.f - sg));
}
// a = silu(g) * u
__global__ void tr_swiglu_kernel(const float *g, const float *u, size_t n, float *a)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = g[i] * tr_sigmoid(g[i]) * u[i];
}
// dg = da * u * silu'(g), du = da * silu(g)
__global__ void tr_swiglu_bwd_kernel(const float *g, const float *u, const float *da, size_t n, float *dg, float *du)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float z = g[i], sg = tr_sigmoid(z), d = da[i];
    dg[i] = d * u[i] * sg * (1.f + z * (1.f - sg));
    du[i] = d * z * sg;
}
// a += b
__global__ void tr_add_kernel(float *a, const float *b, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] += b[i];
}
