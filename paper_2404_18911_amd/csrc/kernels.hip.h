// Device code of libkangaroo: hand-written HIP kernels for gfx950 (CDNA4, 64-wide wavefronts).
//
// Every decode forward of Kangaroo (draft step of M^s = A o M^b[:l], verification by M^b[l:],
// Sections 3.1-3.2 and Figure 2) has at most 8 rows, so each projection is a weight-streaming
// product bounded by HBM bandwidth (Section 1).  The design here:
//   * weights are re-tiled once at load time into 1 KB tiles of 16 rows x 32 k in exactly the
//     register layout of the A operand of v_mfma_f32_16x16x32_bf16, so a wavefront streams
//     contiguous memory with 16-byte loads straight into MFMA operands (no LDS, no conversion);
//   * activations stay fp32; a row is split into bf16 hi + bf16 lo parts that occupy columns
//     m and m+8 of the 16-column B operand, so one MFMA gives fp32-grade products for 8 rows;
//   * the result for a row never depends on how many other rows are in the batch, which keeps
//     verification bit-identical to one-token decoding (needed for token-exact losslessness);
//   * RMSNorm is folded in: the producer's epilogue stores x*g (hi/lo) and per-tile sums of
//     squares, the consumer's epilogue multiplies by rsqrt(mean square + eps).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

#define KG_ROWS 8

enum { EPI_PLAIN = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_HEAD = 3, EPI_SILU = 4, EPI_QKV = 5, EPI_FEATURE = 6 };

// What a projection kernel does with a finished 16-row tile y[16][8].
struct Epi {
    int kind;
    int M;              // live rows (<= 8)
    int N;              // output features of this projection
    // RMSNorm scale of the projection's input rows: rsqrt(sum(ssq_in[t][m]) * inv_d + eps); null = 1
    const float *ssq_in;
    int nt_in;
    float inv_d, eps;
    const float *scale_in;  // prompt passes in 128-row workgroups: the scales themselves, one per row (pf_rms_scale_kernel)
    // EPI_PLAIN: out[(m + row_shift)][n] = y * scale, rows with m + row_shift < 0 are dropped
    float *out;
    int row_shift;
    int k_pairs;        // head_dim where the key rows of a q, k, v projection are stored in rotation pairs (see map_row), else 0
    // EPI_HEAD: as EPI_PLAIN, plus per-tile statistics of z * inv_temp for the rows kept:
    // hstat[(row * N / 16 + tile) * 4 + {0,1,2}] = max, sum exp(. - max), arg-max index (as float bits):
    // the statistics of one row lie together, for the block that reduces them
    float *hstat;
    float inv_temp;
    // EPI_RESID: x = res[m][n] + y; xout[m][n] = x; act_out <- x * gain[n]; ssq_out[tile][m] = sum x^2
    const float *res;
    float *xout;
    // EPI_SILU: act_out <- silu(y * scale) at K index n (the first map of the two-linear-map adapter)
    // EPI_RESID / EPI_SWIGLU: activation for the next projection (K index = n, or tile*8+i for SwiGLU)
    void *act_out;
    int act_pair;       // prompt passes: layout of act_out, see pf_act_ptr (0 = the 8-row layout above)
    int act_K;
    const float *gain;
    float *ssq_out;
};

// EPI_FEATURE (early features, decode launches): as EPI_RESID with the rows of act_out and ssq_out from act_row on; and once more for
// layer l (act2 <- x * gain2 and ssq2 from row row2 on), and as fp32 rows (xout2, may be null).  An argument of the kernels that have this
// epilogue only: 40 more bytes in every bf16 projection's arguments cost 0.6 % of a 26 us launch.  (gemv_f32_kernel has it for all its
// launches: stand-alone fp32 products of 256 x 256 to 2048 x 1024 took what they took without it, within 2 %.)
struct Feature {
    int act_row, row2;
    void *act2;
    const float *gain2;
    float *ssq2, *xout2;
};

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// A value the compiler must materialise in a register: what is computed from it cannot be fused
// with what computed it (a * b + c stays a rounded product followed by a sum), so that the same
// source expression rounds alike in every kernel it is written in.
__device__ __forceinline__ float rounded(float v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// device-scope relaxed accesses for data exchanged between workgroups inside one kernel
__device__ __forceinline__ void st_dev(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float ld_dev(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Store activation value v of row m, feature k, for a consumer projection with K features.
// BF: bf16 hi/lo parts in 1 KB tiles per 32 features, [k/32][row m][part hi|lo][k%32/8][k%8]: the
// 128 bytes of one batch row and k-step are contiguous, so a wave that needs M rows touches M cache
// lines per tile.  MFMA lane (g = lane/16, column j) reads slot ((j%8)*2 + j/8)*4 + g, see b_slot().
// else: plain float [m][K].
template <bool BF>
__device__ __forceinline__ void store_act(void *buf, int K, int m, int k, float v)
{
    if (BF) {
        // the low part is taken from the rounded fp32 value v (fused with a product that made v it
        // would use the unrounded product, and then depend on the caller's expression)
        v = rounded(v);
        uint16_t hi = f2bf(v);
        uint16_t lo = f2bf(v - bf2f(hi));
        uint16_t *p = (uint16_t *)buf;
        size_t base = (size_t)(k >> 5) * 512 + (size_t)(m * 8 + ((k >> 3) & 3)) * 8 + (k & 7);
        p[base] = hi;
        p[base + 32] = lo;
    } else {
        ((float *)buf)[(size_t)m * K + k] = v;
    }
}
// 16-byte slot of MFMA lane `lane` inside a B-operand tile (column j < 8: hi part of row j; j >= 8: lo part of row j-8)
__device__ __forceinline__ int b_slot(int lane) { return (((lane & 7) * 2 + ((lane >> 3) & 1)) << 2) + (lane >> 4); }

// scale[m] = rsqrt(mean square of the input row + eps), from per-tile partial sums, fixed order.
// Wave w of an 8-wave block serves batch row w.  The partials (at most 8 per lane: d <= 8192) are
// fetched by scale_fetch at kernel start so that their latency hides behind the weight stream;
// scale_finish reduces them.  Result valid after the next __syncthreads().
// Loads of which some lanes want nothing go through a buffer whose bounds the others respect (a lane out of bounds gets 0 and moves no
// bytes): a masked load is a branch around it, after which the compiler no longer knows how many loads are in flight and waits for
// more of them than are needed, in a weight stream for the very chunk it has just asked for.  us per launch in a 7B request, masked
// activation loads and sums of squares / here: q,k,v 17.2 / 16.7, o_proj 8.0 / 7.6, gate+up 28.8 / 28.3, LM head 40.1 / 38.8; seven
// rows: q,k,v 18.9 / 18.4, gate+up 32.6 / 32.3.  Stand-alone, 4096 x 4096, one row 7.31 / 6.76; 13840 x 5136, 7 rows 26.3 / 24.5.
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t buffer_of(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
// a pointer that is the same in all lanes, where the compiler cannot tell
template <typename T> __device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}
#define BUFFER_NONE 0x80000000u     // a byte offset no buffer here reaches

struct ScaleRegs { float v[8]; };
__device__ __forceinline__ void scale_fetch(const float *ssq_in, int M, int nt_in, ScaleRegs &r)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 8; j++) r.v[j] = 0.f;
    if (!ssq_in || wave >= M) return;
    const buffer_t b = buffer_of(ssq_in, (uint32_t)nt_in * KG_ROWS * 4);
#pragma unroll
    for (int j = 0; j < 8; j++)
        r.v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (lane + 64 * j) * KG_ROWS * 4 + wave * 4, 0, 0));
}
__device__ __forceinline__ void scale_finish(const Epi &e, const ScaleRegs &r, float *sc)
{
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave < e.M) {
        float s = 1.f;
        if (e.ssq_in) {
            s = 0.f;
#pragma unroll
            for (int j = 0; j < 8; j++) s += rounded(r.v[j]);       // (or the compiler adds, and waits, where the loads are)
            for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
            s = rsqrtf(fmaf(s, e.inv_d, e.eps));
        }
        if (lane == 0) sc[wave] = s;
    }
}

// Epilogue on a finished tile: yt[16][8] in LDS (row in tile, batch row), all 256 threads call it.
// Prompt passes: where the producer of a projection's input puts row m of 8-row block b, feature k.
// Returns the address of the hi part; the lo part lies lo_off elements further.
// pair = 0: the block's own tiles [k/32][row m][hi|lo][k%32/8][k%8], what the 8-row kernels read.
// pair = 1: tiles of two blocks, [k/32][hi|lo][lane (8 (b % 2) + m) + 16 (k%32/8)][k%8]: the B operand of a
// 16-row MFMA as one contiguous KB, which a mover wave fetches with one coalesced access per four lanes
// (gathered from the 8-row layout the same tile costs one access per lane: neighbouring lanes then
// read 128 bytes apart).
__device__ __forceinline__ uint16_t *pf_act_ptr(void *base, size_t blk_bytes, int b, int m, int k, int pair, int &lo_off)
{
    uint16_t *p = (uint16_t *)base;
    if (pair) {
        lo_off = 512;
        return p + (size_t)(b >> 1) * blk_bytes + (size_t)(k >> 5) * 1024 + (size_t)(((b & 1) * 8 + m) + 16 * ((k >> 3) & 3)) * 8 + (k & 7);
    }
    lo_off = 32;
    return p + (size_t)b * (blk_bytes >> 1) + (size_t)(k >> 5) * 512 + (size_t)(m * 8 + ((k >> 3) & 3)) * 8 + (k & 7);
}
// one value, split as store_act splits it
__device__ __forceinline__ void store_act_pf(void *base, size_t blk_bytes, int b, int m, int k, float v, int pair)
{
    int lo_off;
    uint16_t *p = pf_act_ptr(base, blk_bytes, b, m, k, pair, lo_off);
    v = rounded(v);
    const uint16_t hi = f2bf(v);
    p[0] = hi;
    p[lo_off] = f2bf(v - bf2f(hi));
}

// Column of the q, k, v row that packed row n of the projection gives (e.k_pairs is a power of two; the second third holds the keys)
__device__ __forceinline__ int plain_column(const Epi &e, int n)
{
    if (e.k_pairs) {
        const int d = e.N / 3, w = (n - d) & (e.k_pairs - 1);
        if (n >= d && n < 2 * d) n += (w >> 1) + (w & 1) * (e.k_pairs >> 1) - w;
    }
    return n;
}

// (EPI_FEATURE only where the kernel is compiled for it: in the one-projection kernel of every launch its arguments, loaded ahead of the
// weights, cost 0.4 % of a decode forward.)
// PAIRS: the rows may be those of a q, k, v projection with key rows in pairs (not in the stand-alone product).
template <bool BF, bool FEATURE = !BF, bool PAIRS = BF>
__device__ __forceinline__ void epilogue(const Epi &e, int rt, float (*yt)[KG_ROWS], const float *sc,
                                         float (*sq)[KG_ROWS], float resv = 0.f, float gainv = 1.f,
                                         bool prefetched = false, int t = threadIdx.x, const Feature *ft = nullptr)
{
    if (e.kind == EPI_PLAIN || e.kind == EPI_HEAD) {
        if (t < 128) {
            int row = t >> 3, m = t & 7;
            int mo = m + e.row_shift;
            float z = yt[row][m] * sc[m];
            if (m < e.M && mo >= 0) e.out[(size_t)mo * e.N + (PAIRS ? plain_column(e, rt * 16 + row) : rt * 16 + row)] = z;
            sq[row][m] = z * e.inv_temp;
        }
        if (e.kind == EPI_HEAD) {
            __syncthreads();
            int mo = t + e.row_shift;
            if (t < e.M && mo >= 0) {
                float best = sq[0][t];
                int bi = 0;
                for (int r = 1; r < 16; r++)
                    if (sq[r][t] > best) { best = sq[r][t]; bi = r; }
                float sum = 0.f;
                for (int r = 0; r < 16; r++) sum += __expf(sq[r][t] - best);
                float *hs = e.hstat + ((size_t)mo * (e.N >> 4) + rt) * 4;
                hs[0] = best;
                hs[1] = sum;
                hs[2] = __int_as_float(rt * 16 + bi);
            }
        }
    } else if (e.kind == EPI_RESID) {
        if (t < 128) {
            int row = t >> 3, m = t & 7;
            float v = 0.f;
            if (m < e.M) {
                int n = rt * 16 + row;
                if (!prefetched) {
                    resv = e.res[(size_t)m * e.N + n];
                    gainv = e.gain ? e.gain[n] : 1.f;
                }
                v = resv + yt[row][m];
                e.xout[(size_t)m * e.N + n] = v;
                if (e.act_out) store_act<BF>(e.act_out, e.act_K, m, n, e.gain ? v * gainv : v);
            }
            sq[row][m] = v * v;
        }
        if (e.ssq_out) {
            __syncthreads();
            if (t < KG_ROWS) {
                float s = 0.f;
                for (int r = 0; r < 16; r++) s += sq[r][t];
                e.ssq_out[(size_t)rt * KG_ROWS + t] = s;
            }
        }
    } else if (FEATURE && e.kind == EPI_FEATURE) {
        if (t < 128) {
            int row = t >> 3, m = t & 7;
            float v = 0.f;
            if (m < e.M) {
                const int n = rt * 16 + row;
                const size_t at = (size_t)m * e.N + n;
                v = resv + yt[row][m];          // (operands fetched ahead by all kernels that have this epilogue)
                e.xout[at] = v;
                if (ft->xout2) ft->xout2[at] = v;
                store_act<BF>(e.act_out, e.act_K, m + ft->act_row, n, v * gainv);
                store_act<BF>(ft->act2, e.act_K, m + ft->row2, n, v * ft->gain2[n]);
            }
            sq[row][m] = v * v;
        }
        __syncthreads();
        if (t < e.M) {
            float s = 0.f;
            for (int r = 0; r < 16; r++) s += sq[r][t];
            e.ssq_out[(size_t)rt * KG_ROWS + t + ft->act_row] = s;
            ft->ssq2[(size_t)rt * KG_ROWS + t + ft->row2] = s;
        }
    } else if (e.kind == EPI_SILU) {
        if (t < 128) {
            int row = t >> 3, m = t & 7;
            if (m < e.M) {
                float g = yt[row][m] * sc[m];
                store_act<BF>(e.act_out, e.act_K, m, rt * 16 + row, g / (1.f + __expf(-g)));
            }
        }
    } else { // EPI_SWIGLU: tile rows (2i, 2i+1) = (gate, up) of feed-forward feature rt*8 + i
        if (t < 64) {
            int i = t >> 3, m = t & 7;
            if (m < e.M) {
                float g = yt[2 * i][m] * sc[m], u = yt[2 * i + 1][m] * sc[m];
                float a = g / (1.f + __expf(-g)) * u;
                store_act<BF>(e.act_out, e.act_K, m, rt * 8 + i, a);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Order of a row tile's KS weight tiles in memory.  The eight waves of a projection block split
// the k-steps into contiguous ranges (wave w starts at ks0(w) = w KS / 8, rounded down) and walk
// them in step; the tiles are stored in the order the block asks for them, the i-th tile of every
// wave next to each other, so that at any moment the block reads one contiguous stretch of memory
// instead of eight stretches KS / 8 KB apart (measured: 18.5 against 19.1 us per projection launch
// at the 7B shape).  Ranges are q = KS / 8 or q + 1 tiles long; the first tile of each of the
// E = KS - 8 q long ranges comes first (in wave order), then the other tiles at E + 8 j + w.
// Which k-steps a wave sums, and in which order, does not depend on where the tiles are stored.
__host__ __device__ __forceinline__ int tile_pos_in_range(int w, int ks, int KS)
{
    const int q = KS >> 3, E = KS - 8 * q;
    const int ks0 = (w * KS) >> 3, len = (((w + 1) * KS) >> 3) - ks0, i = ks - ks0;
    if (len > q) return i == 0 ? ks0 - w * q : E + (i - 1) * 8 + w;
    return E + i * 8 + w;
}
__host__ __device__ __forceinline__ int tile_pos(int ks, int KS) { return tile_pos_in_range((8 * ks + 7) / KS, ks, KS); }

// k-step held by the tile stored at position p of a row tile: the inverse of tile_pos
__host__ __device__ __forceinline__ int kstep_at_pos(int p, int KS)
{
    const int q = KS >> 3, E = KS - 8 * q;
    if (p < E) return ((8 * (p + 1) + E - 1) / E - 1) * q + p;      // first tile of the (p + 1)-th long range
    const int w = (p - E) & 7, j = (p - E) >> 3;
    return w * q + (((w + 1) * E) >> 3) + j;                        // a long range's first tile lies in front: skipped here
}

// ---------------------------------------------------------------------------------------------
// Projection, bf16 weights: one block (8 waves) per 16-row tile; the waves split K; each wave
// streams its 1 KB weight tiles with 16-byte non-temporal loads and issues one MFMA per tile.
// W: tiles [rt][tile_pos(ks)][64 lanes][8 bf16]; act: B-operand tiles [ks][64 lanes][8 bf16].

// B operand of one k-step as a lane loads it, and the 16 bytes the multiplication takes.
// FROM_ACT: activation tiles written by the producer (hi / lo parts, see store_act).
// FROM_ROWS, FROM_ROWS_UNALIGNED: plain fp32 rows x[M][K] (the stand-alone product), split by the lanes
// themselves into the very parts store_act would have stored.  Of the 8 consecutive k of a row that lanes j (hi
// part) and j + 8 (lo part) share, each lane reads four, splits them, keeps the part it stands for and passes
// the other one on: as many bytes through the L1 as the activation tiles take, and 20 vector operations a tile
// (4096 x 4096, one row: 11.1 us a call with two launches that clear and fill activation tiles, 8.0 without; 32000 x
// 4096: 42.8 -> 39.1; with every lane reading and splitting all 8 k, 13840 x 5136 with 7 rows took 35.9 us against
// 34.1 with the two launches).
enum { FROM_ACT = 0, FROM_ROWS = 1, FROM_ROWS_UNALIGNED = 2 };
template <int SRC> struct BRaw { float v[4]; };
template <> struct BRaw<FROM_ACT> { u32x4_t v; };

template <int SRC> struct BSource {
    buffer_t buf;
    uint32_t off;               // this lane's 16 bytes of k-step 0 (its slot, or its row at its four k); BUFFER_NONE: the column stands for no row
    const float *row;           // FROM_ROWS_UNALIGNED: the same as an address
    int k, K;                   // first of the pair's 8 k, features
    bool on, lo;                // the lane's column stands for a live row; for the lo part of it
    __device__ __forceinline__ BSource(const void *act, int M, int lane, int K_)
    {
        on = (lane & 7) < M;
        lo = (lane & 8) != 0;
        k = (lane >> 4) * 8;
        K = K_;
        buf = buffer_of(act, 0x7FFFFFFFu);
        const uint32_t at = (uint32_t)(lane & 7) * K_ + k + (lo ? 4 : 0);
        off = !on ? BUFFER_NONE : SRC == FROM_ACT ? 16 * b_slot(lane) : 4 * at;
        row = (const float *)act + (size_t)(lane & 7) * K_ + k + (lo ? 4 : 0);
    }
    __device__ __forceinline__ BRaw<SRC> load(int ks) const
    {
        BRaw<SRC> r;
        if constexpr (SRC == FROM_ACT) {
            r.v = __builtin_amdgcn_raw_buffer_load_b128(buf, off, ks * 1024, 0);
        } else if constexpr (SRC == FROM_ROWS) {
            // (K is a multiple of 16: the last k-step may be half empty)
            const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(buf, k + 32 * ks + 8 <= K ? off : BUFFER_NONE, ks * 128, 0);
#pragma unroll
            for (int i = 0; i < 4; i++) r.v[i] = __uint_as_float(v[i]);
        } else {
            const float *p = row + 32 * ks;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            if (on && k + 32 * ks + 8 <= K) a = make_float4(p[0], p[1], p[2], p[3]);
            r.v[0] = a.x; r.v[1] = a.y; r.v[2] = a.z; r.v[3] = a.w;
        }
        return r;
    }
    // all 64 lanes call it
    __device__ __forceinline__ bf16x8_t operand(const BRaw<SRC> &r) const
    {
        if constexpr (SRC == FROM_ACT) {
            return __builtin_bit_cast(bf16x8_t, r.v);
        } else {
            typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
            uint32_t h[2], l[2], o[2];
#pragma unroll
            for (int i = 0; i < 2; i++) {                           // nearest even, as f2bf
                bf16x2_t hi, lw;
                hi[0] = (__bf16)r.v[2 * i]; hi[1] = (__bf16)r.v[2 * i + 1];
                lw[0] = (__bf16)(r.v[2 * i] - (float)hi[0]); lw[1] = (__bf16)(r.v[2 * i + 1] - (float)hi[1]);
                h[i] = __builtin_bit_cast(uint32_t, hi);
                l[i] = __builtin_bit_cast(uint32_t, lw);
                o[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(lo ? h[i] : l[i]), 0x128, 0xF, 0xF, false);    // lane ^ 8 (row_ror:8)
            }
            u32x4_t v;
            v[0] = lo ? o[0] : h[0]; v[1] = lo ? o[1] : h[1];
            v[2] = lo ? l[0] : o[0]; v[3] = lo ? l[1] : o[1];
            return __builtin_bit_cast(bf16x8_t, v);
        }
    }
};

#define GEMV_WAVES 8

// ONE: one chunk of weights in flight per wave, not two (gemv_one_chunk)
template <int SRC, bool FEATURE = false, bool ONE = false>
__device__ __forceinline__ void gemv_bf16_body(const u32x4_t *__restrict__ W, int KS, int M, const void *__restrict__ act,
                                               const float *ssq_in, int nt_in, int N, const float *res, const float *gain,
                                               int K, const Epi &e, const Feature *ft = nullptr)
{
    __shared__ float part[GEMV_WAVES][16][KG_ROWS];
    __shared__ float yt[16][KG_ROWS];
    __shared__ float sq[16][KG_ROWS];
    __shared__ float sc[KG_ROWS];
    const int rt = blockIdx.x;
    // The wave index as a scalar, so that everything derived from it (the k range, whether it is a
    // long one) is tested with scalar branches.  This is needed for correctness, not only speed: an
    // MFMA ignores the EXEC mask, and the compiler drops the skip branch around a short
    // exec-masked region, so an `if` on a per-lane copy of a uniform condition that holds nothing
    // but an MFMA executes it also in the waves where the condition is false, on registers those
    // waves never loaded.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ks0 = (wave * KS) / GEMV_WAVES, ks1 = ((wave + 1) * KS) / GEMV_WAVES;
    // the wave's tiles sit 8 tiles apart (see tile_pos); a long range has one more tile up front
    const int q = KS >> 3, n_long = KS - 8 * q;
    const bool long_range = ks1 - ks0 > q;
    const u32x4_t *wbase = W + (size_t)rt * KS * 64 + lane;
    const u32x4_t *wp = wbase + (size_t)(n_long + wave) * 64;
    const BSource<SRC> bsrc(act, M, lane, K);
    int ks = ks0 + (long_range ? 1 : 0);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    ScaleRegs sr;
    scale_fetch(ssq_in, M, nt_in, sr);
    float resv = 0.f, gainv = 1.f;       // epilogue operands of thread (row, m), fetched early
    if (res && threadIdx.x < 128 && (threadIdx.x & 7) < M) {
        int nn = rt * 16 + (threadIdx.x >> 3);
        resv = res[(size_t)(threadIdx.x & 7) * N + nn];
        if (gain) gainv = gain[nn];
    }
    auto mma = [&](const u32x4_t &w, const BRaw<SRC> &b) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), bsrc.operand(b), acc, 0, 0, 0);
    };
    // chunks of U tiles: all loads of a chunk are issued before its multiplications
    auto load = [&](auto &A, auto &Bv, int U) {
#pragma unroll
        for (int u = 0; u < U; u++) A[u] = __builtin_nontemporal_load(wp + u * 512);
#pragma unroll
        for (int u = 0; u < U; u++) Bv[u] = bsrc.load(ks + u);
        wp += U * 512;
        ks += U;
    };
    auto mul = [&](const auto &A, const auto &Bv, int U) {
#pragma unroll
        for (int u = 0; u < U; u++) mma(A[u], Bv[u]);
    };
    // chunks of 4 tiles, double-buffered: the loads of chunk i+1 are in flight while chunk i is
    // multiplied, so a wave never drains its memory pipe between chunks.  LONG: some waves have a long range (KS is no multiple of 8),
    // with its own load in front; a copy of its own, for with that condition the compiler waits for all loads in every turn of the loop.
#define GEMV_FENCE __builtin_amdgcn_sched_barrier(0)        // (nor is a load moved below a multiplication)
    auto stream = [&](auto has_long) {
        constexpr bool LONG = decltype(has_long)::value;
        u32x4_t a0[4], a1[4];
        BRaw<SRC> b0[4], b1[4];
        int n = q & 3, rem = q >> 2;
        if constexpr (LONG) {
            u32x4_t ax = {0u, 0u, 0u, 0u};                 // first tile of a long range (k-step ks0)
            BRaw<SRC> bx;
            if (long_range) {
                ax = __builtin_nontemporal_load(wbase + (size_t)(ks0 - wave * q) * 64);
                bx = bsrc.load(ks0);
            }
            if (rem) load(a0, b0, 4);
            if (long_range) mma(ax, bx);
        } else if (rem) {
            load(a0, b0, 4);
        }
        if constexpr (ONE)
            for (; rem > 2; rem--) {
                mul(a0, b0, 4);
                GEMV_FENCE;
                load(a0, b0, 4);
                GEMV_FENCE;
            }
        for (; rem > 2; rem -= 2) {
            load(a1, b1, 4);
            GEMV_FENCE;
            mul(a0, b0, 4);
            GEMV_FENCE;
            load(a0, b0, 4);
            GEMV_FENCE;
            mul(a1, b1, 4);
            GEMV_FENCE;
        }
        if (rem == 2) {
            load(a1, b1, 4);
            GEMV_FENCE;
            mul(a0, b0, 4);
            mul(a1, b1, 4);
        } else if (rem == 1) {
            mul(a0, b0, 4);
        }
        if (n >= 2) { load(a0, b0, 2); mul(a0, b0, 2); n -= 2; }
        if (n >= 1) { load(a0, b0, 1); mul(a0, b0, 1); }
    };
#undef GEMV_FENCE
    if (n_long) stream(std::true_type{});
    else stream(std::false_type{});
    scale_finish(e, sr, sc);
    // D layout: lane holds column (lane & 15) and tile rows 4*(lane >> 4) + r.  Columns m and m+8
    // are the hi and lo parts of batch row m: fold them.
#pragma unroll
    for (int r = 0; r < 4; r++) {
        float v = acc[r] + __shfl_xor(acc[r], 8);
        if ((lane & 15) < 8) part[wave][4 * (lane >> 4) + r][lane & 7] = v;
    }
    __syncthreads();
    if (threadIdx.x < 128) {
        int row = threadIdx.x >> 3, m = threadIdx.x & 7;
        float v = part[0][row][m];
#pragma unroll
        for (int w = 1; w < GEMV_WAVES; w++) v += part[w][row][m];
        yt[row][m] = v;
    }
    __syncthreads();
    epilogue<true, FEATURE, SRC == FROM_ACT>(e, rt, yt, sc, sq, resv, gainv, true, threadIdx.x, ft);
}

// Everything a wave needs before its first weight load is a leading scalar argument (a copy of the
// fields of e named alike): those arrive preloaded in SGPRs, a field of the by-value struct costs a
// scalar load from the argument block at the start of every launch.
// 14 dwords fit: W, KS, M, act, ssq_in, nt_in, N, res (null unless the epilogue adds a residual), gain.
__global__ __launch_bounds__(64 * GEMV_WAVES, 2) void gemv_bf16_kernel(const u32x4_t *__restrict__ W, int KS, int M,
                                                                   const u32x4_t *__restrict__ act,
                                                                   const float *ssq_in, int nt_in, int N,
                                                                   const float *res, const float *gain, Epi e)
{
    gemv_bf16_body<FROM_ACT>(W, KS, M, act, ssq_in, nt_in, N, res, gain, 0, e);
}

// the same with one chunk of weights in flight (gemv_one_chunk)
__global__ __launch_bounds__(64 * GEMV_WAVES, 2) void gemv_bf16_one_kernel(const u32x4_t *__restrict__ W, int KS, int M,
                                                                       const u32x4_t *__restrict__ act,
                                                                       const float *ssq_in, int nt_in, int N,
                                                                       const float *res, const float *gain, Epi e)
{
    gemv_bf16_body<FROM_ACT, false, true>(W, KS, M, act, ssq_in, nt_in, N, res, gain, 0, e);
}

// the same for the projection that gives the early features (EPI_FEATURE)
__global__ __launch_bounds__(64 * GEMV_WAVES, 2) void gemv_bf16_feature_kernel(const u32x4_t *__restrict__ W, int KS, int M,
                                                                           const u32x4_t *__restrict__ act, int N, Epi e, Feature ft)
{
    gemv_bf16_body<FROM_ACT, true>(W, KS, M, act, nullptr, 0, N, e.res, e.gain, 0, e, &ft);
}

// the same product from plain rows x[M][K] (stand-alone product: no scale, no residual); y[m][n] fp32
template <int SRC>
__global__ __launch_bounds__(64 * GEMV_WAVES, 4) void gemv_bf16_rows_kernel(const u32x4_t *__restrict__ W, int KS, int M,
                                                                        const float *__restrict__ x, int K, int N, float *y)
{
    Epi e = {};
    e.kind = EPI_PLAIN; e.M = M; e.N = N; e.out = y;
    gemv_bf16_body<SRC>(W, KS, M, x, nullptr, 0, N, nullptr, nullptr, K, e);
}

// Projections of several rows with more weight tiles than compute units: one workgroup per compute unit and NTW tiles per
// workgroup.  gemv_bf16_kernel fetches the activations of a k-step through the L1 once per weight tile (M / 8 of the
// weights' bytes, and they come after them: gate+up of the 7B shape takes 28 us with one row and 36 us with eight);
// here they serve NTW tiles.  Every tile's sums run over the same k in the same order as there: the results are
// the same bits for any number of rows.  The tiles are shared out evenly (no group has more than NTW).
// D k-steps of loads are in flight per wave.  (Two tiles per workgroup in gemv_bf16_body instead, 16 waves a compute
// unit: slower at every row count, 33 .. 36 us for gate+up.)
template <int NTW> __host__ __device__ constexpr int gemv_multi_depth() { return (204 - 4 * NTW) / (4 * (NTW + 1)) > 8 ? 8 : (204 - 4 * NTW) / (4 * (NTW + 1)); }

template <int SRC, int NTW>
__global__ __launch_bounds__(64 * GEMV_WAVES, 2) void gemv_multi_kernel(const u32x4_t *__restrict__ W, int KS, int M,
                                                                    const void *__restrict__ act, const float *ssq_in, int nt_in, int N,
                                                                    int K, Epi e)
{
    constexpr int D = gemv_multi_depth<NTW>(), NY = (NTW + 3) / 4 * 4;      // tiles in the epilogue: four at a time
    __shared__ float part[GEMV_WAVES][NTW][16][KG_ROWS];
    __shared__ float yt[NY][16][KG_ROWS];
    __shared__ float sq[NY][16][KG_ROWS];
    __shared__ float sc[KG_ROWS];
    const int NT = N >> 4, groups = gridDim.x;
    const int rt0 = (int)((long long)blockIdx.x * NT / groups), ntw = (int)((long long)(blockIdx.x + 1) * NT / groups) - rt0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ks0 = (wave * KS) / GEMV_WAVES, n = ((wave + 1) * KS) / GEMV_WAVES - ks0;     // the wave's k-steps
    const int q = KS >> 3, n_long = KS - 8 * q;
    // position of the wave's i-th k-step (see tile_pos): p_rest + 8 i, except the first of a long range
    const int p_first = n > q ? ks0 - wave * q : n_long + wave, p_rest = n > q ? n_long + wave - 8 : n_long + wave;
    const u32x4_t *wsrc[NTW];
#pragma unroll
    for (int t = 0; t < NTW; t++) wsrc[t] = W + (size_t)(rt0 + min(t, ntw - 1)) * KS * 64 + lane;
    const BSource<SRC> bsrc(act, M, lane, K);
    ScaleRegs sr;
    scale_fetch(ssq_in, M, nt_in, sr);
    f32x4_t acc[NTW];
#pragma unroll
    for (int t = 0; t < NTW; t++) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t av[D][NTW];
    BRaw<SRC> bv[D];
    auto load = [&](int s, int i) {
        const int p = i ? p_rest + 8 * i : p_first;
#pragma unroll
        for (int t = 0; t < NTW; t++) av[s][t] = __builtin_nontemporal_load(wsrc[t] + p * 64);
        bv[s] = bsrc.load(ks0 + i);
    };
    auto mul = [&](int s) {
        const bf16x8_t b = bsrc.operand(bv[s]);
#pragma unroll
        for (int t = 0; t < NTW; t++) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av[s][t]), b, acc[t], 0, 0, 0);
    };
    // fewer than 2 D steps are left, the first D of them loaded or on their way
    auto finish = [&](int i) {
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + s < n) {
                mul(s);
                if (i + s + D < n) load(s, i + s + D);
            }
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + D + s < n) mul(s);
    };
    // (two ways apart from the start: after loads that may not have been issued the compiler waits for all of them in every turn.  us with
    // 7 rows, 2048 and 2560 features, that way from 2 D steps on / here: 3 tiles 11.2 and 13.9 / 10.6 and 12.7, 5 tiles 16.8 and 20.1 / 16.2 and 19.1)
    if (n >= D) {
#pragma unroll
        for (int s = 0; s < D; s++) {
            load(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
#pragma unroll
            for (int s = 0; s < D; s++) {
                __builtin_amdgcn_sched_barrier(0);
                mul(s);
                load(s, i + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        finish(i);
    } else {
#pragma unroll
        for (int s = 0; s < D; s++)
            if (s < n) load(s, s);
        finish(0);
    }
    scale_finish(e, sr, sc);
    // fold the hi and lo columns, add the waves' sums in wave order (as gemv_bf16_body)
#pragma unroll
    for (int t = 0; t < NTW; t++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float v = acc[t][r] + __shfl_xor(acc[t][r], 8);
            if ((lane & 15) < 8) part[wave][t][4 * (lane >> 4) + r][lane & 7] = v;
        }
    __syncthreads();
    for (int j = threadIdx.x; j < NTW * 128; j += 64 * GEMV_WAVES) {
        const int t = j >> 7, row = (j >> 3) & 15, m = j & 7;
        float v = part[0][t][row][m];
#pragma unroll
        for (int w = 1; w < GEMV_WAVES; w++) v += part[w][t][row][m];
        yt[t][row][m] = v;
    }
    __syncthreads();
#pragma unroll
    for (int t0 = 0; t0 < NTW; t0 += 4) {
        const int t = t0 + (threadIdx.x >> 7);                              // 128 threads per tile (none where there is no tile)
        epilogue<true, false, SRC == FROM_ACT>(e, rt0 + t, yt[t], sc, sq[t], 0.f, 1.f, false, t < ntw ? (int)(threadIdx.x & 127) : 1 << 20);
    }
}

// The one-row projection on the vector ALUs instead of the matrix units, over the same weight tiles,
// launch shape, k ranges and chunked, double-buffered loads as gemv_bf16_kernel: the comparison that
// backs the choice of an MFMA per tile also at one row (where 7 of its 8 row columns are idle).  A
// lane holds 8 consecutive k of one weight row: it widens them and multiplies by the row's fp32
// activations, the four lanes of a row are added at the end of the wave's range, the waves through LDS.
// y[n] = sum_k W[n][k] x[k], plain fp32 output; used by kg_op_linear_valu only.
__global__ __launch_bounds__(64 * GEMV_WAVES, 2) void gemv_bf16_valu_kernel(const u32x4_t *__restrict__ W, int KS,
                                                                        const float *__restrict__ x, int K, float *y)
{
    __shared__ float part[GEMV_WAVES][16];
    const int rt = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ks0 = (wave * KS) / GEMV_WAVES, ks1 = ((wave + 1) * KS) / GEMV_WAVES;
    const int q = KS >> 3, n_long = KS - 8 * q;
    const bool long_range = ks1 - ks0 > q;
    const u32x4_t *wbase = W + (size_t)rt * KS * 64 + lane;
    const u32x4_t *wp = wbase + (size_t)(n_long + wave) * 64;
    const int g8 = (lane >> 4) * 8;
    int ks = ks0 + (long_range ? 1 : 0);
    float acc = 0.f;
    auto mac = [&](const u32x4_t &a, int kstep) {
        const int k0 = kstep * 32 + g8;
        float4 x0 = make_float4(0.f, 0.f, 0.f, 0.f), x1 = x0;
        if (k0 + 8 <= K) { x0 = *(const float4 *)(x + k0); x1 = *(const float4 *)(x + k0 + 4); }
        acc = fmaf(__uint_as_float(a[0] << 16), x0.x, acc); acc = fmaf(__uint_as_float(a[0] & 0xFFFF0000u), x0.y, acc);
        acc = fmaf(__uint_as_float(a[1] << 16), x0.z, acc); acc = fmaf(__uint_as_float(a[1] & 0xFFFF0000u), x0.w, acc);
        acc = fmaf(__uint_as_float(a[2] << 16), x1.x, acc); acc = fmaf(__uint_as_float(a[2] & 0xFFFF0000u), x1.y, acc);
        acc = fmaf(__uint_as_float(a[3] << 16), x1.z, acc); acc = fmaf(__uint_as_float(a[3] & 0xFFFF0000u), x1.w, acc);
    };
    if (long_range) {
        const u32x4_t ax = __builtin_nontemporal_load(wbase + (size_t)(ks0 - wave * q) * 64);
        mac(ax, ks0);
    }
    int n = q;
    u32x4_t a0[4], a1[4];
    int rem = n >> 2;
    n &= 3;
#define LDV(A) { _Pragma("unroll") for (int u = 0; u < 4; u++) A[u] = __builtin_nontemporal_load(wp + u * 512); wp += 2048; }
#define MACV(A) { _Pragma("unroll") for (int u = 0; u < 4; u++) mac(A[u], ks + u); ks += 4; }
    if (rem) LDV(a0)
    while (rem >= 2) {
        LDV(a1)
        MACV(a0)
        if (rem > 2) LDV(a0)
        MACV(a1)
        rem -= 2;
    }
    if (rem == 1) MACV(a0)
#undef LDV
#undef MACV
    for (; n > 0; n--) {
        const u32x4_t a = __builtin_nontemporal_load(wp);
        wp += 512;
        mac(a, ks++);
    }
    acc += __shfl_xor(acc, 16);
    acc += __shfl_xor(acc, 32);
    if (lane < 16) part[wave][lane] = acc;
    __syncthreads();
    if (threadIdx.x < 16) {
        float v = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < GEMV_WAVES; w++) v += part[w][threadIdx.x];
        y[rt * 16 + threadIdx.x] = v;
    }
}

// Lane exchanges of reductions as data-parallel-primitive moves (no trip through the
// LDS crossbar as __shfl_xor takes).  All 64 lanes must be active.  quad_x1 / quad_x2: the value of
// lane ^ 1 / lane ^ 2.  half_mirror / row_mirror: the value of the mirrored lane inside a group of
// 8 / 16 lanes; where the value is already uniform over groups of 4 / 8 lanes that is the value
// lane ^ 4 / lane ^ 8 holds, so a butterfly built from them gives every lane the bits the xor
// butterfly gives.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float quad_x1(float v) { return dpp_move<0xB1>(v); }       // quad_perm [1,0,3,2]
__device__ __forceinline__ float quad_x2(float v) { return dpp_move<0x4E>(v); }       // quad_perm [2,3,0,1]
__device__ __forceinline__ float half_mirror(float v) { return dpp_move<0x141>(v); }
__device__ __forceinline__ float row_mirror(float v) { return dpp_move<0x140>(v); }
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
// v of the lanes with bit 32 (16, 8, 4) of their number clear and w of the others, each added to that of the lane that far away
__device__ __forceinline__ float fold32(float v, float w)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(w), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float v, float w)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(w), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold8(float v, float w, int lane)
{
    const bool hi = lane & 8;
    const float keep = hi ? w : v, give = hi ? v : w;
    return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xF, 0xF, false));      // row_ror:8
}
__device__ __forceinline__ float fold4(float v, float w, int lane)
{
    const bool hi = lane & 4;
    const float keep = hi ? w : v;
    const int give = __float_as_int(hi ? v : w);
    int other = __builtin_amdgcn_update_dpp(0, give, 0x104, 0xF, 0x5, false);           // row_shl:4 into lanes with bit 4 clear
    other = __builtin_amdgcn_update_dpp(other, give, 0x114, 0xF, 0xA, false);           // row_shr:4 into the others
    return keep + __int_as_float(other);
}

// Projection, fp32 weights (row-major [N][K]) and fp32 activations [8][K], K a multiple of 4: one workgroup (8 waves) per 16 weight
// rows, wave (rh, kp) takes rows 8 rh .. 8 rh + 7 and every fourth step of 64 k.  Lane (b, i) = (lane / 4, lane % 4) loads 4 consecutive k
// from 4 b on of weight rows i and 4 + i and of activation rows i (and 4 + i, MC = 2), for v_mfma_f32_4x4x1_16b_f32: one fused
// multiply-add per k slot b, weight row and activation row; the slots are added by lane exchanges at the end, each leaving half the
// sums in a lane.  (Of the fp32 matrix instructions the one that wastes least on few rows: v_mfma_f32_16x16x4_f32 does 16 columns, and one
// row of 512 x 8192 took 20.9 us with it.)
// The models this serves are small (the float32 configuration: K of 256 and 688, 16 .. 86 workgroups), so a launch is a chain of latencies:
// the row sums of the scale, the operands of the first D steps and those of the epilogue are requested together before any is used, and
// the scale is reduced while the others are on their way.  us per launch in a request of that configuration, one, two and eight rows: 4.4, 4.8
// and 8.1 with 16 threads to a weight row on the vector units and all loads masked; 3.4 (the kernel below), 3.6 and 4.3 here.
// A row's arithmetic does not depend on the others or on their number.  Rows of weights and activations need not be 16-byte aligned.
template <int MC>
__global__ __launch_bounds__(512) void gemv_f32_kernel(const float *__restrict__ W, int K, const float *__restrict__ act, Epi e, Feature ft)
{
    constexpr int D = 4;                    // steps in flight
    typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float red[4][16][KG_ROWS];
    __shared__ float sq[16][KG_ROWS];
    __shared__ float sc[KG_ROWS];
    const int rt = blockIdx.x, t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, i4 = lane & 3, slot = lane >> 2;
    const int rh = wave & 1, kp = wave >> 1;
    const int S = (K + 63) >> 6, n = kp < S ? (S - kp + 3) >> 2 : 0;       // steps, the last one perhaps short; this wave's
    ScaleRegs sr;
    scale_fetch(e.ssq_in, e.M, e.nt_in, sr);
    const float *wr = W + (size_t)(rt * 16 + rh * 8 + i4) * K;
    const buffer_t xb = buffer_of(act, 0x7FFFFFFFu);
    f32x4_t w[D][2];
    u32x4_t x[D][MC];
    auto load = [&](int s, int i) {         // (no lane is masked, see buffer_of; k beyond the last repeats it in the weights, and is 0 in the rows)
        const int k = 64 * (kp + 4 * i) + 4 * slot, kw = min(k, K - 4);
#pragma unroll
        for (int r = 0; r < 2; r++) w[s][r] = *(const f32x4u_t *)(wr + (size_t)4 * r * K + kw);
#pragma unroll
        for (int c = 0; c < MC; c++)
            x[s][c] = __builtin_amdgcn_raw_buffer_load_b128(xb, k < K && 4 * c + i4 < e.M ? 4u * ((4 * c + i4) * K + k) : BUFFER_NONE, 0, 0);
    };
    f32x4_t acc[2][MC];                     // [rows 4 r ..][activation rows 4 c ..][row]
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int c = 0; c < MC; c++) acc[r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](int s, int i) {
        const int k = 64 * (kp + 4 * i);
        if (k + 64 > K && k + 4 * slot >= K) w[s][0] = w[s][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};      // (0 x infinity)
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int r = 0; r < 2; r++)
#pragma unroll
                for (int c = 0; c < MC; c++)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[s][r][j], __uint_as_float(x[s][c][j]), acc[r][c], 0, 0, 0);
    };
    float resv = 0.f, gainv = 1.f;          // epilogue operands of thread (row, m)
    auto operands = [&]() {
        if ((e.kind == EPI_RESID || e.kind == EPI_FEATURE) && t < 128 && (t & 7) < e.M) {
            const int nn = rt * 16 + (t >> 3);
            resv = e.res[(size_t)(t & 7) * e.N + nn];
            if (e.gain) gainv = e.gain[nn];
        }
        scale_finish(e, sr, sc);
    };
    if (n >= D) {
#pragma unroll
        for (int s = 0; s < D; s++) {
            load(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        operands();
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
#pragma unroll
            for (int s = 0; s < D; s++) {
                mul(s, i + s);
                load(s, i + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D; s++) {
            mul(s, i + s);
            if (i + s + D < n) load(s, i + s + D);
        }
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + s + D < n) mul(s, i + s + D);
    } else {
#pragma unroll
        for (int s = 0; s < D - 1; s++)
            if (s < n) load(s, s);
        operands();
#pragma unroll
        for (int s = 0; s < D - 1; s++)
            if (s < n) mul(s, s);
    }
    // lane (b, i): 4 weight rows (registers) x activation row i of k slot b.  After the folds lane bits 32, 16, 8 say which of the 8
    // weight rows it holds the sum of and bit 4 (MC = 2) which four activation rows.
    float v[MC];
#pragma unroll
    for (int c = 0; c < MC; c++) {
        float y[4];
#pragma unroll
        for (int q = 0; q < 4; q++) y[q] = fold32(acc[0][c][q], acc[1][c][q]);
        v[c] = fold8(fold16(y[0], y[2]), fold16(y[1], y[3]), lane);
    }
    const float sum = fold4(v[0], v[MC - 1], lane);
    const int row = 8 * rh + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1), m = i4 + (lane & 4);
    red[kp][row][m] = sum;                  // (MC = 1: the same number twice, the second of no use)
    __syncthreads();
    if (t < 128) red[0][t >> 3][t & 7] = (red[0][t >> 3][t & 7] + red[1][t >> 3][t & 7]) + (red[2][t >> 3][t & 7] + red[3][t >> 3][t & 7]);
    __syncthreads();
    epilogue<false>(e, rt, red[0], sc, sq, resv, gainv, true, t, &ft);
}

// The same sums of one row on the vector units (a k slot's products one after another, slots and quarters of the steps in the order
// above): 16 consecutive lanes read 256 bytes of a weight row, where the matrix instruction's operand has neighbouring lanes in four rows.
// us, one row, matrix / vector: 2048 x 1024 4.18 / 3.78, 512 x 8192 17.6 / 9.9, 256 x 688 3.37 / 3.37; from two rows on the matrix form is as
// fast or faster at the sizes of small models (2048 x 1024, two rows, 4.37 against 4.75 with two rows on the vector units).  Few rows of many
// features take it from two rows on too (512 x 8192, 2, 4 and 8 rows 19.9, 23.3 and 30.7 us; with 16 threads to a weight row 33, 46 and 83).
__global__ __launch_bounds__(256) void gemv_f32_row_kernel(const float *__restrict__ W, int K, const float *__restrict__ act, Epi e, Feature ft)
{
    constexpr int D = 8;                    // steps of 64 k in flight
    typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float yt[16][KG_ROWS];
    __shared__ float sq[16][KG_ROWS];
    __shared__ float sc[KG_ROWS];
    const int rt = blockIdx.x, t = threadIdx.x, row = t >> 4, slot = t & 15;
    const int S = (K + 63) >> 6;
    ScaleRegs sr;
    scale_fetch(e.ssq_in, 1, e.nt_in, sr);
    const float *wr = W + (size_t)(rt * 16 + row) * K;
    f32x4_t w[D], x[D];
    auto load = [&](int s, int i) {
        const int k = min(64 * i + 4 * slot, K - 4);
        w[s] = *(const f32x4u_t *)(wr + k);
        x[s] = *(const f32x4u_t *)(act + k);
    };
    float acc[4] = {0.f, 0.f, 0.f, 0.f};    // steps i % 4
    auto mul = [&](int s, int i) {
        if (64 * i + 64 > K && 64 * i + 4 * slot >= K) w[s] = x[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; j++) acc[s & 3] = fmaf(w[s][j], x[s][j], acc[s & 3]);
    };
    float resv = 0.f, gainv = 1.f;          // epilogue operands of thread (row, 0)
    auto operands = [&]() {
        if ((e.kind == EPI_RESID || e.kind == EPI_FEATURE) && t < 128 && (t & 7) == 0) {
            const int nn = rt * 16 + (t >> 3);
            resv = e.res[nn];
            if (e.gain) gainv = e.gain[nn];
        }
        scale_finish(e, sr, sc);
    };
    if (S >= D) {
#pragma unroll
        for (int s = 0; s < D; s++) {
            load(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        operands();
        int i = 0;
        for (; i + 2 * D <= S; i += D) {
#pragma unroll
            for (int s = 0; s < D; s++) {
                mul(s, i + s);
                load(s, i + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D; s++) {
            mul(s, i + s);
            if (i + s + D < S) load(s, i + s + D);
        }
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + s + D < S) mul(s, i + s + D);
    } else {
#pragma unroll
        for (int s = 0; s < D - 1; s++)
            if (s < S) load(s, s);
        operands();
#pragma unroll
        for (int s = 0; s < D - 1; s++)
            if (s < S) mul(s, s);
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        acc[j] += dpp_move<0x128>(acc[j]);                              // lane ^ 8 (row_ror:8)
        acc[j] = fold4(acc[j], acc[j], t);
        acc[j] += quad_x2(acc[j]);
        acc[j] += quad_x1(acc[j]);
    }
    if (slot == 0) yt[row][0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    epilogue<false>(e, rt, yt, sc, sq, resv, gainv, true, t, &ft);
}

// ---------------------------------------------------------------------------------------------
// Projection for the prompt (prefill): Y[T][N] = X[T][K] . W^T for T up to a few hundred rows, a
// dense contraction on the MFMA units.  Rows are handled in blocks of 8 (hi/lo columns of one
// MFMA, exactly as in decoding), so every output is computed by the same instruction sequence as
// in gemv_bf16_kernel: per output tile the k-steps are split into the same 8 ranges, each range is
// accumulated in order by MFMA, hi and lo are folded, and the 8 range sums are added in order.
// A cache prefilled by this kernel and the 8-row attention is therefore bit-identical to one written
// token by token (the bfloat16 / float32 cache options; with the half-precision cache long passes use
// gemm_prefill2_body and pf_attn_kernel below, which sum in another order).
//   A workgroup handles a group of CBW row blocks (CBW = 8: 64 rows) and a group of 8 * TW weight tiles.
//   It has 12 waves: waves 8..11 only move data, waves 0..7 only multiply.  The movers bring the
//   weight tiles and the activation tiles of a stage (PF_KC k-steps) straight from memory into LDS
//   (global_load_lds: no registers in between), two stages ahead of the multiplication, into a ring
//   of PF_NB stage buffers, and wait with explicit counts for the stage that is due; the
//   multipliers read operands from LDS only, so they never wait on memory.  Wave w of the
//   multipliers owns TW weight tiles and TW * CBW accumulators: every activation tile read from
//   LDS feeds TW MFMAs.  Activation tiles sit in LDS in MFMA lane order (lane l fetches the piece it
//   will use), so a read touches 64 consecutive 16-byte pieces, free of bank conflicts.  Rows
//   beyond the last one of a block are not masked: an MFMA column only depends on its own column of
//   B, and the results of those columns are never stored.
//   The workgroups that stream the same weight tiles for different row groups run next to each other on
//   one XCD and share its L2 (pf_work).
#define PF_KC 2
#define PF_CBW 8
#define PF_NB 3

// Where the keys and values of a prompt pass's q, k, v projection go (EPI_QKV, half-precision cache): the epilogue rotates the keys, which
// arrive in rotation pairs (map_row), and writes both to the rows' pages in the cache's own type; only the queries go to e.out.
// (A launch of its own that read them back cost 4.8 us a layer at 45 rows, 7 at 256, 55 at 4096; the projection takes 0.6 .. 1 us longer.  Whole
// prompts at the 7B shape: 45 tokens 4.13 -> 4.06 ms, 4096 tokens 95.2 -> 93.8; at 256 tokens, where the power limit takes back what the
// shorter pause gives, 8.10 -> 8.09.)
struct KvOut {
    uint16_t *kv;           // pool: [phys page][slot][head][K|V][P][hd], half bit patterns
    const int *page_table;
    const float2 *rope;     // [max_seq][hd/2]
    int slot, n_slots, H, log_hd, logP, pos0;
    int d, n0;              // width of the model; packed row of the stacked projection at which this launch's weights start
};
struct PfArgs {
    const u32x4_t *W;       // weight tiles [NT][tile_pos(ks)][64]
    int KS, NT;
    const u32x4_t *act;     // activation tiles, block b at act + b * act_blk
    size_t act_blk;         // 16-byte units per 8-row block
    int T;                  // rows in this pass
    int ssq_in_blk, ssq_out_blk;   // floats per 8-row block of the sum-of-squares arrays
    size_t act_out_blk;     // bytes per 8-row block of the output activation
    int gx, gy;             // row groups, tile groups (the grid holds 8 * ceil(gx * gy / 8) workgroups, see pf_work)
    float *part;            // gemm_prefill2_body: partial sums [slice = blockIdx.y][T][N] for pf_reduce_rows_kernel; null: the epilogue
    KvOut kv;               // EPI_QKV
};

__device__ __forceinline__ Epi pf_block_epi(const Epi &e, const PfArgs &a, int b)
{
    Epi eb = e;
    eb.M = min(KG_ROWS, a.T - 8 * b);
    if (eb.ssq_in) eb.ssq_in += (size_t)b * a.ssq_in_blk;
    if (eb.out) eb.out += (size_t)8 * b * e.N;
    if (eb.res) eb.res += (size_t)8 * b * e.N;
    if (eb.xout) eb.xout += (size_t)8 * b * e.N;
    if (eb.act_out) eb.act_out = (char *)eb.act_out + (size_t)b * a.act_out_blk;
    if (eb.ssq_out) eb.ssq_out += (size_t)b * a.ssq_out_blk;
    return eb;
}

__device__ __forceinline__ float half_bits_to_f32(uint32_t low16) { return (float)__builtin_bit_cast(_Float16, (uint16_t)low16); }
__device__ __forceinline__ uint16_t f32_to_half_bits(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }

// rotation of the pair (x0, x1) by the angle whose (cos, sin) is cs; written with explicit fused
// operations so that every instantiation rounds alike
__device__ __forceinline__ float rot_lo(float x0, float x1, float2 cs) { return fmaf(x0, cs.x, -__fmul_rn(x1, cs.y)); }
__device__ __forceinline__ float rot_hi(float x0, float x1, float2 cs) { return fmaf(x1, cs.x, __fmul_rn(x0, cs.y)); }

// position of row `row` of the pass inside its page's keys of head 0
__device__ __forceinline__ uint16_t *kv_out_row(const KvOut &k, int row)
{
    const int pos = k.pos0 + row, page = k.page_table[pos >> k.logP];
    return k.kv + (((size_t)page * k.n_slots + k.slot) * k.H << (k.logP + k.log_hd + 1)) + ((size_t)(pos & ((1 << k.logP) - 1)) << k.log_hd);
}
// four packed rows n .. n + 3 of the launch (n a multiple of 4), scaled, for one row of the pass
__device__ __forceinline__ void store_qkv(const KvOut &k, float *out, uint16_t *kv_row, int row, int n, float y0, float y1, float y2, float y3)
{
    n += k.n0;
    const int d = k.d, hd = 1 << k.log_hd;
    if (n < d) {
        *(float4 *)(out + (size_t)row * 3 * d + n) = make_float4(y0, y1, y2, y3);
        return;
    }
    const bool key = n < 2 * d;
    const int m = n - (key ? d : 2 * d), h = m >> k.log_hd, w = m & (hd - 1);
    uint16_t *p = kv_row + ((size_t)h << (k.logP + k.log_hd + 1));
    if (key) {
        const int j = w >> 1;
        const float4 cs = *(const float4 *)(k.rope + (size_t)(k.pos0 + row) * (hd >> 1) + j);      // (cos, sin) of pairs j, j + 1
        const float a0 = rounded(y0), b0 = rounded(y1), a1 = rounded(y2), b1 = rounded(y3);
        const float2 c0 = make_float2(cs.x, cs.y), c1 = make_float2(cs.z, cs.w);
        *(uint32_t *)(p + j) = f32_to_half_bits(rounded(rot_lo(a0, b0, c0))) | ((uint32_t)f32_to_half_bits(rounded(rot_lo(a1, b1, c1))) << 16);
        *(uint32_t *)(p + j + (hd >> 1)) = f32_to_half_bits(rounded(rot_hi(a0, b0, c0))) | ((uint32_t)f32_to_half_bits(rounded(rot_hi(a1, b1, c1))) << 16);
    } else {
        *(uint2 *)(p + ((size_t)1 << (k.logP + k.log_hd)) + w) =
            make_uint2(f32_to_half_bits(rounded(y0)) | ((uint32_t)f32_to_half_bits(rounded(y1)) << 16),
                       f32_to_half_bits(rounded(y2)) | ((uint32_t)f32_to_half_bits(rounded(y3)) << 16));
    }
}

// (row group, group of weight tiles) of this workgroup.  Workgroups go to the 8 XCDs in turn; XCD x takes the x-th
// eighth of the pairs in the order "all row groups of a tile group, then the next tile group".  (Whole tile
// groups dealt out to the XCDs leave some with twice the work of others where there are few: 10 groups of 32
// tiles, o_proj of the 13B shape at 3000 rows, took 488 us, two rounds on two XCDs.)
__device__ __forceinline__ bool pf_work(const PfArgs &a, int &row_group, int &tile_group)
{
    const int total = a.gx * a.gy, per = (total + 7) >> 3, j = blockIdx.x >> 3, i = (blockIdx.x & 7) * per + j;
    if (j >= per || i >= total) return false;
    row_group = __builtin_amdgcn_readfirstlane(i % a.gx);       // (scalars: they are needed again after the main loop)
    tile_group = __builtin_amdgcn_readfirstlane(i / a.gx);
    return true;
}

struct PfStage { int r, k, n; };   // k-range index (0..7, 8 = end), first k-step, k-steps in the stage

// the stage that starts at k-step k of range r (or the first stage of the next non-empty range)
__device__ __forceinline__ PfStage pf_stage_at(int r, int k, int KS)
{
    while (r < 8) {
        int k1 = ((r + 1) * KS) >> 3;
        if (k < k1) return PfStage{r, k, min(PF_KC, k1 - k)};
        r++;
        k = (r * KS) >> 3;
    }
    return PfStage{8, 0, 0};
}

template <int PF_TW, int CBW>
__device__ __forceinline__ void gemm_prefill_body(const PfArgs &a, const Epi &e)
{
    constexpr int NTW = 8 * PF_TW;                         // weight tiles of the workgroup
    __shared__ u32x4_t As[PF_NB][PF_KC][NTW][64];
    __shared__ u32x4_t Bs[PF_NB][PF_KC][CBW][64];
    __shared__ float scs[CBW][KG_ROWS];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const bool mover = wave >= 8;
    const int nb = (a.T + 7) >> 3;
    int rgi, gyi;
    if (!pf_work(a, rgi, gyi)) return;
    const int b0 = rgi * CBW;
    const int nbw = min(CBW, nb - b0);
    const int rt0 = (gyi * 8 + (wave & 7)) * PF_TW;
    const int KS = a.KS;

    // RMS scales of this block group's rows: wave w serves row block w; all partial sums of its 8
    // rows are fetched at once, then every row is reduced exactly as in decoding (lane sums in index
    // order, then the same butterfly)
    static_assert(CBW <= 8, "one wave per row block");
    if (wave < nbw) {
        const Epi eb = pf_block_epi(e, a, b0 + wave);
        float pv[KG_ROWS][8];
#pragma unroll
        for (int m = 0; m < KG_ROWS; m++)
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int i = lane + 64 * j;
                pv[m][j] = (eb.ssq_in && m < eb.M && i < eb.nt_in) ? eb.ssq_in[(size_t)i * KG_ROWS + m] : 0.f;
            }
#pragma unroll
        for (int m = 0; m < KG_ROWS; m++) {
            float sv = 1.f;
            if (eb.ssq_in) {
                sv = 0.f;
#pragma unroll
                for (int j = 0; j < 8; j++) sv += pv[m][j];
                for (int o = 32; o >= 1; o >>= 1) sv += __shfl_xor(sv, o);
                sv = rsqrtf(fmaf(sv, eb.inv_d, eb.eps));
            }
            if (lane == 0) scs[wave][m] = sv;
        }
    }

    // A stage is up to PF_KC k-steps of one k-range (a range ends a stage early, so the accumulators
    // are folded between stages only).  Per stage the movers issue a fixed number of tile loads
    // (pieces beyond the stage's end, beyond the last weight tile or the last row block read a valid
    // address again; nobody uses them), so the explicit wait counts below are exact.
    constexpr int TL = PF_KC * (NTW + CBW);             // tile loads of a stage
    constexpr int LPW = TL / 4;                            // ... per mover wave
    static_assert(TL % 4 == 0, "tile loads spread evenly over the 4 mover waves");
    bool valid[PF_TW];
#pragma unroll
    for (int tw = 0; tw < PF_TW; tw++) valid[tw] = rt0 + tw < a.NT;
    const int bsl = b_slot(lane);
    // movers: the address of every tile of the wave at k-step 0 is computed once (tile j = wave - 8 + 4 i is
    // uniform in the wave; the first PF_KC * NTW tiles of a stage are weight tiles [kk][tile], the others
    // activation tiles [kk][row block]); a stage then adds the position of its k-steps
    const u32x4_t *src0[LPW];
    if (mover) {
#pragma unroll
        for (int i = 0; i < LPW; i++) {
            const int j = (wave - 8) + 4 * i;
            if (j < PF_KC * NTW) {
                const int rt = min(gyi * NTW + j % NTW, a.NT - 1);
                src0[i] = a.W + (size_t)rt * KS * 64 + lane;
            } else {
                const int cb = (j - PF_KC * NTW) % CBW;
                src0[i] = a.act + (size_t)(b0 + min(cb, nbw - 1)) * a.act_blk + bsl;
            }
        }
    }
    auto issue = [&](const PfStage &sg, int buf) {         // movers: loads of stage sg into ring slot buf
        const int k0 = sg.r < 8 ? sg.k : 0, n = sg.r < 8 ? sg.n : 0;
        int wpos[PF_KC], apos[PF_KC];
#pragma unroll
        for (int kk = 0; kk < PF_KC; kk++) {
            const int ks = k0 + (kk < n ? kk : 0);
            wpos[kk] = tile_pos_in_range(sg.r < 8 ? sg.r : 0, ks, KS) * 64;
            apos[kk] = ks * 64;
        }
#pragma unroll
        for (int i = 0; i < LPW; i++) {
            const int j = (wave - 8) + 4 * i;              // uniform in the wave
            if (j < PF_KC * NTW) {
                const int kk = j / NTW, tile = j % NTW;
                __builtin_amdgcn_global_load_lds(src0[i] + wpos[kk], &As[buf][kk][tile][0], 16, 0, 0);
            } else {
                const int jb = j - PF_KC * NTW, kk = jb / CBW, cb = jb % CBW;
                __builtin_amdgcn_global_load_lds(src0[i] + apos[kk], &Bs[buf][kk][cb][0], 16, 0, 0);
            }
        }
    };
    auto next_of = [&](const PfStage &sg) { return sg.r < 8 ? pf_stage_at(sg.r, sg.k + sg.n, KS) : sg; };

    // The waves meet at bare barriers: the movers wait explicitly for exactly the loads that are due
    // (a fence would wait for all of them, also those issued two stages ahead), and an LDS-direct
    // load has written its tile once it is counted as complete.  Movers and multipliers run loops
    // of their own with the same number of barriers.
    auto meet = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    PfStage cur = pf_stage_at(0, 0, KS), nx1 = next_of(cur);
    int buf = 0;
    if (mover) {
        PfStage nx2 = next_of(nx1);
        issue(cur, 0);
        issue(nx1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW) : "memory");     // the first stage has landed
        __syncthreads();
        while (cur.r < 8) {
            // slot buf + 2 held the stage multiplied before the last barrier; the stage after the
            // current one must have landed before the next barrier
            issue(nx2, buf >= 1 ? buf - 1 : 2);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW) : "memory");
            meet();
            cur = nx1;
            nx1 = nx2;
            nx2 = next_of(nx2);
            buf = buf == PF_NB - 1 ? 0 : buf + 1;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no load may still be on its way into LDS at the end
        return;
    }
    f32x4_t acc[PF_TW][CBW], tot[PF_TW][CBW];
#pragma unroll
    for (int tw = 0; tw < PF_TW; tw++)
#pragma unroll
        for (int cb = 0; cb < CBW; cb++) {
            acc[tw][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            tot[tw][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }

    __syncthreads();         // first stage in LDS, RMS scales published
    while (cur.r < 8) {
#pragma unroll
        for (int kk = 0; kk < PF_KC; kk++)
            if (kk < cur.n) {
                bf16x8_t av[PF_TW];
#pragma unroll
                for (int tw = 0; tw < PF_TW; tw++) av[tw] = __builtin_bit_cast(bf16x8_t, As[buf][kk][wave * PF_TW + tw][lane]);
#pragma unroll
                for (int cb = 0; cb < CBW; cb++) {
                    const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, Bs[buf][kk][cb][lane]);
#pragma unroll
                    for (int tw = 0; tw < PF_TW; tw++)
                        acc[tw][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[tw], bv, acc[tw][cb], 0, 0, 0);
                }
            }
        if (nx1.r != cur.r) {      // end of a k-range: fold hi/lo, add the range sum in range order
#pragma unroll
            for (int tw = 0; tw < PF_TW; tw++)
#pragma unroll
                for (int cb = 0; cb < CBW; cb++) {
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        float v = acc[tw][cb][r] + __shfl_xor(acc[tw][cb][r], 8);
                        tot[tw][cb][r] = (cur.r == 0) ? v : tot[tw][cb][r] + v;
                    }
                    acc[tw][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
            // empty ranges between cur.r and the next stage's contribute exact zeros
        }
        meet();
        cur = nx1;
        nx1 = next_of(nx1);
        buf = buf == PF_NB - 1 ? 0 : buf + 1;
    }

    // Epilogue straight from the accumulators: after the fold, lane (column m = lane % 16 < 8, group
    // g = lane / 16) holds rows 4g..4g+3 of the 16-row tile for batch row m, i.e. four consecutive
    // output features: vector loads and stores, no staging.  Same arithmetic as the one-token epilogue.
    const int col = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int tw = 0; tw < PF_TW; tw++) {
        const int rt = rt0 + tw;
        const int n0 = rt * 16 + 4 * g4;
        const bool okl = valid[tw] && col < KG_ROWS;
        if (e.kind == EPI_RESID) {
            float4 rv[CBW];
            const float4 gv = (okl && e.gain) ? *(const float4 *)(e.gain + n0) : make_float4(1.f, 1.f, 1.f, 1.f);
#pragma unroll
            for (int cb = 0; cb < CBW; cb++) {
                const int M = min(KG_ROWS, a.T - 8 * (b0 + cb));
                rv[cb] = (okl && cb < nbw && col < M) ? *(const float4 *)(e.res + ((size_t)8 * (b0 + cb) + col) * e.N + n0)
                                                       : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int cb = 0; cb < CBW; cb++) {
                if (cb >= nbw) break;
                const Epi eb = pf_block_epi(e, a, b0 + cb);
                const bool live = okl && col < eb.M;
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                if (live) {
                    v[0] = rv[cb].x + tot[tw][cb][0]; v[1] = rv[cb].y + tot[tw][cb][1];
                    v[2] = rv[cb].z + tot[tw][cb][2]; v[3] = rv[cb].w + tot[tw][cb][3];
                    *(float4 *)(eb.xout + (size_t)col * eb.N + n0) = make_float4(v[0], v[1], v[2], v[3]);
                    if (eb.act_out) {
                        const float gq[4] = {gv.x, gv.y, gv.z, gv.w};
                        uint16_t hi[4], lo[4];
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            const float x = rounded(eb.gain ? v[r] * gq[r] : v[r]);
                            hi[r] = f2bf(x);
                            lo[r] = f2bf(x - bf2f(hi[r]));
                        }
                        int lo_off;
                        uint16_t *pa = pf_act_ptr(e.act_out, a.act_out_blk, b0 + cb, col, n0, e.act_pair, lo_off);
                        *(uint2 *)pa = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
                        *(uint2 *)(pa + lo_off) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
                    }
                }
                if (eb.ssq_out) {
                    // sum of squares over the 16 rows of the tile in row order: a chain through the 4 lane groups
                    float sq = 0.f;
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const float up = __shfl(sq, (lane & 15) + 16 * (g > 0 ? g - 1 : 0));
                        if (g4 == g) {
                            float c = g ? up : 0.f;
#pragma unroll
                            for (int r = 0; r < 4; r++) c += rounded(v[r] * v[r]);
                            sq = c;
                        }
                    }
                    if (valid[tw] && g4 == 3 && col < KG_ROWS) eb.ssq_out[(size_t)rt * KG_ROWS + col] = sq;
                }
            }
        } else {
            // a tile of a q, k, v projection's key rows (a tile holds nothing else then): two rotation pairs a lane
            const bool keys = e.k_pairs && __builtin_amdgcn_readfirstlane(rt) >= e.N / 48 && __builtin_amdgcn_readfirstlane(rt) < 2 * (e.N / 48);
            const int c0 = keys ? plain_column(e, n0) : n0;
#pragma unroll
            for (int cb = 0; cb < CBW; cb++) {
                if (cb >= nbw) break;
                const Epi eb = pf_block_epi(e, a, b0 + cb);
                if (!(okl && col < eb.M)) continue;
                const float sc = scs[cb][col];
                if (eb.kind == EPI_PLAIN) {
                    float *o = eb.out + (size_t)col * eb.N + c0;
                    const float y[4] = {tot[tw][cb][0] * sc, tot[tw][cb][1] * sc, tot[tw][cb][2] * sc, tot[tw][cb][3] * sc};
                    if (keys) {
                        *(float2 *)o = make_float2(y[0], y[2]);
                        *(float2 *)(o + (e.k_pairs >> 1)) = make_float2(y[1], y[3]);
                    } else *(float4 *)o = make_float4(y[0], y[1], y[2], y[3]);
                } else {                          // EPI_SWIGLU: rows (2i, 2i+1) = (gate, up) of feature rt*8 + i
                    uint16_t hi[2], lo[2];
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        const float g = tot[tw][cb][2 * i] * sc, u = tot[tw][cb][2 * i + 1] * sc;
                        const float av = rounded(g / (1.f + __expf(-g)) * u);
                        hi[i] = f2bf(av);
                        lo[i] = f2bf(av - bf2f(hi[i]));
                    }
                    const int k0 = rt * 8 + 2 * g4;
                    int lo_off;
                    uint16_t *pa = pf_act_ptr(e.act_out, a.act_out_blk, b0 + cb, col, k0, e.act_pair, lo_off);
                    *(uint32_t *)pa = hi[0] | ((uint32_t)hi[1] << 16);
                    *(uint32_t *)(pa + lo_off) = lo[0] | ((uint32_t)lo[1] << 16);
                }
            }
        }
    }
}

// one or two weight tiles per multiplying wave; row groups of PF_CBW blocks, or of 4 for projections
// with so few weight tiles that groups of 8 would leave compute units without a workgroup
__global__ __launch_bounds__(768) void gemm_prefill_kernel_tw1(PfArgs a, Epi e) { gemm_prefill_body<1, PF_CBW>(a, e); }
__global__ __launch_bounds__(768) void gemm_prefill_kernel_tw2(PfArgs a, Epi e) { gemm_prefill_body<2, PF_CBW>(a, e); }
__global__ __launch_bounds__(768) void gemm_prefill_kernel_tw1_cb4(PfArgs a, Epi e) { gemm_prefill_body<1, 4>(a, e); }

// ---------------------------------------------------------------------------------------------
// RMSNorm scale of every row of a prompt pass: rsqrt(sum of the row's tile sums of squares / d + eps),
// the sums taken in the order of the one-token kernels (a lane adds its tiles lane, lane + 64, .., then
// the lanes are folded).  One workgroup per 8-row block, one wave per row; rows beyond the pass get the
// scale of an all-zero row and are not used.
__global__ __launch_bounds__(512) void pf_rms_scale_kernel(const float *ssq, int ssq_blk, int nt_in, int T, float inv_d,
                                                           float eps, float *scale)
{
    const int b = blockIdx.x, m = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int M = min(KG_ROWS, T - KG_ROWS * b);
    const float *p = ssq + (size_t)b * ssq_blk;
    float pv[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = lane + 64 * j;
        pv[j] = (m < M && i < nt_in) ? p[(size_t)i * KG_ROWS + m] : 0.f;
    }
    float sv = 0.f;
#pragma unroll
    for (int j = 0; j < 8; j++) sv += pv[j];
    for (int o = 32; o >= 1; o >>= 1) sv += __shfl_xor(sv, o);
    if (lane == 0) scale[(size_t)b * KG_ROWS + m] = rsqrtf(fmaf(sv, inv_d, eps));
}

// ---------------------------------------------------------------------------------------------
// Projection for prompt passes of more than 96 rows (192 in narrow models; half-precision cache): the same contraction as
// gemm_prefill_body, organised for reuse instead of for the one-token kernel's summation order (a prompt row then
// differs from the same row decoded alone in the order of its sums only, far inside the logit tolerance).  A
// workgroup owns 6 .. 32 weight tiles x 80 .. 128 rows (pf2_plan picks the numbers that fill whole rounds of
// workgroups, and the rows of the pass, best); a projection with few weight tiles (o_proj, down_proj) is also cut along k, one slice per
// blockIdx.y, into partial sums that pf_reduce_rows_kernel adds with what follows the projection.  The hi and lo
// halves of the activations are two B operands of 16 distinct rows each (two
// 8-row blocks) that are multiplied into the SAME accumulator, so nothing is folded and no per-range
// totals are kept: a weight tile fetched from the L2 serves all rows of the group and an activation tile serves up to
// 512 weight rows.  The activations arrive in the pair layout of pf_act_ptr (a B operand = one KB).
//   12 waves: waves 8..11 move, waves 0..7 multiply.  The movers bring the operand tiles of a k-step
// straight into an LDS ring of NB stage buffers (global_load_lds), NB - 1 stages ahead, and wait with
// exact counts; their loop holds nothing but the loads: every tile's address at step 0 is computed
// once, and the k loop walks a row tile's weight tiles in the order they are stored (contiguous memory;
// the sum over k may take any order here) and works out the k-step each one holds (kstep_at_pos) to pick the
// matching activation tile.
//   PIPE (all but 32 tiles): the multiplying waves are arranged 4 x 2 (2 x 4 for 6 tiles), so that a wave reads
// few operands from LDS per multiplication; all reads of a k-step are issued together, the hi halves are
// multiplied into every accumulator before the lo halves, and the operands of k-step ks + 1 are read under the
// second half of step ks (two register sets).  Without PIPE (32 tiles, whose 128 accumulator registers leave no
// room for a second set) a wave owns 4 weight tiles x all pairs of the group.
// AW x (8 / AW) multiplying waves; a wave owns WA weight tiles x its share of the workgroup's NP pairs of 8-row blocks; NB
// stage buffers
template <int AW, int WA, int NP, int NB, bool PIPE>
__device__ __forceinline__ void gemm_prefill2_body(const PfArgs &a, const Epi &e)
{
    constexpr int NTW = AW * WA, RB = 2 * NP;               // weight tiles and 8-row blocks of the workgroup
    constexpr int PG = 8 / AW, WPM = (NP + PG - 1) / PG;    // the pairs are shared out to PG groups of waves: WPM pairs, the last group the rest
    static_assert(PG <= 2 || NP % PG == 0, "with more than two groups of waves every group owns as many pairs");
    __shared__ u32x4_t As[NB][NTW][64];                     // ring of NB stage buffers, one k-step each
    __shared__ u32x4_t Bs[NB][NP][2][64];
    __shared__ float scs[RB][KG_ROWS];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const bool mover = wave >= 8;
    const int nb = (a.T + 7) >> 3;
    int rgi, gyi;
    if (!pf_work(a, rgi, gyi)) return;
    const int b0 = rgi * RB;
    const int nbw = min(RB, nb - b0);
    const int KS = a.KS;
    // a projection cut along k: this workgroup's slice of the positions of a row tile
    const int p_lo = PIPE ? __builtin_amdgcn_readfirstlane((int)(blockIdx.y * KS / gridDim.y)) : 0;
    const int p_hi = PIPE ? __builtin_amdgcn_readfirstlane((int)((blockIdx.y + 1) * KS / gridDim.y)) : KS;
    const int col = lane & 15, g4 = lane >> 4;
    const int a0 = (wave % AW) * WA;                        // first weight tile and first pair of a multiplying wave
    const int wg = (wave & 7) / AW, g0 = wg * WPM;

    // RMS scales of the group's rows (computed once per pass by pf_rms_scale_kernel: every workgroup summing
    // the tile sums of its rows again cost a tenth of a short pass); read after the main loop's barriers
    if (t < nbw * KG_ROWS) scs[t >> 3][t & 7] = e.scale_in ? e.scale_in[(size_t)b0 * KG_ROWS + t] : 1.f;

    constexpr int TL = NTW + RB;                            // tile loads of a stage
    constexpr int LPW = (TL + 3) / 4;                       // ... per mover wave (one too many for some: it repeats the last tile)
    auto meet = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // the movers run NB - 1 stages ahead: when stage ks is multiplied, stages ks + 1 .. ks + NB - 1 are on
    // their way or have landed; after issuing one more, at most NB - 2 stages may still be in flight
    // for the next stage to be complete
    static_assert((NB - 2) * LPW <= 63, "the wait count must fit the instruction's field");
    int buf = 0;
    if (mover) {
        const u32x4_t *src0[LPW];                           // the wave's tiles at k-step 0 (tile j = wave - 8 + 4 i: uniform in the wave)
#pragma unroll
        for (int i = 0; i < LPW; i++) {
            const int j = min((wave - 8) + 4 * i, TL - 1);
            if (j < NTW) {
                const int rt = min(gyi * NTW + j, a.NT - 1);
                src0[i] = a.W + (size_t)rt * KS * 64 + lane;
            } else {
                const int jb = j - NTW, grp = jb >> 1, part = jb & 1;
                const int pr = min((b0 >> 1) + grp, (nb - 1) >> 1);
                src0[i] = a.act + (size_t)pr * 2 * a.act_blk + part * 64 + lane;
            }
        }
        int next_apos = kstep_at_pos(p_lo, KS) * 128;       // worked out a stage ahead, under the loads (in place: 0.4 % of a 777-token prompt)
        auto issue = [&](int ks, int bf) {                  // operands of position ks (clamped: late stages reload a valid one)
            const int wpos = min(ks, p_hi - 1) * 64, apos = next_apos;
            next_apos = kstep_at_pos(min(ks + 1, p_hi - 1), KS) * 128;
#pragma unroll
            for (int i = 0; i < LPW; i++) {
                const int j = min((wave - 8) + 4 * i, TL - 1);
                if (j < NTW) __builtin_amdgcn_global_load_lds(src0[i] + wpos, &As[bf][j][0], 16, 0, 0);
                else __builtin_amdgcn_global_load_lds(src0[i] + apos, &Bs[bf][(j - NTW) >> 1][(j - NTW) & 1][0], 16, 0, 0);
            }
        };
#pragma unroll
        for (int s0 = 0; s0 < NB - 1; s0++) issue(p_lo + s0, s0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * LPW) : "memory");
        __syncthreads();
        for (int ks = p_lo; ks < p_hi; ks++) {
            issue(ks + NB - 1, buf >= 1 ? buf - 1 : NB - 1);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * LPW) : "memory");
            meet();
            buf = buf == NB - 1 ? 0 : buf + 1;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    // a multiplying wave with WP pairs from pair g0 on
    auto multiply = [&](auto pairs) {
    constexpr int WP = decltype(pairs)::value;
    f32x4_t acc[WA][WP];
#pragma unroll
    for (int ta = 0; ta < WA; ta++)
#pragma unroll
        for (int gb = 0; gb < WP; gb++) acc[ta][gb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (PIPE) {
        struct Frag { bf16x8_t av[WA], bh[WP], bl[WP]; };
        auto fetch = [&](Frag &f, int bf) {
#pragma unroll
            for (int ta = 0; ta < WA; ta++) f.av[ta] = __builtin_bit_cast(bf16x8_t, As[bf][a0 + ta][lane]);
#pragma unroll
            for (int gb = 0; gb < WP; gb++) f.bh[gb] = __builtin_bit_cast(bf16x8_t, Bs[bf][g0 + gb][0][lane]);
#pragma unroll
            for (int gb = 0; gb < WP; gb++) f.bl[gb] = __builtin_bit_cast(bf16x8_t, Bs[bf][g0 + gb][1][lane]);
        };
        // Between the halves of a step: the barrier after which stage ks + 1 has landed (and no wave still
        // reads the stage before), and the reads of that stage.
        auto step = [&](const Frag &cur, Frag &nxt) {
#pragma unroll
            for (int gb = 0; gb < WP; gb++)
#pragma unroll
                for (int ta = 0; ta < WA; ta++)
                    acc[ta][gb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.av[ta], cur.bh[gb], acc[ta][gb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            meet();
            buf = buf == NB - 1 ? 0 : buf + 1;
            __builtin_amdgcn_sched_barrier(0);
            fetch(nxt, buf);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int gb = 0; gb < WP; gb++)
#pragma unroll
                for (int ta = 0; ta < WA; ta++)
                    acc[ta][gb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.av[ta], cur.bl[gb], acc[ta][gb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        __syncthreads();
        Frag fa, fb;
        fetch(fa, 0);
        // (the reads after the last step's barrier fetch a stage the movers filled with a valid, unused k-step)
        for (int ks = p_lo; ks < p_hi; ks += 2) {
            step(fa, fb);
            if (ks + 1 < p_hi) step(fb, fa);
        }
    } else {
        __syncthreads();
        for (int ks = p_lo; ks < p_hi; ks++) {
            bf16x8_t av[WA];
#pragma unroll
            for (int ta = 0; ta < WA; ta++) av[ta] = __builtin_bit_cast(bf16x8_t, As[buf][a0 + ta][lane]);
#pragma unroll
            for (int gb = 0; gb < WP; gb++) {
                const bf16x8_t bh = __builtin_bit_cast(bf16x8_t, Bs[buf][g0 + gb][0][lane]);
                const bf16x8_t bl = __builtin_bit_cast(bf16x8_t, Bs[buf][g0 + gb][1][lane]);
#pragma unroll
                for (int ta = 0; ta < WA; ta++) {
                    acc[ta][gb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ta], bh, acc[ta][gb], 0, 0, 0);
                    acc[ta][gb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ta], bl, acc[ta][gb], 0, 0, 0);
                }
            }
            meet();
            buf = buf == NB - 1 ? 0 : buf + 1;
        }
    }

    // Epilogue from the accumulators: lane (column c, group g4) holds weight rows 4 g4 .. 4 g4 + 3 of a
    // tile for row c of its pair of blocks.  (Rows are addressed from the launch's own pointers: copies per
    // 8-row block spilled registers here, 35 us per round of workgroups of 32 tiles.)
    const int rt0 = gyi * NTW + a0;
#pragma unroll
    for (int gb = 0; gb < WP; gb++) {
        const int lrow = (g0 + gb) * 16 + col, row = b0 * KG_ROWS + lrow;      // row in the group, in the pass
        const bool row_ok = row < a.T;
        const float sc = (e.kind != EPI_RESID && row_ok) ? scs[lrow >> 3][lrow & 7] : 1.f;
        uint16_t *kv_row = e.kind == EPI_QKV && row_ok ? kv_out_row(a.kv, row) : nullptr;
#pragma unroll
        for (int ta = 0; ta < WA; ta++) {
            const int rt = rt0 + ta, n0 = rt * 16 + 4 * g4;
            const bool live = rt < a.NT && row_ok;
            const f32x4_t y = acc[ta][gb];
            if (PIPE && a.part) {
                if (live) *(float4 *)(a.part + ((size_t)blockIdx.y * a.T + row) * e.N + n0) = make_float4(y[0], y[1], y[2], y[3]);
            } else if (e.kind == EPI_RESID) {
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                if (live) {
                    const size_t at = (size_t)row * e.N + n0;
                    const float4 rv = *(const float4 *)(e.res + at);
                    v[0] = rv.x + y[0]; v[1] = rv.y + y[1]; v[2] = rv.z + y[2]; v[3] = rv.w + y[3];
                    *(float4 *)(e.xout + at) = make_float4(v[0], v[1], v[2], v[3]);
                    if (e.act_out) {
                        const float4 gv = e.gain ? *(const float4 *)(e.gain + n0) : make_float4(1.f, 1.f, 1.f, 1.f);
                        const float gq4[4] = {gv.x, gv.y, gv.z, gv.w};
                        uint16_t hi[4], lo[4];
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            const float xv = rounded(v[r] * gq4[r]);
                            hi[r] = f2bf(xv);
                            lo[r] = f2bf(xv - bf2f(hi[r]));
                        }
                        int lo_off;
                        uint16_t *pa = pf_act_ptr(e.act_out, a.act_out_blk, row >> 3, row & 7, n0, 1, lo_off);
                        *(uint2 *)pa = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
                        *(uint2 *)(pa + lo_off) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
                    }
                }
                if (e.ssq_out) {                 // sum of squares of the tile's 16 outputs per row: 4 in the lane, then the 4 lane groups
                    float sq = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                    sq += __shfl_xor(sq, 16);
                    sq += __shfl_xor(sq, 32);
                    if (live && g4 == 0) e.ssq_out[(size_t)(row >> 3) * a.ssq_out_blk + (size_t)rt * KG_ROWS + (row & 7)] = sq;
                }
            } else if (live) {
                if (e.kind == EPI_QKV) {
                    store_qkv(a.kv, e.out, kv_row, row, n0, y[0] * sc, y[1] * sc, y[2] * sc, y[3] * sc);
                } else {                          // EPI_SWIGLU: rows (2i, 2i+1) = (gate, up) of feature rt*8 + i
                    uint16_t hi[2], lo[2];
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        const float gt = y[2 * i] * sc, up = y[2 * i + 1] * sc;
                        const float av2 = rounded(gt / (1.f + __expf(-gt)) * up);
                        hi[i] = f2bf(av2);
                        lo[i] = f2bf(av2 - bf2f(hi[i]));
                    }
                    int lo_off;
                    uint16_t *pa = pf_act_ptr(e.act_out, a.act_out_blk, row >> 3, row & 7, rt * 8 + 2 * g4, 1, lo_off);
                    *(uint32_t *)pa = hi[0] | ((uint32_t)hi[1] << 16);
                    *(uint32_t *)(pa + lo_off) = lo[0] | ((uint32_t)lo[1] << 16);
                }
            }
        }
    }
    };
    if (NP % PG == 0 || wg == 0) multiply(std::integral_constant<int, WPM>{});
    else multiply(std::integral_constant<int, NP - (PG - 1) * WPM>{});
}
// named by the weight tiles and the pairs of 8-row blocks of a workgroup
#define PF2_KERNEL(tiles, np, AW, WA, NB, PIPE) \
    __global__ __launch_bounds__(768) void gemm_prefill2_kernel_t##tiles##_p##np(PfArgs a, Epi e) { gemm_prefill2_body<AW, WA, np, NB, PIPE>(a, e); }
#define PF2_KERNELS(tiles, AW, WA, NB, PIPE) \
    PF2_KERNEL(tiles, 5, AW, WA, NB, PIPE) PF2_KERNEL(tiles, 6, AW, WA, NB, PIPE) PF2_KERNEL(tiles, 7, AW, WA, NB, PIPE) PF2_KERNEL(tiles, 8, AW, WA, NB, PIPE)
PF2_KERNEL(6, 8, 2, 3, 6, true)
PF2_KERNELS(8, 4, 2, 6, true)
PF2_KERNELS(12, 4, 3, 5, true)
PF2_KERNELS(16, 4, 4, 4, true)
PF2_KERNELS(32, 8, 4, 3, false)
#undef PF2_KERNELS
#undef PF2_KERNEL

// ---------------------------------------------------------------------------------------------
// Projection for short prompt passes (half-precision cache, 9 rows and more): Y[T][N] = X[T][K] . W^T where
// reading the weights is still what bounds the launch (up to about 96 rows, in narrow models its latency), so the kernel is
// built as a weight stream.  A workgroup of 8 waves owns up to NTW weight tiles x R pairs of 8-row blocks (16 R
// rows); its waves take the k-steps of the row tiles in turn, in the order the tiles are stored, and each wave
// multiplies its k-steps into accumulators of its own: weights and activations go from memory straight into
// registers in operand order (the activations in the pair layout of pf_act_ptr, a 16-row operand = one
// contiguous KB), with no LDS and no barrier until the waves' sums are added at the end.  Per k-step a wave
// reads NTW + 2 R KB for 2 NTW R multiplications: with both sides this small the L1 (64 bytes a clock) is kept
// below the memory's share of a compute unit (about 12 bytes a clock) times that ratio.
//   Loads run D k-steps ahead (a ring of D register sets).  Where the accumulators leave no room for two sets
// (D = 1) the weights are double-buffered and an activation operand is fetched again, for the next step, as
// soon as its multiplications are issued.
//   Projections with few weight tiles (o_proj, down_proj) are cut along k into `slices` (1, 2, 4 or 8; a
// workgroup's slice is fixed by its XCD, so an XCD's L2 holds one slice of the activations) and write partial
// sums; pf_reduce_rows_kernel adds them, in slice order, with what follows the projection.
struct PfStreamArgs {
    const u32x4_t *W;       // weight tiles [NT][tile_pos(ks)][64]
    int KS, NT;
    const u32x4_t *act;     // activations, pair layout; pair p at act + p * act_pair16
    size_t act_pair16;      // 16-byte units per pair of 8-row blocks
    int T;
    int slices, groups, gx; // k slices, groups of weight tiles, groups of 16 R rows
    float *part;            // partial sums [slice][T][N] for pf_reduce_rows_kernel; null: the epilogue (one slice)
    size_t act_out_blk;     // bytes per 8-row block of the output activation (SwiGLU)
    KvOut kv;               // EPI_QKV
};

// Waves of a workgroup: 8, of 256 registers each, while those hold the accumulators and the operands of a step
// and a half; else 4 waves of 512 registers (gate+up of the 7B shape at 96 .. 128 rows: one round of 230
// workgroups of 6 tiles instead of two rounds of workgroups of 3).
__host__ __device__ constexpr int pf_stream_waves(int NTW, int R) { return NTW <= (R <= 2 ? 8 : R == 3 ? 7 : R == 4 ? 6 : 4) ? 8 : 4; }
// register sets of the ring: what a wave's registers leave beside the accumulators and the addresses
__host__ __device__ constexpr int pf_stream_depth(int NTW, int R)
{
    const int free = (pf_stream_waves(NTW, R) == 8 ? 204 : 440) - 4 * NTW * R, set = 4 * (NTW + 2 * R), d = free / set;
    return d < 2 ? 1 : d > 8 ? 8 : d;
}

template <int NTW, int R>
__global__ __launch_bounds__(64 * pf_stream_waves(NTW, R), pf_stream_waves(NTW, R) / 4) void gemm_stream_kernel(const PfStreamArgs a, const Epi e)
{
    constexpr int D = pf_stream_depth(NTW, R), NW = pf_stream_waves(NTW, R);
    constexpr int NACC = NTW * R, CH = NACC < 8 ? NACC : 8;         // accumulator tiles added per round at the end
    __shared__ f32x4_t red[NW][CH][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int slice = xcd % a.slices, per = 8 / a.slices;
    const int rg = j % a.gx, tg = (j / a.gx) * per + xcd / a.slices;
    if (tg >= a.groups) return;
    // the NT tiles are shared out evenly: groups differ by at most one tile, none has more than NTW
    const int rt0 = (int)((long long)tg * a.NT / a.groups), ntw = (int)((long long)(tg + 1) * a.NT / a.groups) - rt0;
    const int KS = a.KS;
    const int p_lo = (int)((long long)slice * KS / a.slices), p_hi = (int)((long long)(slice + 1) * KS / a.slices);
    const int p0 = p_lo + wave;
    const int n = p0 < p_hi ? (p_hi - p0 + NW - 1) / NW : 0;      // the wave's k-steps: positions p0, p0 + NW, ..
    const int n_pairs = (a.T + 15) >> 4;
    const u32x4_t *wsrc[NTW], *bsrc[R];
#pragma unroll
    for (int t = 0; t < NTW; t++) wsrc[t] = a.W + (size_t)(rt0 + min(t, ntw - 1)) * KS * 64 + lane;
#pragma unroll
    for (int r = 0; r < R; r++) bsrc[r] = a.act + (size_t)min(rg * R + r, n_pairs - 1) * a.act_pair16 + lane;
    f32x4_t acc[NTW][R];
#pragma unroll
    for (int t = 0; t < NTW; t++)
#pragma unroll
        for (int r = 0; r < R; r++) acc[t][r] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mma = [](const u32x4_t &w, const u32x4_t &b, f32x4_t &c) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    };
    if (D >= 2) {
        u32x4_t av[D][NTW], bv[D][R][2];
        auto load = [&](int s, int i) {
            const int p = p0 + NW * i, ks = kstep_at_pos(p, KS);
#pragma unroll
            for (int t = 0; t < NTW; t++) av[s][t] = __builtin_nontemporal_load(wsrc[t] + p * 64);
#pragma unroll
            for (int r = 0; r < R; r++) {
                bv[s][r][0] = bsrc[r][ks * 128];
                bv[s][r][1] = bsrc[r][ks * 128 + 64];
            }
        };
        auto mul = [&](int s) {
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int r = 0; r < R; r++)
#pragma unroll
                    for (int t = 0; t < NTW; t++) mma(av[s][t], bv[s][r][h], acc[t][r]);
        };
#pragma unroll
        for (int s = 0; s < D; s++)
            if (s < n) load(s, s);
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
#pragma unroll
            for (int s = 0; s < D; s++) {
                mul(s);
                load(s, i + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // fewer than 2 D steps are left, the first D of them loaded or on their way
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + s < n) {
                mul(s);
                if (i + s + D < n) load(s, i + s + D);
            }
        i += D;
#pragma unroll
        for (int s = 0; s < D; s++)
            if (i + s < n) mul(s);
    } else if (n > 0) {
        u32x4_t av[2][NTW], bv[R][2];
        auto load_w = [&](int s, int i) {
#pragma unroll
            for (int t = 0; t < NTW; t++) av[s][t] = __builtin_nontemporal_load(wsrc[t] + (p0 + NW * i) * 64);
        };
        // step i on weight set s; the weights of step i + 1 are requested before, its activations under the multiplications
        auto step = [&](int s, int i) {
            const int in = min(i + 1, n - 1), ks = kstep_at_pos(p0 + NW * in, KS) * 128;     // (the last step fetches itself again)
            load_w(s ^ 1, in);
#pragma unroll
            for (int r = 0; r < R; r++) {
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int t = 0; t < NTW; t++) mma(av[s][t], bv[r][h], acc[t][r]);
                bv[r][0] = bsrc[r][ks];
                bv[r][1] = bsrc[r][ks + 64];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        load_w(0, 0);
        const int ks = kstep_at_pos(p0, KS) * 128;
#pragma unroll
        for (int r = 0; r < R; r++) { bv[r][0] = bsrc[r][ks]; bv[r][1] = bsrc[r][ks + 64]; }
        int i = 0;
        for (; i + 2 <= n; i += 2) { step(0, i); step(1, i + 1); }
        if (i < n) step(0, i);
    }
    // Add the waves' sums, CH accumulator tiles at a time (wave w finishes tiles c + w, c + w + NW, ..), in wave order.
    // Lane (column c, group g4) then holds weight rows 4 g4 .. 4 g4 + 3 of a tile for row c % 8 of its block.
    const int col = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int c = 0; c < NACC; c += CH) {
        if (c) __syncthreads();
#pragma unroll
        for (int u = 0; u < CH; u++)
            if (c + u < NACC) red[wave][u][lane] = acc[(c + u) / R][(c + u) % R];
        __syncthreads();
        for (int u = wave; u < CH; u += NW) {
            const int at = c + u, ta = at / R, r = at % R;
            if (at >= NACC || ta >= ntw) continue;
            f32x4_t y = red[0][u][lane];
#pragma unroll
            for (int w = 1; w < NW; w++) y += red[w][u][lane];
            const int rt = rt0 + ta, n0 = rt * 16 + 4 * g4, row = (rg * R + r) * 16 + col;
            if (row >= a.T) continue;
            if (a.part) {
                *(float4 *)(a.part + ((size_t)slice * a.T + row) * e.N + n0) = make_float4(y[0], y[1], y[2], y[3]);
                continue;
            }
            const float sc = e.scale_in ? e.scale_in[row] : 1.f;
            if (e.kind == EPI_QKV) {
                store_qkv(a.kv, e.out, kv_out_row(a.kv, row), row, n0, y[0] * sc, y[1] * sc, y[2] * sc, y[3] * sc);
            } else {                          // EPI_SWIGLU: rows (2i, 2i+1) = (gate, up) of feature rt*8 + i
                uint16_t hi[2], lo[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const float gt = y[2 * i] * sc, up = y[2 * i + 1] * sc;
                    const float av2 = rounded(gt / (1.f + __expf(-gt)) * up);
                    hi[i] = f2bf(av2);
                    lo[i] = f2bf(av2 - bf2f(hi[i]));
                }
                int lo_off;
                uint16_t *pa = pf_act_ptr(e.act_out, a.act_out_blk, row >> 3, row & 7, rt * 8 + 2 * g4, 1, lo_off);
                *(uint32_t *)pa = hi[0] | ((uint32_t)hi[1] << 16);
                *(uint32_t *)(pa + lo_off) = lo[0] | ((uint32_t)lo[1] << 16);
            }
        }
    }
}

// What follows a projection cut along k: x = res + the slices' partial sums (slice order), xout = x, the next
// projection's input x * gain (pair layout) and the row's RMSNorm scale.  One workgroup per row.
__global__ __launch_bounds__(1024) void pf_reduce_rows_kernel(const float *part, int slices, int T, int d, const float *res, float *xout,
                                                             const float *gain, void *act_out, size_t act_blk, float inv_d, float eps,
                                                             float *scale)
{
    __shared__ float red[16];
    const int row = blockIdx.x, t = threadIdx.x;
    float ss = 0.f;
    for (int k = 4 * t; k < d; k += 4096) {
        float4 v = *(const float4 *)(res + (size_t)row * d + k);
        float4 p[8];
#pragma unroll
        for (int s = 0; s < 8; s++)
            if (s < slices) p[s] = *(const float4 *)(part + ((size_t)s * T + row) * d + k);
        float4 y = p[0];
#pragma unroll
        for (int s = 1; s < 8; s++)
            if (s < slices) { y.x += p[s].x; y.y += p[s].y; y.z += p[s].z; y.w += p[s].w; }
        v.x += y.x; v.y += y.y; v.z += y.z; v.w += y.w;
        *(float4 *)(xout + (size_t)row * d + k) = v;
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        if (act_out) {
            const float4 g = gain ? *(const float4 *)(gain + k) : make_float4(1.f, 1.f, 1.f, 1.f);
            const float q[4] = {v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w};
            uint16_t hi[4], lo[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float x = rounded(q[i]);
                hi[i] = f2bf(x);
                lo[i] = f2bf(x - bf2f(hi[i]));
            }
            int lo_off;
            uint16_t *pa = pf_act_ptr(act_out, act_blk, row >> 3, row & 7, k, 1, lo_off);
            *(uint2 *)pa = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
            *(uint2 *)(pa + lo_off) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
        }
    }
    for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
    if ((t & 63) == 0) red[t >> 6] = ss;
    __syncthreads();
    if (t == 0) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < 16; w++) s += red[w];
        scale[row] = rsqrtf(fmaf(s, inv_d, eps));
    }
}

// ---------------------------------------------------------------------------------------------
// Rows -> activation for the first projection of a stack: x[m] = E[tok[m]] (emb != null) or the
// given fp32 rows; writes xout (optional), act = x * gain (hi/lo), ssq[tile][m].  One block per
// 16 features.
struct Tok8 { int t[KG_ROWS]; int vocab; };   // token ids given by the host; vocab bounds the ids read from device memory too

template <bool BF>
__global__ __launch_bounds__(128) void pack_rows_kernel(const void *emb, Tok8 tok, const int *tok_dev,
                                                        const float *rows, int d, int M, const float *gain,
                                                        float *xout, void *act, float *ssq,
                                                        size_t act_blk_bytes = 0, int ssq_blk = 0, int act_pair = 0)
{
    __shared__ float sq[16][KG_ROWS];
    // blockIdx.y selects a block of 8 rows (prefill passes many blocks in one launch; M is then the
    // total row count and every per-row pointer advances by 8 rows per block)
    const int blk = blockIdx.y;
    void *const act_base = act;
    if (blk) {
        M -= 8 * blk;
        if (tok_dev) tok_dev += 8 * blk;
        if (rows) rows += (size_t)8 * blk * d;
        if (xout) xout += (size_t)8 * blk * d;
        act = (char *)act + (size_t)blk * act_blk_bytes;
        if (ssq) ssq += (size_t)blk * ssq_blk;
    }
    if (M > KG_ROWS) M = KG_ROWS;
    int rt = blockIdx.x, row = threadIdx.x >> 3, m = threadIdx.x & 7;
    int n = rt * 16 + row;
    float v = 0.f;
    if (m < M) {
        if (emb) {
            // token ids from the host or from device memory; an id a kernel produced from non-finite
            // logits may be anything: it is clamped so that the gather stays inside the table (the host
            // reports the bad token)
            const int id = min(max(tok_dev ? tok_dev[m] : tok.t[m], 0), tok.vocab - 1);
            size_t idx = (size_t)id * d + n;
            v = BF ? bf2f(((const uint16_t *)emb)[idx]) : ((const float *)emb)[idx];
        } else {
            v = rows[(size_t)m * d + n];
        }
        if (xout) xout[(size_t)m * d + n] = v;
        if (BF && act_pair) store_act_pf(act_base, act_blk_bytes, blk, m, n, gain ? v * gain[n] : v, 1);
        else store_act<BF>(act, d, m, n, gain ? v * gain[n] : v);
    }
    sq[row][m] = v * v;
    __syncthreads();
    if (threadIdx.x < KG_ROWS && ssq) {
        float s = 0.f;
        for (int r = 0; r < 16; r++) s += sq[r][threadIdx.x];
        ssq[(size_t)rt * KG_ROWS + threadIdx.x] = s;
    }
}

// ---------------------------------------------------------------------------------------------
// Weight re-tiling.  Destination row of source row r: mode 0: row_off + r; mode 1 (gate): 16*(r/8)
// + 2*(r%8); mode 2 (up): the same + 1, so a tile holds 8 (gate, up) pairs.  qkv_rows(d, head_dim): row_off + r of the stacked q, k, v
// rows, with the keys of a head stored in rotation pairs (0, hd/2), (1, hd/2 + 1), ..: a lane of a prompt projection then holds
// whole pairs, and its epilogue can rotate them and write the cache.
__host__ __device__ __forceinline__ constexpr int qkv_rows(int d, int head_dim) { return (d << 8) | head_dim; }
__device__ __forceinline__ int map_row(int r, int row_off, int mode)
{
    if (mode > 2) {
        const int d = mode >> 8, hd = mode & 255, R = row_off + r, j = (R - d) & (hd - 1);
        return (R >= d && R < 2 * d) ? R - j + 2 * (j & ((hd >> 1) - 1)) + (j >= (hd >> 1)) : R;
    }
    return mode == 0 ? row_off + r : 16 * (r >> 3) + 2 * (r & 7) + (mode - 1);
}

__global__ void pack_w_bf16_kernel(const uint16_t *src, int rows, int K, u32x4_t *dst, int KS, int row_off,
                                   int mode)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)rows * KS * 4;
    if (i >= total) return;
    int g = (int)(i & 3);
    int ks = (int)((i >> 2) % KS);
    int r = (int)((i >> 2) / KS);
    int k0 = ks * 32 + g * 8;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (k0 + 8 <= K) v = *(const u32x4_t *)(src + (size_t)r * K + k0);
    int R = map_row(r, row_off, mode);
    dst[((size_t)(R >> 4) * KS + tile_pos(ks, KS)) * 64 + g * 16 + (R & 15)] = v;
}

__global__ void pack_w_f32_kernel(const float *src, int rows, int K, float *dst, int row_off, int mode)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * K) return;
    int r = (int)(i / K), k = (int)(i % K);
    dst[(size_t)map_row(r, row_off, mode) * K + k] = src[i];
}

__global__ void gain_to_f32_kernel(const void *src, int bf, int n, float *dst)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = bf ? bf2f(((const uint16_t *)src)[i]) : ((const float *)src)[i];
}

// cos/sin table of the rotary embedding, angle = pos * inv_freq[i] evaluated in double.
__global__ void rope_table_kernel(float2 *tab, int max_seq, int half, const double *inv_freq)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= max_seq * half) return;
    double a = (double)(i / half) * inv_freq[i % half];
    tab[i] = make_float2((float)cos(a), (float)sin(a));
}

// ---------------------------------------------------------------------------------------------
// Decode attention over a paged KV cache for up to 8 query rows at positions pos0..pos0+M-1.
// grid = (heads, pages in use, blocks of 8 rows); block = 512.  A block handles one head and one
// page of P positions: it rotates q (and k), appends the new k/v rows that fall in its page,
// computes scores, a page-local softmax and P.V, and stores an unnormalised partial.  The last
// block to finish for a head merges the partials in an order fixed by the page numbers (so results do not
// depend on arrival order, nor on how many rows or trailing pages the launch had).
// The argument block is only read (never indexed dynamically, never modified): it then stays in
// scalar registers instead of being copied to private memory.
struct AttnArgs {
    const float *qkv;   // [M][3d]: q | k | v, already RMS-scaled projections
    int d, H, M, pos0, P, logP;
    const int *page_table;
    int pages[16];      // copy of the first 16 page-table entries (saves a dependent load)
    void *kv;           // pool: [phys page][slot][head][K|V][P][hd]
    int slot, n_slots;
    const float2 *rope; // [max_seq][hd/2]
    float *opart;       // [row block][H][S][8][hd]
    float *mxs, *sms;   // [row block][H][S][8]
    int *cnt;           // [row block][H], zero between launches
    int S;              // pages covered by this launch = ceil((pos0+M)/P)
    void *act_out;      // attention output as activation for the output projection (K = d)
    int append_only;    // 1: only append k/v
    // prefill: blockIdx.z selects a block of 8 rows; M is then the total row count
    size_t act_blk_bytes;   // bytes per 8-row block of act_out
    int preappended;    // 1: this call's k/v rows are already in the cache (appended by an earlier launch)
    int append_all;     // with append_only: write every row of the block to its own page (grid.y = 1)
};

// Element types of the KV cache: float, uint16_t (bfloat16 bit patterns), kvhalf_t (IEEE half bit
// patterns).  Keys and values are O(1) numbers, far inside the half range; half keeps three more
// significant bits than bfloat16 in the same two bytes.
// A half only ever exists as an integer bit pattern in memory, registers and aggregates here, and is
// converted at the point of use (arrays of structs with a _Float16 member that are filled
// conditionally came out of the compiler with every second element undefined).
struct kvhalf_t { uint16_t bits; };
static_assert(sizeof(kvhalf_t) == 2, "two-byte cache element");
template <typename T> __device__ __forceinline__ float kv_ld(const T *p);
template <> __device__ __forceinline__ float kv_ld<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float kv_ld<uint16_t>(const uint16_t *p) { return bf2f(*p); }
template <> __device__ __forceinline__ float kv_ld<kvhalf_t>(const kvhalf_t *p) { return half_bits_to_f32(p->bits); }
template <typename T> __device__ __forceinline__ float kv_round(float v);     // value as the cache type holds it
template <> __device__ __forceinline__ float kv_round<float>(float v) { return v; }
template <> __device__ __forceinline__ float kv_round<uint16_t>(float v) { return bf2f(f2bf(v)); }
template <> __device__ __forceinline__ float kv_round<kvhalf_t>(float v) { return half_bits_to_f32(f32_to_half_bits(rounded(v))); }
template <typename T> __device__ __forceinline__ void kv_st(T *p, float v);
template <> __device__ __forceinline__ void kv_st<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void kv_st<uint16_t>(uint16_t *p, float v) { *p = f2bf(v); }
template <> __device__ __forceinline__ void kv_st<kvhalf_t>(kvhalf_t *p, float v) { p->bits = f32_to_half_bits(v); }

template <typename T, int N8> struct KvVec;           // N8 groups of 8 cache elements, loaded as 16-byte pieces (byte offset in a buffer)
template <int N8> struct KvVec<uint16_t, N8> {
    u32x4_t r[N8];
    __device__ __forceinline__ void load(buffer_t b, uint32_t off)
    {
#pragma unroll
        for (int i = 0; i < N8; i++) r[i] = __builtin_amdgcn_raw_buffer_load_b128(b, off + 16 * i, 0, 0);
    }
    __device__ __forceinline__ float get(int i) const
    {
        uint32_t w = r[i >> 3][(i >> 1) & 3];
        return __uint_as_float((i & 1) ? (w & 0xFFFF0000u) : (w << 16));
    }
};
template <int N8> struct KvVec<kvhalf_t, N8> {
    u32x4_t r[N8];
    __device__ __forceinline__ void load(buffer_t b, uint32_t off)
    {
#pragma unroll
        for (int i = 0; i < N8; i++) r[i] = __builtin_amdgcn_raw_buffer_load_b128(b, off + 16 * i, 0, 0);
    }
    __device__ __forceinline__ float get(int i) const
    {
        const uint32_t w = r[i >> 3][(i >> 1) & 3];
        return half_bits_to_f32((i & 1) ? (w >> 16) : (w & 0xFFFFu));
    }
};
template <int N8> struct KvVec<float, N8> {
    u32x4_t r[2 * N8];
    __device__ __forceinline__ void load(buffer_t b, uint32_t off)
    {
#pragma unroll
        for (int i = 0; i < 2 * N8; i++) r[i] = __builtin_amdgcn_raw_buffer_load_b128(b, off + 16 * i, 0, 0);
    }
    __device__ __forceinline__ float get(int i) const { return __uint_as_float(r[i >> 2][i & 3]); }
};

// E consecutive cache elements owned by one lane in the P.V pass (E = head_dim / 64)
template <typename T, int E> struct KvLane;
template <> struct KvLane<uint16_t, 2> {
    uint32_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0); }
    __device__ __forceinline__ float get(int e) const { return __uint_as_float(e ? (r & 0xFFFF0000u) : (r << 16)); }
};
template <> struct KvLane<uint16_t, 1> {
    uint16_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b16(b, off, 0, 0); }
    __device__ __forceinline__ float get(int) const { return bf2f(r); }
};
template <> struct KvLane<kvhalf_t, 2> {
    uint32_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0); }
    __device__ __forceinline__ float get(int e) const { return half_bits_to_f32(e ? (r >> 16) : (r & 0xFFFFu)); }
};
template <> struct KvLane<kvhalf_t, 1> {
    uint32_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b16(b, off, 0, 0); }
    __device__ __forceinline__ float get(int) const { return half_bits_to_f32(r); }
};
template <> struct KvLane<float, 2> {
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    u32x2_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0); }
    __device__ __forceinline__ float get(int e) const { return __uint_as_float(r[e]); }
};
template <> struct KvLane<float, 1> {
    uint32_t r;
    __device__ __forceinline__ void load(buffer_t b, uint32_t off) { r = __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0); }
    __device__ __forceinline__ float get(int) const { return __uint_as_float(r); }
};

// physical page of logical page s: the first 16 come from the argument block through a chain of
// selects on constant indices
__device__ __forceinline__ int attn_page(const AttnArgs &a, int s)
{
    if (s >= 16) return ((const __attribute__((address_space(4))) int *)a.page_table)[s];       // (a scalar load: nothing writes the table here)
    int p = a.pages[0];
#pragma unroll
    for (int i = 1; i < 16; i++) p = (s == i) ? a.pages[i] : p;
    return p;
}

// max / sum over the wave of a value that is uniform over groups of 4 lanes, in the order of the
// xor butterfly over offsets 4, 8, 16, 32 (the last two levels combine the four 16-lane rows as
// (r0 . r1) . (r2 . r3), which is what every lane of that butterfly ends with)
__device__ __forceinline__ float wave_max_q4(float v)
{
    v = fmaxf(v, half_mirror(v));
    v = fmaxf(v, row_mirror(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
// values of 16 lanes (a row), of the whole wave; every lane gets the result
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, quad_x1(v));
    v = fmaxf(v, quad_x2(v));
    v = fmaxf(v, half_mirror(v));
    return fmaxf(v, row_mirror(v));
}
__device__ __forceinline__ float row_sum(float v)
{
    v += quad_x1(v);
    v += quad_x2(v);
    v += half_mirror(v);
    return v + row_mirror(v);
}
__device__ __forceinline__ float wave_max(float v)
{
    v = row_max(v);
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v = row_sum(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
__device__ __forceinline__ float wave_sum_q4(float v)
{
    v += half_mirror(v);
    v += row_mirror(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}


// One (head, page) unit, 512 threads, MR >= number of rows (1, 2, 4 or 8: less code and fewer
// registers for the common one- and two-row calls; a row's arithmetic is the same in all of them).
// Scores: 4 lanes per position (a quarter of the head dimension each), all 128 positions of a
// page in one pass.  P.V: a wave walks its 16 positions, every lane owning head_dim/64 output
// elements (no cross-lane reduction).  Softmax statistics are kept per wave, then merged across
// the 8 waves, then across pages; every level rescales by exp(max_part - max_all), in a fixed
// order, so a row's result does not depend on the other rows of the batch or on trailing pages.
template <typename T, int HD, bool BF, int MR>
__global__ __launch_bounds__(512, (sizeof(T) == 2 ? 6 : 1)) void attn_kernel(const AttnArgs a)
{
    constexpr int EL = HD / 4;          // elements of one score lane
    constexpr int EPL = HD / 64;        // output elements of one P.V lane
    constexpr int HH = HD / 2;
    __shared__ __align__(16) float qs[MR][HD];
    __shared__ float kn[MR][HD], vn[MR][HD];     // this call's k, v rows as the cache holds them
    __shared__ float ow[8][MR][HD];
    __shared__ float mw[8][MR], sw[8][MR];
    __shared__ __align__(16) float pw[8][MR][16];   // a wave's probabilities [row][position]
    __shared__ __align__(16) float wtl[MR][8];      // weights of the wave merge [row][wave]
    __shared__ float gml[MR];
    __shared__ int last_flag;
    const int h = blockIdx.x, s = blockIdx.y, zb = blockIdx.z, t = threadIdx.x;
    // the wave index as a scalar: conditions on it (which positions a wave owns) become scalar branches
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int P = a.P, d = a.d, logP = a.logP;
    const int pos0 = a.pos0 + 8 * zb;
    const int M = min(MR, a.M - 8 * zb);
    const int S = (pos0 + M + P - 1) >> logP;               // pages this block of rows attends to
    if (!a.append_all && s >= S) return;
    const int hz = zb * a.H + h;                            // index of (row block, head) in the partial buffers
    const float *qkv = a.qkv + (size_t)8 * zb * 3 * d + h * HD;
    const int p_begin = s << logP;
    const int n_valid = min(P, pos0 + M - p_begin);         // positions of this page that hold data
    const int n_old = a.preappended ? n_valid : min(P, max(0, pos0 - p_begin));   // ... cached before this call
    const size_t unit = (size_t)2 * P * HD;                 // K then V of one (page, slot, head)
    T *const Kp = (T *)a.kv + (((size_t)attn_page(a, s) * a.n_slots + a.slot) * a.H + h) * unit;
    T *const Vp = Kp + (size_t)P * HD;
    void *const act_out = (char *)a.act_out + (size_t)zb * a.act_blk_bytes;

    // All loads first, without a condition per lane or position (see buffer_of): this call's rows (thread = row rm, rotation pair rj),
    // which come from the L2 and are waited for alone, then the rows cached by earlier calls: score lane (position pl, quarter sub); P.V lane owns
    // EPL elements.  (With the cached rows requested under conditions the compiler waited for this call's before it
    // asked for any: 7B shape, one row and two pages 6.4 -> 5.6 us, two rows and one page 5.5 -> 5.1.)
    const bool has_row = t < M * HH;
    const int rm = t / HH, rj = t % HH, rpos = pos0 + rm;
    const bool row_here = has_row && !a.preappended && (a.append_all || (rpos >= p_begin && rpos < p_begin + P));
    const int rq = min(rm, M - 1);
    const float *q = qkv + (size_t)rq * 3 * d;
    const float2 cs = a.rope[(size_t)(pos0 + rq) * HH + rj];
    float q0 = q[rj], q1 = q[rj + HH];
    const float k0 = q[d + rj], k1 = q[d + rj + HH], v0 = q[2 * d + rj], v1 = q[2 * d + rj + HH];      // (of no use if !row_here)
    const int pl = t >> 2, sub = t & 3;
    KvVec<T, EL / 8> kreg;
    KvLane<T, EPL> vreg[16];
    {
        const uint32_t cached = a.append_only ? 0 : __builtin_amdgcn_readfirstlane(n_old) * HD * sizeof(T);
        const buffer_t kb = buffer_of(uniform(Kp), cached), vb = buffer_of(uniform(Vp), cached);
        kreg.load(kb, (pl * HD + sub * EL) * sizeof(T));
#pragma unroll
        for (int i = 0; i < 16; i++) vreg[i].load(vb, ((wave * 16 + i) * HD + EPL * lane) * sizeof(T));
    }
    __builtin_amdgcn_sched_barrier(0);
    q0 = rounded(q0); q1 = rounded(q1);         // (the rotation is not begun, and its operands not waited for, above)
    if (!has_row && t < MR * HH) { qs[rm][rj] = 0.f; qs[rm][rj + HH] = 0.f; }   // unused rows of the instantiation
    if (has_row) {
        const float qscale = rsqrtf((float)HD);
        qs[rm][rj] = rot_lo(q0, q1, cs) * qscale;
        qs[rm][rj + HH] = rot_hi(q0, q1, cs) * qscale;
        if (row_here) {
            const float ka = kv_round<T>(rot_lo(k0, k1, cs)), kb = kv_round<T>(rot_hi(k0, k1, cs));
            const float va = kv_round<T>(v0), vb = kv_round<T>(v1);
            T *Kq = Kp, *Vq = Vp;
            int pp = rpos - p_begin;
            if (a.append_all) {
                pp = rpos & (P - 1);
                Kq = (T *)a.kv + (((size_t)a.page_table[rpos >> logP] * a.n_slots + a.slot) * a.H + h) * unit;
                Vq = Kq + (size_t)P * HD;
            }
            kv_st<T>(Kq + (size_t)pp * HD + rj, ka);
            kv_st<T>(Kq + (size_t)pp * HD + rj + HH, kb);
            kv_st<T>(Vq + (size_t)pp * HD + rj, va);
            kv_st<T>(Vq + (size_t)pp * HD + rj + HH, vb);
            kn[rm][rj] = ka; kn[rm][rj + HH] = kb;
            vn[rm][rj] = va; vn[rm][rj + HH] = vb;
        }
    }
    if (a.append_only) return;
    __syncthreads();
    // positions written by this call are taken from LDS (the very values the cache now holds)
    const bool k_new = pl >= n_old && pl < n_valid;
    const int mk = p_begin + pl - pos0;

    // scores and wave-local softmax
    // Every row's dot product runs over the lane's EL elements in ascending order; the cached keys
    // are widened once per 4 elements and used for all rows (rows beyond M multiply zeros).
    float pr[MR], dot[MR];
#pragma unroll
    for (int m = 0; m < MR; m++) dot[m] = 0.f;
    const bool cached_here = wave * 16 < __builtin_amdgcn_readfirstlane(n_old);      // does the wave have a cached position?
    if (cached_here)
#pragma unroll
    for (int i4 = 0; i4 < EL; i4 += 4) {        // (zeros where no position is cached)
        const float kf0 = kreg.get(i4), kf1 = kreg.get(i4 + 1), kf2 = kreg.get(i4 + 2), kf3 = kreg.get(i4 + 3);
#pragma unroll
        for (int m = 0; m < MR; m++) {
            const float4 qv = *(const float4 *)&qs[m][sub * EL + i4];
            dot[m] = fmaf(kf0, qv.x, dot[m]);
            dot[m] = fmaf(kf1, qv.y, dot[m]);
            dot[m] = fmaf(kf2, qv.z, dot[m]);
            dot[m] = fmaf(kf3, qv.w, dot[m]);
        }
    }
    if (k_new) {
#pragma unroll
        for (int m = 0; m < MR; m++)
            if (m < M) {
                dot[m] = 0.f;
#pragma unroll
                for (int i = 0; i < EL; i++) dot[m] = fmaf(kn[mk][sub * EL + i], qs[m][sub * EL + i], dot[m]);
            }
    }
#pragma unroll
    for (int m = 0; m < MR; m++) {
        pr[m] = 0.f;
        if (m < M) {
            float v = dot[m];
            v += quad_x1(v);
            v += quad_x2(v);
            const float sc = (pl < n_valid && p_begin + pl <= pos0 + m) ? v : -INFINITY;
            const float mx = wave_max_q4(sc);
            const float p = (mx == -INFINITY) ? 0.f : __expf(sc - mx);
            const float sum = wave_sum_q4(p);
            pr[m] = p;
            if (lane == 0) { mw[wave][m] = mx; sw[wave][m] = sum; }
        }
    }
    // P.V over the wave's 16 positions; the probability of position i sits in lane 4 i
    float acc[MR][EPL];
#pragma unroll
    for (int m = 0; m < MR; m++)
#pragma unroll
        for (int e = 0; e < EPL; e++) acc[m][e] = 0.f;
    // With 4 or 8 rows the wave passes its probabilities through a private LDS row and reads them
    // back four positions at a time as broadcasts (one lane read per (position, row) otherwise:
    // a third of this loop's vector instructions); the products and their order are the same.
    if (MR >= 4) {
        if ((lane & 3) == 0) {
#pragma unroll
            for (int m = 0; m < MR; m++) pw[wave][m][lane >> 2] = pr[m];
        }
        __builtin_amdgcn_wave_barrier();
    }
    // probability of row m at the wave's position i (rows beyond M carry 0 and are not stored)
    auto prob = [&](int m, int i) { return MR >= 4 ? pw[wave][m][i] : __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr[m]), 4 * i)); };
    if (cached_here)
#pragma unroll
    for (int i4 = 0; i4 < 16; i4 += 4) {        // cached positions (the values of others are zeros here)
        float4 p4[MR];
        if (MR >= 4) {
#pragma unroll
            for (int m = 0; m < MR; m++) p4[m] = *(const float4 *)&pw[wave][m][i4];
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float vv[EPL];
#pragma unroll
            for (int e = 0; e < EPL; e++) vv[e] = vreg[i4 + j].get(e);
#pragma unroll
            for (int m = 0; m < MR; m++) {
                const float p = MR < 4 ? prob(m, i4 + j) : j == 0 ? p4[m].x : j == 1 ? p4[m].y : j == 2 ? p4[m].z : p4[m].w;
#pragma unroll
                for (int e = 0; e < EPL; e++) acc[m][e] = fmaf(p, vv[e], acc[m][e]);
            }
        }
    }
    for (int pv = max(n_old, wave * 16); pv < min(n_valid, wave * 16 + 16); pv++) {        // this call's (uniform in the wave)
#pragma unroll
        for (int m = 0; m < MR; m++) {
            const float p = prob(m, pv - wave * 16);
#pragma unroll
            for (int e = 0; e < EPL; e++) acc[m][e] = fmaf(p, vn[p_begin + pv - pos0][EPL * lane + e], acc[m][e]);
        }
    }
#pragma unroll
    for (int m = 0; m < MR; m++)
        if (m < M) {
#pragma unroll
            for (int e = 0; e < EPL; e++) ow[wave][m][EPL * lane + e] = acc[m][e];
        }
    __syncthreads();
    // merge the 8 waves; a single page is final, otherwise store the page partial
    const bool single = S == 1;
    const size_t pidx = (size_t)hz * a.S + s;
    // weight exp(max_wave - max_all) of every (row, wave), once per block: thread (m, w) = (t / 8, t % 8);
    // a wave without a valid position gets weight 0 (its sums are 0 too)
    if (t < 8 * MR) {
        const float mv = mw[t & 7][t >> 3];
        float gm = mv;
        gm = fmaxf(gm, quad_x1(gm));
        gm = fmaxf(gm, quad_x2(gm));
        gm = fmaxf(gm, half_mirror(gm));
        wtl[t >> 3][t & 7] = (mv == -INFINITY) ? 0.f : __expf(mv - gm);
        if ((t & 7) == 0) gml[t >> 3] = gm;
    }
    __syncthreads();
    for (int i = t; i < M * HD; i += 512) {
        const int m = i / HD, e = i % HD;
        const float gm = gml[m];
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < 8; w++) {
            const float wt = wtl[m][w];
            num = fmaf(wt, ow[w][m][e], num);
            den = fmaf(wt, sw[w][m], den);
        }
        if (single) {
            store_act<BF>(act_out, d, m, h * HD + e, num / den);
        } else {
            st_dev(&a.opart[(pidx * KG_ROWS + m) * HD + e], num);
            if (e == 0) {
                st_dev(&a.mxs[pidx * KG_ROWS + m], gm);
                st_dev(&a.sms[pidx * KG_ROWS + m], den);
            }
        }
    }
    if (single) return;
    // The last block of this head merges the pages, every fourth one and then the four sums, the weights' sum as a tree over the
    // pages: in one order however many pages the launch covers, since those of its last row may be more than the earlier rows have (pages
    // a row does not reach add zeros).  The partials are exchanged with device-scope relaxed atomic stores / loads (write-through,
    // cache-bypassing accesses); every wave waits for its stores to be acknowledged before the block bumps the head's counter.  A
    // device-scope fence would write back and invalidate the whole L2 and costs several microseconds here.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
        const int old = __hip_atomic_fetch_add(&a.cnt[hz], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last_flag = (old == S - 1);
    }
    __syncthreads();
    if (!last_flag) return;
    const size_t hb = (size_t)hz * a.S;
    if (S <= 8) {     // few pages: every load of the merge is issued before any is used
        for (int i = t; i < M * HD; i += 512) {
            const int m = i / HD, e = i % HD;
            float mv[8], ov[8], sv[8];
#pragma unroll
            for (int ss = 0; ss < 8; ss++) {
                const bool in = ss < S;
                mv[ss] = in ? ld_dev(&a.mxs[(hb + ss) * KG_ROWS + m]) : -INFINITY;
                ov[ss] = in ? ld_dev(&a.opart[((hb + ss) * KG_ROWS + m) * HD + e]) : 0.f;
                sv[ss] = in ? ld_dev(&a.sms[(hb + ss) * KG_ROWS + m]) : 0.f;
            }
            float gm = -INFINITY;
#pragma unroll
            for (int ss = 0; ss < 8; ss++) gm = fmaxf(gm, mv[ss]);
            float num[4] = {0.f, 0.f, 0.f, 0.f}, dp[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ss = 0; ss < 8; ss++) {
                if (ss < S) {
                    const float w = (mv[ss] == -INFINITY) ? 0.f : __expf(mv[ss] - gm);
                    num[ss & 3] = fmaf(w, ov[ss], num[ss & 3]);
                    dp[ss] = fmaf(w, sv[ss], 0.f);      // (a product that no addition is fused with)
                }
            }
            const float den = ((dp[0] + dp[4]) + (dp[2] + dp[6])) + ((dp[1] + dp[5]) + (dp[3] + dp[7]));
            store_act<BF>(act_out, d, m, h * HD + e, (((num[0] + num[1]) + num[2]) + num[3]) / den);
        }
        if (t == 0) __hip_atomic_store(&a.cnt[hz], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    // Many pages: four groups of HD threads take every fourth page, as above, MB rows and JB pages of loads in flight; the first of them fly
    // while wave m works out the page weights exp(max_page - max_all) and the sum of row m, which go through LDS, as do the groups' sums (added
    // in group order).  (One group and weights read twice, 8 loads at a time: a launch of one row at 4000 positions 17.7 us, of seven 30.2; here
    // 16.1 and 28.2.  Seven rows, four of them and 8 pages at a time: 20.2 us at 9 pages, 21.0 at 16, half of the loads of no use; here 19.2 and 20.0.)
    constexpr int G = 4, MB = MR < 2 ? 1 : MR < 4 ? 2 : HD == 128 ? MR : MR / 2, JB = MR < 8 ? 8 : 4;
    float (*gsum)[MR][HD] = ow;                             // [group - 1][row][element]
    float (*wgt)[MR] = (float (*)[MR]) & ow[3][0][0];       // [page][row], S <= 128 <= 5 * HD
    float *denl = &sw[0][0];
    const int e = t % HD, grp = __builtin_amdgcn_readfirstlane(t / HD);
    float ov[MB][JB], num[MR];
    auto load = [&](int m0, int j0) {
#pragma unroll
        for (int r = 0; r < MB; r++)
#pragma unroll
            for (int j = 0; j < JB; j++) {
                const int ss = min(grp + G * (j0 + j), S - 1), m = min(m0 + r, M - 1);
                ov[r][j] = ld_dev(&a.opart[((hb + ss) * KG_ROWS + m) * HD + e]);
            }
    };
    if (grp < G) load(0, 0);
    if (wave < M) {
        const int s0 = min(lane, S - 1), s1 = min(lane + 64, S - 1);
        const float x0 = ld_dev(&a.mxs[(hb + s0) * KG_ROWS + wave]), x1 = ld_dev(&a.mxs[(hb + s1) * KG_ROWS + wave]);
        const float d0 = ld_dev(&a.sms[(hb + s0) * KG_ROWS + wave]), d1 = ld_dev(&a.sms[(hb + s1) * KG_ROWS + wave]);
        float gm = fmaxf(x0, x1);
        for (int o = 32; o >= 1; o >>= 1) gm = fmaxf(gm, __shfl_xor(gm, o));
        const float w0 = lane < S && x0 != -INFINITY ? __expf(x0 - gm) : 0.f, w1 = lane + 64 < S && x1 != -INFINITY ? __expf(x1 - gm) : 0.f;
        if (lane < S) wgt[lane][wave] = w0;
        if (lane + 64 < S) wgt[lane + 64][wave] = w1;
        float den = fmaf(w1, d1, w0 * d0);
        for (int o = 32; o >= 1; o >>= 1) den += __shfl_xor(den, o);
        if (lane == 0) denl[wave] = den;
    }
    __syncthreads();
    const int J = (S + G - 1) / G;
#pragma unroll
    for (int m0 = 0; m0 < MR; m0 += MB) {
        if (m0 >= M || grp >= G) break;
#pragma unroll
        for (int r = 0; r < MB; r++) num[m0 + r] = 0.f;
        for (int j0 = 0; j0 < J; j0 += JB) {
            if (m0 || j0) load(m0, j0);
#pragma unroll
            for (int j = 0; j < JB; j++) {
                const int ss = grp + G * (j0 + j);
                if (ss < S) {
#pragma unroll
                    for (int r = 0; r < MB; r++) num[m0 + r] = fmaf(wgt[ss][min(m0 + r, M - 1)], ov[r][j], num[m0 + r]);
                }
            }
        }
    }
    if (grp > 0 && grp < G) {
#pragma unroll
        for (int m = 0; m < MR; m++)
            if (m < M) gsum[grp - 1][m][e] = num[m];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
        for (int m = 0; m < MR; m++)
            if (m < M) {
                float v = num[m];
#pragma unroll
                for (int g = 1; g < G; g++) v += gsum[g - 1][m][e];
                store_act<BF>(act_out, d, m, h * HD + e, v / denl[m]);
            }
    }
    if (t == 0) __hip_atomic_store(&a.cnt[hz], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------------------------
// Attention of the prompt rows (prefill) on the matrix units, for a half-precision KV cache.  The keys and values of all rows
// of this pass are already in the cache (written by the q, k, v projection).  A wave owns 32 query rows and walks the cache:
//   S^T = K Q^T   A = 32 keys (as stored: one position's 8 consecutive dimensions per lane), B = the rotated, scaled queries held
//         in registers as half hi + lo parts (two MFMAs per step, fp32-grade scores); a lane gets one query row (its column) and
//         positions 8 (r / 4) + 4 (lane / 32) + r % 4 in its 16 registers;
//   row softmax   running maximum and sum per query row (flash-attention recurrence) in powers of two: over a
//         lane's own registers and the lane 32 away, nothing else, since
//   O^T = V^T P   B = the probabilities straight from the score registers, rounded to half (the contraction index may be enumerated
//         in any order as long as both operands agree), A = V^T, which ds_read_b64_tr_b16 gathers from values stored as they are (per 16
//         lanes 4 positions x 16 dimensions, transposed), leaves a query's outputs in the same column: rescaling needs no lane exchange.
// Rows are masked causally; rows beyond the pass are computed and dropped.  The output goes to the activation tiles of the
// output projection (hi + lo bf16 parts per 8-row block), like the decode kernel's.  Numerically the rows differ from the decode
// kernel's in the order of the sums and in the half-precision probabilities (relative 2^-12), far inside the logit tolerance.
//   32 x 32 tiles, because what bounds 16 x 16 ones is the way of K and V out of LDS (512 KB per 128 rows and 128 positions, 4096
// cycles, against 3072 of matrix instructions per SIMD; here 256 KB).  us per launch, 32 heads of 128: 16 x 16 tiles with values transposed
// on the way into LDS / here: 45 rows 10.1 / 6.9, 256 rows 15.0 / 12.4, 777 rows 32.7 / 29.6, 1024 rows 38 / 34, 2048 rows 84 / 71,
// 4096 rows 287 / 208 (0.66 PFLOP/s, hi and lo counted; matrix units busy half the time, the vector units with exponentials and sums the rest).
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));

struct PfAttnArgs {
    const float *qkv;        // [T][3d] rows of this pass: q | k | v, RMS-scaled projections, not rotated
    int d, H, T, pos0, logP;
    const int *page_table;
    const kvhalf_t *kv;      // pool: [phys page][slot][head][K|V][P][hd]
    int slot, n_slots;
    const float2 *rope;      // [max_seq][hd/2]
    void *act_out;           // activation tiles of the output projection, one per 8-row block
    size_t act_blk_bytes;
    int act_pair;            // layout of act_out (pf_act_ptr)
};

// A lane's query (column lane % 32 of the wave's rows from row0 on): rotated, scaled by 1 / sqrt(hd), split into half hi + lo, in
// B-operand order: step ks holds dimensions 16 ks + 8 (lane / 32) .. + 7.
template <int HD>
__device__ __forceinline__ void pf_attn_queries(const PfAttnArgs &a, int h, int row0, int lane, f16x8_t (&qhi)[HD / 16], f16x8_t (&qlo)[HD / 16])
{
    constexpr int HH = HD / 2, KH = HD / 32;        // steps ks and ks + KH hold the two halves of the same rotation pairs
    const int row = min(row0 + (lane & 31), a.T - 1), g = lane >> 5;
    const float *q = a.qkv + (size_t)row * 3 * a.d + h * HD;
    const float2 *rp = a.rope + (size_t)(a.pos0 + row) * HH;
    const float qscale = rsqrtf((float)HD);
    float4 x0[KH][2], x1[KH][2], cs[KH][4];
#pragma unroll
    for (int ks = 0; ks < KH; ks++) {
        const int i0 = 16 * ks + 8 * g;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            x0[ks][j] = *(const float4 *)(q + i0 + 4 * j);
            x1[ks][j] = *(const float4 *)(q + i0 + HH + 4 * j);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) cs[ks][j] = *(const float4 *)(rp + i0 + 2 * j);
    }
#pragma unroll
    for (int ks = 0; ks < KH; ks++) {
        const float xa[8] = {x0[ks][0].x, x0[ks][0].y, x0[ks][0].z, x0[ks][0].w, x0[ks][1].x, x0[ks][1].y, x0[ks][1].z, x0[ks][1].w};
        const float xb[8] = {x1[ks][0].x, x1[ks][0].y, x1[ks][0].z, x1[ks][0].w, x1[ks][1].x, x1[ks][1].y, x1[ks][1].z, x1[ks][1].w};
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float4 c4 = cs[ks][e >> 1];
            const float2 c = (e & 1) ? make_float2(c4.z, c4.w) : make_float2(c4.x, c4.y);
            const float va = rounded(rot_lo(xa[e], xb[e], c) * qscale), vb = rounded(rot_hi(xa[e], xb[e], c) * qscale);
            const _Float16 ha = (_Float16)va, hb = (_Float16)vb;
            qhi[ks][e] = ha; qlo[ks][e] = (_Float16)(va - (float)ha);
            qhi[ks + KH][e] = hb; qlo[ks + KH][e] = (_Float16)(vb - (float)hb);
        }
    }
}

__device__ __forceinline__ f32x16_t f32x16_zero()
{
    return f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

// the larger of a lane's value and that of the lane 32 away; their sum
__device__ __forceinline__ float pair_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Probabilities of NS x 32 scores per query row (s is the lane's: positions as above) relative to 2^m_run, m_run the row's running maximum,
// and their sum.  (The factor log2 e of the exponent comes with the subtraction, as one fused multiply-add: in the queries it would take a
// third of the half range from them.)  Where a row's maximum has grown, what was summed so far (o, l_run) is multiplied by the difference; no
// other row of the wave shows in a row's bits.  A row that has seen no position yet has m_run = -inf and sums 0.
//   m_run is the maximum itself: a row's largest probability is then 1 and exact in half precision.  Following it with a lag of 8 (FlashAttention-4's
// conditional rescaling) saves nothing here (4096 rows of the 7B width, 4 layers: 9.53 ms with, 9.53 without) and costs precision: error of the
// attention output against 64 bits, 1000 rows, 1.5e-4 with, 1.1e-4 without, and with scores 16 times as large 8.5e-5 and 2.3e-5.
template <int NS, int DT>
__device__ __forceinline__ void pf_attn_softmax(f32x16_t (&s)[NS], f16x8_t (&p)[2 * NS], float &m_run, float &l_run, f32x16_t (&o)[DT])
{
    float mx = s[0][0];
#pragma unroll
    for (int i = 0; i < NS; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) mx = fmaxf(mx, s[i][r]);
    constexpr float LOG2E = 1.44269504088896341f;
    mx = pair_max(mx) * LOG2E;
    if (__any(mx > m_run)) {
        const float m_new = fmaxf(m_run, mx);           // (where it stays, scale is 1, or 0 times the zeros of a row without a position)
        const float scale = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));     // 0 for the first positions a row sees
#pragma unroll
        for (int dt = 0; dt < DT; dt++) o[dt] *= scale;
        l_run *= scale;
        m_run = m_new;
    }
    const float m_ref = m_run == -INFINITY ? 0.f : m_run;
    float sum[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NS; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const float v = __builtin_amdgcn_exp2f(fmaf(s[i][r], LOG2E, -m_ref));        // 0 for a masked score
            sum[r & 1] += v;
            p[2 * i + (r >> 3)][r & 7] = (_Float16)v;
        }
    l_run += sum[0] + sum[1];
}

// Values in LDS as [position][HD] halves, the 32-byte pieces of a row permuted so that four rows of one piece lie in different banks.
template <int HD> __device__ __forceinline__ int pf_v_piece(int pos, int piece) { return piece ^ (HD == 128 ? pos & 7 : pos & 3); }

// a lane's 8 values of V^T for dimension 32 dt + lane % 32: positions 16 u + 4 (lane / 32) + {0 .. 3, 8 .. 11} of the 16-position step u
template <int HD>
__device__ __forceinline__ f16x8_t pf_v_operand(const uint16_t *v, int u, int dt, int lane)
{
    const int i = lane & 15, p0 = 16 * u + 4 * (lane >> 5) + (i >> 2);
    f16x4_t part[2];
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const uint16_t *p = v + (p0 + 8 * e) * HD + pf_v_piece<HD>(p0 + 8 * e, 2 * dt + ((lane >> 4) & 1)) * 16 + (i & 3) * 4;
        part[e] = __builtin_bit_cast(f16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)p));
    }
    return __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// 4 consecutive output dimensions k .. k + 3 of a row of the pass
__device__ __forceinline__ void pf_attn_store(const PfAttnArgs &a, int row, int k, const float (&v)[4])
{
    uint16_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float x = rounded(v[i]);
        hi[i] = f2bf(x);
        lo[i] = f2bf(x - bf2f(hi[i]));
    }
    int lo_off;
    uint16_t *p = pf_act_ptr(a.act_out, a.act_blk_bytes, row >> 3, row & 7, k, a.act_pair, lo_off);
    *(uint2 *)p = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
    *(uint2 *)(p + lo_off) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
}

// 16 bytes per lane straight from memory into LDS: from base + off (or addr) of each lane to `lds` (a byte address, uniform in the
// wave) + 16 lane.  In assembly because the compiler, which cannot tell the buffers of a ring apart, would wait for all such loads before
// any read of LDS; it does not count these: whoever reads what they bring waits for them himself (lds_loads_landed, then a barrier).
__device__ __forceinline__ void lds_load16(const void *base, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" ::"s"(base), "v"(off), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void lds_load16(const void *addr, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void lds_loads_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_address(const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p; }

// Longer passes: one workgroup per (head, 128 rows), 4 waves of 32 rows, two workgroups per compute unit (one multiplies while the other
// is at its softmax or its barrier).  Tiles of 64 positions of K and V, two of each in LDS; the next tile comes straight into LDS under
// this one's work (4096 rows: 208 us; through registers, keys under the scores and values under P.V, 223; with two heads at a time on an XCD
// instead of the late row blocks of all its heads first, 245).
template <int HD>
__global__ __launch_bounds__(256, 2) void pf_attn_kernel(const PfAttnArgs a)
{
    constexpr int KS = HD / 16, DT = HD / 32;
    constexpr int CPR = HD / 8, RPL = 64 / CPR; // 16-byte chunks per row; rows a wave's load covers
    constexpr int CH = 16 / RPL;                // loads per wave of a K tile (and of a V tile)
    constexpr int KM = CPR - 1;                 // the chunks of a key row are permuted by the low bits of its position (no bank conflicts)
    __shared__ __align__(16) uint16_t Ks[2][64 * HD];
    __shared__ __align__(16) uint16_t Vs[2][64 * HD];
    __shared__ int pages[128];                  // the page table (a context has at most 128 pages)
    const int h = blockIdx.x, t = threadIdx.x;
    const int rb = (int)gridDim.y - 1 - (int)blockIdx.y;        // late row blocks (most tiles) are scheduled first
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int P = 1 << a.logP;
    const int row0 = rb * 128 + wave * 32;                        // the wave's first row
    const int row = row0 + (lane & 31), qpos = a.pos0 + row;
    const int last_pos = a.pos0 + min(a.T, rb * 128 + 128) - 1;     // last position any row of the block attends to
    const int n_tiles = (last_pos >> 6) + 1;
    const int wave_first = a.pos0 + row0, wave_last = a.pos0 + min(a.T, row0 + 32) - 1;
    const size_t unit = (size_t)2 * P * HD;
    const size_t page_stride = (size_t)a.n_slots * a.H * unit;              // elements per physical page
    const kvhalf_t *kv_head = a.kv + ((size_t)a.slot * a.H + h) * unit;     // this layer's and head's keys in physical page 0
    if (t <= (last_pos >> a.logP) && t < 128) pages[t] = a.page_table[t];
    __syncthreads();

    // a lane's part of a wave's load: row (of RPL), place in the row, and the chunks of a key row and of a value row that belong there
    const int lrow = RPL * wave + lane / CPR, place = lane % CPR;
    const int kc = place ^ (lrow & KM), vc = 2 * pf_v_piece<HD>(lrow, place >> 1) + (place & 1);
    const uint32_t koff = (lrow * HD + 8 * kc) * 2, voff = (lrow * HD + 8 * vc) * 2;
    const uint32_t lds_k = lds_address(&Ks[0][0]) + 1024 * wave, lds_v = lds_address(&Vs[0][0]) + 1024 * wave;
    auto load_tile = [&](int tile0, int b) {
        if (a.logP >= 6 && tile0 + 63 <= last_pos) {        // 64 rows of one page
            const kvhalf_t *src = kv_head + (size_t)__builtin_amdgcn_readfirstlane(pages[tile0 >> a.logP]) * page_stride + (size_t)(tile0 & (P - 1)) * HD;
#pragma unroll
            for (int i = 0; i < CH; i++) lds_load16(src + 4 * RPL * HD * i, koff, lds_k + 128 * HD * b + 4096 * i);
#pragma unroll
            for (int i = 0; i < CH; i++) lds_load16(src + (size_t)P * HD + 4 * RPL * HD * i, voff, lds_v + 128 * HD * b + 4096 * i);
        } else {                                            // (positions beyond the block's reach repeat the last one: finite, and masked below)
#pragma unroll
            for (int i = 0; i < CH; i++) {
                const int ap = min(tile0 + lrow + 4 * RPL * i, last_pos);
                const kvhalf_t *src = kv_head + (size_t)pages[ap >> a.logP] * page_stride + (ap & (P - 1)) * HD;
                lds_load16(src + 8 * kc, lds_k + 128 * HD * b + 4096 * i);
                lds_load16(src + (size_t)P * HD + 8 * vc, lds_v + 128 * HD * b + 4096 * i);
            }
        }
    };
    load_tile(0, 0);
    f16x8_t qhi[KS], qlo[KS];
    pf_attn_queries<HD>(a, h, row0, lane, qhi, qlo);
    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++) o[dt] = f32x16_zero();
    float m_run = -INFINITY, l_run = 0.f;       // running maximum of the row (same in its two lanes), this lane's share of the sum
    lds_loads_landed();
    __syncthreads();
    for (int kt = 0; kt < n_tiles; kt++) {
        const int tile0 = kt << 6, b = kt & 1;
        if (kt + 1 < n_tiles) load_tile(tile0 + 64, b ^ 1);     // no wave reads the other buffers any more: their tile was finished before the last barrier
        if (tile0 <= wave_last) {               // else nothing of this tile is visible to the wave's rows
            f32x16_t s[2] = {f32x16_zero(), f32x16_zero()};
            // a step's keys are read under the step before
            auto keys = [&](int ks, int i) {
                const int pos = 32 * i + (lane & 31);
                return __builtin_bit_cast(f16x8_t, *(const u32x4_t *)&Ks[b][pos * HD + 8 * ((2 * ks + (lane >> 5)) ^ (pos & KM))]);
            };
            f16x8_t kk[2][2] = {{keys(0, 0), keys(0, 1)}};
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                __builtin_amdgcn_sched_barrier(0);
                if (ks + 1 < KS) { kk[(ks + 1) & 1][0] = keys(ks + 1, 0); kk[(ks + 1) & 1][1] = keys(ks + 1, 1); }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2; i++) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kk[ks & 1][i], qhi[ks], s[i], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 2; i++) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kk[ks & 1][i], qlo[ks], s[i], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // causal mask (only a tile that reaches beyond the wave's first row needs it).  Every row sees position 0, so its maximum is
            // finite from the first tile on; rows beyond the pass are computed like the others (on the last row's queries) and dropped.
            if (tile0 + 63 > wave_first) {
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int r = 0; r < 16; r++)
                        s[i][r] = tile0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) <= qpos ? s[i][r] : -INFINITY;
            }
            f16x8_t p[4];
            pf_attn_softmax<2, DT>(s, p, m_run, l_run, o);
#pragma unroll
            for (int u = 0; u < 4; u++)
#pragma unroll
                for (int dt = 0; dt < DT; dt++)
                    o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pf_v_operand<HD>(Vs[b], u, dt, lane), p[u], o[dt], 0, 0, 0);
        }
        lds_loads_landed();
        __syncthreads();
    }
    // normalise and store: lane holds dimensions 32 dt + 8 (r / 4) + 4 (lane / 32) + r % 4 of its row
    const float l = pair_sum(l_run), inv = l > 0.f ? 1.f / l : 0.f;
    if (row < a.T) {
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
#pragma unroll
            for (int rr = 0; rr < 4; rr++) {
                const float v[4] = {o[dt][4 * rr] * inv, o[dt][4 * rr + 1] * inv, o[dt][4 * rr + 2] * inv, o[dt][4 * rr + 3] * inv};
                pf_attn_store(a, row, h * HD + 32 * dt + 8 * rr + 4 * (lane >> 5), v);
            }
    }
}

// Short passes, whose blocks of 128 rows would leave compute units idle: one workgroup per (head, 32 rows); its 4 waves take the tiles of 32
// positions in turn, keys straight from memory in operand order, values through a piece of LDS of their own, with no barrier before
// their sums are added.
template <int HD>
__global__ __launch_bounds__(256, 2) void pf_attn_short_kernel(const PfAttnArgs a)
{
    constexpr int KS = HD / 16, DT = HD / 32, NW = 4;
    constexpr int CPR = HD / 8, CH = 32 * CPR / 64;     // 16-byte chunks per row of values; per lane of a tile
    constexpr int NG = 4 * DT;                          // groups of 4 output registers of a lane
    __shared__ __align__(16) float part[NW][NG][64][4]; // a wave's values (32 x HD halves), then its sums
    __shared__ float mw[NW][32], lw[NW][32];
    __shared__ int pages[128];
    const int h = blockIdx.x, t = threadIdx.x;
    const int row0 = 32 * ((int)gridDim.y - 1 - (int)blockIdx.y);
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, q = lane & 31, g = lane >> 5;
    const int P = 1 << a.logP;
    const int row = row0 + q, qpos = a.pos0 + row;
    const int last_pos = a.pos0 + min(a.T, row0 + 32) - 1, n_tiles = (last_pos >> 5) + 1;
    const size_t unit = (size_t)2 * P * HD;
    const size_t page_stride = (size_t)a.n_slots * a.H * unit;
    const kvhalf_t *kv_head = a.kv + ((size_t)a.slot * a.H + h) * unit;
    if (t <= (last_pos >> a.logP) && t < 128) pages[t] = a.page_table[t];
    __syncthreads();
    uint16_t *vs = (uint16_t *)&part[wave][0][0][0];

    u32x4_t kreg[KS], vreg[CH];
    auto load_tile = [&](int tile0) {       // (positions beyond the block's reach repeat the last one: finite, and masked below)
        const int kp = min(tile0 + q, last_pos);
        const kvhalf_t *Kp = kv_head + (size_t)pages[kp >> a.logP] * page_stride + (kp & (P - 1)) * HD;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) kreg[ks] = *(const u32x4_t *)(Kp + 16 * ks + 8 * g);
#pragma unroll
        for (int i = 0; i < CH; i++) {
            const int c = lane + 64 * i, vp = min(tile0 + c / CPR, last_pos);
            vreg[i] = *(const u32x4_t *)(kv_head + (size_t)pages[vp >> a.logP] * page_stride + ((P + (vp & (P - 1))) * HD + 8 * (c % CPR)));
        }
    };
    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++) o[dt] = f32x16_zero();
    float m_run = -INFINITY, l_run = 0.f;
    if (wave < n_tiles) {
        load_tile(32 * wave);
        f16x8_t qhi[KS], qlo[KS];
        pf_attn_queries<HD>(a, h, row0, lane, qhi, qlo);
        for (int kt = wave; kt < n_tiles; kt += NW) {
            const int tile0 = 32 * kt;
            __builtin_amdgcn_wave_barrier();        // (a wave's accesses to LDS take effect in program order)
#pragma unroll
            for (int i = 0; i < CH; i++) {
                const int c = lane + 64 * i, pos = c / CPR, dq = c % CPR;
                *(u32x4_t *)&vs[pos * HD + 16 * pf_v_piece<HD>(pos, dq >> 1) + 8 * (dq & 1)] = vreg[i];
            }
            __builtin_amdgcn_wave_barrier();
            f32x16_t s[1] = {f32x16_zero()};
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                s[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, kreg[ks]), qhi[ks], s[0], 0, 0, 0);
                s[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, kreg[ks]), qlo[ks], s[0], 0, 0, 0);
            }
            if (kt + NW < n_tiles) load_tile(tile0 + 32 * NW);
            if (tile0 + 31 > a.pos0 + row0) {
#pragma unroll
                for (int r = 0; r < 16; r++) s[0][r] = tile0 + 8 * (r >> 2) + 4 * g + (r & 3) <= qpos ? s[0][r] : -INFINITY;
            }
            f16x8_t p[2];
            pf_attn_softmax<1, DT>(s, p, m_run, l_run, o);
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int dt = 0; dt < DT; dt++)
                    o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pf_v_operand<HD>(vs, u, dt, lane), p[u], o[dt], 0, 0, 0);
        }
    }
    // Merge: the waves' sums weighted by 2^(maximum of the wave - maximum of all), added in wave order; wave w finishes the w-th
    // quarter of the registers.
    l_run = pair_sum(l_run);
    if (g == 0) { mw[wave][q] = m_run; lw[wave][q] = l_run; }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < NG; j++)
        *(float4 *)part[wave][j][lane] = make_float4(o[j >> 2][4 * (j & 3)], o[j >> 2][4 * (j & 3) + 1], o[j >> 2][4 * (j & 3) + 2], o[j >> 2][4 * (j & 3) + 3]);
    __syncthreads();
    if (row >= a.T) return;
    const int nw = min(NW, n_tiles);
    float mx = -INFINITY, l = 0.f, wt[NW];
#pragma unroll
    for (int w = 0; w < NW; w++) mx = fmaxf(mx, mw[w][q]);      // finite: every row sees position 0
#pragma unroll
    for (int w = 0; w < NW; w++) {
        wt[w] = __builtin_amdgcn_exp2f(mw[w][q] - mx);
        l = fmaf(wt[w], lw[w][q], l);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int jj = 0; jj < NG / NW; jj++) {
        const int j = wave * (NG / NW) + jj;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; w++)
            if (w < nw) {
                const float4 y = *(const float4 *)part[w][j][lane];
                v[0] = fmaf(wt[w], y.x, v[0]); v[1] = fmaf(wt[w], y.y, v[1]); v[2] = fmaf(wt[w], y.z, v[2]); v[3] = fmaf(wt[w], y.w, v[3]);
            }
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] *= inv;
        pf_attn_store(a, row, h * HD + 32 * (j >> 2) + 8 * (j & 3) + 4 * g, v);
    }
}

// ---------------------------------------------------------------------------------------------
// Random numbers of sampling mode: Philox4x32-10 (Salmon et al., SC 2011), a counter-based generator,
// so that the number for (absolute token position, purpose) can be produced by whichever kernel
// needs it, with no state to carry and independent of the control flow that led there.
// Ten rounds on the counter words (c0, c1, c2, c3) under the key (k0, k1):
//   (c0, c1, c2, c3) <- (mulhi(B, c2) ^ c1 ^ k0, B * c2, mulhi(A, c0) ^ c3 ^ k1, A * c0),
// A = 0xD2511F53, B = 0xCD9E8D57, products mod 2^32; the key grows by (0x9E3779B9, 0xBB67AE85)
// between rounds.  Returns the first word of the block for counter (position, purpose, 0, 0).
__device__ __forceinline__ uint32_t philox_word(uint32_t k0, uint32_t k1, uint32_t position, uint32_t purpose)
{
    uint32_t a = position, b = purpose, c = 0u, d = 0u;
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint32_t ha = __umulhi(0xD2511F53u, a), la = 0xD2511F53u * a;
        const uint32_t hc = __umulhi(0xCD9E8D57u, c), lc = 0xCD9E8D57u * c;
        a = hc ^ b ^ (k0 + (uint32_t)r * 0x9E3779B9u);
        c = ha ^ d ^ (k1 + (uint32_t)r * 0xBB67AE85u);
        b = lc;
        d = la;
    }
    return a;
}
// uniform number in [0, 1) with 24 random bits
__device__ __forceinline__ float philox_uniform(uint32_t k0, uint32_t k1, uint32_t position, uint32_t purpose)
{
    return (float)(philox_word(k0, k1, position, purpose) >> 8) * (1.f / 16777216.f);
}

__global__ void philox_words_kernel(uint32_t k0, uint32_t k1, uint32_t pos0, uint32_t purpose, int n, uint32_t *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = philox_word(k0, k1, pos0 + (uint32_t)i, purpose);
}

// Where the uniform numbers of a launch's rows come from: the generator keyed by the seed, evaluated
// at the absolute position each row decides, or numbers the caller supplied (a test hook).
struct USrc {
    int from_seed;
    uint32_t k0, k1;
    int pos[KG_ROWS];
    float u0[KG_ROWS], u1[KG_ROWS];     // caller's numbers for the launch's first / second purpose
};
__device__ __forceinline__ float row_uniform(const USrc &s, int row, int purpose, int which)
{
    // constant indices only: the argument block stays in scalar registers
    float tv = 0.f;
    int pv = 0;
#pragma unroll
    for (int i = 0; i < KG_ROWS; i++)
        if (i == row) { tv = which ? s.u1[i] : s.u0[i]; pv = s.pos[i]; }
    return s.from_seed ? philox_uniform(s.k0, s.k1, (uint32_t)pv, (uint32_t)purpose) : tv;
}

// ---------------------------------------------------------------------------------------------
// Block-wide inverse-CDF draw (1024 threads): smallest index n with w(0) + .. + w(n) > u * total,
// walking ascending indices; weights are accumulated in double.  Returns -1 when total == 0.
// All threads must call it; all get the result.  The weight of index i is w(za[i], zb[i]) (zb may be
// null: its value is then 0).
// Up to 32768 indices every thread owns 32 consecutive ones: it fetches them with 16-byte loads,
// computes their weights once and keeps them in registers for the sum, the walk and the fallback;
// larger index sets are walked in chunks with the weights recomputed.
struct I8 { int v[KG_ROWS]; };

template <class F>
__device__ int block_inverse_cdf(const float *za, const float *zb, F w, int V, float u)
{
    __shared__ double wsum[16];
    __shared__ int found, lastpos;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const bool in_regs = V <= 32768 && (V & 3) == 0;
    const int chunk = in_regs ? 32 : (V + 1023) >> 10;
    const int i0 = min(V, t * chunk), i1 = min(V, i0 + chunk);
    float wv[32];
    double local = 0.0;
    if (in_regs) {
#pragma unroll
        for (int j = 0; j < 32; j += 4) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
            const bool in = i0 + j < i1;                       // V % 4 == 0: a group of four is all in or all out
            if (in) {
                a = *(const float4 *)(za + i0 + j);
                if (zb) b = *(const float4 *)(zb + i0 + j);
            }
            wv[j] = in ? w(a.x, b.x) : 0.f;
            wv[j + 1] = in ? w(a.y, b.y) : 0.f;
            wv[j + 2] = in ? w(a.z, b.z) : 0.f;
            wv[j + 3] = in ? w(a.w, b.w) : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 32; j++) local += (double)wv[j];
    } else {
        for (int i = i0; i < i1; i++) local += (double)w(za[i], zb ? zb[i] : 0.f);
    }
    double incl = local;                                   // inclusive scan inside the wave
    for (int o = 1; o < 64; o <<= 1) {
        double v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    if (t == 0) { found = -1; lastpos = -1; }
    __syncthreads();
    double base = 0.0, total = 0.0;
    for (int k = 0; k < 16; k++) {
        if (k < wave) base += wsum[k];
        total += wsum[k];
    }
    if (total <= 0.0) return -1;
    const double thr = (double)u * total;
    const double excl = base + incl - local;
    if (excl <= thr && excl + local > thr) {
        double acc = excl;
        if (in_regs) {
            int f = -1;
#pragma unroll
            for (int j = 0; j < 32; j++) {
                acc += (double)wv[j];
                if (f < 0 && acc > thr) f = i0 + j;
            }
            if (f >= 0) found = f;
        } else {
            for (int i = i0; i < i1; i++) {
                acc += (double)w(za[i], zb ? zb[i] : 0.f);
                if (acc > thr) { found = i; break; }
            }
        }
    }
    __syncthreads();
    if (found >= 0) return found;
    // u * total landed beyond the accumulated mass by rounding: last index with weight
    int lp = -1;
    if (in_regs) {
#pragma unroll
        for (int j = 0; j < 32; j++) if (wv[j] > 0.f) lp = i0 + j;
    } else {
        for (int i = i0; i < i1; i++) if (w(za[i], zb ? zb[i] : 0.f) > 0.f) lp = i;
    }
    if (lp >= 0) atomicMax(&lastpos, lp);
    __syncthreads();
    return lastpos;
}

// The LM head's statistics of a row's tiles (16 consecutive tokens each), tile i at hs[4 i] = (max of z / T, sum exp(z / T - max), index of
// the max), shared out over 1024 threads in ascending stretches.  Up to 8 tiles of a thread are kept in registers, all requested
// together (vocabularies of up to 131072 tokens); those of a longer stretch are read again each time.
struct TileStats {
    const float *hs;
    int i0, n;              // this thread's tiles
    float4 v[8];
    __device__ __forceinline__ TileStats(const float *hs_, int n_tiles)
    {
        hs = hs_;
        const int chunk = (n_tiles + 1023) >> 10, t = threadIdx.x;
        i0 = min(n_tiles, t * chunk);
        n = min(n_tiles, i0 + chunk) - i0;
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (k < chunk) v[k] = *(const float4 *)(hs + (size_t)min(i0 + k, n_tiles - 1) * 4);
    }
    template <class F> __device__ __forceinline__ void each(F f) const      // f(statistics, tile)
    {
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (k < n) f(v[k], i0 + k);
        for (int k = 8; k < n; k++) f(*(const float4 *)(hs + (size_t)(i0 + k) * 4), i0 + k);
    }
};
// weight of a tile under the row's maximum mx of z / T (none for one of -infinity, whose own sum is not a number)
__device__ __forceinline__ float tile_weight(const float4 &h, float mx) { return h.x == -INFINITY ? 0.f : h.y * __expf(h.x - mx); }

// Block-wide inverse-CDF draw from softmax(z / T) through the tile statistics (1024 threads): the tile that holds u * total is
// found from the tiles' weights, and only its 16 logits are looked at.  Walks ascending token indices;
// sums in double.  Returns -1 when the total is not positive.  All threads must call it; all get the result.
__device__ int tile_inverse_cdf(const TileStats &ts, const float *z, float inv_temp, float mx, float u)
{
    __shared__ double wsum[16];
    __shared__ int cand[16];
    __shared__ int found;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    double local = 0.0;
    ts.each([&](const float4 &h, int) { local += (double)tile_weight(h, mx); });
    double incl = local;                                   // inclusive scan inside the wave
    for (int o = 1; o < 64; o <<= 1) {
        double v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    if (t == 0) found = -1;
    __syncthreads();
    double base = 0.0, total = 0.0;
    for (int k = 0; k < 16; k++) {
        if (k < wave) base += wsum[k];
        total += wsum[k];
    }
    if (!(total > 0.0)) return -1;
    const double thr = (double)u * total;                  // u < 1: below the total
    const double excl = base + incl - local;
    // the stretch that holds the threshold: the last one that starts at or below it
    const unsigned long long starts_below = __ballot(ts.n > 0 && excl <= thr);
    if (lane == 0) cand[wave] = starts_below ? wave * 64 + 63 - __builtin_clzll(starts_below) : -1;
    __syncthreads();
    int owner = -1;
    for (int k = 0; k < 16; k++) owner = max(owner, cand[k]);
    if (t == owner) {
        double acc = excl, last = 0.0;
        int tile = -1;
        bool hit = false;
        ts.each([&](const float4 &h, int i) {
            const double wt = (double)tile_weight(h, mx);
            if (hit || !(wt > 0.0)) return;
            acc += last;                                   // pass the tile before: the threshold lies beyond it
            last = wt;
            tile = i;
            hit = acc + wt > thr;
        });
        // (a stretch whose sums fall short of the threshold by rounding ends at its last tile with weight)
        if (tile >= 0) {
            // inside the tile the 16 weights are recomputed; if their sum misses the tile's own by rounding,
            // the tile's last token with weight is the draw
            float zv[16];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float4 q = *(const float4 *)(z + tile * 16 + 4 * j);
                zv[4 * j] = q.x; zv[4 * j + 1] = q.y; zv[4 * j + 2] = q.z; zv[4 * j + 3] = q.w;
            }
            int f = -1, lastw = -1;
#pragma unroll
            for (int j = 0; j < 16; j++) {
                const float wj = __expf(zv[j] * inv_temp - mx);
                acc += (double)wj;
                if (wj > 0.f) lastw = tile * 16 + j;
                if (f < 0 && acc > thr) f = tile * 16 + j;
            }
            found = f >= 0 ? f : lastw;
        }
    }
    __syncthreads();
    return found;
}

// A result word for the host, which knows it by the launch number in its upper half (pinned memory; one 8-byte store, so the
// word is complete when its number is there).
__device__ __forceinline__ void post(unsigned long long *slot, unsigned seq, uint32_t v)
{
    __hip_atomic_store(slot, ((unsigned long long)seq << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// emb.table: row 0's token is looked up at once and becomes the first activation of the pass that follows, as pack_rows_kernel
// makes it from a token in device memory: 1 us more here at 4096 features, for a launch less (2.7 and 4.6 us) and the gap before it.
struct EmbedOut {
    const void *table;      // [V][d], bfloat16 or fp32; null: no lookup
    int bf, d;
    const float *gain;
    float *xout, *ssq;
    void *act;
};
// gain: this thread's features 4 t .. 4 t + 3 and those 4096 further on
template <bool BF>
__device__ __forceinline__ void embed_row(const EmbedOut &o, int tok, int V, const float4 (&gain)[2], float *sq)
{
    const int id = min(max(tok, 0), V - 1);
    float v[2][4];
#pragma unroll
    for (int j = 0; j < 2; j++) {               // d <= 8192
        const int n = 4 * threadIdx.x + 4096 * j;
        if (n >= o.d) continue;
        const size_t idx = (size_t)id * o.d + n;
        if (BF) {
            const uint2 q = *(const uint2 *)((const uint16_t *)o.table + idx);
            v[j][0] = __uint_as_float(q.x << 16); v[j][1] = __uint_as_float(q.x & 0xFFFF0000u);
            v[j][2] = __uint_as_float(q.y << 16); v[j][3] = __uint_as_float(q.y & 0xFFFF0000u);
        } else {
            const float4 q = *(const float4 *)((const float *)o.table + idx);
            v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
        }
    }
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int n = 4 * threadIdx.x + 4096 * j;
        if (n >= o.d) continue;
        *(float4 *)(o.xout + n) = make_float4(v[j][0], v[j][1], v[j][2], v[j][3]);
        const float g[4] = {gain[j].x, gain[j].y, gain[j].z, gain[j].w};
        if (BF) {                               // as store_act, four features at a time
            uint16_t hi[4], lo[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float x = rounded(v[j][i] * g[i]);
                hi[i] = f2bf(x);
                lo[i] = f2bf(x - bf2f(hi[i]));
            }
            uint16_t *p = (uint16_t *)o.act + (size_t)(n >> 5) * 512 + ((n >> 3) & 3) * 8 + (n & 7);
            *(uint2 *)p = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
            *(uint2 *)(p + 32) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
        } else {
            *(float4 *)((float *)o.act + n) = make_float4(v[j][0] * g[0], v[j][1] * g[1], v[j][2] * g[2], v[j][3] * g[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) sq[n + i + (n >> 4)] = v[j][i] * v[j][i];
    }
    __syncthreads();
    for (int rt = threadIdx.x; rt < o.d >> 4; rt += 1024) {
        float s = 0.f;
        for (int r = 0; r < 16; r++) s += sq[17 * rt + r];
        o.ssq[(size_t)rt * KG_ROWS] = s;
    }
}

// Final reduction of the per-tile LM-head statistics for one row per block: arg-max (lowest index
// among equal maxima) and top-1 probability of softmax(z / T) = 1 / sum exp((z - max) / T).
// mode 1 additionally draws the token from softmax(z / T) with the row's uniform number (of the
// given purpose: 0 a draft token, 2 a first / plain token).
// stat_out[row] = (max of z/T, sum exp(z/T - max)).
// host[row], host[KG_ROWS + row]: the result words with the row's token and the bits of its top-1 probability.
// One workgroup that waits: every load that does not depend on another is issued at the start, the statistics are read once, the
// maximum is found before any sum is taken (no rescaling on the way), and the last step over 16 waves is taken by 16 lanes.  us at
// 32000 tokens, statistics read twice, both reductions pairwise with the last step by one thread, the look-up feature by feature / here:
// seven verification rows 5.9 / 4.0, a draft with its look-up 8.4 / 5.0, with a draw 12.6 / 7.9; 1024 tokens 4.8 / 3.3.
__global__ __launch_bounds__(1024) void head_final_kernel(const float *hstat, int n_tiles, const float *logits,
                                                          int V, float inv_temp, int mode, USrc us, int purpose,
                                                          unsigned long long *host, unsigned seq, float *stat_out, EmbedOut emb)
{
    constexpr int NONE = 0x7FFFFFFF;
    __shared__ float bm[16], bs[16], sq[8192 + 512];      // d <= 8192; one float of padding per 16: embed_row's sums read without conflicts
    __shared__ int bi[16];
    const int m = blockIdx.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const TileStats ts(hstat + (size_t)m * n_tiles * 4, n_tiles);
    const bool look_up = emb.table && m == 0;
    float4 gain[2];
#pragma unroll
    for (int j = 0; j < 2; j++)
        if (look_up && 4 * t + 4096 * j < emb.d) gain[j] = *(const float4 *)(emb.gain + 4 * t + 4096 * j);
    const float u = mode != 0 ? row_uniform(us, m, purpose, 0) : 0.f;
    float best = -INFINITY;
    int idx = NONE;
    ts.each([&](const float4 &h, int) {
        if (h.x > best || (h.x == best && idx == NONE)) { best = h.x; idx = __float_as_int(h.z); }      // (a row of -infinity has a first token too)
    });
    // stretches, waves and lanes ascend, so the first of equal maxima has the lowest index
    const float wm = wave_max(best);
    const unsigned long long have = __ballot(best == wm && idx != NONE);
    const int wi = have ? __builtin_amdgcn_readlane(idx, __builtin_ctzll(have)) : NONE;
    if (lane == 0) { bm[wave] = wm; bi[wave] = wi; }
    __syncthreads();
    const float wv = bm[lane & 15], mx = row_max(wv);
    const unsigned have16 = (unsigned)__ballot(wv == mx && bi[lane & 15] != NONE) & 0xFFFFu;
    int tok = have16 ? bi[__builtin_ctz(have16)] : NONE;
    float part = 0.f;
    ts.each([&](const float4 &h, int) { part += tile_weight(h, mx); });
    part = wave_sum(part);
    if (lane == 0) bs[wave] = part;
    if (mode != 0) {
        const int drawn = tile_inverse_cdf(ts, logits + (size_t)m * V, inv_temp, mx, u);
        if (drawn >= 0) tok = drawn;
    } else {
        __syncthreads();
    }
    const float sum = row_sum(bs[lane & 15]);
    if (t == 0) {
        post(host + KG_ROWS + m, seq, __float_as_uint(1.f / sum));
        post(host + m, seq, (uint32_t)tok);
        stat_out[2 * m] = mx;
        stat_out[2 * m + 1] = sum;
    }
    if (!look_up) return;
    if (emb.bf) embed_row<true>(emb, tok, V, gain, sq);
    else embed_row<false>(emb, tok, V, gain, sq);
}

// Speculative-sampling acceptance of one round (Section 3: the first rejected draft discards the
// rest; the sampling distribution of the target is preserved).  Draft d_i ~ q_i is kept while
// u_acc[i] < min(1, p_i(d_i) / q_i(d_i)); the first rejected position is redrawn from
// normalize(max(0, p_i - q_i)); if all k are kept a bonus token is drawn from p_k.
// Row i decides the token at us.pos[i]; its acceptance number has purpose 1 (us.u0), its redraw /
// bonus number purpose 2 (us.u1).
// zt: target logits [k+1][V], zd: draft logits [k][V]; tstat/dstat: (max, sum exp) per row of z/T.
// host[0], host[1]: the result words with the number of accepted drafts and the redrawn / bonus token.
__global__ __launch_bounds__(1024) void accept_sample_kernel(const float *zt, const float *zd, const float *tstat,
                                                             const float *dstat, const float *hstat_t, int V, int k,
                                                             float inv_temp, I8 drafts, USrc us, unsigned long long *host, unsigned seq)
{
    __shared__ int n_acc;
    const int t = threadIdx.x;
    // the k acceptance tests are independent: lane n tests draft n, the first failure ends the run
    if (t < 64) {
        bool keep = true;
        if (t < k) {
            int dd = 0;
#pragma unroll
            for (int i = 0; i < KG_ROWS; i++)
                if (i == t) dd = drafts.v[i];
            const float pp = __expf(zt[(size_t)t * V + dd] * inv_temp - tstat[2 * t]) / tstat[2 * t + 1];
            const float qq = __expf(zd[(size_t)t * V + dd] * inv_temp - dstat[2 * t]) / dstat[2 * t + 1];
            float uv = 0.f;
#pragma unroll
            for (int i = 0; i < KG_ROWS; i++)
                if (i == t) uv = row_uniform(us, i, 1, 0);
            keep = uv < fminf(1.f, pp / qq);
        }
        const unsigned long long rejected = __ballot(!keep);
        if (t == 0) n_acc = rejected ? min(k, __builtin_ctzll(rejected)) : k;
    }
    __syncthreads();
    const int n = n_acc;
    const float *zp = zt + (size_t)n * V;
    const float pm = tstat[2 * n], ps = 1.f / tstat[2 * n + 1];
    int tok = -1;
    if (n < k) {
        const float *zq = zd + (size_t)n * V;
        const float qm = dstat[2 * n], qs = 1.f / dstat[2 * n + 1];
        tok = block_inverse_cdf(
            zp, zq, [&](float a, float b) { return fmaxf(0.f, __expf(a * inv_temp - pm) * ps - __expf(b * inv_temp - qm) * qs); }, V,
            row_uniform(us, n, 2, 1));
        __syncthreads();
    }
    // all drafts kept (or an empty residual): the bonus token from p_n, through the target head's tile statistics
    if (tok < 0) tok = tile_inverse_cdf(TileStats(hstat_t + (size_t)n * (V / 16) * 4, V / 16), zp, inv_temp, pm, row_uniform(us, n, 2, 1));
    if (t == 0) { post(host, seq, (uint32_t)n); post(host + 1, seq, (uint32_t)tok); }
}

// Streaming read of a buffer with no dependencies between the loads: the bandwidth that a weight
// stream could reach at best on this device (the measured ceiling the projections are compared
// with).  Persistent grid, 8 x 16-byte loads in flight per lane; out[block] keeps the loads alive.
__global__ __launch_bounds__(512, 2) void stream_read_kernel(const u32x4_t *__restrict__ src, size_t n16, unsigned *out)
{
    // a block takes 64 KB pieces; inside a piece every wave reads 8 consecutive KB (as a wave of a
    // projection reads consecutive 1 KB weight tiles)
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const size_t pieces = (n16 + 4095) >> 12;
    unsigned x = 0;
    for (size_t pc = blockIdx.x; pc < pieces; pc += gridDim.x) {
        const size_t base = (pc << 12) + (size_t)wave * 512 + lane;
        u32x4_t v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const size_t i = base + (size_t)u * 64;
            v[u] = i < n16 ? __builtin_nontemporal_load(src + i) : u32x4_t{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 8; u++) x ^= v[u][0] ^ v[u][3];
    }
    for (int o = 32; o >= 1; o >>= 1) x ^= __shfl_xor(x, o);
    if (lane == 0) atomicXor(&out[blockIdx.x], x);
}

// dst[i] = src[i] (a launch that a stream capture records like any other)
__global__ void copy_rows_kernel(const float *src, size_t n, float *dst)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// Copy cached k and v rows of one position, widened to float (test / debug access).
template <typename T>
__global__ void kv_read_kernel(const void *kv, const int *page_table, int slot, int n_slots, int H, int hd,
                               int P, int logP, int pos, float *k_out, float *v_out)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= H * hd) return;
    int h = i / hd, e = i % hd;
    const T *Kp = (const T *)kv + ((((size_t)page_table[pos >> logP] * n_slots + slot) * H + h) * 2) * (size_t)P * hd;
    int pl = pos & (P - 1);
    k_out[i] = kv_ld<T>(Kp + (size_t)pl * hd + e);
    v_out[i] = kv_ld<T>(Kp + (size_t)P * hd + (size_t)pl * hd + e);
}
