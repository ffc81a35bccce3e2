// How a long prompt pass (gemm_prefill2_body) and a training contraction (tr_gemm_body) are cut into workgroups: plain host arithmetic, no
// device code.
#pragma once
#include <cmath>
#include <cstddef>

// Projections cut along k write at most PF_SLICES partial sums per output, PF_PART_ROWS rows of them in all.
constexpr int PF_SLICES = 8, PF_PART_ROWS = 4096;

// The kernel's variants: weight tiles and pairs of 8-row blocks of a workgroup, and microseconds per k-step of a workgroup where
// all compute units have one (s with 8 pairs; a share f of it does not depend on the pairs: 0.29 us with 5 pairs and 0.41 with 8 at 8
// tiles, 0.39 / 0.54 at 12, 0.47 / 0.68 at 16, 1.09 / 1.69 at 32).
#define PF2_SIZES(V, t, s, f) V(t, 5, s, f) V(t, 6, s, f) V(t, 7, s, f) V(t, 8, s, f)
#define PF2_VARIANTS(V) \
    V(6, 8, 0.38, 0.2) PF2_SIZES(V, 8, 0.46, 0.216) PF2_SIZES(V, 12, 0.63, 0.152) PF2_SIZES(V, 16, 0.775, 0.149) PF2_SIZES(V, 32, 1.465, 0.1)

struct Pf2Variant { int ntw, pairs; double step_us; };
#define PF2_V(t, p, s, f) {t, p, s * (f + (1.0 - f) * p / 8)},
const Pf2Variant pf2_variants[] = {PF2_VARIANTS(PF2_V)};
#undef PF2_V
constexpr int PF2_N = (int)(sizeof(pf2_variants) / sizeof(pf2_variants[0]));

// Which variant, in how many slices along k (`split` allowed: EPI_RESID).  A workgroup fills a compute unit, so a
// launch takes whole rounds of them; a partly filled last round runs at a higher clock (0.75 of a round when nearly
// empty).  Partial sums are written at 5 TB/s and added by pf_reduce_rows_kernel (4 us + what it moves at 6 TB/s, against
// 5 us for the scales of rows that are finished in place).  The model is within a tenth of the measured launches (us,
// real passes): 7B shape, 256 rows: q,k,v 6 tiles 54, 8 tiles 59, 12 tiles 71; gate+up 12 tiles 81, 16 tiles 89; down_proj
// 16 tiles in 8 slices 50, 8 tiles in 4 slices 47, 8 tiles uncut 111; 1024 rows: gate+up 16 tiles 288, 12 tiles 313, 32
// tiles 359; down_proj 16 tiles in 2 slices 138, 8 tiles uncut 163; 4096 rows: q,k,v 32 tiles 607, 16 tiles 660;
// gate+up 16 tiles 1133, 32 tiles 1152.  Passes that long run at the card's power limit, where the tile that moves
// fewer bytes per multiplication also leaves the other launches a higher clock: 32 tiles are entered 3 % cheaper than
// they measure alone (4096 rows, whole pass: 94.5 ms with 32 tiles for gate+up, 96.9 ms with 16; 3000 rows, where 32
// tiles need a fifth round for the last 8 workgroups: 76.4 against 74.6 ms).
//   Groups of 80, 96 or 112 rows where they fit the pass's rows or the rounds better than groups of 128: rows multiplied for nothing
// cost as much as the others, in time and in power (these launches run at 1.6 .. 1.9 GHz on random data, at 2.4 GHz on zeros).  us,
// 128 rows at their best / the group picked: 7B, 300 rows: q,k,v 78 / 57 (12 tiles, 80 rows), gate+up 156 / 132 (12, 80), down_proj 60 / 51
// (16, 80, 4 slices); 400 rows: 87 / 68, 194 / 151, 71 / 62; 777 rows: q,k,v 184 / 144 (32, 80); 13B, 777 rows: 275 / 245 (32, 112),
// gate+up 443 / 401 (16, 112), o_proj 92 / 79 (12, 96).  They have to be 4 % ahead: nearer than that the fit does not rank them
// (7B, 512 rows, whole pass: 2.69 ms with 128 rows, 2.75 where it took 32 tiles x 112 rows for gate+up as 2 % ahead).
//   Workgroups go to the 8 XCDs in turn and pf_work deals a slice's out to them in equal shares, so a cut launch fills whole eighths: 36
// workgroups in 7 slices are 5 x 7 = 35 on some XCDs of 32 compute units, a second round for all, though 252 would fit the device
// (d_model 3072, 240 rows, down_proj: 48 us; 5 slices of 12 tiles 31.  700 rows 113 / 68; 13B, 640 rows 200 / 147, 384 rows, o_proj 76 / 48).
//   Picked against the best of all variants and slices (each timed in place, ten widths of d_model 1024 .. 8192, 36 passes of 104 ..
// 4096 rows): q,k,v 0.2 % longer on average, at most 5; o_proj 0.5 and 11; gate+up 0.7 and 11 (d_model 8192); down_proj 1.5 and 31 (d_model
// 1024, 4096 rows: 62 us where 16 tiles x 80 rows take 47; all other widths at most 8).  Without groups of fewer than 128 rows: 6 .. 9 % longer.
struct Pf2Plan { int variant, slices; };
inline Pf2Plan pf2_plan(int n_cus, int NT, int KS, int T, bool split)
{
    const int pairs = (T + 15) / 16;
    Pf2Plan best = {0, 1};
    double best_cost = -1.0;
    for (int v = 0; v < PF2_N; v++)
        for (int S = 1; S <= (split ? PF_SLICES : 1); S++) {
            if (S > 1 && (S * T > PF_PART_ROWS || KS < 8 * S || pf2_variants[v].ntw == 32)) break;
            const Pf2Variant &pv = pf2_variants[v];
            const int gx = (pairs + pv.pairs - 1) / pv.pairs;
            const int slice = gx * ((NT + pv.ntw - 1) / pv.ntw);
            const double wgs = S > 1 ? (double)((slice + 7) / 8 * 8) * S : slice, whole = std::floor(wgs / n_cus), rest = wgs / n_cus - whole;
            const double rounds = whole + (rest > 0 ? 0.75 + 0.25 * rest : 0.0), bytes = (double)T * NT * 64;
            const double step = pv.step_us * (pv.pairs < 8 ? 1.04 : 1.0);
            const double cost = rounds * ((double)KS / S * step + 4.0) + (S > 1 ? S * bytes / 5e6 + (S + 3) * bytes / 6e6 + 4.0 : split ? 5.0 : 0.0);
            if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = {v, S}; }
        }
    return best;
}

constexpr int TRG_K = 32, TRG_M = 128, TRG_N = 256;     // k per step and tile of C of tr_gemm_kernel
constexpr int TR_SPLIT_MAX = 8;

// Are the tiles of one column of C (of gn) dealt to one XCD, column c to XCD c % 8?  (Its L2 keeps that part of B; not where columns would
// leave XCDs idle.)
inline bool trg_by_column(int gn) { return gn % 8 == 0 || gn >= 16; }

// Into how many slices of `chunk` numbers k a training contraction of M x N x K is cut: whole rounds of workgroups of one tile each (6 us
// apart from their steps of 32 k: 1.9 us a step with all compute units at work, 1.4 against bf16 tiles), counted on the XCD with the most columns
// (of 20 some have three and some two), partial sums written and added at 4.5 TB/s by a launch of 4 us.  So few tiles are cut to fill the
// device, and a launch whose last round is half empty to halve the rounds (1000 x 12288 x 4096, 384 tiles on 256 compute units: 690 us -> 554 and 35
// for the sums).  No slice is empty.  (700 x 5120 x 15360: 2 slices are 240 tiles, but 36 on an XCD of 32 compute units, two rounds, 1067 us; 4 are
// 72, three rounds of half the steps, 842; 7 are 126, four rounds, 715 and 27 for the sums.)
struct TrSlices { int slices, chunk; };
inline TrSlices tr_slices(int n_cus, int M, int N, int K, bool tiles16, size_t part_floats)
{
    const int gm = (M + TRG_M - 1) / TRG_M, gn = (N + TRG_N - 1) / TRG_N;
    const int tiles = trg_by_column(gn) ? gm * ((gn + 7) / 8) : gm * gn, cus = trg_by_column(gn) ? n_cus / 8 : n_cus;
    TrSlices best = {1, 0};
    double best_us = -1.0;
    for (int S = 1; S <= TR_SPLIT_MAX; S++) {
        if (S > 1 && (K / S < 128 || (size_t)S * M * N > part_floats)) break;
        const int chunk = ((K + S - 1) / S + TRG_K - 1) / TRG_K * TRG_K;
        if (S > 1 && (S - 1) * chunk >= K) continue;
        const int rounds = (tiles * S + cus - 1) / cus;
        const double us = rounds * (chunk / TRG_K * (tiles16 ? 1.4 : 1.9) + 6.0) + (S > 1 ? 4.0 + (S + 1) * (double)M * N * 4 / 4.5e6 : 0.0);
        if (best_us < 0 || us < best_us) { best_us = us; best = {S, chunk}; }
    }
    return best;
}
