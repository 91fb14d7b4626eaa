// Host-side launchers of the libtm kernels (all asynchronous on a stream).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdlib>

#include "tm_types.h"

namespace tmk {

// integer tuning knob from the environment (read once by its callers)
inline int env_knob(const char *name, int dflt)
{
    const char *e = getenv(name);
    return e ? atoi(e) : dflt;
}

// Chunk of the timeslice walk: cy rows (y) x cz planes (z) of full x rows with
// cy | Ly, cz | Lz, one site per thread; the block has whole waves, the lanes
// beyond the last site idle.  busy: the share of lanes with a site.  tiles:
// reduction tiles (one per wave) of a half field, 0 if no chunk fits (a row
// longer than a block) or the walk is switched off (TM_LDS_WALK=0).
constexpr int WALK_MAX = 256;  // threads per block
struct WalkPlan {
    int cy = 0, cz = 0, threads = 0, chunks = 0, tiles = 0;
    double busy = 0.0;
};
// Waves of the walk on a CU: its launch bounds allow 2 (FP64), 3 (FP32) and 4 per
// SIMD, and the LDS of a block, which is that of 256 sites, 3 blocks in FP64 and 6
// otherwise.
inline int walk_blocks_per_cu(int sp, int waves_per_block, int waves_per_simd)
{
    return std::min(sp == P64 ? 3 : 6, std::max(1, 4 * waves_per_simd / waves_per_block));
}
// The shape with the least modelled time per site, among equals the largest,
// then the one with more rows:
// - 1 + 0.09 per halo neighbour (2/cy + 2/cz, no term for a dimension the chunk
//   spans): the measured slope (FP32, 12 right-hand sides, 32^3x64: 840 us at 1.0
//   halo neighbours per site, 876 us at 1.5);
// - 0.3 of a 128-byte line (8 sites) per run of sites that are consecutive in
//   memory, unless runs are whole lines; 0.1 in half precision, which is bound
//   by issue rather than by traffic;
// - over the share of busy lanes: idle ones cost their issue slots;
// - over the share of 6 (FP64) or 8 waves that fit a CU: a block of one wave has
//   the LDS of 256 sites too.
// All shapes were timed on 38 lattices (12 right-hand sides, Mhat): this choice
// is within 1.4% (FP64), 1.5% (FP32) and 0.9% (FP16) of the best on average, 13%
// at worst; by halo and busy lanes alone, 3.6, 2.9 and 2.8%, 51% at worst.
// FP64 / FP32 / FP16: 2 x 14 -> 14 x 2 at 14^3x28 179 / 79 / 69 -> 148 / 73 / 66 us, 1 x 13
// -> 13 x 1 at 26^4 1413 / 668 / 401 -> 1093 / 507 / 346 us, 6 x 2 in one wave -> 15 x 2
// in three at 10x30x26x14 342 / 119 / 128 -> 255 / 103 / 94 us.
// It depends on lattice and precision alone, so a slot's reduction tiles are the
// same in every batch.
inline WalkPlan walk_plan(const Geom &g, int sp)
{
    static const bool on = env_knob("TM_LDS_WALK", 1) != 0;
    WalkPlan p;
    if (!on) return p;
    const bool half = sp == P16 || sp == PBF;
    double best = 1e30;
    int sites = 0;
    for (int y = 1; y <= g.L[1]; y++) {
        if (g.L[1] % y) continue;
        for (int z = 1; z <= g.L[2]; z++) {
            const int cs = y * z * g.lxh;
            if (cs > WALK_MAX) break;
            if (g.L[2] % z) continue;
            const int threads = (cs + 63) & ~63;
            const double halo = (y < g.L[1] ? 2.0 / y : 0.0) + (z < g.L[2] ? 2.0 / z : 0.0);
            const int wpb = threads / 64, fit = wpb * walk_blocks_per_cu(sp, wpb, sp == P64 ? 2 : sp == P32 ? 3 : 4);
            const int run = g.lxh * y * (y == g.L[1] ? z : 1);
            const double lines = run % 8 ? (half ? 0.1 : 0.3) * 8 / run : 0.0, full = sp == P64 ? 6 : 8;
            const double cost = (1.0 + 0.09 * halo + lines) * threads / cs * std::max(1.0, full / fit);
            if (cost < best - 1e-9 || (cost < best + 1e-9 && cs >= sites)) {
                best = cost;
                sites = cs;
                p.cy = y;
                p.cz = z;
                p.threads = threads;
            }
        }
    }
    if (!sites) return p;
    p.chunks = (g.L[1] / p.cy) * (g.L[2] / p.cz);
    p.tiles = p.chunks * (p.threads / 64) * g.L[3];
    p.busy = (double)sites / p.threads;
    return p;
}

// Lattices that the register kernel, which has no idle lanes, serves instead: few
// busy lanes, and too many tiles for one wave per neighbour direction.  Mhat, 12
// right-hand sides, register kernel / walk: FP16, 0.53 busy (34^3x8), 245 / 368 us;
// 0.69 (66x34x16^2) 465 / 503; 0.72 (46^3x8) 634 / 757; 0.80 (102x22^2x8) 326 / 301.
// FP64, 0.53 busy, 903 / 1025; 0.59 (38^3x8) 1280 / 1300, but one right-hand side
// 134 / 112.  FP32, 0.53 busy, 457 / 411.
inline bool register_lattice(const WalkPlan &p, int sp)
{
    return !p.tiles || (p.tiles > 128 && p.busy < (sp == P64 ? 0.55 : sp == P32 ? 0.0 : 0.75));
}

// Timeslices walked per block, a divisor of Lt up to 8 (TM_LDS_TWALK), for n
// right-hand sides and parities, waves of the kernel per SIMD.  A block that
// walks tw timeslices takes tw steps and a shorter one that stages the first
// two (0.3 of a step).  The busiest of the 256 CUs runs its blocks in rounds of
// as many as fit; a round takes one step's latency per step, or longer
// where more waves are resident than it takes to keep the SIMDs issuing (FP64 6,
// FP32 8, half 16 per CU).  Lengths 1 to 8 were timed on 22 lattices from 6^3x12
// to 46^3x8 with 1, 3 and 12 right-hand sides: this rule's choice is within 0.9%
// (FP64), 0.8% (FP32) and 1.3% (FP16) of the best on average, 12, 7 and 16% at
// worst; with a whole step for the first two timeslices and rounds that all
// cost the same, 2.7, 1.4 and 3.0%, 36, 10 and 30% at worst (three FP16
// right-hand sides at 46^3x8: 2 timeslices 186 us, 8 of them 241 us).
// beside: the kernels of another batch run at the same time, so latency hides
// behind them and the work counts: FP64 walks then pay a whole step for the
// first two timeslices and the same for every round (12 FP64 solves beside four
// mixed ones at 16^3x32, truncated-solver estimate: 8 timeslices 52.6 ms, 2 of
// them 53.7; alone 15.9 and 15.1).  FP32 and half precision gained nothing by it.
// The outputs have the same bits.
inline int walk_length(const Geom &g, const WalkPlan &p, int n, int sp, int waves, bool beside)
{
    static const int most = std::max(1, env_knob("TM_LDS_TWALK", 8));
    const int wpb = p.threads / 64, fit = walk_blocks_per_cu(sp, wpb, waves);
    const double sat = sp == P64 ? 6 : sp == P32 ? 8 : 16;
    const int exact = sp == P16 || sp == PBF ? 4 : 8;  // rounds beyond which the blocks of a CU even out
    const bool work = beside && sp == P64;
    auto round = [&](double blocks) { return work ? 1.0 : std::max(1.0, blocks * wpb / sat); };
    double best = 1e30;
    int len = 1;
    for (int tw = std::min(most, g.L[3]); tw >= 1; tw--) {
        if (g.L[3] % tw) continue;
        const long blocks = (long)p.chunks * (g.L[3] / tw) * n, q = (blocks + 255) / 256;
        const double rounds = q > (long)exact * fit ? round(fit) * blocks / 256 / fit
                                                    : q / fit * round(fit) + (q % fit ? round(q % fit) : 0.0);
        const double cost = rounds * (tw + (work ? 1.0 : 0.3));
        if (cost < best - 1e-9) {
            best = cost;
            len = tw;
        }
    }
    return len;
}

// Order of the eight neighbours in half precision: a lattice with a chunk of
// whole waves on aligned 64-site tiles adds the backward t neighbour first and
// the forward one last, every other lattice both t neighbours last, as the
// register kernel does.  The order shows in the low bits of a half-precision
// spinor (4e-4 of a truncated FP16 solve), so it goes by the lattice alone.
inline bool both_t_last(const Geom &g)
{
    for (int y = 1; y <= g.L[1]; y++)
        for (int z = 1; g.L[1] % y == 0 && z <= g.L[2] && y * z * g.lxh <= WALK_MAX; z++) {
            const int cs = y * z * g.lxh;
            if (g.L[2] % z == 0 && cs % 64 == 0 && (y == g.L[1] || (y * g.lxh) % 64 == 0)) return false;
        }
    return true;
}

// Dslash with epilogue; sp = storage precision of in/in2/out/p and of x, r
// in the CG update (links of the same precision).  Returns -1 on an
// unsupported combination.
int launch_dslash(int sp, bool dag, int epi, bool in2, const DslashArgs &A, hipStream_t s);
// plain Dslash on full fields (A.in, A.in2, A.out), both output parities in
// one launch where the timeslice walk serves the lattice, else in two
int launch_dslash_full(int sp, bool dag, bool in2, DslashArgs A, hipStream_t s);
// the last preparation Dslash of a noise run with EPI_START: v = Mhat^dag bhat
// (A.in = A^-dag D'_oe bhat, A.in2 = bhat, both in precision sp: P32, or the
// half precision po itself) written as r (A.r), p (A.out) and x = 0 (A.x) in
// half precision po (P16 or PBF), with |v|^2 partials; -1 when no
// timeslice-walk chunk fits the lattice or the pair is not built (nothing
// launched)
int launch_dslash_start(int sp, int po, const DslashArgs &A, hipStream_t s);
// plain-epilogue Dslash with Z4-code inputs, uniform (kappa, a):
//   src 3: hop input A^-1 eta (parity 1 - out_par) and site input eta (prep:
//          bhat = eta + k D A^-1 eta); output in any storage precision
//   src 2: hop input a field, site input eta (reconstruction: A^-1 (eta + k D s)); P64 or P32
int launch_dslash_codes(int sp, int src, const DslashArgs &A, hipStream_t s);

// ---- CG scalars (one block per slot, fixed summation order) ----
void launch_cg_alpha(SlotState *st, const double *partial, int nslot, int nblk, hipStream_t s);
void launch_cg_beta(SlotState *st, const double *partial, int nslot, int nblk, hipStream_t s);
// end of a CG iteration: x += alpha p for slots whose iteration took a step
// (skipped when x is null: after reliable updates), then p = r + beta p for
// running slots (sp = p precision, xr = x and r precision)
void launch_p_update(int sp, int xr, const Geom &g, char *p, size_t p_slot, const char *r, size_t r_slot, char *x,
                     size_t x_slot, SlotState *st, int nslot, int swz, hipStream_t s);
// the same update with per-slot coefficients given by value (every slot
// steps x if x is not null and updates p); fields of one precision sp,
// slot i at base + i * slot_bytes
struct UpdateCoefs {
    double alpha[MAX_SLOTS], beta[MAX_SLOTS];
};
void launch_p_update_coefs(int sp, const Geom &g, char *p, const char *r, char *x, size_t slot_bytes,
                           const UpdateCoefs &c, int nslot, int swz, hipStream_t s);
// start n consecutive slots: rr0 = sum of the slot's nblk partials, status
// RUNNING (or CONVERGED if rr0 == 0); parameters per slot
struct SlotStartParams {
    double kappa[MAX_SLOTS], a[MAX_SLOTS], tol2[MAX_SLOTS], delta2[MAX_SLOTS];
    int max_iter[MAX_SLOTS];
    int mixed;
};
void launch_slot_start(SlotState *st, const double *partial, int nblk, const SlotStartParams &P, int n,
                       hipStream_t s);
// after FP64 reliable updates of n consecutive slots: rr_true = sum(partial);
// decide convergence, set beta
void launch_reliable_finish(SlotState *st, const double *partial, int nblk, int n, hipStream_t s);
// out[k] = sum(partial[k*nblk .. (k+1)*nblk)) for k < n (fixed order)
void launch_reduce(const double *partial, int nblk, int n, double *out, hipStream_t s);

// ---- site-local vector kernels on nslot consecutive half fields ----
void launch_convert(int pin, int pout, const Geom &g, const char *in, size_t in_slot, char *out, size_t out_slot,
                    int nslot, hipStream_t s);
void launch_zero(int p, const Geom &g, char *f, size_t slot, int nslot, hipStream_t s);
// r = p = in (rounded to pout), x = 0 for nslot slots; r, p and x share the pitch out_slot; pin P32 or P64
void launch_cg_start(int pin, int pout, const Geom &g, const char *in, size_t in_slot, char *r, char *p, char *x,
                     size_t out_slot, int nslot, hipStream_t s);
// x64 += x32; x32 = 0 (if x32_zero), n consecutive slots with strides s64, s32
void launch_accum_x(const Geom &g, char *x64, size_t s64, const char *x32_in, char *x32_zero, size_t s32, int n,
                    hipStream_t s);
// |f|^2 partials (ntile_of(g, P64) per field) of n FP64 half fields, pitch bytes apart
void launch_norm_partial(const Geom &g, const char *f, size_t pitch, int n, double *partial, hipStream_t s);

// ---- noise ----
// Z4 codes of both parities: codes[par*vh + cb]
void launch_z4_codes(const Geom &g, uint64_t seed, uint64_t src, uint32_t *codes, hipStream_t s);
// the same for n sources (n <= MAX_SLOTS) into codes + i * 2 * vh; source i
// is zero outside the timeslices t = tph[i] mod tmod[i] when tmod[i] > 0
struct Z4Sources {
    uint64_t seed[MAX_SLOTS], src[MAX_SLOTS];
    int tmod[MAX_SLOTS], tph[MAX_SLOTS];
};
void launch_z4_codes(const Geom &g, const Z4Sources &Z, int n, uint32_t *codes, hipStream_t s);
// eta of one parity as an FP64 half field (times A^-1 when ainv != 0)
void launch_z4_field(const Geom &g, const uint32_t *codes_par, int ainv, double a, char *out, hipStream_t s);
// canonical FP64 layout [V][4][3][2]
void launch_z4_canonical(const Geom &g, uint64_t seed, uint64_t src, double *out, hipStream_t s);

// ---- contractions ----
int contract_nchunk(const Geom &g);
// spin matrices of one source into raw_out [9][T][16][2]: s and links in FP64
// or FP32 (sps; gauge must be that precision's link array), accumulation FP64
void launch_contract(int sps, const Geom &g, const void *gauge, const char *s_even, const char *s_odd,
                     const uint32_t *codes, double *cpart, double *raw_out, hipStream_t s);
// n sources at once (n <= MAX_SLOTS): source i has s_even + i * s_stride,
// s_odd + i * s_stride, codes + i * 2 * vh, partials cpart + i * contract_part_doubles
// and output raw_out[i]
struct RawOuts {
    double *p[MAX_SLOTS];
};
size_t contract_part_doubles(const Geom &g);
void launch_contract(int sps, const Geom &g, const void *gauge, const char *s_even, const char *s_odd,
                     size_t s_stride, const uint32_t *codes, double *cpart, const RawOuts &raw, int n, hipStream_t s);
// the same with a field as the left vector (the one-end trick): left fields
// l_even/l_odd + i * l_stride, right fields s_even/s_odd + i * s_stride, all
// in precision sps; raw = (sr + i si) * the spin-matrix sums
void launch_contract_lr(int sps, const Geom &g, const void *gauge, const char *s_even, const char *s_odd,
                        size_t s_stride, const char *l_even, const char *l_odd, size_t l_stride, double *cpart,
                        const RawOuts &raw, int n, double sr, double si, hipStream_t s, bool local_only = false);
// local spin matrices only (kind 0 of raw[i]; other kinds untouched) of n
// sources with Z4-code left vectors, as launch_contract
void launch_contract_local(int sps, const Geom &g, const char *s_even, const char *s_odd, size_t s_stride,
                           const uint32_t *codes, double *cpart, const RawOuts &raw, int n, hipStream_t s);
// exact part of the hopping parameter expansion as local spin matrices
// raw[0][T][16][2] (kinds 1..8 untouched); even extents >= 4
void launch_hpe_exact(const Geom &g, double kappa, double a, double *raw, hipStream_t s);
// raw [n][9][T][16][2] -> ops [n][90][T][2]; gtab: [16][4] (col | phase << 2)
void launch_project(int n, int lt, const double *raw, double *ops, const int *gtab_host, hipStream_t s);
// TSM combination over per-source ops; est += ops_add when given; entries
// (op, t) with valid[op * T + t] == 0 are NaN (estimate and variances)
void launch_tsm_combine(int n_hp, int n_lp, int lt, const double *ops_hp, const double *ops_lp_corr,
                        const double *ops_lp_bulk, double *est, double *var_re, double *var_im, hipStream_t s,
                        const double *ops_add = nullptr, const unsigned char *valid = nullptr);
// out[i] = sum_k in[i * nph + k] in order k = 0..nph-1, i < n, per doubles each
void launch_sum_phases(const double *in, double *out, int n, int nph, size_t per, hipStream_t s);

// ---- layout ----
// canonical FP64 gauge (device) -> per-precision link arrays
void launch_gauge_pack(int p, const Geom &g, const double *canon, void *out, hipStream_t s);
// canonical full-lattice spinors <-> layout (full field = even half, then odd half)
void launch_field_import(int p, const Geom &g, int nrhs, const double *canon, char *field, hipStream_t s);
void launch_field_export(int p, const Geom &g, int nrhs, const char *field, double *canon, hipStream_t s);

// n consecutive canonical FP64 sources into FP64 halves even + i * pitch and
// odd + i * pitch (the odd half times A^-1 with ainv)
void launch_eta_import(const Geom &g, int n, const double *canon, char *even, char *odd, size_t pitch, bool ainv,
                       double a, hipStream_t s);
// n FP64 fields from halves with pitches of their own to consecutive canonical ones
void launch_halves_export(const Geom &g, int n, const char *even, size_t even_pitch, const char *odd, size_t odd_pitch,
                          double *canon, hipStream_t s);

// streaming copy probe
void launch_stream_copy(const void *src, void *dst, size_t bytes, hipStream_t s);

// gamma table for the projection: [16][4] entries (column | phase << 2),
// phase 0..3 = 1, i, -1, -i; built from the four basis matrices.
const int *gamma_table();

__host__ __device__ inline size_t half_bytes(int p, const Geom &g)
{
    return (size_t)g.vh * (p == P64 ? 192 : p == P32 ? 96 : 52);
}
inline size_t link_array_bytes(int p, const Geom &g)
{
    return (size_t)2 * 4 * g.vh * (p == P64 ? 96 : p == P32 ? 48 : HALF_LINK_BYTES);
}
__host__ __device__ inline int nblk_of(const Geom &g) { return (g.vh + BLOCK - 1) / BLOCK; }
// per-slot partial sums: one per wave of the timeslice walk, or per 64-site
// tile of the register kernel
inline int ntile_of(const Geom &g, int sp)
{
    const WalkPlan p = walk_plan(g, sp);
    return register_lattice(p, sp) ? (g.vh + TILE - 1) / TILE : p.tiles;
}
// the largest count of any precision
inline int ntile_most(const Geom &g)
{
    int n = 0;
    for (int sp : {P64, P32, P16, PBF}) n = std::max(n, ntile_of(g, sp));
    return n;
}

}  // namespace tmk
