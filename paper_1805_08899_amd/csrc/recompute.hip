// B3: the fused recomputation kernel.  For every valid (b, i, j, h) it
// re-evaluates t = tanh(Qp[b,i,h] + Kp[b,j,h]) (Section 3.4: redo the cheap
// forward nodes when the backward pass starts; Section 6.1: the nodes on the
// recomputation path fused into one kernel) and accumulates
//     dQp[b,i,h] = v[h] sum_j dS[b,i,j] (1 - t^2)        (Section 3.2: tanh' = 1 - tanh^2)
//     dKp[b,j,h] = v[h] sum_i dS[b,i,j] (1 - t^2)
//     dv[h]     += sum_{i,j} dS[b,i,j] t                  (Eq. 2: needs the tanh map as the input of the v projection)
// without the B x Tq x Tk x H map ever existing in memory.
//
// A block owns one sample and one slice of HW = 64, 32 or 16 columns of h; lanes run along h, and with a slice narrower
// than the wave the 64 / HW lane groups own different query rows.  dS[b,i,j] is uniform over a lane group and dQp, dKp, dv
// are plain per-lane sums.
// With r = 1 / (exp(2(q+k)) + 1):  t = 1 - 2r  and  1 - t^2 = 4 r (1 - r).
// Wave w owns query rows; all waves walk the keys together in tiles of RJ.
// The key tile (exponentials) and the dS tile are fetched one tile ahead and
// shared through LDS.  Per tile a wave adds its partial column sums into LDS, and after the
// barrier wave jj sums key jj of the tile over the waves in fixed order and
// owns that element of dKp for the whole kernel (first block of rows stores,
// later ones add), so no atomics are needed and results are reproducible.
//
// STASH reads t from a stored map instead (the keep-the-feature-map baseline,
// comparison only).
//
// Samples of many query rows take the form of recompute_rows.hip on grids of more than half a round of blocks (recompute_takes_rows).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace echo {

constexpr int RC_RI = 8;      // query rows per wave and pass
constexpr int RC_RJ = 8;      // keys per tile (== kDsPad)
constexpr int RC_W = 8;       // waves per block (== RC_RJ: wave jj finishes key jj of a tile)
constexpr int RC_THREADS = 64 * RC_W;
constexpr int RC_ROUND = 512; // blocks that run at a time: two on every compute unit
static_assert(RC_RJ == kDsPad, "dS rows are padded to the key tile");
static_assert(RC_W == RC_RJ, "one finishing wave per key of a tile");
static_assert(RC_W == 8, "rows are dealt to eight waves");

enum RcMode { RC_FACTOR = 0, RC_EXACT = 1, RC_STASH = 2 };


// One RI x RJ register tile.  NI = number of live rows (compile time so the
// accumulators stay in registers and the NI*RJ chains interleave freely).
//   RC_FACTOR: fq = exp(2q), fk = exp(2k)        r = 1 / (fq fk + 1)
//   RC_EXACT : fq = 2 log2e q, fk = 2 log2e k    r = 1 / (exp2(fq + fk) + 1)
//   RC_STASH : t read from the stored map        r = (1 - t) / 2
// ds_tile points at dS[b, i0, j0] (wave-uniform values, zero at masked keys);
// t_tile at tmap[b, i0, 0, h] of this lane, kcol[c] = key index of column c
// clamped into the valid range.
template <int NI, int MODE, int NJ>
__device__ __forceinline__ void rc_tile(const float (&fq)[RC_RI], const float (&fk)[RC_RJ],
                                        const float *__restrict__ ds_tile, int pitch,
                                        const float *__restrict__ t_tile, size_t t_row, size_t t_key,
                                        const int (&kcol)[RC_RJ],
                                        float (&accQ)[RC_RI], float (&accK)[RC_RJ], float (&accV)[4]) {
    // Row by row; the eight evaluations of a row are issued as batches (multiply-adds, reciprocals, ...) so
    // that no instruction waits for the one before it.
#pragma unroll
    for (int a = 0; a < NI; ++a) {
        const float4 d0 = *reinterpret_cast<const float4 *>(ds_tile + a * pitch);
        const float4 d1 = NJ > 4 ? *reinterpret_cast<const float4 *>(ds_tile + a * pitch + 4) : d0;
        const float d[RC_RJ] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        float r[NJ], u[NJ];
        if (MODE == RC_STASH) {
#pragma unroll
            for (int c = 0; c < NJ; ++c) r[c] = __builtin_fmaf(-0.5f, t_tile[a * t_row + kcol[c] * t_key], 0.5f);
        } else {
#pragma unroll
            for (int c = 0; c < NJ; ++c)
                r[c] = MODE == RC_FACTOR ? __builtin_fmaf(fq[a], fk[c], 1.0f) : fast_exp2(fq[a] + fk[c]) + 1.0f;
            trans_begin();
#pragma unroll
            for (int c = 0; c < NJ; ++c) r[c] = fast_rcp(r[c]);
            trans_end();
        }
#pragma unroll
        for (int c = 0; c < NJ; ++c) u[c] = __builtin_fmaf(-r[c], r[c], r[c]);      // r (1 - r) = (1 - t^2) / 4
        float q0 = 0.f, q1 = 0.f;
#pragma unroll
        for (int c = 0; c < NJ; c += 2) {
            accK[c] = __builtin_fmaf(d[c], u[c], accK[c]);
            q0 = __builtin_fmaf(d[c], u[c], q0);
            accV[c & 3] = __builtin_fmaf(d[c], r[c], accV[c & 3]);
            accK[c + 1] = __builtin_fmaf(d[c + 1], u[c + 1], accK[c + 1]);
            q1 = __builtin_fmaf(d[c + 1], u[c + 1], q1);
            accV[(c + 1) & 3] = __builtin_fmaf(d[c + 1], r[c + 1], accV[(c + 1) & 3]);
        }
        accQ[a] += q0 + q1;
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int MODE>
__device__ __forceinline__ void rc_tile_n(int ni, int live, const float (&fq)[RC_RI], const float (&fk)[RC_RJ],
                                          const float *__restrict__ ds_tile, int pitch,
                                          const float *__restrict__ t_tile, size_t t_row, size_t t_key,
                                          const int (&kcol)[RC_RJ],
                                          float (&accQ)[RC_RI], float (&accK)[RC_RJ], float (&accV)[4]) {
#define RC_CASE(N) \
    case N:                                                                                              \
        if (live <= 4) rc_tile<N, MODE, 4>(fq, fk, ds_tile, pitch, t_tile, t_row, t_key, kcol, accQ, accK, accV); \
        else rc_tile<N, MODE, RC_RJ>(fq, fk, ds_tile, pitch, t_tile, t_row, t_key, kcol, accQ, accK, accV);       \
        break;
    switch (ni) {
        RC_CASE(1) RC_CASE(2) RC_CASE(3) RC_CASE(4) RC_CASE(5) RC_CASE(6) RC_CASE(7) RC_CASE(8)
        default: break;
    }
#undef RC_CASE
}

template <typename T, bool STASH, int HW>
__global__ __launch_bounds__(RC_THREADS, 4) void k_recompute(
    const T *__restrict__ Qp, const T *__restrict__ Kp, const T *__restrict__ v,
    const int *__restrict__ order, const float *__restrict__ dS, const float *__restrict__ ds_rowsum,
    const float *__restrict__ tmap, float *__restrict__ dQp, float *__restrict__ dKp, float *dv_part,
    unsigned long long *dv_flag, unsigned long long epoch, float *__restrict__ dv,
    int Tq, int Tk, int H, int pitch, int rows_per_pass, int acc) {
    // Key tile staged once per block, double buffered: exp(2k) for the factor
    // path, 2 log2e k for the exact path, and per key a flag "beyond the factor limit".
    __shared__ float s_fk[2][RC_RJ][HW];
    __shared__ float s_sk[2][RC_RJ][HW];
    __shared__ int s_kbig[2][RC_RJ];
    constexpr int NS = 64 / HW;                             // lane groups
    constexpr int ROWS = RC_W * RC_RI * NS;                 // rows of a pass at most
    __shared__ __align__(16) float s_ds[2][ROWS * RC_RJ];   // dS of the pass rows x tile keys, [row][key]
    __shared__ float s_part[2][RC_W][RC_RJ][64];
    __shared__ float s_dv[RC_W][64];
    __shared__ float s_rowsum;
    __shared__ int s_seen[RC_W];

    // slot -> sample (the heaviest samples start first) and its clamped key length, packed by the ranking block
    const int packed = order[blockIdx.y];
    const int b = packed & 0xffff, L = packed >> 16;
    const int lane = lane_id(), w = wave_id();
    const int sub = lane / HW, hl = lane % HW;
    const int h = blockIdx.x * HW + hl;
    const bool hv = h < H;
    const int hc = hv ? h : H - 1;
    // v of this lane's h: requested here, first touched behind the first loads of a pass (as a guarded load followed
    // by its scaling the compiler waited for it on the spot: a trip to memory before anything else had been requested)
    float v_raw = ld(v, hc);

    float *dQb = dQp ? dQp + (size_t)b * Tq * H : nullptr;
    float *dKb = dKp + (size_t)b * Tk * H;

    // masked keys: exact zeros (when adding to earlier decoder steps they hold zeros already)
    if (!acc)
        for (int j = L + w * NS + sub; j < Tk; j += RC_W * NS)
            if (hv) dKb[(size_t)j * H + h] = 0.f;
    if (L == 0 && dQp) {                            // block-uniform
        for (int i = w * NS + sub; i < Tq; i += RC_W * NS)
            if (hv) dQb[(size_t)i * H + h] = 0.f;
    }
    // sum of this sample's dS (zero in exact arithmetic): the part of sum dS t that comes from t = 1 - 2r.  The last
    // wave adds it up behind the first loads of the first pass, so that its rows are not a trip to memory late.
    auto sum_rows = [&]() {
        float rs = 0.f;
        for (int i = lane; i < Tq; i += 64) rs += ds_rowsum[(size_t)b * Tq + i];
        rs = wave_sum(rs);
        if (lane == 0) s_rowsum = rs;
    };
    if (L == 0 && w == RC_W - 1) sum_rows();

    float accV[4] = {0.f, 0.f, 0.f, 0.f};
    if (L > 0) {
        const T *qb = Qp + (size_t)b * Tq * H;
        const T *kb = Kp + (size_t)b * Tk * H;
        const float *dsb = dS + (size_t)b * Tq * pitch;
        const int n_jt = (L + RC_RJ - 1) / RC_RJ;

        // Tile staging, one tile ahead of the arithmetic.  Wave w fetches key w of the
        // tile (RC_W == RC_RJ) and every thread an element of the pass's dS
        // rows or four; the loads are issued before the current tile is evaluated and
        // committed to the other LDS buffer after it.
        // (one lane group: 64 rows, an element per thread; more: four elements of a row)
        constexpr int DN = NS == 1 ? 1 : 4;
        const int t_row = threadIdx.x / (RC_RJ / DN), t_col = DN * (threadIdx.x % (RC_RJ / DN));
        const bool t_on = RC_THREADS / (RC_RJ / DN) <= ROWS || t_row < ROWS;
        typedef RawElem<T> Raw;
        typename Raw::type kx_raw = 0;
        typedef float DVec __attribute__((ext_vector_type(DN)));
        DVec dx = 0.f;
        auto fetch = [&](int jt, int i_pass0, int nrows) {
            const int j = jt * RC_RJ + w;
            kx_raw = 0;
            if (!STASH && j < L) kx_raw = Raw::load(kb, (size_t)j * H + hc);
            dx = 0.f;
            if (t_row < nrows)
                dx = *reinterpret_cast<const DVec *>(dsb + (size_t)(i_pass0 + t_row) * pitch + jt * RC_RJ + t_col);
        };
        auto commit = [&](int jt, int buf) {
            const int j = jt * RC_RJ + w;
            if (t_on) *reinterpret_cast<DVec *>(&s_ds[buf][t_row * RC_RJ + t_col]) = dx;
            if (STASH) return;
            asm volatile("" : "+v"(kx_raw));
            const float kx = Raw::value(kx_raw);
            if (NS == 1 || sub == 0) s_sk[buf][w][hl] = kTwoLog2e * kx;
            if (NS == 1 || sub == 0) s_fk[buf][w][hl] = (j < L) ? fast_exp2(kTwoLog2e * kx) : 0.f;
            const int big = __any(fabsf(kx) > kFactorLimit) ? 1 : 0;
            if (lane == 0) s_kbig[buf][w] = big;
        };

        int pass = 0;
        for (int i_pass0 = 0; i_pass0 < Tq; i_pass0 += rows_per_pass, ++pass) {
            const int nrows = min(rows_per_pass, Tq - i_pass0);
            // rows are dealt to the waves NS at a time, one to each lane group: this lane's rows are i0 + NS a
            const int n_rg = (nrows + NS - 1) / NS;
            const int g_lo = deal8_begin(n_rg, w), ni = deal8_begin(n_rg, w + 1) - g_lo;   // ni: 0..RC_RI
            const int r_lo = g_lo * NS + sub;
            const int i0 = i_pass0 + r_lo;

            fetch(0, i_pass0, nrows);
            float fq[RC_RI], sq[RC_RI], accQ[RC_RI];
            bool qbig = false;
            {
                typename Raw::type xr[RC_RI];
#pragma unroll
                for (int a = 0; a < RC_RI; ++a) {
                    xr[a] = 0;
                    if (!STASH && a < ni) xr[a] = Raw::load(qb, (size_t)(NS == 1 ? i0 + a : min(i0 + NS * a, Tq - 1)) * H + hc);
                }
                if (pass == 0 && w == RC_W - 1) sum_rows();
                asm volatile("" : "+v"(v_raw));
                float x[RC_RI];
#pragma unroll
                for (int a = 0; a < RC_RI; ++a) {
                    asm volatile("" : "+v"(xr[a]));
                    x[a] = Raw::value(xr[a]);
                }
#pragma unroll
                for (int a = 0; a < RC_RI; ++a) {
                    accQ[a] = 0.f;
                    qbig |= fabsf(x[a]) > kFactorLimit;
                    sq[a] = kTwoLog2e * x[a];
                    fq[a] = fast_exp2(sq[a]);
                }
            }
            const float v4 = hv ? 4.f * v_raw : 0.f;
            const bool wave_qbig = __any(qbig);
            commit(0, 0);
            lds_barrier();

            for (int jt = 0; jt < n_jt; ++jt) {
                const int buf = jt & 1;
                const int j0 = jt * RC_RJ;
                const bool more = jt + 1 < n_jt;
                // valid keys of this tile: a last tile with at most four evaluates half the columns (finer steps
                // make the backward pass alone faster, but the code grows and forward + backward, which alternate
                // in a training step, get slower)
                const int live = L - j0;
                if (more) fetch(jt + 1, i_pass0, nrows);
                float accK[RC_RJ], fk[RC_RJ];
                int kcol[RC_RJ];
#pragma unroll
                for (int c = 0; c < RC_RJ; ++c) {
                    accK[c] = 0.f;
                    kcol[c] = min(j0 + c, L - 1);
                }
                const float *ds_tile = &s_ds[buf][r_lo * RC_RJ];     // wave-uniform reads, pitch RC_RJ
                if (STASH) {
                    const float *t_tile = tmap + (((size_t)b * Tq + i0) * Tk) * H + hc;
#pragma unroll
                    for (int c = 0; c < RC_RJ; ++c) fk[c] = 0.f;
                    rc_tile_n<RC_STASH>(ni, live, fq, fk, ds_tile, NS * RC_RJ, t_tile, (size_t)Tk * H, (size_t)H, kcol, accQ, accK,
                                        accV);
                } else {
                    int kbig = 0;
#pragma unroll
                    for (int c = 0; c < RC_RJ; ++c) kbig |= s_kbig[buf][c];
                    if (!(wave_qbig || kbig)) {
#pragma unroll
                        for (int c = 0; c < RC_RJ; ++c) fk[c] = s_fk[buf][c][hl];
                        rc_tile_n<RC_FACTOR>(ni, live, fq, fk, ds_tile, NS * RC_RJ, nullptr, 0, 0, kcol, accQ, accK, accV);
                    } else {
#pragma unroll
                        for (int c = 0; c < RC_RJ; ++c) fk[c] = s_sk[buf][c][hl];
                        rc_tile_n<RC_EXACT>(ni, live, sq, fk, ds_tile, NS * RC_RJ, nullptr, 0, 0, kcol, accQ, accK, accV);
                    }
                }
                if (more) commit(jt + 1, buf ^ 1);
#pragma unroll
                for (int c = 0; c < RC_RJ; ++c) s_part[buf][w][c][lane] = accK[c];
                lds_barrier();
                // wave w finishes key j0 + w of this tile: sum over the waves in fixed order
                const int j = j0 + w;
                float tot = 0.f;
#pragma unroll
                for (int w2 = 0; w2 < RC_W; ++w2) tot += s_part[buf][w2][w][lane];
                if constexpr (NS >= 2) tot = transpose_pair<32>(tot, tot, lane);     // the lane groups
                if constexpr (NS >= 4) tot = transpose_pair<16>(tot, tot, lane);
                if (j < L && hv && (NS == 1 || sub == 0)) {
                    float *dst = dKb + (size_t)j * H + h;
                    const float val = v4 * tot;
                    if (pass == 0 && !acc) store_streaming(dst, val);
                    else *dst = *dst + val;
                }
            }
            if (hv && dQp) {
#pragma unroll
                for (int a = 0; a < RC_RI; ++a)
                    if (a < ni && (NS == 1 || i0 + NS * a < i_pass0 + nrows))
                        store_streaming(&dQb[(size_t)(i0 + NS * a) * H + h], v4 * accQ[a]);
            }
            lds_barrier();   // the next pass restages buffer 0 and reuses s_part
        }
    }

    // dv partial of this sample: sum dS t = sum dS - 2 sum dS r
    s_dv[w][lane] = (accV[0] + accV[1]) + (accV[2] + accV[3]);
    lds_barrier();
    const int n_slots = gridDim.y;
    unsigned long long *flags = dv_flag + (size_t)blockIdx.x * n_slots;      // of this slice of h, one per sample
    if (w == 0) {
        float tot = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < RC_W; ++w2) tot += s_dv[w2][lane];
        if constexpr (NS >= 2) tot = transpose_pair<32>(tot, tot, lane);
        if constexpr (NS >= 4) tot = transpose_pair<16>(tot, tot, lane);
        send_part(&dv_part[(size_t)b * H + h], __builtin_fmaf(-2.f, tot, s_rowsum), hv && (NS == 1 || sub == 0), &flags[b], epoch);
    }
    // B4 without a launch of its own: the block of the last slot, which starts last, adds the parts of its slice of h
    if ((int)blockIdx.y != n_slots - 1) return;
    lds_barrier();                                   // s_dv is reused below
    const float tot = sum_parts<HW, RC_W>(dv_part, flags, n_slots, H, h, epoch, [](int) { return false; }, &s_dv[0][0], s_seen);
    if (w == 0 && lane < HW && hv) dv[h] = acc ? dv[h] + tot : tot;
}

template <typename T, bool STASH, int HW>
static hipError_t launch_recompute_t(const AttnShape &s, const void *Qp, const void *Kp, const void *v,
                                     const int *order, const float *dS, const float *ds_rowsum, const float *tmap,
                                     float *dQp, float *dKp, float *dv_part, unsigned long long *dv_flag,
                                     unsigned long long epoch, float *dv, hipStream_t st) {
    const int max_rows = RC_W * RC_RI * (64 / HW);
    // full passes first, the remainder last: with the rows split evenly over the passes, waves of 7 and of 8
    // rows meet at every tile's barrier (100 rows: 64 + 36 instead of 50 + 50; backward 141.5 -> 139.8 us at B = 128)
    const int rows_per_pass = s.Tq > max_rows ? max_rows : s.Tq;
    dim3 grid((s.H + HW - 1) / HW, s.B);
    k_recompute<T, STASH, HW><<<grid, RC_THREADS, 0, st>>>((const T *)Qp, (const T *)Kp, (const T *)v, order, dS, ds_rowsum,
                                                           tmap, dQp, dKp, dv_part, dv_flag, epoch, dv, s.Tq, s.Tk, s.H,
                                                           ds_pitch(s.Tk), rows_per_pass, s.acc ? 1 : 0);
    return hipGetLastError();
}

// Expected time of a launch with slices of `hw` columns, in units of one row of a wave against one key tile.  A block walks
// every key tile once per pass over its rows; a tile costs the rows of a wave plus about three rows' worth of staging, sums and
// barriers, the block itself about ten (its prologue, its part of dv).  The samples' mean key count is taken as 0.8 Tk.  Up to
// RC_ROUND blocks the launch lasts as long as a full sample's block (heavy and light samples share a compute unit); beyond, the
// blocks of a round pass through it one after the other, and half a block is lost at the end.
static float recompute_time(const AttnShape &s, int hw) {
    const int ns = 64 / hw, max_rows = RC_W * RC_RI * ns;
    const float passes = (float)((s.Tq + max_rows - 1) / max_rows);
    const float tile = (float)s.Tq / (RC_W * ns) + 3.f * passes;
    const float full = tile * ((s.Tk + RC_RJ - 1) / RC_RJ) + 10.f, mean = 0.8f * tile * s.Tk / RC_RJ + 10.f;
    const float blocks = (float)s.B * ((s.H + hw - 1) / hw);
    const float all = blocks / RC_ROUND * mean + 0.5f * mean;
    return blocks <= RC_ROUND || full > all ? full : all;
}

// Width of a block's slice of h: 64, 32 or 16.  A narrower slice means more blocks of less work each (lane groups share the
// rows): it fills the chip, balances it better, makes do with fewer passes over the keys (one pass takes 64, 128 or 256 rows) and
// leaves fewer columns idle, but a wave has fewer rows to share a key tile's fixed costs.  Taken where recompute_time
// expects at least 2 % from it; over 104 shapes of 20 and more keys the whole backward was within 4 % of the best of the
// three widths on all but one (7 %).  Measured (recompute launch): B = 32, T = 100, H = 512, 64 -> 32 columns 56 -> 33 us; B = 16, T = 300, H = 512, 64 ->
// 16 401 -> 145.  Backward: B = 27, T = 181 / 233, H = 340, 32 -> 16 218 -> 176; B = 101, T = 199 / 240, H = 268, 64 -> 16 492 -> 412; B = 32,
// T = 194 / 182, H = 577, 64 -> 16 295 -> 198; B = 58, T = 108 / 163, H = 568, 64 -> 32 155 -> 132.  The wider ones win
// on few rows (B = 64, T = 50, H = 512: 30 us at 64 columns, 38 at 32) and where they fill one round just so (B = 32, T = 300, H =
// 1024: 644 against 702).  With a wave's rows already down to three a narrower slice gives nothing.  An H that fits the
// narrower slice whole takes it in any case.
static int recompute_width(const AttnShape &s) {
    int hw = 64;
    for (int narrow = 32; narrow >= 16; narrow /= 2)
        if (s.H <= narrow || (s.Tq > 3 * RC_W && recompute_time(s, narrow) < 0.98f * recompute_time(s, hw))) hw = narrow;
    return hw;
}

// The form of recompute_rows.hip where its expected time is 5 % ahead, 13 % on grids just past a round (whose few blocks more cost it,
// with its slices of 64 columns, more than the estimate says: 515 blocks at B = 103, T = 83 / 68, H = 272 84.7 us backward against 76.5).
// Over 420 shapes of 60 to 480 rows from 256 of its blocks on the whole backward takes 0.938 of the time without it, over the 244 that
// take it 0.895, two of them 3 and 5 % more; over 600 of 240 to 1100 blocks and any H 0.965, over the 228 that take it 0.913, five of them 2
// to 14 % more (most where the keys per sample differ much and the heaviest sample's block decides: B = 31, T = 128 / 166, H = 816 in
// bf16, 17 to 166 keys, 74.6 us without it, 85.1 with).  A margin of 7 % would leave out 64 of them, 0.949 of the time on average.
// B = 128, T = 100, H = 512 135 -> 119 us; B = 32, T = 300, H = 1024 604 -> 516; B = 64, T = 200 / 30, H = 512 65 -> 58.
static bool recompute_takes_rows(const AttnShape &s) {
    const float rows = recompute_rows_time(s);
    const long long blocks = (long long)s.B * ((s.H + 63) / 64);
    return rows > 0.f && rows * (blocks > RC_ROUND && blocks <= RC_ROUND * 5 / 4 ? 1.13f : 1.05f) < recompute_time(s, recompute_width(s));
}

// In a grid that runs all at once the first RC_ROUND / 2 blocks have a compute unit each and the others join them in turn, so sample n +
// first meets sample n.  That the second half of the samples meets the first holds for a full round alone: with the order laid out
// that on every grid, the form by rows took up to 18 % more for the backward than narrower slices did (B = 22, T = 132 / 136, H = 1000 in bf16,
// 352 blocks, 85.4 us without it: 97.0 -> 80.1; B = 58, T = 271 / 190, H = 376 in bf16, 348 blocks, 281: 285 -> 250).  Over 466 grids of
// 257 to 512 blocks the backward takes 0.976 of the time it took, 0.83 to 1.02.
// Rounded down: with the last of them over the edge the heaviest samples' blocks share a unit (up to 39 % more).
int recompute_first_samples(const AttnShape &s, bool stash) {
    const int hw = stash || recompute_takes_rows(s) ? 64 : recompute_width(s);
    const int slices = (s.H + hw - 1) / hw;
    if ((long long)s.B * slices > RC_ROUND) return 0;
    return std::min(s.B, std::max(RC_ROUND / 2 / slices, (s.B + 1) / 2));
}

template <typename T>
static hipError_t launch_recompute_w(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order,
                                     const float *dS, const float *ds_rowsum, const float *tmap, float *dQp, float *dKp,
                                     float *dv_part, unsigned long long *dv_flag, unsigned long long epoch, float *dv,
                                     hipStream_t st) {
    if (tmap) return launch_recompute_t<T, true, 64>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag, epoch, dv, st);
    switch (recompute_width(s)) {
        case 16: return launch_recompute_t<T, false, 16>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag, epoch, dv, st);
        case 32: return launch_recompute_t<T, false, 32>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag, epoch, dv, st);
        default: return launch_recompute_t<T, false, 64>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag, epoch, dv, st);
    }
}

hipError_t launch_recompute(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order,
                            const float *dS, const float *ds_rowsum, const float *tmap, float *dQp, float *dKp,
                            float *dv_part, unsigned long long *dv_flag, unsigned long long epoch, float *dv,
                            hipStream_t st) {
    if (!tmap && recompute_takes_rows(s))
        return launch_recompute_rows(s, Qp, Kp, v, order, dS, ds_rowsum, dQp, dKp, dv_part, dv_flag, epoch, dv, st);
    return s.bf16 ? launch_recompute_w<bf16_t>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag,
                                               epoch, dv, st)
                  : launch_recompute_w<float>(s, Qp, Kp, v, order, dS, ds_rowsum, tmap, dQp, dKp, dv_part, dv_flag,
                                              epoch, dv, st);
}

}  // namespace echo
