// The fused recomputation (recompute.hip) for launches that would leave most of the chip idle.
//
// k_recompute gives every sample and slice of h to one block, which evaluates each tanh once and spends it on
// dQp, dKp and dv alike.  With B ceil(H / 16), its blocks at the narrowest, below the number of compute units a handful of
// blocks walk a whole sample each while the rest of the chip waits.  Here the sums are split so
// that no block needs another's partial result: blocks of one kind own query rows and sum over the keys (dQp), blocks of
// the other kind own keys and sum over the query rows (dKp and the sample's part of dv).  Every tanh is evaluated twice
// (15 issue slots per element instead of 9), but the work spreads over as many blocks and waves as wanted.
//
// A block owns up to XW * 8 * NS rows ("x": queries or keys) of one sample and a slice of HW columns of h, HW = 16, 32 or
// 64: the 64 lanes are NS = 64 / HW groups of HW columns, so that a narrow H does not leave lanes idle.  Its eight waves
// are XW groups of rows times YS shares of the other axis ("y"), XW YS = 8; a lane owns eight rows of its group and walks
// its wave's share of y in chunks of four, the y values of the next chunk already requested.  The dS entries of the block's
// rows are staged in LDS, one range of y at a time.  With YS > 1 the waves' sums meet in LDS at the end.  The order of all
// additions is fixed.
//
// k_bwd_small is the same with everything that comes before it: the whole backward of a small batch in one launch.
//
// dv: every key-owning block hands its part (per column of h) to the last block of the slice, which starts last and adds the
// parts in order (send_part, sum_parts).
#include "common.hpp"
#include "kernels.hpp"

namespace echo {

constexpr int RS_W = 8;                    // waves per block
constexpr int RS_THREADS = 64 * RS_W;
constexpr int RS_R = 8;                    // rows a lane owns
constexpr int RS_C = 4;                    // y per chunk
constexpr int RS_TILE = 6144;              // floats of staged dS (24 KB)

struct RsAxis {                            // how a kind of block cuts its axes (the same for the whole launch)
    int groups;                            // blocks per sample and slice
    int ys;                                // waves that share a row group (1, 2, 4, 8)
    int y_tile;                            // y per staged range: a multiple of RS_C, rows * (y_tile + RS_C) <= RS_TILE
};
// rows of one block
__host__ __device__ constexpr int rs_rows(int hw, int ys) { return RS_W / ys * RS_R * (64 / hw); }

// row pitch of the staged dS: an odd multiple of four floats, so that the lane groups of a narrow slice read their rows from
// different banks
__host__ __device__ constexpr int rs_pitch(int y_tile) { return RS_C * ((y_tile / RS_C) | 1); }

// One chunk: eight rows of a lane against four y.  EXACT: fx, fy hold 2 log2e x and the exponential of the sum is taken.
template <bool EXACT, bool DV>
__device__ __forceinline__ void rs_chunk(const float (&fx)[RS_R], const float (&fy)[RS_C], const float *__restrict__ d_row,
                                         int d_step, float (&acc)[RS_R], float (&acc_v)[RS_C]) {
#pragma unroll
    for (int a0 = 0; a0 < RS_R; a0 += 2) {                 // two rows at a time: eight independent evaluations
        float4 d4[2];
        float r[2][RS_C], u[2][RS_C];
#pragma unroll
        for (int a = 0; a < 2; ++a) d4[a] = *reinterpret_cast<const float4 *>(d_row + (a0 + a) * d_step);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int c = 0; c < RS_C; ++c)
                r[a][c] = EXACT ? fast_exp2(fx[a0 + a] + fy[c]) + 1.0f : __builtin_fmaf(fx[a0 + a], fy[c], 1.0f);
        trans_begin();
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int c = 0; c < RS_C; ++c) r[a][c] = fast_rcp(r[a][c]);
        trans_end();
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int c = 0; c < RS_C; ++c) u[a][c] = __builtin_fmaf(-r[a][c], r[a][c], r[a][c]);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const float d[RS_C] = {d4[a].x, d4[a].y, d4[a].z, d4[a].w};
            float p = d[0] * u[a][0], q = d[1] * u[a][1];
            p = __builtin_fmaf(d[2], u[a][2], p);
            q = __builtin_fmaf(d[3], u[a][3], q);
            acc[a0 + a] += p + q;
            if (DV) {
#pragma unroll
                for (int c = 0; c < RS_C; ++c) acc_v[c] = __builtin_fmaf(d[c], r[a][c], acc_v[c]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// X: rows of the owned axis [n_x valid rows, row stride H], Y: rows of the axis summed over [n_y rows].  out: rows of the
// result.  KEYS: x = keys, y = queries (dKp, dv), else x = queries, y = keys (dQp).
// stage(y0, ny): puts the dS entries of the block's rows for y0 .. y0 + ny - 1 into s_d [row][y], zeros where they are to add
// nothing, and returns this thread's share of their sum; it is called after the first loads of the block (or range) have
// been requested, and a barrier follows it.  s_red: RS_W RS_R 64 floats, s_v: RS_W 65 floats.
template <typename T, int HW, bool KEYS, typename Stage>
__device__ __forceinline__ void rs_block(const T *__restrict__ X, const T *__restrict__ Y, const T *__restrict__ v,
                                         float *__restrict__ out, bool add, float *part,
                                         unsigned long long *flag, unsigned long long epoch, int x_first, int n_x,
                                         int n_out, int n_y, int H, int h0, int ys, int y_tile,
                                         const float *__restrict__ s_d, int d_pitch, float *__restrict__ s_red,
                                         float *__restrict__ s_v, Stage stage) {
    constexpr int NS = 64 / HW;
    typedef RawElem<T> Raw;
    const int lane = lane_id(), w = wave_id();
    const int sub = lane / HW;
    const int h = h0 + lane % HW;
    const bool hv = h < H;
    const int hc = hv ? h : H - 1;
    const int yg = w & (ys - 1), xg = w / ys;
    const int xl = xg * RS_R * NS + sub;                    // this lane's rows: x_first + xl + NS a
    const bool wave_on = x_first + xg * RS_R * NS < n_x;    // the wave has valid rows

    typename Raw::type v_raw = Raw::load(v, hc);
    typename Raw::type x_raw[RS_R];
#pragma unroll
    for (int a = 0; a < RS_R; ++a) x_raw[a] = Raw::load(X, (size_t)min(x_first + xl + NS * a, n_x - 1) * H + hc);

    float acc[RS_R], acc_v[RS_C] = {0.f, 0.f, 0.f, 0.f}, fx[RS_R], sx[RS_R];
#pragma unroll
    for (int a = 0; a < RS_R; ++a) acc[a] = 0.f;
    bool x_big = false, first = true;
    float d_sum = 0.f;
    for (int y0 = 0; y0 < n_y; y0 += y_tile) {
        const int ny = min(y_tile, n_y - y0);
        const int ny4 = (ny + RS_C - 1) & ~(RS_C - 1);
        // the first chunk of this wave's share leaves together with the dS of the range
        typename Raw::type y_raw[RS_C];
        auto fetch = [&](int y) {
#pragma unroll
            for (int c = 0; c < RS_C; ++c) y_raw[c] = Raw::load(Y, (size_t)min(y0 + y + c, n_y - 1) * H + hc);
        };
        fetch(RS_C * yg);
        if (!first) lds_barrier();                          // everybody is done with the previous range
        d_sum += stage(y0, ny);
        if (first) {
            asm volatile("" : "+v"(v_raw));
#pragma unroll
            for (int a = 0; a < RS_R; ++a) {
                asm volatile("" : "+v"(x_raw[a]));
                const float x = Raw::value(x_raw[a]);
                x_big |= fabsf(x) > kFactorLimit;
                sx[a] = kTwoLog2e * x;
                fx[a] = fast_exp2(sx[a]);
            }
            first = false;
        }
        lds_barrier();
        if (wave_on) {
            for (int y = RS_C * yg; y < ny4; y += RS_C * ys) {
                float sy[RS_C], fy[RS_C];
                bool big = x_big;
#pragma unroll
                for (int c = 0; c < RS_C; ++c) asm volatile("" : "+v"(y_raw[c]));
#pragma unroll
                for (int c = 0; c < RS_C; ++c) {
                    const float k = Raw::value(y_raw[c]);
                    big |= fabsf(k) > kFactorLimit;
                    sy[c] = kTwoLog2e * k;
                    fy[c] = fast_exp2(sy[c]);
                }
                fetch(min(y + RS_C * ys, ny4 - RS_C));
                const float *d_row = s_d + xl * d_pitch + y;
                if (!__any(big)) rs_chunk<false, KEYS>(fx, fy, d_row, NS * d_pitch, acc, acc_v);
                else rs_chunk<true, KEYS>(sx, sy, d_row, NS * d_pitch, acc, acc_v);
            }
        }
    }

    const float v4 = hv ? 4.f * Raw::value(v_raw) : 0.f;
    int x_out = x_first + xl;
    asm volatile("" : "+v"(x_out));                         // addresses formed here, not kept since the loads
    auto store = [&](int x, float val) {
        if (x >= n_out || !hv) return;
        float *dst = out + (size_t)x * H + h;
        if (x >= n_x) {
            if (!add) *dst = 0.f;                           // masked key (adding: it holds a zero already)
        } else if (add) {
            *dst += val;
        } else {
            store_streaming(dst, val);
        }
    };
    if (ys == 1) {
#pragma unroll
        for (int a = 0; a < RS_R; ++a) store(x_out + NS * a, v4 * acc[a]);
    } else {
#pragma unroll
        for (int a = 0; a < RS_R; ++a) s_red[(w * RS_R + a) * 64 + lane] = acc[a];
    }
    if (KEYS) {
        s_v[w * 64 + lane] = (acc_v[0] + acc_v[1]) + (acc_v[2] + acc_v[3]);
        d_sum = wave_sum(d_sum);
        if (lane == 0) s_v[RS_W * 64 + w] = d_sum;
    }
    if (KEYS || ys > 1) lds_barrier();
    if (ys > 1) {
        // row a of group xg: its YS partial sums, added by the group's waves in turn
        for (int a = yg; a < RS_R; a += ys) {
            float tot = 0.f;
            for (int k = 0; k < ys; ++k) tot += s_red[((xg * ys + k) * RS_R + a) * 64 + lane];
            store(x_out + NS * a, v4 * tot);
        }
    }
    if (KEYS && w == 0) {
        float tot = 0.f, dtot = 0.f;
#pragma unroll
        for (int k = 0; k < RS_W; ++k) {
            tot += s_v[k * 64 + lane];
            dtot += s_v[RS_W * 64 + k];
        }
        if constexpr (NS >= 2) tot += __shfl_xor(tot, 32);
        if constexpr (NS >= 4) tot += __shfl_xor(tot, 16);
        send_part(part + h, __builtin_fmaf(-2.f, tot, dtot), sub == 0 && hv, flag, epoch);   // sum dS t = sum dS - 2 sum dS r
    }
}

// Stager from memory: the sample's dS [query][key], rows x_first ..; n_x valid rows.
template <int HW, bool KEYS>
__device__ __forceinline__ float rs_stage(const float *__restrict__ ds, int pitch, int x_first, int n_x, int ys, int y0, int ny,
                                          float *__restrict__ s_d, int d_pitch) {
    const int rows = rs_rows(HW, ys);
    const int ny4 = (ny + RS_C - 1) & ~(RS_C - 1);
    float d_sum = 0.f;
    // dS of (rows, range), four entries of a dS row per load, all loads of the range under way together; the pads of a
    // dS row and its masked keys are stored zeros, rows past the end become zeros here: they add nothing
    constexpr int U = (RS_TILE / 4 + RS_THREADS - 1) / RS_THREADS;
    const int n_vec = rows * ny4 / 4, per_row = KEYS ? rows / 4 : ny4 / 4;
    const float inv = fast_rcp((float)per_row);         // (e + 0.5) inv: exact quotient for e < 2^16
    float4 d4[U];
    int at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = (int)threadIdx.x + u * RS_THREADS;
        const int r = (int)(((float)e + 0.5f) * inv), c = 4 * (e - r * per_row);
        const int xr = KEYS ? c : r, yr = KEYS ? r : c;
        at[u] = e < n_vec ? xr * d_pitch + yr : -1;
        d4[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (KEYS ? (e < n_vec && yr < ny && x_first + xr < pitch) : (e < n_vec && x_first + xr < n_x))
            d4[u] = KEYS ? ld4(ds, (size_t)(y0 + yr) * pitch + x_first + xr) : ld4(ds, (size_t)(x_first + xr) * pitch + y0 + yr);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (at[u] < 0) continue;
        if (KEYS) {
            s_d[at[u]] = d4[u].x;
            s_d[at[u] + d_pitch] = d4[u].y;
            s_d[at[u] + 2 * d_pitch] = d4[u].z;
            s_d[at[u] + 3 * d_pitch] = d4[u].w;
            d_sum += (d4[u].x + d4[u].y) + (d4[u].z + d4[u].w);
        } else {
            *reinterpret_cast<float4 *>(s_d + at[u]) = d4[u];
        }
    }
    return d_sum;
}

// grid (slices of h, samples heaviest first, groups of keys then groups of queries)
template <typename T, int HW>
__global__ __launch_bounds__(RS_THREADS, 4) void k_recompute_split(
    const T *__restrict__ Qp, const T *__restrict__ Kp, const T *__restrict__ v, const int *__restrict__ order,
    const float *__restrict__ dS, float *__restrict__ dQp, float *__restrict__ dKp, float *parts,
    unsigned long long *flags, unsigned long long epoch, float *__restrict__ dv, int Tq, int Tk, int H, int pitch, RsAxis ka, RsAxis qa, int acc) {
    __shared__ __align__(16) float s_d[RS_TILE];
    __shared__ __align__(16) float s_red[RS_W * RS_R * 64 + RS_W * 64 + RS_W];
    __shared__ int s_seen[RS_W];
    const int packed = order[blockIdx.y];
    const int b = packed & 0xffff, L = packed >> 16;
    const int h0 = blockIdx.x * HW;
    const int n_slots = gridDim.y;
    const int z = blockIdx.z;
    unsigned long long *slice_flags = flags + (size_t)blockIdx.x * n_slots * ka.groups;
    const T *qb = Qp + (size_t)b * Tq * H, *kb = Kp + (size_t)b * Tk * H;
    const float *dsb = dS + (size_t)b * Tq * pitch;
    if (z < ka.groups) {
        const int x0 = z * rs_rows(HW, ka.ys);
        if (x0 < L) {
            const int dp = rs_pitch(ka.y_tile);
            rs_block<T, HW, true>(kb, qb, v, dKp + (size_t)b * Tk * H, acc != 0,
                                  parts + ((size_t)blockIdx.y * ka.groups + z) * H, slice_flags + blockIdx.y * ka.groups + z,
                                  epoch, x0, L, Tk, Tq, H, h0, ka.ys, ka.y_tile, s_d, dp, s_red, s_red + RS_W * RS_R * 64,
                                  [&](int y0, int ny) { return rs_stage<HW, true>(dsb, pitch, x0, L, ka.ys, y0, ny, s_d, dp); });
        } else if (!acc) {                                  // masked keys only: exact zeros
            const int n = min(rs_rows(HW, ka.ys), Tk - x0), lh = threadIdx.x % HW;
            for (int x = threadIdx.x / HW; x < n; x += RS_THREADS / HW)
                if (h0 + lh < H) dKp[((size_t)b * Tk + x0 + x) * H + h0 + lh] = 0.f;
        }
    } else {
        const int x0 = (z - ka.groups) * rs_rows(HW, qa.ys);
        float *out = dQp + (size_t)b * Tq * H;
        if (L > 0) {
            const int dp = rs_pitch(qa.y_tile);
            rs_block<T, HW, false>(qb, kb, v, out, false, nullptr, nullptr, 0, x0, Tq, Tq, L, H, h0, qa.ys, qa.y_tile, s_d, dp,
                                   s_red, s_red + RS_W * RS_R * 64,
                                   [&](int y0, int ny) { return rs_stage<HW, false>(dsb, pitch, x0, Tq, qa.ys, y0, ny, s_d, dp); });
        } else {
            const int n = min(rs_rows(HW, qa.ys), Tq - x0), lh = threadIdx.x % HW;
            for (int x = threadIdx.x / HW; x < n; x += RS_THREADS / HW)
                if (h0 + lh < H) out[(size_t)(x0 + x) * H + h0 + lh] = 0.f;
        }
    }
    if (z != (int)gridDim.z - 1 || (int)blockIdx.y != n_slots - 1) return;

    // ---- the last block of the slice: dv = the parts of all samples and key groups; groups past a sample's last valid key
    // send nothing
    lds_barrier();                                          // s_red is reused
    const int h = h0 + lane_id() % HW, key_rows = rs_rows(HW, ka.ys);
    const float tot = sum_parts<HW, RS_W>(parts, slice_flags, n_slots * ka.groups, H, h, epoch,
                                          [&](int p) { return (p % ka.groups) * key_rows >= (order[p / ka.groups] >> 16); },
                                          s_red, s_seen);
    if (wave_id() == 0 && lane_id() < HW && h < H) dv[h] = acc ? dv[h] + tot : tot;
}

// ---- the whole backward in one launch -------------------------------------------------------------------------------

constexpr int BS_ROWS = 64;                // most query rows and most keys
constexpr int BS_PITCH = BS_ROWS + 4;      // floats: an odd multiple of 16 bytes

// What a block of k_bwd_small keeps in LDS.
struct BsLds {
    float stage[2 * BS_ROWS * BS_PITCH];   // a piece of dC and of V; then dP, in parts; then (second half) the last reduction
    float d[BS_ROWS * BS_PITCH];           // the dS entries of the block's rows
    float s_v[RS_W * 64 + RS_W];
    int seen[RS_W];
};
constexpr int BS_HALF = BS_ROWS * BS_PITCH;

// dS of the block's rows from dC, V and P.  Every block forms the whole dP of its sample: the softmax backward needs whole rows,
// and at up to 16 tiles of 16 x 16 this is cheaper than a launch of its own and the trip of dS through memory.  dC and V pass
// through LDS in pieces of 64, 128 or 256 columns (64, 32 or 16 rows of each: two 16-byte loads of each per thread), the next
// piece on its way in registers.  The tiles are dealt to the waves; with four or fewer, the columns of a piece are too.
template <typename T>
struct BsScores {
    const float *dC;
    const T *V;
    int Tq, Tk, Dv, cols_log;              // columns of a piece: 1 << cols_log
    float pr[8];                           // P of the rows this wave finishes: w, w + 8, ..; a key per lane
    float4 c4[2];
    RawKey<T> v4[2];

    __device__ __forceinline__ void fetch(int d0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {      // rows and columns past the ends repeat the last ones
            const int e = (int)threadIdx.x + u * RS_THREADS;
            const int row = e >> (cols_log - 2), col = min(d0 + 4 * (e & ((1 << (cols_log - 2)) - 1)), Dv - 4);
            c4[u] = ld4(dC, (size_t)min(row, Tq - 1) * Dv + col);
            v4[u].load(V, (size_t)min(row, Tk - 1) * Dv + col);
        }
    }
    // what does not depend on the sample's key count
    __device__ __forceinline__ void start(const float *P) {
        const int rows = max(Tq, Tk);
        cols_log = rows <= 16 ? 8 : rows <= 32 ? 7 : 6;
        fetch(0);
#pragma unroll
        for (int t = 0; t < 8; ++t) pr[t] = P[min(wave_id() + 8 * t, Tq - 1) * Tk + min(lane_id(), Tk - 1)];
    }
    // dS into lds.d (KEYS: [key - x0][query], else [query - x0][key]), zeros beyond Tq and the L > 0 valid keys; returns this
    // thread's share of the sum over the block's keys (KEYS)
    template <bool KEYS>
    __device__ __forceinline__ float finish(int x0, int rows, int L, BsLds &lds) {
        const int lane = lane_id(), w = wave_id();
        const int lm = lane & 15, lk = lane >> 4;
        const int mt = (Tq + 15) / 16, nt = (L + 15) / 16;
        // both counts rounded up to powers of two: waves side by side, one tile (of 16: two) each, and shares of a piece's columns
        const int m_log = mt > 2 ? 2 : mt - 1, n_log = nt > 2 ? 2 : nt - 1;
        const int dealt_log = min(m_log + n_log, 3), shares = RS_W >> dealt_log, share = w >> dealt_log;
        const int tm = (w & ((1 << dealt_log) - 1)) >> n_log, tn = w & ((1 << n_log) - 1);      // tiles (tm, tn), (tm + 2, tn)
        const int pitch = (1 << cols_log) + 4;
        f32x4 acc[2];
        acc[0] = acc[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int d0 = 0; d0 < Dv; d0 += 1 << cols_log) {
            if (d0 > 0) lds_barrier();                       // everybody is done with the previous piece
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = (int)threadIdx.x + u * RS_THREADS;
                const int row = e >> (cols_log - 2), col = 4 * (e & ((1 << (cols_log - 2)) - 1));
                // columns past Dv add nothing
                *reinterpret_cast<float4 *>(lds.stage + row * pitch + col) = d0 + col < Dv ? c4[u] : make_float4(0.f, 0.f, 0.f, 0.f);
                *reinterpret_cast<float4 *>(lds.stage + BS_HALF + row * pitch + col) = v4[u].get();
            }
            if (d0 + (1 << cols_log) < Dv) fetch(d0 + (1 << cols_log));
            lds_barrier();
            const int n_u = (min(1 << cols_log, Dv - d0) + 15) / 16;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (tm + 2 * t < mt && tn < nt && (t == 0 || m_log + n_log == 4)) {            // uniform
                    const float *a_row = lds.stage + (16 * (tm + 2 * t) + lm) * pitch + 4 * lk;
                    const float *b_row = lds.stage + BS_HALF + (16 * tn + lm) * pitch + 4 * lk;
                    for (int u = share; u < n_u; u += shares) {
                        const float4 a = *reinterpret_cast<const float4 *>(a_row + 16 * u);
                        const float4 b = *reinterpret_cast<const float4 *>(b_row + 16 * u);
                        acc[t] = mfma16(a.x, b.x, acc[t]);
                        acc[t] = mfma16(a.y, b.y, acc[t]);
                        acc[t] = mfma16(a.z, b.z, acc[t]);
                        acc[t] = mfma16(a.w, b.w, acc[t]);
                    }
                }
            }
        }
        lds_barrier();
        // the shares' tiles, then their sums: shares x 16 mt rows fit, as shares mt <= 8
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (tm + 2 * t < mt && tn < nt && (t == 0 || m_log + n_log == 4)) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    lds.stage[(16 * (share * mt + tm + 2 * t) + 4 * lk + q) * BS_PITCH + 16 * tn + lm] = acc[t][q];
            }
        }
        lds_barrier();
        // softmax backward, two rows of a wave at a time: dS = P (dP - sum_j P dP)
        const bool on = lane < L;                            // elsewhere nothing has been written
        float d_sum = 0.f;
#pragma unroll
        for (int t0 = 0; t0 < 8; t0 += 2) {
            if (8 * t0 >= ((Tq + 3) & ~3)) break;            // uniform
            float dp[2], prod[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int i = w + 8 * (t0 + t);
                float x = 0.f;
                for (int k = 0; k < shares; ++k) x += lds.stage[min(16 * mt * k + i, 2 * BS_ROWS - 1) * BS_PITCH + lane];
                const bool valid = on && i < Tq;
                if (!valid) pr[t0 + t] = 0.f;
                dp[t] = valid ? x : 0.f;
                prod[t] = pr[t0 + t] * dp[t];
            }
            const float tot = wave_transpose_sum<2>(prod);   // of row t in lanes 32 t .. 32 t + 31
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float x = pr[t0 + t] * (dp[t] - lane_value(tot, 32 * t));
                const int i = w + 8 * (t0 + t);
                if (KEYS) {
                    if (lane >= x0 && lane < x0 + rows) {
                        lds.d[(lane - x0) * BS_PITCH + i] = x;
                        d_sum += x;
                    }
                } else if (i >= x0 && i < x0 + rows) {
                    lds.d[(i - x0) * BS_PITCH + lane] = x;
                }
            }
        }
        return d_sum;
    }
};

// dV of all keys and 64 columns: wave w forms the tile of keys 16 (w % 4) from one half of the query rows (w / 4).
// s_part: 4 x 16 x 64 floats.
__device__ __forceinline__ void bs_dv(const float *__restrict__ P, const float *__restrict__ dC, float *__restrict__ dV,
                                      float *__restrict__ s_part, int Tq, int Tk, int L, int Dv, int n0, bool add) {
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int m0 = 16 * (w % 4), ncol = n0 + 4 * lm;
    const int half = ((Tq + 7) / 8) * 4, k_lo = (w / 4) * half;
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (m0 < L) {                                            // uniform
        float a[8];
        float4 bv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k_lo + 4 * u + lk;
            const bool on = 4 * u + lk < half && k < Tq;
            a[u] = on && m0 + lm < L ? P[(size_t)k * Tk + m0 + lm] : 0.f;
            bv[u] = on && ncol < Dv ? ld4(dC, (size_t)k * Dv + ncol) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (4 * u < half) {                              // uniform
                acc[0] = mfma16(a[u], bv[u].x, acc[0]);
                acc[1] = mfma16(a[u], bv[u].y, acc[1]);
                acc[2] = mfma16(a[u], bv[u].z, acc[2]);
                acc[3] = mfma16(a[u], bv[u].w, acc[3]);
            }
        }
    }
    float *mine = s_part + (size_t)(w % 4) * 16 * 64 + 4 * lm;
    if (w >= 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(mine + (4 * lk + q) * 64) = make_float4(acc[0][q], acc[1][q], acc[2][q], acc[3][q]);
    }
    lds_barrier();
    if (w >= 4 || ncol >= Dv) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = m0 + 4 * lk + q;
        if (m < Tk) {
            const float4 x = *reinterpret_cast<const float4 *>(mine + (4 * lk + q) * 64);
            float4 o = make_float4(acc[0][q] + x.x, acc[1][q] + x.y, acc[2][q] + x.z, acc[3][q] + x.w);
            float *dst = dV + (size_t)m * Dv + ncol;
            if (add) {
                const float4 old = *reinterpret_cast<const float4 *>(dst);
                o.x += old.x;
                o.y += old.y;
                o.z += old.z;
                o.w += old.w;
            }
            store4_streaming(dst, o);
        }
    }
}

// grid (slices of h or pieces of 64 columns of dV, samples, 1 + groups of keys + groups of queries); z = 0: dV
// Bound by its chain of trips: key count and rows, dP, dS, the exchange of dv.  One block per compute unit: within 128
// registers (two) it spills and was slower at every grid it is taken for.
template <typename T, int HW>
__global__ __launch_bounds__(RS_THREADS, 2) void k_bwd_small(
    const float *__restrict__ dC, const float *__restrict__ P, const T *__restrict__ V, const T *__restrict__ Qp,
    const T *__restrict__ Kp, const T *__restrict__ v, const int *__restrict__ key_len, float *__restrict__ dQp,
    float *__restrict__ dKp, float *__restrict__ dV, float *parts, unsigned long long *flags, unsigned long long epoch,
    float *__restrict__ dv, int Tq, int Tk, int H, int Dv, RsAxis ka, RsAxis qa, int acc) {
    __shared__ __align__(16) BsLds lds;
    const int b = blockIdx.y, slice = blockIdx.x;
    if (blockIdx.z == 0) {
        if (64 * slice < Dv)
            bs_dv(P + (size_t)b * Tq * Tk, dC + (size_t)b * Tq * Dv, dV + (size_t)b * Tk * Dv, lds.stage, Tq, Tk,
                  clamp_len(key_len[b], Tk), Dv, 64 * slice, acc != 0);
        return;
    }
    if (slice * HW >= H) return;
    const int z = (int)blockIdx.z - 1;
    const int h0 = slice * HW;
    BsScores<T> scores{dC + (size_t)b * Tq * Dv, V + (size_t)b * Tk * Dv, Tq, Tk, Dv};
    scores.start(P + (size_t)b * Tq * Tk);
    const int L = clamp_len(key_len[b], Tk);
    const int B = gridDim.y;
    unsigned long long *slice_flags = flags + (size_t)slice * B * ka.groups;
    const T *qb = Qp + (size_t)b * Tq * H, *kb = Kp + (size_t)b * Tk * H;
    const bool keys = z < ka.groups;
    const int rows = rs_rows(HW, keys ? ka.ys : qa.ys), x0 = (keys ? z : z - ka.groups) * rows;
    float *out = keys ? dKp + (size_t)b * Tk * H : dQp + (size_t)b * Tq * H;
    if (keys && x0 < L) {
        rs_block<T, HW, true>(kb, qb, v, out, acc != 0, parts + ((size_t)b * ka.groups + z) * H, slice_flags + b * ka.groups + z,
                              epoch, x0, L, Tk, Tq, H, h0, ka.ys, BS_ROWS, lds.d, BS_PITCH, lds.stage + BS_HALF,
                              lds.s_v, [&](int, int) { return scores.template finish<true>(x0, rows, L, lds); });
    } else if (!keys && L > 0) {
        rs_block<T, HW, false>(qb, kb, v, out, false, nullptr, nullptr, 0, x0, Tq, Tq, L, H, h0, qa.ys, BS_ROWS, lds.d, BS_PITCH,
                               lds.stage + BS_HALF, lds.s_v, [&](int, int) { return scores.template finish<false>(x0, rows, L, lds); });
    } else if (!keys || !acc) {                              // masked keys only, or none valid: exact zeros
        const int n = min(rows, (keys ? Tk : Tq) - x0), lh = threadIdx.x % HW;
        for (int x = threadIdx.x / HW; x < n; x += RS_THREADS / HW)
            if (h0 + lh < H) out[(size_t)(x0 + x) * H + h0 + lh] = 0.f;
    }
    if (z != ka.groups + qa.groups - 1 || b != B - 1) return;

    lds_barrier();                                          // the reduction's region is reused
    const int h = h0 + lane_id() % HW, key_rows = rs_rows(HW, ka.ys);
    const float tot = sum_parts<HW, RS_W>(parts, slice_flags, B * ka.groups, H, h, epoch,
                                          [&](int p) { return (p % ka.groups) * key_rows >= clamp_len(key_len[p / ka.groups], Tk); },
                                          lds.s_v, lds.seen);
    if (wave_id() == 0 && lane_id() < HW && h < H) dv[h] = acc ? dv[h] + tot : tot;
}

// ---- host side ------------------------------------------------------------------------------------------------------

constexpr int RS_ROUND = 512;              // two blocks on every compute unit (128 registers per lane)
constexpr float RS_BLOCK_US = 4.0f, RS_CHUNK_US = 1.1f;
constexpr int BS_ROUND = 256;              // one block of k_bwd_small per compute unit
constexpr int BS_MOST_BLOCKS = 340;
constexpr int RS_MOST_BLOCKS = 192;
constexpr size_t RS_MOST_PARTS = 1 << 20;  // floats: 4 MB
constexpr int RS_MOST_GROUPS = 65535;      // the groups are a grid's z

// Blocks of one kind per sample and slice when n_x rows are owned and ys waves share a row group.
static int rs_groups(int hw, int ys, int n_x) { return (n_x + rs_rows(hw, ys) - 1) / rs_rows(hw, ys); }

static RsAxis rs_axis(int hw, int ys, int n_x, int n_y) {
    RsAxis a;
    a.ys = ys;
    a.groups = rs_groups(hw, ys, n_x);
    a.y_tile = (RS_TILE / rs_rows(hw, ys) - RS_C) / RS_C * RS_C;
    const int n_y4 = (n_y + RS_C - 1) / RS_C * RS_C;
    if (a.y_tile > n_y4) a.y_tile = n_y4;
    return a;
}

// How a launch is cut, and what it is expected to take.
struct RsPlan {
    int hw;
    RsAxis ka, qa;
    float us;
};

// Expected time of a cut in microseconds: a block lives RS_BLOCK_US (launch, its trips to memory, its last reduction) plus
// RS_CHUNK_US per chunk that its waves walk one after the other, RS_ROUND blocks run at a time (half of them: a chunk
// takes half the time), and the launch takes as long as its longest block or as all blocks together.
static RsPlan rs_plan(const AttnShape &s) {
    RsPlan best{};
    for (int hw = 64; hw >= 16; hw /= 2) {
        const float per_group = (float)s.B * ((s.H + hw - 1) / hw);
        for (int ys = 1; ys <= RS_W; ys *= 2) {
            auto fit = [](int y, int n) {          // not more waves than chunks
                while (y > 1 && y * RS_C > n + RS_C - 1) y /= 2;
                return y;
            };
            RsPlan p;
            p.hw = hw;
            p.ka = rs_axis(hw, fit(ys, s.Tq), s.Tk, s.Tq);
            p.qa = rs_axis(hw, fit(ys, s.Tk), s.Tq, s.Tk);
            const float nk = per_group * p.ka.groups, nq = per_group * p.qa.groups;
            const float chunk = nk + nq <= RS_ROUND / 2 ? RS_CHUNK_US / 2 : RS_CHUNK_US;
            const float tk = RS_BLOCK_US + chunk * ((s.Tq + RS_C * p.ka.ys - 1) / (RS_C * p.ka.ys));
            const float tq = RS_BLOCK_US + chunk * ((s.Tk + RS_C * p.qa.ys - 1) / (RS_C * p.qa.ys));
            const float all = (nk * tk + nq * tq) / RS_ROUND, longest = tk > tq ? tk : tq;
            p.us = all > longest ? all : longest;
            if (best.hw == 0 || p.us < 0.95f * best.us) best = p;
        }
    }
    return best;
}

// Taken while recompute.hip's narrowest slices would leave a quarter of the compute units without a block (measured: at 192
// blocks the two forms meet, 10.7 against 11.6 us at B = 16, T = 40, H = 181; below it this one is ahead by up to 4 times,
// 53 -> 13 us at B = 3, T = 200, H = 76; above it evaluating every tanh twice loses).  Samples of hardly more than a key tile
// and a row per wave stay with the other form, which is then done before this one has exchanged its parts of dv (7.4
// against 9.5 us at B = 50, T = 9 / 15), and close to the limit those of up to 600 pairs do (T = 20, H = 32, B = 90, 180 blocks: 9.2
// against 10.2; ahead again at T = 30, H = 48, B = 60: 10.3 against 11.2).  Row counts whose groups no grid holds (B = 1, Tk = 32,
// H = 4: from 524 thousand rows on) stay with the other form, which walks them in passes.
bool recompute_split_applies(const AttnShape &s, size_t *part_floats, size_t *flag_words) {
    const long long blocks = (long long)s.B * ((s.H + 15) / 16), pairs = (long long)s.Tq * s.Tk;
    if (blocks > RS_MOST_BLOCKS || pairs <= (blocks > 160 ? 600 : 150)) return false;
    const RsPlan p = rs_plan(s);
    *part_floats = (size_t)s.B * p.ka.groups * s.H;
    *flag_words = (size_t)s.B * p.ka.groups * ((s.H + p.hw - 1) / p.hw);
    return *part_floats <= RS_MOST_PARTS && p.ka.groups + p.qa.groups <= RS_MOST_GROUPS;
}

template <typename T, int HW>
static hipError_t launch_split_t(const AttnShape &s, const RsPlan &p, const void *Qp, const void *Kp, const void *v, const int *order,
                                 const float *dS, float *dQp, float *dKp, float *parts, unsigned long long *flags, unsigned long long epoch,
                                 float *dv,
                                 hipStream_t st) {
    const RsAxis ka = p.ka;
    RsAxis qa = p.qa;
    if (!dQp) qa.groups = 0;
    dim3 grid((s.H + HW - 1) / HW, s.B, ka.groups + qa.groups);
    k_recompute_split<T, HW><<<grid, RS_THREADS, 0, st>>>((const T *)Qp, (const T *)Kp, (const T *)v, order, dS, dQp, dKp, parts, flags,
                                                          epoch, dv, s.Tq, s.Tk, s.H, ds_pitch(s.Tk), ka, qa, s.acc ? 1 : 0);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_split_hw(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order,
                                  const float *dS, float *dQp, float *dKp, float *parts, unsigned long long *flags, unsigned long long epoch,
                                  float *dv,
                                  hipStream_t st) {
    const RsPlan p = rs_plan(s);
    switch (p.hw) {
        case 16: return launch_split_t<T, 16>(s, p, Qp, Kp, v, order, dS, dQp, dKp, parts, flags, epoch, dv, st);
        case 32: return launch_split_t<T, 32>(s, p, Qp, Kp, v, order, dS, dQp, dKp, parts, flags, epoch, dv, st);
        default: return launch_split_t<T, 64>(s, p, Qp, Kp, v, order, dS, dQp, dKp, parts, flags, epoch, dv, st);
    }
}

hipError_t launch_recompute_split(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order,
                                  const float *dS, float *dQp, float *dKp, float *parts, unsigned long long *flags, unsigned long long epoch,
                                  float *dv,
                                  hipStream_t st) {
    return s.bf16 ? launch_split_hw<bf16_t>(s, Qp, Kp, v, order, dS, dQp, dKp, parts, flags, epoch, dv, st)
                  : launch_split_hw<float>(s, Qp, Kp, v, order, dS, dQp, dKp, parts, flags, epoch, dv, st);
}

// Taken for up to 64 query rows and keys while every block gets a compute unit of its own and what each block repeats, the dP of
// its sample, stays short: about 0.6 us per piece of columns plus the products (a tile takes 32 clocks per four columns on one
// of the four matrix cores).  A launch and the trips of dS through memory saved, together 4.9 + 6.4 -> 8.6 us at B = 4,
// T = 6 / 7, H = 16; 5.9 + 6.8 -> 9.2 at B = 1, T = 33 / 53, H = 48; 6.2 + 8.7 -> 12.1 at B = 10, T = 24, H = 256; 5.5 + 8.0 -> 9.3
// at B = 20, T = 16, H = 128 (340 blocks); level at B = 2, T = 20, H = 512; behind at B = 2, T = 64, Dv = 512 (14.9 -> 24) and
// at B = 16, T = 40, H = 181 (16 -> 23).  Past one block per compute unit only a third more than a round: 380 blocks at B = 38, T =
// 11, H = 224 lose (13.4 -> 15.3).
bool bwd_small_applies(const AttnShape &s, size_t *part_floats, size_t *flag_words) {
    if (s.Tq > BS_ROWS || s.Tk > BS_ROWS || s.B > BS_MOST_BLOCKS) return false;
    const RsPlan p = rs_plan(s);
    const int slices = (s.H + p.hw - 1) / p.hw;
    const long long blocks = (long long)s.B * ((s.Dv + 63) / 64 + (long long)slices * (p.ka.groups + p.qa.groups));
    const int rows = s.Tq > s.Tk ? s.Tq : s.Tk, tiles = ((s.Tq + 15) / 16) * ((s.Tk + 15) / 16);
    const int piece = rows <= 16 ? 256 : rows <= 32 ? 128 : 64;
    const float us = 0.6f * ((s.Dv + piece - 1) / piece) + 8.f / 2400 * tiles * (s.Dv / 4);
    if (!(blocks <= BS_ROUND ? us <= 3.5f : blocks <= BS_MOST_BLOCKS && us <= 1.2f)) return false;
    *part_floats = (size_t)s.B * p.ka.groups * s.H;
    *flag_words = (size_t)s.B * p.ka.groups * slices;
    return true;
}

template <typename T, int HW>
static hipError_t launch_small_t(const AttnShape &s, const RsPlan &p, const float *dC, const float *P, const void *V,
                                 const void *Qp, const void *Kp, const void *v, const int *key_len, float *dQp, float *dKp, float *dV,
                                 float *parts, unsigned long long *flags, unsigned long long epoch, float *dv, hipStream_t st) {
    const int slices = (s.H + HW - 1) / HW, dv_cols = (s.Dv + 63) / 64;
    dim3 grid(slices > dv_cols ? slices : dv_cols, s.B, 1 + p.ka.groups + p.qa.groups);
    k_bwd_small<T, HW><<<grid, RS_THREADS, 0, st>>>(dC, P, (const T *)V, (const T *)Qp, (const T *)Kp, (const T *)v, key_len, dQp,
                                                    dKp, dV, parts, flags, epoch, dv, s.Tq, s.Tk, s.H, s.Dv, p.ka, p.qa,
                                                    s.acc ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_bwd_small(const AttnShape &s, const float *dC, const float *P, const void *V, const void *Qp, const void *Kp,
                            const void *v, const int *key_len, float *dQp, float *dKp, float *dV, float *parts,
                            unsigned long long *flags, unsigned long long epoch, float *dv, hipStream_t st) {
    const RsPlan p = rs_plan(s);
#define ECHO_SMALL(T)                                                                                                         \
    switch (p.hw) {                                                                                                           \
        case 16: return launch_small_t<T, 16>(s, p, dC, P, V, Qp, Kp, v, key_len, dQp, dKp, dV, parts, flags, epoch, dv, st); \
        case 32: return launch_small_t<T, 32>(s, p, dC, P, V, Qp, Kp, v, key_len, dQp, dKp, dV, parts, flags, epoch, dv, st); \
        default: return launch_small_t<T, 64>(s, p, dC, P, V, Qp, Kp, v, key_len, dQp, dKp, dV, parts, flags, epoch, dv, st); \
    }
    if (s.bf16) {
        ECHO_SMALL(bf16_t)
    }
    ECHO_SMALL(float)
#undef ECHO_SMALL
}

}  // namespace echo
