// Backward pass of one decoder step (Section 2: the decoder produces one query at a time against the same
// encoder states) in ONE launch.  With a single query per sample every quantity of the backward pass except dv
// is local to the sample, so a block takes a sample through all of it:
//   dP[j]  = sum_d dC[d] V[j,d]                      (Eq. 2: from the inputs alone)
//   dS[j]  = P[j] (dP[j] - sum_j P dP)
//   t      = tanh(q[h] + k[j,h]) re-evaluated        (Section 3.4)
//   dQp[h] = v[h] sum_j dS[j] (1 - t^2),   dKp[j,h] += v[h] dS[j] (1 - t^2),   dV[j,:] += P[j] dC
//   dv_part[b,h] += sum_j dS[j] t                    (per sample; summed over the samples once per sentence)
// One launch instead of three.  What bounds a step is memory, not arithmetic: every step reads K and V of the
// valid keys and reads and writes the whole dKp and dV accumulators (23 MB at 64 sentences of 30 keys, H = Dv =
// 512), traffic that the batched call pays once for all steps.  The sum over samples that dv needs is deferred to
// one small launch at the end of the sentence.  Results do not depend on the order in which blocks run: every
// element has one owner.
#include "common.hpp"
#include "kernels.hpp"

namespace echo {

__device__ __forceinline__ float comp4(const float4 &x, int c) { return c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w; }

constexpr int ST_W = 8;                   // waves per block
constexpr int ST_THREADS = 64 * ST_W;
constexpr int ST_KB = 4;                  // keys per wave and batch: a batch of the block is 32 consecutive keys

// Block = (sample b, 64-wide slice of h); it also owns the matching slice of the columns of dV.  Wave w takes
// keys 32 n + 4 w .. + 3 of every batch n; the first batch's K, old dKp and old dV are requested before dP is
// formed.  dP is formed by every h slice of a sample for itself (a few ten thousand multiply-adds, V comes from
// the L2 that the slices of a sample share).
//
// DEFER: the key-side sums are left to one batched call at the end of the sentence.  The step then only reads: it
// writes dQp, and the block of the first h slice writes the step's row of dS (row `ds_row` of the sample's
// `ds_rows` rows of `ds_pitch` floats, zeros at masked keys and pads) and its sum; dKp, dV and dv_part are not
// touched.
template <typename T, bool DEFER>
__global__ __launch_bounds__(ST_THREADS) void k_step_bwd(
    const float *__restrict__ dC, const float *__restrict__ P, const T *__restrict__ Qp, const T *__restrict__ Kp,
    const T *__restrict__ V, const T *__restrict__ v, const int *__restrict__ key_len, float *__restrict__ dQp,
    float *__restrict__ dKp, float *__restrict__ dV, float *__restrict__ dv_part, float *__restrict__ ds_out,
    float *__restrict__ ds_sum_out, int ds_rows, int ds_row, int ds_pitch, int Tk, int H, int Dv, int cw) {
    extern __shared__ float s_step[];     // [Tk] P, then [Tk] dP
    float *s_p = s_step, *s_dp = s_step + Tk;
    __shared__ float s_q[ST_W][64], s_r[ST_W][64];
    const int hs = blockIdx.x, b = blockIdx.y;
    const int lane = lane_id(), w = wave_id();
    const int h = hs * 64 + lane;
    const bool hv = h < H;
    const int hc = hv ? h : H - 1;
    const int L = clamp_len(key_len[b], Tk);
    float *ds_dst = DEFER ? ds_out + ((size_t)b * ds_rows + ds_row) * ds_pitch : nullptr;
    if (DEFER && hs == 0) {               // masked keys and pads of the stored dS row: zeros
        for (int j = L + (int)threadIdx.x; j < ds_pitch; j += ST_THREADS) ds_dst[j] = 0.f;
        if (L == 0 && threadIdx.x == 0) ds_sum_out[(size_t)b * ds_rows + ds_row] = 0.f;
    }
    if (L == 0) {                         // no valid key: the query gets no gradient, the sums get nothing
        if (w == 0 && hv) dQp[(size_t)b * H + h] = 0.f;
        return;
    }
    const float *dCb = dC + (size_t)b * Dv;
    const float *Pb = P + (size_t)b * Tk;
    const T *Vb = V + (size_t)b * Tk * Dv;
    const T *Kb = Kp + (size_t)b * Tk * H;
    float *dKb = dKp + (size_t)b * Tk * H;
    float *dVb = dV + (size_t)b * Tk * Dv;
    const int c_lo = hs * cw, c_hi = min(c_lo + cw, Dv);         // this block's columns of dV
    const int n_batch = (L + 8 * ST_KB - 1) / (8 * ST_KB);

    // ---- requests of the first batch: K and old dKp at this lane's h, old dV at this lane's first column
    float k0[ST_KB], oldk0[ST_KB], oldv0[ST_KB];
    const int c0 = min(c_lo + lane, Dv - 1);
#pragma unroll
    for (int u = 0; u < ST_KB; ++u) {
        const int j = min(ST_KB * w + u, L - 1);
        k0[u] = ld(Kb, (size_t)j * H + hc);
        oldk0[u] = DEFER ? 0.f : dKb[(size_t)j * H + hc];
        oldv0[u] = DEFER ? 0.f : dVb[(size_t)j * Dv + c0];
    }
    const float sq = kTwoLog2e * ld(Qp, (size_t)b * H + hc);
    float v_raw = ld(v, (size_t)hc);     // scaled behind the barrier below: as a guarded load with its scaling it was
                                         // awaited on the spot, before the loads of the dP loop had been requested

    // ---- dP[j] = sum_d dC[d] V[j,d] for this wave's keys of every batch; P to LDS (its first ST_THREADS entries are
    //      requested here and stored behind the loop: stored at once, they were a trip to memory that the loads of the
    //      loop had to wait for)
    const int jp = min((int)threadIdx.x, L - 1);
    const float p_first = Pb[jp];
    for (int n = 0; n < n_batch; ++n) {
        const int j0 = 8 * ST_KB * n + ST_KB * w;
        if (j0 >= L) break;                                       // wave-uniform
        float acc[ST_KB] = {0.f, 0.f, 0.f, 0.f};
        for (int d = 4 * lane; d < Dv; d += 256) {
            const float4 c = ld4(dCb, (size_t)d);
            float4 x[ST_KB];
#pragma unroll
            for (int u = 0; u < ST_KB; ++u) x[u] = ld4(Vb, (size_t)min(j0 + u, L - 1) * Dv + d);
#pragma unroll
            for (int u = 0; u < ST_KB; ++u)
                acc[u] += (c.x * x[u].x + c.y * x[u].y) + (c.z * x[u].z + c.w * x[u].w);
        }
#pragma unroll
        for (int u = 0; u < ST_KB; ++u) {
            const float tot = wave_sum(acc[u]);
            if (lane == 0 && j0 + u < L) s_dp[j0 + u] = tot;
        }
    }
    if ((int)threadIdx.x < L) s_p[threadIdx.x] = p_first;
    for (int j = threadIdx.x + ST_THREADS; j < L; j += ST_THREADS) s_p[j] = Pb[j];
    __syncthreads();
    asm volatile("" : "+v"(v_raw));
    const float v4 = hv ? 4.f * v_raw : 0.f;

    // ---- the two row sums, formed by every wave for itself (same arithmetic, same result in all waves)
    float r = 0.f;
    for (int j = lane; j < L; j += 64) r += s_p[j] * s_dp[j];
    r = wave_sum(r);
    float dsum = 0.f;
    for (int j = lane; j < L; j += 64) dsum += s_p[j] * (s_dp[j] - r);
    dsum = wave_sum(dsum);                // sum_j dS[j]: zero in exact arithmetic; kept so that sum dS t is exact in fp32

    // ---- recomputation at (this wave's keys, this lane's h):  r' = 1 / (exp(2 (q + k)) + 1),
    //      t = 1 - 2 r',  1 - t^2 = 4 r' (1 - r');  and dV at this lane's columns
    float accQ = 0.f, accR = 0.f;
    for (int n = 0; n < n_batch; ++n) {
        const int j0 = 8 * ST_KB * n + ST_KB * w;
        if (j0 >= L) break;                                       // wave-uniform
        float k[ST_KB], oldk[ST_KB];
#pragma unroll
        for (int u = 0; u < ST_KB; ++u) {
            if (n == 0) {
                k[u] = k0[u];
                oldk[u] = oldk0[u];
            } else {
                const size_t at = (size_t)min(j0 + u, L - 1) * H + hc;
                k[u] = ld(Kb, at);
                oldk[u] = DEFER ? 0.f : dKb[at];
            }
        }
#pragma unroll
        for (int u = 0; u < ST_KB; ++u) {
            if (j0 + u < L) {                                     // wave-uniform
                const float ds = s_p[j0 + u] * (s_dp[j0 + u] - r);
                const float rr = fast_rcp(fast_exp2(__builtin_fmaf(kTwoLog2e, k[u], sq)) + 1.0f);
                const float g = ds * __builtin_fmaf(-rr, rr, rr);
                accQ += g;
                accR = __builtin_fmaf(ds, rr, accR);
                if (!DEFER && hv) store_streaming(&dKb[(size_t)(j0 + u) * H + h], __builtin_fmaf(v4, g, oldk[u]));
                if (DEFER && hs == 0 && lane == 0) ds_dst[j0 + u] = ds;
            }
        }
        for (int c = c_lo + lane, m = 0; !DEFER && c < c_hi; c += 64, ++m) {
            const float dc = dCb[c];
#pragma unroll
            for (int u = 0; u < ST_KB; ++u) {
                if (j0 + u < L) {
                    float *at = dVb + (size_t)(j0 + u) * Dv + c;
                    const float old = (n == 0 && m == 0) ? oldv0[u] : *at;
                    store_streaming(at, __builtin_fmaf(s_p[j0 + u], dc, old));
                }
            }
        }
    }
    s_q[w][lane] = accQ;
    s_r[w][lane] = accR;
    __syncthreads();
    if (w == 0 && hv) {
        float tq = 0.f, tr = 0.f;
#pragma unroll
        for (int k2 = 0; k2 < ST_W; ++k2) {
            tq += s_q[k2][lane];
            tr += s_r[k2][lane];
        }
        store_streaming(&dQp[(size_t)b * H + h], v4 * tq);
        if (!DEFER) {
            float *dvp = dv_part + (size_t)b * H + h;
            *dvp += __builtin_fmaf(-2.f, tr, dsum);
        } else if (hs == 0 && lane == 0) {
            ds_sum_out[(size_t)b * ds_rows + ds_row] = dsum;
        }
    }
}

// Forward pass of one decoder step in one block of eight waves per sample, for steps of few keys (see step_fwd_takes_rows): scores
// with the eight waves taking four keys each per batch and the lanes along h, softmax over the valid keys, context with a thread
// per column.  tanh is taken from the exponential of the sum here (one exponential and one reciprocal per
// element): a step is a few thousand elements per wave, nothing to save by factoring it.
template <typename T>
__global__ __launch_bounds__(ST_THREADS) void k_step_fwd_rows(
    const T *__restrict__ Qp, const T *__restrict__ Kp, const T *__restrict__ V, const T *__restrict__ v,
    const int *__restrict__ key_len, float *__restrict__ C, float *__restrict__ P, int Tk, int H, int Dv) {
    extern __shared__ float s_step[];     // [Tk] scores, then probabilities
    float *s_s = s_step;
    const int b = blockIdx.x;
    const int lane = lane_id(), w = wave_id();
    const int L = clamp_len(key_len[b], Tk);
    float *Pb = P + (size_t)b * Tk;
    float *Cb = C + (size_t)b * Dv;
    if (L == 0) {                         // no valid key: zeros
        for (int j = threadIdx.x; j < Tk; j += ST_THREADS) Pb[j] = 0.f;
        for (int d = threadIdx.x; d < Dv; d += ST_THREADS) Cb[d] = 0.f;
        return;
    }
    const T *qb = Qp + (size_t)b * H;
    const T *Kb = Kp + (size_t)b * Tk * H;
    const T *Vb = V + (size_t)b * Tk * Dv;
    const int n_batch = (L + 8 * ST_KB - 1) / (8 * ST_KB);
    const int H4 = (H % 4 == 0) ? H : 0;  // rows are read four elements at a time when every row starts aligned

    // ---- scores: S[j] = sum_h v[h] tanh(q[h] + k[j,h]),  tanh = 1 - 2 / (exp(2 (q + k)) + 1)
    for (int n = 0; n < n_batch; ++n) {
        const int j0 = 8 * ST_KB * n + ST_KB * w;
        float acc[ST_KB] = {0.f, 0.f, 0.f, 0.f};
        if (j0 < L) {                                             // wave-uniform
            for (int h = 4 * lane; h < H4; h += 256) {
                const float4 q4 = ld4(qb, (size_t)h), v4 = ld4(v, (size_t)h);
                float4 k4[ST_KB];
#pragma unroll
                for (int u = 0; u < ST_KB; ++u) k4[u] = ld4(Kb, (size_t)min(j0 + u, L - 1) * H + h);
#pragma unroll
                for (int u = 0; u < ST_KB; ++u) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x = kTwoLog2e * (comp4(q4, c) + comp4(k4[u], c));
                        acc[u] += comp4(v4, c) * __builtin_fmaf(-2.f, fast_rcp(fast_exp2(x) + 1.0f), 1.0f);
                    }
                }
            }
            for (int h = H4 + lane; h < H; h += 64) {             // rows that do not start aligned: one element at a time
                const float qh = ld(qb, (size_t)h), vh = ld(v, (size_t)h);
#pragma unroll
                for (int u = 0; u < ST_KB; ++u) {
                    const float x = kTwoLog2e * (qh + ld(Kb, (size_t)min(j0 + u, L - 1) * H + h));
                    acc[u] += vh * __builtin_fmaf(-2.f, fast_rcp(fast_exp2(x) + 1.0f), 1.0f);
                }
            }
#pragma unroll
            for (int u = 0; u < ST_KB; ++u) {
                const float tot = wave_sum(acc[u]);
                if (lane == 0 && j0 + u < L) s_s[j0 + u] = tot;
            }
        }
    }
    lds_barrier();

    // ---- softmax over the valid keys: every wave forms the maximum and the sum itself (same arithmetic in all)
    float mx = -INFINITY;
    for (int j = lane; j < L; j += 64) mx = fmaxf(mx, s_s[j]);
    mx = wave_max(mx);
    float z = 0.f;
    for (int j = lane; j < L; j += 64) z += fast_exp2((s_s[j] - mx) * 1.4426950408889634f);
    z = wave_sum(z);
    const float inv = 1.0f / z;
    lds_barrier();
    for (int j = threadIdx.x; j < Tk; j += ST_THREADS) {
        const float p = j < L ? fast_exp2((s_s[j] - mx) * 1.4426950408889634f) * inv : 0.f;
        if (j < L) s_s[j] = p;
        store_streaming(&Pb[j], p);
    }
    lds_barrier();

    // ---- context: a thread per column, eight value rows in flight
    for (int d = threadIdx.x; d < Dv; d += ST_THREADS) {
        float acc = 0.f;
        for (int j0 = 0; j0 < L; j0 += 8) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = ld(Vb, (size_t)min(j0 + u, L - 1) * Dv + d);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (j0 + u < L) acc = __builtin_fmaf(s_s[j0 + u], x[u], acc);
        }
        store_streaming(&Cb[d], acc);
    }
}

// ---- one block of sixteen waves per sample: forward, and the query side of the backward ------------------------------
//
// What bounds these is the rate at which one CU draws a sample's rows (about 100 KB/us when enough whole-row loads are under
// way), so a wave loads whole pieces of rows (64 lanes x 16 bytes), 16 waves x 8 loads make a batch (64 rows x 512 columns), and
// two batches are under way: where one batch holds a sample's keys and one its values (ONE), all rows of the step are
// requested before anything is evaluated, else two batches of keys at a time, and the first two of the second half of the
// step (V forward, K backward) before the softmax in between.  Both passes have the same frame: a value per key from the rows of one matrix (score from K,
// dP from V), a step on the row of values (softmax, its backward), then sums over the keys into columns (context from V, dQp
// from K), which the waves form for their rows and add up in LDS.
// (With eight waves, four keys at a time and a thread per column, one trip to memory after the other, a step of 80 samples,
// 100 keys, H = Dv = 512 took 20 us; this takes 9.1.  64 samples of 50 keys: 8.0 with a column's values in registers, 6.6.)
constexpr int SB_W = 16;                  // waves
constexpr int SB_THREADS = 64 * SB_W;
constexpr int SB_U = 4;                   // rows per wave and batch: row w + 16 u
constexpr int SB_ROWS = SB_W * SB_U;
constexpr int SB_C = 2;                   // 256-wide chunks of columns per batch
constexpr int SB_COLS = 256 * SB_C;

// Where the group of four columns that belongs at `col` is loaded from (NARROW: rows of fewer than four elements).
template <bool NARROW> __device__ __forceinline__ int piece_at(int width, int col) { return NARROW ? col : min(col, width - 4); }

// A batch of a wave's rows: rows j0 + w + 16 u below L, columns c0 + 256 c + 4 lane.  Groups of four that reach past the width
// are loaded as the row's last four; chunks from `end` on are not loaded.  Row and chunk are scalars, the lane's place a small
// offset to them.
template <typename T> struct RowBatch {
    RawKey<T> x[SB_C][SB_U];
    template <bool NARROW>
    __device__ __forceinline__ void load(const T *base, int width, int end, int L, int j0, int c0, int lane, int w) {
        const int back = c0 > 0 ? 4 : 0;  // so that no offset is negative
        unsigned off[SB_C];
#pragma unroll
        for (int c = 0; c < SB_C; ++c)
            off[c] = (unsigned)min(256 * c + 4 * lane + back, width - 4 - c0 + back) * (unsigned)sizeof(T);
        const T *first = base + (c0 - back);
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            const int j = j0 + w + SB_W * u;
            if (j < L) {                                          // uniform
                const T *row = first + (size_t)j * width;
#pragma unroll
                for (int c = 0; c < SB_C; ++c) {
                    if (c0 + 256 * c >= end) x[c][u].zero();      // uniform
                    else if (NARROW) x[c][u].load_some(row, width - 4 * lane);
                    else x[c][u].load(reinterpret_cast<const T *>(reinterpret_cast<const char *>(row) + off[c]), 0);
                }
            } else {
#pragma unroll
                for (int c = 0; c < SB_C; ++c) x[c][u].zero();
            }
        }
    }
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int c = 0; c < SB_C; ++c)
#pragma unroll
            for (int u = 0; u < SB_U; ++u) x[c][u].pin();
    }
};
// Walks the rows of one matrix in batches: all chunks of columns of 64 rows before the next 64 (ROWS_OUTER), or all rows of a
// chunk of columns before the next chunk.  The same in all lanes.
template <bool ROWS_OUTER> struct Walk {
    int begin, width, L, j, c;            // columns begin .. width - 1
    __device__ __forceinline__ Walk(int begin_, int width_, int L_) : begin(begin_), width(width_), L(L_), j(0), c(begin_) {}
    __device__ __forceinline__ Walk after() const {
        Walk n = *this;
        n.next();
        return n;
    }
    __device__ __forceinline__ bool more() const { return ROWS_OUTER ? j < L : c < width; }
    __device__ __forceinline__ void next() {
        if (ROWS_OUTER) {
            c += SB_COLS;
            if (c >= width) {
                c = begin;
                j += SB_ROWS;
            }
        } else {
            j += SB_ROWS;
            if (j >= L) {
                j = 0;
                c += SB_COLS;
            }
        }
    }
};

// Four columns of a vector at c0 + 256 c + 4 lane; columns past the width, and those that a last group loaded as the row's last
// four repeats, are zero if `masked`.
template <bool NARROW, typename T>
__device__ __forceinline__ float4 vec_piece(const T *p, int width, int col, bool masked) {
    const int at = piece_at<NARROW>(width, col);
    RawKey<T> raw;
    if (NARROW) raw.load_some(p, width - col);
    else raw.load(p, (size_t)(unsigned)at);
    float4 r = raw.get();
    if (masked) {
        if (at + 0 < col) r.x = 0.f;
        if (at + 1 < col) r.y = 0.f;
        if (at + 2 < col) r.z = 0.f;
        if (at + 3 < col) r.w = 0.f;
    }
    return r;
}

// Partial sums of the waves, [wave][column of the chunk], added in wave order: column t of thread t < SB_COLS.
__device__ __forceinline__ float sum_over_waves(float (&s_part)[SB_W][SB_COLS], const float4 (&acc)[SB_C], int lane, int w) {
    lds_barrier();                                                // the previous use of s_part is over
#pragma unroll
    for (int c = 0; c < SB_C; ++c) *reinterpret_cast<float4 *>(&s_part[w][256 * c + 4 * lane]) = acc[c];
    lds_barrier();
    float tot = 0.f;
    if (threadIdx.x < SB_COLS) {
#pragma unroll
        for (int k = 0; k < SB_W; ++k) tot += s_part[k][threadIdx.x];
    }
    return tot;
}

// Forward: S[j] = sum_h v[h] tanh(q[h] + k[j,h]), tanh = 1 - 2 / (exp(2 (q + k)) + 1).  One exponential and one reciprocal per
// element: nothing to save by factoring when every key meets one query.  The exponent is taken from q + k, so that its rounding
// error follows the sum and not the operands where these cancel, and the terms v tanh are summed, not v / (exp(2 (q + k)) + 1),
// whose partial sums stay large where the tanh terms are small.
template <typename T, bool NARROW, bool ONE>
__global__ __launch_bounds__(SB_THREADS) void k_step_fwd(
    const T *__restrict__ Qp, const T *__restrict__ Kp, const T *__restrict__ V, const T *__restrict__ v,
    const int *__restrict__ key_len, float *__restrict__ C, float *__restrict__ P, int Tk, int H, int Dv, int part) {
    extern __shared__ float s_step[];     // [Tk] scores, then probabilities
    float *s_s = s_step;
    __shared__ __align__(16) float s_part[SB_W][SB_COLS];
    const int b = blockIdx.x;
    const int lane = lane_id(), w = wave_id();
    const int L = clamp_len(key_len[b], Tk);
    float *Pb = P + (size_t)b * Tk;
    float *Cb = C + (size_t)b * Dv;
    if (L == 0) {                         // no valid key: zeros
        if (blockIdx.y > 0) return;
        for (int j = threadIdx.x; j < Tk; j += SB_THREADS) Pb[j] = 0.f;
        for (int d = threadIdx.x; d < Dv; d += SB_THREADS) Cb[d] = 0.f;
        return;
    }
    const T *qb = Qp + (size_t)b * H;
    const T *Kb = Kp + (size_t)b * Tk * H;
    const T *Vb = V + (size_t)b * Tk * Dv;
    // two batches at a time: of the first matrix, or (ONE: each matrix is a single batch) one of both
    RowBatch<T> x[2];
    const int d_lo = blockIdx.y * part, d_hi = min(d_lo + part, Dv);     // this block's columns of the context
    Walk<true> kw(0, H, L);
    Walk<false> vw(d_lo, d_hi, L);
    auto load_keys = [&](RowBatch<T> &r, const Walk<true> &at) {
        if (at.more()) r.template load<NARROW>(Kb, H, H, L, at.j, at.c, lane, w);
    };
    auto load_values = [&](RowBatch<T> &r, const Walk<false> &at) {
        if (at.more()) r.template load<false>(Vb, Dv, d_hi, L, at.j, at.c, lane, w);
    };
    if (ONE) load_keys(x[0], kw);
    float4 q4[SB_C], v4[SB_C];
    auto load_qv = [&](int h0) {
#pragma unroll
        for (int c = 0; c < SB_C; ++c) {
            q4[c] = vec_piece<NARROW>(qb, H, h0 + 256 * c + 4 * lane, false);
            v4[c] = vec_piece<NARROW>(v, H, h0 + 256 * c + 4 * lane, true);
        }
    };
    load_qv(0);
    if (ONE) load_values(x[1], vw);

    float acc[SB_U];
    auto scores = [&](RowBatch<T> &kx, int j0, int h0) {
        if (h0 == 0) {
#pragma unroll
            for (int u = 0; u < SB_U; ++u) acc[u] = 0.f;
        }
        if (H > SB_COLS && (j0 > 0 || h0 > 0)) load_qv(h0);
        kx.pin();
#pragma unroll
        for (int c = 0; c < SB_C; ++c) {
            if (h0 + 256 * c >= H) continue;                      // uniform
#pragma unroll
            for (int u = 0; u < SB_U; ++u) {
                if (j0 + w + SB_W * u >= L) continue;             // uniform
                const float4 k4 = kx.x[c][u].get();
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = kTwoLog2e * (comp4(q4[c], e) + comp4(k4, e));
                    acc[u] = __builtin_fmaf(comp4(v4[c], e), __builtin_fmaf(-2.f, fast_rcp(fast_exp2(x) + 1.0f), 1.0f), acc[u]);
                }
            }
        }
        if (h0 + SB_COLS >= H) {                                  // the scores of these rows are complete
            const float tot = wave_transpose_sum<SB_U>(acc);      // key u in lanes 16 u ..
            const int j = j0 + w + SB_W * (lane >> 4);
            if ((lane & 15) == 0 && j < L) s_s[j] = tot;
        }
    };
    if (ONE) {
        scores(x[0], 0, 0);
    } else {
        while (kw.more()) {
            load_keys(x[0], kw);
            load_keys(x[1], kw.after());
            scores(x[0], kw.j, kw.c);
            kw.next();
            if (kw.more()) scores(x[1], kw.j, kw.c);
            kw.next();
        }
        load_values(x[0], vw);
        load_values(x[1], vw.after());
    }
    lds_barrier();

    // ---- softmax over the valid keys: every wave forms the maximum and the sum itself (same arithmetic in all)
    float mx = -INFINITY;
    for (int j = lane; j < L; j += 64) mx = fmaxf(mx, s_s[j]);
    mx = wave_max(mx);
    float z = 0.f;
    for (int j = lane; j < L; j += 64) z += fast_exp2((s_s[j] - mx) * 1.4426950408889634f);
    z = wave_sum(z);
    const float inv = 1.0f / z;
    lds_barrier();
    for (int j = threadIdx.x; j < Tk; j += SB_THREADS) {
        const float p = j < L ? fast_exp2((s_s[j] - mx) * 1.4426950408889634f) * inv : 0.f;
        if (j < L) s_s[j] = p;
        if (blockIdx.y == 0) store_streaming(&Pb[j], p);
    }
    lds_barrier();

    // ---- context
    float4 accC[SB_C];
    auto context = [&](RowBatch<T> &vx, int j0, int d0) {
        if (j0 == 0) {
#pragma unroll
            for (int c = 0; c < SB_C; ++c) accC[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        vx.pin();
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            if (j0 + w + SB_W * u >= L) continue;                 // uniform
            const float p = s_s[j0 + w + SB_W * u];
#pragma unroll
            for (int c = 0; c < SB_C; ++c) {
                const float4 x = vx.x[c][u].get();
                accC[c].x = __builtin_fmaf(p, x.x, accC[c].x);
                accC[c].y = __builtin_fmaf(p, x.y, accC[c].y);
                accC[c].z = __builtin_fmaf(p, x.z, accC[c].z);
                accC[c].w = __builtin_fmaf(p, x.w, accC[c].w);
            }
        }
        if (j0 + SB_ROWS >= L) {
            const float tot = sum_over_waves(s_part, accC, lane, w);
            const int d = d0 + (int)threadIdx.x;
            if (threadIdx.x < SB_COLS && d < d_hi) store_streaming(&Cb[d], tot);
        }
    };
    if (ONE) {
        context(x[1], 0, d_lo);
        return;
    }
    for (;;) {
        context(x[0], vw.j, vw.c);
        vw.next();
        if (vw.more()) context(x[1], vw.j, vw.c);
        vw.next();
        if (!vw.more()) break;
        load_values(x[0], vw);
        load_values(x[1], vw.after());
    }
}

// The query side of the backward step: dP[j] = sum_d dC[d] V[j,d], dS = P (dP - sum_j P dP), dQp[h] = v[h] sum_j dS (1 - t^2) with
// t re-evaluated (1 - t^2 = 4 r (1 - r)).  Also leaves the step's row of dS (row `ds_row` of the sample's `ds_rows` rows of
// `ds_pitch` floats, zeros at masked keys and pads) and its sum.
template <typename T, bool ONE>
__global__ __launch_bounds__(SB_THREADS) void k_step_bwd_query(
    const float *__restrict__ dC, const float *__restrict__ P, const T *__restrict__ Qp, const T *__restrict__ Kp,
    const T *__restrict__ V, const T *__restrict__ v, const int *__restrict__ key_len, float *__restrict__ dQp,
    float *__restrict__ ds_out, float *__restrict__ ds_sum_out, int ds_rows, int ds_row, int ds_pitch, int Tk, int H, int Dv,
    int part) {
    extern __shared__ float s_step[];     // [Tk] P, then [Tk] dP, later dS
    float *s_p = s_step, *s_dp = s_step + Tk;
    __shared__ __align__(16) float s_part[SB_W][SB_COLS];
    const int b = blockIdx.x;
    const int lane = lane_id(), w = wave_id();
    const int L = clamp_len(key_len[b], Tk);
    float *ds_dst = ds_out + ((size_t)b * ds_rows + ds_row) * ds_pitch;
    const bool first = blockIdx.y == 0;   // of the sample's blocks: it leaves the row of dS
    if (!first && L == 0) return;
    if (first)
        for (int j = L + (int)threadIdx.x; j < ds_pitch; j += SB_THREADS) ds_dst[j] = 0.f;
    if (L == 0) {                         // no valid key: the query gets no gradient
        if (threadIdx.x == 0) ds_sum_out[(size_t)b * ds_rows + ds_row] = 0.f;
        for (int h = threadIdx.x; h < H; h += SB_THREADS) dQp[(size_t)b * H + h] = 0.f;
        return;
    }
    const float *dCb = dC + (size_t)b * Dv;
    const float *Pb = P + (size_t)b * Tk;
    const T *qb = Qp + (size_t)b * H;
    const T *Kb = Kp + (size_t)b * Tk * H;
    const T *Vb = V + (size_t)b * Tk * Dv;
    RowBatch<T> x[2];                     // see k_step_fwd
    const int h_lo = blockIdx.y * part, h_hi = min(h_lo + part, H);      // this block's part of dQp
    Walk<true> vw(0, Dv, L);
    Walk<false> kw(h_lo, h_hi, L);
    auto load_values = [&](RowBatch<T> &r, const Walk<true> &at) {
        if (at.more()) r.template load<false>(Vb, Dv, Dv, L, at.j, at.c, lane, w);
    };
    auto load_keys = [&](RowBatch<T> &r, const Walk<false> &at) {
        if (at.more()) r.template load<false>(Kb, H, h_hi, L, at.j, at.c, lane, w);
    };
    if (ONE) load_values(x[0], vw);
    float4 c4[SB_C], q4[SB_C];
    auto load_dc = [&](int d0) {
#pragma unroll
        for (int c = 0; c < SB_C; ++c) c4[c] = vec_piece<false>(dCb, Dv, d0 + 256 * c + 4 * lane, true);
    };
    auto load_q = [&](int h0) {
#pragma unroll
        for (int c = 0; c < SB_C; ++c) q4[c] = vec_piece<false>(qb, H, h0 + 256 * c + 4 * lane, false);
    };
    load_dc(0);
    const float p_first = Pb[min((int)threadIdx.x, L - 1)];
    load_q(h_lo);
    if (ONE) load_keys(x[1], kw);

    float acc[SB_U];
    auto dots = [&](RowBatch<T> &vx, int j0, int d0) {
        if (d0 == 0) {
#pragma unroll
            for (int u = 0; u < SB_U; ++u) acc[u] = 0.f;
        }
        if (Dv > SB_COLS && (j0 > 0 || d0 > 0)) load_dc(d0);
        vx.pin();
#pragma unroll
        for (int c = 0; c < SB_C; ++c)
#pragma unroll
            for (int u = 0; u < SB_U; ++u) {
                const float4 x = vx.x[c][u].get();
                acc[u] += (c4[c].x * x.x + c4[c].y * x.y) + (c4[c].z * x.z + c4[c].w * x.w);
            }
        if (d0 + SB_COLS >= Dv) {
            const float tot = wave_transpose_sum<SB_U>(acc);
            const int j = j0 + w + SB_W * (lane >> 4);
            if ((lane & 15) == 0 && j < L) s_dp[j] = tot;
        }
    };
    if (ONE) {
        dots(x[0], 0, 0);
    } else {
        while (vw.more()) {
            load_values(x[0], vw);
            load_values(x[1], vw.after());
            dots(x[0], vw.j, vw.c);
            vw.next();
            if (vw.more()) dots(x[1], vw.j, vw.c);
            vw.next();
        }
        load_keys(x[0], kw);
        load_keys(x[1], kw.after());
    }
    if ((int)threadIdx.x < L) s_p[threadIdx.x] = p_first;
    for (int j = threadIdx.x + SB_THREADS; j < L; j += SB_THREADS) s_p[j] = Pb[j];
    __syncthreads();

    // ---- the row sums, formed by every wave for itself (same arithmetic, same result in all waves)
    float r = 0.f;
    for (int j = lane; j < L; j += 64) r += s_p[j] * s_dp[j];
    r = wave_sum(r);
    float dsum = 0.f;
    for (int j = lane; j < L; j += 64) dsum += s_p[j] * (s_dp[j] - r);
    dsum = wave_sum(dsum);                // zero in exact arithmetic; kept so that the key-side sums are exact in fp32
    lds_barrier();
    for (int j = threadIdx.x; j < L; j += SB_THREADS) {
        const float ds = s_p[j] * (s_dp[j] - r);
        s_dp[j] = ds;
        if (first) ds_dst[j] = ds;
    }
    if (first && threadIdx.x == 0) ds_sum_out[(size_t)b * ds_rows + ds_row] = dsum;
    lds_barrier();

    float4 accQ[SB_C];
    auto query = [&](RowBatch<T> &kx, int j0, int h0) {
        if (j0 == 0) {
            if (h0 > h_lo) load_q(h0);
#pragma unroll
            for (int c = 0; c < SB_C; ++c) accQ[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        kx.pin();
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            if (j0 + w + SB_W * u >= L) continue;                 // uniform
            const float ds = s_dp[j0 + w + SB_W * u];
#pragma unroll
            for (int c = 0; c < SB_C; ++c) {
                if (h0 + 256 * c >= h_hi) continue;               // uniform
                const float4 k4 = kx.x[c][u].get();
                float g[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float rr = fast_rcp(fast_exp2(__builtin_fmaf(kTwoLog2e, comp4(k4, e), kTwoLog2e * comp4(q4[c], e))) + 1.0f);
                    g[e] = ds * __builtin_fmaf(-rr, rr, rr);
                }
                accQ[c].x += g[0];
                accQ[c].y += g[1];
                accQ[c].z += g[2];
                accQ[c].w += g[3];
            }
        }
        if (j0 + SB_ROWS >= L) {
            const float tot = sum_over_waves(s_part, accQ, lane, w);
            // thread t holds the sum of the lane that loaded column piece_at(4 (t / 4)) + t % 4 of this chunk: a last group of
            // fewer than four columns lies further right than its place
            const int g4 = h0 + ((int)threadIdx.x & ~3), h = piece_at<false>(H, g4) + ((int)threadIdx.x & 3);
            if (threadIdx.x < SB_COLS && g4 < h_hi && h >= g4 && h < H)
                store_streaming(&dQp[(size_t)b * H + h], 4.f * ld(v, (size_t)h) * tot);
        }
    };
    if (ONE) {
        query(x[1], 0, h_lo);
        return;
    }
    for (;;) {
        query(x[0], kw.j, kw.c);
        kw.next();
        if (kw.more()) query(x[1], kw.j, kw.c);
        kw.next();
        if (!kw.more()) break;
        load_keys(x[0], kw);
        load_keys(x[1], kw.after());
    }
}

// Blocks per sample: while the chip has room, the columns that the second half of the step sums into are split in parts of
// whole multiples of `unit`; every block of a sample forms the values per key for itself.  256 columns where the second half
// re-evaluates tanh (7.0 -> 6.0 us at 100 samples of 50 keys, H = 512; 18.3 -> 11.1 at 2 of 128, H = 1024), 512 for the context,
// which 256 slowed down (9.0 -> 9.6 us at 80 samples of 100 keys).
static int step_parts(int B, int width, int unit) {
    const int units = (width + unit - 1) / unit, room = 256 / B;
    return room < 2 || units < 2 ? 1 : (room < units ? room : units);
}
static int step_part_width(int width, int unit, int parts) { return ((width + unit - 1) / unit + parts - 1) / parts * unit; }
static bool step_one_batch(const AttnShape &s) { return s.Tk <= SB_ROWS && s.H <= SB_COLS && s.Dv <= SB_COLS; }
constexpr size_t SB_MOST_LDS = 64 * 1024;     // next to the 32 KB in which the waves' sums meet

template <typename T, bool NARROW, bool ONE>
static hipError_t launch_step_fwd_t(const AttnShape &s, size_t lds, const void *Qp, const void *Kp, const void *V, const void *v,
                                    const int *key_len, float *C, float *P, hipStream_t st) {
    if (lds > 16 * 1024) {
        static LdsGrants granted;
        hipError_t e = ensure_dynamic_lds((const void *)k_step_fwd<T, NARROW, ONE>, lds, granted);
        if (e != hipSuccess) return e;
    }
    const int parts = step_parts(s.B, s.Dv, SB_COLS);
    k_step_fwd<T, NARROW, ONE><<<dim3(s.B, parts), SB_THREADS, lds, st>>>((const T *)Qp, (const T *)Kp, (const T *)V, (const T *)v,
                                                                          key_len, C, P, s.Tk, s.H, s.Dv,
                                                                          step_part_width(s.Dv, SB_COLS, parts));
    return hipGetLastError();
}

// Steps that the block of eight waves does sooner (us per launch, it against the sixteen waves).  Past 256 samples: four of its
// blocks share a compute unit that one block of sixteen waves fills, so those take a second round (H = 640, 300 samples of 4
// keys: 5.3 against 10.4, of 17: 9.0 against 11.5, of 32: 14.4 against 13.6; in bf16 level at 17).  On few keys its chain is
// the shorter one, but its trips to memory, one per 32 keys and 256 columns, are not overlapped: ahead up to 16 keys while the
// rows are narrow (H = 75, bf16, 10 keys: 3.8 against 4.2; not in f32 beside value rows of more than a batch: H = 8, Dv = 972,
// 13 keys: 5.9 against 4.7), up to 10 past 128 samples (level at H = 772, 160 samples of 10 keys), else up to 6 in f32 (H =
// 516, 40 samples of 4 keys: 5.0 against 5.4); rows that do not start aligned it reads element by element (H = 587, 88 samples
// of 5 keys: 6.3 against 5.9; up to 4 keys past 128 samples).  A row of fewer than four elements gives the sixteen waves no
// whole pieces to load: level at 32 keys, past 256 samples at 100 (12.3 against 14.0). Where one batch of whole groups of four
// holds the step, all its rows are under way at once and the sixteen waves are ahead from the first key on.
static bool step_fwd_takes_rows(const AttnShape &s) {
    const bool two_rounds = s.B > 256;
    if (s.H < 4) return s.Tk <= (two_rounds ? 100 : 32);
    if (s.H % 4 == 0 && step_one_batch(s)) return false;
    if (two_rounds) return s.Tk <= (s.bf16 ? 17 : 32);
    if (s.H <= 128 && (s.bf16 || s.Dv <= SB_COLS)) return s.Tk <= 16;
    if (s.H % 4 != 0) return s.B > 128 && s.Tk <= 4;
    return s.Tk <= (s.B > 128 ? 10 : s.bf16 ? 0 : 6);
}

hipError_t launch_step_fwd(const AttnShape &s, const void *Qp, const void *Kp, const void *V, const void *v,
                           const int *key_len, float *C, float *P, hipStream_t st) {
    const size_t lds = (size_t)s.Tk * sizeof(float);
    if (lds > SB_MOST_LDS) return hipErrorInvalidValue;
    if (step_fwd_takes_rows(s)) {
        if (s.bf16)
            k_step_fwd_rows<bf16_t><<<s.B, ST_THREADS, lds, st>>>((const bf16_t *)Qp, (const bf16_t *)Kp, (const bf16_t *)V,
                                                                  (const bf16_t *)v, key_len, C, P, s.Tk, s.H, s.Dv);
        else
            k_step_fwd_rows<float><<<s.B, ST_THREADS, lds, st>>>((const float *)Qp, (const float *)Kp, (const float *)V,
                                                                 (const float *)v, key_len, C, P, s.Tk, s.H, s.Dv);
        return hipGetLastError();
    }
#define ECHO_STEP(T, NARROW, ONE) launch_step_fwd_t<T, NARROW, ONE>(s, lds, Qp, Kp, V, v, key_len, C, P, st)
    if (s.H < 4) return s.bf16 ? ECHO_STEP(bf16_t, true, false) : ECHO_STEP(float, true, false);
    if (step_one_batch(s)) return s.bf16 ? ECHO_STEP(bf16_t, false, true) : ECHO_STEP(float, false, true);
    return s.bf16 ? ECHO_STEP(bf16_t, false, false) : ECHO_STEP(float, false, false);
#undef ECHO_STEP
}

size_t step_lds_bytes(const AttnShape &s) { return 2 * (size_t)s.Tk * sizeof(float); }

template <typename T, bool DEFER>
static hipError_t launch_step_bwd_t(const AttnShape &s, const float *dC, const float *P, const void *Qp,
                                    const void *Kp, const void *V, const void *v, const int *key_len, float *dQp,
                                    float *dKp, float *dV, float *dv_part, float *ds_out, float *ds_sum_out,
                                    int ds_rows, int ds_row, hipStream_t st) {
    const size_t lds = step_lds_bytes(s);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    if (lds > 40 * 1024) {
        static LdsGrants granted;
        hipError_t e = ensure_dynamic_lds((const void *)k_step_bwd<T, DEFER>, lds, granted);
        if (e != hipSuccess) return e;
    }
    const int n_hs = (s.H + 63) / 64;
    const int cw = (s.Dv + n_hs - 1) / n_hs;                     // columns of dV per h slice
    dim3 grid(n_hs, s.B);
    k_step_bwd<T, DEFER><<<grid, ST_THREADS, lds, st>>>(dC, P, (const T *)Qp, (const T *)Kp, (const T *)V,
                                                        (const T *)v, key_len, dQp, dKp, dV, dv_part, ds_out,
                                                        ds_sum_out, ds_rows, ds_row, ds_pitch(s.Tk), s.Tk, s.H, s.Dv,
                                                        cw);
    return hipGetLastError();
}

hipError_t launch_step_bwd(const AttnShape &s, const float *dC, const float *P, const void *Qp, const void *Kp,
                           const void *V, const void *v, const int *key_len, float *dQp, float *dKp, float *dV,
                           float *dv_part, hipStream_t st) {
    return s.bf16 ? launch_step_bwd_t<bf16_t, false>(s, dC, P, Qp, Kp, V, v, key_len, dQp, dKp, dV, dv_part, nullptr,
                                                     nullptr, 1, 0, st)
                  : launch_step_bwd_t<float, false>(s, dC, P, Qp, Kp, V, v, key_len, dQp, dKp, dV, dv_part, nullptr,
                                                    nullptr, 1, 0, st);
}

template <typename T, bool ONE>
static hipError_t launch_step_bwd_query_t(const AttnShape &s, const float *dC, const float *P, const void *Qp, const void *Kp,
                                          const void *V, const void *v, const int *key_len, float *dQp, float *ds_out,
                                          float *ds_sum_out, int steps, int step, hipStream_t st) {
    const size_t lds = step_lds_bytes(s);
    if (lds > SB_MOST_LDS) return hipErrorInvalidValue;
    if (lds > 16 * 1024) {
        static LdsGrants granted;
        hipError_t e = ensure_dynamic_lds((const void *)k_step_bwd_query<T, ONE>, lds, granted);
        if (e != hipSuccess) return e;
    }
    const int parts = step_parts(s.B, s.H, 256);
    k_step_bwd_query<T, ONE><<<dim3(s.B, parts), SB_THREADS, lds, st>>>(
        dC, P, (const T *)Qp, (const T *)Kp, (const T *)V, (const T *)v, key_len, dQp, ds_out, ds_sum_out, steps, step,
        ds_pitch(s.Tk), s.Tk, s.H, s.Dv, step_part_width(s.H, 256, parts));
    return hipGetLastError();
}

// Query gradients for which k_step_bwd is done sooner: its blocks of eight waves, one per 64 columns of h, request K together
// with V and four of them share a compute unit, but every one forms dP of its sample again.  (us per launch, this form against
// the sixteen waves, f32 with Dv = H; over 2180 shapes about 30 are more than 5 % slower than the better form.)
//   Up to a block for every fourth compute unit: up to 300 keys (H = 640, 4 samples of 32: 4.0 against 5.6); where the sixteen
//   waves need several batches for a row, at up to 32 blocks any number (H = 640, 1 sample of 400: 14.8 against 16.8).
//   Beyond, while the value rows that the blocks read together stay below 32 MB, 16 where a row is one batch of the sixteen
//   waves (H = 312, 21 samples of 160, 21 MB: 12.7 against 10.4; not past 256 samples, where these take a second round) or
//   where short rows make the many blocks the cost (bf16, more than a block per unit), and
//     up to a block per unit: up to 300 keys (H = 75, 100 samples of 200: 11.4 against 11.6);
//     more: one batch of 32 keys (H = 75, 160 samples of 32: 4.8 against 5.0, of 48: 5.9 against 5.4) on at most 900 blocks (H
//     = 640, 100 samples of 4: 5.0 against 5.3), 600 where one batch of the sixteen waves holds the step (H = 256, 100 samples
//     of 32: 4.4 against 4.6; H = 301, 160 samples of 4, 800 blocks: 5.1 against 4.6);
//     past 256 samples 100 keys on at most 1500 blocks (H = 128, 300 samples of 32: 5.3 against 7.6; H = 256, 300 samples of
//     32, 39 MB: 9.1 against 7.6).
// One slice of h repeats nothing: always past 256 samples (H = 32, 300 samples of 100: 8.5 against 12.9).  Rows of fewer than
// four elements in any case (H = 3, 64 samples of 17: 4.3 against 6.0).
static bool step_bwd_takes_slices(const AttnShape &s) {
    const long long slices = (s.H + 63) / 64, blocks = slices * s.B;
    if (s.H < 4 || (slices == 1 && s.B > 256)) return true;
    if (blocks <= 64) return s.Tk <= 300 || (blocks <= 32 && s.H > SB_COLS);
    const bool one_column_batch = s.H <= SB_COLS && s.Dv <= SB_COLS;
    const long long bytes = blocks * s.Tk * s.Dv * (s.bf16 ? 2 : 4);
    if (bytes > ((one_column_batch && s.B <= 256) || (s.bf16 && blocks > 256) ? 16 << 20 : 32 << 20)) return false;
    if (blocks <= 256) return s.Tk <= 300;
    return s.B > 256 ? blocks <= 1500 && s.Tk <= 100 : blocks <= (step_one_batch(s) ? 600 : 900) && s.Tk <= 32;
}

hipError_t launch_step_bwd_query(const AttnShape &s, const float *dC, const float *P, const void *Qp, const void *Kp,
                                 const void *V, const void *v, const int *key_len, float *dQp, float *ds_out,
                                 float *ds_sum_out, int steps, int step, hipStream_t st) {
    if (step_bwd_takes_slices(s))
        return s.bf16 ? launch_step_bwd_t<bf16_t, true>(s, dC, P, Qp, Kp, V, v, key_len, dQp, nullptr, nullptr, nullptr, ds_out,
                                                        ds_sum_out, steps, step, st)
                      : launch_step_bwd_t<float, true>(s, dC, P, Qp, Kp, V, v, key_len, dQp, nullptr, nullptr, nullptr, ds_out,
                                                       ds_sum_out, steps, step, st);
#define ECHO_QUERY(T, ONE) \
    launch_step_bwd_query_t<T, ONE>(s, dC, P, Qp, Kp, V, v, key_len, dQp, ds_out, ds_sum_out, steps, step, st)
    if (step_one_batch(s)) return s.bf16 ? ECHO_QUERY(bf16_t, true) : ECHO_QUERY(float, true);
    return s.bf16 ? ECHO_QUERY(bf16_t, false) : ECHO_QUERY(float, false);
#undef ECHO_QUERY
}

}  // namespace echo
