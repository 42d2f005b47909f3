// The dense contractions of the layer on the matrix cores, fp32 in and out
// (v_mfma_f32_16x16x4_f32; past the smallest launches B1 as six bf16 products of split operands, split.hpp):
//   F3  context[b] = P[b] . V[b]                 (Section 2, step 2)
//   B1  dV[b] = P[b]^T . dC[b],  dP[b] = dC[b] . V[b]^T   (Eq. 2: only inputs needed)
//   B2  dS = P (dP - rowsum(P dP)), fused behind dP so dP never leaves the CU
//
// Operand layout of one 16x16x4 step, lane l:  A[m = l%16][k = l/16],
// B[k = l/16][n = l%16], D[m = 4*(l/16) + r][n = l%16] in accumulator r.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"
#include "split.hpp"

namespace echo {

__device__ __forceinline__ float comp4(const float4 &x, int c) { return c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w; }

// ---------------------------------------------------------------------------
// out[b, m, n] = sum_k A(m, k) * Bm[b, k, n]
//   TRANS_A = false: A(m, k) = P[b, m, k]   M = Tq, K = L_b   (context)
//   TRANS_A = true : A(m, k) = P[b, k, m]   M = Tk, K = Tq    (dV; rows m >= L_b are zero)
// A wave owns 16 rows x 64 columns: each lane loads four consecutive columns
// of Bm (one 16-byte load) and feeds component c to column tile c, so the
// output columns of tile c are n0 + 4*(l%16) + c and the store is 16 bytes too.
// N must be a multiple of 4.
template <typename TB, bool TRANS_A>
__device__ __forceinline__ void pv_block(const float *__restrict__ P, const TB *__restrict__ Bm,
                                         const int *__restrict__ key_len, float *__restrict__ out,
                                         int Tq, int Tk, int N, int b, int by, int bx, int acc_out) {
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int M = TRANS_A ? Tk : Tq;
    const int K = TRANS_A ? Tq : L;
    const int Mvalid = TRANS_A ? L : Tq;      // rows that can be non-zero
    const int m0 = by * 16;
    const int n0 = (bx * 4 + w) * 64;
    if (n0 >= N) return;
    const int lm = lane & 15, lk = lane >> 4;
    const int ncol = n0 + 4 * lm;             // first of this lane's four columns
    const bool nok = ncol < N;
    const float *Pb = P + (size_t)b * Tq * Tk;
    const TB *Bb = Bm + (size_t)b * (TRANS_A ? Tq : Tk) * N;

    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};

    if (m0 < Mvalid) {
        const int m = m0 + lm;
        constexpr int U = TRANS_A ? 16 : 8;       // k-steps whose loads are in flight together
        for (int kb0 = 0; kb0 < K; kb0 += 4 * U) {
            float a[U];
            float4 bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb0 + 4 * u + lk;
                a[u] = 0.f;
                bv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (kb0 + 4 * u < K) {            // uniform
                    if (m < Mvalid && k < K) a[u] = TRANS_A ? Pb[(size_t)k * Tk + m] : Pb[(size_t)m * Tk + k];
                    if (k < K && nok) bv[u] = ld4(Bb, (size_t)k * N + ncol);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kb0 + 4 * u < K) {
                    acc[0] = mfma16(a[u], bv[u].x, acc[0]);
                    acc[1] = mfma16(a[u], bv[u].y, acc[1]);
                    acc[2] = mfma16(a[u], bv[u].z, acc[2]);
                    acc[3] = mfma16(a[u], bv[u].w, acc[3]);
                }
            }
        }
    }
    if (!nok) return;
    float *ob = out + (size_t)b * M * N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + 4 * lk + r;
        if (m < M) {
            float4 o = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
            float4 *dst = reinterpret_cast<float4 *>(ob + (size_t)m * N + ncol);
            if (acc_out) {                       // add to what the earlier decoder steps left
                const float4 old = *dst;
                o.x += old.x;
                o.y += old.y;
                o.z += old.z;
                o.w += old.w;
            }
            store4_streaming(ob + (size_t)m * N + ncol, o);
        }
    }
}

template <typename TB, bool TRANS_A>
__global__ __launch_bounds__(256) void k_pv(const float *__restrict__ P, const TB *__restrict__ Bm,
                                            const int *__restrict__ key_len, float *__restrict__ out,
                                            int Tq, int Tk, int N) {
    pv_block<TB, TRANS_A>(P, Bm, key_len, out, Tq, Tk, N, blockIdx.z, blockIdx.y, blockIdx.x, 0);
}

hipError_t launch_context(const AttnShape &s, const float *P, const void *V, const int *key_len, float *C,
                          hipStream_t st) {
    dim3 grid((s.Dv + 255) / 256, (s.Tq + 15) / 16, s.B);
    if (s.bf16)
        k_pv<bf16_t, false><<<grid, 256, 0, st>>>(P, (const bf16_t *)V, key_len, C, s.Tq, s.Tk, s.Dv);
    else
        k_pv<float, false><<<grid, 256, 0, st>>>(P, (const float *)V, key_len, C, s.Tq, s.Tk, s.Dv);
    return hipGetLastError();
}

// The finishing phase of a dS block on a long key axis: dP of its 16 rows stands in LDS, wave w turns rows w, w + 4, ...
// into dS = P (dP - sum_j P dP), with zeros at masked keys and pads.
__device__ __forceinline__ void dscore_finish(const float *__restrict__ P, float *__restrict__ dS,
                                              float *__restrict__ ds_rowsum, const float *__restrict__ s_dp, int b, int i0,
                                              int Tq, int Tk, int L, int pitch, int pitch16) {
    const int lane = lane_id(), w = wave_id();
    // P of the rows this wave finishes (w, w + 4, ...), the first NP keys per lane of each: requested together
    // before the barrier (the registers of the product loop are free by now), where loading row after row inside
    // the loop below put one trip to memory behind the other
    constexpr int NP = 5, NR = 4;
    float pr[NR][NP];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const float *p = P + ((size_t)b * Tq + min(i0 + w + 4 * t, Tq - 1)) * Tk;
#pragma unroll
        for (int c = 0; c < NP; ++c) pr[t][c] = p[min(lane + 64 * c, Tk - 1)];
    }
    lds_barrier();

#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int rr = w + 4 * t, i = i0 + rr;
        if (i < Tq) {
            const float *p = P + ((size_t)b * Tq + i) * Tk;
            const float *dp = s_dp + rr * pitch16;
            float *ds = dS + ((size_t)b * Tq + i) * pitch;
            float r = 0.f;
#pragma unroll
            for (int c = 0; c < NP; ++c)
                if (lane + 64 * c < L) r += pr[t][c] * dp[lane + 64 * c];
            for (int j = lane + 64 * NP; j < L; j += 64) r += p[j] * dp[j];
            r = wave_sum(r);
            float tot = 0.f;
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                const int j = lane + 64 * c;
                if (j < pitch) {
                    float x = 0.f;
                    if (j < L) x = pr[t][c] * (dp[j] - r);
                    ds[j] = x;
                    tot += x;
                }
            }
            for (int j = lane + 64 * NP; j < pitch; j += 64) {
                float x = 0.f;
                if (j < L) x = p[j] * (dp[j] - r);
                ds[j] = x;
                tot += x;
            }
            tot = wave_sum(tot);
            if (lane == 0) ds_rowsum[(size_t)b * Tq + i] = tot;
        }
    }
}

// ---------------------------------------------------------------------------
// dS for (b, 16 query rows).  Waves take key tiles of 16 in turn and compute
// dP[i, j] = sum_d dC[i, d] V[j, d] into LDS; then each wave finishes four
// rows: r = sum_j P dP, dS = P (dP - r).  dS rows have pitch `pitch` floats and
// are zero at j >= L_b (pads included).  Dv must be a multiple of 4.
// A lane loads four consecutive d of its row for both operands and spends
// them on four MFMA steps, so the k index of step c is d0 + 4*(l/16) + c on
// both sides.
template <typename TV>
__device__ __forceinline__ void dscore_block(const float *__restrict__ dC, const TV *__restrict__ V,
                                             const float *__restrict__ P, const int *__restrict__ key_len,
                                             float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                             float *__restrict__ s_dp, int b, int i0, int Tq, int Tk, int Dv,
                                             int pitch) {
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int pitch16 = (Tk + 15) / 16 * 16 + 4;
    const float *dCb = dC + (size_t)b * Tq * Dv;
    const TV *Vb = V + (size_t)b * Tk * Dv;

    // Wave w takes key tiles w, w+4, ..., G at a time so that one fragment of dC feeds G products (the
    // kernel is bound by what the L2 can deliver, not by the matrix cores); tiles past the sample's last one are
    // neither loaded nor multiplied.  The sum over d runs
    // in stages of U 16-wide slices; the loads of the next stage are in flight while the current one is multiplied.
    // Rows and keys past the end are clamped for loading; what they produce is never read.  Columns past Dv are zeroed.
    const int n_jt = (L + 15) / 16;
    constexpr int G = 4, U = 2;
    const int n_st = (Dv + 16 * U - 1) / (16 * U);            // stages
    const bool ragged = Dv % (16 * U) != 0;
    const float *dCrow = dCb + (size_t)min(i0 + lm, Tq - 1) * Dv;
    for (int jt0 = w; jt0 < n_jt; jt0 += 4 * G) {              // this wave's tiles jt0, jt0 + 4, jt0 + 8, ...
        const TV *vrow[G];
#pragma unroll
        for (int k = 0; k < G; ++k) vrow[k] = Vb + (size_t)min((jt0 + 4 * k) * 16 + lm, Tk - 1) * Dv;
        float4 a[U], bv[G][U], an[U], bn[G][U];
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u) bv[k][u] = bn[k][u] = make_float4(0.f, 0.f, 0.f, 0.f);
        // key tiles of this group that exist (the same in all lanes): the others are neither loaded nor multiplied
        bool live[G];
#pragma unroll
        for (int k = 0; k < G; ++k) live[k] = jt0 + 4 * k < n_jt;
        auto load = [&](float4 (&da)[U], float4 (&db)[G][U], int st) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int d = min((st * U + u) * 16 + 4 * lk, Dv - 4);
                da[u] = ld4(dCrow, (size_t)d);
#pragma unroll
                for (int k = 0; k < G; ++k)
                    if (live[k]) db[k][u] = ld4(vrow[k], (size_t)d);
            }
        };
        load(a, bv, 0);
        f32x4 acc[G];
#pragma unroll
        for (int k = 0; k < G; ++k) acc[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int st = 0; st < n_st; ++st) {
            load(an, bn, min(st + 1, n_st - 1));
            if (ragged && st == n_st - 1) {                      // columns past Dv add nothing
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((st * U + u) * 16 + 4 * lk >= Dv) a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < G; ++k) if (live[k]) acc[k] = mfma16(a[u].x, bv[k][u].x, acc[k]);
#pragma unroll
                for (int k = 0; k < G; ++k) if (live[k]) acc[k] = mfma16(a[u].y, bv[k][u].y, acc[k]);
#pragma unroll
                for (int k = 0; k < G; ++k) if (live[k]) acc[k] = mfma16(a[u].z, bv[k][u].z, acc[k]);
#pragma unroll
                for (int k = 0; k < G; ++k) if (live[k]) acc[k] = mfma16(a[u].w, bv[k][u].w, acc[k]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = an[u];
#pragma unroll
                for (int k = 0; k < G; ++k) bv[k][u] = bn[k][u];
            }
        }
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int jt = jt0 + 4 * k;
            if (jt < n_jt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) s_dp[(4 * lk + r) * pitch16 + jt * 16 + lm] = acc[k][r];
            }
        }
    }
    dscore_finish(P, dS, ds_rowsum, s_dp, b, i0, Tq, Tk, L, pitch, pitch16);
}

// The same for short key axes (Tk <= kDsplitMaxTk): latency, not arithmetic, decides here, so the four waves
// split d instead of the key tiles.  Wave w owns the columns d of every fourth 128-wide chunk, keeps its slice
// of the 16 dC rows in registers across the key tiles when Dv <= 512, has the V slice of the next key tile in
// flight while the current one is multiplied, and leaves a partial dP tile in its own LDS plane; the planes
// are added in wave order by the finishing phase, whose P rows were requested at the very start.
// Rows and keys past the end are clamped for loading; what they produce is never read.
constexpr int kDsplitMaxTk = 128;

// The finishing phase of a dS block for short key axes: the four waves' planes of partial dP are added in wave order,
// then dS = P (dP - sum_j P dP) for rows w, w+4, w+8, w+12 of the tile (pr: their P, two keys per lane).
__device__ __forceinline__ void dsplit_finish(const float (&pr)[4][2], const float *__restrict__ s_dp,
                                              float *__restrict__ dS, float *__restrict__ ds_rowsum, int b, int i0,
                                              int Tq, int L, int pitch, int pitch16, int plane) {
    const int lane = lane_id(), w = wave_id();

    // the four rows together: r = sum_j P dP and sum_j dS by transposing reductions (sum of row t ends up in
    // lanes 16 t .. 16 t + 15), so the exchanges of the rows overlap instead of queueing behind each other
    float dp[4][2], rsum[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int rr = w + 4 * t;
        rsum[t] = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = lane + 64 * u;
            const float *q = s_dp + rr * pitch16 + min(j, pitch16 - 1);
            const float x = ((q[0] + q[plane]) + q[2 * plane]) + q[3 * plane];
            dp[t][u] = j < L ? x : 0.f;
            rsum[t] = __builtin_fmaf(j < L ? pr[t][u] : 0.f, dp[t][u], rsum[t]);
        }
    }
    const float r4 = wave_transpose_sum<4>(rsum);
    float tsum[4], dsv[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r4), 16 * t));
        tsum[t] = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = lane + 64 * u;
            dsv[t][u] = j < L ? pr[t][u] * (dp[t][u] - r) : 0.f;
            tsum[t] += dsv[t][u];
        }
    }
    const float t4 = wave_transpose_sum<4>(tsum);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int i = i0 + w + 4 * t;
        if (i < Tq) {
            float *ds = dS + ((size_t)b * Tq + i) * pitch;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (lane + 64 * u < pitch) store_streaming(&ds[lane + 64 * u], dsv[t][u]);
            if (lane == 16 * t) ds_rowsum[(size_t)b * Tq + i] = t4;
        }
    }
}

// The general form (any width of the value rows): two register groups of a whole round of V slices each, one in
// flight; with more than one round the dC slices are fetched per key tile and round.
template <typename TV>
__device__ __forceinline__ void dscore_block_dsplit(const float *__restrict__ dC, const TV *__restrict__ V,
                                                    const float *__restrict__ P, const int *__restrict__ key_len,
                                                    float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                                    float *__restrict__ s_dp, int b, int i0, int Tq, int Tk,
                                                    int Dv, int pitch) {
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int pitch16 = (Tk + 15) / 16 * 16 + 4;
    const int plane = 16 * pitch16;
    // P of the rows this wave finishes (rows w, w+4, w+8, w+12 of the tile), two keys per lane
    float pr[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int i = min(i0 + w + 4 * t, Tq - 1);
#pragma unroll
        for (int u = 0; u < 2; ++u) pr[t][u] = P[((size_t)b * Tq + i) * Tk + min(lane + 64 * u, Tk - 1)];
    }
    const float *dCrow = dC + ((size_t)b * Tq + min(i0 + lm, Tq - 1)) * Dv;
    const TV *Vb = V + (size_t)b * Tk * Dv;
    constexpr int U = 8;                          // 16-wide slices of d per wave and round
    const int rounds = (Dv + 64 * U - 1) / (64 * U);
    float4 a[U], bcur[U], bnxt[U];
    auto load_a = [&](int r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int d = (4 * r + w) * 16 * U + 16 * u + 4 * lk;
            const float4 x = ld4(dCrow, (size_t)min(d, Dv - 4));
            a[u] = d < Dv ? x : make_float4(0.f, 0.f, 0.f, 0.f);     // columns past Dv add nothing
        }
    };
    auto load_b = [&](float4 (&dst)[U], int it) {
        const int jt = it / rounds, r = it % rounds;
        const TV *row = Vb + (size_t)min(jt * 16 + lm, Tk - 1) * Dv;
#pragma unroll
        for (int u = 0; u < U; ++u) dst[u] = ld4(row, (size_t)min((4 * r + w) * 16 * U + 16 * u + 4 * lk, Dv - 4));
    };
    // the first slices do not depend on the sample's key count (key tile 0 always exists in memory): they
    // leave before key_len[b] has arrived
    load_b(bcur, 0);
    load_a(0);
    const int L = clamp_len(key_len[b], Tk);
    const int n_jt = (L + 15) / 16;
    const int items = n_jt * rounds;
    f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < items; ++it) {
        const int jt = it / rounds, r = it % rounds;
        load_b(bnxt, min(it + 1, items - 1));
        if (rounds > 1 && it > 0) load_a(r);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = mfma16(a[u].x, bcur[u].x, acc);
            acc = mfma16(a[u].y, bcur[u].y, acc);
            acc = mfma16(a[u].z, bcur[u].z, acc);
            acc = mfma16(a[u].w, bcur[u].w, acc);
        }
        if (r == rounds - 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) s_dp[w * plane + (4 * lk + q) * pitch16 + jt * 16 + lm] = acc[q];
            acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) bcur[u] = bnxt[u];
    }
    lds_barrier();
    dsplit_finish(pr, s_dp, dS, ds_rowsum, b, i0, Tq, L, pitch, pitch16, plane);
}

// Short key axes, value rows of at most 1024 columns, operands through LDS.  A quarter of a wave that reads the operand
// layout of the matrix cores straight from memory asks for the same 16 bytes of 16 different rows; with rows a
// multiple of 128 bytes apart these requests queue in the CU's L1 (measured: 37 KB/us per CU, against 90 to 110
// for loads of whole row pieces, and 67 with rows 2064 bytes apart).  Here a wave loads its 128 columns of 16 rows
// as 8 loads of two 512-byte row pieces each (lanes along d), writes them row by row into its own 16 x 132 floats
// of LDS and reads them back in operand layout (row l % 16, 16 bytes at column 16 u + 4 (l / 16): conflict-free at
// this pitch).  The region belongs to one wave, so no barrier is involved; the V slice of the next key tile is in
// flight in registers while the current one is multiplied.
// ROUNDS = 1 (up to 512 columns): the partial dP tiles stay in registers until the end and then go into the same
// region, which the finishing phase reads as the wave's plane.
// ROUNDS = 2 (513 to 1024 columns): the dC slices of both rounds stay in registers, the steps run over (key tile,
// round), and the partial dP tiles go to planes of their own behind the staging regions as each key tile finishes
// (there is no room to keep eight of them in registers next to two rounds of dC).  The general form above fetches
// the dC slices again for every key tile and round and waits for them each time.
constexpr int kPartKeys = 64;                    // keys of a block that forms a part of the rows of dP (PART)
constexpr int kStagePitch = 132;                 // floats; 16 rows of it are a wave's region
template <typename TV, int ROUNDS, bool PART>
__device__ __forceinline__ void dscore_block_dsplit_lds(const float *__restrict__ dC, const TV *__restrict__ V,
                                                        const float *__restrict__ P, const int *__restrict__ key_len,
                                                        float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                                        float *__restrict__ s_stage, int b, int i0, int Tq, int Tk,
                                                        int Dv, int pitch, int j_first) {
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int pitch16 = PART ? kPartKeys + 4 : (Tk + 15) / 16 * 16 + 4;
    constexpr int region = 16 * kStagePitch;
    constexpr int MAX_JT = (PART ? kPartKeys : kDsplitMaxTk) / 16;
    constexpr int NT = ROUNDS == 1 ? MAX_JT : 1;       // dP tiles kept in registers
    // the planes of partial dP: the staging regions themselves (one round) or planes behind them
    float *planes = ROUNDS == 1 ? s_stage : s_stage + 4 * region;
    const int plane = ROUNDS == 1 ? region : 16 * pitch16;
    // P of the rows this wave finishes (rows w, w+4, w+8, w+12 of the tile), two keys per lane
    float pr[4][2];
    if (!PART) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int i = min(i0 + w + 4 * t, Tq - 1);
#pragma unroll
            for (int u = 0; u < 2; ++u) pr[t][u] = P[((size_t)b * Tq + i) * Tk + min(lane + 64 * u, Tk - 1)];
        }
    }
    constexpr int U = 8;                          // 16-wide slices of d per wave and round
    float *st = s_stage + w * region;             // this wave's region
    const int cr = lane >> 5, cc = 4 * (lane & 31);               // loading: row of the pair, column in the chunk
    const float *dCb = dC + (size_t)b * Tq * Dv;
    const TV *Vb = V + ((size_t)b * Tk + j_first) * Dv;
    const int n_keys = PART ? min(kPartKeys, Tk - j_first) : Tk;          // keys of this block, masked ones included
    float4 a[ROUNDS][U], bcur[U], bnxt[U];
    auto col_of = [&](int r) { return min((4 * r + w) * 16 * U + cc, Dv - 4); };   // clamped for loading
    auto load_v = [&](float4 (&dst)[U], int it) {                 // step it = (key tile, round): 16 keys, two per load
        const int jt = it / ROUNDS, r = it % ROUNDS;
        const int col = col_of(r);
#pragma unroll
        for (int u = 0; u < U; ++u) dst[u] = ld4(Vb + (size_t)min(jt * 16 + 2 * u + cr, n_keys - 1) * Dv, (size_t)col);
    };
    auto through_lds = [&](float4 (&dst)[U], const float4 (&src)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) *reinterpret_cast<float4 *>(st + (2 * u + cr) * kStagePitch + cc) = src[u];
#pragma unroll
        for (int u = 0; u < U; ++u) dst[u] = *reinterpret_cast<const float4 *>(st + lm * kStagePitch + 16 * u + 4 * lk);
    };
    // the first loads do not depend on the sample's key count (key tile 0 always exists in memory)
    load_v(bnxt, 0);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int col = col_of(r);
#pragma unroll
        for (int u = 0; u < U; ++u) a[r][u] = ld4(dCb + (size_t)min(i0 + 2 * u + cr, Tq - 1) * Dv, (size_t)col);
    }
    const int L = clamp_len(key_len[b] - j_first, n_keys);
    const int n_jt = (L + 15) / 16;
    const int items = n_jt * ROUNDS;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        through_lds(a[r], a[r]);
#pragma unroll
        for (int u = 0; u < U; ++u)                               // columns past Dv add nothing
            if ((4 * r + w) * 16 * U + 16 * u + 4 * lk >= Dv) a[r][u] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    through_lds(bcur, bnxt);
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jt = 0; jt < MAX_JT; ++jt) {
        if (jt < n_jt) {                                           // uniform
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                load_v(bnxt, min(jt * ROUNDS + r + 1, max(items - 1, 0)));
                f32x4 &d = acc[ROUNDS == 1 ? jt : 0];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    d = mfma16(a[r][u].x, bcur[u].x, d);
                    d = mfma16(a[r][u].y, bcur[u].y, d);
                    d = mfma16(a[r][u].z, bcur[u].z, d);
                    d = mfma16(a[r][u].w, bcur[u].w, d);
                }
                through_lds(bcur, bnxt);
            }
            if (ROUNDS > 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q) planes[w * plane + (4 * lk + q) * pitch16 + jt * 16 + lm] = acc[0][q];
                acc[0] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    if (ROUNDS == 1) {                            // the wave's plane of partial dP into its own region
#pragma unroll
        for (int jt = 0; jt < MAX_JT; ++jt)
            if (jt < n_jt) {
#pragma unroll
                for (int q = 0; q < 4; ++q) st[(4 * lk + q) * pitch16 + jt * 16 + lm] = acc[ROUNDS == 1 ? jt : 0][q];
            }
    }
    lds_barrier();
    if (PART) {
        // dP of the block's keys (the softmax backward needs whole rows: k_ds_finish); masked keys are not written
        static_assert(kPartKeys == 64, "one key per lane");
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int rr = w + 4 * t, i = i0 + rr;
            if (i < Tq && lane < L) {
                const float *q = planes + rr * pitch16 + lane;
                dS[((size_t)b * Tq + i) * pitch + j_first + lane] = ((q[0] + q[plane]) + q[2 * plane]) + q[3 * plane];
            }
        }
        return;
    }
    dsplit_finish(pr, planes, dS, ds_rowsum, b, i0, Tq, L, pitch, pitch16, plane);
}

// dV of 16 keys and 64 columns, the four waves taking a quarter of the query rows each and adding their tiles in LDS: for
// launches of few blocks, where the length of a wave's walk over the rows decides.  s_part: 3 x 16 x 64 floats.
__device__ __forceinline__ void dv_rows_block(const float *__restrict__ P, const float *__restrict__ dC,
                                              const int *__restrict__ key_len, float *__restrict__ dV,
                                              float *__restrict__ s_part, int Tq, int Tk, int Dv, int b, int by, int bx,
                                              int acc_out) {
    constexpr int U = 8;                      // k-steps of four rows whose loads are in flight together
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int m0 = by * 16, ncol = bx * 64 + 4 * lm;
    const bool nok = ncol < Dv;
    const float *Pb = P + (size_t)b * Tq * Tk + min(m0 + lm, Tk - 1);
    const float *Cb = dC + (size_t)b * Tq * Dv + min(ncol, Dv - 4);
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (m0 < L) {                             // block-uniform
        const int per = ((Tq + 15) / 16) * 4; // rows per wave, a multiple of four
        const int k_lo = w * per, k_hi = min(k_lo + per, Tq);
        for (int kb0 = k_lo; kb0 < k_hi; kb0 += 4 * U) {
            float a[U];
            float4 bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = min(kb0 + 4 * u + lk, Tq - 1);
                a[u] = Pb[(size_t)k * Tk];
                bv[u] = ld4(Cb, (size_t)k * Dv);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kb0 + 4 * u < k_hi) {     // uniform
                    // rows of the next wave or past Tq add nothing, nor do masked keys
                    const float x = kb0 + 4 * u + lk < k_hi && m0 + lm < L ? a[u] : 0.f;
                    acc[0] = mfma16(x, bv[u].x, acc[0]);
                    acc[1] = mfma16(x, bv[u].y, acc[1]);
                    acc[2] = mfma16(x, bv[u].z, acc[2]);
                    acc[3] = mfma16(x, bv[u].w, acc[3]);
                }
            }
        }
        if (w > 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<float4 *>(s_part + ((w - 1) * 16 + 4 * lk + r) * 64 + 4 * lm) =
                    make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
        }
        lds_barrier();
    }
    if (w > 0 || !nok) return;
    float *ob = dV + (size_t)b * Tk * Dv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + 4 * lk + r;
        if (m < Tk) {
            float4 o = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
            if (m0 < L) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float4 x = *reinterpret_cast<const float4 *>(s_part + (k * 16 + 4 * lk + r) * 64 + 4 * lm);
                    o.x += x.x;
                    o.y += x.y;
                    o.z += x.z;
                    o.w += x.w;
                }
            }
            if (acc_out) {                       // add to what the earlier decoder steps left
                const float4 old = *reinterpret_cast<const float4 *>(ob + (size_t)m * Dv + ncol);
                o.x += old.x;
                o.y += old.y;
                o.z += old.z;
                o.w += old.w;
            }
            store4_streaming(ob + (size_t)m * Dv + ncol, o);
        }
    }
}

// dS for (b, 32 query rows) as products of split operands (split.hpp), all of the sample's keys.  The eight waves are KW key groups times
// 8 / KW groups of d: wave w takes the key tiles of 32 w % KW, + KW, ..., at most two, and of every 64 columns of d the pairs of
// 32-wide chunks that fall to its group w / KW.  A wave loads whole row pieces of a chunk (8 rows of 128 bytes per load), passes them
// through LDS of its own to reach operand layout (conflict-free at these pitches) and splits them; what comes next is under
// way meanwhile.  dC is staged by each wave for itself, or, where all of them need the same chunk (KW = 8), split once for the
// block, an eighth of two chunks by each, one buffer ahead (a barrier per two chunks).  The partial sums of the groups of d meet in LDS planes.
// Rows and keys past the end are clamped for loading; what they produce is never read.  Columns of d past Dv are zeroed in dC.
// Results that are not finite are formed again in fp32 by the same waves, several loads under way at a time (backward at B = 64, T = 50, H = Dv =
// 512 27 -> 34 us with one infinity per sample, at B = 32, T = 300, H = Dv = 1024 461 -> 538, 564 with nothing but NaN; two columns per load: 62,
// 740 and 876).
// What bounds it: a wave alone on its SIMD issues a vector instruction in four clocks and overlaps little of that with its products, about ten
// instructions per product of 32 x 32 x 16, so sixteen waves of at most 128 registers share a CU (eight of 250, each with four key tiles and a
// software pipeline, took as long as four of them).  Counters of the launch at B = 32, T = 300, Dv = 1024, one block per CU: vector issue 23 % of the
// SIMDs' clocks, matrix cores 27 %; bf16, B = 128, T = 50, Dv = 1024 24 and 13 %.
// The launch of k_bwd_pre, dS and dV blocks, before (fp32 products; 16 or 32 rows) and with split operands, us: B = 32, T = 300, Dv = 1024
// 126 -> 73, 83 with one block per CU, as it is launched now; bf16 V, B = 128, T = 50, Dv = 1024 28.4 -> 18.6; B = 64, T = 50, Dv = 512 9.7 -> 9.0.
template <typename TV> struct SplitStage;
template <> struct SplitStage<float> {
    static constexpr int PITCH = 36;          // of 32 elements
    static __device__ __forceinline__ void put(float *p, float4 x) { *reinterpret_cast<float4 *>(p) = x; }
    struct Raw { float4 x, y; };
    typedef Split8 Frag;
    static __device__ __forceinline__ Raw get(const float *p) {
        return {*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 4)};
    }
    static __device__ __forceinline__ Frag split(const Raw &r) {
        const float v[8] = {r.x.x, r.x.y, r.x.z, r.x.w, r.y.x, r.y.y, r.y.z, r.y.w};
        return split8(v);
    }
};
template <> struct SplitStage<bf16_t> {
    static constexpr int PITCH = 40;
    static __device__ __forceinline__ void put(bf16_t *p, uint2 x) { *reinterpret_cast<uint2 *>(p) = x; }
    typedef u32x4 Raw;
    typedef u32x4 Frag;
    static __device__ __forceinline__ Raw get(const bf16_t *p) { return *reinterpret_cast<const u32x4 *>(p); }
    static __device__ __forceinline__ Frag split(const Raw &r) { return r; }
};
// floats of LDS: a wave's key tile and its rows of dC; or, KW = 8, two buffers of two chunks of split dC for the block (rows of 80 bytes)
constexpr int kSplitTileFloats = 32 * 36, kSplitPlane = 32 * 5;             // (plane: 16-byte words)
__host__ __device__ constexpr int split_stage_floats(int kw) {
    return 8 * kSplitTileFloats + (kw == 8 ? 4 * 3 * kSplitPlane * 4 : 8 * kSplitTileFloats);
}
constexpr size_t kAloneLdsBytes = 84 * 1024;                                // (of 160 KB)
__host__ __device__ constexpr int split_dp_pitch(int Tk) { return (Tk + 31) / 32 * 32 + 4; }
__host__ __device__ constexpr int split_lds_floats(int kw, int Tk) {
    return split_stage_floats(kw) > 8 / kw * 32 * split_dp_pitch(Tk) ? split_stage_floats(kw) : 8 / kw * 32 * split_dp_pitch(Tk);
}

// The finishing phase: dS = P (dP - sum_j P dP) of the rows w, w + 8, ... of the block, NP keys per lane.
template <int PLANES, int NP>
__device__ __forceinline__ void split_finish(const float (&pr)[4][NP], float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                             const float *__restrict__ s_dp, int b, int i0, int Tq, int L, int pitch, int dp_pitch) {
    const int lane = lane_id(), w = wave_id();
    float dp[4][NP], sum[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        sum[t] = 0.f;
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const float *q = s_dp + (w + 8 * t) * dp_pitch + min(lane + 64 * c, dp_pitch - 1);
            float x = q[0];
#pragma unroll
            for (int p = 1; p < PLANES; ++p) x += q[p * 32 * dp_pitch];
            dp[t][c] = lane + 64 * c < L ? x : 0.f;
            sum[t] = __builtin_fmaf(lane + 64 * c < L ? pr[t][c] : 0.f, dp[t][c], sum[t]);
        }
    }
    const float r4 = wave_transpose_sum<4>(sum);                  // lane l: row l / 16
    float tot[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float r = lane_value(r4, 16 * t);
        tot[t] = 0.f;
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            dp[t][c] = lane + 64 * c < L ? pr[t][c] * (dp[t][c] - r) : 0.f;
            tot[t] += dp[t][c];
        }
    }
    const float t4 = wave_transpose_sum<4>(tot);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int i = i0 + w + 8 * t;
        if (i < Tq) {
            float *ds = dS + ((size_t)b * Tq + i) * pitch;
#pragma unroll
            for (int c = 0; c < NP; ++c)
                if (lane + 64 * c < pitch) store_streaming(&ds[lane + 64 * c], dp[t][c]);
            if (lane == 16 * t) ds_rowsum[(size_t)b * Tq + i] = t4;
        }
    }
}

// The products of a wave with NL key tiles.  APART: those of each chunk summed on their own (add16).
template <typename TV, int NL, int KW, bool APART>
__device__ __forceinline__ void dscore_split_tiles(const BufferRows<float> &rows_a, const BufferRows<TV> &rows_v,
                                                   float *__restrict__ s_mem, f32x16 (&acc)[2], int last_row, int last_key, int Dv) {
    constexpr bool SHARED = KW == 8;
    constexpr int DW = 8 / KW, NA = SHARED ? 1 : 4;
    typedef SplitStage<TV> VS;
    typedef SplitStage<float> AS;
    const int lane = lane_id(), w = wave_id();
    const int kw = w % KW, dw = w / KW;
    const int n = lane & 31, half = lane >> 5;
    TV *sv = reinterpret_cast<TV *>(s_mem + w * kSplitTileFloats);
    float *sa = s_mem + (8 + w) * kSplitTileFloats;                // (dC of the wave)
    u32x4 *sp = reinterpret_cast<u32x4 *>(s_mem + 8 * kSplitTileFloats);                                        // (of the block)
    const int lr = lane >> 3, lc = 4 * (lane & 7);                // loading: row of the eight, column in the chunk
    const int n_ch = (Dv + 31) / 32, pairs = (n_ch + 1) / 2;
    // chunk s of this wave: pair dw + DW (s / 2), its (s % 2)th chunk; the last pair may hold one chunk only
    const int my_pairs = (pairs - dw + DW - 1) / DW;
    const int steps = SHARED ? n_ch : dw < pairs ? 2 * my_pairs - ((n_ch & 1) && (pairs - 1) % DW == dw ? 1 : 0) : 0;
    if (steps == 0) return;
    constexpr int R = SHARED && NL == 1 ? 2 : 1;                   // (tile chunks on their way)
    float4 na[NA];
    Raw4<TV> nv[R][4];                                             // the chunks of key tiles that come next
    // Buffer loads: row group and chunk are the scalar offset, the lane's row in the group and its columns the vector offset.  The
    // descriptors end behind the last row of the block and the last valid key (the hardware checks the range; the scalar offset stays
    // below it); a last chunk of fewer than 32 columns runs on into the next row.
    const unsigned a_off = (unsigned)(lr * Dv + lc) * 4u, v_off = (unsigned)(lr * Dv + lc) * (unsigned)sizeof(TV);
    auto chunk_of = [&](int s) { return SHARED ? 32 * s : 32 * (2 * (dw + DW * (s >> 1)) + (s & 1)); };          // its first column
    // (SHARED: the first four waves take the rows of the even chunks, the others those of the odd ones)
    auto load_a = [&](int s) {
        const int c = min(chunk_of(s), Dv - 4);
#pragma unroll
        for (int u = 0; u < NA; ++u)
            na[u] = rows_a.load4_raw(a_off, (unsigned)(min(8 * (SHARED ? w & 3 : u), last_row) * Dv + c) * 4u);
    };
    auto load_v = [&](Raw4<TV> (&dst)[4], int s, int k) {
        const int c = min(chunk_of(s), Dv - 4);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            dst[u] = rows_v.load4_raw(v_off, (unsigned)(min((kw + KW * k) * 32 + 8 * u, last_key) * Dv + c) * (unsigned)sizeof(TV));
    };
    auto put_a = [&](int s) {
        if (chunk_of(s) + 32 > Dv && chunk_of(s) + lc >= Dv) {     // columns past Dv add nothing
#pragma unroll
            for (int u = 0; u < NA; ++u) na[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const float4 x = na[u];
            if constexpr (SHARED) {
                uint2 p[3];
                split2(x.x, x.y, p[0].x, p[1].x, p[2].x);
                split2(x.z, x.w, p[0].y, p[1].y, p[2].y);
                uint2 *dst = reinterpret_cast<uint2 *>(sp + (s & 3) * 3 * kSplitPlane) + (8 * (w & 3) + lr) * 10 + (lane & 7);
#pragma unroll
                for (int q = 0; q < 3; ++q) dst[q * 2 * kSplitPlane] = p[q];
            } else {
                AS::put(sa + (8 * u + lr) * AS::PITCH + lc, x);
            }
        }
    };
    auto frag_a = [&](int s, int ks) {
        if constexpr (SHARED) {
            const u32x4 *src = sp + (s & 3) * 3 * kSplitPlane + n * 5 + 2 * ks + half;
            Split8 f;
#pragma unroll
            for (int q = 0; q < 3; ++q) f.p[q] = src[q * kSplitPlane];
            return f;
        } else {
            return AS::split(AS::get(sa + n * AS::PITCH + 16 * ks + 8 * half));
        }
    };
    const int odd = w >> 2;                                        // (SHARED: the chunk of each pair whose dC this wave splits)
    load_a(SHARED ? odd : 0);
    if constexpr (NL > 0) load_v(nv[0], 0, 0);
    if constexpr (R == 2) load_v(nv[1], 1, 0);
    if constexpr (SHARED) {
        put_a(odd);
        load_a(2 + odd);
    }
    f32x16 run = zero16();                                         // (APART)
    auto step = [&](Raw4<TV> (&now)[4], int s) {
        if constexpr (SHARED) {
            if ((s & 1) == 0) {
                lds_barrier();                                     // dC of chunks s and s + 1 is there, that of s - 2 and s - 1 no longer read
                put_a(s + 2 + odd);
                load_a(s + 4 + odd);
            }
        } else {
            put_a(s);
            load_a(s + 1);
        }
        Split8 a0, a1;
        if constexpr (NL > 0) {
            a0 = frag_a(s, 0);
            a1 = frag_a(s, 1);
        }
#pragma unroll
        for (int k = 0; k < NL; ++k) {
#pragma unroll
            for (int u = 0; u < 4; ++u) VS::put(sv + (8 * u + lr) * VS::PITCH + lc, now[u]);
            load_v(now, k + 1 < NL ? s : s + R, k + 1 < NL ? k + 1 : 0);
            loads_stay();
            const TV *t = sv + n * VS::PITCH + 8 * half;
            if constexpr (APART) {                                  // (the run before this one is done by now, where an add behind its own waits)
                const auto b0 = VS::split(VS::get(t));
                add16(acc[k > 0 ? k - 1 : NL - 1], run);
                run = mfma32(a1, VS::split(VS::get(t + 16)), mfma32(a0, b0, zero16()));
            } else {
                acc[k] = mfma32(a0, VS::split(VS::get(t)), acc[k]);
                acc[k] = mfma32(a1, VS::split(VS::get(t + 16)), acc[k]);
            }
        }
    };
    for (int s = 0; s < steps; s += 2) {
        step(nv[0], s);
        if (s + 1 < steps) step(nv[R - 1], s + 1);
    }
    if constexpr (APART && NL > 0) add16(acc[NL - 1], run);
}

template <typename TV, int KW, bool APART>
__device__ __forceinline__ void dscore_split_block(const float *__restrict__ dC, const TV *__restrict__ V,
                                                   const float *__restrict__ P, const int *__restrict__ key_len,
                                                   float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                                   float *__restrict__ s_mem, int *__restrict__ s_inf, int b, int i0, int Tq,
                                                   int Tk, int Dv, int pitch) {
    constexpr int DW = 8 / KW, NP = KW;                             // 64 KW keys at most
    const int lane = lane_id(), w = wave_id();
    const int kw = w % KW, dw = w / KW;
    const int n = lane & 31, half = lane >> 5;
    const float *dCb = dC + ((size_t)b * Tq + i0) * Dv;
    const TV *Vb = V + (size_t)b * Tk * Dv;
    const int last_row = min(32, Tq - i0) - 1;
    // P of the rows this wave finishes: requested at the start where it takes few registers, else before the block meets
    float pr[4][NP];
    auto load_p = [&]() {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float *p = P + ((size_t)b * Tq + min(i0 + w + 8 * t, Tq - 1)) * Tk;
#pragma unroll
            for (int c = 0; c < NP; ++c) pr[t][c] = p[min(lane + 64 * c, Tk - 1)];
        }
    };
    if constexpr (NP <= 2) load_p();
    const int L = clamp_len(key_len[b], Tk);
    const int mine = __builtin_amdgcn_readfirstlane(((L + 31) / 32 - kw + KW - 1) / KW);       // this wave's key tiles
    f32x16 acc[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
    if (L > 0) {                                                    // (block-uniform)
        const BufferRows<float> rows_a(dCb, (unsigned)(last_row + 1) * (unsigned)Dv);
        const BufferRows<TV> rows_v(Vb, (unsigned)L * (unsigned)Dv);
        if (mine == 2) dscore_split_tiles<TV, 2, KW, APART>(rows_a, rows_v, s_mem, acc, last_row, L - 1, Dv);
        else if (mine == 1) dscore_split_tiles<TV, 1, KW, APART>(rows_a, rows_v, s_mem, acc, last_row, L - 1, Dv);
        else if constexpr (KW == 8) dscore_split_tiles<TV, 0, KW, APART>(rows_a, rows_v, s_mem, acc, last_row, L - 1, Dv);
    }
    // a result of a valid key that is not finite: infinities among the operands, perhaps (see split.hpp)
    float odd = 0.f;
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (k < mine) {
            float x = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) x = __builtin_fmaf(acc[k][r], 0.f, x);
            odd += (kw + KW * k) * 32 + n < L ? x : 0.f;
        }
    if constexpr (NP > 2) load_p();
    const int dp_pitch = split_dp_pitch(Tk);
    if (lane == 0) s_inf[w] = 0;
    if (odd != 0.f) s_inf[w] = 1;                                   // (NaN)
    lds_barrier();                                                  // the staging regions become the rows of dP
    int again = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) again |= s_inf[k];
    float back = split_back<TV>;
    if (KW == 8 ? again : __builtin_expect(again, 0)) {             // the wave's products again, in fp32 (KW = 8: the hint costs registers)
        back = 1.f;
        const float *arow = dCb + (size_t)min(n, last_row) * Dv;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k >= mine) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
            const TV *vrow = Vb + (size_t)min((kw + KW * k) * 32 + n, Tk - 1) * Dv;
            // PC pieces of 8 columns of d at a time, all loads of them before the first product: step c of a piece is column 4 half + c
            constexpr int PC = KW == 8 ? 2 : 4;
            for (int d0 = 8 * PC * dw; d0 < Dv; d0 += 8 * PC * DW) {
                float4 a[PC], x[PC];
#pragma unroll
                for (int u = 0; u < PC; ++u) {
                    const int d = d0 + 8 * u + 4 * half;
                    a[u] = ld4(arow, (size_t)min(d, Dv - 4));
                    x[u] = ld4(vrow, (size_t)min(d, Dv - 4));
                    if (d >= Dv) a[u] = x[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int u = 0; u < PC; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp4(a[u], c), comp4(x[u], c), acc[k], 0, 0, 0);
            }
        }
    }
    float *plane = s_mem + dw * 32 * dp_pitch;
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (k < mine)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                plane[mfma32_row(r, lane) * dp_pitch + (kw + KW * k) * 32 + n] = acc[k][r] * back;
    lds_barrier();
    split_finish<DW, NP>(pr, dS, ds_rowsum, s_mem, b, i0, Tq, L, pitch, dp_pitch);
}

// dV of one sample for a panel of up to 64 keys and 256 columns, 32 columns per wave: dV[j, n] = sum_i P[i, j] dC[i, n] as products of
// split operands (split.hpp).  Steps of 64 query rows.  The P values of a step are split once for all waves: a thread takes 8 rows of a
// key, lanes along the keys, and leaves them in LDS as the lanes of the products will read them, 16 bytes each, in one of two
// buffers (one barrier per step).  A lane's dC values, one column of 8 rows per product, come straight from memory (a row piece of 128
// bytes per half wave), two products ahead, and are split in registers: every element of the block's columns is loaded
// once, for all keys of the panel.  Rows past Tq and masked keys count as zero.
constexpr int kDvKeys = 64;                   // keys of a panel
constexpr int kDvSplitLdsBytes = 2 * 3 * 8 * kDvKeys * 16;
template <bool APART>
__device__ __forceinline__ void dv_split_block(const float *__restrict__ P, const float *__restrict__ dC,
                                               const int *__restrict__ key_len, float *__restrict__ dV, u32x4 *__restrict__ s_a, int Tq,
                                               int Tk, int Dv, int b, int j0, int cg, int acc_out) {
    constexpr int W = 8, NT = kDvKeys / 32, KEYS = kDvKeys, ROWS = 8 * W, NK = ROWS / 16;
    constexpr int BUF = 3 * W * KEYS;                                        // (16-byte words of a buffer)
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, half = lane >> 5;
    const int col = (cg * W + w) * 32 + n;
    const float *Pb = P + (size_t)b * Tq * Tk;
    const float *Cb = dC + (size_t)b * Tq * Dv;
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    const int live = min((L - j0 + 31) / 32, NT);                            // key tiles that hold a valid key (block-uniform)
    const unsigned b_col = (unsigned)min(col, Dv - 1);
    float back = split_back<float>;
    if (live > 0) {
        const int n_st = (Tq + ROWS - 1) / ROWS;
        // staging: rows 8 w .. + 7 of the step; key `lane` of the panel
        const unsigned a_col = (unsigned)min(j0 + lane, Tk - 1);
        const bool a_on = j0 + lane < L;
        const bool has_cols = (cg * W + w) * 32 < Dv;
        float pa[8], pb[2][8];
        // offsets within a step in 32 bits; rows past Tq are read as the last one
        auto load_a = [&](int st) {
            const float *base = Pb + (size_t)st * ROWS * Tk;
            const int lim = Tq - 1 - ROWS * st;
#pragma unroll
            for (int e = 0; e < 8; ++e) pa[e] = (base + (size_t)min(8 * w + e, lim) * Tk)[a_col];        // (scalar row)
        };
        // scalar row below Tq, the halves eight rows apart; rows past Tq read as the last one or, past the descriptor, as zero
        const BufferRows<float> rows_b(Cb, (unsigned)Tq * (unsigned)Dv);
        const unsigned b_off = ((unsigned)(8 * half * Dv) + b_col) * 4u;
        auto load_b = [&](float (&dst)[8], int st, int ks) {
            const int row = st * ROWS + 16 * ks;
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[e] = rows_b.load_raw(b_off, (unsigned)(min(row + e, Tq - 1) * Dv) * 4u);
        };
        load_a(0);
        if (has_cols) {
            load_b(pb[0], 0, 0);
            load_b(pb[1], 0, 1);
        }
        for (int st = 0; st < n_st; ++st) {
            u32x4 *buf = s_a + (st & 1) * BUF;
            const int rows = Tq - ROWS * st, next = min(st + 1, n_st - 1);
            {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = a_on && 8 * w + e < rows ? pa[e] : 0.f;
                const Split8 s = split8(x);
#pragma unroll
                for (int p = 0; p < 3; ++p) buf[(p * W + w) * KEYS + lane] = s.p[p];
            }
            load_a(next);
            loads_stay();
            lds_barrier();
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                if (16 * ks < rows && has_cols) {                            // uniform
                    const Split8 sb = split8(pb[ks & 1]);
                    if (ks + 2 < NK) load_b(pb[ks & 1], st, ks + 2);
                    else load_b(pb[ks & 1], next, ks + 2 - NK);
                    loads_stay();
                    const u32x4 *frag = buf + (2 * ks + half) * KEYS + n;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        if (t < live) {
                            Split8 sa;
#pragma unroll
                            for (int p = 0; p < 3; ++p) sa.p[p] = frag[p * W * KEYS + 32 * t];
                            if constexpr (APART) add16(acc[t], mfma32(sa, sb, zero16()));
                            else acc[t] = mfma32(sa, sb, acc[t]);
                        }
                }
            }
        }
        // a result of a valid key that is not finite: infinities among the operands, perhaps (see split.hpp); the wave's columns again,
        // in fp32
        float odd = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t < live) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    odd = __builtin_fmaf(j0 + 32 * t + mfma32_row(r, lane) < L ? acc[t][r] : 0.f, 0.f, odd);
            }
        if (__builtin_expect(__any(odd != 0.f), 0)) {
            back = 1.f;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
            for (int i = 0; i < Tq; i += 16) {                               // all loads of 16 rows before their first product
                float x[NT][8], y[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int row = min(i + 2 * u + half, Tq - 1);
                    y[u] = Cb[(size_t)row * Dv + b_col];
#pragma unroll
                    for (int t = 0; t < NT; ++t) x[t][u] = Pb[(size_t)row * Tk + min(j0 + 32 * t + n, Tk - 1)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool on = i + 2 * u + half < Tq;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        if (t < live)
                            acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(on && j0 + 32 * t + n < L ? x[t][u] : 0.f, on ? y[u] : 0.f,
                                                                          acc[t], 0, 0, 0);
                }
            }
        }
    }
    if (col >= Dv) return;
    float *ob = dV + ((size_t)b * Tk + j0) * Dv + col;
    const int rows = min(KEYS, Tk - j0);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int j = 32 * t + mfma32_row(r, lane);
            if (j < rows) {
                float *dst = ob + (size_t)j * Dv;
                // (masked keys of a tile were multiplied by zeros, which leave a NaN of dC standing)
                const float x = j0 + j < L ? acc[t][r] * back : 0.f;
                store_streaming(dst, acc_out ? x + *dst : x);      // add to what the earlier decoder steps left
            }
        }
}

// dV of one sample for a panel of 64 keys and 256 columns, 64 columns per wave: dV[j, n] = sum_i P[i, j] dC[i, n].
// Per step of four query rows a lane loads four consecutive keys of a P row and four consecutive columns of the dC
// row (16 bytes each) and spends them on 16 products: component ca of the keys with component cb of the columns,
// so product (ca, cb) holds keys m0 + 4 (row of the result tile) + ca and columns n0 + 4 (l % 16) + cb.  Two bytes
// of operands per lane and product, against five in the form with one key per lane (pv_block), which at the larger
// workloads was bound by what the L2 could deliver.  Needs Tk % 4 == 0 (16-byte loads of P rows).  Batches of U
// steps are double buffered.  Rows of masked keys (j >= L) come out as exact zeros whatever P holds there.
__device__ __forceinline__ void dv_tile64(const float *__restrict__ P, const float *__restrict__ dC,
                                          const int *__restrict__ key_len, float *__restrict__ dV, int Tq, int Tk,
                                          int Dv, int b, int by, int bx, int acc_out) {
    constexpr int U = 4;
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int m0 = by * 64, n0 = (bx * 4 + w) * 64;
    if (n0 >= Dv) return;
    const int kcol = m0 + 4 * lm;             // first of this lane's four keys
    const int ncol = n0 + 4 * lm;             // first of this lane's four columns
    const bool nok = ncol < Dv;
    const float *Pb = P + (size_t)b * Tq * Tk;
    const float *Cb = dC + (size_t)b * Tq * Dv;
    f32x4 acc[4][4];
#pragma unroll
    for (int ca = 0; ca < 4; ++ca)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[ca][cb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (m0 < L) {
        const int kc = min(kcol, Tk - 4), nc = min(ncol, Dv - 4);       // clamped for loading
        float4 a[U], bv[U], an[U], bn[U];
        auto load = [&](float4 (&da)[U], float4 (&db)[U], int kb0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = min(kb0 + 4 * u + lk, Tq - 1);
                da[u] = ld4(Pb, (size_t)k * Tk + kc);
                db[u] = ld4(Cb, (size_t)k * Dv + nc);
            }
        };
        load(a, bv, 0);
        for (int kb0 = 0; kb0 < Tq; kb0 += 4 * U) {
            load(an, bn, min(kb0 + 4 * U, Tq - 1));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool row_on = kb0 + 4 * u + lk < Tq;               // rows past Tq add nothing
                float x[4];
#pragma unroll
                for (int ca = 0; ca < 4; ++ca) x[ca] = (row_on && kcol + ca < L) ? comp4(a[u], ca) : 0.f;
#pragma unroll
                for (int ca = 0; ca < 4; ++ca)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) acc[ca][cb] = mfma16(x[ca], comp4(bv[u], cb), acc[ca][cb]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = an[u];
                bv[u] = bn[u];
            }
        }
    }
    if (!nok) return;
    float *ob = dV + (size_t)b * Tk * Dv;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ca = 0; ca < 4; ++ca) {
            const int m = m0 + 16 * lk + 4 * r + ca;
            if (m < Tk) {
                float4 o = make_float4(acc[ca][0][r], acc[ca][1][r], acc[ca][2][r], acc[ca][3][r]);
                if (acc_out) {                       // add to what the earlier decoder steps left
                    const float4 old = *reinterpret_cast<const float4 *>(ob + (size_t)m * Dv + ncol);
                    o.x += old.x;
                    o.y += old.y;
                    o.z += old.z;
                    o.w += old.w;
                }
                store4_streaming(ob + (size_t)m * Dv + ncol, o);
            }
        }
}

// dV of one sample for a 64-wide group of columns and all of at most 64 keys: dV[j, n0 .. n0+63] = sum_i P[i, j] dC[i, n0 ..].
// The block's slice of dC (Tq rows of 256 bytes) passes through the CU once.  Wave w owns the key tile of 16: per step of four query rows
// a lane loads one value of P and four consecutive columns of dC (one 16-byte load) and issues 4 products.
// Batches of U steps are double buffered: the loads of the next batch are in flight during the products of this one.
// Rows of masked keys (j >= L) come out as exact zeros.
__device__ __forceinline__ void dv_cols_block(const float *__restrict__ P, const float *__restrict__ dC,
                                              const int *__restrict__ key_len, float *__restrict__ dV, int Tq, int Tk,
                                              int Dv, int b, int cg, int acc_out) {
    constexpr int U = 8;
    const int L = clamp_len(key_len[b], Tk);
    const int lane = lane_id(), w = wave_id();
    const int lm = lane & 15, lk = lane >> 4;
    const int ncol = cg * 64 + 4 * lm;
    const int n_steps = (Tq + 3) / 4;
    if (16 * w >= Tk) return;
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (16 * w < L) {                                               // uniform: else all of the tile's keys are masked
        const float *Pb = P + (size_t)b * Tq * Tk + min(16 * w + lm, Tk - 1);
        const float *dCb = dC + (size_t)b * Tq * Dv + min(ncol, Dv - 4);
        float a[2][U];
        float4 bv[2][U];
        auto load = [&](int buf, int st0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kc = min(4 * (st0 + u) + lk, Tq - 1);
                a[buf][u] = Pb[(size_t)kc * Tk];
                bv[buf][u] = ld4(dCb, (size_t)kc * Dv);
            }
        };
        auto mult = [&](int buf, int st0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (st0 + u < n_steps) {                            // uniform
                    // query rows past Tq (last step only) were loaded from row Tq - 1: they add nothing.
                    // Masked here, at the point of use, so that nothing waits for the loads earlier.
                    const float av = 4 * (st0 + u) + lk < Tq ? a[buf][u] : 0.f;
                    acc[0] = mfma16(av, bv[buf][u].x, acc[0]);
                    acc[1] = mfma16(av, bv[buf][u].y, acc[1]);
                    acc[2] = mfma16(av, bv[buf][u].z, acc[2]);
                    acc[3] = mfma16(av, bv[buf][u].w, acc[3]);
                }
            }
        };
        load(0, 0);
        for (int st0 = 0; st0 < n_steps; st0 += 2 * U) {
            if (st0 + U < n_steps) load(1, st0 + U);
            mult(0, st0);
            if (st0 + 2 * U < n_steps) load(0, st0 + 2 * U);
            if (st0 + U < n_steps) mult(1, st0 + U);
        }
    }
    if (ncol >= Dv) return;
    float *dVb = dV + (size_t)b * Tk * Dv + ncol;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = 16 * w + 4 * lk + r;
        if (j < Tk) {
            float4 o = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
            if (j >= L) o = make_float4(0.f, 0.f, 0.f, 0.f);      // masked key: its P column was not zeroed above
            float *dst = dVb + (size_t)j * Dv;
            if (acc_out) {                                       // add to what the earlier decoder steps left
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

// For the recompute kernel: order[n] = b | L_b << 16, the samples by valid keys, the most first (ties by index), or in index order
// when `sorted` is 0.  first > 0: sample n's blocks share their compute units with those of sample first + n (n < B - first), the
// samples between have theirs alone (recompute_first_samples).  The 2 first - B heaviest then stay alone, and of the others the
// heavier half meets the lighter one, the heaviest the lightest.  (One alone: in the middle of the samples, whose unit it may share.)
__device__ __forceinline__ void rank_block(const int *__restrict__ key_len, int *__restrict__ order,
                                           int *__restrict__ s_len, int B, int Tk, int sorted, int first) {
    if (sorted)
        for (int o = threadIdx.x; o < B; o += (int)blockDim.x) s_len[o] = clamp_len(key_len[o], Tk);
    lds_barrier();
    const int paired = B - first, alone = first - paired > 1 ? first - paired : 0;
    for (int cand = threadIdx.x; cand < B; cand += (int)blockDim.x) {
        int r = cand;
        const int lc = sorted ? s_len[cand] : clamp_len(key_len[cand], Tk);
        if (sorted) {
            r = 0;
            for (int o = 0; o < B; ++o) {
                const int lo = s_len[o];
                r += (lo > lc) || (lo == lc && o < cand);
            }
        }
        int at = r;
        if (first > 0) at = r < alone ? paired + r : r < first ? r - alone : first + (B - 1 - r);
        order[at] = cand | (lc << 16);
    }
}

// Everything the backward pass needs before the recomputation, in one launch:
// blocks that produce dS (B1 + B2), blocks that produce dV (B1) and one block
// that ranks the samples.  The three kinds of block do not depend on each other.
// dV blocks of a sample: groups of columns times groups of keys.  dv_split_block and dv_tile64: 256 columns, 64 keys; dv_cols_block:
// 64 columns, all keys; pv_block: 256 columns, 16 keys.
__host__ __device__ constexpr int dv_col_groups(int kw, int Tk, int Dv) { return kw == 0 && Tk <= 64 ? (Dv + 63) / 64 : (Dv + 255) / 256; }
__host__ __device__ constexpr int dv_key_groups(int kw, bool panels, int Tk) {
    return kw || panels ? (Tk + kDvKeys - 1) / kDvKeys : Tk <= 64 ? 1 : (Tk + 15) / 16;
}

// The dS blocks of a launch: KW key groups of a block of eight waves, 32 query rows and at most 64 KW keys (dscore_split_block), or, KW = 0,
// 16 rows on the fp32 matrix instructions in blocks of four waves.  ALT: with KW = 0 dV in panels (dv_tile64), with KW = 8 short
// runs of products summed on their own.
template <typename TV, int KW, bool ALT>
__global__ __launch_bounds__(KW ? 512 : 256, KW ? 4 : 3) void k_bwd_pre(const float *__restrict__ dC, const TV *__restrict__ V,
                                                 const float *__restrict__ P, const int *__restrict__ key_len,
                                                 float *__restrict__ dS, float *__restrict__ ds_rowsum,
                                                 int *__restrict__ order, float *__restrict__ dV, int B, int sorted,
                                                 int first,
                                                 int Tq, int Tk, int Dv, int pitch, int s_tiles, int s_rows, int acc) {
    // dS blocks: [s_rows][pitch16], four planes of 16 rows when Tk <= kDsplitMaxTk; dV blocks: two buffers of split P
    extern __shared__ __align__(16) float s_dp[];
    __shared__ int s_len[kMaxSortedB];
    // The hardware deals blocks to the eight XCDs round-robin, so block id mod 8 names the XCD.  Sample b is
    // worked on by XCD b mod 8 only: its dC, V and P then pass through one L2 instead of eight.  Within an XCD the
    // long dS blocks of all its samples come first, then the dV blocks; the last block of the grid ranks.
    constexpr int kXcd = 8;
    const int spx = (B + kXcd - 1) / kXcd;                     // sample slots per XCD
    const int v_cols = dv_col_groups(KW, Tk, Dv), per_b = v_cols * dv_key_groups(KW, KW == 0 && ALT, Tk);       // dV blocks per sample
    const int per_xcd = spx * (s_tiles + per_b);
    if ((int)blockIdx.x == kXcd * per_xcd) {
        rank_block(key_len, order, s_len, B, Tk, sorted, first);
        return;
    }
    const int xcd = blockIdx.x % kXcd;
    int li = blockIdx.x / kXcd;
    if (li < spx * s_tiles) {
        const int b = xcd + kXcd * (li / s_tiles), i0 = (li % s_tiles) * s_rows;
        if (b >= B) return;
        if constexpr (KW > 0) {
            dscore_split_block<TV, KW, ALT>(dC, V, P, key_len, dS, ds_rowsum, s_dp, s_len, b, i0, Tq, Tk, Dv, pitch);
        } else if (Tk <= kDsplitMaxTk) {
            if (Dv <= 512) dscore_block_dsplit_lds<TV, 1, false>(dC, V, P, key_len, dS, ds_rowsum, s_dp, b, i0, Tq, Tk, Dv, pitch, 0);
            else if (Dv <= 1024) dscore_block_dsplit_lds<TV, 2, false>(dC, V, P, key_len, dS, ds_rowsum, s_dp, b, i0, Tq, Tk, Dv, pitch, 0);
            else dscore_block_dsplit<TV>(dC, V, P, key_len, dS, ds_rowsum, s_dp, b, i0, Tq, Tk, Dv, pitch);
        } else {
            dscore_block<TV>(dC, V, P, key_len, dS, ds_rowsum, s_dp, b, i0, Tq, Tk, Dv, pitch);
        }
        return;
    }
    li -= spx * s_tiles;
    const int b = xcd + kXcd * (li / per_b), rem = li % per_b;
    if (b >= B) return;
    if constexpr (KW > 0)
        dv_split_block<ALT>(P, dC, key_len, dV, reinterpret_cast<u32x4 *>(s_dp), Tq, Tk, Dv, b, (rem / v_cols) * kDvKeys, rem % v_cols, acc);
    else if constexpr (ALT) dv_tile64(P, dC, key_len, dV, Tq, Tk, Dv, b, rem / v_cols, rem % v_cols, acc);
    else if (Tk <= 64) dv_cols_block(P, dC, key_len, dV, Tq, Tk, Dv, b, rem, acc);
    else pv_block<float, true>(P, dC, key_len, dV, Tq, Tk, Dv, b, rem / v_cols, rem % v_cols, acc);
}

// The same work for launches that k_bwd_pre would run in too few, too long blocks (key axes past 128 keys): dP in blocks of 16
// query rows x 64 keys, dV in blocks of 16 keys x 64 columns, in no particular place; the softmax backward, which needs whole
// rows, follows in a launch of its own (k_ds_finish).  Blocks 0 .. n_s - 1: dP; then dV; the last one ranks.
template <typename TV, int ROUNDS>
__global__ __launch_bounds__(256, 3) void k_bwd_pre_parts(const float *__restrict__ dC, const TV *__restrict__ V,
                                                       const float *__restrict__ P, const int *__restrict__ key_len,
                                                       float *__restrict__ dP, int *__restrict__ order,
                                                       float *__restrict__ dV, int B, int first, int Tq, int Tk, int Dv, int pitch,
                                                       int row_tiles, int parts, int with_ds, int acc) {
    extern __shared__ float s_dp[];
    __shared__ int s_len[kMaxSortedB];
    const int n_s = with_ds ? B * row_tiles * parts : 0;
    int id = blockIdx.x;
    if (id == (int)gridDim.x - 1) {
        rank_block(key_len, order, s_len, B, Tk, 1, first);
        return;
    }
    if (id < n_s) {
        const int b = id / (row_tiles * parts), rem = id % (row_tiles * parts);
        const int i0 = (rem / parts) * 16, j_first = (rem % parts) * kPartKeys;
        if (j_first >= clamp_len(key_len[b], Tk)) return;
        dscore_block_dsplit_lds<TV, ROUNDS, true>(dC, V, P, key_len, dP, nullptr, s_dp, b, i0, Tq, Tk, Dv, pitch, j_first);
        return;
    }
    id -= n_s;
    const int cols = (Dv + 63) / 64, keys = (Tk + 15) / 16;
    const int b = id / (cols * keys), rem = id % (cols * keys);
    dv_rows_block(P, dC, key_len, dV, s_dp, Tq, Tk, Dv, b, rem / cols, rem % cols, acc);
}

// dS = P (dP - sum_j P dP) in place of dP, a wave per query row; zeros at masked keys and pads, and the rows' sums.
__global__ __launch_bounds__(256) void k_ds_finish(const float *__restrict__ P, const int *__restrict__ key_len, float *dS,
                                                   float *__restrict__ ds_rowsum, int rows, int Tq, int Tk, int pitch) {
    const int row = blockIdx.x * 4 + wave_id();
    if (row >= rows) return;
    const int lane = lane_id();
    const int L = clamp_len(key_len[row / Tq], Tk);
    const float *p = P + (size_t)row * Tk;
    float *ds = dS + (size_t)row * pitch;
    constexpr int NP = 6;                                         // keys per lane held in registers (384)
    float pr[NP], dp[NP];
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        const int j = lane + 64 * c;
        pr[c] = j < L ? p[j] : 0.f;
        dp[c] = j < L ? ds[j] : 0.f;
    }
    float r = 0.f;
#pragma unroll
    for (int c = 0; c < NP; ++c) r = __builtin_fmaf(pr[c], dp[c], r);
    for (int j = lane + 64 * NP; j < L; j += 64) r = __builtin_fmaf(p[j], ds[j], r);
    r = wave_sum(r);
    float tot = 0.f;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        const int j = lane + 64 * c;
        const float x = pr[c] * (dp[c] - r);                      // zero at masked keys
        if (j < pitch) store_streaming(&ds[j], x);
        tot += x;
    }
    for (int j = lane + 64 * NP; j < pitch; j += 64) {
        const float x = j < L ? p[j] * (ds[j] - r) : 0.f;
        store_streaming(&ds[j], x);
        tot += x;
    }
    tot = wave_sum(tot);
    if (lane == 0) ds_rowsum[row] = tot;
}

// What the blocks of split operands take: at most 512 keys, 32-bit offsets within 32 rows of dC, a sample's V and its dC.
static bool split_fits(const AttnShape &s) { return s.Tk <= 512 && s.Dv < (1 << 20) && (long long)s.Tq * s.Dv < (1LL << 29); }

// k_bwd_pre's dS blocks take all keys and all of d; with few of them the shorter blocks win what the extra launch costs (4 to 5 us; B = 1, T = 400,
// Dv = 512 70 -> 14 us for the pre-kernel as it was on fp32 products).  Where they would be blocks of split operands, up to 50 blocks of 32 rows:
// backward on these against parts, 150 shapes of 129 to 512 keys, up to 14 blocks 1.17 of the time, to 29 1.12, to 44 1.03, to 59 0.98, to 74
// 0.96, to 200 0.75 to 0.97.  Where they would be fp32 blocks of 16 rows, up to 100, 200 where the rows are wide: without parts B = 8, T = 600,
// H = Dv = 512 468 -> 523 us, bf16 B = 5, T = 600, Dv = 512 91 -> 189; 22 shapes of more than 512 keys 1.28 (0.99 to 2.07).
static int most_parts_fp32(const AttnShape &s) { return s.Dv >= 384 ? 200 : 100; }
bool bwd_pre_in_parts(const AttnShape &s) {
    const int most = split_fits(s) ? 50 : most_parts_fp32(s);
    return s.Tk > kDsplitMaxTk && s.Dv <= 1024 && s.B <= kMaxSortedB && (long long)s.B * ((s.Tq + 31) / 32) <= most;
}

template <typename TV, int ROUNDS>
static hipError_t launch_parts_t(const AttnShape &s, const float *dC, const void *V, const float *P, const int *key_len,
                                 float *dS, int *order, float *dV, hipStream_t st, bool with_ds, int first) {
    const int row_tiles = (s.Tq + 15) / 16, parts = (s.Tk + kPartKeys - 1) / kPartKeys;
    const long long blocks = 1 + (with_ds ? (long long)s.B * row_tiles * parts : 0) +
                             (long long)s.B * ((s.Dv + 63) / 64) * ((s.Tk + 15) / 16);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = (size_t)(4 * 16 * kStagePitch + (ROUNDS > 1 ? 64 * (kPartKeys + 4) : 0)) * sizeof(float);
    if (lds > 48 * 1024) {
        static LdsGrants granted;
        hipError_t e = ensure_dynamic_lds((const void *)k_bwd_pre_parts<TV, ROUNDS>, lds, granted);
        if (e != hipSuccess) return e;
    }
    k_bwd_pre_parts<TV, ROUNDS><<<(unsigned)blocks, 256, lds, st>>>(dC, (const TV *)V, P, key_len, dS, order, dV, s.B, first, s.Tq,
                                                                    s.Tk, s.Dv, ds_pitch(s.Tk), row_tiles, parts,
                                                                    with_ds ? 1 : 0, s.acc ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_ds_finish(const AttnShape &s, const float *P, const int *key_len, float *dS, float *ds_rowsum, hipStream_t st) {
    const int rows = s.B * s.Tq;
    k_ds_finish<<<(rows + 3) / 4, 256, 0, st>>>(P, key_len, dS, ds_rowsum, rows, s.Tq, s.Tk, ds_pitch(s.Tk));
    return hipGetLastError();
}

hipError_t launch_bwd_pre(const AttnShape &s, const float *dC, const void *V, const float *P, const int *key_len,
                          float *dS, float *ds_rowsum, int *order, float *dV, int first, hipStream_t st, bool with_ds) {
    const int sorted = s.B <= kMaxSortedB ? 1 : 0;
    if (!sorted) first = 0;
    if (bwd_pre_in_parts(s)) {
        if (s.Dv <= 512)
            return s.bf16 ? launch_parts_t<bf16_t, 1>(s, dC, V, P, key_len, dS, order, dV, st, with_ds, first)
                          : launch_parts_t<float, 1>(s, dC, V, P, key_len, dS, order, dV, st, with_ds, first);
        return s.bf16 ? launch_parts_t<bf16_t, 2>(s, dC, V, P, key_len, dS, order, dV, st, with_ds, first)
                      : launch_parts_t<float, 2>(s, dC, V, P, key_len, dS, order, dV, st, with_ds, first);
    }
    // Split operands (KW > 0) for what their blocks take (split_fits).  Not where tiles of 32 would be mostly empty, nor, in f32, on few
    // blocks, where latency decides and the splitting of both operands is a part of it (backward, 350 shapes of up to 128 keys: at most 16
    // rows or 16 keys 1.02 of the time of the fp32 form, up to 1.13; fewer than 64 blocks of 32 rows 1.00 in f32, 0.75 to 1.12, and 0.92 in
    // bf16; 64 to 160 blocks 0.94; more and longer ones 0.93, see dscore_split_block).
    const long long blocks32 = (long long)s.B * ((s.Tq + 31) / 32);
    // dV alone (the keys' call of the decoder) on short key axes: blocks of 64 columns up to two rounds of them (512 of them 5.8 us against 7.8;
    // 2048 19.4 against 13).
    const bool few_dv = !with_ds && s.Tk <= 64 && (long long)s.B * ((s.Dv + 63) / 64) <= 1024;
    // dV alone of few rows, any number of keys: a step of 64 rows and the splitting of all of dC for it are a waste there (fp32 blocks over
    // split ones, 129 to 500 keys: 29 launches of up to 12 rows 0.95 of the time, 0.92 to 1.01; 16 rows and more level).  With dS, whose rows
    // of V are split once for up to 32 rows of dC, split operands stay ahead past 128 keys at any number of rows: 51 shapes of 1 to 16
    // rows 0.87 of the time that the backward takes on the fp32 forms (0.47 to 1.25; at 64 value columns 0.99, 0.87 to 1.19).
    const bool few_rows_dv = !with_ds && s.Tq <= 12;
    const bool small = s.Tk <= 128 && (s.Tq <= 16 || s.Tk <= 16 || (with_ds && !s.bf16 && blocks32 < 64) || few_dv);
    // f32, 65 to 128 keys, value rows that fill the four waves' 128 columns of the fp32 form to seven eighths and more, and a block for every CU:
    // there the launch itself gains least from split operands (B = 128, T = 100, Dv = 512 39 -> 33 us), and on cards that answer dense bf16
    // products with a lower shader clock the launches around it lose more, one block per CU or two.  Forward and backward over fp32 products on
    // a card that reacts and on one that does not: ten shapes inside 1.03 (0.99 to 1.05) and 0.97 (0.93 to 1.03); 384 to 447 columns 0.98
    // (0.92 to 1.01) and 0.95; more than 512 0.93 (0.90 to 0.98) and 0.91; 448 to 512 and fewer blocks 0.96 and 0.94.
    const bool dense = with_ds && !s.bf16 && s.Tk > 64 && s.Tk <= 128 && s.Dv >= 448 && s.Dv <= 512 && blocks32 >= 256;
    const int kw = !split_fits(s) || small || few_rows_dv || dense ? 0 : s.Tk <= 64 ? 1 : s.Tk <= 128 ? 2 : 8;
    // fp32 products past 128 keys: dV in panels of 64 keys where P rows allow 16-byte loads and the panels still fill the chip, or there are
    // few rows to share a block's start among (blocks of 16 keys over panels: 28 shapes of 516 to 1000 keys with 800 panels and more 1.02 of the
    // backward's time, 0.98 to 1.07; ten of 96 to 793 panels 0.94, 0.86 to 0.99; up to 12 rows and 132 to 500 keys 1.03, 1.00 to 1.09).
    const bool panels = kw == 0 && s.Tk > kDsplitMaxTk && s.Tk % 4 == 0 &&
                        (s.Tq <= 16 || s.B * ((s.Dv + 255LL) / 256) * ((s.Tk + kDvKeys - 1) / kDvKeys) >= 800);
    // Few blocks of split operands past 128 keys: short runs of products are summed on their own, as the parts, which these grids ran in on fp32
    // products, sum in four shorter chains.  Error against float64 of dV and dP (300 keys, T = 300, Dv = 512): parts 1.6e-7 and 2.3e-7, one
    // chain of split products 2.6e-7 and 3.5e-7, this 1.0e-7 and 1.4e-7, for 0.5 to 1.5 % of forward and backward, 1 to 5 % (once 9) of the
    // backward where there are few rows.  On more blocks one chain of fp32 products, 3.1e-7 and 4.2e-7, came before.
    const bool apart = kw == 8 && blocks32 <= most_parts_fp32(s);
    const int s_rows = kw ? 32 : 16;
    const int s_tiles = with_ds ? (s.Tq + s_rows - 1) / s_rows : 0;
    const int v_groups = dv_col_groups(kw, s.Tk, s.Dv) * dv_key_groups(kw, panels, s.Tk);
    const long long blocks = 1 + 8LL * ((s.B + 7) / 8) * (s_tiles + (long long)v_groups);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const int pitch16 = (s.Tk + 15) / 16 * 16 + 4;
    // short key axes: four planes of 16 rows, or (one round over d) the four waves' staging regions, which the
    // planes then share
    const size_t ds_lds = s_tiles == 0          ? 0
                          : kw > 0              ? (size_t)split_lds_floats(kw, s.Tk) * sizeof(float)
                          : s.Tk > kDsplitMaxTk ? (size_t)s_rows * pitch16 * sizeof(float)
                          : s.Dv <= 512         ? (size_t)4 * 16 * kStagePitch * sizeof(float)
                          : s.Dv <= 1024        ? (size_t)(4 * 16 * kStagePitch + 64 * pitch16) * sizeof(float)
                                                : (size_t)64 * pitch16 * sizeof(float);
    // One block per CU, by asking for more than half of its LDS, for f32 on long key axes and wide value rows, once there is a dS block for every
    // CU and they are full to three quarters.  Two of them keep the matrix cores so busy with dense bf16 products that some cards lower the
    // shader clock, by up to 10 %, for the launches around this one too; one does not, and loses less than that.  Forward and backward
    // over fp32 products, two blocks and one: B = 32, T = 300, H = 1024 0.97 to 1.00 and 0.94 on a card that reacts, 0.92 and 0.93 on three that do not; twice the samples 1.05 and 0.97,
    // 0.97 and 0.97; 24 shapes of 200 to 480 keys that take this line 1.01 (0.87 to 1.05) and 0.95 (0.89 to 1.00), 0.92 and 0.94; with 400
    // columns 1.01 and 1.03 on the first.  From 129 to 192 keys, where waves have no key tile, 1.01 (up to 1.07) and 0.99, 0.93 and 0.96.
    // Blocks of few rows do not make them busy (256 samples of 4 and 16 rows, 300 and 200 keys, 1024 columns: two blocks 152 and 111 us for the
    // backward, one 176 and 135).
    const bool alone = kw == 8 && with_ds && !s.bf16 && s.Tk > 192 && s.Dv >= 512 && blocks32 >= 256 &&
                       4LL * s.B * s.Tq >= 3 * 32 * blocks32;
    const size_t lds = std::max(ds_lds, alone ? kAloneLdsBytes : kw ? (size_t)kDvSplitLdsBytes : (size_t)0);
#define ECHO_PRE_LAUNCH(TV, KW, ALT)                                                                                \
    do {                                                                                                            \
        if (lds > 48 * 1024) { /* beyond the default dynamic LDS limit (up to 160 KB per block on gfx950) */        \
            static LdsGrants granted;                                                                               \
            hipError_t e = ensure_dynamic_lds((const void *)k_bwd_pre<TV, KW, ALT>, lds, granted);                  \
            if (e != hipSuccess) return e;                                                                          \
        }                                                                                                           \
        k_bwd_pre<TV, KW, ALT><<<(unsigned)blocks, KW ? 512 : 256, lds, st>>>(                                      \
            dC, (const TV *)V, P, key_len, dS, ds_rowsum, order, dV, s.B, sorted, first, s.Tq, s.Tk, s.Dv,          \
            ds_pitch(s.Tk), s_tiles, s_rows, s.acc ? 1 : 0);                                                        \
    } while (0)
#define ECHO_PRE_KW(TV)                                 \
    switch (kw) {                                       \
        case 1: ECHO_PRE_LAUNCH(TV, 1, false); break;   \
        case 2: ECHO_PRE_LAUNCH(TV, 2, false); break;   \
        case 8:                                         \
            if (apart) ECHO_PRE_LAUNCH(TV, 8, true);    \
            else ECHO_PRE_LAUNCH(TV, 8, false);         \
            break;                                      \
        default:                                        \
            if (panels) ECHO_PRE_LAUNCH(TV, 0, true);   \
            else ECHO_PRE_LAUNCH(TV, 0, false);         \
            break;                                      \
    }
    if (s.bf16) {
        ECHO_PRE_KW(bf16_t)
    } else {
        ECHO_PRE_KW(float)
    }
#undef ECHO_PRE_KW
#undef ECHO_PRE_LAUNCH
    return hipGetLastError();
}

}  // namespace echo
