// The fused recomputation (recompute.hip) in the form for samples of many query rows on grids of more than half of the blocks that run
// at a time (recompute_takes_rows: from about 280 of 512 on).
//
// k_recompute deals the query rows of a sample to eight waves, eight rows each at most, and meets at a barrier for every eight
// keys; what a wave adds to a key, one value per column and eight evaluations, passes through LDS.  Here a lane owns up to 25
// query rows, so that a key's partial sum leaves the registers twice per 25 evaluations, and a barrier comes once per 25 rows x 8 keys.
// Where the rows of a sample need only half of the waves, the lanes of a wave take different keys:
//
// Block = (sample, 64 columns of h), eight waves = G slices of 64 / G columns x 8 / G groups of query rows, G = 2 or 1 (up to
// 100 or 200 rows per pass).  The 64 lanes of a wave are G groups of 64 / G columns; lane group g takes the keys j with j % G = g of
// a step.  A step covers 8 G keys, eight per lane (the first one what is left over).  Per step a wave evaluates its rows one by one
// against eight keys; dQp stays in registers for the whole pass, the step's sums for dKp go to LDS, and behind the barrier the
// waves add them up over the row groups in fixed order and store them (first pass) or add them (later ones).  At the end of a pass
// the lane groups' dQp are added by lane exchanges and leave as whole rows.  Rows, keys and dS reach the lanes through LDS.
//
// Bound by issue slots, nine per tanh as in recompute.hip (five plain instructions and a reciprocal).  The register file decides its
// shape: a lane's rows are a compile-time number (15 to 25 with G = 2, 13 to 25 with G = 1), all waves evaluate as many, and a row that a wave does not
// have carries a zero dS; counted at run time the compiler keeps two copies of the sums.  No instance spills: with a dozen spilled
// registers the prologue alone took 10 us instead of 3 (T = 50, H = 512, B = 64).  Sums are kept in chains as short as
// recompute.hip's (dQp: eight keys, then the steps; dKp: halves of a lane's rows; dv: a step, then the steps), so that the errors
// against float64 are no larger: B = 57, T = 100, H = 512 dQp 4.7e-7 of the tensor's norm in both, dKp 2.0e-7 in both, dv 5.4e-7 in
// both; B = 30, T = 300, H = 1024 1.1e-6, 2.0e-7 and 6.8e-7, dv there 2.8e-6.
// Entries beyond the factor limit cost the wave or the step concerned an exponential and an addition per evaluation, and no digits.  The whole
// backward in us without such entries / with one row of them in every sample / with nothing else in a column: B = 128, T = 100, H = 512
// 122 / 137 / 158 (through k_recompute 144 / 144 / 165), B = 32, T = 304, H = 1024 629 / 680 / 866 (815 / 843 / 1092).
// Measured, the launch without the pre-kernel: B = 128, T = 100, H = 512 97 -> 82 us; B = 32, T = 300, H = 1024 455 -> 366.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace echo {

constexpr int RR_W = 8;                    // waves per block
constexpr int RR_THREADS = 64 * RR_W;
constexpr int RR_R = 25;                   // query rows a lane owns at most: what 128 registers hold
constexpr int RR_NJ = 8;                   // keys of a lane per step
constexpr int RR_COLS = 64;                // columns of h per block
constexpr int RR_ROUND = 512;              // blocks that run at a time: two on every compute unit

// One row of a lane against its first NJ (even) keys of the step.
//   BY_SUM false: x = exp(2q), fk = exp(2k)         r = 1 / (exp(2(q+k)) + 1) = 1 / (x fk + 1)
//   BY_SUM true : x = 2 log2e q, fk = 2 log2e k     r = 1 / (exp2(x + fk) + 1), for operands beyond the factor limit
// The empty statements keep the compiler from evaluating the first instructions of all rows up front and from moving the sums into
// a later block, either of which takes registers by the dozen.
template <int NJ, bool BY_SUM>
__device__ __forceinline__ void rr_row(float x, float (&fk)[RR_NJ], const float *__restrict__ d_row, float &acc_q,
                                       float (&acc_k)[RR_NJ], float (&acc_v)[4]) {
#pragma unroll
    for (int c = 0; c < NJ; ++c) asm volatile("" : "+v"(fk[c]));
    const float4 d0 = *reinterpret_cast<const float4 *>(d_row);
    const float4 d1 = NJ > 4 ? *reinterpret_cast<const float4 *>(d_row + 4) : d0;
    const float d[RR_NJ] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
    float r[NJ];
#pragma unroll
    for (int c = 0; c < NJ; ++c) r[c] = BY_SUM ? x + fk[c] : __builtin_fmaf(x, fk[c], 1.0f);
    trans_begin();
    if (BY_SUM) {
#pragma unroll
        for (int c = 0; c < NJ; ++c) r[c] = fast_exp2(r[c]);
#pragma unroll
        for (int c = 0; c < NJ; ++c) r[c] += 1.0f;
    }
#pragma unroll
    for (int c = 0; c < NJ; ++c) r[c] = fast_rcp(r[c]);
    trans_end();
    float q0 = 0.f, q1 = 0.f;
#pragma unroll
    for (int c0 = 0; c0 < NJ; c0 += 4) {
        float u[4];
#pragma unroll
        for (int c = c0; c < c0 + 4 && c < NJ; ++c) u[c - c0] = __builtin_fmaf(-r[c], r[c], r[c]);      // (1 - t^2) / 4
#pragma unroll
        for (int c = c0; c < c0 + 4 && c < NJ; ++c) {
            acc_k[c] = __builtin_fmaf(d[c], u[c - c0], acc_k[c]);
            float &q = (c & 1) ? q1 : q0;
            q = c < 2 ? d[c] * u[c - c0] : __builtin_fmaf(d[c], u[c - c0], q);
            acc_v[c & 3] = __builtin_fmaf(d[c], r[c], acc_v[c & 3]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    acc_q += q0 + q1;
    asm volatile("" : "+v"(acc_q), "+v"(acc_v[0]), "+v"(acc_v[1]), "+v"(acc_v[2]), "+v"(acc_v[3]));
#pragma unroll
    for (int c = 0; c < NJ; ++c) asm volatile("" : "+v"(acc_k[c]));
    __builtin_amdgcn_sched_barrier(0);
}

// grid (64-column pieces of h, samples in the order of the ranking)
template <typename T, int G, int R>
__global__ __launch_bounds__(RR_THREADS, 4) void k_recompute_rows(
    const T *__restrict__ Qp, const T *__restrict__ Kp, const T *__restrict__ v, const int *__restrict__ order,
    const float *__restrict__ dS, const float *__restrict__ ds_rowsum, float *__restrict__ dQp, float *__restrict__ dKp,
    float *dv_part, unsigned long long *dv_flag, unsigned long long epoch, float *__restrict__ dv, int Tq, int Tk, int H, int pitch,
    int rows_per_pass, int acc) {
    constexpr int W = RR_W;
    constexpr int HW = 64 / G;                             // columns of a wave
    constexpr int RG = W / G;                              // groups of query rows
    constexpr int STEP = RR_NJ * G;                        // keys of a step
    constexpr bool FRESH = R > (G == 1 ? 23 : 15);         // see fetch
    constexpr int ROWS = R * RG;                           // rows of a pass at most
    constexpr int DP = STEP;                               // a staged row of dS: [lane group][key of the group]
    constexpr int PART = W * RR_NJ * 64;                   // sums of a step for dKp: [wave][key of the lane][lane]
    // exp(2q) of the pass's rows, then the steps' sums (two buffers), then dQp of the pass's rows
    __shared__ __align__(16) float s_rows[ROWS * RR_COLS > 2 * PART ? ROWS * RR_COLS : 2 * PART];
    __shared__ float s_fk[2][STEP][RR_COLS];               // exp(2k) of a step's keys
    __shared__ __align__(16) float s_ds[2][ROWS * DP];
    __shared__ float s_dv[W][64];
    __shared__ float s_rowsum;
    __shared__ __align__(8) unsigned char s_kbig[2][W];    // a key that wave w has staged is beyond the factor limit
    __shared__ int s_qbig[RG];                             // a row of the group is
    __shared__ int s_seen[W];

    // the phases that wait on memory go first when they have something to issue: next to the loop of the CU's other block a
    // prologue would get hardly any issue slots
    __builtin_amdgcn_s_setprio(3);
    const int packed = order[blockIdx.y];
    const int b = packed & 0xffff, L = packed >> 16;
    const int lane = lane_id(), w = wave_id();
    const int slice = w % G, rg = w / G;
    const int col = slice * HW + lane % HW;                // this lane's column of the block's in the evaluations
    const int h0 = blockIdx.x * RR_COLS, ho = h0 + lane;   // and the column it loads and stores
    const bool hov = ho < H;
    const unsigned hoc = hov ? ho : H - 1;
    typename RawElem<T>::type vo_raw = RawElem<T>::load(v, hoc);

    float *dQb = dQp ? dQp + (size_t)b * Tq * H : nullptr;
    float *dKb = dKp + (size_t)b * Tk * H;
    if (!acc)                                              // masked keys: exact zeros (adding: they hold zeros already)
        for (int j = L + w; j < Tk; j += W)
            if (hov) dKb[(size_t)j * H + ho] = 0.f;
    if (L == 0 && dQp)
        for (int i = w; i < Tq; i += W)
            if (hov) dQb[(size_t)i * H + ho] = 0.f;
    auto sum_rows = [&]() {                                // sum of the sample's dS: the part of sum dS t that comes from t = 1 - 2 r
        float rs = 0.f;
        for (int i = lane; i < Tq; i += 64) rs += ds_rowsum[(size_t)b * Tq + i];
        rs = wave_sum(rs);
        if (lane == 0) s_rowsum = rs;
    };
    if (L == 0 && w == W - 1) sum_rows();

    // The sample's part of dv, sum dS t = sum dS - 2 sum dS r, leaves before dQp does, so that its trip to memory and back (see
    // send_part) passes behind that.
    const int n_slots = gridDim.y;
    unsigned long long *flags = dv_flag + (size_t)blockIdx.x * n_slots;
    auto put_part = [&]() {
        if (w == 0) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            float tot = 0.f;
            if (L > 0) {
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int k = 0; k < G; ++k) tot += s_dv[ln / HW + G * g][k * HW + ln % HW];
            }
            if (h0 + ln < H) store_agent(&dv_part[(size_t)b * H + h0 + ln], __builtin_fmaf(-2.f, tot, s_rowsum));
        }
    };
    auto put_flag = [&]() {
        if (w == 0) {
            wait_all_memory_ops();
            if (lane == 0) store_agent(&flags[b], epoch);
        }
    };
    float tot_v = 0.f;
    if (L > 0) {                                           // the same for the block
        const T *qb = Qp + (size_t)b * Tq * H, *kb = Kp + (size_t)b * Tk * H;
        const float *dsb = dS + (size_t)b * Tq * pitch;
        // the first step takes what is left over, n0 keys, the others STEP each
        const int n_steps = (L + STEP - 1) / STEP, n0 = L - (n_steps - 1) * STEP;
        // staging: a thread moves four neighbouring keys of a row; rows [row group][row of the group], zeros where a group has
        // fewer than R
        static_assert(ROWS * STEP <= 4 * RR_THREADS, "one piece per thread at most");
        constexpr int T_PER_ROW = STEP / 4;
        const int t_row = threadIdx.x / T_PER_ROW;
        const int t_rg = t_row / R;
        const BufferRows<T> k_rows(kb, (unsigned)L * (unsigned)H);
        const BufferRows<T> q_rows(qb, (unsigned)Tq * (unsigned)H);
        const BufferRows<float> d_rows(dsb, (unsigned)Tq * (unsigned)pitch);
        const unsigned row_bytes = (unsigned)H * (unsigned)sizeof(T);
        f32x4 dx;
        constexpr int KPW = STEP / W;                      // wave w stages, and later finishes, keys w and w + 8 of a step
        typename BufferRows<T>::Raw k_raw[KPW];
        // FRESH: what a step needs of the lane's number is formed anew from ln, a copy that the compiler cannot see through; kept
        // through the steps these addresses take the registers of several pairs of rows
        auto fetch = [&](int j0, unsigned d_at, int ln) {
            const unsigned at_col = (unsigned)min(h0 + ln, H - 1) * (unsigned)sizeof(T);
#pragma unroll
            for (int k = 0; k < KPW; ++k) k_raw[k] = k_rows.load_raw(at_col, (unsigned)min(j0 + w + W * k, L - 1) * row_bytes);
            dx = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(d_rows.rsrc, d_at, (unsigned)j0 * 4u, 0));
        };
        auto commit = [&](int buf, int ln, int cnt) {
            bool big = false;
#pragma unroll
            for (int k = 0; k < KPW; ++k) {
                const float x = BufferRows<T>::value(k_raw[k]);
                s_fk[buf][w + W * k][ln] = fast_exp2(kTwoLog2e * x);
                big |= fabsf(x) > kFactorLimit;
            }
            s_kbig[buf][w] = __any(big) ? 1 : 0;
            const int row_at = w * (64 / T_PER_ROW) + ln / T_PER_ROW, key = 4 * (ln % T_PER_ROW);
            if (row_at >= ROWS) return;
            float *row = &s_ds[buf][row_at * DP];
#pragma unroll
            for (int c = 0; c < 4; ++c) row[((key + c) % G) * RR_NJ + (key + c) / G] = key + c < cnt ? dx[c] : 0.f;
        };

        int pass = 0;
        for (int i_pass0 = 0; i_pass0 < Tq; i_pass0 += rows_per_pass, ++pass) {
            const int nrows = min(rows_per_pass, Tq - i_pass0);
            // the row that this thread stages, -1: none
            const int t_i = nrows * t_rg / RG + t_row - t_rg * R;
            const int i_t = t_rg < RG && t_i < nrows * (t_rg + 1) / RG ? i_pass0 + t_i : -1;
            const unsigned d_at = i_t >= 0 ? (unsigned)(i_t * pitch + 4 * (int)(threadIdx.x % T_PER_ROW)) * 4u : 0x80000000u;
            fetch(0, d_at, lane);
            // the rows, four columns per lane and four rows per wave-level load; positions [row group][row of the group]
            {
                constexpr int PER = (ROWS + 31) / 32;
                RawKey<T> xr[PER];
                int t = threadIdx.x;
                asm volatile("" : "+v"(t));                            // what is derived from it is not kept through the steps
                const int c4 = 4 * (t % 16);
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int at = t / 16 + 32 * u, g = at / R;
                    const int i = i_pass0 + nrows * g / RG + at - g * R;
                    const T *row = qb + (size_t)min(i, Tq - 1) * H + h0 + c4;     // rows that count nothing have a zero dS
                    if (h0 + c4 + 4 <= H) xr[u].load(row, 0);
                    else xr[u].load_some(row, H - h0 - c4);
                }
                if (pass == 0 && w == W - 1) sum_rows();
                asm volatile("" : "+v"(vo_raw));
                if (threadIdx.x < RG) s_qbig[threadIdx.x] = 0;
                lds_barrier();
#pragma unroll
                for (int u = 0; u < PER; ++u) xr[u].pin();
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int at = t / 16 + 32 * u;
                    const float4 x = xr[u].get();
                    if (ROWS % 32 == 0 || at < ROWS) {
                        *reinterpret_cast<float4 *>(&s_rows[at * RR_COLS + c4]) =
                            make_float4(fast_exp2(kTwoLog2e * x.x), fast_exp2(kTwoLog2e * x.y), fast_exp2(kTwoLog2e * x.z),
                                        fast_exp2(kTwoLog2e * x.w));
                        if (fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))) > kFactorLimit) s_qbig[at / R] = 1;
                    }
                }
            }
            commit(0, lane, n0);
            lds_barrier();
            float fq[R], acc_q[R];
#pragma unroll
            for (int a = 0; a < R; ++a) {
                fq[a] = s_rows[(rg * R + a) * RR_COLS + col];
                acc_q[a] = 0.f;
            }
            const bool q_big = __builtin_amdgcn_readfirstlane(s_qbig[rg]) != 0;
            lds_barrier();                                             // the region is used for the steps' sums from here on

            // Operands beyond the factor limit: the exponential of the sum, in all steps for a wave with such a row, in the step for
            // such a key.  2 log2e k of the step and, as its turn comes, 2 log2e q of a row are then read from memory (q kept in registers spills,
            // k in LDS beside exp(2k) costs the factor path 2 to 3 %); the sums and their order are those of the factor path.
            auto by_sum = [&](int st) {
                const uint2 f = *reinterpret_cast<const uint2 *>(&s_kbig[st & 1][0]);
                return q_big || __builtin_amdgcn_readfirstlane(f.x | f.y) != 0;
            };
            auto step = [&](auto n, auto mode, int st, int j0, int cnt) {
                constexpr int NJ = decltype(n)::value;                 // keys of a lane
                constexpr bool BY_SUM = decltype(mode)::value;
                const int buf = st & 1;
                const bool more = st + 1 < n_steps;
                int ln = lane;
                if (FRESH) asm volatile("" : "+v"(ln));
                float acc_k[RR_NJ], acc_v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < RR_NJ; ++k) acc_k[k] = 0.f;
                float fk[RR_NJ];
                unsigned at_col = 0;                                   // BY_SUM
                if constexpr (BY_SUM) {
                    at_col = (unsigned)min(h0 + slice * HW + ln % HW, H - 1) * (unsigned)sizeof(T);
                    typename BufferRows<T>::Raw raw[RR_NJ];
#pragma unroll
                    for (int k = 0; k < RR_NJ; ++k) raw[k] = k_rows.load_raw(at_col + (unsigned)min(j0 + k * G + ln / HW, L - 1) * row_bytes, 0);
#pragma unroll
                    for (int k = 0; k < RR_NJ; ++k) fk[k] = kTwoLog2e * BufferRows<T>::value(raw[k]);
                } else {
#pragma unroll
                    for (int k = 0; k < RR_NJ; ++k) fk[k] = s_fk[buf][k * G + ln / HW][slice * HW + ln % HW];
                }
                if (more) fetch(j0 + cnt, d_at, ln);
                int ds_at = (buf * ROWS + rg * R) * DP + ln / HW * RR_NJ;
                asm volatile("" : "+v"(ds_at));                        // one address, the rows are its immediate offsets
                const float *ds_tile = &s_ds[0][0] + ds_at;
                // the sums over the rows in two parts: shorter chains of additions
                auto first_part = [&]() {
#pragma unroll
                    for (int k = 0; k < NJ; ++k) {
                        s_rows[buf * PART + (w * RR_NJ + k) * 64 + ln] = acc_k[k];
                        acc_k[k] = 0.f;
                    }
                };
                if constexpr (BY_SUM) {
                    int i0 = i_pass0 + nrows * rg / RG;
                    asm volatile("" : "+s"(i0));                       // the rows' offsets are not kept through the steps
                    auto load = [&](int a) { return q_rows.load_raw(at_col, (unsigned)min(i0 + a, Tq - 1) * row_bytes); };
                    auto raw = load(0);
#pragma unroll
                    for (int a = 0; a < R; ++a) {
                        const float x = kTwoLog2e * BufferRows<T>::value(raw);
                        if (a + 1 < R) raw = load(a + 1);
                        rr_row<NJ, true>(x, fk, ds_tile + a * DP, acc_q[a], acc_k, acc_v);
                        if (a == R / 2 - 1) first_part();
                    }
                } else {
#pragma unroll
                    for (int a = 0; a < R; ++a) {
                        rr_row<NJ, false>(fq[a], fk, ds_tile + a * DP, acc_q[a], acc_k, acc_v);
                        if (a == R / 2 - 1) first_part();
                    }
                }
                tot_v += (acc_v[0] + acc_v[1]) + (acc_v[2] + acc_v[3]);
                if (FRESH) asm volatile("" : "+v"(ln));
                if (more) commit(buf ^ 1, ln, STEP);
#pragma unroll
                for (int k = 0; k < NJ; ++k) s_rows[buf * PART + (w * RR_NJ + k) * 64 + ln] += acc_k[k];
                lds_barrier();
                // the step's keys, finished by the waves in turn: lane = column, sums over the row groups in fixed order
                const int part0 = ln / HW, pcol = ln % HW;
#pragma unroll
                for (int k = 0; k < KPW; ++k) {
                    const int jj = w + W * k;
                    if (jj < cnt) {                                    // uniform
                        float tot = 0.f;
#pragma unroll
                        for (int g = 0; g < RG; ++g) tot += s_rows[buf * PART + ((part0 + G * g) * RR_NJ + jj / G) * 64 + (jj % G) * HW + pcol];
                        if (h0 + ln < H) {
                            float *dst = dKb + (size_t)(j0 + jj) * H + h0 + ln;
                            const float val = 4.f * RawElem<T>::value(vo_raw) * tot;
                            if (pass == 0 && !acc) store_streaming(dst, val);
                            else *dst = *dst + val;
                        }
                    }
                }
            };
            __builtin_amdgcn_s_setprio(0);
            int st = 0;
            const int pairs = (n0 + 2 * G - 1) / (2 * G);              // of keys of a lane in the first step
            if (pairs < 4 && !by_sum(0)) {
                if (pairs == 1) step(std::integral_constant<int, 2>(), std::false_type{}, 0, 0, n0);
                else if (pairs == 2) step(std::integral_constant<int, 4>(), std::false_type{}, 0, 0, n0);
                else step(std::integral_constant<int, 6>(), std::false_type{}, 0, 0, n0);
                st = 1;
            }
            auto full_step = [&](auto mode) {
                step(std::integral_constant<int, RR_NJ>(), mode, st, st == 0 ? 0 : n0 + (st - 1) * STEP, st == 0 ? n0 : STEP);
            };
            // (loops of their own: with the two kinds of step as branches of one loop the compiler keeps two copies of acc_q and spills)
            while (st < n_steps) {
                for (; st < n_steps && !by_sum(st); ++st) full_step(std::false_type{});
                for (; st < n_steps && by_sum(st); ++st) full_step(std::true_type{});
            }
            __builtin_amdgcn_s_setprio(3);
            const bool last = i_pass0 + rows_per_pass >= Tq;
            if (last) s_dv[w][lane] = tot_v;
            lds_barrier();                                             // everybody is done with the last step's sums
            if (last) put_part();
            if (dQp) {
                // the lane groups' sums (of two neighbouring rows lanes 32 and up keep the second), then whole rows out through LDS
                int l = lane;
                asm volatile("" : "+v"(l));
#pragma unroll
                for (int a = 0; a < R; a += G) {
                    const int a1 = a + 1 < R ? a + 1 : a;              // (an odd last row: both halves hold its sum)
                    const float x = G == 1 ? acc_q[a] : transpose_pair<32>(acc_q[a], acc_q[a1], l);
                    s_rows[(rg * R + (G == 1 || l < 32 ? a : a1)) * RR_COLS + slice * HW + l % HW] = x;
                }
                lds_barrier();
                if (last) put_flag();
                for (int at = w; at < ROWS; at += W) {
                    const int g = at / R, i = nrows * g / RG + at - g * R;
                    if (i < nrows * (g + 1) / RG && h0 + l < H)
                        store_streaming(dQb + (size_t)(i_pass0 + i) * H + h0 + l, 4.f * RawElem<T>::value(vo_raw) * s_rows[at * RR_COLS + l]);
                }
            }
            lds_barrier();   // the next pass stages its rows in the same place
        }
    }

    if (L == 0) {
        lds_barrier();                                     // the sum of the dS rows
        put_part();
    }
    if (L == 0 || !dQp) put_flag();
    if ((int)blockIdx.y != n_slots - 1) return;
    lds_barrier();                                   // s_dv is reused
    const float tot = sum_parts<RR_COLS, W>(dv_part, flags, n_slots, H, ho, epoch, [](int) { return false; }, &s_dv[0][0], s_seen);
    if (w == 0 && hov) dv[ho] = acc ? dv[ho] + tot : tot;
}

// passes over the rows with rg groups of them, and the rows per lane that they then take
static int rr_passes(int Tq, int rg) { return (Tq + RR_R * rg - 1) / (RR_R * rg); }
static int rr_rows(int Tq, int rg) {
    const int passes = rr_passes(Tq, rg), rows = (Tq + passes - 1) / passes;
    return (rows + rg - 1) / rg;
}

static int rr_groups(int Tq) { return Tq <= RR_R * RR_W / 2 ? 2 : 1; }

// Expected time of a launch in the units of recompute.hip's recompute_time (one row of a wave against eight keys of a lane): a step
// costs a lane's rows and about one more, a block about twenty (prologue, dQp, its part of dv).  Negative: not for this form.  Fewer
// than 60 rows leave a lane too few for the prologue to pay: over 504 shapes of 46 to 59 rows, 30 to 64 keys, half a round to eight rounds of
// blocks, both types, the backward takes 1.019 of k_recompute's time (0.94 to 1.10; ahead, by 0.2 %, at a round and a half alone; B = 64, T = 50,
// H = 512 29.6 us against 28.5, B = 128, T = 50, H = 1024 in bf16 71.6 against 70.5).  Rows are addressed by 32-bit byte offsets.
float recompute_rows_time(const AttnShape &s) {
    const long long e = s.bf16 ? 2 : 4, most = 1LL << 31, T = s.Tq > s.Tk ? s.Tq : s.Tk;
    if (s.Tq < 60 || T * s.H * e >= most || (long long)s.Tq * ds_pitch(s.Tk) * 4 >= most) return -1.f;
    const int g = rr_groups(s.Tq), step = RR_NJ * g;
    const float tile = rr_passes(s.Tq, RR_W / g) * (rr_rows(s.Tq, RR_W / g) + 1.f);
    const float full = tile * ((s.Tk + step - 1) / step) + 20.f, mean = 0.8f * tile * s.Tk / step + 20.f;
    const float blocks = (float)s.B * ((s.H + RR_COLS - 1) / RR_COLS), all = blocks / RR_ROUND * mean + 0.5f * mean;
    return blocks <= RR_ROUND || full > all ? full : all;
}

template <typename T, int G, int R>
static hipError_t launch_rows_r(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order, const float *dS,
                                 const float *ds_rowsum, float *dQp, float *dKp, float *dv_part, unsigned long long *dv_flag,
                                 unsigned long long epoch, float *dv, hipStream_t st) {
    const int passes = rr_passes(s.Tq, RR_W / G), rows_per_pass = (s.Tq + passes - 1) / passes;
    dim3 grid((s.H + RR_COLS - 1) / RR_COLS, s.B);
    k_recompute_rows<T, G, R><<<grid, RR_THREADS, 0, st>>>((const T *)Qp, (const T *)Kp, (const T *)v, order, dS, ds_rowsum, dQp, dKp, dv_part,
                                                            dv_flag, epoch, dv, s.Tq, s.Tk, s.H, ds_pitch(s.Tk), rows_per_pass, s.acc ? 1 : 0);
    return hipGetLastError();
}

// From 60 rows on with two groups of lanes, 15 to 25 per lane; from 101 with one, in one pass or in equal ones, 13 to 25.
template <typename T, int G>
static hipError_t launch_rows_t(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order, const float *dS,
                                const float *ds_rowsum, float *dQp, float *dKp, float *dv_part, unsigned long long *dv_flag,
                                unsigned long long epoch, float *dv, hipStream_t st) {
#define ECHO_R(N) \
    case N:                                                                                                                     \
        if constexpr (G == 1 || N >= 15)                                                                                        \
            return launch_rows_r<T, G, N>(s, Qp, Kp, v, order, dS, ds_rowsum, dQp, dKp, dv_part, dv_flag, epoch, dv, st);       \
        break
    switch (rr_rows(s.Tq, RR_W / G)) {
        ECHO_R(13); ECHO_R(14); ECHO_R(15); ECHO_R(16); ECHO_R(17); ECHO_R(18); ECHO_R(19); ECHO_R(20); ECHO_R(21); ECHO_R(22);
        ECHO_R(23); ECHO_R(24); ECHO_R(25);
        default: break;
    }
#undef ECHO_R
    return hipErrorInvalidValue;
}

hipError_t launch_recompute_rows(const AttnShape &s, const void *Qp, const void *Kp, const void *v, const int *order, const float *dS,
                                 const float *ds_rowsum, float *dQp, float *dKp, float *dv_part, unsigned long long *dv_flag,
                                 unsigned long long epoch, float *dv, hipStream_t st) {
    const bool two = rr_groups(s.Tq) == 2;
#define ECHO_ROWS(T)                                                                                                                  \
    return two ? launch_rows_t<T, 2>(s, Qp, Kp, v, order, dS, ds_rowsum, dQp, dKp, dv_part, dv_flag, epoch, dv, st)                    \
               : launch_rows_t<T, 1>(s, Qp, Kp, v, order, dS, ds_rowsum, dQp, dKp, dv_part, dv_flag, epoch, dv, st)
    if (s.bf16) ECHO_ROWS(bf16_t);
    ECHO_ROWS(float);
#undef ECHO_ROWS
}

}  // namespace echo
