// tridiag.hip -- Householder reduction of Gram matrices by groups of
// workgroups that keep the matrix on the chip, for sides from SVD_GROUP_MIN to
// SVD_GROUP_MAX (the singular values of an unfolding are the square roots of
// its Gram matrix's eigenvalues; Section 4.2, "Matching Equivalent Tensors").
//
// One group of G workgroups reduces one n x n matrix.  Local row j of member w
// is matrix row j G + w, so every member keeps work as the matrix shrinks; a
// member's rows stay in its registers and LDS for the whole reduction (above
// side 3072 a few do not fit: they are the first to retire and live in L2), so
// a step reads and writes no memory beyond what the members tell each other.
// A step has one exchange: every member publishes p_i = beta (A u)_i of its own
// rows, and the owner of the next row that row.  Each member then derives by
// itself the whole w = p - K u, the updated next row, and from it the next
// reflector, whose products with the member's rows start the next step.
//
// Exchange: a double travels as two 64-bit words, each half of it beside a
// 32-bit step number.  A reader polls the words it needs until both carry the
// step (64-bit relaxed atomics at device scope: a word is never seen in
// parts, and no order between words is assumed, so no fence or flush is
// needed).  Two buffers alternate: a member writes step k's words only after
// it has read all of step k - 1's, whose writers had by then read step
// k - 2's.  The words start at zero, which no step carries.  Every poll is
// bounded in time; a member that gives up marks the call failed and leaves,
// and the others follow when their own waits end, about a second in all (a look
// at the mark in the polls cost every step 1 %).  The members are launched
// cooperatively (all resident together; the runtime puts cooperative launches
// of several streams one after the other).
//
// What bounds it: the exchange, about 2 us for 8 members and 3.4 us for 256 (a
// probe that exchanges n doubles and does nothing else), then the latency of
// a step's two workgroup reductions.  Words in the order in which members
// write them (four to a 64-byte piece) matter: scattered 16-byte writes made
// the same exchange 4.4 to 5.9 us.  Measured per reduction, against four
// launches a step over the whole device (above 512) or one workgroup working
// from L2 (up to 512): side 512 1.67 ms (21.9), 768 2.6 ms (about 20), 1024 3.7
// ms, 2048 9.6 ms, 3072 17.2 ms, 4096 46.6 ms (218); eight matrices of side
// 512, or four of 768, take the time of one.  Side 4096 is another matter: its
// first 1,024 steps take 29.7 ms, 29 us each against 7.4 us in the class below.
// Beside the four rows that a member then keeps in memory, the kernel of that
// class spills 128 vector registers (244 bytes of scratch a lane).

#include <algorithm>
#include <cfloat>

#include "mag_internal.hpp"

namespace mag {

namespace {

constexpr int TG_WAVES = 8;  // most waves of a member
constexpr int TG_RUN = 4;  // consecutive slots of one member (one 64-byte piece of words)
constexpr int TG_MAX_ROWS = 16;  // rows of one member, all kinds
// 0.25 s of the 100 MHz wall clock for one wait; the waits of a step (four to
// six, an exchange takes microseconds) follow one another
constexpr uint64_t TG_PATIENCE = 25000000ull;

template <int CTRL>
__device__ __forceinline__ double dpp_row(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// sum over the 16 lanes of a row, in every lane of it (rotations by 8, 4, 2, 1)
__device__ __forceinline__ double row_total(double x)
{
    x += dpp_row<0x128>(x);
    x += dpp_row<0x124>(x);
    x += dpp_row<0x122>(x);
    x += dpp_row<0x121>(x);
    return x;
}

// lanes 0..31: a summed over lane pairs (l, l + 32); lanes 32..63: b likewise
__device__ __forceinline__ double fold32(double a, double b)
{
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

// rows 0 and 2 of 16 lanes: a summed with the row after; rows 1 and 3: b
// summed with the row before
__device__ __forceinline__ double fold16(double a, double b)
{
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

// sums of four values over the wave: row r of 16 lanes holds value
// {0, 2, 1, 3}[r] in every lane
__device__ __forceinline__ double wave_total4(double a, double b, double c, double d)
{
    return row_total(fold16(fold32(a, b), fold32(c, d)));
}

__device__ __forceinline__ double wave_total1(double a)
{
    return row_total(fold16(fold32(a, a), fold32(a, a)));
}

// a lane's value as a scalar
__device__ __forceinline__ double lane_value(double v, int l)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// a uniform value that the compiler takes as new here: what is computed from
// it is not computed ahead of the loop around and kept in registers
__device__ __forceinline__ int scalar_here(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ void put_word2(uint64_t* w, double v, uint32_t tag)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    __hip_atomic_store(w, ((uint64_t)tag << 32) | (uint32_t)b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, ((uint64_t)tag << 32) | (uint32_t)(b >> 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t get_word(const uint64_t* w)
{
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool both_carry(uint64_t a, uint64_t b, uint32_t tag)
{
    return (uint32_t)(a >> 32) == tag && (uint32_t)(b >> 32) == tag;
}

__device__ __forceinline__ double from_words(uint64_t a, uint64_t b)
{
    return __longlong_as_double((long long)((b << 32) | (uint32_t)a));
}

// N doubles of a step, element i in the two words `at` bytes past
// w + i * stride words; lanes whose bit i of `need` is clear do not want
// element i.  False: they did not come in time
template <int N>
__device__ __forceinline__ bool poll_words(const uint64_t* w, int stride, uint32_t at, unsigned need,
                                           uint32_t tag, double* v)
{
    uint64_t a[N], b[N];
    auto word = [&](int i) { return (const uint64_t*)((const char*)(w + i * stride) + at); };
#pragma unroll
    for (int i = 0; i < N; ++i) {
        a[i] = get_word(word(i));
        b[i] = get_word(word(i) + 1);
    }
    need &= (1u << N) - 1u;
    uint64_t since = 0;
    for (int spins = 0;; ++spins) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (((need >> i) & 1u) && both_carry(a[i], b[i], tag)) {
                v[i] = from_words(a[i], b[i]);
                need &= ~(1u << i);
            }
        if (need == 0) return true;
        if ((spins & 1023) == 1023) {
            const uint64_t now = wall_clock64();
            if (since == 0) since = now;
            if (now - since > TG_PATIENCE) return false;
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((need >> i) & 1u) {
                a[i] = get_word(word(i));
                b[i] = get_word(word(i) + 1);
            }
    }
}

// square root and reciprocal without the library's range checks (half its
// latency), for arguments from 2^-900 to 2^900: the hardware's estimates refined
// by Newton steps.  From an estimate off by up to 2^-24 (the reciprocal's was
// measured to 2^-24.4), none of 2e7 random arguments gave anything but the
// correctly rounded result
__device__ __forceinline__ double sqrt_near(double v)
{
    const double y = __builtin_amdgcn_rsq(v);
    double g = v * y, h = 0.5 * y;
    double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, v), h, g);
}

__device__ __forceinline__ double recip_near(double v)
{
    double r = __builtin_amdgcn_rcp(v);
    r = fma(r, fma(-v, r, 1.0), r);
    r = fma(r, fma(-v, r, 1.0), r);
    return fma(r, fma(-v, r, 1.0), r);
}

// a column with at most this much below its subdiagonal entry (squared) counts
// as reduced.  The entries of a Gram matrix of fp32 data lie between 2^-300
// and 2^300 in magnitude (zeros apart), so that leaving out entries below
// 2^-450 changes no eigenvalue that doubles can hold beside them
constexpr double TAIL_MIN = 0x1p-900;

__host__ __device__ constexpr int tg_dots(int q) { return q <= 2 ? 1 : q <= 4 ? 2 : 4; }

struct TgShared {
    double red[TG_WAVES][TG_MAX_ROWS + 4];  // the waves' parts of (A u)_i, then of w.u and u'.u
    double us[2][TG_MAX_ROWS + 2], ws[2][TG_MAX_ROWS + 2];  // u and w of the member's rows, by step parity
    double redt[TG_WAVES];
    double x0;
    int dead;
};

// Q: slots of a thread (a slot is one column, the same numbering as the rows'
// slots: slot s is run s / TG_RUN, run t of member t % G; local row
// (t / G) TG_RUN + s % TG_RUN of that member).  RR: rows of a member in
// registers; before them in local order come n_lds rows in LDS, and before
// those n_mem rows in the matrix itself.
//
// Step k, with A holding the updates of the steps before k - 1 and (u', w) the
// pending one of step k - 1:
//   p = beta (A u - u' (w.u) - w (u'.u)) of the member's rows goes out, with
//   the member's part of p.u; then the pending update is applied, while the
//   others' words are on their way; then w = p - K u, row k + 1 after step k
//   and the norm of its tail.  The owner of row k + 1 sends it out, with the
//   pending update, before its products, so that it arrives ahead of p.
// Every wave reads p_{k+1} and the members' parts of p.u itself, which leaves
// two workgroup barriers a step: for A u, and for the tail's norm.
template <int TH, int RR, int Q>
__global__ __launch_bounds__(TH) void k_tri_group(const TriGroupJobs jobs, int lost_at,
                                                  int32_t* failed)
{
    constexpr int WV = TH / 64;
    constexpr int RC = RR * Q <= 64 ? 8 : 4;  // register rows handled at a time
    constexpr int PQ = Q <= 4 ? Q : Q / 2;   // slots polled at a time
    constexpr int KD = tg_dots(Q);  // members a lane reads p.u of
    __shared__ TgShared sm;
    extern __shared__ double lds_rows[];  // [n_lds][Q * TH]
    int jb = 0;
    while (jb + 1 < jobs.count && (int)blockIdx.x >= jobs.job[jb + 1].wg0) ++jb;
    const TriGroupJob& job = jobs.job[jb];
    const int n = job.n, G = job.G, mem = (int)blockIdx.x - job.wg0;
    const int64_t lda = job.lda;
    double* const A = job.A;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n_mem = job.n_mem, n_out = n_mem + job.n_lds, rows = job.rows;
    constexpr int NS = Q * TH;  // slots that have words (those past job.slots are never written)
    // the member that stays to the end writes the tridiagonal form
    const bool lead = (n - 1) % G == mem;
    const int last_row = (n - 1 - mem) / G * G + mem;
    // words of a step: p at slot s, then row k + 1 at slot s, then the
    // members' parts of p.u
    uint64_t* const words = job.words;
    constexpr int wrow = 2 * NS, wdot = 4 * NS;
    constexpr size_t wstep = 4 * (size_t)NS + 2 * 64 * KD;

    int col[Q];              // column of a slot
    unsigned own_bits = 0u;  // slots that are rows of the member
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int s = tid + q * TH, run = s / TG_RUN;
        const int j = run / G * TG_RUN + s % TG_RUN, c = j * G + run % G;
        col[q] = (s < job.slots && c < n) ? c : -1;
        if (col[q] >= 0 && run % G == mem) own_bits |= 1u << q;
    }
    int dot_last[KD];  // last row of the members whose p.u the lane reads
#pragma unroll
    for (int i = 0; i < KD; ++i) {
        const int m = lane + 64 * i;
        dot_last[i] = m < G ? (n - 1 - m) / G * G + m : -1;
    }
    // the word of row tid of the member (the threads below `rows` publish p)
    const int p_at = 2 * ((tid / TG_RUN * G + mem) * TG_RUN + tid % TG_RUN);

    // the member's rows
    double a[RR][Q];
#pragma unroll
    for (int r = 0; r < RR; ++r) {
        const int i = (n_out + r) * G + mem;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            a[r][q] = (i < n && col[q] >= 0) ? A[(size_t)i * lda + col[q]] : 0.0;
    }
    for (int j = n_mem; j < n_out; ++j) {
        const int i = j * G + mem;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            lds_rows[(j - n_mem) * Q * TH + tid + q * TH] =
                (i < n && col[q] >= 0) ? A[(size_t)i * lda + col[q]] : 0.0;
    }
    // entry q of local row j, one of the member's
    auto entry = [&](int j, int q) -> double {
        double v = 0.0;
        if (j < n_mem) {
            if (col[q] >= 0) v = A[(size_t)(j * G + mem) * lda + col[q]];
        } else if (j < n_out) {
            v = lds_rows[(j - n_mem) * Q * TH + tid + q * TH];
        } else {
            const int jr = scalar_here(j - n_out);
#pragma unroll
            for (int r = 0; r < RR; ++r)
                if (jr == r) v = a[r][q];
        }
        return v;
    };

    // x: row k after step k - 1; the first one as it is
    double x[Q], u[Q], w[Q], un[Q];
    double tail = 0.0;
    if (tid == 0) sm.dead = *(volatile int32_t*)failed;  // (by a launch before this one)
    if (tid < TG_MAX_ROWS + 2) sm.us[0][tid] = sm.us[1][tid] = sm.ws[0][tid] = sm.ws[1][tid] = 0.0;
    __syncthreads();
    if (sm.dead) return;  // uniform
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        x[q] = col[q] >= 0 ? A[col[q]] : 0.0;
        u[q] = w[q] = 0.0;
        if (col[q] >= 2) tail += x[q] * x[q];
        if (col[q] == 1) sm.x0 = x[q];
        if (col[q] == 0 && lead) job.d[0] = x[q];
    }
    tail = wave_total1(tail);
    if (lane == 0) sm.redt[wave] = tail;
    __syncthreads();

    int m1 = 1 % G, j1 = 1 / G;  // member and local row of row k + 1
    const int steps = (mem == 0 && lost_at >= 0) ? min(lost_at, job.stop) : job.stop;
    for (int k = 0; k < steps; ++k) {
        const uint32_t tag = job.tag0 + (uint32_t)k + 1;
        uint64_t* const now = words + (tag & 1) * wstep;
        const int cur = k & 1, prev = cur ^ 1;

        // ---- the reflector of column k (every thread derives its scalars):
        // u = (x0 - alpha, x1, ...), H = I - beta u u^T
        tail = 0.0;
#pragma unroll
        for (int v = 0; v < WV; ++v) tail += sm.redt[v];
        const double x0 = sm.x0;
        const bool live = tail > TAIL_MIN;
        const double norm = sqrt_near(x0 * x0 + tail);
        const double alpha = (x0 >= 0.0) ? -norm : norm;
        const double u0 = live ? x0 - alpha : 0.0;
        if (tid == 0 && lead) job.e2[k] = live ? alpha * alpha : x0 * x0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            un[q] = (col[q] == k + 1) ? u0 : (live && col[q] > k + 1) ? x[q] : 0.0;
        }
        if (own_bits != 0u) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if ((own_bits >> q) & 1u) sm.us[cur][col[q] / G] = un[q];
        }
        // row k + 1, with the pending update
        if (mem == m1) {
            const double ui = sm.us[prev][j1], wi = sm.ws[prev][j1];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (col[q] > k)
                    put_word2(now + wrow + 2 * (tid + q * TH), fma(-ui, w[q], fma(-wi, u[q], entry(j1, q))), tag);
        }
        // slots whose columns are all reduced, and the member's first live row
        const int qdead = min((k + 1) / (TG_RUN * G) * (TG_RUN * G) / TH, Q - 1);
        const int j0 = (k + G - mem) / G;  // rows j >= j0 are matrix rows > k

        // ---- A u of the member's rows, w.u and u'.u
        double beta;
        {
            // (its division overlaps the products)
            beta = live ? 2.0 * recip_near(u0 * u0 + tail) : 0.0;
            double s1 = 0.0, s2 = 0.0;
            const int row = lane >> 4, v4 = ((row & 1) << 1) | (row >> 1);
#pragma unroll
            for (int g = 0; g < RR; g += RC) {
                double y[RC];
#pragma unroll
                for (int r = 0; r < RC; ++r) y[r] = 0.0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (Q > 2 && q < qdead) continue;
#pragma unroll
                    for (int r = 0; r < RC; ++r) y[r] = fma(a[g + r][q], un[q], y[r]);
                }
#pragma unroll
                for (int r = 0; r < RC; r += 4) {
                    const double s = wave_total4(y[r], y[r + 1], y[r + 2], y[r + 3]);
                    if ((lane & 15) == 0) sm.red[wave][n_out + g + r + v4] = s;
                }
                __builtin_amdgcn_sched_barrier(0);  // (registers: a chunk at a time)
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                s1 = fma(w[q], un[q], s1);
                s2 = fma(u[q], un[q], s2);
            }
            const double s = wave_total4(s1, s2, s1, s2);
            if ((lane & 15) == 0 && v4 < 2) sm.red[wave][TG_MAX_ROWS + v4] = s;
            // rows in memory: loaded once a step, for the product and the
            // pending update (dead columns are read too: u is zero there)
            for (int j = j0; j < n_mem; ++j) {
                const int i = j * G + mem;
                double* const row = A + (size_t)i * lda;
                const double ui = sm.us[prev][j], wi = sm.ws[prev][j];
                double z = 0.0, t[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) t[q] = row[max(col[q], 0)];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    z = fma(t[q], un[q], z);
                    t[q] = fma(-ui, w[q], fma(-wi, u[q], t[q]));
                }
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (col[q] > k) row[col[q]] = t[q];
                z = wave_total1(z);
                if (lane == 0) sm.red[wave][j] = z;
            }
            for (int j = max(j0, n_mem); j < n_out; ++j) {
                const double* lrow = lds_rows + (j - n_mem) * Q * TH + tid;
                double z = 0.0;
#pragma unroll
                for (int q = 0; q < Q; ++q) z = fma(lrow[q * TH], un[q], z);
                z = wave_total1(z);
                if (lane == 0) sm.red[wave][j] = z;
            }
        }
        __syncthreads();
        double pj = 0.0, uj = 0.0;  // of the member's row tid
        if (wave == 0) {
            double s = 0.0;
            const int jr = min(lane, TG_MAX_ROWS + 1);
#pragma unroll
            for (int v = 0; v < WV; ++v) s += sm.red[v][jr];
            const double t1 = lane_value(s, TG_MAX_ROWS), t2 = lane_value(s, TG_MAX_ROWS + 1);
            const bool mine = lane < rows && lane >= j0 && lane * G + mem < n;
            uj = sm.us[cur][jr];
            pj = beta * fma(-sm.us[prev][jr], t1, fma(-sm.ws[prev][jr], t2, s));
            if (!mine) pj = uj = 0.0;
            if (mine) put_word2(now + p_at, pj, tag);
            const double part = wave_total1(pj * uj);
            if (lane == 0) put_word2(now + wdot + 2 * mem, part, tag);
        }
        // a member whose last row this was leaves without reading the step's
        // words: the others do not wait for it again, so they may be reused
        if (last_row <= k + 1) return;

        // ---- the pending update, while the words travel (the rows' u and w as
        // scalars: lane r of every wave fetches row r's)
        {
            const int rl = n_out + min(lane, RR - 1);
            const double ul = sm.us[prev][rl], wl = sm.ws[prev][rl];
#pragma unroll
            for (int r = 0; r < RR; ++r) {
                const double ui = lane_value(ul, r), wi = lane_value(wl, r);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (Q > 2 && q < qdead) continue;
                    a[r][q] = fma(-ui, w[q], fma(-wi, u[q], a[r][q]));
                    // (done here: the compiler would move it behind the polls)
                    asm volatile("" : "+v"(a[r][q]));
                }
            }
        }
        for (int j = max(j0, n_mem); j < n_out; ++j) {
            const double ui = sm.us[prev][j], wi = sm.ws[prev][j];
            double* lrow = lds_rows + (j - n_mem) * Q * TH + tid;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                lrow[q * TH] = fma(-ui, w[q], fma(-wi, u[q], lrow[q * TH]));
        }

        // ---- row k + 1 and p from every member; p_{k+1} and p.u for the wave
        double p[Q], dots[KD], p1[1];
        {
            unsigned need = 0, need_dot = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                u[q] = un[q];
                p[q] = x[q] = 0.0;
                if (col[q] > k) need |= 1u << q;
            }
#pragma unroll
            for (int i = 0; i < KD; ++i) {
                dots[i] = 0.0;
                if (dot_last[i] > k) need_dot |= 1u << i;
            }
            const int p1_at = 2 * ((j1 / TG_RUN * G + m1) * TG_RUN + j1 % TG_RUN);
            const uint32_t at = 16u * (uint32_t)tid;
            constexpr int stride = 2 * TH;
            bool ok = true;
#pragma unroll
            for (int q = 0; q < Q; q += PQ)
                ok = ok && poll_words<PQ>(now + wrow + q * stride, stride, at, need >> q, tag, x + q);
#pragma unroll
            for (int q = 0; q < Q; q += PQ)
                ok = ok && poll_words<PQ>(now + q * stride, stride, at, need >> q, tag, p + q);
            ok = ok && poll_words<1>(now + p1_at, 0, 0u, 1u, tag, p1) &&
                 poll_words<KD>(now + wdot, 128, 16u * (uint32_t)lane, need_dot, tag, dots);
            if (!ok) sm.dead = 1;
        }
        double dot = dots[0];
#pragma unroll
        for (int i = 1; i < KD; ++i) dot += dots[i];
        dot = wave_total1(dot);

        // ---- w = p - K u, and row k + 1 after this step
        const double K2 = 0.5 * beta * dot;
        const double w0 = fma(-K2, u0, p1[0]);
        tail = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            w[q] = fma(-K2, u[q], p[q]);
            x[q] -= fma(u0, w[q], w0 * u[q]);
            if (col[q] > k + 2) tail += x[q] * x[q];
            if (col[q] == k + 2) sm.x0 = x[q];
            if (lead && col[q] == k + 1) job.d[k + 1] = x[q];
            // the last step leaves a corner: its off-diagonal entry, and the
            // last row's diagonal entry, which has this step's update to take
            if (lead && k + 3 == n && col[q] == n - 1) {
                job.e2[n - 2] = x[q] * x[q];
                job.d[n - 1] = fma(-2.0 * u[q], w[q], entry((n - 1) / G, q));
            }
        }
        if (wave == 0 && lane < TG_MAX_ROWS) sm.ws[cur][lane] = fma(-K2, uj, pj);
        tail = wave_total1(tail);
        if (lane == 0) sm.redt[wave] = tail;
        if (++m1 == G) {
            m1 = 0;
            ++j1;
        }
        __syncthreads();
        if (sm.dead) {  // uniform
            if (tid == 0) atomicOr(failed, 1);
            return;
        }
        // after the last step: the rest of the matrix, with the pending update,
        // for the group that takes over
        if (k + 1 == job.stop && job.stop != n - 2) {
            const int rl = n_out + min(lane, RR - 1);
            const double ul = sm.us[cur][rl], wl = sm.ws[cur][rl];
            int i = scalar_here(n_out * G + mem);  // (no row's address is kept through the loop)
            const int step = scalar_here(G);
#pragma unroll
            for (int r = 0; r < RR; ++r, i += step) {
                const double ui = lane_value(ul, r), wi = lane_value(wl, r);
                if (i <= k || i >= n) continue;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (col[q] > k)
                        A[(size_t)i * lda + col[q]] = fma(-ui, w[q], fma(-wi, u[q], a[r][q]));
            }
            i = scalar_here(mem);
            for (int j = 0; j < n_out; ++j, i += step) {
                if (i <= k || i >= n) continue;
                const double ui = sm.us[cur][j], wi = sm.ws[cur][j];
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (col[q] > k) {
                        double* v = &A[(size_t)i * lda + col[q]];
                        const double old =
                            j < n_mem ? *v : lds_rows[(j - n_mem) * Q * TH + tid + q * TH];
                        *v = fma(-ui, w[q], fma(-wi, u[q], old));
                    }
            }
        }
    }
    if (steps < job.stop && tid == 0) atomicOr(failed, 1);
}

// One workgroup of W waves per matrix, for sides up to min(W R, 64 C): lane l
// of every wave holds columns l, l + 64, ..., wave h the rows h, h + W, ... of
// them, all in registers.  Every wave keeps the step's vectors whole (entry c
// in lane c % 64), takes the rows' entries of them as scalars, and derives the
// step's scalars by itself, so a step has one barrier: for the waves' parts of
// A u, and row k + 1, through LDS.  The update with (u, w) and the products
// with the next reflector are one pass over the rows.
//
// What bounds it: instruction issue, one wave a SIMD: six lane reads and 3 C
// multiply-adds a row, and about 250 instructions for the rest of a step.
// Measured for the 192 matrices (sides 32 and 128) of 64 tensors [32, 128,
// 128]: 169 us, against 358 us for the matrix in LDS, eight waves and three
// barriers a step (187 us with range checks around the square root and the
// reciprocal, and the form stored entry by entry).
template <int W, int C>
struct OneShared {
    double part[2][W][64 * C];
    double row[2][64 * C];
};

// entry `at` (uniform) of a vector held C to a lane
template <int C>
__device__ __forceinline__ double entry_at(const double (&v)[C], int at)
{
    double s = lane_value(v[0], at & 63);
#pragma unroll
    for (int c = 1; c < C; ++c)
        if (at >> 6 == c) s = lane_value(v[c], at & 63);
    return s;
}

template <int W, int R, int C>
__device__ void tri_one(const double* A, int n, double* d, double* e2, OneShared<W, C>& sm)
{
    static_assert((64 * C) % (4 * W) == 0 && R % 4 == 0, "rows and lanes");
    const int lane = threadIdx.x & 63;
    const int h = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    double a[R][C];
    double x[C], u[C], w[C], un[C], y[C];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = r * W + h;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int col = lane + 64 * c;
            a[r][c] = (j < n && col < n) ? A[(size_t)j * n + col] : 0.0;
        }
    }
    double tail = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int col = lane + 64 * c;
        x[c] = col < n ? A[col] : 0.0;
        u[c] = w[c] = 0.0;
        if (col >= 2) tail += x[c] * x[c];
    }
    double dv[C], ev[C];  // the form's entries c, in their lanes
#pragma unroll
    for (int c = 0; c < C; ++c) {
        dv[c] = x[c];
        ev[c] = 0.0;
    }
    for (int k = 0; k + 1 < n; ++k) {
        // ---- the reflector of column k, from x: row k after step k - 1 (the last
        // step's is zero: its tail is)
        tail = wave_total1(tail);
        const double x0 = entry_at(x, k + 1);
        const bool live = tail > TAIL_MIN;
        const double norm = sqrt_near(x0 * x0 + tail);
        const double alpha = (x0 >= 0.0) ? -norm : norm;
        const double u0 = live ? x0 - alpha : 0.0;
        const double beta = live ? 2.0 * recip_near(u0 * u0 + tail) : 0.0;
        const double off = live ? alpha * alpha : x0 * x0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int col = lane + 64 * c;
            ev[c] = (col == k) ? off : ev[c];
            un[c] = (col == k + 1) ? u0 : (live && col > k + 1) ? x[c] : 0.0;
            y[c] = 0.0;
        }
        // ---- the update of step k - 1 and the products with u
        const int i0 = (k + W - h) / W;  // rows r >= i0 are matrix rows > k
#pragma unroll
        for (int g = 0; g < R; g += 4) {
            if (g + 4 <= i0) continue;
#pragma unroll
            for (int r = g; r < g + 4; ++r) {
                // row r W + h: lane (r W + h) % 64 of entry r W / 64
                const int vc = r * W / 64, l = r * W % 64 + h;
                const double ui = lane_value(u[vc], l), wi = lane_value(w[vc], l);
                const double ni = lane_value(un[vc], l);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    a[r][c] = fma(-ui, w[c], fma(-wi, u[c], a[r][c]));
                    y[c] = fma(a[r][c], ni, y[c]);
                }
            }
        }
        const int buf = k & 1;
#pragma unroll
        for (int c = 0; c < C; ++c) sm.part[buf][h][lane + 64 * c] = y[c];
        if ((k + 1) % W == h) {
            const int i = (k + 1) / W;
#pragma unroll
            for (int g = 0; g < R; g += 4) {
                if (i >> 2 != g >> 2) continue;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    double v = a[g][c];
#pragma unroll
                    for (int r = 1; r < 4; ++r)
                        if ((i & 3) == r) v = a[g + r][c];
                    sm.row[buf][lane + 64 * c] = v;
                }
            }
        }
        __syncthreads();
        double dot = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            double s = 0.0;
#pragma unroll
            for (int v = 0; v < W; ++v) s += sm.part[buf][v][lane + 64 * c];
            x[c] = sm.row[buf][lane + 64 * c];
            u[c] = un[c];
            w[c] = beta * s;
            dot = fma(w[c], un[c], dot);
        }
        // ---- w = p - K u, and row k + 1 after this step
        const double K2 = 0.5 * beta * wave_total1(dot);
        const double w0 = fma(-K2, u0, entry_at(w, k + 1));
        tail = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int col = lane + 64 * c;
            w[c] = col > k ? fma(-K2, u[c], w[c]) : 0.0;
            x[c] -= fma(u0, w[c], w0 * u[c]);
            if (col > k + 2) tail += x[c] * x[c];
            dv[c] = (col == k + 1) ? x[c] : dv[c];
        }
    }
    if (h == 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int col = lane + 64 * c;
            if (col < n) d[col] = dv[c];
            if (col + 1 < n) e2[col] = ev[c];
        }
    }
}

// sides up to 128 (four waves), by their own size
__global__ __launch_bounds__(256) void k_tri_small(const SvdTask* tasks)
{
    __shared__ union {
        OneShared<4, 1> one;
        OneShared<4, 2> two;
    } sm;
    const SvdTask& t = tasks[blockIdx.x];
    const int n = (int)t.K;
    if (n <= 32)
        tri_one<4, 8, 1>(t.gram, n, t.tri, t.tri + n, sm.one);
    else if (n <= 64)
        tri_one<4, 16, 1>(t.gram, n, t.tri, t.tri + n, sm.one);
    else if (n <= TRI_SMALL)
        tri_one<4, 32, 2>(t.gram, n, t.tri, t.tri + n, sm.two);
}

// sides up to 192 (eight waves)
__global__ __launch_bounds__(512) void k_tri_middle(const SvdTask* tasks)
{
    __shared__ OneShared<8, 3> sm;
    const SvdTask& t = tasks[blockIdx.x];
    const int n = (int)t.K;
    if (n > TRI_SMALL && n <= TRI_MIDDLE) tri_one<8, 24, 3>(t.gram, n, t.tri, t.tri + n, sm);
}

// the Gershgorin interval of each tridiagonal form, and the form as the counts
// read it: scaled by a power of two so that the interval lies within (-1, 1],
// the pairs {d_i, e2_{i-1}} side by side, padded to whole steps of STURM_STEP
// with diagonal entries above the interval (which change no count), and
// whether it splits: some squared off-diagonal is below SPLIT_MIN (a diagonal
// or block tensor, channels that are always zero)
constexpr int STURM_STEP = 8;
constexpr int PREP_THREADS = 256;
// With |d_i - x| <= 5 and e2 >= SPLIT_MIN, max(|p_i|, |p_{i-1}|) of the minors'
// recurrence falls by at most 6 / SPLIT_MIN a term (e2_{i-1} |p_{i-2}| <= |p_i| +
// 5 |p_{i-1}|), so the STURM_STEP terms between two scalings stay above
// 2^-(8 * 123) and none underflows
constexpr double SPLIT_MIN = 0x1p-120;
// an eigenvalue below this, of a form scaled to (-1, 1], counts as zero
constexpr double STURM_LEAST = 0x1p-323;

__global__ __launch_bounds__(PREP_THREADS) void k_tri_prep(const SvdTask* tasks)
{
    __shared__ double red[3][PREP_THREADS / 64];
    const SvdTask& t = tasks[blockIdx.x];
    const int n = (int)t.K, tid = threadIdx.x;
    const double* d = t.tri;
    const double* e2 = t.tri + n;
    double glo = INFINITY, ghi = -INFINITY, least = INFINITY;
    for (int i = tid; i < n; i += PREP_THREADS) {
        const double r = (i > 0 ? sqrt(e2[i - 1]) : 0.0) + (i + 1 < n ? sqrt(e2[i]) : 0.0);
        glo = fmin(glo, d[i] - r);
        ghi = fmax(ghi, d[i] + r);
        if (i + 1 < n) least = fmin(least, e2[i]);
    }
    for (int off = 32; off > 0; off >>= 1) {
        glo = fmin(glo, __shfl_xor(glo, off));
        ghi = fmax(ghi, __shfl_xor(ghi, off));
        least = fmin(least, __shfl_xor(least, off));
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = glo;
        red[1][tid >> 6] = ghi;
        red[2][tid >> 6] = least;
    }
    __syncthreads();
    for (int v = 0; v < PREP_THREADS / 64; ++v) {
        glo = fmin(glo, red[0][v]);
        ghi = fmax(ghi, red[1][v]);
        least = fmin(least, red[2][v]);
    }
    const double span = fmax(fabs(glo), fabs(ghi));
    // (a matrix of zeros, or one that is not finite, is left unscaled)
    const int ex = (span > 0.0 && span < INFINITY) ? ilogb(span) + 2 : 0;
    const double wide = span > 0.0 ? 2.0 * DBL_EPSILON : 0.0;
    double2* pairs = tri_pairs(t.tri, n);
    const int np = tri_padded(n);
    for (int i = tid; i < np; i += PREP_THREADS) {
        double2 v = make_double2(4.0, 0.0);
        if (i < n) {
            v.x = ldexp(d[i], -ex);
            v.y = i > 0 ? ldexp(ldexp(e2[i - 1], -ex), -ex) : 0.0;
        }
        pairs[i] = v;
    }
    if (tid == 0) {
        double* b = tri_bounds(t.tri, n);
        b[0] = ldexp(glo, -ex) - wide;
        b[1] = ldexp(ghi, -ex) + wide;
        b[2] = (double)ex;
        b[3] = ldexp(ldexp(least, -ex), -ex) >= SPLIT_MIN ? 0.0 : 1.0;
    }
}

// number of eigenvalues below x: the sign changes of the leading principal
// minors' sequence p_i = (d_i - x) p_{i-1} - e2_{i-1} p_{i-2}, scaled every
// STURM_STEP terms.  One fused multiply-add separates a term from the next
// (the ratio of successive terms, which needs no scaling, needs a division
// there).  Each term is exact for a matrix whose d_i - x and e2_{i-1} are off
// by a few units of rounding, as with the ratios.
typedef __attribute__((address_space(3))) const double2 lds_pair;

__device__ __forceinline__ int sturm_count(lds_pair* pairs, int steps, double x)
{
    double p = 1.0, pp = 0.0;
    uint32_t signs = 0u;
    int c = 0;
    for (int i = 0; i < steps; ++i) {
        double2 f[STURM_STEP];
#pragma unroll
        for (int u = 0; u < STURM_STEP; ++u) {
            f[u].x = pairs[i * STURM_STEP + u].x;
            f[u].y = pairs[i * STURM_STEP + u].y;
        }
#pragma unroll
        for (int u = 0; u < STURM_STEP; ++u) {
            const double np = fma(f[u].x - x, p, -(f[u].y * pp));
            pp = p;
            p = np;
            signs = __builtin_amdgcn_alignbit(signs, (uint32_t)((uint64_t)__double_as_longlong(p) >> 32), 31);
        }
        c += __popc((signs ^ (signs >> 1)) & ((1u << STURM_STEP) - 1u));
        const int s = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
        p = ldexp(p, s);
        pp = ldexp(pp, s);
    }
    return c;
}

// the same for a form that splits, whose terms may vanish: scaled at every term,
// and a term that is zero takes the sign opposite to the one before (x counts
// as above that minor's eigenvalue), so that the block after it starts from
// a nonzero term.  About three times the instructions of a term above
__device__ __forceinline__ int sturm_count_split(lds_pair* pairs, int steps, double x)
{
    double p = 1.0, pp = 0.0;
    uint32_t signs = 0u;
    int c = 0;
    for (int i = 0; i < steps; ++i) {
#pragma unroll
        for (int u = 0; u < STURM_STEP; ++u) {
            double np = fma(pairs[i * STURM_STEP + u].x - x, p, -(pairs[i * STURM_STEP + u].y * pp));
            if (np == 0.0) np = copysign(0x1p-1000, -p);
            const int s = -__builtin_amdgcn_frexp_exp(fmax(fabs(np), fabs(p)));
            pp = ldexp(p, s);
            p = ldexp(np, s);
            signs = __builtin_amdgcn_alignbit(signs, (uint32_t)((uint64_t)__double_as_longlong(p) >> 32), 31);
        }
        c += __popc((signs ^ (signs >> 1)) & ((1u << STURM_STEP) - 1u));
    }
    return c;
}

// every eigenvalue of the tridiagonal forms, G neighbouring lanes each (a
// power of two): a round counts at G points inside every eigenvalue's
// interval and keeps the part that holds it, to two units of rounding.  Below
// STURM_LEAST of the scaled span an eigenvalue is zero; a form that splits, which
// may have many of them, finds them by one count there.
// Counting at more points at once takes fewer, costlier rounds, so G is just
// large enough to give every SIMD a wave.  What bounds it: the LDS reads of a
// term's coefficients, the same for every lane, about 16 cycles for each of a
// CU's waves, then the issue of its five to six instructions.  Measured for
// 64 tensors [32, 128, 128] and for one side of 4096: 74 us and 1.43 ms; with
// the coefficients as scalars, requested a group ahead, 78 us and 1.59 ms (in
// the group that uses them 85 us, 1.95 ms); broadcast from a row of 16 lanes
// by DPP 83 us, 1.93 ms.
__global__ __launch_bounds__(STURM_LANES) void k_sturm(const SvdTask* tasks, int n_tasks,
                                                       int64_t n_items, int G)
{
    extern __shared__ double lds_rows[];  // a form's pairs
    const int64_t item = blockIdx.x;
    if (item >= n_items) return;  // uniform
    int lo_t = 0, hi_t = n_tasks - 1;  // the last task whose first item is <= item
    while (lo_t < hi_t) {
        const int mid = (lo_t + hi_t + 1) >> 1;
        if (tasks[mid].eig0 <= item) lo_t = mid; else hi_t = mid - 1;
    }
    const SvdTask& t = tasks[lo_t];
    const int n = (int)t.K, np = tri_padded(n);
    const double2* pairs = tri_pairs(t.tri, n);
    double2* const staged = reinterpret_cast<double2*>(lds_rows);
    for (int i = threadIdx.x; i < np; i += STURM_LANES) staged[i] = pairs[i];
    const double* b = tri_bounds(t.tri, n);
    double lo = b[0], hi = b[1];
    const int ex = (int)b[2];
    const bool split = __builtin_amdgcn_readfirstlane((int)b[3]) != 0;
    const int per = STURM_LANES / G;
    // (a group of lanes past the last eigenvalue has nothing to do)
    const int k = (int)(item - t.eig0) * per + (int)threadIdx.x / G, g = threadIdx.x % G;
    bool done = k >= n;
    __syncthreads();
    if (split) {
        if (sturm_count_split((lds_pair*)staged, np / STURM_STEP, STURM_LEAST) > k)
            done = true;  // (lo is not above zero)
        else
            lo = fmax(lo, STURM_LEAST);
    }
    for (int it = 0; it < 340; ++it) {
        done = done || !(hi - lo > 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + STURM_LEAST);
        if (__ballot(!done) == 0ull) break;
        const double h = (hi - lo) / (double)(G + 1);
        const double x = lo + h * (double)(g + 1);
        const int c = split ? sturm_count_split((lds_pair*)staged, np / STURM_STEP, x)
                            : sturm_count((lds_pair*)staged, np / STURM_STEP, x);
        double nlo = lo, nhi = hi;
        if (c <= k) nlo = fmax(nlo, x);
        else nhi = fmin(nhi, x);
        for (int off = 1; off < G; off <<= 1) {
            nlo = fmax(nlo, __shfl_xor(nlo, off));
            nhi = fmin(nhi, __shfl_xor(nhi, off));
        }
        if (nlo == lo && nhi == hi) done = true;  // no representable progress
        if (!done) {
            lo = nlo;
            hi = nhi;
        }
    }
    if (g == 0 && k < n)
        t.out[n - 1 - k] = lo <= 0.0 ? 0.0 : sqrt(ldexp(fmax(0.5 * (lo + hi), 0.0), ex));
}

// how a matrix of side n is spread over a group: rows per member (a multiple
// of TG_RUN), members, and where the rows are kept
constexpr int TG_LDS = 155 << 10;  // most LDS for a member's rows (beside TgShared)
static_assert(TG_LDS + sizeof(TgShared) <= 160 * 1024, "LDS of one workgroup");
struct TgShape {
    int th, q, rows, G, slots, n_mem, n_lds;
};

// classes by slots per thread: sides up to th * q take the first that they fit.
// n rounded up to whole members fits the slots, for rows divides them; the
// smallest group (side 193) has 13 members, the largest 256
struct TgClass {
    int th, q, rr, rows;
};
constexpr TgClass TG_CLASS[] = {
    {256, 2, 16, 16}, {512, 2, 16, 16}, {512, 4, 16, 16}, {512, 6, 8, 12}, {512, 8, 8, 16}};
constexpr bool tg_classes_fit()
{
    int top = 0;
    for (const TgClass& c : TG_CLASS) {
        const int slots = c.th * c.q;
        if (slots <= top || slots % c.rows || c.rows % TG_RUN || c.rows > TG_MAX_ROWS ||
            slots / c.rows > 64 * tg_dots(c.q) || c.th > 64 * TG_WAVES)
            return false;
        top = slots;
    }
    return top == SVD_GROUP_MAX;
}
static_assert(tg_classes_fit(), "rows, members and slots of the classes");

TgShape tg_shape(int n)
{
    int i = 0;
    while (n > TG_CLASS[i].th * TG_CLASS[i].q) ++i;  // n <= SVD_GROUP_MAX
    const TgClass& c = TG_CLASS[i];
    const int G = (n + c.rows - 1) / c.rows, out = c.rows - std::min(c.rows, c.rr);
    const int n_lds = std::min(out, TG_LDS / (int)(sizeof(double) * c.q * c.th));
    return TgShape{c.th, c.q, c.rows, G, c.rows * G, out - n_lds, n_lds};
}

// (a kernel's attribute belongs to the whole process: every call sets the same
// value, so that no other thread's launch meets a smaller one)
template <int TH, int RR, int Q>
hipError_t launch_group(const TriGroupJobs& jobs, int wgs, int lds, int lost_at,
                        int32_t* failed, hipStream_t stream)
{
    hipError_t e = hipFuncSetAttribute((const void*)k_tri_group<TH, RR, Q>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, TG_LDS);
    if (e != hipSuccess) return e;
    void* args[] = {(void*)&jobs, (void*)&lost_at, (void*)&failed};
    return hipLaunchCooperativeKernel((const void*)k_tri_group<TH, RR, Q>, dim3((unsigned)wgs),
                                      dim3(TH), args, (unsigned)lds, stream);
}

}  // namespace

bool tri_group_fits(int n)
{
    return n >= SVD_GROUP_MIN && n <= SVD_GROUP_MAX && tg_shape(n).G <= device_cu_count();
}

int tri_group_rounds(const int* n, int count)
{
    const int cus = device_cu_count();
    int rounds = 1, used = 0;
    for (int i = 0; i < count; ++i) {
        const int G = tg_shape(n[i]).G;
        if (used + G > cus) {
            ++rounds;
            used = 0;
        }
        used += G;
    }
    return rounds;
}

// A matrix is reduced class by class: when what is left of it fits the next
// smaller class, its rows go back to memory and a smaller group takes over (a
// step costs less the fewer members exchange words and the fewer slots a
// thread has), together with the matrices of the batch that start there.
hipError_t launch_tri_groups(TriMatrix* m, int count, int lost_at, int32_t* failed,
                             hipStream_t stream)
{
    const int cus = device_cu_count();
    const int limits[] = {SVD_GROUP_MAX, 3072, 2048, 1024, 512, 0};
    for (int level = 0; level + 1 < (int)(sizeof(limits) / sizeof(limits[0])); ++level) {
        const int top = limits[level], next = limits[level + 1];
        for (int i = 0; i < count;) {
            TriGroupJobs jobs{};
            int wgs = 0, lds = 0, cls = -1;
            for (; i < count && jobs.count < TRI_GROUP_JOBS; ++i) {
                if (m[i].n <= next || m[i].n > top) continue;
                const TgShape s = tg_shape(m[i].n);
                if (m[i].n < SVD_GROUP_MIN || s.G > cus) return hipErrorInvalidValue;
                if ((cls >= 0 && s.th * s.q != cls) || wgs + s.G > cus) break;
                cls = s.th * s.q;
                const int n = m[i].n, stop = next > 0 ? n - next : n - 2;
                jobs.job[jobs.count++] =
                    TriGroupJob{m[i].A, m[i].d, m[i].e2, m[i].words, m[i].lda, n, s.G, wgs, s.slots,
                                s.rows, s.n_mem, s.n_lds, stop, m[i].tag};
                wgs += s.G;
                lds = std::max(lds, s.n_lds * s.q * s.th * (int)sizeof(double));
                m[i].A += (size_t)stop * m[i].lda + stop;
                m[i].d += stop;
                m[i].e2 += stop;
                m[i].n = next > 0 ? next : 0;
                m[i].tag += (uint32_t)stop;
            }
            if (jobs.count == 0) break;
            hipError_t e;
            switch (cls) {
            case 512: e = launch_group<256, 16, 2>(jobs, wgs, lds, lost_at, failed, stream); break;
            case 1024: e = launch_group<512, 16, 2>(jobs, wgs, lds, lost_at, failed, stream); break;
            case 2048: e = launch_group<512, 16, 4>(jobs, wgs, lds, lost_at, failed, stream); break;
            case 3072: e = launch_group<512, 8, 6>(jobs, wgs, lds, lost_at, failed, stream); break;
            default: e = launch_group<512, 8, 8>(jobs, wgs, lds, lost_at, failed, stream); break;
            }
            if (e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

hipError_t launch_tri_one(const SvdTask* tasks, int n_tasks, bool small, bool middle,
                          hipStream_t stream)
{
    if (n_tasks <= 0) return hipSuccess;
    if (small)
        hipLaunchKernelGGL(k_tri_small, dim3((unsigned)n_tasks), dim3(256), 0, stream, tasks);
    if (middle)
        hipLaunchKernelGGL(k_tri_middle, dim3((unsigned)n_tasks), dim3(512), 0, stream, tasks);
    return hipGetLastError();
}

int sturm_lanes(int64_t values)
{
    // enough lanes to give every SIMD of the 256 CUs a wave (no device is
    // asked: the workspace's size follows from this)
    const int64_t lanes = 256 * 4 * 64;
    int G = 1;
    while (G < 32 && values * G * 2 <= lanes + lanes / 4) G *= 2;
    return G;
}

hipError_t launch_sturm(const SvdTask* tasks, int n_tasks, int64_t n_items, int G, int n_max,
                        hipStream_t stream)
{
    if (n_tasks <= 0) return hipSuccess;
    const int lds = tri_padded(n_max) * (int)sizeof(double2);
    hipError_t e = hipFuncSetAttribute((const void*)k_sturm,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       tri_padded(SVD_MAX_K) * (int)sizeof(double2));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tri_prep, dim3((unsigned)n_tasks), dim3(PREP_THREADS), 0, stream, tasks);
    hipLaunchKernelGGL(k_sturm, dim3((unsigned)n_items), dim3(STURM_LANES), (size_t)lds, stream,
                       tasks, n_tasks, n_items, G);
    return hipGetLastError();
}

}  // namespace mag
