// Exponential windows by sliding sums (FP64).
//
// For one tau and one channel y (a^2, b^2, ab with u = e^(-2 T_sft / tau);
// Re / Im of F_a, F_b of a bin with u = e^(-T_sft / tau)) the window of row m
// holds the slots [lo, hi), lo = clamp(k0_m, 0, K), hi = clamp(k0_m + L_m, 0,
// K), L_m = ceil((3 tau - delta_m) / T_sft) (section 2, eq. winexp), and its
// sum normalised to slot lo is
//   G_m = sum_{k in [lo, hi)} u^(k - lo) y_k.
// The row's own scale e^(-(t_lo - t0_m) / tau), squared on A, B, C, cancels
// in 2F = 2 (B |F_a|^2 + A |F_b|^2 - 2 C Re F_a F_b*) / D and in the
// degenerate-window rule, so G is all a cell needs.  Going down the rows both
// window ends move down: a slot entering at the front is G <- u G + y, a slot
// leaving at the back is G <- G - u^(k - lo) y_k.  Section 3 finds no reuse
// of the exponential sums across tau; along t0 there is one, and a cell costs
// the slots between two rows instead of its whole window.
//
// Lane = tau, wave = 64 taus x BG bins x one segment of rows, from the
// segment's last row down.  A front slot is the same in every lane (scalar
// loads); a back slot is the lane's own (gathered from a stage in LDS, or
// through the caches where the taus of a wave span too many slots).  A
// segment starts from H(k) = sum_{j >= k} u^(j - k) y_j at its last row's two
// ends, G = H(lo) - u^(hi - lo) H(hi); slide_anchor_kernel leaves H at every
// range_len-th slot.
//
// Errors.  The factors are below one, so rounding errors fade with the
// weights.  A slot enters by multiplications with the rounded rho and leaves
// with a weight of its own, so what it leaves behind is up to n 2^-53 of it, n
// the slots that the segment slid since (strong slots side by side add up).  A
// cell whose A or B is below 2^-13 of the largest slot's a^2 or b^2 (an empty
// window, or one of weak SFTs only) is summed directly, so that the degenerate
// rule decides as on direct sums (D keeps about 38 bits of A B for n of a few
// slots).  What data may spread over (set_ranges in the runtime) follows from
// the same: simulated with a stretch of 64 strong slots, windows of 1200 slots
// and segments of 3000 rows, the cells after it are off by 3e-12 in 2F at a
// spread of 2^10 (double precision slides up to that) and 2e-9 at 2^19 (the
// others up to 2^20); 5e-14 without.  Atoms beyond, or not finite, keep the
// direct forms.
#include "tfstat_device.h"

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <stdint.h>

namespace tfs {

namespace {

template <typename T>
using ConstParams = const __attribute__((address_space(4))) T;
template <typename T>
__device__ inline ConstParams<T> *const_ptr(const T *p) {
    return reinterpret_cast<ConstParams<T> *>(reinterpret_cast<uintptr_t>(p));
}

// The lane's tau: decay per slot and 3 tau in slots (q) and seconds left (r).
struct LaneTau {
    double c;        // ln rho = -T_sft / tau
    double rho, rho2;
    int q, r;
};

__device__ inline LaneTau lane_tau(int64_t tau, int64_t T) {
    LaneTau t;
    t.c = -(double)T / (double)tau;
    t.rho = exp(t.c);
    t.rho2 = exp(2.0 * t.c);
    span_qr(tau, 3, T, t.q, t.r);
    return t;
}

__device__ inline int clamp_slot(int k, int K) { return min(max(k, 0), K); }
// End slot of the window of row (k0, delta) for 3 tau = q T + r: slots
// k0 .. k0 + L - 1 with L = q + (r > delta).
__device__ inline int end_slot(int k0, int delta, int q, int r, int K) {
    return clamp_slot(k0 + q + (r > delta ? 1 : 0), K);
}

// h <- f h + y with y in scalar registers (the compiler would copy y to vector
// registers first, two moves a double).
__device__ __attribute__((always_inline)) inline void fma_scalar(double &h, double f, double y) {
    asm("v_fma_f64 %0, %1, %0, %2" : "+v"(h) : "v"(f), "s"(y));
}

// Channel sums of BG bins and the antenna.
template <int BG>
struct Sums {
    double a[3];
    double x[BG][4];
    __device__ inline void zero() {
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = 0.0;
#pragma unroll
        for (int b = 0; b < BG; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[b][c] = 0.0;
    }
    // this <- (fa, fx) this + y
    __device__ inline void shift(double fa, double fx, const Sums &y) {
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = fma(fa, a[c], y.a[c]);
#pragma unroll
        for (int b = 0; b < BG; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[b][c] = fma(fx, x[b][c], y.x[b][c]);
    }
    // the same for a slot that is uniform over the wave
    __device__ inline void shift_uniform(double fa, double fx, const Sums &y) {
#pragma unroll
        for (int c = 0; c < 3; ++c) fma_scalar(a[c], fa, y.a[c]);
#pragma unroll
        for (int b = 0; b < BG; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) fma_scalar(x[b][c], fx, y.x[b][c]);
    }
    // this <- this + (fa, fx) y
    __device__ inline void add(double fa, double fx, const Sums &y) {
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = fma(fa, y.a[c], a[c]);
#pragma unroll
        for (int b = 0; b < BG; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[b][c] = fma(fx, y.x[b][c], x[b][c]);
    }
};

// Slot k (the same in every lane; scalar loads).  Bins past the last repeat it.
template <int BG, typename PP>
__device__ __attribute__((always_inline)) inline Sums<BG> uniform_slot(PP &p, int k, int bin0) {
    Sums<BG> y;
    ConstParams<double> *ab = const_ptr(p.abc) + (size_t)k * 4;
#pragma unroll
    for (int c = 0; c < 3; ++c) y.a[c] = ab[c];
#pragma unroll
    for (int b = 0; b < BG; ++b) {
        ConstParams<double> *x = const_ptr(p.x64) + ((size_t)k * p.n_bins + min(bin0 + b, p.n_bins - 1)) * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) y.x[b][c] = x[c];
    }
    return y;
}

// The first slot from k (at most K) on that holds an SFT, K if none does.
template <typename PP>
__device__ __attribute__((always_inline)) inline int next_sft(PP &p, int k) {
    return const_ptr(reinterpret_cast<const int *>(p.abc))[(size_t)k * 8 + 6];
}

// H at slot k taken down to slot lo, front slots added.
template <int BG, int U, typename PP>
__device__ __attribute__((always_inline)) inline void run_down(PP &p, const LaneTau &t, int bin0, int k, int lo,
                                                               Sums<BG> &H) {
#pragma unroll 1
    for (; k > lo; k -= U) {
        Sums<BG> y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = uniform_slot<BG>(p, max(k - 1 - u, 0), bin0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k - 1 - u >= lo) H.shift_uniform(t.rho2, t.rho, y[u]);
    }
}

// ---------------------------------------------------------------------------
// Anchors.  Workgroup = one (tau tile, bin group or antenna) x kSlideWaves
// consecutive ranges (a super-range): every range's sum T = H over its own
// slots; then wave = range, by a Horner step over the later ranges of the
// workgroup the local H at its end (anc) and, for the whole super-range, the
// sum at its start (sup).
//
// T is a contraction, weights [64 taus x slots] times data [slots x 4 BG
// channels], the weights the same for every range: maps of two bins or more
// run it on the FP64 matrix cores (four 16-tau tiles; ranges side by side where
// a group has fewer than 16 channels), whose operands are one coalesced load
// and one product per four slots.  The antenna's three channels and one-bin
// maps, which would leave most of the chip idle, run it as a wave per range
// with scalar loads.  64 bins, 703 taus, 3001 slots: 97 us with every group on
// the VALU, 56 us now, of which the writes of H (45 MB) are about 10 us and the
// rest is waits of the chain over a range's slots.
// ---------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Range sums in LDS, [range][channel][64 taus] (channels: 4 BG, or the
// antenna's 3).
template <int BG>
constexpr int anchor_smem() {
    return kSlideWaves * 4 * BG * 64;   // doubles
}

// Range sums of the workgroup's ranges from slot k0 (its first) on.
template <int BG, typename PP>
__device__ __attribute__((always_inline)) inline void range_sums_mfma(PP &p, double *tot, int tt, int bin0, int k0,
                                                                    int kend) {
    constexpr int CH = 4 * BG;
    constexpr int kSide = 16 / CH;               // ranges side by side in the 16 columns
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave * kSide >= kSlideWaves) return;
    const int col = lane & 15, kg = lane >> 4;   // column (channel), slot within a step of four
    const int side = col / CH;
    const int ch = col - side * CH;
    const int RL = p.range_len;
    const int kb = k0 + (wave * kSide + min(side, kSide - 1)) * RL;
    const int ke = side < kSide && bin0 + (ch >> 2) < p.n_bins ? min(kb + RL, kend) : kb;   // (columns without data: none)
    double w[4], r4[4];                          // the weight of slot kg of the step, and rho^4
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double c = -(double)p.t_sft / (double)p.tau[min(tt * 64 + 16 * t + col, p.n_tau - 1)];
        w[t] = exp(c * (double)kg);
        r4[t] = exp(c * 4.0);
    }
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    const double *x = p.x64 + bin0 * 4 + (ke > kb ? ch : 0);
    const size_t row = (size_t)p.n_bins * 4;
    // four steps (range_len is a multiple of 16) at a time, the next four's
    // loads in flight
    constexpr int kStep = 4;
    auto load = [&](int i, double *y) {
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            const int k = kb + i + 4 * u + kg;
            y[u] = x[(size_t)(k < ke ? k : p.K) * row];   // row K is zero
        }
    };
    double y[kStep], nx[kStep];
    load(0, y);
#pragma unroll 1
    for (int i = 0; i < RL; i += 4 * kStep) {
        load(i + 4 * kStep, nx);
#pragma unroll
        for (int u = 0; u < kStep; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[t], y[u], acc[t], 0, 0, 0);
                w[t] *= r4[t];
            }
#pragma unroll
        for (int u = 0; u < kStep; ++u) y[u] = nx[u];
    }
    // register r of lane (col, kg): tau 16 t + 4 r + kg of the tile
    if (side < kSide) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[((wave * kSide + side) * CH + ch) * 64 + 16 * t + 4 * r + kg] = acc[t][r];
    }
}

// Anchors of CH channels whose decay per slot is e^c, from the range sums.
template <int CH>
__device__ __attribute__((always_inline)) inline void anchor_horner(const double *tot, double c, int RL, int n_first, bool any,
                                                                  double *anc, double *sup) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // ranges after this one, from the last: full ranges decay by f (a short
    // or empty one is last, where the sum so far is zero)
    const double f = exp(c * (double)RL);
    double E[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) E[q] = 0.0;
    for (int w = kSlideWaves - 1; w > wave; --w) {
#pragma unroll
        for (int q = 0; q < CH; ++q) E[q] = fma(f, E[q], tot[(w * CH + q) * 64 + lane]);
    }
    if (any) {
#pragma unroll
        for (int q = 0; q < CH; ++q) anc[((size_t)wave * CH + q) * 64 + lane] = E[q];
    }
    if (wave == 0) {
        const double l = exp(c * (double)n_first);
#pragma unroll
        for (int q = 0; q < CH; ++q) sup[(size_t)q * 64 + lane] = fma(l, E[q], tot[q * 64 + lane]);
    }
}

// The pass's column (tau tile, bin group) in the anchors' memory.
template <typename PP>
__device__ __attribute__((always_inline)) inline size_t pass_column(PP &p, int tt, int bg) {
    return (size_t)(tt - p.tt0) * p.pass_bg + (bg - p.bg0);
}

// bg == p.n_bg: the antenna's channels.
template <int BG, typename PP>
__device__ __attribute__((always_inline)) inline void slide_anchor(PP &p, double *tot, int tt, int bg, int sup) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kend = const_ptr(p.tiles)[tt].kend;
    const int RL = p.range_len;
    const int g0 = sup * kSlideWaves;
    const int k0 = p.kbeg + g0 * RL;
    if (k0 >= kend) return;   // the whole workgroup: no slots
    const int kb = k0 + wave * RL;
    const int ke = min(kb + RL, kend);
    const int n_first = min(RL, kend - k0);   // slots of the first range
    const double c = -(double)p.t_sft / (double)p.tau[min(tt * 64 + lane, p.n_tau - 1)];
    const bool ant = bg == p.n_bg;
    if (!ant && (BG > 1 || p.n_bins > 1)) {
        range_sums_mfma<BG>(p, tot, tt, bg * BG, k0, kend);
    } else {
        // one wave per range, a slot's channels by scalar loads
        const int nc = ant ? 3 : 4;
        const double rho = exp(ant ? 2.0 * c : c);
        ConstParams<double> *y = ant ? const_ptr(p.abc) : const_ptr(p.x64) + bg * 4;
        const size_t row = ant ? 4 : (size_t)p.n_bins * 4;
        double H[4] = {0.0, 0.0, 0.0, 0.0};
        constexpr int U = 8;
#pragma unroll 1
        for (int k = ke; k > kb; k -= U) {
            double v[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[u][q] = y[(size_t)max(k - 1 - u, 0) * row + q];   // (the antenna's fourth: no use)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k - 1 - u >= kb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) H[q] = fma(rho, H[q], v[u][q]);
        }
        for (int q = 0; q < nc; ++q) tot[(wave * nc + q) * 64 + lane] = H[q];
    }
    __syncthreads();
    if (ant) {
        const size_t at = tt - p.tt0;
        anchor_horner<3>(tot, 2.0 * c, RL, n_first, kb < ke, p.anc_a + (at * p.n_range + g0) * 3 * 64,
                         p.sup_a + (at * p.n_sup + sup) * 3 * 64);
    } else {
        const size_t col = pass_column(p, tt, bg);
        anchor_horner<4 * BG>(tot, c, RL, n_first, kb < ke, p.anc + (col * p.n_range + g0) * (4 * BG) * 64,
                              p.sup + (col * p.n_sup + sup) * (4 * BG) * 64);
    }
}

// The super-ranges' sums of one (tau tile, bin group or antenna) into H at
// their ends, in place: thread = (channel, tau), from the last down.
template <typename PP>
__device__ __attribute__((always_inline)) inline void slide_supers(PP &p, int tt, int bg) {
    const bool ant = bg == p.n_bg;
    const int CH = ant ? 3 : 4 * p.bg;
    const int len = kSlideWaves * p.range_len;
    const int n = (const_ptr(p.tiles)[tt].kend - p.kbeg + len - 1) / len;
    const int lane = threadIdx.x & 63;
    const double c = -(double)p.t_sft / (double)p.tau[min(tt * 64 + lane, p.n_tau - 1)] * (double)len;
    const double f = exp(ant ? 2.0 * c : c);
    for (int q = threadIdx.x >> 6; q < CH; q += 4) {
        double *s = ant ? p.sup_a + (size_t)(tt - p.tt0) * p.n_sup * 3 * 64 : p.sup + pass_column(p, tt, bg) * p.n_sup * CH * 64;
        s += q * 64 + lane;
        double H = 0.0;   // (a short super-range is the last: nothing comes after it)
#pragma unroll 8
        for (int u = n - 1; u >= 0; --u) {
            const double v = s[(size_t)u * CH * 64];
            s[(size_t)u * CH * 64] = H;
            H = fma(f, H, v);
        }
    }
}

// ---------------------------------------------------------------------------
// Rows.  Bound by VALU issue where segments are long: a row of a wave of four
// bins is about 220 instructions plus 30 a front and 50 a back slot, nearly all
// FP64 (counters at 256 bins x 500 x 500: VALU busy 77 %, 250 instructions a
// row).  Short segments wait for their starts and, with taus far apart, for the
// back slots' LDS reads (64 bins x 611 x 703: VALU busy 56 %, half of the LDS
// cycles in conflicts; one bin x 1000 x 1000 54 %; a mixed batch of 24 43 %).
// What it took to get there: G changed in place (branches around its update
// cost a move of all its registers a row), four waves per SIMD, the first front
// slot and the next row's plan loaded a row ahead, back slots from LDS.  Rows
// kernel at 64 bins x 611 x 703 on 3001 slots: 464 us with the back slots
// through the caches, 268 us staged, 196 us now; 256 bins x 500 x 500: 481, 340,
// 199 us.
// ---------------------------------------------------------------------------
// The segment's rows, from the last down, on one wave.  STAGED: the back slots
// are in LDS from slot w_lo on.
template <int BG, bool STAGED, typename PP>
__device__ __attribute__((always_inline)) inline void slide_segment(PP &p, double *lds, int tt, int col, int bin0, int seg,
                                                                  int w_lo) {   // col: of the pass
    const int lane = threadIdx.x & 63;
    const int n_bins = p.n_bins;
    const int K = p.K;
    const int RL = p.range_len;
    const int cap = p.stage;
    ConstParams<RowPlan> *rows = const_ptr(p.rows);
    const int kbeg = p.kbeg, kend = const_ptr(p.tiles)[tt].kend;
    const int n = tt * 64 + lane;
    const bool n_ok = n < p.n_tau;
    const double2 *const s_ab = reinterpret_cast<const double2 *>(lds);
    const float4 *const s_x = reinterpret_cast<const float4 *>(s_ab + cap + 1);
    const double *const s_c = reinterpret_cast<const double *>(s_x + BG * (cap + 1));
    const LaneTau t = lane_tau(p.tau[min(n, p.n_tau - 1)], p.t_sft);

    // the lane's back slot k, zero where !on (byte offsets fit 32 bits: the
    // plan's limit)
    auto lane_slot = [&](int k, bool on) {
        Sums<BG> y;
        float4 v[BG];
        if constexpr (STAGED) {
            const int i = on ? k - w_lo : cap;
            const double2 ab = s_ab[i];
            y.a[0] = ab.x;
            y.a[1] = ab.y;
            y.a[2] = s_c[i];
#pragma unroll
            for (int b = 0; b < BG; ++b) v[b] = s_x[b * (cap + 1) + i];
        } else {
            const unsigned kk = on ? k : K;   // row K is zero
            const char *ab = reinterpret_cast<const char *>(p.abc);
            const double2 u = *reinterpret_cast<const double2 *>(ab + kk * 32u);
            y.a[0] = u.x;
            y.a[1] = u.y;
            y.a[2] = *reinterpret_cast<const double *>(ab + 16 + kk * 32u);
            const unsigned e = (kk * (unsigned)n_bins + (unsigned)bin0) * 4u;
            if (!p.exact32) {
                const char *x = reinterpret_cast<const char *>(p.x64);
#pragma unroll
                for (int b = 0; b < BG; ++b) {
                    const char *xb = x + 32 * min(b, n_bins - 1 - bin0);
                    const double2 u0 = *reinterpret_cast<const double2 *>(xb + e * 8u);
                    const double2 u1 = *reinterpret_cast<const double2 *>(xb + 16 + e * 8u);
                    y.x[b][0] = u0.x;
                    y.x[b][1] = u0.y;
                    y.x[b][2] = u1.x;
                    y.x[b][3] = u1.y;
                }
                return y;
            }
            const char *x = reinterpret_cast<const char *>(p.x32);
#pragma unroll
            for (int b = 0; b < BG; ++b)
                v[b] = *reinterpret_cast<const float4 *>(x + 16 * min(b, n_bins - 1 - bin0) + e * 4u);
        }
#pragma unroll
        for (int b = 0; b < BG; ++b) {
            y.x[b][0] = v[b].x;
            y.x[b][1] = v[b].y;
            y.x[b][2] = v[b].z;
            y.x[b][3] = v[b].w;
        }
        return y;
    };
    // channel c of anchor g, or of H at the end of super-range g
    const double *anc = p.anc + (size_t)col * p.n_range * (4 * BG) * 64 + lane;
    const double *sup = p.sup + (size_t)col * p.n_sup * (4 * BG) * 64 + lane;
    const double *anc_a = p.anc_a + (size_t)(tt - p.tt0) * p.n_range * 3 * 64 + lane;
    const double *sup_a = p.sup_a + (size_t)(tt - p.tt0) * p.n_sup * 3 * 64 + lane;
    auto load_sums = [&](const double *x, const double *a, int g) {
        Sums<BG> y;
#pragma unroll
        for (int c = 0; c < 3; ++c) y.a[c] = a[((size_t)g * 3 + c) * 64];
#pragma unroll
        for (int c = 0; c < 4 * BG; ++c) y.x[c >> 2][c & 3] = x[((size_t)g * (4 * BG) + c) * 64];
        return y;
    };
    const int n_range = (kend - kbeg + RL - 1) / RL;
    constexpr int kU = BG == 1 ? 4 : BG == 2 ? 2 : 1;   // slots in flight
    // H at the first range end at or after slot k (kbeg <= k < kend; lanes with
    // !on: anything finite), and that end
    auto range_end = [&](int k, bool on, Sums<BG> &H) {
        const int g = on ? max((k - kbeg + RL - 1) / RL - 1, 0) : n_range - 1;
        const int u = g / kSlideWaves;
        H = load_sums(anc, anc_a, g);
        const int ge = min(kbeg + (g + 1) * RL, kend);
        const int ue = kbeg + (u + 1) * kSlideWaves * RL;
        if (__any(ue < kend)) {   // super-ranges follow
            const double f = ue < kend ? exp(t.c * (double)(ue - ge)) : 0.0;
            H.add(f * f, f, load_sums(sup, sup_a, u));
        }
        return ge;
    };

    const int m_lo = seg * p.seg_rows;
    int m = min(m_lo + p.seg_rows, p.n_t0) - 1;
    int k0 = rows[m].k0, delta = rows[m].delta;
    int lo = clamp_slot(k0, K);
    int hi = max(end_slot(k0, delta, t.q, t.r, K), lo);
    Sums<BG> G;
    G.zero();
    if (__any(hi > lo)) {
        Sums<BG> H;
        // G = H(lo) - rho^(hi - lo) H(hi)
        const bool back = hi > lo && hi < kend;
        if (__any(back)) {
            int k = range_end(hi, back, H);
#pragma unroll 1
            for (; __any(back && k > hi); --k) {
                const bool on = back && k > hi;
                const Sums<BG> y = lane_slot(k - 1, on);
                H.shift(on ? t.rho2 : 1.0, on ? t.rho : 1.0, y);
            }
            const double w = back ? -exp(t.c * (double)(hi - lo)) : 0.0;
            const double w2 = -w * w;
            G.add(w2, w, H);
        }
        int k = range_end(lo, true, H);
        k = __builtin_amdgcn_readfirstlane(k);
        run_down<BG, kU>(p, t, bin0, k, lo, H);
        const double in = hi > lo ? 1.0 : 0.0;
        G.add(in, in, H);
    }
    // rho^q and rho^(q + 1): weights of the first slot past a window
    const double wq = exp(t.c * (double)t.q), wq1 = wq * t.rho;
    const double ga = p.guard_a, gb = p.guard_b;
    const size_t bin_cells = (size_t)p.n_t0 * p.n_tau;
    float *out = p.twoF ? p.twoF + (size_t)bin0 * bin_cells + (size_t)m * p.n_tau + tt * 64 : nullptr;   // row m, bin bin0
    const int nb = min(BG, n_bins - bin0);
    const bool write = out && n_ok;

    double fm[BG], fs[BG];
    int im[BG];
#pragma unroll
    for (int b = 0; b < BG; ++b) {
        fm[b] = -INFINITY;
        fs[b] = 0.0;
        im[b] = 0;
    }
    // The loop below changes G in place, without branches around a change:
    // where paths with a changed and an unchanged G meet, the compiler moves
    // all its registers.
#pragma unroll 1
    for (;;) {
        // the next row and its first front slot (row K of the atoms, zeros, if
        // none enters), on their way while this row is finished
        const int mn = max(m - 1, m_lo);
        const int k0_n = rows[mn].k0, delta_n = rows[mn].delta;
        const int lo_n = clamp_slot(k0_n, K);
        int k = lo_n < lo ? lo - 1 : K;
        Sums<BG> y = uniform_slot<BG>(p, k, bin0);
        const bool direct = hi > lo && (G.a[0] < ga || G.a[1] < gb);
        if (__any(direct)) {
            // too weak beside what has left the window: the plain sums, from
            // SFT to SFT (most such windows hold none, or a few at their end
            // after a gap: stepping through the gaps slot by slot took 2.8 of
            // 3.2 ms of 64 bins x 600 x 700 with one gap of 500 slots)
            const int j0 = next_sft(p, lo);
            const bool some = __any(direct && j0 < hi);
            const double w0 = some ? exp(t.c * (double)(j0 - lo)) : 0.0;
#pragma unroll
            for (int b = 0; b < BG; ++b) {
                Sums<1> S;
                S.zero();
                if (some) {
                    double w = w0;
                    int j = j0;
#pragma unroll 1
                    do {
                        const double ww = j < hi ? w : 0.0;
                        S.add(ww * ww, ww, uniform_slot<1>(p, j, bin0 + b));
                        const int jn = next_sft(p, j + 1);
#pragma unroll 1
                        for (; j < jn; ++j) w *= t.rho;
                    } while (__any(direct && j < hi));
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) G.x[b][c] = direct ? S.x[0][c] : G.x[b][c];
                if (b == BG - 1) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) G.a[c] = direct ? S.a[c] : G.a[c];
                }
            }
        }
        // the cell (m, n): 1 / D by two Newton steps (the plan keeps D's range
        // normal), then each bin's F = 2F / 2
        const double A = G.a[0], B = G.a[1], C = G.a[2];
        const double AB = A * B;
        const double D = fma(-C, C, AB);
        double r = __builtin_amdgcn_rcp(D);
        r = fma(r, fma(-D, r, 1.0), r);
        r = fma(r, fma(-D, r, 1.0), r);
        r = hi > lo && D > kDegenerateRtol * AB ? r : 0.0;
        const double qa = r * A, qb = r * B, qc = -2.0 * r * C;
        float F2[BG];
#pragma unroll
        for (int b = 0; b < BG; ++b) {
            const double *f = G.x[b];
            const double F = fma(qb, fma(f[0], f[0], f[1] * f[1]),
                                 fma(qa, fma(f[2], f[2], f[3] * f[3]), qc * fma(f[0], f[2], f[1] * f[3])));
            F2[b] = 2.f * (float)F;
            // running maximum (the earlier row on a tie) and sum of
            // exp(F - max), one FP32 exponential
            const double d = F - fm[b];
            const bool up = d >= 0.0;
            const float e = __expf(-fabsf((float)d));
            fs[b] = fma(fs[b], (double)(up ? e : 1.f), (double)(up ? 1.f : e));
            fm[b] = up ? F : fm[b];
            im[b] = up ? m : im[b];
        }
        if (write) {
#pragma unroll
            for (int b = 0; b < BG; ++b)
                if (b < nb) out[b * bin_cells + lane] = F2[b];
        }
        if (m == m_lo) break;
        --m;
        if (out) out -= p.n_tau;
        k0 = k0_n;
        delta = delta_n;
        // slots that enter at the front
        const double u = lo_n < lo ? t.rho : 1.0, u2 = lo_n < lo ? t.rho2 : 1.0;
        lo = lo_n;
#pragma unroll 1
        for (;;) {
            G.shift_uniform(u2, u, y);
            if (--k < lo || k >= K - 1) break;
            y = uniform_slot<BG>(p, k, bin0);
        }
        // slots that leave at the back: weight rho^(k - lo)
        const int hi_n = max(end_slot(k0, delta, t.q, t.r, K), lo);
        double w = hi_n - lo == t.q ? wq : wq1;
        // (rows that start before the data: a shorter window)
        if (k0 < 0) w = exp(t.c * (double)(hi_n - lo));
        w = -w;
        int j = hi_n;
#pragma unroll 1
        do {
            const Sums<BG> v = lane_slot(j, j < hi);
            G.add(-w * w, w, v);
            w *= t.rho;
            ++j;
        } while (__any(j < hi));
        hi = hi_n;
    }

#pragma unroll
    for (int b = 0; b < BG; ++b) {
        const Partial w = wave_state(fm[b], fs[b], im[b], n, n_ok, p.n_tau);
        if (lane == 0 && b < nb) p.part[(size_t)(bin0 + b) * p.n_tiles + (size_t)tt * p.n_seg + seg] = w;
    }
}

// Workgroup = up to kRowsWaves segments of one column.  The back slots that
// its segments drop, and those between their last ends and the next range
// boundary, are staged in LDS once (sized by the plan): [a^2, b^2], ab, then
// each bin's data; the last entry is zero (lanes without a slot to drop read
// it).  Maps whose tiles' taus span more slots than fit (or whose data are not
// single-precision numbers) read them through the caches, a line per lane and
// slot.
template <int BG, bool STAGED, typename PP>
__device__ __attribute__((always_inline)) inline void slide_rows(PP &p, double *lds, int col, int group) {
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int at = col / p.pass_bg;
    const int tt = p.tt0 + at;
    const int bin0 = (p.bg0 + col - at * p.pass_bg) * BG;
    const int n_bins = p.n_bins;
    const int K = p.K;
    const int RL = p.range_len;
    const int W = p.waves;
    const int cap = p.stage;
    ConstParams<RowPlan> *rows = const_ptr(p.rows);
    auto &tile = const_ptr(p.tiles)[tt];
    const int kbeg = p.kbeg, kend = tile.kend;
    double2 *const s_ab = reinterpret_cast<double2 *>(lds);
    float4 *const s_x = reinterpret_cast<float4 *>(s_ab + cap + 1);
    double *const s_c = reinterpret_cast<double *>(s_x + BG * (cap + 1));

    const int s0 = group * W;
    int w_lo = 0;
    if constexpr (STAGED) {
        const int m_a = s0 * p.seg_rows, m_b = min((s0 + W) * p.seg_rows, p.n_t0) - 1;
        w_lo = end_slot(rows[m_a].k0, rows[m_a].delta, tile.q0, tile.r0, K);
        int w_hi = max(end_slot(rows[m_b].k0, rows[m_b].delta, tile.q1, tile.r1, K), kbeg);
        w_hi = min(kbeg + (w_hi - kbeg + RL - 1) / RL * RL, kend);
        const int n_w = min(w_hi - w_lo, cap);   // (the plan's stage holds them all)
        for (int i = tid; i < n_w; i += 64 * W) {
            const double *ab = p.abc + (size_t)(w_lo + i) * 4;
            s_ab[i] = *reinterpret_cast<const double2 *>(ab);
            s_c[i] = ab[2];
#pragma unroll
            for (int b = 0; b < BG; ++b)
                s_x[b * (cap + 1) + i] = *reinterpret_cast<const float4 *>(
                    p.x32 + ((size_t)(w_lo + i) * n_bins + min(bin0 + b, n_bins - 1)) * 4);
        }
        if (tid == 0) {
            s_ab[cap] = double2{0.0, 0.0};
            s_c[cap] = 0.0;
#pragma unroll
            for (int b = 0; b < BG; ++b) s_x[b * (cap + 1) + cap] = float4{0.f, 0.f, 0.f, 0.f};
        }
        __syncthreads();
    }
    const int seg = s0 + wave;
    if (seg < p.n_seg) slide_segment<BG, STAGED>(p, lds, tt, col, bin0, seg, w_lo);
}

// ---------------------------------------------------------------------------
// Once per upload: the FP32 plane, and the ranges of the atoms' values.
// Workgroup = up to kAtomBins bins (the last group: the antenna) x a chunk of
// 64-slot stretches.  Eight lanes share a (stretch, bin), every eighth slot
// each, so that a stretch is one round of loads in flight (bound by that
// latency, and by the copies around it) and lanes next to each other read slots
// or bins next to each other.  The findings go straight to pinned host memory,
// a record per workgroup, which the host combines: a copy back costs more than
// the kernel (an upload of one bin x 200 slots: 52 us with one workgroup per 16
// columns and a copy, 26 us now, 24 us without the ranges; 16 bins x 8000 slots:
// the kernel 47 and 13 us).
// ---------------------------------------------------------------------------
// v over the n (a power of two) lanes that lie `stride` apart around this one,
// `at` its place among them.
template <typename T, typename Op>
__device__ __attribute__((always_inline)) inline T ring(T v, int lane, int stride, int at, int n, Op op) {
    const int first = lane - at * stride;
    for (int o = n / 2; o > 0; o >>= 1) v = op(v, __shfl(v, first + ((at + o) & (n - 1)) * stride, 64));
    return v;
}

__global__ __launch_bounds__(64 * kAtomWaves) void atoms_kernel(const double *x64, const double *abc, float *x32,
                                                               int32_t K, int32_t n_bins, RangeInfo *out) {
    constexpr int kSlots = 64 / kAtomLanes;              // slots of a lane
    __shared__ double smax[kAtomWaves][4][kAtomBins], smin[kAtomWaves][4][kAtomBins];
    __shared__ double sslot[kAtomWaves][kAtomBins], sjoint[kAtomWaves][kAtomBins];
    __shared__ int sflags;
    auto larger = [](double x, double y) { return fmax(x, y); };
    auto smaller = [](double x, double y) { return fmin(x, y); };
    auto sum = [](int x, int y) { return x + y; };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool ant = blockIdx.x == gridDim.x - 1;
    const int b0 = ant ? 0 : blockIdx.x * kAtomBins;
    const int row = ant ? 1 : n_bins;                    // groups of four values per slot
    const int W = min(row - b0, kAtomBins);              // bins of this workgroup
    const int subs = W == 1 ? 8 : W == 2 ? 4 : W <= 4 ? 2 : 1;   // stretches of a wave
    const int t = lane / W;
    const int b = lane - t * W, s8 = t % kAtomLanes, sub = t / kAtomLanes;
    const double *in = (ant ? abc : x64) + 4 * b0;
    if (threadIdx.x == 0) sflags = 0;
    __syncthreads();
    double mx[4], mn[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        mx[c] = 0.0;
        mn[c] = INFINITY;
    }
    double slot = INFINITY, joint = INFINITY;   // of all four columns together
    bool bad = false, inexact = false;
    for (int k0 = (blockIdx.y * kAtomWaves + wave) * subs * 64; k0 < K; k0 += gridDim.y * kAtomWaves * subs * 64) {
        const int kb = k0 + sub * 64 + s8;
        double v[kSlots][4];
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int k = kb + i * kAtomLanes;
            const bool on = sub < subs && k < K;
            const double *x = in + ((size_t)(on ? k : 0) * row + b) * 4;
            const double2 u0 = *reinterpret_cast<const double2 *>(x);
            const double2 u1 = *reinterpret_cast<const double2 *>(x + 2);
            v[i][0] = on ? u0.x : 0.0;
            v[i][1] = on ? u0.y : 0.0;
            v[i][2] = on ? u1.x : 0.0;
            v[i][3] = on ? u1.y : 0.0;
        }
        double m[4] = {0.0, 0.0, 0.0, 0.0};
        int n_sft = 0;   // slots with data
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int k = kb + i * kAtomLanes;
            float4 f;
            f.x = (float)v[i][0];
            f.y = (float)v[i][1];
            f.z = (float)v[i][2];
            f.w = (float)v[i][3];
            if (!ant && sub < subs && k < K)
                *reinterpret_cast<float4 *>(x32 + ((size_t)k * n_bins + b0 + b) * 4) = f;
            inexact |= f.x != v[i][0] || f.y != v[i][1] || f.z != v[i][2] || f.w != v[i][3];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bad |= !(fabs(v[i][c]) < INFINITY);
                m[c] = fmax(m[c], fabs(v[i][c]));
            }
            const double all = fmax(fmax(fabs(v[i][0]), fabs(v[i][1])), fmax(fabs(v[i][2]), fabs(v[i][3])));
            if (all > 0.0) slot = fmin(slot, all);
            n_sft += all > 0.0;
        }
        // (a stretch of a few SFTs has no level of its own: of one SFT's values
        // three in a million lie 2^-20 below their column's largest by chance,
        // which is one a map where 256 bins have hundreds of such stretches)
        const bool counts = ring(n_sft, lane, W, s8, kAtomLanes, sum) >= kAtomSfts;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            m[c] = ring(m[c], lane, W, s8, kAtomLanes, larger);   // the stretch's
            mx[c] = fmax(mx[c], m[c]);
            if (counts && m[c] > 0.0) mn[c] = fmin(mn[c], m[c]);
        }
        const double all = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
        if (counts && all > 0.0) joint = fmin(joint, all);
    }
    if (!ant && blockIdx.y == 0 && threadIdx.x < W) {   // row K is zero
        const float4 z = {0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<float4 *>(x32 + ((size_t)K * n_bins + b0 + threadIdx.x) * 4) = z;
    }
    const int flags = (__any(bad) ? 1 : 0) | (__any(inexact) ? 2 : 0);
    if (lane == 0 && flags) atomicOr(&sflags, flags);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        mx[c] = ring(mx[c], lane, kAtomLanes * W, sub, subs, larger);
        mn[c] = ring(mn[c], lane, kAtomLanes * W, sub, subs, smaller);
        if (lane < W) {
            smax[wave][c][lane] = mx[c];
            smin[wave][c][lane] = mn[c];
        }
    }
    slot = ring(slot, lane, W, s8, kAtomLanes, smaller);
    slot = ring(slot, lane, kAtomLanes * W, sub, subs, smaller);
    joint = ring(joint, lane, kAtomLanes * W, sub, subs, smaller);
    if (lane < W) {
        sslot[wave][lane] = slot;
        sjoint[wave][lane] = joint;
    }
    __syncthreads();
    // the waves': sixteen lanes a (bin, column)
    RangeInfo &r = out[blockIdx.y * gridDim.x + blockIdx.x];
    if (threadIdx.x == 0) r.flags = sflags;
    const int e = threadIdx.x / kAtomWaves, w = threadIdx.x % kAtomWaves;
    const int eb = e >> 2, ec = e & 3;
    if (eb < W) {   // (whole groups of sixteen lanes)
        double x = smax[w][ec][eb], n = smin[w][ec][eb];
        double y = ec ? sjoint[w][eb] : sslot[w][eb];   // (columns 2 and 3: the same again)
#pragma unroll
        for (int o = 1; o < kAtomWaves; o <<= 1) {
            x = fmax(x, __shfl_xor(x, o, kAtomWaves));
            n = fmin(n, __shfl_xor(n, o, kAtomWaves));
            y = fmin(y, __shfl_xor(y, o, kAtomWaves));
        }
        if (w == 0) {
            r.most[eb][ec] = x;
            r.least[eb][ec] = n;
            if (ec == 0) r.slot[eb] = y;
            if (ec == 1) r.joint[eb] = y;
        }
    }
}

template <int BG>
__global__ __launch_bounds__(64 * kSlideWaves) void slide_anchor_kernel(SlideParams p) {
    __shared__ double tot[anchor_smem<BG>()];
    const int at = blockIdx.x / (p.pass_bg + 1);
    const int i = blockIdx.x - at * (p.pass_bg + 1);   // (the last: the antenna)
    slide_anchor<BG>(p, tot, p.tt0 + at, i == p.pass_bg ? p.n_bg : p.bg0 + i, blockIdx.y);
}

template <int BG, bool STAGED>
__global__ __launch_bounds__(64 * kRowsWaves) void slide_rows_kernel(SlideParams p) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    slide_rows<BG, STAGED>(p, lds, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void slide_supers_kernel(SlideParams p) {
    const int at = blockIdx.x / (p.pass_bg + 1);
    const int i = blockIdx.x - at * (p.pass_bg + 1);
    slide_supers(p, p.tt0 + at, i == p.pass_bg ? p.n_bg : p.bg0 + i);
}

// Many maps, one workgroup per entry; the bins per group are the map's.
template <typename T>
__device__ inline ConstParams<T> &const_params(const T *p) {
    return *const_ptr(p);
}
__global__ __launch_bounds__(64 * kSlideWaves) void slide_anchor_batch_kernel(SlideBatchParams b) {
    __shared__ double tot[anchor_smem<4>()];
    ConstParams<int32_t> *e = const_ptr(b.anchors) + 4 * (size_t)blockIdx.x;
    auto &p = const_params(b.jobs + e[0]);
    switch (p.bg) {
    case 1: slide_anchor<1>(p, tot, e[1], e[2], e[3]); break;
    case 2: slide_anchor<2>(p, tot, e[1], e[2], e[3]); break;
    case 3: slide_anchor<3>(p, tot, e[1], e[2], e[3]); break;
    default: slide_anchor<4>(p, tot, e[1], e[2], e[3]); break;
    }
}
// (an anchor entry's first super-range stands for its column)
__global__ __launch_bounds__(256) void slide_supers_batch_kernel(SlideBatchParams b) {
    ConstParams<int32_t> *e = const_ptr(b.anchors) + 4 * (size_t)blockIdx.x;
    if (e[3] == 0) slide_supers(const_params(b.jobs + e[0]), e[1], e[2]);
}
__global__ __launch_bounds__(64 * kRowsWaves) void slide_rows_batch_kernel(SlideBatchParams b) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    ConstParams<int32_t> *e = const_ptr(b.rows) + 4 * (size_t)blockIdx.x;
    auto &p = const_params(b.jobs + e[0]);
    if ((int)threadIdx.x >= 64 * p.waves) return;
    if (p.stage > 0) {
        switch (p.bg) {
        case 1: slide_rows<1, true>(p, lds, e[1], e[2]); break;
        case 2: slide_rows<2, true>(p, lds, e[1], e[2]); break;
        case 3: slide_rows<3, true>(p, lds, e[1], e[2]); break;
        default: slide_rows<4, true>(p, lds, e[1], e[2]); break;
        }
    } else {
        switch (p.bg) {
        case 1: slide_rows<1, false>(p, lds, e[1], e[2]); break;
        default: slide_rows<2, false>(p, lds, e[1], e[2]); break;   // (the plan's limit)
        }
    }
}

}  // namespace

hipError_t launch_slide_batch(const SlideBatchParams &p, hipStream_t s) {
    SlideBatchParams q = p;
    for (int32_t i = 0; i < p.n_anchors; i += kLaunchMost) {
        q.anchors = p.anchors + 4 * (size_t)i;
        q.n_anchors = std::min(p.n_anchors - i, kLaunchMost);
        hipLaunchKernelGGL(slide_anchor_batch_kernel, dim3((unsigned)q.n_anchors), dim3(64 * kSlideWaves), 0, s, q);
    }
    for (int32_t i = 0; i < p.n_anchors; i += kLaunchMost) {
        q.anchors = p.anchors + 4 * (size_t)i;
        q.n_anchors = std::min(p.n_anchors - i, kLaunchMost);
        hipLaunchKernelGGL(slide_supers_batch_kernel, dim3((unsigned)q.n_anchors), dim3(256), 0, s, q);
    }
    for (int32_t i = 0; i < p.n_rows; i += kLaunchMost) {
        q.rows = p.rows + 4 * (size_t)i;
        q.n_rows = std::min(p.n_rows - i, kLaunchMost);
        hipLaunchKernelGGL(slide_rows_batch_kernel, dim3((unsigned)q.n_rows), dim3(64 * kRowsWaves), q.lds_bytes, s, q);
    }
    return hipGetLastError();
}

hipError_t launch_atoms(const double *x64, const double *abc, float *x32, int32_t K, int32_t n_bins, RangeInfo *out,
                        hipStream_t s) {
    static_assert(4 * kAtomBins * kAtomWaves <= 64 * kAtomWaves, "a lane for every (bin, column, wave)");
    hipLaunchKernelGGL(atoms_kernel, dim3((unsigned)atom_groups(n_bins), (unsigned)atom_chunks(K, n_bins)),
                       dim3(64 * kAtomWaves), 0, s, x64, abc, x32, K, n_bins, out);
    return hipGetLastError();
}

hipError_t launch_slide_anchors(const SlideParams &p, hipStream_t s) {
    if (p.n_tau <= 0 || p.n_t0 <= 0 || p.seg_rows < 1 || p.range_len < 16 || p.range_len % 16) return hipErrorInvalidValue;
    const dim3 g((unsigned)(p.pass_tt * (p.pass_bg + 1)), (unsigned)p.n_sup), b(64 * kSlideWaves);
    if (g.y > 65535u) return hipErrorInvalidValue;
    switch (p.bg) {
    case 1: hipLaunchKernelGGL(slide_anchor_kernel<1>, g, b, 0, s, p); break;
    case 2: hipLaunchKernelGGL(slide_anchor_kernel<2>, g, b, 0, s, p); break;
    case 3: hipLaunchKernelGGL(slide_anchor_kernel<3>, g, b, 0, s, p); break;
    case 4: hipLaunchKernelGGL(slide_anchor_kernel<4>, g, b, 0, s, p); break;
    default: return hipErrorInvalidValue;
    }
    if (p.n_sup > 1) hipLaunchKernelGGL(slide_supers_kernel, dim3(g.x), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_slide_rows(const SlideParams &p, hipStream_t s) {
    const unsigned lds = slide_stage_bytes(p.bg, p.stage);
    if (p.waves < 1 || p.waves > kRowsWaves || p.stage < 0 || lds > kSlideStageBytes) return hipErrorInvalidValue;
    const dim3 g((unsigned)(p.pass_tt * p.pass_bg), (unsigned)((p.n_seg + p.waves - 1) / p.waves)), b(64u * p.waves);
    if (g.y > 65535u) return hipErrorInvalidValue;
    switch (2 * p.bg + (p.stage > 0)) {
    case 2: hipLaunchKernelGGL((slide_rows_kernel<1, false>), g, b, 0, s, p); break;
    case 3: hipLaunchKernelGGL((slide_rows_kernel<1, true>), g, b, lds, s, p); break;
    case 4: hipLaunchKernelGGL((slide_rows_kernel<2, false>), g, b, 0, s, p); break;
    case 5: hipLaunchKernelGGL((slide_rows_kernel<2, true>), g, b, lds, s, p); break;
    case 7: hipLaunchKernelGGL((slide_rows_kernel<3, true>), g, b, lds, s, p); break;
    case 9: hipLaunchKernelGGL((slide_rows_kernel<4, true>), g, b, lds, s, p); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tfs
