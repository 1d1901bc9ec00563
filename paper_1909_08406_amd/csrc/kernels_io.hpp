// Kernels of the RD3Q41 library besides the step: equilibrium
// initialisation, moments, FP64 conservation totals and Fourier
// projections, population I/O and the debug pull map. Included by the host
// side of the library only (lbm.hip).
#pragma once

#include "kernels.hpp"

namespace lbm {

// Device-held step counter read by graph replays (one vector store).
__global__ void k_set_counter(uint32_t* __restrict__ ctr, uint32_t v)
{
    if (threadIdx.x == 0) ctr[0] = v;
}

// ---------------------------------------------------------------------------
// Initialisation at equilibrium from FP64 fields (one chunk of nodes).
// ---------------------------------------------------------------------------
constexpr int INIT_NEWTON = 6;

// Whether the step of this squared length was the last one needed: the error
// left is quadratic in it, after one below 1e-9 a few 1e-18, where a context
// of 32- or 16-bit storage keeps 6e-8. FP64 storage takes every step.
template <bool F64>
__host__ __device__ inline bool newton_done(double step2)
{
    return !F64 && !(step2 > 1e-18);
}

// Node state of (rho, u, theta) relative to the reference state w_q rho_ref.
__host__ __device__ inline NodeDev<double> node_dev_f64(double rho, double ux, double uy, double uz, double theta,
                                                        double rho_ref)
{
    NodeDev<double> st;
    st.rho_ref = rho_ref;
    st.rho = rho;
    st.irho = d_rcp<double>(rho);
    st.drho = rho - rho_ref * SUM_W;
    st.j[0] = rho * ux;
    st.j[1] = rho * uy;
    st.j[2] = rho * uz;
    st.de2 = rho * (ux * ux + uy * uy + uz * uz + 3.0 * theta) - rho_ref * SUM_WC2;
    return st;
}

// Multipliers of the equilibrium of (rho, u, theta): MODEL_E2, or MODEL_ISO
// (theta unused).
template <bool F64>
__host__ __device__ inline Mult<double> solve_f64(const NodeDev<double>& st, double ux, double uy, double uz,
                                                  double theta, int model)
{
    Mult<double> m;
    if (model == MODEL_ISO) {
        m.b[0] = ux / THETA0;
        m.b[1] = uy / THETA0;
        m.b[2] = uz / THETA0;
        m.g = 0.0;
#pragma clang loop unroll(disable)
        for (int it = 0; it < INIT_NEWTON; ++it)
            if (newton_done<F64>(newton_step<double, false>(m, st))) break;
    } else {
        m.b[0] = d_div<double>(ux, theta);
        m.b[1] = d_div<double>(uy, theta);
        m.b[2] = d_div<double>(uz, theta);
        m.g = d_div<double>(0.5, theta) - 0.5 / THETA0;
#pragma clang loop unroll(disable)
        for (int it = 0; it < INIT_NEWTON; ++it)
            if (newton_done<F64>(newton_step<double>(m, st))) break;
    }
    return m;
}

// D_q of solved multipliers, to each(q, D_q).
template <class F>
__host__ __device__ __forceinline__ void gibbs_each_f64(const Mult<double>& m, const Shells<double>& S, double kap,
                                                        F&& each)
{
    static_for<Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        each(qc, dmul(gibbs_dev<q, double>(S), kap));
    });
}

// Deviations D_q (f_eq,q = w_q rho_ref (1 + D_q)) of the equilibrium of
// (rho, u, theta) in FP64, relative to the reference state w_q rho_ref, to
// each(q, D_q). model: MODEL_E2, MODEL_ISO (theta unused) or MODEL_SERIES.
// solved (E2 and ISO only) receives the multipliers b, g and kappa, from
// which gibbs_each_f64 forms the same D_q again.
template <bool F64, class F>
__host__ __device__ __forceinline__ void equilibrium_each_f64(double rho, double ux, double uy, double uz,
                                                              double theta, double rho_ref, int model,
                                                              double solved[5], F&& each)
{
    const NodeDev<double> st = node_dev_f64(rho, ux, uy, uz, theta, rho_ref);
    model &= MODEL_BASE_MASK;  // the path length plays no part in the equilibrium
    if (model == MODEL_SERIES) {
        SeriesCoef<double> sc;
        series_coef<double>(ux, uy, uz, theta / THETA0 - 1.0, sc);
        const double kap = st.drho / (rho_ref * SUM_W);
        static_for<Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            each(qc, dmul(series_eps<q, double>(sc), kap));
        });
        return;
    }
    const Mult<double> m = solve_f64<F64>(st, ux, uy, uz, theta, model);
    Shells<double> S;
    shells_at<double>(m, S);
    const double kap = kappa_of<double>(st, S);
    solved[0] = m.b[0];
    solved[1] = m.b[1];
    solved[2] = m.b[2];
    solved[3] = m.g;
    solved[4] = kap;
    gibbs_each_f64(m, S, kap, each);
}

__host__ inline void equilibrium_dev_f64(double rho, double ux, double uy, double uz, double theta, double rho_ref,
                                         int model, double D[Q])
{
    double solved[5];
    equilibrium_each_f64<true>(rho, ux, uy, uz, theta, rho_ref, model, solved,
                               [&](auto qc, double d) { D[decltype(qc)::value] = d; });
}

// v rounded to FP32 with the last bit set when inexact (round to odd): a
// following round to nearest of the 16-bit forms then gives what one rounding
// of v gives, without the 28-instruction conversion from FP64 to 16 bits.
// Decided on magnitudes: t has v's sign also where it is 0 (|v| below half
// the smallest FP32 subnormal), so one more in its bits is one unit away from
// 0 there too. Zeros, infinities and NaN stay as they are; past the FP32 range
// t is the largest finite value, which rounds to infinity in 16 bits.
__host__ __device__ inline float to_f32_odd(double v)
{
    const float t = float(v);
    const uint32_t u = __builtin_bit_cast(uint32_t, t);
    const double m = fabs(double(t)), a = fabs(v);
    const uint32_t other = m < a ? u + 1u : m > a ? u - 1u : u;
    return __builtin_bit_cast(float, (u & 1u) == 0u ? other : u);
}

__device__ inline void block_max_float(float v, float* out)
{
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    __shared__ float sm[BLOCK / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) sm[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = sm[0];
        for (int i = 1; i < BLOCK / 64; ++i) r = fmaxf(r, sm[i]);
        // non-negative floats order like their bit patterns
        atomicMax(reinterpret_cast<unsigned int*>(out), __float_as_uint(r));
    }
}

// Nodal FP64 fields of one chunk of nodes (host data staged on the device,
// or device arrays of the caller), element i for node n0 + i.
struct InitFields {
    const double* rho;
    const double* ux;
    const double* uy;
    const double* uz;
    const double* th;
};

// What a launch of k_init does.
constexpr int INIT_STORE = 0;    // solve and store the encoded populations
constexpr int INIT_MEASURE = 1;  // solve and measure max_q |f_q - w_q rho0| 2^{k_shell} (for the shifted storage
                                 // exponent); keep the solution in `solved` when that is not null
constexpr int INIT_RESTORE = 2;  // store the populations from the kept solution (no fields read)

// The shifted 16-bit forms need the largest deviation of all nodes before the
// first value can be encoded. The measuring launch keeps its solution, five
// doubles per node, in the other population buffer (82 bytes per node, unused
// until the first step), and the storing launch forms the populations from it
// again without the fields or a second solve. Bound by FP64 arithmetic (the
// measuring launch: about 700 instructions per Newton step, two wavefronts per
// SIMD). 160^3 FP16 from device fields: 1.4 + 1.4 -> 0.47 + 0.27 ms, the whole
// call 3.56 -> 0.74 ms (with the Newton exit, to_f32_odd and the tile lists
// written on the device).
template <class ST, int MODE>
__global__ __launch_bounds__(BLOCK) void k_init(typename ST::T* __restrict__ f, uint32_t qs, uint32_t n0,
                                                uint32_t count, InitFields fields, StepParams p,
                                                double* __restrict__ solved, float* maxdev)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    float dev = 0.f;
    if (i < count) {
        const size_t N = p.g.N, n = size_t(n0) + i;
        // storage reference: rho0 for the shifted forms, the weights themselves otherwise
        const double rref = ST::shifted ? p.rho_ref : 1.0;
        bool bad = false;
        // range of D_q per shell, and a sum that is NaN once a D_q is not finite
        double lo[6], hi[6], sum0 = 0.0;
        for (int sh = 0; sh < 6; ++sh) lo[sh] = hi[sh] = 0.0;
        auto each = [&](auto qc, double D) {
            constexpr int q = decltype(qc)::value;
            constexpr int sh = VEL[q].shell;
            if constexpr (MODE != INIT_RESTORE) {
                lo[sh] = fmin(lo[sh], D);
                hi[sh] = fmax(hi[sh], D);
                sum0 = fma(D, 0.0, sum0);
            }
            if constexpr (MODE != INIT_MEASURE) {
                const double d = SHELL_W[sh] * rref * D;  // f_eq,q - w_q rref
                double v;
                if constexpr (ST::shifted) v = d * double(p.scale[sh]);
                else v = SHELL_W[sh] + d;
                if constexpr (sizeof(typename ST::T) == 2) ST::store(f + size_t(q) * qs + n, to_f32_odd(v));
                else ST::store(f + size_t(q) * qs + n, typename ST::R(v));
            }
        };
        if constexpr (MODE == INIT_RESTORE) {
            Mult<double> m;
            m.b[0] = solved[n];
            m.b[1] = solved[N + n];
            m.b[2] = solved[2 * N + n];
            m.g = solved[3 * N + n];
            const double kap = solved[4 * N + n];
            Shells<double> S;
            shells_at<double>(m, S);
            gibbs_each_f64(m, S, kap, each);
        } else {
            const double rho = fields.rho[i], ux = fields.ux[i], uy = fields.uy[i], uz = fields.uz[i],
                         th = fields.th[i];
            // the domain: rho > 0, theta > 0 (checked but unused by the
            // isothermal model), all finite
            bad = !(rho > 0.0 && th > 0.0 && fabs(rho) < 1e300 && fabs(th) < 1e300 && fabs(ux) < 1e300 &&
                    fabs(uy) < 1e300 && fabs(uz) < 1e300);
            double sol[5];
            equilibrium_each_f64<sizeof(typename ST::T) == 8>(rho, ux, uy, uz, th, rref, int(p.model), sol, each);
            if constexpr (MODE == INIT_MEASURE)
                if (solved) {
#pragma unroll
                    for (int k = 0; k < 5; ++k) solved[k * N + n] = sol[k];
                }
            // the checks and the measure are monotonic in D_q: taken on the
            // ends of its range they are those of every population
            bad |= !(sum0 == 0.0);
#pragma unroll
            for (int sh = 0; sh < 6; ++sh) {
                const double d0 = SHELL_W[sh] * rref * lo[sh], d1 = SHELL_W[sh] * rref * hi[sh];
                const double dmax = fmax(-d0, d1);
                bad |= !(dmax < 1e300) || !(SHELL_W[sh] * rref + d0 > 0.0);
                if constexpr (MODE == INIT_MEASURE) dev = fmaxf(dev, float(dmax * double(1u << SHELL_K[sh])));
            }
        }
        if (bad) atomicOr(p.flag, 1u);
    }
    if constexpr (MODE == INIT_MEASURE) block_max_float(dev, maxdev);
}

// (box, tile) lists of the batched launch, one grid row per block size: entry
// t of list i belongs to the last box whose first tile is not after t.
struct TileLists {
    uint2* list[NBLK];
    uint32_t count[NBLK];
};
__global__ __launch_bounds__(BLOCK) void k_tiles(const BatchBox* __restrict__ boxes, uint32_t nboxes, TileLists L)
{
    const int i = blockIdx.y;
    const uint32_t t = blockIdx.x * BLOCK + threadIdx.x;
    if (t >= L.count[i]) return;
    uint32_t lo = 0, hi = nboxes;  // the box is in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (boxes[mid].tile0[i] <= t) lo = mid;
        else hi = mid;
    }
    L.list[i][t] = make_uint2(lo, t - boxes[lo].tile0[i]);
}

// ---------------------------------------------------------------------------
// FP64 decoding helpers for the diagnostics kernels.
// ---------------------------------------------------------------------------
template <class ST, int q>
__device__ inline double dev64(const typename ST::T* f, size_t qs, uint32_t n, const StepParams& p)
{
    double v = double(ST::load(f + size_t(q) * qs + n));
    if constexpr (ST::shifted) v *= double(p.inv_scale[VEL[q].shell]);
    return v;
}

// rho, jx, jy, jz, E of node n in FP64.
template <class ST>
__device__ inline void node_moments64(const typename ST::T* f, size_t qs, uint32_t n, const StepParams& p,
                                      double m[5])
{
    double rd = 0, jx = 0, jy = 0, jz = 0, e4 = 0;
    static_for<Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        constexpr HalfVel v = VEL[q];
        const double d = dev64<ST, q>(f, qs, n, p);
        rd += d;
        jx += double(v.x) * d;
        jy += double(v.y) * d;
        jz += double(v.z) * d;
        e4 += double(v.x * v.x + v.y * v.y + v.z * v.z) * d;
    });
    m[0] = p.rho_ref + rd;
    m[1] = 0.5 * jx;
    m[2] = 0.5 * jy;
    m[3] = 0.5 * jz;
    m[4] = 0.5 * (p.e2_ref + 0.25 * e4);
}

template <class ST>
__global__ __launch_bounds__(BLOCK) void k_moments(const typename ST::T* __restrict__ f, uint32_t qs, uint32_t n0,
                                                   uint32_t count, StepParams p, double* __restrict__ out)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= count) return;
    double m[5];
    node_moments64<ST>(f, qs, n0 + i, p, m);
#pragma unroll
    for (int k = 0; k < 5; ++k) out[size_t(k) * count + i] = m[k];
}

// Block-wide FP64 sum of K values: wavefront butterfly (64 lanes), then the
// wave partials in LDS. Result valid in thread 0.
template <int K>
__device__ inline void block_sum(double v[K], double out[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k)
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    __shared__ double sm[BLOCK / 64][K];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0)
        for (int k = 0; k < K; ++k) sm[wv][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int k = 0; k < K; ++k) {
            double s = sm[0][k];
            for (int i = 1; i < BLOCK / 64; ++i) s += sm[i][k];
            out[k] = s;
        }
}

__device__ inline void block_sum5(double v[5], double out[5]) { block_sum<5>(v, out); }

constexpr int TOTAL_BLOCKS = 1024;

// Per-block partial sums of the node moments (fixed assignment of nodes to
// threads, so the result does not depend on timing).
// sat_check: flag a stored magnitude at the saturation value of the
// stochastic-rounding FP16 encoder (contexts with stochastic rounding).
template <class ST>
__global__ __launch_bounds__(BLOCK) void k_totals(const typename ST::T* __restrict__ f, uint32_t N, StepParams p,
                                                  double* __restrict__ partials, uint32_t sat_check = 0)
{
    double acc[5] = {0, 0, 0, 0, 0};
    for (uint32_t n = blockIdx.x * BLOCK + threadIdx.x; n < N; n += gridDim.x * BLOCK) {
        double m[5];
        node_moments64<ST>(f, p.g.qs, n, p, m);
        if constexpr (ST::SAT > 0.f) {
            if (sat_check) {
                bool sat = false;
                for (int q = 0; q < Q; ++q) sat |= !(fabsf(float(f[size_t(q) * p.g.qs + n])) < ST::SAT);
                if (sat) atomicOr(p.flag, 1u);
            }
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] += m[k];
    }
    double r[5];
    block_sum<5>(acc, r);
    if (threadIdx.x == 0)
        for (int k = 0; k < 5; ++k) partials[blockIdx.x * 5 + k] = r[k];
}

template <int K>
__global__ __launch_bounds__(BLOCK) void k_reduce_partials(const double* __restrict__ partials, uint32_t nblk,
                                                           double* __restrict__ out)
{
    double acc[K];
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    for (uint32_t b = threadIdx.x; b < nblk; b += BLOCK)
        for (int k = 0; k < K; ++k) acc[k] += partials[b * K + k];
    double r[K];
    block_sum<K>(acc, r);
    if (threadIdx.x == 0)
        for (int k = 0; k < K; ++k) out[k] = r[k];
}

// Fourier amplitudes (1/N) sum_n m(n) e^{-i k.x_n} of rho, jx, jy, jz, E and
// theta = (2E/rho - u^2)/3 at the true node positions (sublattice 1 at
// +1/2 in every direction): per-block partial sums of 12 values.
constexpr int PROJ_FIELDS = 6;

template <class ST>
__global__ __launch_bounds__(BLOCK) void k_project(const typename ST::T* __restrict__ f, StepParams p, double kx,
                                                   double ky, double kz, double* __restrict__ partials)
{
    const uint32_t N = p.g.N;
    double acc[2 * PROJ_FIELDS];
    for (int k = 0; k < 2 * PROJ_FIELDS; ++k) acc[k] = 0.0;
    for (uint32_t n = blockIdx.x * BLOCK + threadIdx.x; n < N; n += gridDim.x * BLOCK) {
        double m[5];
        node_moments64<ST>(f, p.g.qs, n, p, m);
        const Coord c = decode(n, p.g);
        const double h = 0.5 * double(c.s);
        const double ph = kx * (double(c.x) + h) + ky * (double(c.y) + h) + kz * (double(c.z) + h);
        double sn, cs;
        sincos(ph, &sn, &cs);
        const double u2 = (m[1] * m[1] + m[2] * m[2] + m[3] * m[3]) / (m[0] * m[0]);
        const double th = (2.0 * m[4] / m[0] - u2) / 3.0;
        const double v[PROJ_FIELDS] = {m[0], m[1], m[2], m[3], m[4], th};
        for (int k = 0; k < PROJ_FIELDS; ++k) {
            acc[2 * k] += v[k] * cs;
            acc[2 * k + 1] -= v[k] * sn;
        }
    }
    double r[2 * PROJ_FIELDS];
    block_sum<2 * PROJ_FIELDS>(acc, r);
    if (threadIdx.x == 0)
        for (int k = 0; k < 2 * PROJ_FIELDS; ++k) partials[blockIdx.x * 2 * PROJ_FIELDS + k] = r[k];
}

// ---------------------------------------------------------------------------
// Population I/O in FP64: nodes [n0, n0 + count) of consecutive q-blocks from
// q0 on, one grid row each, staged as [q - q0][count] (the host's order, so
// that one copy moves them all).
// ---------------------------------------------------------------------------
__host__ __device__ inline int shell_of(uint32_t q)
{
    return q == 0 ? 0 : q < 7 ? 1 : q < 13 ? 2 : q < 25 ? 3 : q < 33 ? 4 : 5;
}

// Stored value h of shell s: f = wref + h inv_scale, h = (f - wref) scale.
struct IoScale {
    float scale[6], inv_scale[6];
    double wref[6];
};

template <class ST>
__global__ __launch_bounds__(BLOCK) void k_get(const typename ST::T* __restrict__ f, uint32_t qs, uint32_t q0,
                                               uint32_t n0, uint32_t count, IoScale c, double* __restrict__ out)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x, q = q0 + blockIdx.y;
    if (i >= count) return;
    const int sh = shell_of(q);
    double v = double(ST::load(f + size_t(q) * qs + n0 + i));
    if constexpr (ST::shifted) v *= double(c.inv_scale[sh]);
    out[size_t(blockIdx.y) * count + i] = c.wref[sh] + v;
}

template <class ST>
__global__ __launch_bounds__(BLOCK) void k_set(typename ST::T* __restrict__ f, uint32_t qs, uint32_t q0, uint32_t n0,
                                               uint32_t count, IoScale c, const double* __restrict__ in)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x, q = q0 + blockIdx.y;
    if (i >= count) return;
    const int sh = shell_of(q);
    double v = in[size_t(blockIdx.y) * count + i] - c.wref[sh];
    if constexpr (ST::shifted) v *= double(c.scale[sh]);
    ST::store(f + size_t(q) * qs + n0 + i, typename ST::R(v));
}

template <class ST>
__global__ __launch_bounds__(BLOCK) void k_gather(const typename ST::T* __restrict__ f, uint32_t N,
                                                  const int64_t* __restrict__ idx, uint32_t count, StepParams p,
                                                  double* __restrict__ out)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= count) return;
    const int64_t k = idx[i];
    const uint32_t q = uint32_t(k / N), n = uint32_t(k - int64_t(q) * N);
    const int sh = shell_of(q);
    double v = double(ST::load(f + size_t(q) * p.g.qs + n));
    if constexpr (ST::shifted) v *= double(p.inv_scale[sh]);
    out[i] = SHELL_W[sh] * p.rho_ref + v;
}

// Source node of every (q, node) of a chunk, by the same code as k_step.
__global__ __launch_bounds__(BLOCK) void k_pull_map(Geom g, uint32_t n0, uint32_t count, int64_t* __restrict__ out)
{
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= count) return;
    const Coord c = decode(n0 + i, g);
    Nbr nb;
    make_nbr(g, c, nb);
    static_for<Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        out[size_t(q) * count + i] = int64_t(pull_src<q>(nb));
    });
}

// ---------------------------------------------------------------------------
// Plain copy of n 16-byte words: reads and writes in equal amounts, fully
// coalesced, no arithmetic. Its rate is what a streaming kernel reaches on
// the device, reported beside the step's own rate. One word per lane in
// 256-lane blocks measured fastest on gfx950 (6.2 TB/s read + write on
// 4 GiB, against 5.6-5.8 with two or four words per lane, 4.2 with eight,
// 5.1-5.4 with 512- and 1024-lane blocks, 5.9 with non-temporal hints).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_copy16(const uint4* __restrict__ in, uint4* __restrict__ out, uint64_t n)
{
    const uint64_t i = uint64_t(blockIdx.x) * BLOCK + threadIdx.x;
    if (i < n) out[i] = in[i];
}

}  // namespace lbm
