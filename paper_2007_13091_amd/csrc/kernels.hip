// HIP kernels of one UGKWP time step for gfx950 (FP64 path and the FP32-transport form).
//
// Order inside a step (paper Sec. 2.3, the four-step particle procedure, and Eq.
// update_macro_variables):
//   k_prim_dt      S0  primitives, tau = mu_ref T^omega / p, min Omega/Lambda     (Sec. 2.4(a))
//   k_cell_prep    S0  dt, exp(-dt/tau), rho^h, sample counts N_sam            (Sec. 2.4(b));
//                  counts of the particles entering through far-field faces
//   k_offsets      exclusive prefixes of both counts, capacity check
//   k_grad         S1  least-squares gradients and limiters (second order only)
//   k_flux(2)      S2  wave flux F^eq + F^{fr,wave} per face                    (Sec. 2.2, 2.4)
//   k_sample       S3  antithetic Maxwellian pairs, uniform positions; start sums S
//   k_inject       S5  free-stream particles entering through far-field faces
//   k_stream         S4+S5 free-flight times and the flights that meet no face, cell by cell:
//                  stayers are written to their cell's region of the next buffer and summed,
//                  the others listed
//   k_stream_long    S4+S5 the same by a block per cell of many particles (small meshes)
//   k_stream_in      S5  flights of the particles entering through far-field faces
//   k_track        S5  the listed flights, face to face; bucket sizes
//   scan           exclusive prefix of the bucket sizes
//   k_scatter      the leavers by end cell
//   k_gather       S6  arrivals in a fixed order, sums E and W^p (k_gather_long: long buckets
//                  by a block)
//   k_update       S6  update of W; step bookkeeping
//   k_avg_cells,   time averaging for steady states, when turned on        (Sec. 2.4(c))
//   k_avg_fin
// No floating-point atomics: per-cell sums use fixed reduction trees, so a run is bitwise
// reproducible.  Integer atomics only hand out bucket slots and counts; the order inside a
// bucket is then fixed by sorting the source indices.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "device_common.hpp"
#include "launch.hpp"

namespace ugkwp {

namespace {

constexpr double kPi = 3.141592653589793238462643383279502884;

// Whole-line stores of particle records with the non-temporal hint: neither the transport nor
// the gather reads back what it writes, and the next kernel's reads of ~1 GB of records do
// not fit in the L2 (measured: transport and gather 3-5% faster)
typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_nt(uint4 *p, const uint4 &v) {
    const u32x4_nt x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<u32x4_nt *>(p));
}
constexpr int kWave = 64;
constexpr int kCountBS = 256;      // cells (far-field faces) per block of k_cell_prep
constexpr int kGatherWaves = 1;    // waves per block in k_gather
constexpr int kSampleCells = 8;     // consecutive cells per wave in k_sample (meshes of 32768 cells or more)
constexpr int kSampleCellsMin = 32768;

// ---------------------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror & Shaw, SC'11); counter = (uid, step, tag<<32|sub, 0),
// key = (seed, 0).
// ---------------------------------------------------------------------------------------
struct U4 {
    uint64_t v[4];
};

// 64 x 64 -> 128-bit product from four 32 x 32 + 64 multiply-adds (v_mad_u64_u32); the low
// half reuses the partial products of the high half
__device__ __forceinline__ void mulhilo64(uint64_t a, uint64_t b, uint64_t &hi, uint64_t &lo) {
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
    const uint64_t p0 = (uint64_t)al * bl;
    const uint64_t t = (uint64_t)al * bh + (p0 >> 32);
    const uint64_t v = (uint64_t)ah * bl + (t & 0xFFFFFFFFULL);
    hi = (uint64_t)ah * bh + ((t >> 32) + (v >> 32));
    lo = (v << 32) | (p0 & 0xFFFFFFFFULL);
}

__device__ __forceinline__ U4 philox(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0, uint64_t k1) {
    constexpr uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    constexpr uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0, lo0, hi1, lo1;
        mulhilo64(M0, c0, hi0, lo0);
        mulhilo64(M1, c2, hi1, lo1);
        uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += W0;
        k1 += W1;
    }
    U4 o;
    o.v[0] = c0;
    o.v[1] = c1;
    o.v[2] = c2;
    o.v[3] = c3;
    return o;
}

// counter (particle id, step, tag << 32 | sub, instance), key (seed, 0)
__device__ __forceinline__ U4 draw(uint64_t seed, uint64_t uid, long long step, int tag, uint32_t sub, int inst) {
    return philox(uid, (uint64_t)step, ((uint64_t)tag << 32) | sub, (uint64_t)inst, seed, 0ULL);
}

// instance of a cell (a single instance needs no table)
__device__ __forceinline__ int inst_of(const Dev &D, int c) { return D.n_inst > 1 ? D.cinst[c] : 0; }

// what the transport of one particle needs from its instance
struct StepCtx {
    unsigned long long seed;
    long long step;
    int inst, max_cross;
};

// uniform in (0, 1), never 0 or 1: FP64 (top 52 bits + 1/2) * 2^-52; FP32 (top 23 bits + 1/2)
// * 2^-23, the leading bits of the same draw
template <typename R>
__device__ __forceinline__ R unif(uint64_t r);
template <>
__device__ __forceinline__ double unif<double>(uint64_t r) {
    return ((double)(r >> 12) + 0.5) * 0x1p-52;
}
template <>
__device__ __forceinline__ float unif<float>(uint64_t r) {
    return ((float)(uint32_t)(r >> 41) + 0.5f) * 0x1p-23f;
}

__device__ __forceinline__ uint64_t make_uid(long long step, int cell, long long k) {
    return (((uint64_t)step & 0x7FFFFULL) << 44) | (((uint64_t)cell & 0xFFFFFFULL) << 20) | ((uint64_t)k & 0xFFFFFULL);
}

// ---------------------------------------------------------------------------------------
// Maxwellian moments in a face frame (R = 1, K = 0), lambda = 1/(2T).
// m[k] = <u_n^k> over the full line (rng 0), u_n > 0 (rng 1) or u_n < 0 (rng -1);
// <u^{k+2}> = U <u^{k+1}> + (k+1)/(2 lambda) <u^k> holds on each half line as well.
// The transport type R is double (plain form) or float (FP32 form).
// ---------------------------------------------------------------------------------------
template <typename R>
struct Prim {
    R rho, un, v, w, lam, T;
    int K;  // internal degrees of freedom (Sec. 2.1): <xi^2> = K / (2 lambda)
};

// temperature of a conservative state with K internal degrees of freedom (R = 1):
// rho E = rho |U|^2 / 2 + (3 + K) rho T / 2
__device__ __forceinline__ double temp_k(const double W[5], int K) {
    return (2.0 / (3.0 + K)) * (W[4] - 0.5 * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]) / W[0]) / W[0];
}

template <typename R>
__device__ __forceinline__ void moments4(int rng, R U, R lam, R m[4]) {
    const R pi = (R)kPi;
    if (rng == 0) {
        m[0] = (R)1;
        m[1] = U;
    } else if (rng > 0) {
        m[0] = (R)0.5 * erfc(-sqrt(lam) * U);
        m[1] = U * m[0] + (R)0.5 * exp(-lam * U * U) / sqrt(pi * lam);
    } else {
        m[0] = (R)0.5 * erfc(sqrt(lam) * U);
        m[1] = U * m[0] - (R)0.5 * exp(-lam * U * U) / sqrt(pi * lam);
    }
    m[2] = U * m[1] + (R)1 / ((R)2 * lam) * m[0];
    m[3] = U * m[2] + (R)2 / ((R)2 * lam) * m[1];
}

// <psi> (H) and <u_n psi> (G) of a unit-density Maxwellian; psi = (1, u_n, v, w, (|u|^2 + xi^2)/2)
template <typename R>
__device__ __forceinline__ void psi_moments(const Prim<R> &p, const R m[4], R H[5], R G[5]) {
    R tr = p.v * p.v + p.w * p.w + (R)1 / p.lam + (R)p.K / ((R)2 * p.lam);
    H[0] = m[0];
    H[1] = m[1];
    H[2] = m[0] * p.v;
    H[3] = m[0] * p.w;
    H[4] = (R)0.5 * (m[2] + m[0] * tr);
    G[0] = m[1];
    G[1] = m[2];
    G[2] = m[1] * p.v;
    G[3] = m[1] * p.w;
    G[4] = (R)0.5 * (m[3] + m[1] * tr);
}

// face frame: t1 = normalise(e_a x n), a = axis of the smallest |n_a| (lowest on ties); t2 = n x t1
template <typename R>
__device__ __forceinline__ void face_frame(const R n[3], R t1[3], R t2[3]) {
    int a = 0;
    if (fabs(n[1]) < fabs(n[a])) a = 1;
    if (fabs(n[2]) < fabs(n[a])) a = 2;
    R e0 = a == 0 ? (R)1 : (R)0, e1 = a == 1 ? (R)1 : (R)0, e2 = a == 2 ? (R)1 : (R)0;
    R c0 = e1 * n[2] - e2 * n[1], c1 = e2 * n[0] - e0 * n[2], c2 = e0 * n[1] - e1 * n[0];
    R l = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    t1[0] = c0 / l;
    t1[1] = c1 / l;
    t1[2] = c2 / l;
    t2[0] = n[1] * t1[2] - n[2] * t1[1];
    t2[1] = n[2] * t1[0] - n[0] * t1[2];
    t2[2] = n[0] * t1[1] - n[1] * t1[0];
}

// primitives of a cell state in the face frame; the energy -> temperature recovery is FP64
template <typename R>
__device__ __forceinline__ Prim<R> to_frame(const double W[5], const R n[3], const R t1[3], const R t2[3], int K) {
    Prim<R> p;
    const double U = W[1] / W[0], V = W[2] / W[0], Z = W[3] / W[0];
    const double T = temp_k(W, K);
    const R u = (R)U, v = (R)V, z = (R)Z;
    p.rho = (R)W[0];
    p.un = u * n[0] + v * n[1] + z * n[2];
    p.v = u * t1[0] + v * t1[1] + z * t1[2];
    p.w = u * t2[0] + v * t2[1] + z * t2[2];
    p.T = (R)T;
    p.lam = (R)1 / ((R)2 * p.T);
    p.K = K;
    return p;
}

// Taylor coefficients (-1)^k/k! and (-1)^k (k-1)/k!, k = 2..24, for the series forms of
//   q1/tau = x - 1 + e^-x   and   (q4 - dt e)/tau = 1 - (1 + x) e^-x.
// For second order also (k = 3..24), with q2, q3, q5 + dt^2 e / 2 = tau^2 x^3 times
//   sum (-1)^k (k-2)/k! x^(k-3),  -sum (-1)^k / k! x^(k-3),  sum (-1)^k (k-1)(k-2)/(2 k!) x^(k-3).
struct QSeries {
    double a[25], b[25], c[25], d[25], e[25];
    float af[25], bf[25], cf[25], df[25], ef[25];
    constexpr QSeries() : a(), b(), c(), d(), e(), af(), bf(), cf(), df(), ef() {
        double f = 1.0;
        for (int k = 1; k <= 24; ++k) {
            f = f * k;
            double s = (k % 2 == 0) ? 1.0 : -1.0;
            a[k] = s / f;
            b[k] = s * (k - 1) / f;
            c[k] = s * (k - 2) / f;
            d[k] = -s / f;
            e[k] = s * (double)((k - 1) * (k - 2)) / (2.0 * f);
            af[k] = (float)a[k];
            bf[k] = (float)b[k];
            cf[k] = (float)c[k];
            df[k] = (float)d[k];
            ef[k] = (float)e[k];
        }
    }
};
__constant__ QSeries kQ = QSeries();

// q1 and q4 - dt e of the time-integrated interface distribution (Eq. of q1..q5), x = dt/tau:
// series below x = 1 (terms x^2..x^24 in FP64, x^2..x^12 in FP32, Horner), closed forms above
template <typename R>
__device__ __forceinline__ void qcoef(R dt, R tau, R &q1, R &q4m) {
    const R x = dt / tau;
    if (x < (R)1) {
        R s1 = (R)0, s4 = (R)0;
        if constexpr (sizeof(R) == 8) {
#pragma unroll
            for (int k = 24; k >= 2; --k) {
                s1 = s1 * x + kQ.a[k];
                s4 = s4 * x + kQ.b[k];
            }
        } else {
#pragma unroll
            for (int k = 12; k >= 2; --k) {
                s1 = s1 * x + kQ.af[k];
                s4 = s4 * x + kQ.bf[k];
            }
        }
        q1 = tau * (s1 * x * x);
        q4m = tau * (s4 * x * x);
    } else {
        const R e = exp(-x);
        q1 = tau * (x - (R)1 + e);
        q4m = tau * ((R)1 - ((R)1 + x) * e);
    }
}

// First-order wave flux between two face-frame states (gks: the wave-only start phase, in which
// no particle is sampled and the waves carry the whole free transport q4 g^h of the hydro part):
//   F = rho0 q1 <u_n psi>_0 + (q4 - dt e) (rhoh_l <u_n psi>_{l,u>0} + rhoh_r <u_n psi>_{r,u<0})
// with g0 from the upwind moments of both sides and tau at the face from g0 plus the
// numerical dissipation C2 |pl - pr| / (pl + pr) dt of Sec. 2.4(d).
// Shakhov model (qsh != 0): the g0 term becomes g0^+ = g0 [1 + (1 - Pr) c.q (|c|^2/T - 5) / (5 p T)],
// whose correction carries, over all velocities, no mass or momentum and the energy flux
// (1 - Pr) q.n for any g0 (Gaussian moments <c_n^2 |c|^2> = 5 T^2, <c_n^2 |c|^4> = 35 T^3): F^eq
// gains q1 qsh in energy, qsh = (1 - Pr) q_f.n with q_f the heat flux at the face (shakhov_qsh).
template <typename R>
__device__ __forceinline__ void flux_pair(const Prim<R> &l, const Prim<R> &r, R hl, R hr, R dt, R mu_ref, R omega,
                                          R c2, bool gks, R qsh, R Ff[5]) {
    R ml[4], mr[4], Hl[5], Gl[5], Hr[5], Gr[5];
    moments4<R>(1, l.un, l.lam, ml);
    moments4<R>(-1, r.un, r.lam, mr);
    psi_moments<R>(l, ml, Hl, Gl);
    psi_moments<R>(r, mr, Hr, Gr);
    R W0[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) W0[k] = l.rho * Hl[k] + r.rho * Hr[k];
    Prim<R> z;
    z.rho = W0[0];
    z.un = W0[1] / W0[0];
    z.v = W0[2] / W0[0];
    z.w = W0[3] / W0[0];
    z.K = l.K;
    z.T = ((R)2 / (R)(3 + z.K)) * (W0[4] - (R)0.5 * (W0[1] * W0[1] + W0[2] * W0[2] + W0[3] * W0[3]) / W0[0]) / W0[0];
    z.lam = (R)1 / ((R)2 * z.T);
    R pl = l.rho * l.T, pr = r.rho * r.T;
    R tau = mu_ref * pow(z.T, omega) / (z.rho * z.T) + c2 * (fabs(pl - pr) / (pl + pr)) * dt;
    R q1, q4m;
    qcoef<R>(dt, tau, q1, q4m);
    if (gks) q4m = q4m + dt * exp(-dt / tau);  // wave-only start: the waves carry all of W^h
    R m0[4], H0[5], G0[5];
    moments4<R>(0, z.un, z.lam, m0);
    psi_moments<R>(z, m0, H0, G0);
#pragma unroll
    for (int k = 0; k < 5; ++k) Ff[k] = q1 * z.rho * G0[k] + q4m * (hl * Gl[k] + hr * Gr[k]);
    if (qsh != (R)0) Ff[4] = Ff[4] + q1 * qsh;
}

// ---------------------------------------------------------------------------------------
// wave reductions with a fixed butterfly (deterministic)
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = v + __shfl_xor(v, s);
    return v;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = v + __shfl_xor(v, s);
    return v;
}

// a value that every lane of the wave holds, as a scalar
__device__ __forceinline__ long long uniform64(long long v) {
    return ((long long)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((int)v);
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, s));
    return v;
}

// ---------------------------------------------------------------------------------------
// slots of a particle buffer (layout: see Particles)
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int hi32(unsigned long long v) { return (int)(v >> 32); }
__device__ __forceinline__ int lo32(unsigned long long v) { return (int)(v & 0xFFFFFFFFULL); }

// empty slots in the regions of the cells before c
__device__ __forceinline__ int empty_before(const Dev &D, int b, int c) {
    const unsigned long long o = D.off[c];
    return D.v0[b][c] - (hi32(o) - lo32(o));
}
// slot of place a >= D.cap - span of the second part of buffer b: the regions' empty slots in order
__device__ __forceinline__ int empty_slot(const Dev &D, int b, int h) {
    int lo = 0, hi = D.nc;
    while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if (empty_before(D, b, mid) <= h)
            lo = mid;
        else
            hi = mid;
    }
    const unsigned long long o0 = D.off[lo], o1 = D.off[lo + 1];
    const int stay = (hi32(o1) - lo32(o1)) - (hi32(o0) - lo32(o0));
    return D.v0[b][lo] + stay + (h - empty_before(D, b, lo));
}
// slot of place a of the second part
__device__ __forceinline__ int slot_of(const Dev &D, int b, long long span, long long a) {
    return a < D.cap - span ? (int)(span + a) : empty_slot(D, b, (int)(a - (D.cap - span)));
}

// the step's most crossings of one particle: a block's maximum raises the step's (reset by
// k_prim_dt); the atomic is issued only when it would change it (the value read first only
// grows during the step, so a stale read costs at most an extra atomic)
__device__ __forceinline__ void raise_max_cross(const Dev &D, unsigned m) {
    if (m > *(volatile unsigned *)&D.sc->max_cross) atomicMax(&D.sc->max_cross, m);
}

// Totals over the wave of P[0..4] and C[0..4], lane k < 5 receiving P_k and C_k.  Each total
// is built from the same pairwise additions as wave_sum (partial sums of lanes that differ
// in bit 5, then 4, ..., then 0), so it is bitwise wave_sum's; but at each of the first levels
// a lane keeps half of the values it carries and hands its partner the other half: 13
// exchanges instead of 60.
__device__ __forceinline__ void wave_sum_pc(const double P[5], const double C[5], double &pk, double &ck) {
    const int lane = lane_id();
    const bool b5 = (lane & 32) != 0, b4 = (lane & 16) != 0, b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
    double x[6];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const double send = b5 ? P[k] : C[k];
        const double keep = b5 ? C[k] : P[k];
        x[k] = keep + __shfl_xor(send, 32);
    }
    x[5] = 0.0;  // lanes with bit 5 clear now carry the P partial sums, the others the C ones
    double y[4];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double send = b4 ? x[j] : x[3 + j];
        const double keep = b4 ? x[3 + j] : x[j];
        y[j] = keep + __shfl_xor(send, 16);
    }
    y[3] = 0.0;
    double z[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const double send = b3 ? y[j] : y[2 + j];
        const double keep = b3 ? y[2 + j] : y[j];
        z[j] = keep + __shfl_xor(send, 8);
    }
    double q;
    {
        const double send = b2 ? z[0] : z[1];
        const double keep = b2 ? z[1] : z[0];
        q = keep + __shfl_xor(send, 4);
    }
    q = q + __shfl_xor(q, 2);
    q = q + __shfl_xor(q, 1);
    // a lane's total is component 3 b4 + 2 b3 + b2 (combinations above 4, or with b3 and b2
    // both set below bit 4, carry the zero padding): P_0..P_4 sit in lanes 0, 4, 8, 16, 20 and
    // C_k 32 lanes above P_k
    const int src = lane < 3 ? 4 * lane : (lane < 5 ? 4 * lane + 4 : 0);
    pk = __shfl(q, src);
    ck = __shfl(q, src + 32);
}

// ---------------------------------------------------------------------------------------
// S0: primitives, tau, min Omega / Lambda
// ---------------------------------------------------------------------------------------
// min Omega / Lambda of an instance, as bits: the blocks' minima go to dt_slots words, each in a
// memory line of its own: the atomics on a line are served one after the other (349,224
// tetrahedra, 1,365 blocks on one word: 22 us, now 9.2; 32 cavities of 32^3 cells, 70 us, now 16)
__device__ __forceinline__ unsigned long long *dt_slot(const Dev &D, int inst, int slot) {
    return D.dtmin + ((long long)inst * D.dt_slots + slot) * D.dt_stride;
}
__device__ __forceinline__ double step_dt(const Dev &D, int inst) {
    unsigned long long m = *dt_slot(D, inst, 0);
    if (D.dt_slots == kDtSlots) {
#pragma unroll
        for (int k = 1; k < kDtSlots; ++k) m = min(m, *dt_slot(D, inst, k));
    }
    return D.ip[inst].cfl * __longlong_as_double((long long)m);
}

__global__ void __launch_bounds__(256) k_prim_dt(Dev D) {
    __shared__ double smin[256 / kWave];
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        Scalars *s = D.sc;
        s->n_sampled = 0;
        s->max_cross = 0u;
        s->n_big = 0u;
    }
    // partial sums of crossings and wall hits of this step's transport
    if (blockIdx.x == 0 && threadIdx.x < 2 * kWallSeg) D.spart[threadIdx.x] = 0ULL;
    double r = INFINITY;
    int inst = 0;
    if (c < D.nc) {
        const int nc = D.nc;
        inst = inst_of(D, c);
        const InstP &P = D.ip[inst];
        double rho = D.W[c], m0 = D.W[nc + c], m1 = D.W[2 * nc + c], m2 = D.W[3 * nc + c], E = D.W[4 * nc + c];
        bool bad = !(rho > 0.0) || !isfinite(rho);
        double T = 0.0;
        double U = 0.0, V = 0.0, Z = 0.0;
        if (!bad) {
            U = m0 / rho;
            V = m1 / rho;
            Z = m2 / rho;
            T = (2.0 / (3.0 + D.K)) * (E - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) / rho) / rho;
            bad = !(T > 0.0) || !isfinite(T);
        }
        // geometry loaded with W, before any store
        const double dS0 = D.dS[c], dS1 = D.dS[nc + c], dS2 = D.dS[2 * nc + c], vol = D.vol[c];
        if (bad) {
            atomicOr(&D.sc->err, kErrNonPhys);
            D.tau[c] = 1.0;
        } else {
            D.tau[c] = P.mu_ref * pow(T, P.omega) / (rho * T);
            double cs = 3.0 * sqrt(T);
            double lam = (fabs(U) + cs) * dS0 + (fabs(V) + cs) * dS1 + (fabs(Z) + cs) * dS2;
            r = vol / lam;
        }
    }
    // the min over each instance's cells; a block whose cells straddle two instances
    // reports per cell (positive doubles order as their bit patterns)
    const int cfirst = blockIdx.x * blockDim.x;
    const int clast = min(cfirst + (int)blockDim.x, D.nc) - 1;
    const int slot = (int)blockIdx.x & (D.dt_slots - 1);
    if (D.n_inst > 1 && D.cinst[cfirst] != D.cinst[clast]) {
        if (r < INFINITY && r > 0.0) atomicMin(dt_slot(D, inst, slot), (unsigned long long)__double_as_longlong(r));
        return;
    }
#pragma unroll
    for (int m = kWave / 2; m > 0; m >>= 1) r = fmin(r, __shfl_xor(r, m));
    if (lane_id() == 0) smin[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < 256 / kWave; ++w) r = fmin(r, smin[w]);
    if (r < INFINITY && r > 0.0)
        atomicMin(dt_slot(D, inst_of(D, cfirst), slot), (unsigned long long)__double_as_longlong(r));
}

// ---------------------------------------------------------------------------------------
// S0 (cont.): dt, collisionless fraction, hydro density, number of particles to sample
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ long long cell_prep(const Dev &D, int c) {
    const int inst = inst_of(D, c);
    const InstP &P = D.ip[inst];
    const double dt = step_dt(D, inst);
    const long long step = D.is[inst].step;
    // every per-cell value loaded before the first store
    const double vol = D.vol[c];
    const double Pm = D.P[c];
    const double rho = D.W[c];
    const double tau = D.tau[c];
    const int nleft = hi32(D.off[c + 1]) - hi32(D.off[c]);
    // bucket counters of this step's transport (survivors ending in c, collided ending in c)
    D.cnt64[c] = 0ULL;
    D.cnt64[D.nc + c] = 0ULL;
    if (c == P.cell0) {
        D.is[inst].dt = dt;
        if (inst == 0) D.sc->dt = dt;
    }
    const double rhop = Pm / vol;
    // the hydro density is a difference of sums; below 1e-12 rho it is roundoff of that
    // subtraction (particles hold all the mass) and counts as zero
    const double rh = rho - rhop;
    const double rhoh = rh > 1e-12 * rho ? rh : 0.0;
    // wave-only start phase: no particle is sampled
    const double e = step < P.gks_steps ? 0.0 : exp(-dt / tau);
    D.rhoh[c] = rhoh;
    D.ec[c] = e;
    const double rhohp = e * rhoh;
    long long ns = 0;
    if (rhohp > 0.0 && rhop + rhohp > 0.0) {
        double r = (0.5 * P.n_ref) * (rhohp / (rhop + rhohp));
        double cr = ceil(r);
        if (!(cr <= 524288.0)) {
            atomicOr(&D.sc->err, kErrCellCount);
        } else {
            ns = 2 * (long long)cr;
            long long need = (long long)P.n_min - nleft;
            if (need > 0) {
                long long ne = 2 * ((need + 1) / 2);
                if (ne > ns) ns = ne;
            }
            if (ns > (1LL << 20)) {
                atomicOr(&D.sc->err, kErrCellCount);
                ns = 0;
            }
        }
    }
    D.nsam[c] = ns;
    return ns;
}

// Diffuse isothermal wall (Sec. 2.4(e)), first order at the state l (n out of the domain):
// incoming q1 g + (q4 - dt e) g^h with the cell tau; the wall emits rho_w M(T_w, U_w) over
// u_n < 0 for the step, rho_w from zero net mass flux; the mass component is exactly 0.
template <typename R>
__device__ __forceinline__ void diffuse_flux(const Prim<R> &l, R h, R tau_c, const R n[3], const R t1[3],
                                             const R t2[3], const DevBC &bc, R dt, bool gks, R Ff[5]) {
    R q1, q4m;
    qcoef<R>(dt, tau_c, q1, q4m);
    if (gks) q4m = q4m + dt * exp(-dt / tau_c);
    R ml[4], Hl[5], Gl[5];
    moments4<R>(1, l.un, l.lam, ml);
    psi_moments<R>(l, ml, Hl, Gl);
    R Fin[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) Fin[k] = q1 * l.rho * Gl[k] + q4m * h * Gl[k];
    const R uw[3] = {(R)bc.Uw[0], (R)bc.Uw[1], (R)bc.Uw[2]};
    Prim<R> w;
    w.rho = (R)1;
    w.un = uw[0] * n[0] + uw[1] * n[1] + uw[2] * n[2];
    w.v = uw[0] * t1[0] + uw[1] * t1[1] + uw[2] * t1[2];
    w.w = uw[0] * t2[0] + uw[1] * t2[1] + uw[2] * t2[2];
    w.T = (R)bc.Tw;
    w.lam = (R)1 / ((R)2 * w.T);
    w.K = l.K;
    R mw[4], Hw[5], Gw[5];
    moments4<R>(-1, w.un, w.lam, mw);
    psi_moments<R>(w, mw, Hw, Gw);
    const R rhow = -Fin[0] / (dt * Gw[0]);
#pragma unroll
    for (int k = 0; k < 5; ++k) Ff[k] = Fin[k] + dt * rhow * Gw[k];
    Ff[0] = (R)0;
}

// Shakhov term of face f (owner c, neighbour nb), FP64: (1 - Pr) q_f.n with the heat flux at the
// face the mean of the two cells' (a far-field face: the free stream's is zero); walls keep the
// BGK flux (0 here).  0 for Pr = 1.
__device__ __forceinline__ double shakhov_qsh(const Dev &D, const InstP &P, int f, int c, int nb) {
    if (P.pr == 1.0) return 0.0;
    if (nb < 0 && D.bc[-1 - nb].type != 2) return 0.0;
    const int nc = D.nc, nf = D.nf;
    const double qa[3] = {D.qh[c], D.qh[nc + c], D.qh[2 * nc + c]};
    double qb[3] = {0.0, 0.0, 0.0};
    if (nb >= 0) {
        qb[0] = D.qh[nb];
        qb[1] = D.qh[nc + nb];
        qb[2] = D.qh[2 * nc + nb];
    }
    const double qn = (0.5 * (qa[0] + qb[0])) * D.fn[f] + (0.5 * (qa[1] + qb[1])) * D.fn[nf + f] +
                      (0.5 * (qa[2] + qb[2])) * D.fn[2 * nf + f];
    return (1.0 - P.pr) * qn;
}

// ---------------------------------------------------------------------------------------
// S2: wave flux per face, times the area, oriented owner -> neighbour.  Arithmetic in R
// (FP32 form: float), inputs recovered from the FP64 state, result stored in FP64.
// ---------------------------------------------------------------------------------------
template <typename R, int BS>
__global__ void __launch_bounds__(BS) k_flux(Dev D) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= D.nf) return;
    const int nc = D.nc, nf = D.nf;
    const int c = D.fown[f];
    const int inst = inst_of(D, c);
    const InstP &P = D.ip[inst];
    if (P.recon != 0) return;
    const R dt = (R)D.is[inst].dt;
    const R mu = (R)P.mu_ref, om = (R)P.omega, c2 = (R)P.c2;
    const bool gks = D.is[inst].step < P.gks_steps;
    const int nb = D.fnb[f];
    R n[3] = {(R)D.fn[f], (R)D.fn[nf + f], (R)D.fn[2 * nf + f]};
    R t1[3], t2[3];
    face_frame<R>(n, t1, t2);
    double Wl[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) Wl[k] = D.W[k * nc + c];
    const Prim<R> l = to_frame<R>(Wl, n, t1, t2, D.K);
    const R qsh = (R)shakhov_qsh(D, P, f, c, nb);
    R Ff[5];
    if (nb >= 0) {
        double Wr[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) Wr[k] = D.W[k * nc + nb];
        const Prim<R> r = to_frame<R>(Wr, n, t1, t2, D.K);
        flux_pair<R>(l, r, (R)D.rhoh[c], (R)D.rhoh[nb], dt, mu, om, c2, gks, qsh, Ff);
    } else {
        const DevBC bc = D.bc[-1 - nb];
        if (bc.type == 0) {
            // specular wall: mirror state, keep only the normal momentum
            Prim<R> g = l;
            g.un = -l.un;
            const R h = (R)D.rhoh[c];
            flux_pair<R>(l, g, h, h, dt, mu, om, c2, gks, (R)0, Ff);
            Ff[0] = (R)0;
            Ff[2] = (R)0;
            Ff[3] = (R)0;
            Ff[4] = (R)0;
        } else if (bc.type == 1) {
            diffuse_flux<R>(l, (R)D.rhoh[c], (R)D.tau[c], n, t1, t2, bc, dt, gks, Ff);
        } else {
            // far field: the free stream as the right state (hydro density = its density)
            const Prim<R> r = to_frame<R>(bc.Winf, n, t1, t2, D.K);
            flux_pair<R>(l, r, (R)D.rhoh[c], (R)bc.Winf[0], dt, mu, om, c2, gks, qsh, Ff);
        }
    }
    const R a = (R)D.farea[f];
    D.Phi[f] = (double)(Ff[0] * a);
#pragma unroll
    for (int d = 0; d < 3; ++d) D.Phi[(1 + d) * nf + f] = (double)((Ff[1] * n[d] + Ff[2] * t1[d] + Ff[3] * t2[d]) * a);
    D.Phi[4 * nf + f] = (double)(Ff[4] * a);
}

// ---------------------------------------------------------------------------------------
// Second order (Sec. 2.2 with slopes and time derivative; Sec. 2.4 for the wave part).
// ---------------------------------------------------------------------------------------

// q1, q2, q3, q4 - dt e, q5 + dt^2 e / 2 (series below x = 1, closed forms above)
template <typename R>
__device__ __forceinline__ void qcoef5(R dt, R tau, R q[5]) {
    const R x = dt / tau;
    if (x < (R)1) {
        R s1 = (R)0, s4 = (R)0, s2 = (R)0, s3 = (R)0, s5 = (R)0;
        constexpr int K = sizeof(R) == 8 ? 24 : 12;
#pragma unroll
        for (int k = K; k >= 2; --k) {
            if constexpr (sizeof(R) == 8) {
                s1 = s1 * x + kQ.a[k];
                s4 = s4 * x + kQ.b[k];
                if (k >= 3) {
                    s2 = s2 * x + kQ.c[k];
                    s3 = s3 * x + kQ.d[k];
                    s5 = s5 * x + kQ.e[k];
                }
            } else {
                s1 = s1 * x + kQ.af[k];
                s4 = s4 * x + kQ.bf[k];
                if (k >= 3) {
                    s2 = s2 * x + kQ.cf[k];
                    s3 = s3 * x + kQ.df[k];
                    s5 = s5 * x + kQ.ef[k];
                }
            }
        }
        q[0] = tau * (s1 * x * x);
        q[3] = tau * (s4 * x * x);
        q[1] = tau * tau * (s2 * x * x * x);
        q[2] = tau * tau * (s3 * x * x * x);
        q[4] = tau * tau * (s5 * x * x * x);
    } else {
        const R e = exp(-x);
        q[0] = tau * (x - (R)1 + e);
        q[3] = tau * ((R)1 - ((R)1 + x) * e);
        q[1] = tau * tau * ((R)2 * ((R)1 - e) - x * ((R)1 + e));
        q[2] = tau * tau * ((R)0.5 * x * x - x + (R)1 - e);
        q[4] = tau * tau * (((R)1 + x + (R)0.5 * x * x) * e - (R)1);
    }
}

// <u^k>, k < N, over a range (0 all, +1 u > 0, -1 u < 0)
template <typename R, int N>
__device__ __forceinline__ void moments_n(int rng, R U, R lam, R m[N]) {
    R m4[4];
    moments4<R>(rng, U, lam, m4);
    m[0] = m4[0];
    m[1] = m4[1];
#pragma unroll
    for (int k = 0; k + 2 < N; ++k) m[k + 2] = U * m[k + 1] + (R)(k + 1) / ((R)2 * lam) * m[k];
}

// normal moments over a range to order 6, tangential ones over the full line to order 5, and
// of the K internal components: x2 = <xi^2> = K / (2 lambda), x4 = <xi^4> = K (K + 2) / (4 lambda^2)
template <typename R>
struct Mom3 {
    R u[7], v[6], w[6];
    R x2, x4;
};
template <typename R>
__device__ __forceinline__ void mom3(int rng, const Prim<R> &g, Mom3<R> &M) {
    moments_n<R, 7>(rng, g.un, g.lam, M.u);
    moments_n<R, 6>(0, g.v, g.lam, M.v);
    moments_n<R, 6>(0, g.w, g.lam, M.w);
    M.x2 = (R)g.K / ((R)2 * g.lam);
    M.x4 = (R)(g.K * (g.K + 2)) / ((R)4 * g.lam * g.lam);
}
template <int I, int J, int K, typename R>
__device__ __forceinline__ R mono(const Mom3<R> &M) {
    return M.u[I] * M.v[J] * M.w[K];
}
// < u^I v^J w^K (a . psi) >, a . psi = a0 + a1 u + a2 v + a3 w + a4 (u^2 + v^2 + w^2 + xi^2) / 2
template <int I, int J, int K, typename R>
__device__ __forceinline__ R amom(const Mom3<R> &M, const R a[5]) {
    return a[0] * mono<I, J, K>(M) + a[1] * mono<I + 1, J, K>(M) + a[2] * mono<I, J + 1, K>(M) +
           a[3] * mono<I, J, K + 1>(M) +
           (R)0.5 * a[4] * (mono<I + 2, J, K>(M) + mono<I, J + 2, K>(M) + mono<I, J, K + 2>(M) + mono<I, J, K>(M) * M.x2);
}
// < u^I v^J w^K (a . psi) xi^2 > (the xi components are independent of u, v, w)
template <int I, int J, int K, typename R>
__device__ __forceinline__ R amom_xi(const Mom3<R> &M, const R a[5]) {
    return M.x2 * (a[0] * mono<I, J, K>(M) + a[1] * mono<I + 1, J, K>(M) + a[2] * mono<I, J + 1, K>(M) +
                   a[3] * mono<I, J, K + 1>(M) +
                   (R)0.5 * a[4] * (mono<I + 2, J, K>(M) + mono<I, J + 2, K>(M) + mono<I, J, K + 2>(M))) +
           (R)0.5 * a[4] * mono<I, J, K>(M) * M.x4;
}
// out_k = < u^P v^Q w^S (a . psi) psi_k >
template <int P, int Q, int S, typename R>
__device__ __forceinline__ void gvec(const Mom3<R> &M, const R a[5], R out[5]) {
    out[0] = amom<P, Q, S>(M, a);
    out[1] = amom<P + 1, Q, S>(M, a);
    out[2] = amom<P, Q + 1, S>(M, a);
    out[3] = amom<P, Q, S + 1>(M, a);
    out[4] = (R)0.5 * (amom<P + 2, Q, S>(M, a) + amom<P, Q + 2, S>(M, a) + amom<P, Q, S + 2>(M, a) +
                       amom_xi<P, Q, S>(M, a));
}
// out_k = < u psi_k >
template <typename R>
__device__ __forceinline__ void uvec(const Mom3<R> &M, R out[5]) {
    out[0] = mono<1, 0, 0>(M);
    out[1] = mono<2, 0, 0>(M);
    out[2] = mono<1, 1, 0>(M);
    out[3] = mono<1, 0, 1>(M);
    out[4] = (R)0.5 * (mono<3, 0, 0>(M) + mono<1, 2, 0>(M) + mono<1, 0, 2>(M) + mono<1, 0, 0>(M) * M.x2);
}

// micro slope a with <(a . psi) psi> = b over the unit Maxwellian g, N = 3 + K:
//   R = 2 b5 - (|U|^2 + N/(2 lambda)) b1, R_i = b_{i+1} - U_i b1, a5 = 4 lambda^2/N (R - 2 U.R_i),
//   a_{i+1} = 2 lambda R_i - U_i a5, a1 = b1 - U.a_{2..4} - a5 (|U|^2 + N/(2 lambda))/2
template <typename R>
__device__ __forceinline__ void slope(const Prim<R> &g, const R b[5], R a[5]) {
    const R U0 = g.un, U1 = g.v, U2 = g.w, lam = g.lam;
    const R N = (R)(3 + g.K);
    const R q2 = U0 * U0 + U1 * U1 + U2 * U2;
    const R th = N / ((R)2 * lam);
    const R Rr = (R)2 * b[4] - (q2 + th) * b[0];
    const R R0 = b[1] - U0 * b[0], R1 = b[2] - U1 * b[0], R2 = b[3] - U2 * b[0];
    a[4] = ((R)4 * lam * lam / N) * (Rr - (R)2 * (U0 * R0 + U1 * R1 + U2 * R2));
    a[1] = (R)2 * lam * R0 - U0 * a[4];
    a[2] = (R)2 * lam * R1 - U1 * a[4];
    a[3] = (R)2 * lam * R2 - U2 * a[4];
    a[0] = b[0] - (U0 * a[1] + U1 * a[2] + U2 * a[3]) - (R)0.5 * a[4] * (q2 + th);
}
template <typename R>
__device__ __forceinline__ void slope_of(const Prim<R> &g, const R dW[5], R a[5]) {
    R b[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) b[k] = dW[k] / g.rho;
    slope<R>(g, b, a);
}

// one side of a face in the face frame: reconstructed state and hydro state with their
// derivatives along n, t1, t2 (hydro density 0: no hydro part)
template <typename R>
struct Side2 {
    Prim<R> g, h;
    R dW[3][5], dWh[3][5];
};

// derivatives of a conservative state along n, t1, t2 from its gradient (G at [3k+d] of a
// [15][stride] array), in frame components
template <typename R>
__device__ __forceinline__ void frame_derivs(const double *G, long long stride, long long idx, const R n[3],
                                             const R t1[3], const R t2[3], R out[3][5]) {
    R g[5][3];
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int d = 0; d < 3; ++d) g[k][d] = (R)G[(3 * k + d) * stride + idx];
    const R *e[3] = {n, t1, t2};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        R dk[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) dk[k] = g[k][0] * e[d][0] + g[k][1] * e[d][1] + g[k][2] * e[d][2];
        out[d][0] = dk[0];
        out[d][1] = dk[1] * n[0] + dk[2] * n[1] + dk[3] * n[2];
        out[d][2] = dk[1] * t1[0] + dk[2] * t1[1] + dk[3] * t1[2];
        out[d][3] = dk[1] * t2[0] + dk[2] * t2[1] + dk[3] * t2[2];
        out[d][4] = dk[4];
    }
}

// W0 of a face from the upwind half moments, as primitives
template <typename R>
__device__ __forceinline__ void face_state(const Side2<R> &L, const Side2<R> &Rs, const Mom3<R> &ML, const Mom3<R> &MR,
                                           Prim<R> &z) {
    R W0[5];
    {
        const R one[5] = {(R)1, (R)0, (R)0, (R)0, (R)0};
        R Hl[5], Hr[5];
        gvec<0, 0, 0, R>(ML, one, Hl);
        gvec<0, 0, 0, R>(MR, one, Hr);
#pragma unroll
        for (int k = 0; k < 5; ++k) W0[k] = L.g.rho * Hl[k] + Rs.g.rho * Hr[k];
    }
    z.rho = W0[0];
    z.un = W0[1] / W0[0];
    z.v = W0[2] / W0[0];
    z.w = W0[3] / W0[0];
    z.K = L.g.K;
    z.T = ((R)2 / (R)(3 + z.K)) * (W0[4] - (R)0.5 * (W0[1] * W0[1] + W0[2] * W0[2] + W0[3] * W0[3]) / W0[0]) / W0[0];
    z.lam = (R)1 / ((R)2 * z.T);
}
// the slope abar_A along axis A (0 n, 1 t1, 2 t2) from
// W_x = rho_l <(a_l . psi) psi>_{>0} + rho_r <(a_r . psi) psi>_{<0}
template <int A, typename R>
__device__ __forceinline__ void face_slope(const Side2<R> &L, const Side2<R> &Rs, const Mom3<R> &ML, const Mom3<R> &MR,
                                           const Prim<R> &z, R abar[5]) {
    R al[5], ar[5], Sl[5], Sr[5], Wx[5];
    slope_of<R>(L.g, L.dW[A], al);
    slope_of<R>(Rs.g, Rs.dW[A], ar);
    gvec<0, 0, 0, R>(ML, al, Sl);
    gvec<0, 0, 0, R>(MR, ar, Sr);
#pragma unroll
    for (int k = 0; k < 5; ++k) Wx[k] = L.g.rho * Sl[k] + Rs.g.rho * Sr[k];
    slope_of<R>(z, Wx, abar);
}
// <u_A (a . psi) psi>, u_A the velocity along axis A, and <u u_A (a . psi) psi>
template <int A, typename R>
__device__ __forceinline__ void gaxis(const Mom3<R> &M, const R a[5], R out[5]) {
    gvec<A == 0, A == 1, A == 2, R>(M, a, out);
}
template <int A, typename R>
__device__ __forceinline__ void guaxis(const Mom3<R> &M, const R a[5], R out[5]) {
    gvec<1 + (A == 0), A == 1, A == 2, R>(M, a, out);
}
// <u u_A (a~_A . psi) psi> of a side's hydro part
template <int A, typename R>
__device__ __forceinline__ void hydro_axis(const Mom3<R> &MH, const Side2<R> &S, R out[5]) {
    R ah[5];
    slope_of<R>(S.h, S.dWh[A], ah);
    guaxis<A, R>(MH, ah, out);
}
template <typename R>
__device__ __forceinline__ void face_q(const Side2<R> &L, const Side2<R> &Rs, const Prim<R> &z, R dt, R mu_ref, R omega,
                                       R c2, bool gks, R q[5]) {
    const R pl = L.g.rho * L.g.T, pr = Rs.g.rho * Rs.g.T;
    const R tau = mu_ref * pow(z.T, omega) / (z.rho * z.T) + c2 * (fabs(pl - pr) / (pl + pr)) * dt;
    qcoef5<R>(dt, tau, q);
    if (gks) {
        // wave-only start: q4 = (q4 - dt e) + dt e, q5 = (q5 + dt^2 e / 2) - dt^2 e / 2
        const R e = exp(-dt / tau);
        q[3] = q[3] + dt * e;
        q[4] = q[4] - (R)0.5 * dt * dt * e;
    }
}
// the equilibrium part of the flux from t = sum_A <u_A (abar_A . psi) psi> and
// X = sum_A <u u_A (abar_A . psi) psi>
template <typename R>
__device__ __forceinline__ void face_eq(const Prim<R> &z, const Mom3<R> &M0, const R t[5], const R X[5], const R q[5],
                                        R Ff[5]) {
    R At[5], bt[5], G0[5], GA[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) bt[k] = -t[k];
    slope<R>(z, bt, At);
    uvec<R>(M0, G0);
    gvec<1, 0, 0, R>(M0, At, GA);
#pragma unroll
    for (int k = 0; k < 5; ++k) Ff[k] = z.rho * (q[0] * G0[k] + q[1] * X[k] + q[2] * GA[k]);
}

// second-order flux between two sides (face frame), per unit area:
//   W0 from the upwind half moments; side slopes; abar_d as above;
//   Abar from <(u abar_n + v abar_t1 + w abar_t2 + Abar) . psi psi> = 0;
//   F = rho0 [q1 <u psi> + q2 <u (u.abar) psi> + q3 <u Abar psi>]
//     + sum_s rho^h_s [(q4 - dt e) <u psi>_s + (q5 + dt^2 e/2) <u (u.a~_s) psi>_s]
// (Shakhov model: + q1 qsh in energy, as in flux_pair)
template <typename R>
__device__ void flux2_pair(const Side2<R> &L, const Side2<R> &Rs, R dt, R mu_ref, R omega, R c2, bool gks, R qsh,
                           R Ff[5]) {
    Mom3<R> ML, MR, M0;
    mom3<R>(1, L.g, ML);
    mom3<R>(-1, Rs.g, MR);
    Prim<R> z;
    face_state<R>(L, Rs, ML, MR, z);
    mom3<R>(0, z, M0);
    R abar[3][5];
    face_slope<0, R>(L, Rs, ML, MR, z, abar[0]);
    face_slope<1, R>(L, Rs, ML, MR, z, abar[1]);
    face_slope<2, R>(L, Rs, ML, MR, z, abar[2]);
    R q[5];
    face_q<R>(L, Rs, z, dt, mu_ref, omega, c2, gks, q);
    {
        R t[5], X[5], y[5], v[5];
        gaxis<0, R>(M0, abar[0], t);
        gaxis<1, R>(M0, abar[1], y);
        gaxis<2, R>(M0, abar[2], v);
#pragma unroll
        for (int k = 0; k < 5; ++k) t[k] = t[k] + y[k] + v[k];
        guaxis<0, R>(M0, abar[0], X);
        guaxis<1, R>(M0, abar[1], y);
        guaxis<2, R>(M0, abar[2], v);
#pragma unroll
        for (int k = 0; k < 5; ++k) X[k] = X[k] + y[k] + v[k];
        face_eq<R>(z, M0, t, X, q, Ff);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const Side2<R> &S = s == 0 ? L : Rs;
        if (!(S.h.rho > (R)0)) continue;
        Mom3<R> MH;
        mom3<R>(s == 0 ? 1 : -1, S.h, MH);
        R Gh[5], Y[5], acc[5];
        uvec<R>(MH, Gh);
        hydro_axis<0, R>(MH, S, acc);
        hydro_axis<1, R>(MH, S, Y);
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] += Y[k];
        hydro_axis<2, R>(MH, S, Y);
#pragma unroll
        for (int k = 0; k < 5; ++k) Ff[k] += S.h.rho * (q[3] * Gh[k] + q[4] * (acc[k] + Y[k]));
    }
    if (qsh != (R)0) Ff[4] = Ff[4] + q[0] * qsh;
}

// Gradients for second order, FP64 in both forms: the unweighted
// least-squares gradient over the face neighbours of the 5 components of W and of the hydro
// state (rho^h / rho) W; boundary ghosts at the centre mirrored in the face plane (specular:
// mirror state; diffuse: the cell's density and temperature, velocity reflected about the
// wall's; far field: the free stream); a limiter per component (Barth-Jespersen or
// Venkatakrishnan with eps^2 = (K h)^3, h = Omega^(1/3)); a cell whose limited face states are
// non-physical (rho <= 0, T <= 0, hydro density < 0 or hydro temperature <= 0) falls back to
// first order; a face hydro density within 1e-12 of the face density of zero counts as zero
// (roundoff of an empty hydro part, which the limiter can pin to a neighbour's zero).
// Bound by the latency of dependent loads and by its FP64 divisions (two a face and component in
// the limiter), not by its bytes.  Five waves have 64 cells, each one component of W and of the hydro
// state; what is a face's (the centres, the neighbour's hydro part, a ghost's state) a wave forms for
// one face and leaves in local memory for all, as the gradients for the face states.  With a thread
// per cell (ten components and their gradients in registers, one wave per SIMD) 32,768 boxes took
// 28.7 us, now 17.7; the 2,709 of a 301 x 3 x 3 tube 26 and 12.6; 262,144 boxes 120 and 109;
// 34,992 tetrahedra 27.7 and 20; 511,104 tetrahedra, which fill the chip either way, 180 and 184 (208
// when every wave formed every face's data).  Ten waves of one component each: 32 us on 32,768 boxes.
constexpr int kGradCells = kWave;

// NF: the faces of a cell at most (4: every cell a tetrahedron).
template <int NF>
__global__ void __launch_bounds__(5 * kGradCells) k_grad(Dev D) {
    __shared__ double sv[10][3][kGradCells];  // limited gradient by component (W, hydro)
    // by face: the neighbour's centre and the face's centre from the cell's, the neighbour's rho^h / rho
    // (a ghost: its state)
    __shared__ double sf[NF][11][kGradCells];
    __shared__ double se[kGradCells];  // eps^2
    __shared__ int sok[kGradCells];
    const int cl = lane_id(), kk = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nc = D.nc, c0 = blockIdx.x * kGradCells + cl;
    const bool in = c0 < nc;
    const int c = in ? c0 : nc - 1;
    const InstP &P = D.ip[inst_of(D, c)];
    const bool live = in && P.recon != 0;
    if (kk == 0) sok[cl] = 1;
    const int nfc = D.nfc[c];
    const double *lfx = D.lfx + (long long)c * 18;
    double Wc[5], g[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    int nb[NF];
    double vj[NF][2];
    // every neighbour's load before the first use
#pragma unroll
    for (int lf = 0; lf < NF; ++lf) nb[lf] = lf < nfc ? D.nbl[c * 6 + lf].x : c;
#pragma unroll
    for (int lf = 0; lf < NF; ++lf) vj[lf][0] = D.W[kk * nc + (nb[lf] >= 0 ? nb[lf] : c)];
#pragma unroll
    for (int i = 0; i < 5; ++i) Wc[i] = D.W[i * nc + c];
    const double fc = D.rhoh[c] / Wc[0];
    const double xc[3] = {D.xc[c], D.xc[nc + c], D.xc[2 * nc + c]};
    // component kk of a state in registers
    auto comp = [kk](const double v[5]) {
        return kk == 0 ? v[0] : kk == 1 ? v[1] : kk == 2 ? v[2] : kk == 3 ? v[3] : v[4];
    };
    double vc[2];
    vc[0] = comp(Wc);
    vc[1] = fc * vc[0];
    // the faces' data: a face a wave, the last of six to the first wave
    for (int lf = kk; lf < nfc && live; lf += 5) {
        const int j = D.nbl[c * 6 + lf].x;
        double xj[3];
        if (j >= 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) xj[d] = D.xc[d * nc + j];
            sf[lf][6][cl] = D.rhoh[j] / D.W[j];
        } else {
            const double4 pl = D.plane[c * 6 + lf];
            const double nn[3] = {pl.x, pl.y, pl.z};
            const double dist = pl.w - (nn[0] * xc[0] + nn[1] * xc[1] + nn[2] * xc[2]);
#pragma unroll
            for (int d = 0; d < 3; ++d) xj[d] = xc[d] + 2.0 * dist * nn[d];
            const DevBC &b = D.bc[-1 - j];
            if (b.type == 2) {
#pragma unroll
                for (int i = 0; i < 5; ++i) sf[lf][6 + i][cl] = b.Winf[i];
            } else {
                const double rho = Wc[0];
                const double U[3] = {Wc[1] / rho, Wc[2] / rho, Wc[3] / rho};
                const double T = temp_k(Wc, D.K);
                double Ug[3];
                if (b.type == 0) {
                    const double un = U[0] * nn[0] + U[1] * nn[1] + U[2] * nn[2];
#pragma unroll
                    for (int d = 0; d < 3; ++d) Ug[d] = U[d] - 2.0 * un * nn[d];
                } else {
#pragma unroll
                    for (int d = 0; d < 3; ++d) Ug[d] = 2.0 * b.Uw[d] - U[d];
                }
                sf[lf][6][cl] = rho;
#pragma unroll
                for (int d = 0; d < 3; ++d) sf[lf][7 + d][cl] = rho * Ug[d];
                sf[lf][10][cl] =
                    0.5 * rho * (Ug[0] * Ug[0] + Ug[1] * Ug[1] + Ug[2] * Ug[2]) + 0.5 * (3.0 + D.K) * rho * T;
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            sf[lf][d][cl] = xj[d] - xc[d];
            sf[lf][3 + d][cl] = lfx[3 * lf + d] - xc[d];
        }
    }
    if (kk == 4 && live && P.recon != 1) {
        const double kh = P.venkat_k * cbrt(D.vol[c]);
        se[cl] = kh * kh * kh;
    }
    __syncthreads();
    if (live) {
#pragma unroll
        for (int lf = 0; lf < NF; ++lf) {
            if (lf >= nfc) break;
            if (nb[lf] >= 0) {
                vj[lf][1] = sf[lf][6][cl] * vj[lf][0];
            } else {
                vj[lf][0] = sf[lf][6 + kk][cl];
                vj[lf][1] = D.bc[-1 - nb[lf]].type == 2 ? vj[lf][0] : fc * vj[lf][0];
            }
        }
        double A00 = 0, A01 = 0, A02 = 0, A11 = 0, A12 = 0, A22 = 0;
        double r[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}}, vmax[2] = {vc[0], vc[1]}, vmin[2] = {vc[0], vc[1]};
#pragma unroll
        for (int lf = 0; lf < NF; ++lf) {
            if (lf >= nfc) break;
            const double dx[3] = {sf[lf][0][cl], sf[lf][1][cl], sf[lf][2][cl]};
            A00 += dx[0] * dx[0];
            A01 += dx[0] * dx[1];
            A02 += dx[0] * dx[2];
            A11 += dx[1] * dx[1];
            A12 += dx[1] * dx[2];
            A22 += dx[2] * dx[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double dv = vj[lf][h] - vc[h];
                r[h][0] += dx[0] * dv;
                r[h][1] += dx[1] * dv;
                r[h][2] += dx[2] * dv;
                vmax[h] = fmax(vmax[h], vj[lf][h]);
                vmin[h] = fmin(vmin[h], vj[lf][h]);
            }
        }
        // inverse of the symmetric normal matrix by cofactors
        const double C00 = A11 * A22 - A12 * A12, C01 = A02 * A12 - A01 * A22, C02 = A01 * A12 - A02 * A11;
        const double C11 = A00 * A22 - A02 * A02, C12 = A02 * A01 - A00 * A12, C22 = A00 * A11 - A01 * A01;
        const double det = A00 * C00 + A01 * C01 + A02 * C02;
        const double eps2 = P.recon != 1 ? se[cl] : 0.0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            g[h][0] = (C00 * r[h][0] + C01 * r[h][1] + C02 * r[h][2]) / det;
            g[h][1] = (C01 * r[h][0] + C11 * r[h][1] + C12 * r[h][2]) / det;
            g[h][2] = (C02 * r[h][0] + C12 * r[h][1] + C22 * r[h][2]) / det;
        }
        double phi[2] = {1.0, 1.0};
        for (int lf = 0; lf < nfc; ++lf) {
            const double dx[3] = {sf[lf][3][cl], sf[lf][4][cl], sf[lf][5][cl]};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double Dk = g[h][0] * dx[0] + g[h][1] * dx[1] + g[h][2] * dx[2];
                double pf = 1.0;
                if (Dk != 0.0) {
                    const double M = Dk > 0.0 ? vmax[h] - vc[h] : vmin[h] - vc[h];
                    if (P.recon == 1)
                        pf = fmin(1.0, M / Dk);
                    else
                        pf = ((M * M + eps2) * Dk + 2.0 * Dk * Dk * M) /
                             (Dk * (M * M + 2.0 * Dk * Dk + M * Dk + eps2));
                }
                phi[h] = fmin(phi[h], pf);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int d = 0; d < 3; ++d) g[h][d] *= phi[h];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int d = 0; d < 3; ++d) sv[5 * h + kk][d][cl] = g[h][d];
    __syncthreads();
    // the states extrapolated to the faces: one face a wave, the last of six to the first wave
    for (int lf = kk; lf < nfc && live; lf += 5) {
        const double dx[3] = {sf[lf][3][cl], sf[lf][4][cl], sf[lf][5][cl]};
        double wf[10];
#pragma unroll
        for (int i = 0; i < 10; ++i)
            wf[i] = (i < 5 ? Wc[i] : fc * Wc[i - 5]) + sv[i][0][cl] * dx[0] + sv[i][1][cl] * dx[1] + sv[i][2][cl] * dx[2];
        bool ok = wf[0] > 0.0 && temp_k(wf, D.K) > 0.0 && wf[5] >= -1e-12 * wf[0];
        if (wf[5] > 1e-12 * wf[0] && !(temp_k(wf + 5, D.K) > 0.0)) ok = false;
        if (!ok) atomicAnd(&sok[cl], 0);
    }
    __syncthreads();
    if (!live) return;
    const bool ok = sok[cl] != 0;
    D.Wh[kk * nc + c] = vc[1];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        D.gW[(3 * kk + d) * nc + c] = ok ? g[0][d] : 0.0;
        D.gH[(3 * kk + d) * nc + c] = ok ? g[1][d] : 0.0;
    }
}

// a cell's state (and hydro state) extrapolated to point x, FP64
__device__ __forceinline__ void extrap(const Dev &D, int c, const double x[3], double W[5], double Wh[5]) {
    const int nc = D.nc;
    const double dx[3] = {x[0] - D.xc[c], x[1] - D.xc[nc + c], x[2] - D.xc[2 * nc + c]};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        W[k] = D.W[k * nc + c] + D.gW[(3 * k) * nc + c] * dx[0] + D.gW[(3 * k + 1) * nc + c] * dx[1] +
               D.gW[(3 * k + 2) * nc + c] * dx[2];
        Wh[k] = D.Wh[k * nc + c] + D.gH[(3 * k) * nc + c] * dx[0] + D.gH[(3 * k + 1) * nc + c] * dx[1] +
                D.gH[(3 * k + 2) * nc + c] * dx[2];
    }
}

// one face at second order: its frame and its two sides' states
template <typename R>
struct Face2 {
    int f, c, nb, type;  // type: the boundary condition's (nb < 0)
    bool pair;           // two sides (an inner face, a mirror, the free stream); else a diffuse wall
    R n[3], t1[3], t2[3];
    R dt;
    bool gks;
    Side2<R> L, Rs;
    double Whl0, Wl0;
};
// the outer side's derivatives at a boundary (specular walls mirror the inner ones: along n and the
// normal momentum flip; the free stream has none)
template <typename R>
__device__ __forceinline__ void mirror_derivs(Face2<R> &F) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const R sg = ((d == 0) != (k == 1)) ? (R)-1 : (R)1;
            F.Rs.dW[d][k] = F.type == 0 ? sg * F.L.dW[d][k] : (R)0;
            F.Rs.dWh[d][k] = F.type == 0 ? sg * F.L.dWh[d][k] : (R)0;
        }
}
// DERIVS: with both sides' derivatives, each side's loaded with its state.  A thread that has a face
// to itself runs at one wave per SIMD, where a second round of loads after the states is not hidden:
// 101,376 faces FP64 53 us with it, 47 without; 1,033,824 faces of tetrahedra 509 and 421.
template <typename R, bool DERIVS>
__device__ __forceinline__ bool open_face(const Dev &D, int f, Face2<R> &F) {
    const int nf = D.nf;
    F.f = f;
    F.c = D.fown[f];
    const int inst = inst_of(D, F.c);
    const InstP &P = D.ip[inst];
    if (P.recon == 0) return false;
    F.dt = (R)D.is[inst].dt;
    F.gks = D.is[inst].step < P.gks_steps;
    F.nb = D.fnb[f];
    F.type = F.nb >= 0 ? -1 : D.bc[-1 - F.nb].type;
    F.pair = F.type != 1;
    F.n[0] = (R)D.fn[f];
    F.n[1] = (R)D.fn[nf + f];
    F.n[2] = (R)D.fn[2 * nf + f];
    face_frame<R>(F.n, F.t1, F.t2);
    const double xf[3] = {D.fx[f], D.fx[nf + f], D.fx[2 * nf + f]};
    auto side = [&](int c, Side2<R> &S, double &w0, double &wh0) {
        double W[5], Wh[5];
        extrap(D, c, xf, W, Wh);
        w0 = W[0];
        wh0 = Wh[0];
        S.g = to_frame<R>(W, F.n, F.t1, F.t2, D.K);
        if (DERIVS) frame_derivs<R>(D.gW, D.nc, c, F.n, F.t1, F.t2, S.dW);
        // a face hydro density at or below 1e-12 of the face density is roundoff of an empty hydro
        // part (the limiter can pin it exactly to a neighbour's zero): no hydro wave on that side
        if (Wh[0] > 1e-12 * W[0]) {
            S.h = to_frame<R>(Wh, F.n, F.t1, F.t2, D.K);
            if (DERIVS) frame_derivs<R>(D.gH, D.nc, c, F.n, F.t1, F.t2, S.dWh);
        } else {
            S.h.rho = (R)0;
            S.h.K = D.K;
        }
    };
    side(F.c, F.L, F.Wl0, F.Whl0);
    if (F.nb >= 0) {
        double a, b;
        side(F.nb, F.Rs, a, b);
    } else if (F.type == 0) {
        F.Rs.g = F.L.g;
        F.Rs.h = F.L.h;
        F.Rs.g.un = -F.L.g.un;
        F.Rs.h.un = -F.L.h.un;
    } else if (F.type == 2) {
        F.Rs.g = to_frame<R>(D.bc[-1 - F.nb].Winf, F.n, F.t1, F.t2, D.K);
        F.Rs.h = F.Rs.g;
    }
    if (DERIVS && F.nb < 0) mirror_derivs<R>(F);
    return true;
}
// both sides' derivatives along the frame's axes
template <typename R>
__device__ __forceinline__ void face_derivs(const Dev &D, Face2<R> &F) {
    frame_derivs<R>(D.gW, D.nc, F.c, F.n, F.t1, F.t2, F.L.dW);
    if (F.L.h.rho > (R)0) frame_derivs<R>(D.gH, D.nc, F.c, F.n, F.t1, F.t2, F.L.dWh);
    if (F.nb >= 0) {
        frame_derivs<R>(D.gW, D.nc, F.nb, F.n, F.t1, F.t2, F.Rs.dW);
        if (F.Rs.h.rho > (R)0) frame_derivs<R>(D.gH, D.nc, F.nb, F.n, F.t1, F.t2, F.Rs.dWh);
    } else {
        mirror_derivs<R>(F);
    }
}
// the face's flux, times its area, oriented owner -> neighbour
template <typename R>
__device__ __forceinline__ void close_face(const Dev &D, const Face2<R> &F, R Ff[5]) {
    const int nf = D.nf, f = F.f;
    if (F.type == 0) {
        Ff[0] = (R)0;
        Ff[2] = (R)0;
        Ff[3] = (R)0;
        Ff[4] = (R)0;
    }
    const R a = (R)D.farea[f];
    D.Phi[f] = (double)(Ff[0] * a);
#pragma unroll
    for (int d = 0; d < 3; ++d)
        D.Phi[(1 + d) * nf + f] = (double)((Ff[1] * F.n[d] + Ff[2] * F.t1[d] + Ff[3] * F.t2[d]) * a);
    D.Phi[4 * nf + f] = (double)(Ff[4] * a);
}
template <typename R>
__device__ __forceinline__ void wall_flux2(const Dev &D, const Face2<R> &F, R Ff[5]) {
    diffuse_flux<R>(F.L.g, (R)(F.Whl0 > 1e-12 * F.Wl0 ? F.Whl0 : 0.0), (R)D.tau[F.c], F.n, F.t1, F.t2, D.bc[-1 - F.nb],
                    F.dt, F.gks, Ff);
}

// S2 at second order: per face, states extrapolated to the face centre from both sides
// (limited gradients), the flux of flux2_pair; specular walls mirror the reconstructed field
// (derivatives along n and the normal momentum flip), diffuse walls stay first order at the
// reconstructed face state, far-field faces see the free stream with zero gradients.
template <typename R, int BS>
__global__ void __launch_bounds__(BS) k_flux2(Dev D) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= D.nf) return;
    Face2<R> F;
    if (!open_face<R, true>(D, f, F)) return;
    const InstP &P = D.ip[inst_of(D, F.c)];
    R Ff[5];
    if (F.pair) {
        const R qsh = F.type == 0 ? (R)0 : (R)shakhov_qsh(D, P, f, F.c, F.nb);
        flux2_pair<R>(F.L, F.Rs, F.dt, (R)P.mu_ref, (R)P.omega, (R)P.c2, F.gks, qsh, Ff);
    } else {
        wall_flux2<R>(D, F, Ff);
    }
    close_face<R>(D, F, Ff);
}

// The same for a mesh of few faces, whose waves do not fill the chip: a face is a chain of some
// 7,000 dependent operations, so three waves share 64 faces, one per axis of the face frame.  Each
// forms the states and the sums of its axis and hands them over in local memory; the second also
// has the time coefficients, the first joins the axes in the order of flux2_pair (the same bits).
// It saves a microsecond or two while a block has a CU to itself and a SIMD to each wave, and costs a
// second round beyond.  Microseconds for gradients and fluxes with it and without, FP64 (FP32): 3,300
// faces of boxes 36.2, 37.2 (29.5, 32.7); 9,331 of a 301 x 3 x 3 tube 35.5, 36.0 (30.6, 32.0); 13,056:
// 35.2, 34.7 (30.0, 31.3), where a step with particles is no longer shorter (140, 140; 127, 125);
// 18,468: 51.8, 37.4 (38.9, 33.0).
constexpr int kFluxSplitMax = 10240;
template <typename R>
struct AxisPart {
    R T[5], X[5], Y[2][5];
};
template <int A, typename R>
__device__ __forceinline__ void axis_part(const Dev &D, Face2<R> &F, const Mom3<R> &ML, const Mom3<R> &MR,
                                          const Prim<R> &z, const Mom3<R> &M0, AxisPart<R> &p) {
    face_derivs<R>(D, F);
    R abar[5];
    face_slope<A, R>(F.L, F.Rs, ML, MR, z, abar);
    gaxis<A, R>(M0, abar, p.T);
    guaxis<A, R>(M0, abar, p.X);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const Side2<R> &S = s == 0 ? F.L : F.Rs;
#pragma unroll
        for (int k = 0; k < 5; ++k) p.Y[s][k] = (R)0;
        if (!(S.h.rho > (R)0)) continue;
        Mom3<R> MH;
        mom3<R>(s == 0 ? 1 : -1, S.h, MH);
        hydro_axis<A, R>(MH, S, p.Y[s]);
    }
}
template <typename R>
__global__ void __launch_bounds__(3 * kWave) k_flux2_axes(Dev D) {
    __shared__ R part[2][20][kWave];
    __shared__ R qs[5][kWave];
    const int axis = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
    const int f = blockIdx.x * kWave + lane;
    Face2<R> F;
    Prim<R> z;
    Mom3<R> M0;
    AxisPart<R> p;
    const bool live = f < D.nf && open_face<R, false>(D, f, F);
    if (live && F.pair) {
        Mom3<R> ML, MR;
        mom3<R>(1, F.L.g, ML);
        mom3<R>(-1, F.Rs.g, MR);
        face_state<R>(F.L, F.Rs, ML, MR, z);
        mom3<R>(0, z, M0);
        if (axis == 0)
            axis_part<0, R>(D, F, ML, MR, z, M0, p);
        else if (axis == 1)
            axis_part<1, R>(D, F, ML, MR, z, M0, p);
        else
            axis_part<2, R>(D, F, ML, MR, z, M0, p);
        if (axis > 0) {
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                part[axis - 1][k][lane] = p.T[k];
                part[axis - 1][5 + k][lane] = p.X[k];
                part[axis - 1][10 + k][lane] = p.Y[0][k];
                part[axis - 1][15 + k][lane] = p.Y[1][k];
            }
        }
        if (axis == 1) {
            const InstP &P = D.ip[inst_of(D, F.c)];
            R q[5];
            face_q<R>(F.L, F.Rs, z, F.dt, (R)P.mu_ref, (R)P.omega, (R)P.c2, F.gks, q);
#pragma unroll
            for (int k = 0; k < 5; ++k) qs[k][lane] = q[k];
        }
    }
    __syncthreads();
    if (axis != 0 || !live) return;
    R Ff[5];
    if (F.pair) {
        R q[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) q[k] = qs[k][lane];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                p.T[k] = p.T[k] + part[a][k][lane];
                p.X[k] = p.X[k] + part[a][5 + k][lane];
                p.Y[0][k] = p.Y[0][k] + part[a][10 + k][lane];
                p.Y[1][k] = p.Y[1][k] + part[a][15 + k][lane];
            }
        face_eq<R>(z, M0, p.T, p.X, q, Ff);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const Side2<R> &S = s == 0 ? F.L : F.Rs;
            if (!(S.h.rho > (R)0)) continue;
            Mom3<R> MH;
            mom3<R>(s == 0 ? 1 : -1, S.h, MH);
            R Gh[5];
            uvec<R>(MH, Gh);
#pragma unroll
            for (int k = 0; k < 5; ++k) Ff[k] += S.h.rho * (q[3] * Gh[k] + q[4] * p.Y[s][k]);
        }
        const R qsh = F.type == 0 ? (R)0 : (R)shakhov_qsh(D, D.ip[inst_of(D, F.c)], f, F.c, F.nb);
        if (qsh != (R)0) Ff[4] = Ff[4] + q[0] * qsh;
    } else {
        wall_flux2<R>(D, F, Ff);
    }
    close_face<R>(D, F, Ff);
}

// particle store access for the two forms
__device__ __forceinline__ void store_new(const Particles &pa, long long i, const double x[3], const double u[3],
                                          double m, uint64_t uid) {
    double2 *r = reinterpret_cast<double2 *>(pa.rec + i);
    r[0] = make_double2(x[0], x[1]);
    r[1] = make_double2(x[2], u[0]);
    r[2] = make_double2(u[1], u[2]);
    r[3] = make_double2(m, __longlong_as_double((long long)uid));
}
__device__ __forceinline__ void store_new(const Particles &pa, long long i, const float x[3], const float u[3],
                                          float m, uint64_t uid) {
    float4 *r = reinterpret_cast<float4 *>(pa.rec32 + i);
    r[0] = make_float4(x[0], x[1], x[2], u[0]);
    r[1] = make_float4(u[1], u[2], __uint_as_float((uint32_t)uid), __uint_as_float((uint32_t)(uid >> 32)));
    pa.m32[i] = m;
}

// phi = m (1, u, |u|^2 / 2) of a stored particle, accumulated in FP64
template <typename R>
__device__ __forceinline__ void add_phi(double acc[5], R m_, const R u_[3], R e_ = (R)0) {
    const double m = (double)m_, u0 = (double)u_[0], u1 = (double)u_[1], u2 = (double)u_[2], e = (double)e_;
    acc[0] += m;
    acc[1] += m * u0;
    acc[2] += m * u1;
    acc[3] += m * u2;
    acc[4] += m * (0.5 * (u0 * u0 + u1 * u1 + u2 * u2 + e));
}

// internal energy variable e = T |X|^2 of a particle in equilibrium at temperature T: the first K
// of the standard normals that Box-Muller makes of the draws (seed, uid, step, tag, sub0 + j,
// inst), j = 0, 1 (four per draw)
template <typename R>
__device__ __forceinline__ R internal_energy(uint64_t seed, uint64_t uid, long long step, int tag, uint32_t sub0,
                                             int inst, int K, R T) {
    const R two_pi = (R)2 * (R)kPi;
    R acc = (R)0;
    for (int j = 0; 4 * j < K; ++j) {
        const U4 r = draw(seed, uid, step, tag, sub0 + (uint32_t)j, inst);
        const R r1 = sqrt((R)-2 * log(unif<R>(r.v[0]))), r2 = sqrt((R)-2 * log(unif<R>(r.v[2])));
        const R a1 = two_pi * unif<R>(r.v[1]), a2 = two_pi * unif<R>(r.v[3]);
        const R X[4] = {r1 * cos(a1), r1 * sin(a1), r2 * cos(a2), r2 * sin(a2)};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * j + i < K) acc = acc + X[i] * X[i];
    }
    return T * acc;
}
__device__ __forceinline__ void store_e(const Particles &pa, long long i, double e) { pa.e64[i] = e; }
__device__ __forceinline__ void store_e(const Particles &pa, long long i, float e) { pa.e32[i] = e; }

// Shakhov model: raw moments sum m u_i |u|^2 and sum m u_i u_j of a cell's particles, from which
// the cell's heat flux q = (1/Omega) sum m c |c|^2 / 2 with c = u - U follows by expanding c
__device__ __forceinline__ void add_heat(double m, double u0, double u1, double u2, double H[9]) {
    const double w = m * (u0 * u0 + u1 * u1 + u2 * u2);
    H[0] += w * u0;
    H[1] += w * u1;
    H[2] += w * u2;
    H[3] += m * u0 * u0;
    H[4] += m * u0 * u1;
    H[5] += m * u0 * u2;
    H[6] += m * u1 * u1;
    H[7] += m * u1 * u2;
    H[8] += m * u2 * u2;
}
// q of one cell from its survivors' raw moments H (summed as above, then over the wave), its
// P^{n+1} and W^{n+1}: lane i < 3 returns component i,
//   sum m c_i |c|^2 = S3_i - 2 sum_j U_j S2_ij - U_i tr S2 + |U|^2 S1_i + 2 U_i (U . S1) - U_i |U|^2 S0
__device__ __forceinline__ double heat_of(const double H[9], const double Wn[5], const double Pv[5], double vol) {
    const int lane = lane_id();
    const double U[3] = {Wn[1] / Wn[0], Wn[2] / Wn[0], Wn[3] / Wn[0]};
    const double tr = H[3] + H[6] + H[8];
    const double uu = U[0] * U[0] + U[1] * U[1] + U[2] * U[2];
    const double us1 = U[0] * Pv[1] + U[1] * Pv[2] + U[2] * Pv[3];
    // lane i takes component i (selects, not register-array indexing)
    const double r0 = H[3] * U[0] + H[4] * U[1] + H[5] * U[2];
    const double r1 = H[4] * U[0] + H[6] * U[1] + H[7] * U[2];
    const double r2 = H[5] * U[0] + H[7] * U[1] + H[8] * U[2];
    const double s2u = lane == 0 ? r0 : (lane == 1 ? r1 : r2);
    const double s3 = lane == 0 ? H[0] : (lane == 1 ? H[1] : H[2]);
    const double s1 = lane == 0 ? Pv[1] : (lane == 1 ? Pv[2] : Pv[3]);
    const double ui = lane == 0 ? U[0] : (lane == 1 ? U[1] : U[2]);
    const double t = s3 - 2.0 * s2u - ui * tr + uu * s1 + 2.0 * ui * us1 - ui * uu * Pv[0];
    return 0.5 * t / vol;
}

// ---------------------------------------------------------------------------------------
// Shakhov model: the heat flux of the gas in each cell at the start of the step,
//   q = (1/Omega) sum_k m_k c_k |c_k|^2 / 2,  c_k = u_k - U,  U = (W_1, W_2, W_3) / W_0,
// over the particles the cell holds (the hydro part, a Maxwellian at the cell's U and T,
// carries none), from the raw moments sum m u_i |u|^2 and sum m u_i u_j: lane l sums the cell's
// particles l + 64 k in increasing k, arrivals first, so the bits do not depend on where the
// particles lie (a state that was exported and imported gives the same ones).  One wave per
// cell, at the end of every step and after the state is set.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void load_um(const Particles &pa, long long i, double u[3], double &m, double) {
    const double2 *r = reinterpret_cast<const double2 *>(pa.rec + i);
    const double2 a = r[1], b = r[2], t = r[3];
    u[0] = a.y;
    u[1] = b.x;
    u[2] = b.y;
    m = t.x;
}
__device__ __forceinline__ void load_um(const Particles &pa, long long i, double u[3], double &m, float) {
    const float4 *r = reinterpret_cast<const float4 *>(pa.rec32 + i);
    const float4 a = r[0], b = r[1];
    u[0] = (double)a.w;
    u[1] = (double)b.x;
    u[2] = (double)b.y;
    m = (double)pa.m32[i];
}

template <typename R>
__global__ void __launch_bounds__(256) k_heat(Dev D, int buf) {
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int c = blockIdx.x * 4 + wave;
    if (c >= D.nc) return;
    const int nc = D.nc;
    const bool sh = D.ip[inst_of(D, c)].pr != 1.0;
    double H[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (sh) {
        const unsigned long long o0 = D.off[c], o1 = D.off[c + 1];
        const int n = hi32(o1) - hi32(o0), nm = lo32(o1) - lo32(o0), m0 = lo32(o0), v0 = D.v0[buf][c];
        const long long span = D.sc->span[buf];
        const Particles pa = D.pa[buf];
        for (int k = lane; k < n; k += kWave) {
            double u[3], m;
            load_um(pa, k < nm ? slot_of(D, buf, span, m0 + k) : v0 + (k - nm), u, m, R(0));
            add_heat(m, u[0], u[1], u[2], H);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) H[k] = wave_sum(H[k]);
    }
    double Wn[5], Pv[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        Wn[k] = D.W[k * nc + c];
        Pv[k] = D.P[k * nc + c];
    }
    if (lane < 3) D.qh[lane * nc + c] = sh ? heat_of(H, Wn, Pv, D.vol[c]) : 0.0;
}

// ---------------------------------------------------------------------------------------
// S3: hydro particles in pairs (2p, 2p+1), a lane per pair.  A pair shares X ~ N(0, I) from
// Box-Muller on the draw keyed by the even partner's id: X0, X1 = r1 (cos, sin)(2 pi e1), r1 =
// sqrt(-2 ln e0), and X2 = r2 cos(2 pi e3), r2 = sqrt(-2 ln e2).  Partners get U + sqrt(T) X and
// U - sqrt(T) X, the pair of Sec. 2.4(b), and their own uniform position (box: per axis;
// tetrahedron: Rocchini-Cignoni folding of the unit cube).  With the energy-exact variant
// (sampling = 1, a departure from the paper) the deviations carry one factor s per cell,
// s = sqrt(3 N_pairs / sum_j |X_j|^2): a first pass sums |X|^2 for s.
// S = P + sum of phi over the new particles (fixed order over the cell's lanes).
// ---------------------------------------------------------------------------------------
// sine and cosine from one reduction of the argument (the same bits as the two calls)
__device__ __forceinline__ void sin_cos(double a, double &s, double &c) { sincos(a, &s, &c); }
__device__ __forceinline__ void sin_cos(float a, float &s, float &c) { sincosf(a, &s, &c); }

// a pair's X ~ N(0, I) by Box-Muller on the draw keyed by the even partner's id
template <typename R>
__device__ __forceinline__ void pair_normal(uint64_t seed, uint64_t puid, long long step, int inst, R X[3]) {
    const R two_pi = (R)2 * (R)kPi;
    const U4 rv = draw(seed, puid, step, kTagVel, 0, inst);
    const R r1 = sqrt((R)-2 * log(unif<R>(rv.v[0]))), r2 = sqrt((R)-2 * log(unif<R>(rv.v[2])));
    R sn, cs;
    sin_cos(two_pi * unif<R>(rv.v[1]), sn, cs);
    X[0] = r1 * cs;
    X[1] = r1 * sn;
    X[2] = r2 * cos(two_pi * unif<R>(rv.v[3]));
}
// a uniform point of a cell from the draw (uid, step, kTagPos): per axis in a box, the unit cube
// folded onto the tetrahedron (Rocchini-Cignoni) in a tetrahedron; org + s e1 + t e2 + w e3
template <typename R>
__device__ __forceinline__ void cell_point(uint64_t seed, uint64_t uid, long long step, int inst, const R org[3],
                                           const R Ed[9], bool tet, R x[3]) {
    const R one = (R)1;
    U4 rp = draw(seed, uid, step, kTagPos, 0, inst);
    R s = unif<R>(rp.v[0]), t = unif<R>(rp.v[1]), w = unif<R>(rp.v[2]);
    if (tet) {
        if (s + t > one) {
            s = one - s;
            t = one - t;
        }
        if (t + w > one) {
            R tmp = w;
            w = one - s - t;
            t = one - tmp;
        } else if (s + t + w > one) {
            R tmp = w;
            w = s + t + w - one;
            s = one - t - tmp;
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = org[d] + s * Ed[d] + t * Ed[3 + d] + w * Ed[6 + d];
}

template <typename R>
__device__ __forceinline__ void sample_state(const Dev &D, int c, R U[3], R &T) {
    const int nc = D.nc;
    const double rho = D.W[c], m0 = D.W[nc + c], m1 = D.W[2 * nc + c], m2 = D.W[3 * nc + c], E = D.W[4 * nc + c];
    U[0] = (R)(m0 / rho);
    U[1] = (R)(m1 / rho);
    U[2] = (R)(m2 / rho);
    T = (R)((2.0 / (3.0 + D.K)) * (E - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) / rho) / rho);
}
template <typename R>
__device__ __forceinline__ void sample_geometry(const Dev &D, int c, int ns, R &msam, R org[3], R Ed[9], bool &tet) {
    const int nc = D.nc;
    msam = (R)(D.ec[c] * D.rhoh[c] * D.vol[c] / (double)ns);
#pragma unroll
    for (int q = 0; q < 3; ++q) org[q] = (R)D.orig[q * nc + c];
#pragma unroll
    for (int q = 0; q < 9; ++q) Ed[q] = (R)D.edge[q * nc + c];
    tet = D.ctype[c] == 4;
}
// the two particles of a pair: U + sT X and U - sT X, each at its own point with its internal energy
// e; their sums
template <typename R, bool KE>
__device__ __forceinline__ void put_pair(const Dev &D, const Particles &pa, int buf, long long span, long long place,
                                         uint64_t seed, long long step, int inst, int cl, int k, const R U[3], R sT,
                                         const R X[3], const R e2[2], R msam, const R org[3], const R Ed[9],
                                         bool tet, double acc[5]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint64_t uid = make_uid(step, cl, k + q);
        const long long i = slot_of(D, buf, span, place + q);
        R u[3], x[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) u[d] = q == 0 ? U[d] + sT * X[d] : U[d] - sT * X[d];
        cell_point<R>(seed, uid, step, inst, org, Ed, tet, x);
        store_new(pa, i, x, u, msam, uid);
        R e = (R)0;
        if (KE) {
            e = e2[q];
            store_e(pa, i, e);
        }
        add_phi<R>(acc, msam, u, e);
    }
}
// |X'|^2 of both particles' internal components
template <typename R>
__device__ __forceinline__ void pair_internal(uint64_t seed, long long step, int inst, int cl, int k, int K, R xi2[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) xi2[q] = internal_energy<R>(seed, make_uid(step, cl, k + q), step, kTagInt, 0, inst, K, (R)1);
}

// one cell's ns > 0 new particles by the whole wave, 64 pairs at a time, and its S (c and ns are
// the wave's: the cell's data and the first rounds of the draws stay scalar)
template <typename R, bool KE>
__device__ __forceinline__ void sample_cell(const Dev &D, int buf, int c, int ns) {
    const int lane = lane_id();
    const int nc = D.nc, np = ns / 2;
    const Scalars *sc = D.sc;
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    {
        const Particles pa = D.pa[buf];
        const long long span = sc->span[buf], base = sc->n_mov + D.samoff[c];
        const int inst = __builtin_amdgcn_readfirstlane(inst_of(D, c));
        const InstP &P = D.ip[inst];
        const long long step = uniform64(D.is[inst].step);
        const unsigned long long seed = (unsigned long long)uniform64((long long)P.seed);
        const int cl = __builtin_amdgcn_readfirstlane(c - P.cell0);  // ids carry the cell index within the instance
        const bool exact = P.sampling == 1;
        R U[3], T;
        sample_state<R>(D, c, U, T);
        R sT = sqrt(T), fint = (R)1;
        // this lane's first pair's normal and internal components (energy-exact pass)
        R F[3] = {(R)0, (R)0, (R)0}, Fi[2] = {(R)0, (R)0};
        if (exact) {
            // energy-exact pairs: the pairs carry the momentum exactly; one factor on every thermal
            // deviation of the cell, sqrt(3 N_pairs / sum_j |X_j|^2), makes the energy exact too (a
            // first pass over the pairs' normal draws, summed in FP64); with internal degrees of
            // freedom one factor K N_sam / sum_k |X'_k|^2 on every internal energy as well
            double sx2 = 0.0, se = 0.0;
            for (int p = lane; p < np; p += kWave) {
                R X[3];
                pair_normal<R>(seed, make_uid(step, cl, 2 * p), step, inst, X);
                if (p == lane) {
                    F[0] = X[0];
                    F[1] = X[1];
                    F[2] = X[2];
                }
                const double x0 = (double)X[0], x1 = (double)X[1], x2 = (double)X[2];
                sx2 += x0 * x0 + x1 * x1 + x2 * x2;
                if (KE) {
                    R xi2[2];
                    pair_internal<R>(seed, step, inst, cl, 2 * p, D.K, xi2);
                    if (p == lane) {
                        Fi[0] = xi2[0];
                        Fi[1] = xi2[1];
                    }
                    se += (double)xi2[0] + (double)xi2[1];
                }
            }
            sx2 = wave_sum(sx2);
            sT = (R)((double)sT * sqrt(3.0 * (double)np / sx2));
            if (KE) fint = (R)((double)D.K * (double)ns / wave_sum(se));
        }
        R msam, org[3], Ed[9];
        bool tet;
        sample_geometry<R>(D, c, ns, msam, org, Ed, tet);
        for (int p0 = 0; p0 < np; p0 += kWave) {
            const int p = p0 + lane;
            if (p >= np) continue;
            R X[3] = {F[0], F[1], F[2]}, e2[2] = {Fi[0], Fi[1]};
            if (p0 > 0 || !exact) {
                pair_normal<R>(seed, make_uid(step, cl, 2 * p), step, inst, X);
                if (KE) pair_internal<R>(seed, step, inst, cl, 2 * p, D.K, e2);
            }
            e2[0] = T * e2[0];
            e2[1] = T * e2[1];
            if (exact) {
                e2[0] = e2[0] * fint;
                e2[1] = e2[1] * fint;
            }
            put_pair<R, KE>(D, pa, buf, span, base + 2 * p, seed, step, inst, cl, 2 * p, U, sT, X, e2, msam, org, Ed, tet,
                            acc);
        }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k] = wave_sum(acc[k]);
    double ak = acc[0];
#pragma unroll
    for (int k = 1; k < 5; ++k)
        if (lane == k) ak = acc[k];
    if (lane < 5) D.S[lane * nc + c] = D.P[lane * nc + c] + ak;
}

// segmented sum over consecutive lanes: lane l of the segment [first, last] receives the sum of
// v over the segment (fixed order: an inclusive scan by doubling offsets, read at `last`)
__device__ __forceinline__ double seg_sum(double v, int first, int last) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const double t = __shfl_up(v, (unsigned)o);
        if (lane - o >= first) v = v + t;
    }
    return __shfl(v, last);
}

// Each wave takes G consecutive cells: runs of consecutive cells whose new pairs fit in 64 lanes
// together are sampled at once, a pair per lane in cell order (most cells sample a few
// particles: one wave per cell left most lanes idle).  G = 8 on meshes of 32768 cells or more; a
// smaller mesh would leave most of the chip idle with a wave per 8 cells, and takes G = 1.  A cell
// with more than 64 pairs is k_sample_big's.  The energy-exact factor and S come from segmented
// sums over the cell's lanes.  What bounds it: the vector ALU (Philox, logarithms, sines), so a lane
// takes a whole pair: the pair's draw and its two logarithms and angles are evaluated once
// instead of by both partners.
template <typename R, int WPB, bool KE, int G>
__global__ void __launch_bounds__(WPB * 64) __attribute__((amdgpu_waves_per_eu(3))) k_sample(Dev D, int buf) {
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int c0 = (blockIdx.x * WPB + wave) * G;
    const Scalars *sc = D.sc;
    if (c0 >= D.nc || sc->none) return;
    const int nc = D.nc;
    // new particles of the group's cells; -1 marks a lane without a cell of its own (past the
    // mesh) and a cell of an instance that samples one by one (k_sample_gp's, which also writes
    // its S): neither is sampled nor has S written here
    int myns = -1;
    if (lane < G && c0 + lane < nc) {
        const int c = c0 + lane;
        if (D.gp_any && D.ip[inst_of(D, c)].sampling >= 2)
            myns = -1;
        else
            myns = sc->n_new > 0 ? (int)D.nsam[c] : 0;  // even, at most 2^20
    }
    // wave-uniform pair counts and prefixes (scalar registers)
    int np[G];
    int pre[G + 1];
    pre[0] = 0;
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int n = __builtin_amdgcn_readlane(myns, j);
        np[j] = n > 0 ? n / 2 : n;
        pre[j + 1] = pre[j] + (n <= 0 ? 0 : (np[j] <= kWave ? np[j] : kWave + 1));
    }
    // cells without new particles: S = P (the five loads issued before the first store)
    if (lane < G && myns == 0) {
        const int c = c0 + lane;
        double pv[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) pv[k] = D.P[k * nc + c];
#pragma unroll
        for (int k = 0; k < 5; ++k) D.S[k * nc + c] = pv[k] + 0.0;
    }
    // cells with more than 64 pairs go to k_sample_big's list (one atomic per wave)
    {
        const bool big = lane < G && myns > 2 * kWave;
        const unsigned long long mb = __ballot(big);
        if (mb) {
            const int first = __ffsll((long long)mb) - 1;
            unsigned int at = 0;
            if (lane == first) at = atomicAdd(&D.sc->n_big, (unsigned int)__popcll(mb));
            at = __shfl(at, first);
            const unsigned long long below = lane == 0 ? 0ULL : (~0ULL >> (64 - lane));
            if (big) D.big[at + __popcll(mb & below)] = c0 + lane;
        }
    }
    int g = 0;
    while (g < G) {
        if (c0 + g >= nc) break;
        // wave-uniform: the longest run [g, h) of cells whose pairs fit in 64 lanes
        int h = g + 1, pg = 0, ph = 0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (j == g) {
                pg = pre[j];
                ph = pre[j + 1];
            }
            if (j == h && j > g && c0 + j < nc && pre[j + 1] - pg <= kWave) {
                h = j + 1;
                ph = pre[j + 1];
            }
        }
        const int nrun = ph - pg;
        if (nrun > 0 && nrun <= kWave) {
            // this lane's cell j of the run and its pair p there
            int j = g, first = lane, last = lane, npj = 0;
#pragma unroll
            for (int i = 0; i < G; ++i)
                if (i >= g && i < h && pre[i] - pg <= lane && pre[i + 1] - pg > lane) {
                    j = i;
                    first = pre[i] - pg;
                    last = pre[i + 1] - pg - 1;
                    npj = np[i];
                }
            const bool act = lane < nrun;
            const int k = 2 * (lane - first);  // its even partner's number
            const int c = c0 + j;
            double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
            const Particles pa = D.pa[buf];
            const int inst = inst_of(D, c);
            const InstP &P = D.ip[inst];
            const long long step = D.is[inst].step;
            const unsigned long long seed = P.seed;
            const int cl = c - P.cell0;
            const bool exact = P.sampling == 1;
            R U[3] = {(R)0, (R)0, (R)0}, X[3] = {(R)0, (R)0, (R)0}, e2[2] = {(R)0, (R)0}, sT = (R)0, T = (R)0;
            double sx2 = 0.0, se = 0.0;
            if (act) {
                sample_state<R>(D, c, U, T);
                sT = sqrt(T);
                pair_normal<R>(seed, make_uid(step, cl, k), step, inst, X);
                const double x0 = (double)X[0], x1 = (double)X[1], x2 = (double)X[2];
                sx2 = x0 * x0 + x1 * x1 + x2 * x2;
                if (KE) {
                    pair_internal<R>(seed, step, inst, cl, k, D.K, e2);
                    se = (double)e2[0] + (double)e2[1];
                    e2[0] = T * e2[0];
                    e2[1] = T * e2[1];
                }
            }
            // energy-exact pairs: one factor per cell on every thermal deviation, sqrt(3 N_pairs /
            // sum_j |X_j|^2), and (K > 0) K N_sam / sum_k |X'_k|^2 on every internal energy
            if (__ballot(act && exact)) {
                sx2 = seg_sum(sx2, first, last);
                if (KE) se = seg_sum(se, first, last);
            }
            if (act && exact) {
                sT = (R)((double)sT * sqrt(3.0 * (double)npj / sx2));
                if (KE) {
                    const R fint = (R)((double)D.K * (double)(2 * npj) / se);
                    e2[0] = e2[0] * fint;
                    e2[1] = e2[1] * fint;
                }
            }
            if (act) {
                const long long span = sc->span[buf], base = sc->n_mov + D.samoff[c];
                R msam, org[3], Ed[9];
                bool tet;
                sample_geometry<R>(D, c, 2 * npj, msam, org, Ed, tet);
                put_pair<R, KE>(D, pa, buf, span, base + k, seed, step, inst, cl, k, U, sT, X, e2, msam, org, Ed, tet, acc);
            }
#pragma unroll
            for (int q = 0; q < 5; ++q) acc[q] = seg_sum(acc[q], first, last);
            if (act && lane == last) {
                double pv[5];
#pragma unroll
                for (int q = 0; q < 5; ++q) pv[q] = D.P[q * nc + c];
#pragma unroll
                for (int q = 0; q < 5; ++q) D.S[q * nc + c] = pv[q] + acc[q];
            }
        }
        g = h;
    }
}

// The cells with more than 64 new pairs, which k_sample listed, one wave each (a launch
// of its own, so that its registers do not add to k_sample's); the waves take the list in a
// grid-stride loop (a cell's particles do not depend on which wave samples it).
template <typename R, bool KE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) k_sample_big(Dev D, int buf) {
    const long long nb = (long long)D.sc->n_big;
    const long long waves = (long long)gridDim.x * 8;
    for (long long k = (long long)blockIdx.x * 8 + (int)(threadIdx.x / kWave); k < nb; k += waves) {
        const int c = __builtin_amdgcn_readfirstlane(D.big[k]);
        sample_cell<R, KE>(D, buf, c, __builtin_amdgcn_readfirstlane((int)D.nsam[c]));
    }
}

// ---------------------------------------------------------------------------------------
// S3 with sampling = 2: hydro particles from the first-order g_p (Sec. 2.3).  With g expanded
// about the state W^n the step starts from, at t = dt,
//   g_p = g(W^n) [1 + alpha p],  alpha = dt e/(1 - e) - tau = dt / expm1(dt/tau) - tau,
// and the first-order correction p of the BGK model written in its Chapman-Enskog form
// (X = (u - U)/sqrt(T), z = e_int/T, G_ij = d_j U_i and grad T from the cell's limited
// gradient of W):
//   p = X_i X_j G_ij - (|X|^2 + z)/(3 + K) div U + ((|X|^2 + z)/2 - (5 + K)/2) sqrt(T) X . grad T / T.
// Acceptance-rejection from one stream of proposals per cell: proposal p draws X by Box-Muller
// on (uid_p, step, kTagGP, 0) (X0, X1 = r1 (cos, sin)(2 pi e1), X2 = r2 cos(2 pi e3)), uid_p the
// id a particle p of the cell would have, and, with K > 0, the internal energy T chi^2_K from
// (uid_p, kTagInt, 0 and 1); it is accepted when eta B < 1 + alpha p, eta the first uniform of
// (uid_p, step, kTagGP, 1) in FP64 and
// B = 1 + |alpha| (16 (sum_ij |G_ij| + |div U|) + ((3 + K) 16 + 5 + K)/2 4 sqrt(T) sum_j |d_j T| / T),
// which bounds |1 + alpha p| wherever every normal is at most 4.  The wave tries proposals
// 64 at a time, and the k-th accepted one (in proposal order) becomes particle k, until the
// cell's ns are accepted or min(64 ns, 2^20) proposals are spent; a particle k still missing
// then takes proposal k.  Unlike a proposal loop per particle, no lane idles while the
// slowest lane of its wave keeps rejecting.  Positions as in k_sample.  One wave per cell;
// S = P + the new sums.
// Sampling 3 takes the same draws from the equilibrium itself (weight 1, B = 1: proposal k is
// particle k).  The Shakhov model (Pr != 1) adds (a.X)(|X|^2 - 5) to the weight and 44 |a| to B.
// ---------------------------------------------------------------------------------------
template <typename R, bool KE>
__global__ void __launch_bounds__(256) k_sample_gp(Dev D, int buf) {
    constexpr double kBox = 4.0;
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int c = blockIdx.x * 4 + wave;
    if (c >= D.nc || D.sc->none) return;
    const int nc = D.nc;
    const int inst = inst_of(D, c);
    const InstP &P = D.ip[inst];
    if (P.sampling < 2) return;
    const bool gp = P.sampling == 2, sh = P.pr != 1.0;
    const Scalars *sc = D.sc;
    const long long ns = sc->n_new > 0 ? D.nsam[c] : 0;
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (ns > 0) {
        const Particles pa = D.pa[buf];
        const long long span = sc->span[buf], base = sc->n_mov + D.samoff[c];
        const long long step = D.is[inst].step;
        const unsigned long long seed = P.seed;
        const int cl = c - P.cell0;
        const int K = KE ? D.K : 0;
        const double W[5] = {D.W[c], D.W[nc + c], D.W[2 * nc + c], D.W[3 * nc + c], D.W[4 * nc + c]};
        const double rho = W[0], Ud[3] = {W[1] / rho, W[2] / rho, W[3] / rho};
        const double T = temp_k(W, K);
        // primitive gradients from the limited gradient of W: G[i][j] = d_j U_i, gT[j] = d_j T
        // (sampling 2 only; sampling 3 draws from the equilibrium itself)
        double G[3][3], gT[3], sU = 0.0, divU = 0.0, sTg = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            gT[j] = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) G[i][j] = 0.0;
        }
        double alpha = 0.0, Bgp = 1.0;
        if (gp) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double dr = D.gW[j * nc + c];
                double dU[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) dU[i] = (D.gW[(3 * (1 + i) + j) * nc + c] - Ud[i] * dr) / rho;
                double dT = (D.gW[(12 + j) * nc + c] - W[4] / rho * dr) / rho -
                            (Ud[0] * dU[0] + Ud[1] * dU[1] + Ud[2] * dU[2]);
                dT = 2.0 / (3.0 + K) * dT;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    G[i][j] = dU[i];
                    sU += fabs(dU[i]);
                }
                divU += dU[j];
                gT[j] = dT;
                sTg += fabs(dT);
            }
            const double tau = D.tau[c], dt = D.is[inst].dt;
            alpha = dt / expm1(dt / tau) - tau;
            Bgp = 1.0 + fabs(alpha) * (kBox * kBox * (sU + fabs(divU)) +
                                       0.5 * ((3.0 + K) * kBox * kBox + 5.0 + K) * kBox * sqrt(T) * sTg / T);
        }
        // Shakhov model: g^+ / g = 1 + (a.X)(|X|^2 - 5), a = (1 - Pr) q / (5 rho T^(3/2)) with the
        // cell's heat flux q; 44 |a| bounds the correction on |X| <= 4 (clipped beyond)
        double a[3] = {0.0, 0.0, 0.0}, Bsh = 0.0;
        if (sh) {
            const double fa = (1.0 - P.pr) / (5.0 * W[0] * T * sqrt(T));
#pragma unroll
            for (int d = 0; d < 3; ++d) a[d] = fa * D.qh[d * nc + c];
            Bsh = 44.0 * sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
        }
        const double B = Bgp + Bsh;
        const double sqT = sqrt(T);
        const R U[3] = {(R)Ud[0], (R)Ud[1], (R)Ud[2]};
        const R sT = (R)sqT, TR = (R)T;
        const R msam = (R)(D.ec[c] * D.rhoh[c] * D.vol[c] / (double)ns);
        const R org[3] = {(R)D.orig[c], (R)D.orig[nc + c], (R)D.orig[2 * nc + c]};
        R Ed[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) Ed[q] = (R)D.edge[q * nc + c];
        const bool tet = D.ctype[c] == 4;
        const R two_pi = (R)2 * (R)kPi;
        // proposal p of the cell (draws keyed by the id a particle p would have): its velocity,
        // internal energy and whether it is accepted
        auto propose = [&](long long p, R u[3], R &e) -> bool {
            const uint64_t uidp = make_uid(step, cl, p);
            const U4 rv = draw(seed, uidp, step, kTagGP, 0u, inst);
            const R r1 = sqrt((R)-2 * log(unif<R>(rv.v[0]))), r2 = sqrt((R)-2 * log(unif<R>(rv.v[2])));
            R sn, cs;
            sin_cos(two_pi * unif<R>(rv.v[1]), sn, cs);
            const R X[3] = {(R)(r1 * cs), (R)(r1 * sn), (R)(r2 * cos(two_pi * unif<R>(rv.v[3])))};
#pragma unroll
            for (int d = 0; d < 3; ++d) u[d] = U[d] + sT * X[d];
            e = (R)0;
            if (KE && K > 0) e = internal_energy<R>(seed, uidp, step, kTagInt, 0u, inst, K, TR);
            const U4 ra = draw(seed, uidp, step, kTagGP, 1u, inst);
            const double x0 = (double)X[0], x1 = (double)X[1], x2 = (double)X[2];
            double w = 1.0;
            if (gp) {
                const double s2 = x0 * x0 + x1 * x1 + x2 * x2 + (double)e / T;
                const double Xd[3] = {x0, x1, x2};
                double shear = 0.0, xg = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    xg += Xd[i] * gT[i];
#pragma unroll
                    for (int jj = 0; jj < 3; ++jj) shear += Xd[i] * Xd[jj] * G[i][jj];
                }
                const double pw = shear - s2 / (3.0 + K) * divU + (0.5 * s2 - 0.5 * (5.0 + K)) * sqT * xg / T;
                w = 1.0 + alpha * pw;
            }
            if (sh) w = w + (a[0] * x0 + a[1] * x1 + a[2] * x2) * ((x0 * x0 + x1 * x1 + x2 * x2) - 5.0);
            return unif<double>(ra.v[0]) * B < w;
        };
        // particle k: its id, position, record and sums
        auto put = [&](long long k, const R u[3], R e) {
            const uint64_t uid = make_uid(step, cl, k);
            const long long i = slot_of(D, buf, span, base + k);
            R x[3];
            cell_point<R>(seed, uid, step, inst, org, Ed, tet, x);
            store_new(pa, i, x, u, msam, uid);
            if (KE) store_e(pa, i, e);
            add_phi<R>(acc, msam, u, e);
        };
        // the wave tries 64 proposals at a time; the accepted ones, in proposal order, become the
        // next particles (ballot prefix counts), until ns are accepted or the proposals are spent
        const unsigned long long below = lane == 0 ? 0ULL : (~0ULL >> (64 - lane));
        const long long pmax = 64 * ns < (1LL << 20) ? 64 * ns : (1LL << 20);
        long long cnt = 0;
        for (long long p0 = 0; p0 < pmax && cnt < ns; p0 += kWave) {
            const long long p = p0 + lane;
            R u[3] = {(R)0, (R)0, (R)0}, e = (R)0;
            const bool ok = p < pmax && propose(p, u, e);
            const unsigned long long m = __ballot(ok);
            const long long k = cnt + (long long)__popcll(m & below);
            if (ok && k < ns) put(k, u, e);
            cnt += (long long)__popcll(m);
        }
        // proposals spent: a particle k still missing takes proposal k, accepted or not
        for (long long k = (cnt < ns ? cnt : ns) + lane; k < ns; k += kWave) {
            R u[3], e;
            (void)propose(k, u, e);
            put(k, u, e);
        }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k] = wave_sum(acc[k]);
    double ak = acc[0];
#pragma unroll
    for (int k = 1; k < 5; ++k)
        if (lane == k) ak = acc[k];
    if (lane < 5) D.S[lane * nc + c] = D.P[lane * nc + c] + ak;
}

// ---------------------------------------------------------------------------------------
// S5 (far field): free-stream particles entering through far-field faces.  Outside the
// domain the gas is the free stream W_inf; the part of it that reaches a face without a
// collision in the step, exp(-dt/tau_inf) of its density, crosses the face with the
// one-sided number flux Gamma = sigma (phi(a) + a Phi(a)) (a = U_inf.n_in / sigma, sigma =
// sqrt(T_inf)).  Face of area A on cell Omega: mass exp(-dt/tau_inf) rho_inf Gamma A dt in
// N = ceil(Gamma A dt N_ref / Omega) equal particles, none below a ratio of 1e-9.  Particle
// k: normal speed from the flux-weighted half-Maxwellian, tangential components Gaussian
// about U_inf in the face frame, entry point uniform on the face, entry time uniform in
// the step (drawn again by the transport, which starts it on that face).  Computed in FP64
// in both forms; the FP32 form rounds what it stores.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double npdf(double t) { return exp(-0.5 * t * t) / sqrt(2.0 * kPi); }
__device__ __forceinline__ double ncdf(double t) { return 0.5 * erfc(-t / sqrt(2.0)); }

// z = v_n / sigma has density g(z) = z phi(z - a) / Z(a) on z > 0, Z(a) = phi(a) + a Phi(a), and
// distribution G(z) = (phi(a) - phi(z - a) + a (Phi(z - a) - Phi(-a))) / Z(a); the root of
// G(z) = eta is the result of 60 bisections of [0, max(a, 0) + 40].  Where g is small the
// rounding of G decides their last steps, so that another way to the root ends up to 1e-7 from
// it; the same bisections are therefore made, but G is evaluated only where it has to be.
// Halley's iteration from the mode of g (G''/G' = 1/z - (z - a)) finds the root, and G is
// evaluated at `band` on either side of it: G grows with z, so where it is further from eta than
// `noise` there (several times the rounding of its terms), the side of every point beyond is
// known, whatever the iteration left.  If it is not, the band is widened, at last to the plain
// bisections.  Below a = -3 the cancellation in Z leaves little to gain.  Some 15 evaluations
// instead of 60.
__device__ double flux_speed(double a, double eta) {
    const double pa = npdf(a), Z = pa + a * ncdf(a), cm = ncdf(-a), top = (a > 0.0 ? a : 0.0) + 40.0;
    auto dist = [&](double m) { return (pa - npdf(m - a) + a * (ncdf(m - a) - cm)) / Z; };
    double z = 0.5 * (a + sqrt(a * a + 4.0)), band = 1e9;
    // (at the very ends of the distribution the rounding has no scale: the plain bisections)
    if (a >= -3.0 && eta > 1e-12 && eta < 1.0 - 1e-12) {
        const double noise = 2e-15 * (1.0 + (pa + fabs(a)) / Z);
        double lo = 0.0, hi = top, b = 0.0;
        for (int it = 0; it < 24; ++it) {
            const double t = z - a, p = npdf(t);
            const double f = (pa - p + a * (ncdf(t) - cm)) / Z - eta, g = z * p / Z;
            if (f < 0.0)
                lo = z;
            else
                hi = z;
            double dz = f / g;
            const double den = 1.0 - 0.5 * dz * (1.0 / z - t);
            if (den > 0.5) dz = dz / den;
            double zn = z - dz;
            if (!(zn >= lo && zn <= hi)) zn = 0.5 * (lo + hi);
            const double moved = fabs(zn - z);
            b = 2.0 * noise / g + 2e-15 * (z + 1.0);
            z = zn;
            if (moved <= 1e-6 * fmin(z, 1.0) || moved <= 0.25 * b) break;
        }
        for (int k = 0; k < 3 && band > 1e8; ++k) {
            const double zl = z - b, zr = z + b;
            if ((zl <= 0.0 || dist(zl) < eta - noise) && (zr >= top || dist(zr) > eta + noise)) band = b;
            b = 8.0 * b;
        }
    }
    double lo = 0.0, hi = top;
    for (int it = 0; it < 60; ++it) {
        const double m = 0.5 * (lo + hi);
        bool below = m < z - band;
        if (!below && !(m > z + band)) {
            if (m <= lo || m >= hi) break;  // neighbouring numbers: m is the side it was before
            below = dist(m) < eta;
        }
        if (below)
            lo = m;
        else
            hi = m;
    }
    return 0.5 * (lo + hi);
}

struct Inflow {
    int c, lf, bf, tri, inst;
    double dt;
    long long N;
    double m, sig, a, vt1, vt2, T;
    double nin[3], t1[3], t2[3];
};

__device__ Inflow inflow_face(const Dev &D, int j, double dt) {
    Inflow q;
    const int4 fi = D.ffi[j];
    q.c = fi.x;
    q.inst = inst_of(D, q.c);
    const InstP &P = D.ip[q.inst];
    q.dt = dt;
    q.lf = fi.y & 0xFF;
    q.tri = fi.y >> 8;
    q.bf = fi.z;
    const DevBC &b = D.bc[fi.w];
    const double rho = b.Winf[0];
    const double Ui[3] = {b.Winf[1] / rho, b.Winf[2] / rho, b.Winf[3] / rho};
    const double T = temp_k(b.Winf, D.K);
    q.T = T;
    const double tau = P.mu_ref * pow(T, P.omega) / (rho * T);
    // wave-only start phase: the free stream enters as waves only
    const double e = D.is[q.inst].step < P.gks_steps ? 0.0 : exp(-dt / tau);
    const double4 pl = D.plane[q.c * 6 + q.lf];  // outward: the particle enters along -n
    q.nin[0] = -pl.x;
    q.nin[1] = -pl.y;
    q.nin[2] = -pl.z;
    face_frame<double>(q.nin, q.t1, q.t2);
    q.sig = sqrt(T);
    const double sd = Ui[0] * q.nin[0] + Ui[1] * q.nin[1] + Ui[2] * q.nin[2];
    q.a = sd / q.sig;
    const double Gam = q.sig * (npdf(q.a) + q.a * ncdf(q.a));
    const double area = D.ffg[10 * j + 9];
    const double r = Gam * area * dt * (double)P.n_ref / D.vol[q.c];
    q.N = 0;
    q.m = 0.0;
    if (e * rho > 0.0 && r >= 1e-9) {
        const double cr = ceil(r);
        q.N = cr <= 1048576.0 ? (long long)cr : -1;
        if (q.N > 0) q.m = (e * rho * Gam * area * dt) / (double)q.N;
    }
    q.vt1 = Ui[0] * q.t1[0] + Ui[1] * q.t1[1] + Ui[2] * q.t1[2];
    q.vt2 = Ui[0] * q.t2[0] + Ui[1] * q.t2[1] + Ui[2] * q.t2[2];
    return q;
}

__device__ __forceinline__ long long inject_count(const Dev &D, int j) {
    const Inflow q = inflow_face(D, j, step_dt(D, inst_of(D, D.ffi[j].x)));
    long long n = q.N;
    if (n < 0) {
        atomicOr(&D.sc->err, kErrCellCount);
        n = 0;
    }
    D.ninj[j] = n;
    return n;
}

// The counts of new particles: per cell (its first blocks) and per far-field face (the others),
// with each block's sum for k_offsets, so that no kernel reads the counts only to sum them: a step
// takes two launches to its offsets instead of four (seven with inflow), 7.2 us on 2,709 cells
// against 9.8, 22 against 46 on 349,224 tetrahedra with a far field.
__global__ void __launch_bounds__(kCountBS) k_cell_prep(Dev D) {
    __shared__ long long ws[kCountBS / kWave];
    const int gc = (D.nc + kCountBS - 1) / kCountBS;
    long long n = 0;
    if ((int)blockIdx.x < gc) {
        const int c = blockIdx.x * kCountBS + threadIdx.x;
        if (c < D.nc) n = cell_prep(D, c);
    } else {
        const int j = ((int)blockIdx.x - gc) * kCountBS + threadIdx.x;
        if (j < D.nff) n = inject_count(D, j);
    }
    n = (long long)wave_sum_u64((unsigned long long)n);
    if (lane_id() == 0) ws[threadIdx.x / kWave] = n;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kCountBS / kWave; ++w) n += ws[w];
    D.scan64[blockIdx.x] = n;
}

// one thread per entering particle, whose face it finds among the prefix sums (a face lets a few
// particles in, so a wave per face left most lanes idle: with the bisections 455 us for the
// far field of the Mach 10 cube on 349,224 tetrahedra); they follow the sampled ones
template <typename R>
__global__ void __launch_bounds__(256) k_inject(Dev D, int buf) {
    const Scalars *sc = D.sc;
    const long long n = sc->n_inj;
    const long long span = sc->span[buf], base = sc->n_mov + sc->n_new, list = sc->n_old + sc->n_new;
    const Particles pa = D.pa[buf];
    const double two_pi = 2.0 * kPi;
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
        int j = 0, end = D.nff;  // injoff[j] <= p < injoff[j + 1]
        while (end - j > 1) {
            const int mid = j + (end - j) / 2;
            if (D.injoff[mid] <= p)
                j = mid;
            else
                end = mid;
        }
        const long long k = p - D.injoff[j];
        const Inflow q = inflow_face(D, j, D.is[inst_of(D, D.ffi[j].x)].dt);
        const long long step = D.is[q.inst].step;
        const unsigned long long seed = D.ip[q.inst].seed;
        const double *g = D.ffg + 10 * j;
        const uint64_t uid = (1ULL << 63) | make_uid(step, q.bf, k);
        const U4 rv = draw(seed, uid, step, kTagInject, 0, q.inst);
        const U4 rp = draw(seed, uid, step, kTagPos, 0, q.inst);
        const double vn = q.sig * flux_speed(q.a, unif<double>(rv.v[0]));
        const double rr = sqrt(-2.0 * log(unif<double>(rv.v[1])));
        const double ang = two_pi * unif<double>(rv.v[2]);
        const double X1 = rr * cos(ang), X2 = rr * sin(ang);
        const double w1 = q.vt1 + q.sig * X1, w2 = q.vt2 + q.sig * X2;
        double p1 = unif<double>(rp.v[0]), p2 = unif<double>(rp.v[1]);
        if (q.tri && p1 + p2 > 1.0) {
            p1 = 1.0 - p1;
            p2 = 1.0 - p2;
        }
        R x[3], u[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = (R)(vn * q.nin[d] + w1 * q.t1[d] + w2 * q.t2[d]);
            x[d] = (R)(g[d] + p1 * g[3 + d] + p2 * g[6 + d]);
        }
        const long long i = slot_of(D, buf, span, base + p);
        store_new(pa, i, x, u, (R)q.m, uid);
        D.lkey[list + p] = q.c;  // its start cell, for k_stream_in
        if (D.K > 0) store_e(pa, i, (R)internal_energy<double>(seed, uid, step, kTagInt, 0, q.inst, D.K, q.T));
    }
}

// ---------------------------------------------------------------------------------------
// S4 + S5: face-to-face transport of one particle for time ts (Sec. 2.3).
// Exit time over the faces with n.u > 0 other than the entry face, clamped at 0, lowest local
// face on a tie; an exit time >= the remaining time keeps the particle in the cell.
// Box hexes take a path that evaluates only the three candidate faces; its arithmetic is
// the plane formula (d - n.x) / (n.u) with n = +-e_d, term by term, so both paths give the
// same bits.
// ---------------------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ const R *cell_box(const Dev &D, int c);
template <>
__device__ __forceinline__ const double *cell_box<double>(const Dev &D, int c) {
    return D.box + 6 * c;
}
template <>
__device__ __forceinline__ const float *cell_box<float>(const Dev &D, int c) {
    return D.box32 + 6 * c;
}
template <typename R>
__device__ __forceinline__ R face_far(const Dev &D, int s);
template <>
__device__ __forceinline__ double face_far<double>(const Dev &D, int s) {
    return D.nfar[s];
}
template <>
__device__ __forceinline__ float face_far<float>(const Dev &D, int s) {
    return D.nfar32[s];
}

__device__ __forceinline__ void cell_plane(const Dev &D, int s, double p[4]) {
    const double4 q = D.plane[s];
    p[0] = q.x;
    p[1] = q.y;
    p[2] = q.z;
    p[3] = q.w;
}
__device__ __forceinline__ void cell_plane(const Dev &D, int s, float p[4]) {
    const float4 q = D.plane32[s];
    p[0] = q.x;
    p[1] = q.y;
    p[2] = q.z;
    p[3] = q.w;
}

// diffuse re-emission: u_n = sqrt(-2 T_w ln eta) into the domain, tangential components
// N(U_w, T_w) in the face frame; with K internal degrees of freedom (e != nullptr) the internal
// energy variable leaves in equilibrium at T_w too (full accommodation)
template <typename R>
__device__ __forceinline__ void reemit_diffuse(const DevBC &b, const R n[3], R u[3], uint64_t uid, const StepCtx &sx,
                                               int bounce, R *e = nullptr, int K = 0) {
    U4 r = draw(sx.seed, uid, sx.step, kTagWall, (uint32_t)bounce, sx.inst);
    R t1[3], t2[3];
    face_frame<R>(n, t1, t2);
    const R Tw = (R)b.Tw;
    const R sq = sqrt(Tw);
    const R vn = sqrt((R)-2 * Tw * log(unif<R>(r.v[0])));
    const R rr = sqrt((R)-2 * log(unif<R>(r.v[1])));
    const R a = (R)2 * (R)kPi * unif<R>(r.v[2]);
    const R X1 = rr * cos(a), X2 = rr * sin(a);
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = (R)b.Uw[d] - vn * n[d] + sq * (X1 * t1[d] + X2 * t2[d]);
    if (e) *e = internal_energy<R>(sx.seed, uid, sx.step, kTagWallInt, 2u * (uint32_t)bounce, sx.inst, K, Tw);
}

// Decisions on exit times without a division.  The time to a face is tt = max(a, 0) / un (a its
// distance, un > 0 the speed towards it).  Products decide comparisons of such quotients by a
// relative margin well above the rounding of either; only values within the margin (or so small
// that a product could lose precision) are divided, so every decision is the formula's own.
template <typename R>
struct Margin;
template <>
struct Margin<double> {
    static constexpr double up = 1.0 + 1e-12, dn = 1.0 - 1e-12, tiny = 1e-280;
};
template <>
struct Margin<float> {
    static constexpr float up = 1.0f + 1e-5f, dn = 1.0f - 1e-5f, tiny = 1e-30f;
};
// whether a flight of time ts meets the face (tt < ts)
template <typename R>
__device__ __forceinline__ bool meets_face(R a, R un, R ts) {
    const R reach = un * ts;
    if (reach > Margin<R>::tiny) {
        if (a >= reach * Margin<R>::up) return false;
        if (a < reach * Margin<R>::dn) return true;
    }
    R tt = a / un;
    if (tt < (R)0) tt = (R)0;
    return tt < ts;
}
// the face with the smallest exit time (the lowest local face on a tie): its distance over speed
template <typename R>
struct Exit {
    R a, un;
    int lf;
};
template <typename R>
__device__ __forceinline__ void nearer(Exit<R> &b, R a, R un, R reach, int lf) {
    // a face at distance a >= un trem (1 + margin) has a computed exit time >= trem, so it can
    // be neither the smallest nor a crossing
    if (!(un > (R)0) || !(a < reach * Margin<R>::up || reach <= Margin<R>::tiny) || a != a) return;
    const R ac = a > (R)0 ? a : (R)0;
    bool take = b.lf < 0;
    if (!take) {
        const R l = ac * b.un, r = b.a * un;
        if (fmax(l, r) > Margin<R>::tiny && (l < r * Margin<R>::dn || l > r * Margin<R>::up))
            take = l < r;
        else
            take = ac / un < b.a / b.un;
    }
    b.a = take ? ac : b.a;
    b.un = take ? un : b.un;
    b.lf = take ? lf : b.lf;
}

// Flight of one particle for the time ts from cell `cell`, entered through its local face
// `entry` (-1: none).  Returns 0 (ends inside the domain), 1 (left through a far-field face)
// or -1 (more than max_cross crossings); ncross, nwall and bounce (diffuse re-emissions so
// far, which keys the wall draws) carry on from their values at the call.  MESH 1: every cell
// a box and neighbours share whole faces; 2: every cell a tetrahedron; 0: any mesh.  What a
// crossing costs is the dependent loads of the next cell: one round with MESH 1 (the neighbour
// and its far bound) and 2 (the neighbour, then its planes with its own neighbours), three
// with MESH 0.
template <typename R, int MESH>
__device__ int track(const Dev &D, R x[3], R u[3], int &cell, R &ts, int &entry, uint64_t uid, const StepCtx &sx,
                     int &ncross, int &nwall, int &bounce, R *e = nullptr) {
    int c = cell;
    R trem = ts;
    // bounds of box cell c; on conforming boxes a crossing builds them for the next cell
    R B[6];
    bool haveB = false;
    for (;;) {
        Exit<R> ex{(R)0, (R)1, -1};
        int2 nb = make_int2(0, 0);
        const bool box = MESH == 1 || (MESH == 0 && D.ctype[c] == 8);
        if (box) {
            if (!haveB) {
                const R *Bg = cell_box<R>(D, c);
#pragma unroll
                for (int q = 0; q < 6; ++q) B[q] = Bg[q];
                haveB = true;
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const bool up = u[d] > (R)0;
                const R au = fabs(u[d]), a = up ? B[3 + d] - x[d] : x[d] - B[d];
                const int lf = 2 * d + (up ? 1 : 0);
                if (lf != entry) nearer<R>(ex, a, au, au * trem, lf);
            }
        } else {
            R pl[4][4];
            int2 nbs[4];
#pragma unroll
            for (int lf = 0; lf < 4; ++lf) {
                cell_plane(D, c * 6 + lf, pl[lf]);
                nbs[lf] = D.nbl[c * 6 + lf];
            }
#pragma unroll
            for (int lf = 0; lf < 4; ++lf) {
                const R *p = pl[lf];
                const R un = p[0] * u[0] + p[1] * u[1] + p[2] * u[2];
                const R a = p[3] - (p[0] * x[0] + p[1] * x[1] + p[2] * x[2]);
                if (lf != entry) nearer<R>(ex, a, un, un * trem, lf);
                if (ex.lf == lf) nb = nbs[lf];
            }
        }
        const int bf = ex.lf;
        const R best = ex.a / ex.un;
        if (bf < 0 || best >= trem) {
            x[0] = x[0] + u[0] * trem;
            x[1] = x[1] + u[1] * trem;
            x[2] = x[2] + u[2] * trem;
            cell = c;
            return 0;
        }
        x[0] = x[0] + u[0] * best;
        x[1] = x[1] + u[1] * best;
        x[2] = x[2] + u[2] * best;
        trem = trem - best;
        if (++ncross > sx.max_cross) {
            cell = c;
            return -1;
        }
        // the far bound of the next box, loaded together with the neighbour
        R far = (R)0;
        if (box) {
            nb = D.nbl[c * 6 + bf];
            if (MESH == 1) far = face_far<R>(D, c * 6 + bf);
        }
        if (nb.x >= 0) {
            int ent = nb.y;
            if (ent >= kPeriodicEntry) {
                // periodic face: the particle goes on from the partner face at x + shift
                const DevBC &pb = D.bc[ent / kPeriodicEntry - 1];
                x[0] = x[0] + (R)pb.shift[0];
                x[1] = x[1] + (R)pb.shift[1];
                x[2] = x[2] + (R)pb.shift[2];
                ent = ent % kPeriodicEntry;
                haveB = false;
            } else if (MESH == 1) {
                // the neighbour shares the whole face: its bounds along the face's axis are
                // this cell's bound at the face and the far one
                // (selects: an array indexed at run time would live in scratch memory)
                const int d = bf >> 1;
                const bool up = (bf & 1) != 0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const R lo = B[k], hi = B[3 + k];
                    B[k] = k == d ? (up ? hi : far) : lo;
                    B[3 + k] = k == d ? (up ? far : lo) : hi;
                }
            } else {
                haveB = false;
            }
            entry = ent;
            c = nb.x;
            continue;
        }
        const DevBC &b = D.bc[-1 - nb.x];
        if (b.type == 0) {
            if (box) {
                // u - 2 (u.n) n with n = +-e_d flips exactly component d
                const int d = bf >> 1;
#pragma unroll
                for (int k = 0; k < 3; ++k) u[k] = k == d ? -u[k] : u[k];
            } else {
                R p[4];
                cell_plane(D, c * 6 + bf, p);
                const R un = p[0] * u[0] + p[1] * u[1] + p[2] * u[2];
                u[0] = u[0] - (R)2 * un * p[0];
                u[1] = u[1] - (R)2 * un * p[1];
                u[2] = u[2] - (R)2 * un * p[2];
            }
            entry = bf;
        } else if (b.type == 1) {
            R p[4];
            cell_plane(D, c * 6 + bf, p);
            const R n[3] = {p[0], p[1], p[2]};
            reemit_diffuse<R>(b, n, u, uid, sx, bounce, e, D.K);
            ++bounce;
            ++nwall;
            entry = bf;
        } else {
            cell = c;
            return 1;
        }
    }
}

// store of the transported state of particle i: position and velocity; mass and id (the last 16 bytes
// of an FP64 record, the last 8 of an FP32 one) stay
__device__ __forceinline__ void store_state(const Particles &pa, long long i, const double x[3], const double u[3]) {
    double2 *rp = reinterpret_cast<double2 *>(pa.rec + i);
    rp[0] = make_double2(x[0], x[1]);
    rp[1] = make_double2(x[2], u[0]);
    rp[2] = make_double2(u[1], u[2]);
}
__device__ __forceinline__ void store_state(const Particles &pa, long long i, const float x[3], const float u[3]) {
    float4 *rp = reinterpret_cast<float4 *>(pa.rec32 + i);
    rp[0] = make_float4(x[0], x[1], x[2], u[0]);
    float2 *q = reinterpret_cast<float2 *>(rp + 1);
    q[0] = make_float2(u[1], u[2]);
}

// Free flight of a cell's particles by one wave, 64 at a time in the cell's order (arrivals,
// stayers, new ones).  The free-flight time of an old particle is t_f = -tau ln eta with tau of
// its start cell; it collides iff t_f < dt.  Since t_f < dt <=> eta > exp(-dt/tau), eta below
// exp(-dt/tau) by a relative margin decides the comparison without the logarithm (the same
// decision as the formula, which is evaluated near the threshold and for every collided
// particle).
//
// Every particle is read once here.  A stayer (collisionless, no face met) is written at once,
// moved by u dt, to its cell's region of the next buffer, whose start is known beforehand
// (Particles), and summed into P^{n+1}; a particle that collided before it met a face is summed
// into the cell's part of E and dropped.  The others meet a face: they are put on the cell's
// list with their slot and flight time, and k_track follows them.
//
// What bounds it: the vector ALU (a wave64 instruction holds its SIMD for four cycles), about
// half of it the Philox draw.  So a face is decided without a division: it is met iff its
// distance over the normal speed is below the flight time, which the product of speed and time
// decides by a relative margin well above the rounding; only a particle within the margin takes
// the quotient itself (the same decision as k_track's formula).  And the tracking loop, which
// one lane in seven needs, is left to a kernel whose lanes all need it.  One wave per cell: the
// cell's data (faces, tau, exp(-dt/tau), the instance's constants) are read once, into scalar
// registers, and the first rounds of the draw, on counter words that do not change within
// the instance, are scalar too.

// a record as 16-byte chunks
template <typename R>
struct RecChunks;
template <>
struct RecChunks<double> {
    static constexpr int N = 4;  // x0 x1 | x2 u0 | u1 u2 | m id
};
template <>
struct RecChunks<float> {
    static constexpr int N = 2;  // x0 x1 x2 u0 | u1 u2 id
};
__device__ __forceinline__ uint4 *rec_chunks(const Particles &p, long long i, double) {
    return reinterpret_cast<uint4 *>(p.rec + i);
}
__device__ __forceinline__ uint4 *rec_chunks(const Particles &p, long long i, float) {
    return reinterpret_cast<uint4 *>(p.rec32 + i);
}

// a whole record in registers
template <typename R>
struct Part {
    R x[3], u[3], m, e;
    uint64_t uid;
};
template <bool KE>
__device__ __forceinline__ void load_part(const Particles &pa, long long i, Part<double> &q) {
    const double2 *a = reinterpret_cast<const double2 *>(pa.rec + i);
    const double2 r0 = a[0], r1 = a[1], r2 = a[2], r3 = a[3];
    q.x[0] = r0.x;
    q.x[1] = r0.y;
    q.x[2] = r1.x;
    q.u[0] = r1.y;
    q.u[1] = r2.x;
    q.u[2] = r2.y;
    q.m = r3.x;
    q.uid = (uint64_t)__double_as_longlong(r3.y);
    q.e = KE ? pa.e64[i] : 0.0;
}
template <bool KE>
__device__ __forceinline__ void load_part(const Particles &pa, long long i, Part<float> &q) {
    const float4 *a = reinterpret_cast<const float4 *>(pa.rec32 + i);
    const float4 r0 = a[0], r1 = a[1];
    q.x[0] = r0.x;
    q.x[1] = r0.y;
    q.x[2] = r0.z;
    q.u[0] = r0.w;
    q.u[1] = r1.x;
    q.u[2] = r1.y;
    q.uid = (uint64_t)__float_as_uint(r1.z) | ((uint64_t)__float_as_uint(r1.w) << 32);
    q.m = pa.m32[i];
    q.e = KE ? pa.e32[i] : 0.0f;
}
// a record into its place in a wave's LDS stage
__device__ __forceinline__ void stage_part(uint4 *slot, const Part<double> &q) {
    double2 *d = reinterpret_cast<double2 *>(slot);
    d[0] = make_double2(q.x[0], q.x[1]);
    d[1] = make_double2(q.x[2], q.u[0]);
    d[2] = make_double2(q.u[1], q.u[2]);
    d[3] = make_double2(q.m, __longlong_as_double((long long)q.uid));
}
__device__ __forceinline__ void stage_part(uint4 *slot, const Part<float> &q) {
    float4 *f = reinterpret_cast<float4 *>(slot);
    f[0] = make_float4(q.x[0], q.x[1], q.x[2], q.u[0]);
    f[1] = make_float4(q.u[1], q.u[2], __uint_as_float((uint32_t)q.uid), __uint_as_float((uint32_t)(q.uid >> 32)));
}
// the arrays beside the records: mass (FP32 form) and internal energy
template <bool KE>
__device__ __forceinline__ void store_side(const Particles &pa, long long i, const Part<double> &q) {
    if constexpr (KE) pa.e64[i] = q.e;
}
template <bool KE>
__device__ __forceinline__ void store_side(const Particles &pa, long long i, const Part<float> &q) {
    pa.m32[i] = q.m;
    if constexpr (KE) pa.e32[i] = q.e;
}

// the crossing counts of a block's waves into the step's (called by the whole block)
template <int NW>
__device__ __forceinline__ void block_counts(const Dev &D, unsigned long long nx, unsigned long long nw, unsigned mx,
                                             bool lost, unsigned long long red[3][NW]) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    if (__ballot(lost) && lane == 0) atomicOr(&D.sc->err, kErrLost);
    nx = wave_sum_u64(nx);
    nw = wave_sum_u64(nw);
    mx = wave_max_u32(mx);
    if (lane == 0) {
        red[0][wave] = nx;
        red[1][wave] = nw;
        red[2][wave] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long a = 0, b = 0, m = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            a += red[0][w];
            b += red[1][w];
            m = max(m, red[2][w]);
        }
        if (a) atomicAdd(&D.spart[blockIdx.x & (kWallSeg - 1)], a);
        if (b) atomicAdd(&D.spart[kWallSeg + (blockIdx.x & (kWallSeg - 1))], b);
        raise_max_cross(D, (unsigned)m);
    }
}

// Cells with many particles.  A wave per cell goes through its cell's runs of 64 one after the other, so a few
// cells of hundreds of particles leave the chip idle: on a small mesh (long_from) a cell of more than
// Dev::long_from particles is left to k_stream_long.  There the kLongWaves waves of a block take the
// runs in turn, with the same places for every particle (the runs' counts meet in local memory).
// Every run's terms of the sums go through local memory too and are added lane by lane in the
// order of the runs, as one wave adds them, so the bits do not depend on who takes a cell.
// 64 boxes of 10,000 particles, FP64: k_stream 331 us by waves, 132 by blocks.  Where the line lies
// (long_from), microseconds a step of a cavity by waves and by blocks, FP64 (FP32):
//   64 cells     400 particles: 117, 92 (102, 83)       2,500: 449, 166 (379, 145)
//   1,000 cells  400: 128, 109 (114, 97)                2,500: 547, 277 (466, 228)
//   1,728 cells  1,000: 233, 186 (190, 154)             2,500: 597, 405 (506, 319)
//   4,096 cells  1,000: 344, 335 (268, 257)             8 instances of 512 cells: 385, 387 (293, 297)
// Beyond, blocks cost up to 6% at 600 particles (8,000 cells FP32).  With fewer particles waves are no slower than
// a thread per particle was (64 cells of 300: 103 and 115); with 400 and more they were, by up to a third.
constexpr int kLongCell = 256, kLongWaves = 4;
template <int W>
struct LongShared {
    int4 cnt[W];                 // stayers, listed and collided particles of the waves' runs
    double part[W][10][kWave];   // the runs' terms of P and of the collided particles' sums
};

// One cell's free flight by the W waves of a block (W = 1: by one wave, without a barrier), ILP runs of 64
// particles loaded together.
template <typename R, bool MULTI, int ILP, bool KE, int W>
__device__ __forceinline__ void stream_cell(const Dev &D, int buf, int c, int w, uint4 *st, LongShared<W> *sh) {
    constexpr int CPR = RecChunks<R>::N;
    const Scalars *sc = D.sc;
    const int lane = lane_id();
    const int nc = D.nc;
    const Particles pa = D.pa[buf], pb = D.pa[buf ^ 1];
    const long long n_new = sc->n_new, span = sc->span[buf], n_mov = sc->n_mov;
    const unsigned long long o0 = D.off[c], o1 = D.off[c + 1];
    const long long so = n_new > 0 ? D.samoff[c] : 0;
    const int ns = n_new > 0 ? (int)(D.samoff[c + 1] - so) : 0;
    const int nold = hi32(o1) - hi32(o0), nm = lo32(o1) - lo32(o0);
    const int n = nold + ns;
    // (no list of these cells: a store before the loads below would take them off the scalar unit)
    if ((n > D.long_from) != (W > 1)) return;
    const int v0 = hi32(o0) + (int)so;  // this cell's region of the next buffer
    const int vs = D.v0[buf][c] - nm;   // slot of an old particle k >= nm: vs + k
    // places of its arrivals and of its new particles in the second part of this buffer: am + k
    // for k < nm, an + k for k >= nold
    const long long am = lo32(o0), an = n_mov + so - nold;
    const bool wrap = n_mov + n_new > D.cap - span;
    const int inst = MULTI ? D.cinst[c] : 0;
    const InstP &P = D.ip[inst];
    const unsigned long long seed = P.seed;
    const long long step = D.is[inst].step;
    const R dt = (R)D.is[inst].dt;
    const R e = (R)D.ec[c], tauc = (R)D.tau[c];
    const bool box = D.all_box || D.ctype[c] == 8;
    // the cell's faces: the bounds of a box, or the planes of a tetrahedron
    R F[16];
    if (box) {
        const R *Bg = cell_box<R>(D, c);
#pragma unroll
        for (int q = 0; q < 6; ++q) F[q] = Bg[q];
    } else {
#pragma unroll
        for (int lf = 0; lf < 4; ++lf) cell_plane(D, c * 6 + lf, F + 4 * lf);
    }
    const R elow = e * (sizeof(R) == 8 ? (R)(1.0 - 1e-12) : (R)(1.0f - 1e-5f));
    const unsigned long long below = lane == 0 ? 0ULL : (~0ULL >> (64 - lane));
    double Pn[5] = {0, 0, 0, 0, 0}, Cn[5] = {0, 0, 0, 0, 0};
    int nst = 0, nlv = 0, nco = 0;  // stayers, particles that meet a face, collided here
    double mine[3] = {0, 0, 0};     // (W > 1) the sums that this wave keeps: w, w + W, ...
    for (int r0 = 0; r0 < n; r0 += W * ILP * kWave) {
        const int k0 = r0 + w * kWave;
        Part<R> q[ILP];
        int slot[ILP];
#pragma unroll
        for (int j = 0; j < ILP; ++j) {
            const int k = k0 + j * kWave + lane;
            slot[j] = 0;
            if (k < n) {
                slot[j] = vs + k;
                if (k < nm || k >= nold) {
                    const long long a = (k < nm ? am : an) + k;
                    slot[j] = wrap ? slot_of(D, buf, span, a) : (int)(span + a);
                }
                load_part<KE>(pa, slot[j], q[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < ILP; ++j) {
            const int k = k0 + j * kWave + lane;
            bool meets = false, collided = false;
            R ts = dt;
            if (k < n) {
                if (k < nold) {
                    const U4 r = draw(seed, q[j].uid, step, kTagTF, 0, inst);
                    const R eta = unif<R>(r.v[0]);
                    if (!(eta < elow)) {
                        const R tf = -tauc * log(eta);
                        if (tf < dt) {
                            ts = tf;
                            collided = true;
                        }
                    }
                }
                if (box) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const R ud = q[j].u[d], au = fabs(ud);
                        const R a = ud > (R)0 ? F[3 + d] - q[j].x[d] : q[j].x[d] - F[d];
                        if (au > (R)0) meets = meets || meets_face<R>(a, au, ts);
                    }
                } else {
#pragma unroll
                    for (int lf = 0; lf < 4; ++lf) {
                        const R *p = F + 4 * lf;
                        const R un = p[0] * q[j].u[0] + p[1] * q[j].u[1] + p[2] * q[j].u[2];
                        const R a = p[3] - (p[0] * q[j].x[0] + p[1] * q[j].x[1] + p[2] * q[j].x[2]);
                        if (un > (R)0) meets = meets || meets_face<R>(a, un, ts);
                    }
                }
            }
            const bool stay = k < n && !meets && !collided, own = k < n && !meets && collided;
            const unsigned long long ms = __ballot(stay), ml = __ballot(meets), mo = __ballot(own);
            const int cs = (int)__popcll(ms);
            const int rs = (int)__popcll(ms & below);
            double tP[5] = {0, 0, 0, 0, 0}, tC[5] = {0, 0, 0, 0, 0};
            if (stay) {
                // the transport's last move of a flight that meets no face
#pragma unroll
                for (int d = 0; d < 3; ++d) q[j].x[d] = q[j].x[d] + q[j].u[d] * dt;
                add_phi<R>(W > 1 ? tP : Pn, q[j].m, q[j].u, q[j].e);
                stage_part(st + rs * CPR, q[j]);
            }
            if (mo && own) add_phi<R>(W > 1 ? tC : Cn, q[j].m, q[j].u, q[j].e);
            int ps = nst, pl = nlv, as = cs, al = (int)__popcll(ml), ao = (int)__popcll(mo);  // first places, the round's counts
            if (W > 1) {
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    sh->part[w][i][lane] = tP[i];
                    if (mo) sh->part[w][5 + i][lane] = tC[i];
                }
                if (lane == 0) sh->cnt[w] = make_int4(as, al, ao, 0);
                __syncthreads();
                as = al = ao = 0;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const int4 v = sh->cnt[i];
                    if (i < w) {
                        ps += v.x;
                        pl += v.y;
                    }
                    as += v.x;
                    al += v.y;
                    ao += v.z;
#pragma unroll
                    for (int h = 0; h < 3; ++h) {
                        const int t = w + h * W;
                        if (t < 5 || (t < 10 && v.z)) mine[h] += sh->part[i][t][lane];
                    }
                }
            }
            if (stay) store_side<KE>(pb, v0 + ps + rs, q[j]);
            if (meets) {
                const int li = v0 + pl + (int)__popcll(ml & below);
                D.lsrc[li] = (uint32_t)slot[j] | (k < nold ? 0u : kNewBit);
                reinterpret_cast<R *>(D.perm + li)[0] = collided ? -ts : ts;  // (ts > 0)
            }
            // the wave's LDS accesses stay in order; consecutive lanes on consecutive chunks
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            uint4 *g = rec_chunks(pb, v0 + ps, R(0));
            for (int i = lane; i < cs * CPR; i += kWave) st_nt(&g[i], st[i]);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            nst += as;
            nlv += al;
            nco += ao;
            if (W > 1) __syncthreads();  // (the counts and terms are read before the next round's are written)
        }
    }
    if (W > 1) {
#pragma unroll
        for (int h = 0; h < 3; ++h)
            if (w + h * W < 10) sh->part[0][w + h * W][lane] = mine[h];
        __syncthreads();
        if (w != 0) return;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            Pn[i] = sh->part[0][i][lane];
            Cn[i] = sh->part[0][5 + i][lane];
        }
    }
    // the stayers' part of P^{n+1}; the gather's E - S is P^{n+1} + (collided elsewhere) - S, so
    // what collided here comes off S
    double Pk, Ck;
    wave_sum_pc(Pn, Cn, Pk, Ck);
    if (lane < 5) {
        if (nco) D.S[lane * nc + c] = D.S[lane * nc + c] - Ck;
        D.P[lane * nc + c] = Pk;
    }
    if (lane == 0) {
        D.v0[buf ^ 1][c] = v0;
        D.lrun[c] = ((unsigned long long)(unsigned)v0 << 32) | (unsigned)nlv;
        D.cnt64[c] = (unsigned long long)(unsigned)nst << 32;
        D.cnt64[nc + c] = (unsigned long long)(unsigned)nco << 32;
    }
}

// BS threads per block, a wave per cell
template <typename R, int BS, bool MULTI, int ILP, bool KE>
__device__ __forceinline__ void stream_cells(const Dev &D, int buf) {
    constexpr int CPR = RecChunks<R>::N, WPB = BS / kWave;
    __shared__ uint4 stage[WPB][kWave * CPR];  // output stage of each wave
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int c = blockIdx.x * WPB + wave;
    if (c >= D.nc || D.sc->none) return;
    stream_cell<R, MULTI, ILP, KE, 1>(D, buf, c, 0, stage[wave], nullptr);
}
template <typename R, int BS, bool MULTI, int ILP>
__global__ void __launch_bounds__(BS) k_stream(Dev D, int buf) {
    stream_cells<R, BS, MULTI, ILP, false>(D, buf);
}
// the same for a gas with internal degrees of freedom
template <typename R, int BS, bool MULTI, int ILP>
__global__ void __launch_bounds__(BS) k_stream_e(Dev D, int buf) {
    stream_cells<R, BS, MULTI, ILP, true>(D, buf);
}

// the cells that k_stream leaves, a block each (the blocks of other cells leave at once)
template <typename R, bool MULTI, bool KE>
__global__ void __launch_bounds__(kLongWaves * kWave) k_stream_long(Dev D, int buf) {
    __shared__ uint4 stage[kLongWaves][kWave * RecChunks<R>::N];
    __shared__ LongShared<kLongWaves> sh;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (D.sc->none) return;
    stream_cell<R, MULTI, 1, KE, kLongWaves>(D, buf, (int)blockIdx.x, wave, stage[wave], &sh);
}

// Lanes of a wave grouped by key with ballots only: mine = the lanes that share this lane's
// key (0 for key < 0).  Must be called by the whole wave.
__device__ __forceinline__ unsigned long long key_group(int key) {
    unsigned long long todo = __ballot(key >= 0);
    unsigned long long mine = 0;
    while (todo) {
        const int lkey = __builtin_amdgcn_readlane(key, __ffsll((long long)todo) - 1);
        const unsigned long long same = __ballot(key == lkey);
        if (key == lkey) mine = same;
        todo &= ~same;
    }
    return mine;
}

// bucket counts: one atomic per end bucket of a run (the particles of a run end in a handful of
// cells; an atomic per particle queues at those few addresses: 129 against 33 us in the scatter
// of a cavity of 32^3 cells with 400 particles each)
__device__ __forceinline__ void count_run(const Dev &D, int key) {
    const unsigned long long mine = key_group(key);
    if (mine && lane_id() == __ffsll((long long)mine) - 1) atomicAdd(&D.cnt64[key], (unsigned long long)__popcll(mine));
}

// Lists of G consecutive cells taken by one wave as if they were one: lane j < G holds cell j's
// first entry and length; entry t of all of them is entry k of cell j.
template <int G>
struct Runs {
    int first[G], pre[G + 1];
    __device__ __forceinline__ Runs(int my_first, int my_len) {
        pre[0] = 0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            first[j] = __builtin_amdgcn_readlane(my_first, j);
            pre[j + 1] = pre[j] + __builtin_amdgcn_readlane(my_len, j);
        }
    }
    // cell j of entry t < pre[G] and where its list entry lies
    __device__ __forceinline__ int find(int t, int &j) const {
        int l = first[0] + t;
        j = 0;
#pragma unroll
        for (int i = 1; i < G; ++i)
            if (t >= pre[i]) {
                j = i;
                l = first[i] + (t - pre[i]);
            }
        return l;
    }
};
// Cells per wave of the kernels over the lists and buckets: eight where Dev::list_sparse says so (16,384
// cells or more of fewer than 320 particles each), else two.  A list holds some 15% of a box
// cell's particles and some 30% of a tetrahedron's, so with tens of particles per cell eight
// lists fill the lanes that one leaves idle (tetrahedra, N_ref 50: 178 against 742 us in k_track,
// 106 against 291 us in the gather), while with hundreds two lists are enough and eight leave
// too few waves (box cells, N_ref 400: 216 against 261 us).  A small mesh has few waves anyway.
// Around the limits, microseconds a step with two and with eight, FP64 (FP32):
//   cells, N_ref 50    4,096: 98, 102 (88, 91)       13,824: 172, 160 (146, 139)   19,683: 213, 192 (182, 165)
//   cells, N_ref 150   13,824: 212, 218 (168, 177)   19,683: 272, 272 (213, 216)   32,768: 321, 318 (244, 239)
//   N_ref, 32,768 cells    300: 522, 521 (384, 385)      350: 580, 591 (429, 426)      400: 637, 658 (468, 474)
//   tetrahedra, N_ref 150  13,182: 207, 209 (168, 174)   16,464: 244, 243 (193, 196)   34,992: 345, 328 (261, 258)
constexpr int kListCellsSparse = 8, kListCellsDense = 2;

// S5: the flights that meet a face: the moved state goes back to the particle's slot, its end
// bucket (end cell, or nc + end cell for a collided one, -1 for one that left through a
// far-field face) to its cell's list and into the bucket counts.  Diffuse walls re-emit here.
// One wave takes the lists of G consecutive cells.  What bounds it: the chain of dependent
// loads at each crossing, so the lanes are kept full.
template <typename R, bool KE, int MESH, int G>
__global__ void __launch_bounds__(256) k_track(Dev D, int buf) {
    constexpr int CPR = RecChunks<R>::N;
    __shared__ unsigned long long red[3][4];
    __shared__ uint4 stage[4][kWave * CPR];
    __shared__ int lslot[4][kWave];
    // (before the block's sums: with no particle anywhere they took 9.2 us on 32,768 cells, now 2.3)
    if (D.sc->none) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
    const int c0 = (blockIdx.x * 4 + wave) * G;
    const Particles pa = D.pa[buf];
    unsigned long long nx_ = 0, nw_ = 0;
    unsigned mx_ = 0;
    bool lost = false;
    if (c0 < D.nc) {
        const unsigned long long run = lane < G && c0 + lane < D.nc ? D.lrun[c0 + lane] : 0ULL;
        const Runs<G> L(hi32(run), lo32(run));
        const int n = L.pre[G];
        uint4 *st = stage[wave];
        int *ls = lslot[wave];
        for (int k0 = (int)blockIdx.y * kWave; k0 < n; k0 += D.list_split * kWave) {
            const int k = k0 + lane, nr = min(kWave, n - k0);
            int key = -1, li = 0;
            if (k < n) {
                int j;
                li = L.find(k, j);
                const int slot = (int)(D.lsrc[li] & ~kNewBit);
                R ts = reinterpret_cast<const R *>(D.perm + li)[0];
                int ec = c0 + j;
                const int inst = inst_of(D, ec);
                Part<R> q;
                load_part<KE>(pa, slot, q);
                const InstP &P = D.ip[inst];
                const StepCtx sx{P.seed, D.is[inst].step, inst, P.max_cross};
                const bool collided = ts < (R)0;  // the sign carries it
                ts = fabs(ts);
                int entry = -1, nx = 0, nw = 0, bounce = 0;
                const int rc = track<R, MESH>(D, q.x, q.u, ec, ts, entry, q.uid, sx, nx, nw, bounce, KE ? &q.e : nullptr);
                nx_ += (unsigned long long)nx;
                nw_ += (unsigned long long)nw;
                mx_ = max(mx_, (unsigned)nx);
                lost = lost || rc < 0;
                if (rc != 1) key = collided ? D.nc + ec : ec;
                if (KE && nw > 0) store_e(pa, slot, q.e);
                ls[lane] = slot;
                stage_part(st + lane * CPR, q);
            }
            // whole records, consecutive lanes on consecutive chunks
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            for (int i = lane; i < nr * CPR; i += kWave) rec_chunks(pa, ls[i / CPR], R(0))[i % CPR] = st[i];
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if (k < n) D.lkey[li] = key;
            count_run(D, key);
        }
    }
    block_counts<4>(D, nx_, nw_, mx_, lost, red);
}

// The particles entering through far-field faces, one per thread: from its entry time to the
// end of the step, starting on that face; never a stayer (it did not start in a cell) and
// never collided.  Diffuse walls re-emit here directly.  Their list is one for all of them,
// after the cells' lists.
template <typename R, bool KE, int MESH>
__global__ void __launch_bounds__(256) k_stream_in(Dev D, int buf) {
    __shared__ unsigned long long red[3][4];
    const Scalars *sc = D.sc;
    const long long n = sc->n_inj, l0 = sc->n_old + sc->n_new, a0 = sc->n_mov + sc->n_new, span = sc->span[buf];
    const Particles pa = D.pa[buf];
    unsigned long long nx_ = 0, nw_ = 0;
    unsigned mx_ = 0;
    bool lost = false;
    for (long long i0 = (long long)blockIdx.x * 256; i0 < n; i0 += (long long)gridDim.x * 256) {
        const long long i = i0 + threadIdx.x;
        int key = -1;
        if (i < n) {
            const int slot = slot_of(D, buf, span, a0 + i);
            int c = D.lkey[l0 + i];
            const int inst = inst_of(D, c);
            const InstP &P = D.ip[inst];
            const StepCtx sx{P.seed, D.is[inst].step, inst, P.max_cross};
            Part<R> q;
            load_part<KE>(pa, slot, q);
            const U4 r = draw(sx.seed, q.uid, sx.step, kTagInject, 0, inst);
            R ts = (R)(unif<double>(r.v[3]) * D.is[inst].dt);
            int entry = D.bflf[P.bf0 + (long long)((q.uid >> 20) & 0xFFFFFFULL)];
            int nx = 0, nw = 0, bounce = 0;
            const int rc = track<R, MESH>(D, q.x, q.u, c, ts, entry, q.uid, sx, nx, nw, bounce,
                                                KE ? &q.e : nullptr);
            nx_ += (unsigned long long)nx;
            nw_ += (unsigned long long)nw;
            mx_ = max(mx_, (unsigned)nx);
            lost = lost || rc < 0;
            store_state(pa, slot, q.x, q.u);
            if (KE) store_e(pa, slot, q.e);
            key = rc == 1 ? -1 : c;
            D.lkey[l0 + i] = key;
            D.lsrc[l0 + i] = (uint32_t)slot | kNewBit;
        }
        if (key >= 0) atomicAdd(&D.cnt64[key], 1ULL);
    }
    block_counts<4>(D, nx_, nw_, mx_, lost, red);
}

// the leavers by end bucket: each group of one key takes its places from the bucket's counter,
// which counts down (the order inside a bucket is fixed later by the gather).  An entry is the
// leaver's order (its place in the lists, new particles after old ones) and its slot.  A group's
// places are consecutive, its orders ascending, and, old and new particles apart, no order of
// another group lies between its first and its last; kHeadBit marks where such a piece begins.
__device__ __forceinline__ void scatter_run(const Dev &D, int li, int key, uint32_t src) {
    const unsigned long long mine = key_group(key);
    const int lane = lane_id();
    const unsigned long long fresh = __ballot((src & kNewBit) != 0);
    const int leader = mine ? __ffsll((long long)mine) - 1 : lane;
    const int n = (int)__popcll(mine);
    int at = 0;
    if (mine && lane == leader) at = lo32(atomicAdd(&D.cnt64[key], 0ULL - (unsigned long long)n)) - n;
    at = __shfl(at, leader);
    if (mine) {
        const unsigned long long below = lane == 0 ? 0ULL : (~0ULL >> (64 - lane));
        const unsigned long long before = mine & below;
        const long long j = (long long)lo32(D.off[key]) + at + (int)__popcll(before);
        const int prev = 63 - __clzll((long long)before);  // the group's lane before this one
        const bool head = before == 0 || ((fresh >> prev) & 1ULL) != ((fresh >> lane) & 1ULL);
        D.perm[j] = ((unsigned long long)((uint32_t)li | (src & kNewBit)) << 32) | (src & ~kNewBit) | (head ? kHeadBit : 0u);
    }
}
template <int G>
__global__ void __launch_bounds__(256) k_scatter(Dev D) {
    const int lane = lane_id();
    const int c0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave))) * G;
    if (c0 >= D.nc || D.sc->none) return;
    const unsigned long long run = lane < G && c0 + lane < D.nc ? D.lrun[c0 + lane] : 0ULL;
    const Runs<G> L(hi32(run), lo32(run));
    for (int k0 = (int)blockIdx.y * kWave; k0 < L.pre[G]; k0 += D.list_split * kWave) {
        int j, li = 0, key = -1;
        uint32_t src = 0;
        if (k0 + lane < L.pre[G]) {
            li = L.find(k0 + lane, j);
            key = D.lkey[li];
            src = D.lsrc[li];
        }
        scatter_run(D, li, key, src);
    }
}
// the same for the list of the particles that entered
__global__ void __launch_bounds__(256) k_scatter_in(Dev D) {
    const Scalars *sc = D.sc;
    const int l0 = (int)(sc->n_old + sc->n_new), n = (int)sc->n_inj, lane = lane_id();
    for (int k0 = (int)(blockIdx.x * 256 + threadIdx.x - lane); k0 < n; k0 += (int)(gridDim.x * 256)) {
        const int li = l0 + k0 + lane;
        scatter_run(D, li, k0 + lane < n ? D.lkey[li] : -1, k0 + lane < n ? D.lsrc[li] : 0u);
    }
}

// orders this wave's LDS and global accesses (its lanes run together: no barrier needed)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------------------
// Sort of a list of distinct values by the W waves of a block (t: the thread's number among theirs),
// ascending.  Bitonic network whose comparators all put the smaller value first, so entries past
// len behave as +infinity and are never touched.  a may point to LDS or to global memory; only
// these waves touch it.
// ---------------------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void sort_list(unsigned long long *a, int len, int t) {
    constexpr int BS = W * kWave;
    int bad = 0;
    for (int i = t; i + 1 < len; i += BS) bad |= a[i] > a[i + 1];
    if (W == 1 ? !__any(bad) : !__syncthreads_or(bad)) return;
    int N = 1;
    while (N < len) N <<= 1;
    for (int k = 2; k <= N; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const bool flip = j == (k >> 1);
            for (int p = t; p < N / 2; p += BS) {
                const int i = 2 * (p & ~(j - 1)) + (p & (j - 1));
                const int q = flip ? (i ^ (k - 1)) : i + j;
                if (q < len) {
                    const unsigned long long ai = a[i], aq = a[q];
                    if (ai > aq) {
                        a[i] = aq;
                        a[q] = ai;
                    }
                }
            }
            if (W == 1)
                wave_sync();
            else
                __syncthreads();
        }
    }
}
__device__ __forceinline__ void wave_sort(unsigned long long *a, int len) { sort_list<1>(a, len, lane_id()); }

// A bucket of 64 < n <= 256 entries sorted into lds, by its pieces (kHeadBit) if they are at most
// 64: a piece stays together, behind the pieces whose first order is smaller.  tab: local memory
// for 64 pieces.
__device__ __forceinline__ void sort_pieces(const unsigned long long *a, int n, unsigned long long *lds,
                                            unsigned long long *tab) {
    const int lane = lane_id();
    const unsigned long long upto = ~0ULL >> (63 - lane);
    unsigned long long v[4], heads[4];
    int H = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = q * kWave + lane;
        v[q] = k < n ? a[k] : 0ULL;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool head = q * kWave + lane < n && ((unsigned)v[q] & kHeadBit) != 0;
        heads[q] = __ballot(head);
        const int h = H + (int)__popcll(heads[q] & upto) - 1;
        if (head && h < kWave) tab[h] = (v[q] & ~0xFFFFFFFFULL) | (unsigned)(q * kWave + lane);
        H += (int)__popcll(heads[q]);
    }
    wave_sync();
    if (H > kWave) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q * kWave + lane < n) lds[q * kWave + lane] = v[q];
        wave_sync();
        wave_sort(lds, n);
        return;
    }
    // lane h: piece h's first order, place and length; the places of the pieces before it
    const unsigned long long t = lane < H ? tab[lane] : 0ULL;
    const unsigned key = (unsigned)(t >> 32);
    const int pos = lo32(t), nextp = __shfl_down(pos, 1);
    const int len = lane < H ? (lane == H - 1 ? n : nextp) - pos : 0;
    int base = -pos;
    for (int i = 0; i < H; ++i)
        if ((unsigned)__builtin_amdgcn_readlane((int)key, i) < key) base += __builtin_amdgcn_readlane(len, i);
    int before = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = q * kWave + lane;
        const int shift = __shfl(base, before + (int)__popcll(heads[q] & upto) - 1);
        if (k < n) lds[k + shift] = v[q];
        before += (int)__popcll(heads[q]);
    }
    wave_sync();
}

// ---------------------------------------------------------------------------------------
// S6: the buckets.  Part 0, a cell's arrivals (survivors that left another cell, or came back
// to this one after a wall), sorted by their order at the start of the step: their records go
// to the second part of the next buffer (the stayers are in the first already, k_stream) and
// their sums are added to P^{n+1}.  Part 1, the particles that collided elsewhere and end in
// the cell: their sums come off S (E - S is P^{n+1} - (S - collided)).
// One wave takes G consecutive cells: runs of cells whose entries fit in 64 lanes together are
// sorted, moved and summed at once (segmented sums, whose order depends only on a particle's
// place in its own bucket); a bucket of more than 64 has the wave to itself.  Which of the
// two a bucket takes depends on its own length alone, so the sums do not depend on the cells
// around it: bitwise reproducible, alone or in a batch.
// ---------------------------------------------------------------------------------------
constexpr int kGatherLds = 256;  // longer lists are sorted in place in global memory
template <typename R, int WPB, bool KE, int G>
__device__ __forceinline__ void gather_cells(const Dev &D, int buf) {
    constexpr int BS = kWave;
    constexpr int CPR = RecChunks<R>::N;
    __shared__ unsigned long long lds_all[WPB][kGatherLds];
    __shared__ uint4 st_all[WPB][kWave * CPR];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
    // blocks go round-robin to the 8 XCDs; give each XCD a contiguous range of cells so that
    // neighbouring cells (whose particles are exchanged) share an L2
    const int nb = (int)gridDim.x, bidx = (int)blockIdx.x;
    const int xcd = bidx & 7, q8 = nb >> 3, rr = nb & 7;
    const int c0 = ((xcd * q8 + (xcd < rr ? xcd : rr) + (bidx >> 3)) * WPB + wave) * G;
    const int nc = D.nc;
    if (c0 >= nc || D.sc->none) return;
    unsigned long long *lds = lds_all[wave];
    uint4 *st = st_all[wave];
    const Particles src = D.pa[buf], dst = D.pa[buf ^ 1];
    const long long span = D.sc->span[buf ^ 1];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const unsigned long long *off = D.off + (part == 0 ? 0 : nc);
        double *to = part == 0 ? D.P : D.S;
        int my_first = 0, my_len = 0;
        if (lane < G && c0 + lane < nc) {
            my_first = lo32(off[c0 + lane]);
            my_len = lo32(off[c0 + lane + 1]) - my_first;
        }
        const Runs<G> L(my_first, my_len);  // the G buckets are consecutive in perm
        const int a0 = L.first[0];
        int g = 0;
        while (g < G) {
            // wave-uniform: the longest run [g, h) of buckets whose entries fit in 64 lanes
            int h = g + 1, pg = 0, ph = 0;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if (j == g) {
                    pg = L.pre[j];
                    ph = L.pre[j + 1];
                }
                if (j == h && j > g && L.pre[j + 1] - pg <= BS) {
                    h = j + 1;
                    ph = L.pre[j + 1];
                }
            }
            const int nr = ph - pg;
            if (nr > 0 && nr <= BS) {
                // this lane's bucket j and its first and last lane
                int j = g, first = 0, last = 0;
#pragma unroll
                for (int i = 0; i < G; ++i)
                    if (i >= g && i < h && L.pre[i] - pg <= lane && L.pre[i + 1] - pg > lane) {
                        j = i;
                        first = L.pre[i] - pg;
                        last = L.pre[i + 1] - pg - 1;
                    }
                const bool act = lane < nr;
                if (!act) first = last = lane;
                // Place in the bucket: a piece (kHeadBit) stays together, behind the pieces of the
                // bucket whose first order is smaller.  A cell's particles come from a handful of
                // cells, so these are a handful of comparisons (a bitonic network over 64
                // entries needs 21 exchanges).
                const unsigned long long v = act ? D.perm[a0 + pg + lane] : 0ULL;
                unsigned long long todo = __ballot(act && ((unsigned)v & kHeadBit) != 0);
                const int my_head = act ? 63 - __clzll((long long)(todo & (~0ULL >> (63 - lane)))) : lane;
                const unsigned key = (unsigned)__shfl((int)(v >> 32), my_head);
                int r = first + (lane - my_head);
                while (todo) {
                    const int h = __ffsll((long long)todo) - 1;
                    todo &= todo - 1;
                    const int next = todo ? __ffsll((long long)todo) - 1 : nr;
                    const unsigned kh = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), h);
                    // a piece lies in one bucket, but its successor here may be another bucket's
                    if (h >= first && h <= last && kh < key) r += next - h;
                }
                if (act) lds[r] = v;
                wave_sync();
                Part<R> A;
                double acc[5] = {0, 0, 0, 0, 0};
                if (act) {
                    load_part<KE>(src, (long long)(lo32(lds[lane]) & ~kHeadBit), A);
                    add_phi<R>(acc, A.m, A.u, A.e);
                }
                if (part == 0) {
                    const int pl = a0 + pg;
                    const bool wrap = (long long)pl + nr > D.cap - span;
                    if (act) {
                        const int o = wrap ? slot_of(D, buf ^ 1, span, pl + lane) : (int)span + pl + lane;
                        store_side<KE>(dst, o, A);
                        if (wrap)
                            stage_part(rec_chunks(dst, o, R(0)), A);
                        else
                            stage_part(st + lane * CPR, A);
                    }
                    if (!wrap) {
                        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                        uint4 *gp = rec_chunks(dst, span + pl, R(0));
                        for (int k = lane; k < nr * CPR; k += BS) st_nt(&gp[k], st[k]);
                    }
                }
                double pv[5];
                const int c = c0 + j;
                const bool end = act && lane == last;
                if (end) {
#pragma unroll
                    for (int k = 0; k < 5; ++k) pv[k] = to[k * nc + c];
                }
#pragma unroll
                for (int k = 0; k < 5; ++k) acc[k] = seg_sum(acc[k], first, last);
                if (end) {
#pragma unroll
                    for (int k = 0; k < 5; ++k) to[k * nc + c] = part == 0 ? pv[k] + acc[k] : pv[k] - acc[k];
                }
                wave_sync();
            } else if (nr > kGatherLds && D.long_from < kNoLong) {
                // k_gather_long's
            } else if (nr > 0) {
                // one bucket of more than 64
                const int pl = a0 + pg;
                unsigned long long *list = D.perm + pl;
                if (nr <= kGatherLds) {
                    sort_pieces(list, nr, lds, reinterpret_cast<unsigned long long *>(st));
                    list = lds;
                } else {
                    wave_sort(list, nr);
                }
                double acc[5] = {0, 0, 0, 0, 0};
                for (int k0 = 0; k0 < nr; k0 += BS) {
                    const int k = k0 + lane;
                    if (k < nr) {
                        Part<R> A;
                        load_part<KE>(src, (long long)(lo32(list[k]) & ~kHeadBit), A);
                        add_phi<R>(acc, A.m, A.u, A.e);
                        if (part == 0) {
                            store_side<KE>(dst, slot_of(D, buf ^ 1, span, pl + k), A);
                            stage_part(st + lane * CPR, A);
                        }
                    }
                    if (part == 0) {
                        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                        const int m = min(BS, nr - k0);
                        for (int i = lane; i < m * CPR; i += BS)
                            st_nt(&rec_chunks(dst, slot_of(D, buf ^ 1, span, pl + k0 + i / CPR), R(0))[i % CPR], st[i]);
                        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    }
                }
#pragma unroll
                for (int k = 0; k < 5; ++k) acc[k] = wave_sum(acc[k]);
                double ak = acc[0];
#pragma unroll
                for (int k = 1; k < 5; ++k)
                    if (lane == k) ak = acc[k];
                if (lane < 5) to[lane * nc + c0 + g] = part == 0 ? to[lane * nc + c0 + g] + ak : to[lane * nc + c0 + g] - ak;
                wave_sync();
            }
            g = h;
        }
    }
}

template <typename R, int WPB, bool KE>
__global__ void __launch_bounds__(WPB * 64) k_gather(Dev D, int buf) {
    gather_cells<R, WPB, KE, kListCellsDense>(D, buf);
}
template <typename R, int WPB, bool KE>
__global__ void __launch_bounds__(WPB * 64) k_gather_sparse(Dev D, int buf) {
    gather_cells<R, WPB, KE, kListCellsSparse>(D, buf);
}

// The buckets of more than kGatherLds entries where a block may share a cell's transport (k_stream_long): a
// block each, its waves taking the runs of 64 in turn, the terms of the sums added lane by lane in
// the runs' order as one wave adds them.  What bounds a wave alone there is the sort (78 passes
// over 4,096 entries in global memory); here up to kLongSort entries are sorted in local memory.
// 64 boxes of 10,000 particles: 330 us in k_gather, 33 here.
constexpr int kLongSort = 4096, kSortWaves = 8;
template <typename R, bool KE>
__global__ void __launch_bounds__(kSortWaves * kWave) k_gather_long(Dev D, int buf) {
    __shared__ unsigned long long lds[kLongSort];
    __shared__ double terms[kSortWaves][5][kWave];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
    const int c = (int)blockIdx.x, nc = D.nc;
    if (D.sc->none) return;
    const Particles src = D.pa[buf], dst = D.pa[buf ^ 1];
    const long long span = D.sc->span[buf ^ 1];
    for (int part = 0; part < 2; ++part) {
        const unsigned long long *off = D.off + (part == 0 ? 0 : nc);
        const int first = lo32(off[c]), nr = lo32(off[c + 1]) - first;
        if (nr <= kGatherLds) continue;
        unsigned long long *list = D.perm + first;
        if (nr <= kLongSort) {
            for (int k = threadIdx.x; k < nr; k += kSortWaves * kWave) lds[k] = list[k];
            __syncthreads();
            list = lds;
        }
        sort_list<kSortWaves>(list, nr, (int)threadIdx.x);
        double mine = 0.0;  // the sum that this wave keeps: component w
        for (int k0 = 0; k0 < nr; k0 += kSortWaves * kWave) {
            const int k = k0 + w * kWave + lane;
            double t[5] = {0, 0, 0, 0, 0};
            if (k < nr) {
                Part<R> A;
                load_part<KE>(src, (long long)(lo32(list[k]) & ~kHeadBit), A);
                add_phi<R>(t, A.m, A.u, A.e);
                if (part == 0) {
                    const int o = slot_of(D, buf ^ 1, span, first + k);
                    store_side<KE>(dst, o, A);
                    stage_part(rec_chunks(dst, o, R(0)), A);
                }
            }
#pragma unroll
            for (int i = 0; i < 5; ++i) terms[w][i][lane] = t[i];
            __syncthreads();
            if (w < 5) {
#pragma unroll
                for (int i = 0; i < kSortWaves; ++i) mine += terms[i][w][lane];
            }
            __syncthreads();  // (read before the next round's are written)
        }
        if (w < 5) {
            mine = wave_sum(mine);
            double *to = (part == 0 ? D.P : D.S) + w * nc + c;
            if (lane == 0) *to = part == 0 ? *to + mine : *to - mine;
        }
    }
}

// the particles between two steps in their order (arrivals, stayers, cell by cell), one after
// the other in the other buffer
template <typename R, bool KE>
__global__ void __launch_bounds__(256) k_pack(Dev D, int buf) {
    const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (c >= D.nc) return;
    const unsigned long long o0 = D.off[c], o1 = D.off[c + 1];
    const int n = hi32(o1) - hi32(o0), nm = lo32(o1) - lo32(o0), m0 = lo32(o0), v0 = D.v0[buf][c];
    const long long span = D.sc->span[buf];
    const Particles pa = D.pa[buf], pb = D.pa[buf ^ 1];
    for (int k = lane_id(); k < n; k += kWave) {
        Part<R> q;
        load_part<KE>(pa, k < nm ? slot_of(D, buf, span, m0 + k) : v0 + (k - nm), q);
        const long long o = hi32(o0) + k;
        stage_part(rec_chunks(pb, o, R(0)), q);
        store_side<KE>(pb, o, q);
    }
}

// the step's bookkeeping, one block
__device__ __forceinline__ void finalize(const Dev &D) {
    __shared__ unsigned long long red[2][kWallSeg];
    Scalars *s = D.sc;
    const long long n_old = s->n_old, n_new = s->n_new, n_inj = s->n_inj;
    const long long n_tot = n_old + n_new + n_inj;
    if (threadIdx.x < kWallSeg) {
        red[0][threadIdx.x] = D.spart[threadIdx.x];
        red[1][threadIdx.x] = D.spart[kWallSeg + threadIdx.x];
    }
    __syncthreads();
    for (int h = kWallSeg / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] += red[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    // per instance: its particles occupy the buckets of its cell range, its old ones are those
    // the step before left, its new ones the sampled and entering ranges of its cells and
    // far-field faces; then its own clock advances
    const int nc = D.nc;
    for (int k = threadIdx.x; k < D.n_inst; k += blockDim.x) {
        const InstP &P = D.ip[k];
        InstS &I = D.is[k];
        const long long alive = hi32(D.off[P.cell1]) - hi32(D.off[P.cell0]);
        const long long coll = hi32(D.off[nc + P.cell1]) - hi32(D.off[nc + P.cell0]);
        const long long old = I.n_alive;
        const long long smp = n_new > 0 ? D.samoff[P.cell1] - D.samoff[P.cell0] : 0;
        const long long inj = (n_inj > 0 && P.ff1 > P.ff0) ? D.injoff[P.ff1] - D.injoff[P.ff0] : 0;
        const long long tot = old + smp + inj;
        I.n_alive = alive;
        I.n_collided = coll;
        I.n_escaped = tot - alive - coll;
        I.n_sampled = smp;
        I.n_injected = inj;
        I.moved_total = I.moved_total + tot;
        I.t = I.t + I.dt;
        I.step = I.step + 1;
        for (int i = 0; i < D.dt_slots; ++i) *dt_slot(D, k, i) = 0x7FF0000000000000ULL;
    }
    if (threadIdx.x == 0) {
        const long long alive = hi32(D.off[nc]);
        const long long ended = hi32(D.off[2 * nc]);
        s->n_cross = red[0][0];
        s->n_wall = red[1][0];
        s->n_collided = (unsigned long long)(ended - alive);
        s->n_escaped = (unsigned long long)(n_tot - ended);
        s->moved_total = s->moved_total + (unsigned long long)n_tot;
        s->n_alive = alive;
        s->n_old = alive;
        s->n_mov = lo32(D.off[nc]);
        s->n_new = 0;
        s->n_inj = 0;
        s->t = s->t + s->dt;
        s->step = s->step + 1;
    }
}

// S6: W^{n+1} = W^n + (-sum_f s_f Phi_f + E - S) / Omega, one thread per cell; E - S is P^{n+1}
// minus what k_stream and the gather left of S.  In a step with no particle anywhere (none is
// left, sampled or let in) no kernel between the preparation and this one does anything: then
// P^{n+1} = 0 and S = P^n.
// The last block keeps the step's books meanwhile: nothing that it writes is read by the others.
__global__ void __launch_bounds__(256) k_update(Dev D) {
    if (blockIdx.x == gridDim.x - 1) {
        finalize(D);
        return;
    }
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= D.nc) return;
    const bool none = D.sc->none != 0;
    const int nc = D.nc, nf = D.nf, nfc = D.nfc[c];
    int codes[6];
#pragma unroll
    for (int lf = 0; lf < 6; ++lf) codes[lf] = lf < nfc ? D.cface[c * 6 + lf] : 0;
    const double vol = D.vol[c];
    // every load before the first store (the stores could alias them as far as the compiler
    // knows, which would otherwise keep one round trip per component)
    double ph[5][6], pv[5], sv[5], wv[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
#pragma unroll
        for (int lf = 0; lf < 6; ++lf) {
            const int cd = codes[lf];
            const int f = (cd > 0 ? cd : -cd) - 1;
            ph[k][lf] = lf < nfc ? D.Phi[k * nf + f] : 0.0;
        }
        pv[k] = D.P[k * nc + c];
        sv[k] = D.S[k * nc + c];
        wv[k] = D.W[k * nc + c];
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        double facc = 0.0;
#pragma unroll
        for (int lf = 0; lf < 6; ++lf)  // (unrolled: arrays indexed at run time would live in scratch memory)
            if (lf < nfc) facc = facc - (codes[lf] > 0 ? ph[k][lf] : -ph[k][lf]);
        const double acc = facc + (none ? 0.0 - pv[k] : pv[k] - sv[k]);
        D.W[k * nc + c] = wv[k] + acc / vol;
        if (none) D.P[k * nc + c] = 0.0;
    }
}

// ---------------------------------------------------------------------------------------
// exclusive scan (integers, deterministic): out[i] = sum_{j<i} in[j], out[n] = total
// ---------------------------------------------------------------------------------------
constexpr int kScanBS = 256, kScanPer = 8, kScanTile = kScanBS * kScanPer;
static_assert(kScanTile % kCountBS == 0);

// exclusive prefix over the block's threads
template <typename T, int BS>
__device__ T block_exclusive_scan(T v, T *sh, T &total) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    T incl = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const T t = __shfl_up(incl, d);
        if (lane >= d) incl = incl + t;
    }
    __syncthreads();  // (sh may still be read from the call before)
    if (lane == kWave - 1) sh[wave] = incl;
    __syncthreads();
    T before = T(0);
    total = T(0);
#pragma unroll
    for (int w = 0; w < BS / kWave; ++w) {
        const T t = sh[w];
        if (w < wave) before = before + t;
        total = total + t;
    }
    return before + incl - v;
}
template <typename T, int BS>
__device__ T block_total(T v, T *sh) {
    T total;
    block_exclusive_scan<T, BS>(v, sh, total);
    return total;
}

// The counts' prefixes, a tile per block: an offset is the sum of k_cell_prep's block sums before
// the tile (a few thousand at most, from the L2).  The last block checks the capacity of the step
// (old + sampled + entering must fit) and sets its counts.
__global__ void __launch_bounds__(kScanBS) k_offsets(Dev D, int buf) {
    __shared__ long long sh[kScanBS / kWave];
    const int tc = (D.nc + kScanTile - 1) / kScanTile, ti = (D.nff + kScanTile - 1) / kScanTile;
    const int gc = (D.nc + kCountBS - 1) / kCountBS, gi = (D.nff + kCountBS - 1) / kCountBS;
    const int tile = blockIdx.x;
    auto sum_of = [&](const long long *part, int n) {
        long long o = 0;
        for (int b = threadIdx.x; b < n; b += kScanBS) o += part[b];
        return block_total<long long, kScanBS>(o, sh);
    };
    if (tile == tc + ti) {
        const long long nn = sum_of(D.scan64, gc), ni = sum_of(D.scan64 + gc, gi);
        if (threadIdx.x != 0) return;
        Scalars *s = D.sc;
        const bool fits = s->n_old + nn + ni <= D.cap;
        if (!fits) atomicOr(&s->err, kErrCapacity);
        s->n_new = fits ? nn : 0;
        s->n_inj = fits ? ni : 0;
        s->none = s->n_old + s->n_new + s->n_inj == 0 ? 1u : 0u;
        s->n_sampled = (unsigned long long)s->n_new;
        s->n_injected = (unsigned long long)s->n_inj;
        // the next buffer's regions: a cell's is as long as its old and new particles are many
        s->span[buf ^ 1] = s->n_old + s->n_new;
        D.v0[buf ^ 1][D.nc] = (int32_t)(s->n_old + s->n_new);
        return;
    }
    const bool cells = tile < tc;
    const int t = cells ? tile : tile - tc;
    const long long *in = cells ? D.nsam : D.ninj, *part = cells ? D.scan64 : D.scan64 + gc;
    long long *out = cells ? D.samoff : D.injoff;
    const long long n = cells ? D.nc : D.nff;
    const long long base = (long long)t * kScanTile + (long long)threadIdx.x * kScanPer;
    long long v[kScanPer], s = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) v[q] = base + q < n ? in[base + q] : 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) s += v[q];
    const long long off = sum_of(part, t * (kScanTile / kCountBS));
    long long tot;
    long long ex = block_exclusive_scan<long long, kScanBS>(s, sh, tot) + off;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        if (base + q < n) out[base + q] = ex;
        ex += v[q];
    }
    if (t == (cells ? tc : ti) - 1 && threadIdx.x == 0) out[n] = off + tot;
}

// The prefix of the bucket sizes (all particles of the bucket in the high word, those listed in
// perm in the low one; neither total reaches 2^31).  Up to 8,192 buckets: one launch of one block
// of 1,024 threads (5,418 buckets: 4.0 us against 7.6 in two launches).  More: the tiles' totals
// first (65,536 buckets: 8.9 us; eight such blocks, each summing all that is before its own tile,
// took 15.5).
__device__ __forceinline__ unsigned long long bucket(unsigned long long v) { return v + (v << 32); }

constexpr int kSmallBS = 1024, kSmallPer = 8;
constexpr long long kScanSmall = kSmallBS * kSmallPer;

__global__ void __launch_bounds__(kSmallBS) k_scan_small(const unsigned long long *in, long long n,
                                                         unsigned long long *out) {
    __shared__ unsigned long long sh[kSmallBS / kWave];
    const long long first = (long long)threadIdx.x * kSmallPer;
    unsigned long long v[kSmallPer], s = 0;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) v[q] = first + q < n ? bucket(in[first + q]) : 0;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) s += v[q];
    unsigned long long tot;
    unsigned long long ex = block_exclusive_scan<unsigned long long, kSmallBS>(s, sh, tot);
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        if (first + q < n) out[first + q] = ex;
        ex += v[q];
    }
    if (threadIdx.x == 0) out[n] = tot;
}

__global__ void __launch_bounds__(kScanBS) k_scan_reduce(const unsigned long long *in, long long n,
                                                         unsigned long long *part) {
    __shared__ unsigned long long sh[kScanBS / kWave];
    const long long base = (long long)blockIdx.x * kScanTile + threadIdx.x;
    unsigned long long s = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) s += base + q * kScanBS < n ? bucket(in[base + q * kScanBS]) : 0;
    const unsigned long long tot = block_total<unsigned long long, kScanBS>(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Each block finds its own offset, the totals of the blocks before it (a few thousand at
// most, read from the L2), so no kernel in between scans the block totals; the last block
// writes the grand total to out[n].  Integer sums: the order does not matter.
__global__ void __launch_bounds__(kScanBS) k_scan_apply(const unsigned long long *in, long long n,
                                                        const unsigned long long *part, unsigned long long *out) {
    __shared__ unsigned long long sh[kScanBS / kWave];
    const long long base = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanPer;
    unsigned long long v[kScanPer], s = 0, o = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) v[q] = base + q < n ? bucket(in[base + q]) : 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kScanBS) o += part[b];
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) s += v[q];
    const unsigned long long off = block_total<unsigned long long, kScanBS>(o, sh);
    unsigned long long tot;
    unsigned long long ex = block_exclusive_scan<unsigned long long, kScanBS>(s, sh, tot) + off;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        if (base + q < n) out[base + q] = ex;
        ex += v[q];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = off + tot;
}

__global__ void k_fill(double *p, long long n, double v) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------------------
// Time averaging for steady states (Sec. 2.4(c)): over the steps n > N_avg of an instance,
// Wbar = A / D with A = sum dt^n W^n per cell and D = sum dt^n, and the relative change of
// Wbar in a step, sum_c Omega_c sum_k |Wbar^n - Wbar^{n-1}| / sum_c Omega_c sum_k |Wbar^n|
// (+infinity until two steps are averaged).  k_avg_cells: kAvgBlocks blocks per instance,
// each a contiguous run of its cells, fixed per-thread assignment and reduction tree;
// k_avg_fin: one wave per instance sums its blocks' partials and advances D.  Both run after
// k_update (the instance's step counter and dt are those of the step just taken).
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_avg_cells(Dev D) {
    __shared__ double red[2][256];
    const int inst = (int)blockIdx.x / kAvgBlocks, j = (int)blockIdx.x % kAvgBlocks;
    const InstS &I = D.is[inst];
    if (I.step <= D.avg_from) return;
    const InstP &P = D.ip[inst];
    const int nc = D.nc, t = (int)threadIdx.x;
    const int n = P.cell1 - P.cell0, chunk = (n + kAvgBlocks - 1) / kAvgBlocks;
    const int c0 = P.cell0 + j * chunk, c1 = min(P.cell1, c0 + chunk);
    const double dt = I.dt, d0 = I.avg_D, d1 = d0 + dt;
    const bool prev = I.avg_n > 0;
    double diff = 0.0, mag = 0.0;
    for (int c = c0 + t; c < c1; c += 256) {
        double dc = 0.0, mc = 0.0;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const double a0 = D.avgA[(long long)k * nc + c];
            const double a1 = a0 + dt * D.W[(long long)k * nc + c];
            D.avgA[(long long)k * nc + c] = a1;
            const double wb1 = a1 / d1;
            mc = mc + fabs(wb1);
            if (prev) dc = dc + fabs(wb1 - a0 / d0);
        }
        const double vol = D.vol[c];
        mag = mag + vol * mc;
        diff = diff + vol * dc;
    }
    red[0][t] = diff;
    red[1][t] = mag;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            red[0][t] = red[0][t] + red[0][t + h];
            red[1][t] = red[1][t] + red[1][t + h];
        }
        __syncthreads();
    }
    if (t < 2) D.avgpart[2 * (long long)blockIdx.x + t] = red[t][0];
}

__global__ void __launch_bounds__(64) k_avg_fin(Dev D) {
    const int inst = (int)blockIdx.x, lane = lane_id();
    InstS &I = D.is[inst];
    if (I.step <= D.avg_from) return;
    double diff = 0.0, mag = 0.0;
    for (int b = lane; b < kAvgBlocks; b += kWave) {
        diff = diff + D.avgpart[2 * ((long long)inst * kAvgBlocks + b)];
        mag = mag + D.avgpart[2 * ((long long)inst * kAvgBlocks + b) + 1];
    }
    diff = wave_sum(diff);
    mag = wave_sum(mag);
    if (lane == 0) {
        I.avg_res = I.avg_n > 0 ? diff / mag : __builtin_inf();
        I.avg_D = I.avg_D + I.dt;
        I.avg_n = I.avg_n + 1;
    }
}

// Wbar = A / D into out, [nc][5]
__global__ void k_avg_out(Dev D, double *out) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= D.nc) return;
    const double d = D.is[inst_of(D, c)].avg_D;
    for (int k = 0; k < 5; ++k) out[5 * (long long)c + k] = D.avgA[(long long)k * D.nc + c] / d;
}

// field output for ugkwp_moments, [nc][5] in out
__global__ void k_moments(Dev D, int which, double *out) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= D.nc) return;
    const int nc = D.nc;
    const double vol = D.vol[c];
    double W[5], P[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        W[k] = D.W[k * nc + c];
        P[k] = D.P[k * nc + c] / vol;
    }
    double o[5];
    if (which == 0) {
        for (int k = 0; k < 5; ++k) o[k] = W[k];
    } else if (which == 1) {
        for (int k = 0; k < 5; ++k) o[k] = P[k];
    } else if (which == 2) {
        for (int k = 0; k < 5; ++k) o[k] = W[k] - P[k];
    } else {
        const double rho = W[0];
        o[0] = rho;
        o[1] = W[1] / rho;
        o[2] = W[2] / rho;
        o[3] = W[3] / rho;
        o[4] = temp_k(W, D.K);
    }
    for (int k = 0; k < 5; ++k) out[5 * c + k] = o[k];
}

// A new state from W0 [nc][5] (already in device memory): its check, each block's first bad cell to
// `bad` (LLONG_MAX: none), and if no block found one, every array that a run starts from.  With a
// bad cell nothing is written and the state before stays.
__global__ void __launch_bounds__(kCountBS) k_check_state(Dev D, const double *W0, long long *bad) {
    __shared__ int first;
    if (threadIdx.x == 0) first = kCountBS;
    __syncthreads();
    const int c = blockIdx.x * kCountBS + threadIdx.x;
    if (c < D.nc) {
        const double *w = W0 + 5LL * c;
        const double rho = w[0];
        const double T = (2.0 / (3.0 + D.K)) * (w[4] - 0.5 * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]) / rho) / rho;
        if (!(rho > 0.0) || !(T > 0.0) || !isfinite(rho) || !isfinite(T)) atomicMin(&first, (int)threadIdx.x);
    }
    __syncthreads();
    if (threadIdx.x == 0)
        bad[blockIdx.x] = first < kCountBS ? (long long)blockIdx.x * kCountBS + first : 0x7FFFFFFFFFFFFFFFLL;
}
__global__ void __launch_bounds__(kCountBS) k_take_state(Dev D, const double *W0, const long long *bad, long long *worst) {
    __shared__ long long sm[kCountBS / kWave];
    const int gc = (D.nc + kCountBS - 1) / kCountBS;
    long long m = 0x7FFFFFFFFFFFFFFFLL;
    for (int b = threadIdx.x; b < gc; b += kCountBS) m = min(m, bad[b]);
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) m = min(m, __shfl_xor(m, d));
    if (lane_id() == 0) sm[threadIdx.x / kWave] = m;
    __syncthreads();
    for (int w = 0; w < kCountBS / kWave; ++w) m = min(m, sm[w]);
    const long long i = (long long)blockIdx.x * kCountBS + threadIdx.x;
    if (i == 0) *worst = m;
    if (m != 0x7FFFFFFFFFFFFFFFLL) return;
    const long long nc = D.nc, all = (long long)gridDim.x * kCountBS;
    if (i < nc) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            D.W[k * nc + i] = W0[5 * i + k];
            D.P[k * nc + i] = 0.0;
            D.avgA[k * nc + i] = 0.0;
        }
        D.v0[0][i] = 0;
        D.v0[1][i] = 0;
        D.off[i] = 0ULL;
        D.off[nc + i] = 0ULL;
    }
    if (i == 0) {
        D.v0[0][nc] = 0;
        D.v0[1][nc] = 0;
        D.off[2 * nc] = 0ULL;
    }
    for (long long k = i; k < (long long)D.n_inst * D.dt_slots * D.dt_stride; k += all) D.dtmin[k] = 0x7FF0000000000000ULL;
    uint32_t *const is = reinterpret_cast<uint32_t *>(D.is), *const sc = reinterpret_cast<uint32_t *>(D.sc);
    for (long long k = i; k < (long long)(D.n_inst * (sizeof(InstS) / 4)); k += all) is[k] = 0u;
    for (long long k = i; k < (long long)(sizeof(Scalars) / 4); k += all) sc[k] = 0u;
}

// prefix of the bucket sizes into D.off
void scan_buckets(const Dev &D, hipStream_t s) {
    const long long n = 2LL * D.nc;
    if (n <= kScanSmall) {
        k_scan_small<<<1, kSmallBS, 0, s>>>(D.cnt64, n, D.off);
        return;
    }
    const unsigned nb = (unsigned)((n + kScanTile - 1) / kScanTile);
    k_scan_reduce<<<nb, kScanBS, 0, s>>>(D.cnt64, n, D.scan32);
    k_scan_apply<<<nb, kScanBS, 0, s>>>(D.cnt64, n, D.scan32, D.off);
}
// counts of the new particles and their offsets
void count_new(const Dev &D, int buf, hipStream_t s, Prof *pr) {
    const int gc = (D.nc + kCountBS - 1) / kCountBS, gi = (D.nff + kCountBS - 1) / kCountBS;
    pr->begin(kSlotCellPrep);
    k_cell_prep<<<(unsigned)(gc + gi), kCountBS, 0, s>>>(D);
    pr->end(kSlotCellPrep);
    pr->begin(kSlotScan);
    const int tc = (D.nc + kScanTile - 1) / kScanTile, ti = (D.nff + kScanTile - 1) / kScanTile;
    k_offsets<<<(unsigned)(tc + ti + 1), kScanBS, 0, s>>>(D, buf);
    pr->end(kSlotScan);
}

}  // namespace

int long_from(long long nc, long long per_cell) {
    const bool few = nc <= 1024 ? per_cell >= 400 : nc <= 4096 && per_cell >= 1000;
    return few ? kLongCell : kNoLong;
}
int list_split(long long nc, bool sparse, long long per_cell) {
    // some 30% of a cell's particles meet a face; 4,096 waves fill the chip (64 boxes of 10,000
    // particles: k_track 326 us with one row, 26 with 94, k_scatter 51 and 11)
    const int g = sparse ? kListCellsSparse : kListCellsDense;
    const long long waves = (nc + g - 1) / g, runs = (3 * per_cell * g / 10 + kWave - 1) / kWave;
    return (int)std::max(1LL, std::min({runs, 4096 / waves, 256LL}));
}

long long scan_partials_needed(long long n) { return (n + kScanTile - 1) / kScanTile + 1; }
long long count_partials_needed(long long nc, long long nff) {
    return (nc + kCountBS - 1) / kCountBS + (nff + kCountBS - 1) / kCountBS;
}


void launch_take_state(const Dev &D, const double *W0, long long *worst, hipStream_t s) {
    const unsigned g = (unsigned)((D.nc + kCountBS - 1) / kCountBS);
    k_check_state<<<g, kCountBS, 0, s>>>(D, W0, D.scan64);
    k_take_state<<<g, kCountBS, 0, s>>>(D, W0, D.scan64, worst);
}

void launch_fill_f64(double *p, long long n, double v, hipStream_t s) {
    if (n > 0) k_fill<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, n, v);
}

namespace {
template <typename R, bool MULTI, int ILP>
void launch_stream_i(const Dev &D, int buf, int bs, hipStream_t s) {
    const unsigned g = (unsigned)((D.nc + bs / kWave - 1) / (bs / kWave));
    if (D.K > 0 && bs == 128)
        k_stream_e<R, 128, MULTI, ILP><<<g, 128, 0, s>>>(D, buf);
    else if (D.K > 0 && bs == 512)
        k_stream_e<R, 512, MULTI, ILP><<<g, 512, 0, s>>>(D, buf);
    else if (D.K > 0)
        k_stream_e<R, 256, MULTI, ILP><<<g, 256, 0, s>>>(D, buf);
    else if (bs == 128)
        k_stream<R, 128, MULTI, ILP><<<g, 128, 0, s>>>(D, buf);
    else if (bs == 512)
        k_stream<R, 512, MULTI, ILP><<<g, 512, 0, s>>>(D, buf);
    else
        k_stream<R, 256, MULTI, ILP><<<g, 256, 0, s>>>(D, buf);
}

// the transport of the cells that k_stream leaves to blocks
template <typename R, bool MULTI>
void launch_stream_long(const Dev &D, int buf, hipStream_t s) {
    if (D.long_from == kNoLong) return;
    const unsigned g = (unsigned)D.nc;
    if (D.K > 0)
        k_stream_long<R, MULTI, true><<<g, kLongWaves * kWave, 0, s>>>(D, buf);
    else
        k_stream_long<R, MULTI, false><<<g, kLongWaves * kWave, 0, s>>>(D, buf);
}

// blocks of the kernels that take several cells per wave
unsigned list_grid(const Dev &D, int waves = 4) {
    const int per = waves * (D.list_sparse ? kListCellsSparse : kListCellsDense);
    return (unsigned)((D.nc + per - 1) / per);
}
// The same over the lists, whose runs of 64 entries are independent of one another: D.list_split
// rows of waves take them in turn (one unless a few cells hold long lists).
dim3 list_grid_runs(const Dev &D) { return dim3(list_grid(D), (unsigned)D.list_split); }

template <typename R, bool KE, int MESH>
void launch_track_m(const Dev &D, int buf, hipStream_t s) {
    if (D.nff > 0) k_stream_in<R, KE, MESH><<<256, 256, 0, s>>>(D, buf);
    if (D.list_sparse)
        k_track<R, KE, MESH, kListCellsSparse><<<list_grid_runs(D), 256, 0, s>>>(D, buf);
    else
        k_track<R, KE, MESH, kListCellsDense><<<list_grid_runs(D), 256, 0, s>>>(D, buf);
}

template <typename R, bool KE>
void launch_track(const Dev &D, int buf, hipStream_t s) {
    if (D.all_box)
        launch_track_m<R, KE, 1>(D, buf, s);
    else if (D.all_tet)
        launch_track_m<R, KE, 2>(D, buf, s);
    else
        launch_track_m<R, KE, 0>(D, buf, s);
}

// the transport: flights that meet no face, those of the entering particles, the others
template <typename R>
void launch_stream(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s) {
    if (D.n_inst > 1 && cfg.stream_ilp == 2)
        launch_stream_i<R, true, 2>(D, buf, cfg.stream_bs, s);
    else if (D.n_inst > 1)
        launch_stream_i<R, true, 1>(D, buf, cfg.stream_bs, s);
    else if (cfg.stream_ilp == 2)
        launch_stream_i<R, false, 2>(D, buf, cfg.stream_bs, s);
    else
        launch_stream_i<R, false, 1>(D, buf, cfg.stream_bs, s);
    if (D.n_inst > 1)
        launch_stream_long<R, true>(D, buf, s);
    else
        launch_stream_long<R, false>(D, buf, s);
    if (D.K > 0)
        launch_track<R, true>(D, buf, s);
    else
        launch_track<R, false>(D, buf, s);
}

template <typename R>
void launch_gather_long(const Dev &D, int buf, hipStream_t s) {
    if (D.long_from == kNoLong) return;
    if (D.K > 0)
        k_gather_long<R, true><<<(unsigned)D.nc, kSortWaves * kWave, 0, s>>>(D, buf);
    else
        k_gather_long<R, false><<<(unsigned)D.nc, kSortWaves * kWave, 0, s>>>(D, buf);
}

void launch_scatter(const Dev &D, hipStream_t s) {
    if (D.list_sparse)
        k_scatter<kListCellsSparse><<<list_grid_runs(D), 256, 0, s>>>(D);
    else
        k_scatter<kListCellsDense><<<list_grid_runs(D), 256, 0, s>>>(D);
    if (D.nff > 0) k_scatter_in<<<256, 256, 0, s>>>(D);
}

template <typename R, bool KE, int G>
void launch_sample_g(const Dev &D, int buf, int w, hipStream_t s) {
    const unsigned g = (unsigned)((D.nc + w * G - 1) / (w * G));
    if (w == 1)
        k_sample<R, 1, KE, G><<<g, 64, 0, s>>>(D, buf);
    else if (w == 2)
        k_sample<R, 2, KE, G><<<g, 128, 0, s>>>(D, buf);
    else if (w == 8)
        k_sample<R, 8, KE, G><<<g, 512, 0, s>>>(D, buf);
    else
        k_sample<R, 4, KE, G><<<g, 256, 0, s>>>(D, buf);
}

// the cells of at most 64 new pairs, then those with more
template <typename R, bool KE>
void launch_sample_k(const Dev &D, int buf, int w, hipStream_t s) {
    if (D.nc >= kSampleCellsMin)
        launch_sample_g<R, KE, kSampleCells>(D, buf, w, s);
    else
        launch_sample_g<R, KE, 1>(D, buf, w, s);
    // at most a wave per cell; a grid of a few thousand waves takes any list in turns
    const unsigned gb = (unsigned)std::min<long long>((D.nc + 7) / 8, 2048);
    k_sample_big<R, KE><<<gb, 512, 0, s>>>(D, buf);
}

template <typename R>
void launch_sample(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s) {
    const int w = cfg.sample_wpb, nc = D.nc;
    if (D.K > 0)
        launch_sample_k<R, true>(D, buf, w, s);
    else
        launch_sample_k<R, false>(D, buf, w, s);
    if (D.gp_any) {
        const unsigned g4 = (unsigned)((nc + 3) / 4);
        if (D.K > 0)
            k_sample_gp<R, true><<<g4, 256, 0, s>>>(D, buf);
        else
            k_sample_gp<R, false><<<g4, 256, 0, s>>>(D, buf);
    }
}

template <typename R>
void launch_flux(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s) {
    const int bs = cfg.flux_bs, nf = D.nf;
    const unsigned g = (unsigned)((nf + bs - 1) / bs);
    if (D.recon_any) {
        // second order: gradients, then the faces of reconstructing instances; the first-order
        // kernel takes the others
        const unsigned gg = (unsigned)((D.nc + kGradCells - 1) / kGradCells);
        if (D.all_tet)
            k_grad<4><<<gg, 5 * kGradCells, 0, s>>>(D);
        else
            k_grad<6><<<gg, 5 * kGradCells, 0, s>>>(D);
        if (nf <= kFluxSplitMax)
            k_flux2_axes<R><<<(unsigned)((nf + kWave - 1) / kWave), 3 * kWave, 0, s>>>(D);
        else if (bs == 64)
            k_flux2<R, 64><<<g, 64, 0, s>>>(D);
        else if (bs == 256)
            k_flux2<R, 256><<<g, 256, 0, s>>>(D);
        else
            k_flux2<R, 128><<<g, 128, 0, s>>>(D);
        if (D.recon_all) return;
    }
    if (bs == 64)
        k_flux<R, 64><<<g, 64, 0, s>>>(D);
    else if (bs == 256)
        k_flux<R, 256><<<g, 256, 0, s>>>(D);
    else
        k_flux<R, 128><<<g, 128, 0, s>>>(D);
}
}  // namespace

void launch_heat(const Dev &D, int buf, hipStream_t s) {
    if (!D.sh_any) return;
    if (D.prec == 1)
        k_heat<float><<<(unsigned)((D.nc + 3) / 4), 256, 0, s>>>(D, buf);
    else
        k_heat<double><<<(unsigned)((D.nc + 3) / 4), 256, 0, s>>>(D, buf);
}

bool launch_cfg_valid(const LaunchCfg &c) {
    const bool sb = (c.stream_bs == 128 || c.stream_bs == 256 || c.stream_bs == 512) &&
                    (c.stream_ilp == 1 || c.stream_ilp == 2);
    const bool sw = c.sample_wpb == 1 || c.sample_wpb == 2 || c.sample_wpb == 4 || c.sample_wpb == 8;
    const bool fb = c.flux_bs == 64 || c.flux_bs == 128 || c.flux_bs == 256;
    return sb && sw && fb;
}

void launch_step(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s, Prof *pr) {
    const int nc = D.nc, nf = D.nf;
    const unsigned gc = (unsigned)((nc + 255) / 256);
    Prof none;
    if (!pr) pr = &none;
    pr->begin(kSlotPrim);
    k_prim_dt<<<gc, 256, 0, s>>>(D);
    pr->end(kSlotPrim);
    count_new(D, buf, s, pr);
    const bool f32 = D.prec == 1;
    pr->begin(kSlotFlux);
    if (nf > 0) {
        if (f32)
            launch_flux<float>(D, buf, cfg, s);
        else
            launch_flux<double>(D, buf, cfg, s);
    }
    pr->end(kSlotFlux);
    pr->begin(kSlotSample);
    if (f32)
        launch_sample<float>(D, buf, cfg, s);
    else
        launch_sample<double>(D, buf, cfg, s);
    if (D.nff > 0) {
        if (f32)
            k_inject<float><<<1024, 256, 0, s>>>(D, buf);
        else
            k_inject<double><<<1024, 256, 0, s>>>(D, buf);
    }
    pr->end(kSlotSample);
    pr->begin(kSlotStream);
    if (f32)
        launch_stream<float>(D, buf, cfg, s);
    else
        launch_stream<double>(D, buf, cfg, s);
    pr->end(kSlotStream);
    pr->begin(kSlotScan2);
    scan_buckets(D, s);
    pr->end(kSlotScan2);
    pr->begin(kSlotScatter);
    launch_scatter(D, s);
    pr->end(kSlotScatter);
    pr->begin(kSlotGather);
    {
        constexpr int WPB = kGatherWaves;
        const unsigned g = list_grid(D, WPB);
        if (D.list_sparse && f32 && D.K > 0)
            k_gather_sparse<float, WPB, true><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (D.list_sparse && f32)
            k_gather_sparse<float, WPB, false><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (D.list_sparse && D.K > 0)
            k_gather_sparse<double, WPB, true><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (D.list_sparse)
            k_gather_sparse<double, WPB, false><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (f32 && D.K > 0)
            k_gather<float, WPB, true><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (f32)
            k_gather<float, WPB, false><<<g, WPB * 64, 0, s>>>(D, buf);
        else if (D.K > 0)
            k_gather<double, WPB, true><<<g, WPB * 64, 0, s>>>(D, buf);
        else
            k_gather<double, WPB, false><<<g, WPB * 64, 0, s>>>(D, buf);
    }
    if (f32)
        launch_gather_long<float>(D, buf, s);
    else
        launch_gather_long<double>(D, buf, s);
    k_update<<<gc + 1, 256, 0, s>>>(D);
    launch_heat(D, buf ^ 1, s);
    pr->end(kSlotGather);
    pr->begin(kSlotFinal);
    if (D.avg_from >= 0) {
        k_avg_cells<<<(unsigned)(D.n_inst * kAvgBlocks), 256, 0, s>>>(D);
        k_avg_fin<<<(unsigned)D.n_inst, 64, 0, s>>>(D);
    }
    pr->end(kSlotFinal);
}

// A wave-only step when no particle exists: no particle is sampled or let in (e = 0 in the
// wave-only phase), so the particle kernels would find nothing to do; the bucket counts (zeroed
// by k_cell_prep) are still scanned so that the offsets are those of empty cells.
void launch_step_wave_only(const Dev &D, int buf, const LaunchCfg &cfg, hipStream_t s, Prof *pr) {
    const int nc = D.nc, nf = D.nf;
    const unsigned gc = (unsigned)((nc + 255) / 256);
    Prof none;
    if (!pr) pr = &none;
    pr->begin(kSlotPrim);
    k_prim_dt<<<gc, 256, 0, s>>>(D);
    pr->end(kSlotPrim);
    count_new(D, buf, s, pr);
    pr->begin(kSlotFlux);
    if (nf > 0) {
        if (D.prec == 1)
            launch_flux<float>(D, buf, cfg, s);
        else
            launch_flux<double>(D, buf, cfg, s);
    }
    pr->end(kSlotFlux);
    pr->begin(kSlotScan2);
    scan_buckets(D, s);
    pr->end(kSlotScan2);
    pr->begin(kSlotGather);
    k_update<<<gc + 1, 256, 0, s>>>(D);
    pr->end(kSlotGather);
    pr->begin(kSlotFinal);
    if (D.avg_from >= 0) {
        k_avg_cells<<<(unsigned)(D.n_inst * kAvgBlocks), 256, 0, s>>>(D);
        k_avg_fin<<<(unsigned)D.n_inst, 64, 0, s>>>(D);
    }
    pr->end(kSlotFinal);
}

void launch_pack(const Dev &D, int buf, hipStream_t s) {
    const unsigned g = (unsigned)((D.nc + 3) / 4);
    if (D.prec == 1 && D.K > 0)
        k_pack<float, true><<<g, 256, 0, s>>>(D, buf);
    else if (D.prec == 1)
        k_pack<float, false><<<g, 256, 0, s>>>(D, buf);
    else if (D.K > 0)
        k_pack<double, true><<<g, 256, 0, s>>>(D, buf);
    else
        k_pack<double, false><<<g, 256, 0, s>>>(D, buf);
}

void launch_avg_out(const Dev &D, double *out, hipStream_t s) {
    k_avg_out<<<(unsigned)((D.nc + 255) / 256), 256, 0, s>>>(D, out);
}

void launch_moments(const Dev &D, int which, double *out, hipStream_t s) {
    k_moments<<<(unsigned)((D.nc + 255) / 256), 256, 0, s>>>(D, which, out);
}

}  // namespace ugkwp
