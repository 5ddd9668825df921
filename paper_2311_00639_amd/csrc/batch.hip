// Batched OTOC: many small-N realisations and random vectors in one persistent launch.
//
// A job is one (realisation, Haar vector) pair: the two parity-block chains of the OTOC of
// Eq. (2) over the t grid (the random-state estimator of the supplement).  The host cuts jobs into
// parts (one block's chain over a range of t points) and sorts them by cost; the grid
// holds one workgroup per resident slot; each workgroup takes parts from a device counter
// until none is left and runs a whole part by itself, with no host round trip: Haar state,
// Majorana insertions, overlaps and every Lanczos propagator (matrix-free apply_H with the
// vector staged in LDS, Lanczos recurrence with double reductions, small exponential,
// step control, recombination).  Vectors are complex64 in the standard layout; every
// reduction and the tridiagonal exponential are double.
//
// Small exponential.  c = e^{w T} e_1 for the k x k Lanczos tridiagonal T (k <= 64) is
// evaluated by one wavefront, lane i holding component i: T = a + b Y with [a - b, a + b]
// the Gershgorin interval, e^{w b y} expanded in Chebyshev polynomials on [-1, 1] with
// coefficients from M Chebyshev nodes (a discrete cosine transform), and the series of M terms summed
// with the three-term recurrence of T_n(Y) e_1.  M = 16 for |w b| <= 1, 32 for |w b| <= 8, else 64: the
// truncation, about 2 (|w b| / 2)^M / M!, stays below double rounding.  Accurate to rounding
// while |w b| <= 25; a larger argument counts as not converged, so the step control shortens the
// sub-step.
// The host path (krylov.cpp) uses an eigendecomposition instead; both compute the same
// matrix function.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "batch.hpp"

namespace syk {

namespace {

// Explicit address spaces.  The job code runs in out-of-line functions, where pointers that
// are not typed by address space turn into generic (flat) accesses: slower for LDS, and each
// one waits on both memory counters.
typedef __attribute__((address_space(1))) float2 gf2;          // device memory
typedef __attribute__((address_space(3))) float2 lf2;          // LDS
typedef __attribute__((address_space(1))) const uint32_t gword;
typedef __attribute__((address_space(3))) const uint32_t lword;

// loads and stores through typed pointers use clang's builtin vector types (the HIP vector
// classes cannot be copied from address-space-qualified objects)
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 ld(const gf2 *p) {
    const f32x2 u = *(__attribute__((address_space(1))) const f32x2 *)p;
    return float2{u.x, u.y};
}
__device__ __forceinline__ void st(gf2 *p, float2 v) { *(__attribute__((address_space(1))) f32x2 *)p = f32x2{v.x, v.y}; }
__device__ __forceinline__ float2 ld(const lf2 *p) {
    const f32x2 u = *(__attribute__((address_space(3))) const f32x2 *)p;
    return float2{u.x, u.y};
}
__device__ __forceinline__ void st(lf2 *p, float2 v) { *(__attribute__((address_space(3))) f32x2 *)p = f32x2{v.x, v.y}; }
constexpr int kCheb = 64;               // Chebyshev nodes and series length, at most
constexpr double kMaxArg = 25.0;        // largest |w| b evaluated

__device__ __forceinline__ uint64_t bmix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

// amplitude n (full-space index) of the Haar state with base = mix(seed + (v + 1) G)
__device__ __forceinline__ double2 bhaar(uint64_t base, uint64_t n) {
    const uint64_t G = 0x9E3779B97F4A7C15ULL;
    const uint64_t w1 = bmix(base + (2 * n + 1) * G);
    const uint64_t w2 = bmix(base + (2 * n + 2) * G);
    const double u1 = static_cast<double>((w1 >> 11) + 1) * 0x1p-53;
    const double u2 = static_cast<double>(w2 >> 11) * 0x1p-53;
    const double r = sqrt(-2.0 * log(u1));
    double sn, cs;
    sincos(2.0 * M_PI * u2, &sn, &cs);
    return double2{r * cs, r * sn};
}

// LDS written by some lanes of a wavefront, then read by others of the same wavefront
__device__ __forceinline__ void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

template <int NT>
struct Shared {
    double red[4][NT / 64];
    double al[kMaxKrylov + 2];
    double bt[kMaxKrylov + 2];
    // v_i = sc[i] * stored: basis vector i >= 1 is stored as beta_{i-1} v_i and sc[i] is a float; vector 0 is
    // the caller's, scaled in 64 bits and rounded once per element, as a rounded scale would
    // enter the whole result
    double sc[kMaxKrylov + 2];
    double cre[kMaxKrylov + 2], cim[kMaxKrylov + 2];
    double fre[kCheb], fim[kCheb];
    double cosb[4 * kCheb];            // cos(pi j / (2 kCheb)), j < 4 kCheb
    double ctl_d[4];
    int ctl_i[4];
};

template <int NT>
using LShared = __attribute__((address_space(3))) Shared<NT>;

// whole-workgroup context of one job
template <int NT, int CHB>
struct Ctx {
    const BatchParams &p;
    LShared<NT> &sh;
    lf2 *buf;                          // LDS staging, 2^CHB amplitudes
    const BatchJob &job;
    gf2 *basis;                        // (m + 1) vectors
    gf2 *vec[4];                       // l, r2, r4, tmp
    uint32_t tid;
    lword *lterms[2];                  // the job's terms staged in LDS (null: read from memory)
    long long matvecs = 0;
    int substeps = 0;
    int status = 0;
};

// sum of two doubles over the workgroup, same value and order in every thread
template <int NT>
__device__ __forceinline__ void bsum2(double &a, double &b, LShared<NT> &sh, uint32_t tid) {
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((tid & 63) == 0) {
        sh.red[0][tid >> 6] = a;
        sh.red[1][tid >> 6] = b;
    }
    __syncthreads();
    a = 0.0;
    b = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        a += sh.red[0][w];
        b += sh.red[1][w];
    }
    __syncthreads();
}

// sum of one double over the workgroup, same value and order in every thread
template <int NT>
__device__ __forceinline__ double bsum1(double a, LShared<NT> &sh, uint32_t tid) {
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if ((tid & 63) == 0) sh.red[0][tid >> 6] = a;
    __syncthreads();
    a = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) a += sh.red[0][w];
    __syncthreads();
    return a;
}

// ------------------------------------------------------------------ vector kernels
// Thread tid owns amplitudes r * NT + tid, r < R = 2^L / NT.

// One term on a thread's RC registers: register 4 h + l (l < 4, or fewer where RC < 4) reads partner
// register 4 (h ^ xh) + (l ^ XL).  The low bits XL and ZL are compile-time constants of the run, so a group
// of four registers costs one address (its reads sit at constant offsets, in whatever order) and
// one sign operation, and the signs inside it are operand modifiers.  cur: 16 records, lane l = word l.
template <int NT, int RC, int XL, int ZL, bool IM>
__device__ __forceinline__ void term_regs(float2 (&acc)[RC], lf2 *buf, uint32_t cur, int j, uint32_t tz, uint32_t tb8,
                                          uint32_t signbit) {
    constexpr int Q = 1 << batch_low_bits(RC);       // registers per group
    const uint32_t xb = __builtin_amdgcn_readlane(cur, j), zt = __builtin_amdgcn_readlane(cur, j + 1);
    const uint32_t cw = __builtin_amdgcn_readlane(cur, j + 2);
    // the parity goes to the sign bit of the coefficient: adding 2^31 flips it
    const float cl = __uint_as_float((static_cast<uint32_t>(__popc(tz & zt)) << 31) + cw);
    const uint32_t base = tb8 ^ xb;
    float2 q[RC];
#pragma unroll
    for (int h = 0; h < RC / Q; ++h) {
        const lf2 *b = (const lf2 *)((__attribute__((address_space(3))) char *)buf + (base ^ (h * Q * NT * 8u)));
#pragma unroll
        for (int l = 0; l < Q; ++l) q[Q * h + l] = ld(b + l * NT);
    }
    const uint32_t sg = RC > Q ? __builtin_amdgcn_readlane(cur, j + 3) : 0u;
#pragma unroll
    for (int h = 0; h < RC / Q; ++h) {
        uint32_t sh = sg << (31 - h);
        asm("" : "+s"(sh));                          // one scalar shift, one vector operation
        const float ch = h == 0 ? cl : __uint_as_float(__float_as_uint(cl) ^ (sh & signbit));
#pragma unroll
        for (int l = 0; l < Q; ++l) {
            const float cr = (__builtin_popcount(l & ZL) & 1) ? -ch : ch;
            const float2 p = q[Q * h + (l ^ XL)];
            float2 &a = acc[Q * h + l];
            if (IM) {
                a.x -= cr * p.y;
                a.y += cr * p.x;
            } else {
                a.x += cr * p.x;
                a.y += cr * p.y;
            }
        }
    }
}

// f(integral_constant<int, i>) for i = I .. N - 1
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// y = H_blk v (v: global, standard layout, scaled by vs + vlo as it is staged); returns this thread's
// share of Re <v, y>.  The block is cut into NCH chunks of CH amplitudes; output chunk o is
// accumulated in registers (RC per thread) while every chunk ch of v is staged in LDS in turn, and the
// terms whose partner offset x >> log2(CH) equals o ^ ch are applied from it, run by run.  Up to two
// chunks, y stays in registers (y0: chunk 0 of two, acc: the last chunk) and chunk o of v is the
// last one staged for output chunk o, so its product with y reads LDS and the last chunk of v is still
// there afterwards; four chunks are written to y.
// Bound by LDS reads, 8 bytes per term and amplitude: at N = 32 a term costs 0.92 us per 2^15
// amplitudes, 119 of an assumed 128 bytes a clock (with 16 registers it takes 46 vector operations, 32 of them
// the products; 74 with an address and a sign per register).  The rest of a step at N = 32, about
// 85 us on every CU at once, is Lanczos vectors from memory: 127 us when y went through memory and
// v_j was read again for the products.
template <int NT, int CHB, int L, int RC>
__device__ __forceinline__ double apply_h(Ctx<NT, CHB> &c, int blk, const gf2 *v, gf2 *y, float vs, float vlo,
                                          float2 (&y0)[RC], float2 (&acc)[RC]) {
    constexpr int n = 1 << L;
    constexpr int LCH = L < CHB ? L : CHB;
    constexpr int CH = 1 << LCH;
    constexpr int NCH = n / CH;
    constexpr int LNT = __builtin_ctz(NT);
    constexpr int LOW = batch_low_bits(RC), RUNS = batch_runs(RC);
    static_assert(NCH >= 1 && NCH <= 4 && RC == CH / NT && RC >= 1 && RC <= 16, "chunking");
    const uint32_t tid = c.tid, lane = tid & 63u;
    gword *terms = (gword *)(c.p.terms + c.job.term_off[blk]);
    lword *lterms = c.lterms[blk];
    const uint32_t *runs = c.p.runs + c.job.run_off[blk];
    const bool staged = __builtin_amdgcn_readfirstlane(lterms != nullptr ? 1 : 0) != 0;   // uniform
    const uint32_t last = static_cast<uint32_t>(c.job.K) * 4u - 1u;
    // records 16 i .. 16 i + 15, one word per lane (past the last record: its last word)
    auto load16 = [&](uint32_t i) __attribute__((always_inline)) {
        uint32_t w = i * 64u + lane;
        w = w < last ? w : last;
        return staged ? lterms[w] : terms[w];
    };
    auto scaled = [&](float2 q) __attribute__((always_inline)) {
        return float2{fmaf(vs, q.x, vlo * q.x), fmaf(vs, q.y, vlo * q.y)};
    };
    const uint32_t tb8 = tid * 8u;
    uint32_t signbit = 0x80000000u;
    asm("" : "+v"(signbit));                          // in a VGPR: a sign operation has one scalar operand
    double dre = 0.0;
    int in_lds = -1;                                  // chunk of v staged in LDS
    for (int o = 0; o < NCH; ++o) {
        if (NCH == 2 && o == 1)
#pragma unroll
            for (int r = 0; r < RC; ++r) y0[r] = acc[r];
#pragma unroll
        for (int r = 0; r < RC; ++r) acc[r] = float2{0.0f, 0.0f};
        const uint32_t tz = tid | (static_cast<uint32_t>(o) << LNT);
        for (int i = 0; i < NCH; ++i) {
            // two chunks: the other one, then its own; four: back and forth; the first chunk of
            // an output chunk is the one staged last
            const int ch = NCH <= 2 ? o ^ (NCH - 1 - i) : (o & 1) ? NCH - 1 - i : i;
            if (ch != in_lds) {
                __syncthreads();                          // earlier readers of buf are done
                float2 q[RC];
#pragma unroll
                for (int r = 0; r < RC; ++r) q[r] = ld(v + (ch * CH + r * NT + tid));
#pragma unroll
                for (int r = 0; r < RC; ++r) st(c.buf + (r * NT + tid), scaled(q[r]));
                __syncthreads();
                in_lds = ch;
            }
            // the terms with partner chunk offset x >> LCH == o ^ ch
            const uint32_t *rb = runs + __builtin_amdgcn_readfirstlane((o ^ ch) * (RUNS + 1));
            uint32_t t = __builtin_amdgcn_readfirstlane(rb[0]);
            uint32_t cur = load16(t >> 4);
            static_for<0, RUNS>([&](auto rc) __attribute__((always_inline)) {
                constexpr int run = decltype(rc)::value;
                constexpr int ZL = run & ((1 << LOW) - 1), XL = (run >> LOW) & ((1 << LOW) - 1);
                constexpr bool IM = (run >> (2 * LOW)) != 0;
                const uint32_t e = __builtin_amdgcn_readfirstlane(rb[run + 1]);
                while (t < e) {
                    term_regs<NT, RC, XL, ZL, IM>(acc, c.buf, cur, static_cast<int>(t & 15u) * 4, tz, tb8, signbit);
                    if ((++t & 15u) == 0u) cur = load16(t >> 4);
                }
            });
        }
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const int i = o * CH + r * NT + static_cast<int>(tid);
            float2 q;
            if (NCH <= 2) {
                q = ld(c.buf + (r * NT + tid));           // written by this thread
            } else {
                q = scaled(ld(v + i));
                st(y + i, acc[r]);
            }
            dre += static_cast<double>(q.x) * acc[r].x + static_cast<double>(q.y) * acc[r].y;
        }
    }
    return dre;
}

template <int NT, int CHB, int L>
__device__ double norm2(Ctx<NT, CHB> &c, const gf2 *v) {
    constexpr int R = (1 << L) / NT;
    double a = 0.0;
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
        const float2 q = ld(v + (r * NT + c.tid));
        a += static_cast<double>(q.x) * q.x + static_cast<double>(q.y) * q.y;
    }
    return bsum1<NT>(a, c.sh, c.tid);
}

// <u, v> = sum conj(u) v
template <int NT, int CHB, int L>
__device__ double2 dot(Ctx<NT, CHB> &c, const gf2 *u, const gf2 *v) {
    constexpr int R = (1 << L) / NT;
    double a = 0.0, b = 0.0;
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
        const float2 p = ld(u + (r * NT + c.tid)), q = ld(v + (r * NT + c.tid));
        a += static_cast<double>(p.x) * q.x + static_cast<double>(p.y) * q.y;
        b += static_cast<double>(p.x) * q.y - static_cast<double>(p.y) * q.x;
    }
    bsum2<NT>(a, b, c.sh, c.tid);
    return double2{a, b};
}

// dst = chi block map of Majorana n from block `src_blk` (times sqrt 2: the Pauli string)
template <int NT, int CHB, int L>
__device__ void gamma(Ctx<NT, CHB> &c, bool top, uint32_t x, uint32_t z, int w, int src_blk, const gf2 *src,
                      gf2 *dst) {
    constexpr int R = (1 << L) / NT;
    // scale i^w, or +-i for n = N - 1 (U -> D: +i, D -> U: -i)
    int q = top ? (src_blk == 0 ? 1 : 3) : (w & 3);
    if (top) {
        x = 0;
        z = 0;
    }
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
        const uint32_t m = static_cast<uint32_t>(r * NT) + c.tid;
        const uint32_t k = m ^ x;
        float2 v = ld(src + k);
        if (__popc(k & z) & 1) v = float2{-v.x, -v.y};
        float2 o;
        switch (q) {
            case 0: o = v; break;
            case 1: o = float2{-v.y, v.x}; break;
            case 2: o = float2{-v.x, -v.y}; break;
            default: o = float2{v.y, -v.x}; break;
        }
        st(dst + m, o);
    }
    __syncthreads();
}

// Haar state of this job's vector: block A part into dst, normalised over the full space
template <int NT, int CHB, int L>
__device__ void haar(Ctx<NT, CHB> &c, int A, gf2 *dst) {
    constexpr int R = (1 << L) / NT;
    const uint64_t h = 1ULL << L;
    double a = 0.0;
#pragma unroll 2
    for (int r = 0; r < R; ++r) {
        const uint64_t m = static_cast<uint64_t>(r * NT + c.tid);
        const double2 u = bhaar(c.job.base, m);
        const double2 d = bhaar(c.job.base, h + m);
        a += u.x * u.x + u.y * u.y + d.x * d.x + d.y * d.y;
        const double2 s = A == 0 ? u : d;
        st(dst + m, float2{static_cast<float>(s.x), static_cast<float>(s.y)});
    }
    a = bsum1<NT>(a, c.sh, c.tid);
    const double inv = 1.0 / sqrt(a);
#pragma unroll 2
    for (int r = 0; r < R; ++r) {
        const uint64_t m = static_cast<uint64_t>(r * NT + c.tid);
        const double2 u = A == 0 ? bhaar(c.job.base, m) : bhaar(c.job.base, h + m);
        st(dst + m, float2{static_cast<float>(u.x * inv), static_cast<float>(u.y * inv)});
    }
    __syncthreads();
}

// ------------------------------------------------------------------ Lanczos
// one Lanczos iteration j: V_{j+1}, alpha_j = sh.al[j], beta_{j+1} = sh.bt[j + 1].  v0: the start
// vector, which is basis vector 0 (the others sit in the slot's basis from 1 on)
template <int NT, int CHB, int L>
__device__ __forceinline__ void lanczos_step(Ctx<NT, CHB> &c, int blk, int j, const gf2 *v0) {
    constexpr int R = (1 << L) / NT;
    constexpr int RC = L < CHB ? R : (1 << CHB) / NT, NCH = R / RC;
    const gf2 *vj = j > 0 ? c.basis + static_cast<size_t>(j) * c.p.vec_stride : v0;
    const gf2 *vp = j > 1 ? c.basis + static_cast<size_t>(j - 1) * c.p.vec_stride : v0;
    gf2 *vn = c.basis + static_cast<size_t>(j + 1) * c.p.vec_stride;
    // basis slots hold v_i / sc[i]; the next slot is left unnormalised (its scale 1/beta_j
    // enters wherever it is read), which saves a normalising pass per step
    const double sj = c.sh.sc[j];
    const float shi = static_cast<float>(sj), slo = static_cast<float>(sj - shi);   // slo = 0 for j > 0
    const float fb = j > 0 ? static_cast<float>(c.sh.bt[j] * c.sh.sc[j - 1]) : 0.0f;
    float2 y0[RC], acc[RC];
    const double dre = apply_h<NT, CHB, L, RC>(c, blk, vj, vn, shi, slo, y0, acc);
    double w2 = 0.0, alpha;
    if constexpr (NCH <= 2) {
        // w = y - alpha v_j - beta_{j-1} v_{j-1} from registers; the last chunk of v_j is still staged
        float2 p[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r)
            p[r] = j > 0 ? ld(vp + ((NCH - 1) * RC + r) * NT + c.tid) : float2{0.0f, 0.0f};
        alpha = bsum1<NT>(dre, c.sh, c.tid);
        const float al = static_cast<float>(alpha), fa = static_cast<float>(alpha * sj);
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const int i = ((NCH - 1) * RC + r) * NT + static_cast<int>(c.tid);
            const float2 q = ld(c.buf + (r * NT + c.tid));
            const float2 w = {acc[r].x - al * q.x - fb * p[r].x, acc[r].y - al * q.y - fb * p[r].y};
            st(vn + i, w);
            w2 += static_cast<double>(w.x) * w.x + static_cast<double>(w.y) * w.y;
        }
        if constexpr (NCH == 2) {
            constexpr int G = RC < 8 ? RC : 8;       // loads in flight: 2 G
#pragma unroll
            for (int r0 = 0; r0 < RC; r0 += G) {
                float2 q[G];
#pragma unroll
                for (int r = 0; r < G; ++r) {
                    q[r] = ld(vj + (r0 + r) * NT + c.tid);
                    p[r] = j > 0 ? ld(vp + (r0 + r) * NT + c.tid) : float2{0.0f, 0.0f};
                }
#pragma unroll
                for (int r = 0; r < G; ++r) {
                    const float2 w = {y0[r0 + r].x - fa * q[r].x - fb * p[r].x, y0[r0 + r].y - fa * q[r].y - fb * p[r].y};
                    st(vn + (r0 + r) * NT + c.tid, w);
                    w2 += static_cast<double>(w.x) * w.x + static_cast<double>(w.y) * w.y;
                }
            }
        }
    } else {
        alpha = bsum1<NT>(dre, c.sh, c.tid);
        const float fa = static_cast<float>(alpha * sj);
#pragma unroll 4
        for (int r = 0; r < R; ++r) {
            const int i = r * NT + static_cast<int>(c.tid);
            const float2 q = ld(vj + i);
            float2 w = ld(vn + i);
            w.x -= fa * q.x;
            w.y -= fa * q.y;
            if (j > 0) {
                const float2 p = ld(vp + i);
                w.x -= fb * p.x;
                w.y -= fb * p.y;
            }
            st(vn + i, w);
            w2 += static_cast<double>(w.x) * w.x + static_cast<double>(w.y) * w.y;
        }
    }
    const double beta = sqrt(bsum1<NT>(w2, c.sh, c.tid));
    if (c.tid == 0) {
        c.sh.al[j] = alpha;
        c.sh.bt[j + 1] = beta;
        c.sh.sc[j + 1] = beta > 0.0 ? static_cast<float>(1.0 / beta) : 0.0f;
    }
    __syncthreads();
}

// lane i's neighbours in the wavefront: the value of lane i - 1 or i + 1, 0 beyond the ends
template <int CTRL>
__device__ __forceinline__ double wave_shift(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int kFromBelow = 0x138, kFromAbove = 0x130;      // whole-wave shifts by one lane

// Wavefront 0 only.  c = e^{(wr + i wi) T_k} e_1 into sh.cre / sh.cim; returns |c_{k-1}|,
// or a negative value when the argument exceeds the evaluated range.
template <int NT>
__device__ double small_exp(LShared<NT> &sh, int k, double wr, double wi, uint32_t lane) {
    // Gershgorin interval of T_k (off-diagonal bt[1..k-1])
    double lo = 1e300, hi = -1e300;
    if (static_cast<int>(lane) < k) {
        const double d = sh.al[lane];
        const double e0 = lane > 0 ? fabs(sh.bt[lane]) : 0.0;
        const double e1 = static_cast<int>(lane) + 1 < k ? fabs(sh.bt[lane + 1]) : 0.0;
        lo = d - e0 - e1;
        hi = d + e0 + e1;
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off, 64));
        hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    const double a = 0.5 * (hi + lo);
    const double b = fmax(0.5 * (hi - lo), 1e-300);
    const double ur = wr * b, ui = wi * b;           // argument on [-1, 1]
    const double arg = sqrt(ur * ur + ui * ui);
    if (arg > kMaxArg) return -1.0;
    const int M = __builtin_amdgcn_readfirstlane(arg <= 1.0 ? 16 : arg <= 8.0 ? 32 : kCheb);
    const int stride = kCheb / M;                    // of the cosine table
    // samples at the Chebyshev nodes y_q = cos(pi (q + 1/2) / M)
    if (static_cast<int>(lane) < M) {
        const double y = sh.cosb[(2 * lane + 1) * stride];
        const double er = exp(ur * y);
        double sn, cs;
        sincos(ui * y, &sn, &cs);
        sh.fre[lane] = er * cs;
        sh.fim[lane] = er * sn;
    }
    wave_lds_sync();
    // coefficient n = lane: (2 / M) sum_q f_q cos(pi n (2q + 1) / (2M))
    double cr = 0.0, ci = 0.0;
#pragma unroll 8
    for (int q = 0; q < M; ++q) {
        const double cs = sh.cosb[(lane * (2 * q + 1) * stride) & (4 * kCheb - 1)];
        cr += sh.fre[q] * cs;
        ci += sh.fim[q] * cs;
    }
    cr *= 2.0 / M;
    ci *= 2.0 / M;
    if (lane == 0) {
        cr *= 0.5;
        ci *= 0.5;
    }
    wave_lds_sync();
    sh.fre[lane] = cr;                                // the samples are no longer needed
    sh.fim[lane] = ci;
    wave_lds_sync();
    // sum_n a_n T_n(Y) e_1, Y = (T - a) / b, lane i = component i
    const bool in = static_cast<int>(lane) < k;
    const double d = in ? (sh.al[lane] - a) / b : 0.0;
    const double lo_off = (in && lane > 0) ? sh.bt[lane] / b : 0.0;                    // to i - 1
    const double up_off = (in && static_cast<int>(lane) + 1 < k) ? sh.bt[lane + 1] / b : 0.0;   // to i + 1
    auto applyY = [&](double u) {
        return d * u + lo_off * wave_shift<kFromBelow>(u) + up_off * wave_shift<kFromAbove>(u);
    };
    double u0 = lane == 0 ? 1.0 : 0.0;
    double u1 = applyY(u0);
    double sr = sh.fre[0] * u0 + sh.fre[1] * u1;
    double si = sh.fim[0] * u0 + sh.fim[1] * u1;
#pragma unroll 2
    for (int nn = 2; nn < M; ++nn) {
        const double u2 = 2.0 * applyY(u1) - u0;
        sr += sh.fre[nn] * u2;
        si += sh.fim[nn] * u2;
        u0 = u1;
        u1 = u2;
    }
    // times e^{w a}
    const double er = exp(wr * a);
    double sn, cs;
    sincos(wi * a, &sn, &cs);
    const double gr = er * cs, gi = er * sn;
    const double outr = gr * sr - gi * si, outi = gr * si + gi * sr;
    if (in) {
        sh.cre[lane] = outr;
        sh.cim[lane] = outi;
    }
    const double mag = sqrt(outr * outr + outi * outi);
    return __shfl(mag, k - 1, 64);
}

// Step decision after k Lanczos vectors (wavefront 0): ctl_i[0] = 1 if the sub-step ends
// here, ctl_d[0] = its fraction tau, ctl_i[1] = error; cre/cim hold e^{tau z T} e_1.
template <int NT>
__device__ void decide(LShared<NT> &sh, int k, int m, double remaining, double zr, double zi, double tol,
                       uint32_t lane) {
    double tn = 0.0;
    if (static_cast<int>(lane) < k) tn = fmax(fabs(sh.al[lane]), lane > 0 ? sh.bt[lane] : 0.0);
    for (int off = 32; off > 0; off >>= 1) tn = fmax(tn, __shfl_xor(tn, off, 64));
    const double bk = sh.bt[k];
    const bool breakdown = bk <= 1e-14 * fmax(tn, 1e-300);
    auto err = [&](double f) {
        const double l = small_exp<NT>(sh, k, f * zr, f * zi, lane);
        if (l < 0.0) return 1e300;
        return breakdown ? 0.0 : bk * l;
    };
    int done = 0, fail = 0;
    double tau = 0.0;
    if (!(bk == bk)) {
        fail = 6;
    } else if (err(remaining) <= tol * remaining) {
        tau = remaining;
        done = 1;
    } else if (k == m) {
        double lo = 0.0, hi = remaining;
        for (int it = 0; it < 200; ++it) {
            const double mid = (lo == 0.0) ? hi * 0.5 : sqrt(lo * hi);
            if (err(mid) <= tol * mid)
                lo = mid;
            else
                hi = mid;
            if (lo > 0.0 && hi / lo < 1.0 + 1e-3) break;
            if (lo == 0.0 && hi < 1e-14 * remaining) break;
        }
        if (lo <= 1e-12 * remaining) {
            fail = 5;
        } else {
            tau = lo;
            done = 1;
            err(tau);                                 // leaves e^{tau z T} e_1 in cre / cim
        }
    }
    if (lane == 0) {
        sh.ctl_i[0] = done;
        sh.ctl_i[1] = fail;
        sh.ctl_d[0] = tau;
    }
}

// v <- e^{z H_blk} v (in place), Lanczos with restarts and the step control of the
// single-vector path; nrm = ||v|| on entry, returns the norm of the result
template <int NT, int CHB, int L>
__device__ __attribute__((noinline)) double prop(Ctx<NT, CHB> &c, int blk, double zr, double zi, gf2 *v, double nrm) {
    constexpr int R = (1 << L) / NT;
    if (c.status) return nrm;
    if (nrm == 0.0 || (zr == 0.0 && zi == 0.0)) return nrm;
    if (!(nrm == nrm)) {
        c.status = 6;
        return nrm;
    }
    const int m = c.p.m;
    double remaining = 1.0;
    for (;;) {
        if (++c.substeps > c.p.max_substeps) {
            c.status = 5;
            return nrm;
        }
        if (c.tid == 0) {
            c.sh.bt[0] = 0.0;
            c.sh.sc[0] = 1.0 / nrm;
        }
        __syncthreads();
        int k = 0, done = 0;
        double tau = 0.0;
        for (int j = 0; j < m; ++j) {
            lanczos_step<NT, CHB, L>(c, blk, j, v);
            ++c.matvecs;
            k = j + 1;
            if (k < 4 && k < m) continue;
            if (c.tid < 64) decide<NT>(c.sh, k, m, remaining, zr, zi, c.p.tol, c.tid);
            __syncthreads();
            done = c.sh.ctl_i[0];
            const int fail = c.sh.ctl_i[1];
            tau = c.sh.ctl_d[0];
            __syncthreads();
            if (fail) {
                c.status = fail;
                return nrm;
            }
            if (done) break;
        }
        if (!done) {                                  // m == 0 cannot happen; defensive
            c.status = 5;
            return nrm;
        }
        // v = nrm * sum_i c_i V_i, four vectors of G amplitudes in flight
        constexpr int G = R < 4 ? R : 4;
        double n2 = 0.0;
        for (int r0 = 0; r0 < R; r0 += G) {
            double sr[G], si[G];
            auto add = [&](int i, const float2 (&q)[G]) __attribute__((always_inline)) {
                const double cr = c.sh.cre[i] * c.sh.sc[i], ci = c.sh.cim[i] * c.sh.sc[i];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    sr[g] += cr * q[g].x - ci * q[g].y;
                    si[g] += cr * q[g].y + ci * q[g].x;
                }
            };
            auto get = [&](const gf2 *u, float2 (&q)[G]) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < G; ++g) q[g] = ld(u + ((r0 + g) * NT + c.tid));
            };
#pragma unroll
            for (int g = 0; g < G; ++g) sr[g] = si[g] = 0.0;
            float2 q[4][G];
            get(v, q[0]);
            add(0, q[0]);
            int i = 1;
            for (; i + 4 <= k; i += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) get(c.basis + static_cast<size_t>(i + u) * c.p.vec_stride, q[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) add(i + u, q[u]);
            }
            for (; i < k; ++i) {
                get(c.basis + static_cast<size_t>(i) * c.p.vec_stride, q[0]);
                add(i, q[0]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float2 w = {static_cast<float>(nrm * sr[g]), static_cast<float>(nrm * si[g])};
                st(v + ((r0 + g) * NT + c.tid), w);
                n2 += static_cast<double>(w.x) * w.x + static_cast<double>(w.y) * w.y;
            }
        }
        nrm = sqrt(bsum1<NT>(n2, c.sh, c.tid));       // ends with a barrier
        remaining -= tau;
        if (remaining <= 1e-15) return nrm;
        if (nrm == 0.0) return nrm;
        if (!(nrm == nrm)) {
            c.status = 6;
            return nrm;
        }
    }
}

// one part: block A's chain of the job, F at the t points [k0, k1)
template <int NT, int CHB, int L>
__device__ __attribute__((noinline)) void run_part(Ctx<NT, CHB> &c, int A, int k0, int k1, double2 *F) {
    const BatchJob &jb = c.job;
    const double beta = jb.beta;
    gf2 *l = c.vec[0], *r2 = c.vec[1], *r4 = c.vec[2], *tmp = c.vec[3];
    const int B = 1 - A;
    haar<NT, CHB, L>(c, A, l);
    // norms travel with the vectors: a Majorana string keeps them
    double nl = sqrt(norm2<NT, CHB, L>(c, l));
    nl = prop<NT, CHB, L>(c, A, -beta / 8.0, 0.0, l, nl);                         // r0
    gamma<NT, CHB, L>(c, jb.v_top, jb.vx, jb.vz, jb.vw, A, l, r2);                // V_BA r0
    double nr = prop<NT, CHB, L>(c, B, -beta / 4.0, 0.0, r2, nl);
    long long before = k0 > 0 ? c.matvecs : 0;                                    // another part's
    int before_sub = k0 > 0 ? c.substeps : 0;
    double tprev = 0.0;
    for (int k = 0; k < k1; ++k) {
        const double t = c.p.ts[k];
        const double dt = t - tprev;
        if (dt > 0.0) {
            nr = prop<NT, CHB, L>(c, B, 0.0, -dt, r2, nr);
            nl = prop<NT, CHB, L>(c, A, 0.0, -dt, l, nl);
        }
        tprev = t;
        if (c.status) return;
        if (k < k0) {
            before = c.matvecs;
            before_sub = c.substeps;
            continue;
        }
        gamma<NT, CHB, L>(c, jb.w_top, jb.wx, jb.wz, jb.ww, B, r2, r4);           // W_AB r2
        const double n4 = prop<NT, CHB, L>(c, A, -beta / 4.0, t, r4, nr);
        gamma<NT, CHB, L>(c, jb.v_top, jb.vx, jb.vz, jb.vw, A, r4, tmp);          // V_BA r4
        prop<NT, CHB, L>(c, B, -beta / 4.0, -t, tmp, n4);                         // r6
        gamma<NT, CHB, L>(c, jb.w_top, jb.wx, jb.wz, jb.ww, B, tmp, r4);          // W_AB r6
        const double2 d = dot<NT, CHB, L>(c, l, r4);
        if (c.tid == 0) F[k] = double2{0.25 * d.x, 0.25 * d.y};
        if (c.status) return;
    }
    c.matvecs -= before;
    c.substeps -= before_sub;
}

template <int NT, int CHB, int OCC>
__global__ void __launch_bounds__(NT, OCC * NT / 256) otoc_batch_kernel(BatchParams p) {
    __shared__ Shared<NT> sh;
    __shared__ float2 buf[1 << CHB];
    __shared__ int job_sh;
    // term staging for the job (both blocks), where LDS allows: jobs with more terms read
    // them from memory
    constexpr int TL = NT >= 512 ? 256 : 1;
    __shared__ BatchTerm tl[2][TL];
    const uint32_t tid = threadIdx.x;
    for (int j = tid; j < 4 * kCheb; j += NT) sh.cosb[j] = cos(M_PI * j / (2.0 * kCheb));
    gf2 *slot = (gf2 *)(p.ws + static_cast<size_t>(blockIdx.x) * p.slot_stride);   // address-space cast
    for (;;) {
        __syncthreads();
        if (tid == 0) job_sh = static_cast<int>(atomicAdd(p.counter, 1u));
        __syncthreads();
        const int pi = job_sh;
        if (pi >= p.n_parts) break;
        const BatchPart part = p.parts[pi];
        const BatchJob &jb = p.jobs[part.job];
        double2 *F = reinterpret_cast<double2 *>(p.F) + (static_cast<size_t>(part.job) * 2 + part.A) * p.nt;
        Ctx<NT, CHB> c{p, *(LShared<NT> *)(&sh), (lf2 *)(buf), jb, slot, {slot + static_cast<size_t>(p.m + 1) * p.vec_stride,
                                               slot + static_cast<size_t>(p.m + 2) * p.vec_stride,
                                               slot + static_cast<size_t>(p.m + 3) * p.vec_stride,
                                               slot + static_cast<size_t>(p.m + 4) * p.vec_stride},
                       tid, {nullptr, nullptr}};
        if (TL > 1 && jb.K <= TL) {
            for (int blk = 0; blk < 2; ++blk)
                for (int t = static_cast<int>(tid); t < jb.K; t += NT) tl[blk][t] = p.terms[jb.term_off[blk] + t];
            __syncthreads();
            c.lterms[0] = (lword *)(tl[0]);
            c.lterms[1] = (lword *)(tl[1]);
        }
        // the block size is a compile-time parameter of the job code
        switch (jb.L) {
#define SYK_BL(LL)                                                       \
    case LL:                                                             \
        if constexpr ((1 << LL) >= NT && (1 << LL) <= 4 * (1 << CHB)) run_part<NT, CHB, LL>(c, part.A, part.k0, part.k1, F); \
        else c.status = 2;                                               \
        break;
            SYK_BL(8)
            SYK_BL(9)
            SYK_BL(10)
            SYK_BL(11)
            SYK_BL(12)
            SYK_BL(13)
            SYK_BL(14)
            SYK_BL(15)
#undef SYK_BL
            default:
                c.status = 2;
        }
        if (tid == 0) {
            p.results[pi] = BatchResult{c.matvecs, c.substeps, c.status};
        }
    }
}

}  // namespace

bool batch_variant_supports(const BatchVariant &v, int L) {
    return L >= 8 && L <= 15 && (1 << L) >= v.nt && (1 << L) <= 4 * (1 << v.chb);
}

const std::vector<BatchVariant> &batch_variants() {
    static const std::vector<BatchVariant> v = {{1024, 14, 1}, {512, 13, 2}, {256, 12, 4}};
    return v;
}

void launch_otoc_batch(const BatchVariant &v, const BatchParams &p, int grid, hipStream_t s) {
    if (v.nt == 1024 && v.chb == 14 && v.occ == 1)
        hipLaunchKernelGGL((otoc_batch_kernel<1024, 14, 1>), dim3(grid), dim3(1024), 0, s, p);
    else if (v.nt == 512 && v.chb == 13 && v.occ == 2)
        hipLaunchKernelGGL((otoc_batch_kernel<512, 13, 2>), dim3(grid), dim3(512), 0, s, p);
    else if (v.nt == 256 && v.chb == 12 && v.occ == 4)
        hipLaunchKernelGGL((otoc_batch_kernel<256, 12, 4>), dim3(grid), dim3(256), 0, s, p);
    else
        fail(SYK_EDEVICE, "unknown batch variant");
    SYK_HIP(hipGetLastError());
}

}  // namespace syk
