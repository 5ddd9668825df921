// apply_H of small and of dense blocks, straight from memory (gfx950).
//
// y[m] = sum_a c_a i^{imag_a} (-1)^{popc(m & z_a)} x[m ^ x_a]   (supplement Algorithm 1, with the
// sign parity of x_a & z_a folded into c_a).  Partners are gathered and nothing is staged: a sparse
// block of at most 4 MiB sits in every L2, and a dense one, of up to 2^22 amplitudes (32 or 64 MiB),
// in the last-level cache, where one gather serves all the terms of an x mask.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace syk {

namespace {

template <typename T> struct V2t;
template <> struct V2t<float> { using type = float2; };
template <> struct V2t<double> { using type = double2; };

__device__ __forceinline__ float flip(float c, uint32_t m) { return __int_as_float(__float_as_int(c) ^ static_cast<int>(m)); }
__device__ __forceinline__ double flip(double c, uint32_t m) {
    return __hiloint2double(__double2hiint(c) ^ static_cast<int>(m), __double2loint(c));
}

// one complex amplitude at byte offset voff + soff (soff wave-uniform) of a vector
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float2 load_amp(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return float2{__uint_as_float(v.x), __uint_as_float(v.y)};
}
__device__ __forceinline__ double2 load_amp(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, double) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    return double2{__hiloint2double(static_cast<int>(v.y), static_cast<int>(v.x)),
                   __hiloint2double(static_cast<int>(v.w), static_cast<int>(v.z))};
}

constexpr uint32_t kBufferWord3 = 0x00020000u;   // raw buffer descriptor: 32-bit data format, no swizzle

// The Lanczos epilogue (LanczosFuse) of a workgroup of S waves, S >= 4.  n_j^2 is the sum of the partials
// the previous pass left (at most 1024): the first 256 threads load them before the apply and the
// sum is ready after the barrier that ends it, so no launch of its own is needed for it.
template <typename T, int S>
struct Epilogue {
    using V = typename V2t<T>::type;
    const LanczosFuse<T> &lf;
    double *sh;                               // S + 4 doubles of LDS: norm shares, then row shares
    double norm = 0.0;
    Scale<T> sc;
    T bp = 0;
    __device__ __forceinline__ void load() {
        if (threadIdx.x < 256)
            for (int p = threadIdx.x; p < lf.n_parts; p += 256) norm += lf.norm_parts[p];
    }
    // before the barrier that ends the apply
    __device__ __forceinline__ void share() {
        if (threadIdx.x < 256) {
            for (int off = 32; off > 0; off >>= 1) norm += __shfl_down(norm, off, 64);
            if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = norm;
        }
    }
    // after it: the scales (a zero vector after an exact breakdown stays zero)
    __device__ __forceinline__ void scales() {
        const double n2 = ((sh[0] + sh[1]) + sh[2]) + sh[3];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            lf.norm2[lf.j] = n2;
            __hip_atomic_store(lf.norm2_host, n2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        const double nj = sqrt(n2);
        const double njm = lf.j >= 1 ? sqrt(lf.norm2[lf.j - 1]) : 0.0;
        sc = Scale<T>(nj > 1e-300 ? 1.0 / nj : 0.0);
        bp = njm > 1e-300 ? static_cast<T>(nj / njm) : T(0);
    }
    // w = H v_j - beta_{j-1} v_{j-1} of amplitude m from s = (H u_j)[m]; adds to Re <v_j, w>
    __device__ __forceinline__ V row(V s, uint32_t m, double &sum) {
        V w{sc(s.x), sc(s.y)};
        if (lf.vprev) {
            const V p = reinterpret_cast<const V *>(lf.vprev)[m];
            w.x -= bp * p.x;
            w.y -= bp * p.y;
        }
        const V u = reinterpret_cast<const V *>(lf.vcur)[m];
        const V c{sc(u.x), sc(u.y)};
        sum += static_cast<double>(c.x) * w.x + static_cast<double>(c.y) * w.y;
        return w;
    }
    // every wave's share of Re <v_j, w> -> partials[blockIdx.x]
    __device__ __forceinline__ void finish(double sum) {
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63u) == 0) sh[4 + (threadIdx.x >> 6)] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double v = 0.0;
            for (int k = 0; k < S; ++k) v += sh[4 + k];
            lf.partials[blockIdx.x] = v;
        }
    }
};

// A 16-byte quad: two adjacent complex64 amplitudes or one complex128.  Rows need the
// alignment of one amplitude only (an odd leading dimension).
template <typename T> struct Quad;
template <> struct Quad<float> {
    static constexpr int A = 2;
    typedef float V __attribute__((ext_vector_type(4), aligned(8)));
};
template <> struct Quad<double> {
    static constexpr int A = 1;
    typedef double V __attribute__((ext_vector_type(2)));
};
template <typename T>
__device__ __forceinline__ typename Quad<T>::V load_quad(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    typename Quad<T>::V q;
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    __builtin_memcpy(&q, &v, 16);
    return q;
}

// One wave owns R rows of 64 quads (A amplitudes each: lane l holds base + A (l + 64 r) + e) and one of
// S slices of the term list; the S waves of a group are in one workgroup and their sums are added in
// slice order in LDS, so the result does not depend on scheduling.
//
// Bound by the gathers: an instruction takes 16 clocks of a CU whether its lanes read 8 bytes or 16, in any
// order and wherever the partner is cached, so every lane reads 16 bytes, which is the 64 bytes
// a clock of the vector cache.  Two complex64 amplitudes of a quad have their partners in one quad,
// swapped for odd x masks; the terms are sorted so that the swap is compiled.  The slice is
// wave-uniform, so term records come through scalar loads; the partner of row r is (lane ^ x) in a
// VGPR plus a scalar offset, so a gather costs no vector address arithmetic; the sign of the
// lane and base bits is folded into the coefficient once per term and the sign of the row and the element
// is one XOR; U terms' gathers are in flight at once.  N = 36, k = 8: complex64 10.2 us against 18.1 us
// with 8-byte gathers, complex128 18.5 us (K 2^17 16 bytes at 39 TB/s of all vector caches: 15.4 us); 59 / 68 us with
// one amplitude per thread and per-lane term loads.
template <typename T, int R, int S, bool FUSE>
__global__ void __launch_bounds__(64 * S) gather_sparse(GatherTerms<T> t0, GatherTerms<T> t1,
                                                        const typename V2t<T>::type *__restrict__ x,
                                                        typename V2t<T>::type *__restrict__ y, uint32_t n, uint64_t ld,
                                                        LanczosFuse<T> lf) {
    static_assert(S >= 4, "the epilogue sums with four waves");
    using V = typename V2t<T>::type;
    using Q = typename Quad<T>::V;
    constexpr int A = Quad<T>::A;
    constexpr int SH = sizeof(T) == 4 ? 3 : 4;       // log2 of the bytes per amplitude
    constexpr int U = R >= 4 ? 2 : 4;                // terms in flight
    constexpr uint32_t ROW = 64u * A;                // amplitudes per row
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t slice = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t base = blockIdx.x * (ROW * R);
    __shared__ double sh[S + 4];
    Epilogue<T, S> epi{lf, sh};
    if constexpr (FUSE) epi.load();
    const GatherTerms<T> tb = blockIdx.z == 0 ? t0 : t1;
    const uint64_t vo = static_cast<uint64_t>(blockIdx.y) * ld + static_cast<uint64_t>(blockIdx.z) * n;
    Q acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = Q(T(0));
    {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<V *>(x + vo), 0, static_cast<int>(n << SH), kBufferWord3);
        // blocks below 64 quads: the spare lanes compute copies and store nothing
        const uint32_t lm = (lane * A) & (n - 1u);
        const uint32_t at = lm | base;
        auto terms = [&](auto im, auto odd, auto uc, uint32_t t) __attribute__((always_inline)) {
            constexpr int C = decltype(uc)::value;
            Q q[C][R];
            T c[C];
            uint32_t zs[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const GatherTerm<T> rec = tb.rec[t + u];              // wave-uniform: scalar load
                const uint32_t voff = (lm ^ (rec.x & (ROW - A))) << SH;
                const uint32_t so = base ^ (rec.x & ~(ROW - 1u));
#pragma unroll
                for (int r = 0; r < R; ++r) q[u][r] = load_quad<T>(rs, voff, (so ^ (ROW * r)) << SH);
                c[u] = flip(rec.c, __popc(at & rec.z) << 31);
                zs[u] = rec.z;
            }
#pragma unroll
            for (int u = 0; u < C; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int e = 0; e < A; ++e) {
                        uint32_t sg = __popc(zs[u] & static_cast<uint32_t>(ROW * r + e)) << 31;
                        asm("" : "+s"(sg));                          // keep the sign of row and element scalar
                        const T cr = r + e == 0 ? c[u] : flip(c[u], sg);
                        const int f = A == 2 && decltype(odd)::value ? 1 - e : e;
                        if (decltype(im)::value) {
                            acc[r][2 * e] -= cr * q[u][r][2 * f + 1];
                            acc[r][2 * e + 1] += cr * q[u][r][2 * f];
                        } else {
                            acc[r][2 * e] += cr * q[u][r][2 * f];
                            acc[r][2 * e + 1] += cr * q[u][r][2 * f + 1];
                        }
                    }
        };
        // the slice's share of a run of terms of one phase and swap
        const uint32_t lo = tb.K * slice / S, hi = tb.K * (slice + 1) / S;
        auto run = [&](auto im, auto odd, uint32_t first, uint32_t end) __attribute__((always_inline)) {
            uint32_t t = first > lo ? first : lo;
            end = end < hi ? end : hi;
            for (; t + U <= end; t += U) terms(im, odd, std::integral_constant<int, U>{}, t);
            for (; t < end; ++t) terms(im, odd, std::integral_constant<int, 1>{}, t);
        };
        if constexpr (A == 2) {
            run(std::false_type{}, std::false_type{}, 0, tb.cut[0]);
            run(std::false_type{}, std::true_type{}, tb.cut[0], tb.cut[1]);
            run(std::true_type{}, std::false_type{}, tb.cut[1], tb.cut[2]);
            run(std::true_type{}, std::true_type{}, tb.cut[2], tb.K);
        } else {
            run(std::false_type{}, std::false_type{}, 0, tb.cut[1]);
            run(std::true_type{}, std::false_type{}, tb.cut[1], tb.K);
        }
    }
    __shared__ __attribute__((aligned(16))) T part[S][R][64][2 * A];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 2 * A; ++i) part[slice][r][lane][i] = acc[r][i];
    if constexpr (FUSE) epi.share();
    __syncthreads();
    if constexpr (FUSE) epi.scales();
    double dot = 0.0;
    // wave q sums register rows q, q + S, ..., the slices in order
    for (uint32_t r = slice; r < R; r += S) {
        Q s;
#pragma unroll
        for (int i = 0; i < 2 * A; ++i) s[i] = part[0][r][lane][i];
#pragma unroll
        for (int k = 1; k < S; ++k)
#pragma unroll
            for (int i = 0; i < 2 * A; ++i) s[i] += part[k][r][lane][i];
        const uint32_t m = base + ROW * r + A * lane;
        if (m < n) {
            if constexpr (FUSE) {
#pragma unroll
                for (int e = 0; e < A; ++e) {
                    const V w = epi.row(V{s[2 * e], s[2 * e + 1]}, m + e, dot);
                    s[2 * e] = w.x;
                    s[2 * e + 1] = w.y;
                }
            }
            *reinterpret_cast<Q *>(y + vo + m) = s;
        }
    }
    if constexpr (FUSE) epi.finish(dot);
}

template <typename T, int R, int S>
int go(const GatherTerms<T> (&tb)[2], int nblk, const T *x, T *y, uint32_t n, int nvec, uint64_t ld, hipStream_t s,
       const LanczosFuse<T> *lf) {
    using V = typename V2t<T>::type;
    constexpr uint32_t rows = 64u * Quad<T>::A * R;
    const uint32_t g = (n + rows - 1) / rows;
    if (lf)
        hipLaunchKernelGGL((gather_sparse<T, R, S, true>), dim3(g), dim3(64 * S), 0, s, tb[0], tb[0],
                           reinterpret_cast<const V *>(x), reinterpret_cast<V *>(y), n, ld, *lf);
    else
        hipLaunchKernelGGL((gather_sparse<T, R, S, false>), dim3(g, nvec, nblk), dim3(64 * S), 0, s, tb[0],
                           tb[nblk - 1], reinterpret_cast<const V *>(x), reinterpret_cast<V *>(y), n, ld,
                           LanczosFuse<T>{});
    return static_cast<int>(g);
}

// ------------------------------------------------------------------ one launch per Lanczos step
// u_j = a g - b u_{j-2} - c u_{j-1} with the scales of the unnormalised basis (a zero vector after an exact
// breakdown stays zero): w = g / n_{j-1} - (n_{j-1} / n_{j-2}) u_{j-2} and u_j = w - (alpha_{j-1} / n_{j-1}) u_{j-1},
// alpha_{j-1} = Re <v_{j-1}, w>.  Every wave adds up the sums of the step before in the same order.
template <typename T>
struct StepScales {
    Scale<T> a;
    T b, c;
    __device__ __forceinline__ StepScales(const LanczosStep<T> &st, uint32_t lane, bool publish) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int p = lane; p < st.np; p += 64) {
            s0 += st.parts[3 * p];
            s1 += st.parts[3 * p + 1];
            s2 += st.parts[3 * p + 2];
        }
        const double n2 = st.j >= 2 ? sqrt(st.norm2[st.j - 2]) : 0.0;
        for (int off = 32; off > 0; off >>= 1) {
            s0 += __shfl_xor(s0, off, 64);
            s1 += __shfl_xor(s1, off, 64);
            s2 += __shfl_xor(s2, off, 64);
        }
        const double n1 = sqrt(s0), inv = n1 > 1e-300 ? 1.0 / n1 : 0.0, inv2 = n2 > 1e-300 ? 1.0 / n2 : 0.0;
        const double al = (s0 > 1e-300 ? s1 / s0 : 0.0) - s2 * inv2;
        a = Scale<T>(inv);
        b = static_cast<T>(n1 * inv2);
        c = static_cast<T>(al * inv);
        if (publish) {
            st.norm2[st.j - 1] = s0;
            st.alpha[st.j - 1] = al;
            __hip_atomic_store(st.norm2_host, s0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(st.alpha_host, al, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __device__ __forceinline__ T operator()(T g, T u2, T u1) const {
        const T w = a(g) - b * u2;
        return w - c * u1;
    }
};

// gather_sparse with u_j formed from three quads at every partner.  A small propagation is bound by the
// time from one dependent launch to the next (4 to 5 us) and not by what the kernels do: with two
// launches a step it took 120 us from N = 20 to 32.  Now the chain of one kernel bounds it: the sums of the
// step before, then a slice's terms, four at a time.
template <typename T, int S, bool FIRST>
__global__ void __launch_bounds__(64 * S) lanczos_step(GatherTerms<T> tb, LanczosStep<T> st, uint32_t n) {
    using Q = typename Quad<T>::V;
    constexpr int A = Quad<T>::A;
    constexpr int SH = sizeof(T) == 4 ? 3 : 4;
    constexpr int R = 1, U = 4;                      // rows per wave, terms in flight
    constexpr uint32_t ROW = 64u * A;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t slice = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t base = blockIdx.x * (ROW * R);
    auto vector = [&](const T *v) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(v), 0, static_cast<int>(n << SH), kBufferWord3);
    };
    const bool two = !FIRST && st.j >= 2;
    // constant memory: the loads stay scalar behind this kernel's stores
    using Rec = const __attribute__((address_space(4))) GatherTerm<T>;
    Rec *recs = (Rec *)reinterpret_cast<uintptr_t>(tb.rec);
    const __amdgpu_buffer_rsrc_t rg = vector(st.g), r1 = vector(FIRST ? st.g : st.u1),
                                 r2 = vector(two ? st.u2 : st.g);
    const uint32_t lm = (lane * A) & (n - 1u), at = lm | base;
    // this wave's own row
    const uint32_t mine = base + ROW * slice + A * lane;
    const bool writes = slice < R && mine < n;
    const uint32_t own = (mine & (n - 1u)) << SH;
    Q ug = load_quad<T>(rg, own, 0), u1{}, u2{};
    if constexpr (!FIRST) u1 = load_quad<T>(r1, own, 0);
    if (two) u2 = load_quad<T>(r2, own, 0);
    Scale<T> ca;
    T cb = T(0), cc = T(0);
    if constexpr (!FIRST) {
        const StepScales<T> sc(st, lane, threadIdx.x == 0 && blockIdx.x == 0);
        ca = sc.a, cb = sc.b, cc = sc.c;
    }
    auto form = [&](Q g, Q p2, Q p1) __attribute__((always_inline)) {
        if constexpr (!FIRST) {
#pragma unroll
            for (int i = 0; i < 2 * A; ++i) {
                const T w = ca(g[i]) - cb * p2[i];
                g[i] = w - cc * p1[i];
            }
        }
        return g;
    };
    const Q u = form(ug, u2, u1);
    if (!FIRST && writes) *reinterpret_cast<Q *>(st.u + 2 * static_cast<uint64_t>(mine)) = u;
    Q acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = Q(T(0));
    auto terms = [&](auto im, auto odd, auto uc, uint32_t t) __attribute__((always_inline)) {
        constexpr int C = decltype(uc)::value;
        Q q[C][R], q1[C][R], q2[C][R];
        T c[C];
        uint32_t zs[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const uint32_t x = recs[t + k].x, z = recs[t + k].z;
            const uint32_t voff = (lm ^ (x & (ROW - A))) << SH;
            const uint32_t so = base ^ (x & ~(ROW - 1u));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t off = (so ^ (ROW * r)) << SH;
                q[k][r] = load_quad<T>(rg, voff, off);
                if constexpr (!FIRST) {
                    q1[k][r] = load_quad<T>(r1, voff, off);
                    q2[k][r] = two ? load_quad<T>(r2, voff, off) : Q(T(0));
                }
            }
            c[k] = flip(static_cast<T>(recs[t + k].c), __popc(at & z) << 31);
            zs[k] = z;
        }
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const Q v = FIRST ? q[k][r] : form(q[k][r], q2[k][r], q1[k][r]);
#pragma unroll
                for (int e = 0; e < A; ++e) {
                    uint32_t sg = __popc(zs[k] & static_cast<uint32_t>(ROW * r + e)) << 31;
                    asm("" : "+s"(sg));                              // keep the sign of row and element scalar
                    const T cr = r + e == 0 ? c[k] : flip(c[k], sg);
                    const int f = A == 2 && decltype(odd)::value ? 1 - e : e;
                    if (decltype(im)::value) {
                        acc[r][2 * e] -= cr * v[2 * f + 1];
                        acc[r][2 * e + 1] += cr * v[2 * f];
                    } else {
                        acc[r][2 * e] += cr * v[2 * f];
                        acc[r][2 * e + 1] += cr * v[2 * f + 1];
                    }
                }
            }
    };
    const uint32_t lo = tb.K * slice / S, hi = tb.K * (slice + 1) / S;
    auto run = [&](auto im, auto odd, uint32_t first, uint32_t end) __attribute__((always_inline)) {
        uint32_t t = first > lo ? first : lo;
        end = end < hi ? end : hi;
        for (; t + U <= end; t += U) terms(im, odd, std::integral_constant<int, U>{}, t);
        for (; t < end; ++t) terms(im, odd, std::integral_constant<int, 1>{}, t);
    };
    if constexpr (A == 2) {
        run(std::false_type{}, std::false_type{}, 0, tb.cut[0]);
        run(std::false_type{}, std::true_type{}, tb.cut[0], tb.cut[1]);
        run(std::true_type{}, std::false_type{}, tb.cut[1], tb.cut[2]);
        run(std::true_type{}, std::true_type{}, tb.cut[2], tb.K);
    } else {
        run(std::false_type{}, std::false_type{}, 0, tb.cut[1]);
        run(std::true_type{}, std::false_type{}, tb.cut[1], tb.K);
    }
    __shared__ __attribute__((aligned(16))) T part[S][R][64][2 * A];
    __shared__ double sh[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 2 * A; ++i) part[slice][r][lane][i] = acc[r][i];
    __syncthreads();
    if (slice < R) {
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        if (writes) {
            Q s;
#pragma unroll
            for (int i = 0; i < 2 * A; ++i) s[i] = part[0][slice][lane][i];
#pragma unroll
            for (int k = 1; k < S; ++k)
#pragma unroll
                for (int i = 0; i < 2 * A; ++i) s[i] += part[k][slice][lane][i];
            *reinterpret_cast<Q *>(st.gout + 2 * static_cast<uint64_t>(mine)) = s;
#pragma unroll
            for (int i = 0; i < 2 * A; ++i) {
                d0 += static_cast<double>(u[i]) * u[i];
                d1 += static_cast<double>(u[i]) * s[i];
                if constexpr (!FIRST) d2 += static_cast<double>(u[i]) * u1[i];
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            d0 += __shfl_down(d0, off, 64);
            d1 += __shfl_down(d1, off, 64);
            d2 += __shfl_down(d2, off, 64);
        }
        if (lane == 0) {
            sh[slice][0] = d0;
            sh[slice][1] = d1;
            sh[slice][2] = d2;
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int r = 0; r < R; ++r) v += sh[r][threadIdx.x];
        st.out[3 * blockIdx.x + threadIdx.x] = v;
    }
}

// the end of the sequence: alpha_{j-1} and ||u_j||^2 without H u_j, in one workgroup
template <typename T>
__global__ void __launch_bounds__(1024) lanczos_close(LanczosStep<T> st, uint32_t n) {
    const uint32_t lane = threadIdx.x & 63u;
    const StepScales<T> sc(st, lane, threadIdx.x == 0);
    const bool two = st.j >= 2;
    double sum = 0.0;
    for (uint32_t i = threadIdx.x; i < 2 * n; i += 1024) {
        const T v = sc(st.g[i], two ? st.u2[i] : T(0), st.u1[i]);
        sum += static_cast<double>(v) * v;
    }
    __shared__ double sh[16];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
    if (lane == 0) sh[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
        for (int k = 0; k < 16; ++k) v += sh[k];
        __hip_atomic_store(st.next_host, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ------------------------------------------------------------------ grouped by x mask
// Terms that share an x mask act on the partner x[m ^ x] as one complex diagonal
//   D(m) = sum_t c_t (-1)^popc(m & z_t)   (real-phase terms in Re D, i-phase terms in Im D),
// so a group costs one gather and one complex product per amplitude however many terms it has
// (about 19 in dense SYK).  D is a matrix product: over a tile of 256 amplitudes m = 16 i + j the
// sign splits into (row, term) and (term, column) factors, D = A B with A[i][t] = c_t s_t(base + 16 i)
// and B[t][j] = s_t(j) = +-1, and four terms are one 16 x 16 x 4 matrix instruction (products by
// +-1 are exact, sums are in the vectors' precision or better).  Summed on the vector unit it was
// about six operations per term and amplitude.  Bound by issue: matrix and vector instructions
// of a SIMD add up here, 32 clocks (16 x 16 x 4, 32-bit) and about 16 vector operations per step,
// six to build A and B and the rest the complex product of a group of 16 terms.  Hence the table
// pairs a real with an i-phase step, so that a step needs no phase branch and two sums run
// independently, and the operands of four steps are built before their products, which hides the
// LDS reads: N = 30 86 -> 53 us (complex128), N = 38 0.82 -> 0.62 / 1.29 -> 1.04 ms (complex64 /
// complex128).  Term by term on the vector unit N = 30 took 278 / 391 us, in the tiled kernel N = 38 9.1 ms
// (complex64).
//
// The matrix instruction of a wave's tile, in the precision P of the sums.  rows(l): the amplitude
// offset of the row of A that lane l supplies, cols(l): that of the column of B; both supply
// term l >> 4 of the step, and result r of lane l belongs to amplitude base + l + 64 r.
//
// MfmaTile: 256 amplitudes, columns = amplitude bits 0..3, rows = bits 4..7.  Result r of
// lane l is row 4 (l >> 4) + r of the 32-bit instruction and row 4 r + (l >> 4) of the 64-bit one; rows are
// numbered so that both are amplitude bits 4..7 = (l >> 4) + 4 r.
template <typename P> struct MfmaTile;
template <> struct MfmaTile<float> {
    static constexpr int R = 4;
    typedef float Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t rows(uint32_t l) { return (((l >> 2) & 3u) | ((l & 3u) << 2)) << 4; }
    static __device__ __forceinline__ uint32_t cols(uint32_t l) { return l & 15u; }
};
template <> struct MfmaTile<double> {
    static constexpr int R = 4;
    typedef double Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t rows(uint32_t l) { return (l & 15u) << 4; }
    static __device__ __forceinline__ uint32_t cols(uint32_t l) { return l & 15u; }
};
// MfmaRow: 64 amplitudes, four blocks of 4 x 4: column = amplitude bits 0..1, block = bits 2..3,
// row = bits 4..5 (64-bit sums, whatever the vectors' precision).
struct MfmaRow {
    static constexpr int R = 1;
    typedef double Acc __attribute__((ext_vector_type(1)));
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return Acc{__builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c[0], 0, 0, 0)};
    }
    static __device__ __forceinline__ uint32_t rows(uint32_t l) { return (l & 12u) | ((l & 3u) << 4); }
    static __device__ __forceinline__ uint32_t cols(uint32_t l) { return l & 3u; }
};

// +-1 and +-c with the sign in the parity of p
__device__ __forceinline__ void signed_pair(uint32_t pa, uint32_t pb, float c, float &a, float &b) {
    a = __uint_as_float((pa << 31) + __float_as_uint(c));
    b = __uint_as_float((pb << 31) | 0x3f800000u);
}
__device__ __forceinline__ void signed_pair(uint32_t pa, uint32_t pb, double c, double &a, double &b) {
    a = __hiloint2double(static_cast<int>((pa << 31) + static_cast<uint32_t>(__double2hiint(c))), __double2loint(c));
    b = __hiloint2double(static_cast<int>((pb << 31) | 0x3ff00000u), 0);
}

// A wave owns one tile (R registers of 64 amplitudes) and one of S slices of the steps; the S
// waves of a workgroup share the tile and their sums are added in slice order.  The records of
// kDenseChunk = 16 steps (64 of them, one per lane) are loaded one chunk ahead, pass through
// the wave's own piece of LDS and are read back by the term each lane supplies; the partners of
// a group are gathered while the group before it is summed.
template <typename T, typename P, typename Tile, int S, bool FUSE>
__global__ void __launch_bounds__(64 * S) gather_dense(DenseTerms<P> t0, DenseTerms<P> t1,
                                                       const typename V2t<T>::type *__restrict__ x,
                                                       typename V2t<T>::type *__restrict__ y, uint32_t n, uint64_t ld,
                                                       LanczosFuse<T> lf) {
    using V = typename V2t<T>::type;
    using M = typename Tile::Acc;
    constexpr int R = Tile::R;
    constexpr int SH = sizeof(T) == 4 ? 3 : 4;
    constexpr int PER = kDenseSlices / S;                 // table slices per wave
    constexpr int B = 4;                                  // steps whose operands are built together
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t base = blockIdx.x * (64u * R);
    const DenseTerms<P> tb = blockIdx.z == 0 ? t0 : t1;
    const uint32_t *hdrs = tb.head + kDenseHead;
    const uint64_t vo = static_cast<uint64_t>(blockIdx.y) * ld + static_cast<uint64_t>(blockIdx.z) * n;
    constexpr size_t kRecs = sizeof(DenseTerm<P>) * 64 * S, kPart = sizeof(V) * S * R * 64;
    __shared__ __attribute__((aligned(16))) char lds[kRecs > kPart ? kRecs : kPart];
    __shared__ double sh[S + 4];
    Epilogue<T, S> epi{lf, sh};
    if constexpr (FUSE) epi.load();
    DenseTerm<P> *stage = reinterpret_cast<DenseTerm<P> *>(lds) + 64 * wave;
    V acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = V{T(0), T(0)};
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<V *>(x + vo), 0, static_cast<int>(n << SH), kBufferWord3);
    const uint32_t am = base + Tile::rows(lane), bm = Tile::cols(lane), kq = lane >> 4;
    V q[R];
    auto gather = [&](uint32_t xm) __attribute__((always_inline)) {
        const uint32_t voff = (lane ^ (xm & 63u)) << SH;
        const uint32_t so = base ^ (xm & ~63u);
#pragma unroll
        for (int r = 0; r < R; ++r) q[r] = load_amp(rs, voff, (so ^ (64u * r)) << SH, T(0));
    };
    const uint32_t s0 = tb.head[wave * PER], s1 = tb.head[wave * PER + PER];
    if (s0 < s1) {
        gather(tb.head[kDenseSlices + 1 + wave * PER]);
        M dre{}, dim{};
        // records as plain words (a struct copied whole would be kept in LDS)
        using Raw = std::conditional_t<sizeof(P) == 4, u32x2, u32x4>;
        static_assert(sizeof(Raw) == sizeof(DenseTerm<P>), "record words");
        const Raw *recs = reinterpret_cast<const Raw *>(tb.rec);
        Raw nrec = recs[static_cast<size_t>(s0) * 4 + lane];
        uint32_t nhdr = hdrs[s0 + (lane & 15u)];
        for (uint32_t st = s0; st < s1; st += kDenseChunk) {
            // the wave's reads of the chunk before are done: the products took their results
            reinterpret_cast<Raw *>(stage)[lane] = nrec;
            const uint32_t hdr = nhdr;
            const uint32_t nx = st + kDenseChunk < s1 ? st + kDenseChunk : s0;
            nrec = recs[static_cast<size_t>(nx) * 4 + lane];
            nhdr = hdrs[nx + (lane & 15u)];
            __builtin_amdgcn_wave_barrier();
            for (int u0 = 0; u0 < kDenseChunk; u0 += B) {
                P a[B], b[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const DenseTerm<P> rec = stage[4 * (u0 + u) + kq];
                    signed_pair(__popc(am & rec.z), __popc(bm & rec.z), rec.c, a[u], b[u]);
                }
#pragma unroll
                for (int u = 0; u < B; u += 2) {
                    const uint32_t h = __builtin_amdgcn_readlane(hdr, u0 + u);
                    dre = Tile::mma(a[u], b[u], dre);
                    dim = Tile::mma(a[u + 1], b[u + 1], dim);
                    if (h & kDenseEnd) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const T cr = static_cast<T>(dre[r]), ci = static_cast<T>(dim[r]);
                            acc[r].x += cr * q[r].x - ci * q[r].y;
                            acc[r].y += cr * q[r].y + ci * q[r].x;
                        }
                        dre = M{};
                        dim = M{};
                        gather(h & 0x0fffffffu);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    V *part = reinterpret_cast<V *>(lds);
    __syncthreads();                                      // the record staging is done with
#pragma unroll
    for (int r = 0; r < R; ++r) part[(wave * R + r) * 64 + lane] = acc[r];
    if constexpr (FUSE) epi.share();
    __syncthreads();
    if constexpr (FUSE) epi.scales();
    double dot = 0.0;
    if (wave < R) {                                       // wave r sums register row r, slices in order
        V s = part[wave * 64 + lane];
#pragma unroll
        for (int k = 1; k < S; ++k) {
            s.x += part[(k * R + wave) * 64 + lane].x;
            s.y += part[(k * R + wave) * 64 + lane].y;
        }
        const uint32_t m = base + 64u * wave + lane;
        if constexpr (FUSE) s = epi.row(s, m, dot);
        y[vo + m] = s;
    }
    if constexpr (FUSE) epi.finish(dot);
}

}  // namespace

// nblk = 2: blocks U and D side by side in one vector (D at element offset n)
template <typename T>
int launch_apply_gather(const GatherTerms<T> (&tb)[2], int nblk, const T *x, T *y, uint32_t n, int nvec, uint64_t ld,
                        hipStream_t s, const LanczosFuse<T> *lf) {
    int g;
    // Rows per wave R and slices of the term list S, by block size alone (so that a vector's
    // result does not depend on how many vectors or blocks share the launch): as many rows per wave
    // as leave about 2048 waves, 8 per CU, with at most 16 slices.  Measured with R in {1, 2, 4, 8} and S in
    // {4, 8, 16} from N = 26 to 44: within 10% of each other below 2^10 rows, where the call's
    // host time (6 us) hides the kernel; above, k = 8, R = 4 with S = 8 / R = 4 with S = 4 / R = 2 with S = 16:
    // N = 36 complex64 10.4 / 11.4 / 10.7 us, N = 38 complex128 37.6 / 38.0 / 38.0 us.
    const uint32_t rows = (n / Quad<T>::A + 63u) / 64u;
    if (rows >= 1024u)
        g = go<T, 4, 8>(tb, nblk, x, y, n, nvec, ld, s, lf);
    else if (rows >= 256u)
        g = go<T, 2, 16>(tb, nblk, x, y, n, nvec, ld, s, lf);
    else
        g = go<T, 1, 16>(tb, nblk, x, y, n, nvec, ld, s, lf);
    SYK_HIP(hipGetLastError());
    return g;
}

template <typename T>
int launch_apply_dense(const DeviceTables *const (&tb)[2], int nblk, const T *x, T *y, uint32_t n, int nvec,
                       uint64_t ld, hipStream_t s, const LanczosFuse<T> *lf) {
    using V = typename V2t<T>::type;
    if (n < 64) fail(SYK_EDEVICE, "the grouped gather needs 64 amplitudes");
    int g = 0;
    auto go = [&](auto pc, auto tile, auto sc) {
        using P = decltype(pc);
        using Tile = decltype(tile);
        constexpr int S = decltype(sc)::value;
        DenseTerms<P> d[2];
        for (int b = 0; b < 2; ++b) {
            d[b].head = tb[b]->head;
            if constexpr (sizeof(P) == 4)
                d[b].rec = tb[b]->d32;
            else
                d[b].rec = tb[b]->d64;
        }
        g = static_cast<int>(n / (64 * Tile::R));
        if (lf)
            hipLaunchKernelGGL((gather_dense<T, P, Tile, S, true>), dim3(g), dim3(64 * S), 0, s, d[0], d[0],
                               reinterpret_cast<const V *>(x), reinterpret_cast<V *>(y), n, ld, *lf);
        else
            hipLaunchKernelGGL((gather_dense<T, P, Tile, S, false>), dim3(g, nvec, nblk), dim3(64 * S), 0, s, d[0],
                               d[nblk - 1], reinterpret_cast<const V *>(x), reinterpret_cast<V *>(y), n, ld,
                               LanczosFuse<T>{});
    };
    // Small blocks take 64-amplitude tiles to reach more CUs, larger ones 256 (four times the amplitudes per
    // step).  64 / 256: complex64 N = 28 39 / 52 us, N = 30 51 / 69 us, N = 32 117 / 89 us; complex128 N = 30 53 / 106 us,
    // N = 32 122 / 136 us, N = 34 296 / 176 us.  Sixteen waves share a tile while the tiles are few, and in
    // complex64 always, as its sums are then shorter; complex128 takes eight from 2^17 amplitudes.  Sixteen / eight:
    // complex64 N = 32 89 / 105 us, N = 38 616 / 644 us, error 3.1e-7 / 4.2e-7; complex128 N = 34 176 / 190 us,
    // N = 38 1.10 / 1.04 ms.
    constexpr bool f32 = sizeof(T) == 4;
    if (n <= (f32 ? 1u << kDenseRowL32 : 1u << (kDenseRowL32 + 1)))
        go(double(0), MfmaRow{}, std::integral_constant<int, 16>{});
    else if (f32 || n <= 1u << 16)
        go(T(0), MfmaTile<T>{}, std::integral_constant<int, 16>{});
    else if constexpr (!f32)
        go(T(0), MfmaTile<T>{}, std::integral_constant<int, 8>{});
    SYK_HIP(hipGetLastError());
    return g;
}

template <typename T>
int launch_lanczos_step(const GatherTerms<T> &tb, const LanczosStep<T> &st, uint32_t n, hipStream_t s) {
    // at most 2^13 amplitudes, so one row per wave and at most 128 workgroups
    constexpr uint32_t row = 64u * Quad<T>::A;
    const int g = static_cast<int>((n + row - 1) / row);
    if (st.j == 0)
        hipLaunchKernelGGL((lanczos_step<T, 16, true>), dim3(g), dim3(1024), 0, s, tb, st, n);
    else
        hipLaunchKernelGGL((lanczos_step<T, 16, false>), dim3(g), dim3(1024), 0, s, tb, st, n);
    SYK_HIP(hipGetLastError());
    return g;
}

template <typename T>
void launch_lanczos_close(const LanczosStep<T> &st, uint32_t n, hipStream_t s) {
    hipLaunchKernelGGL(lanczos_close<T>, dim3(1), dim3(1024), 0, s, st, n);
    SYK_HIP(hipGetLastError());
}

#define SYK_INST(T)                                                                                                 \
    template int launch_lanczos_step<T>(const GatherTerms<T> &, const LanczosStep<T> &, uint32_t, hipStream_t);     \
    template void launch_lanczos_close<T>(const LanczosStep<T> &, uint32_t, hipStream_t);                           \
    template int launch_apply_dense<T>(const DeviceTables *const (&)[2], int, const T *, T *, uint32_t, int,        \
                                       uint64_t, hipStream_t, const LanczosFuse<T> *);                              \
    template int launch_apply_gather<T>(const GatherTerms<T> (&)[2], int, const T *, T *, uint32_t, int, uint64_t,  \
                                        hipStream_t, const LanczosFuse<T> *);
SYK_INST(float)
SYK_INST(double)

}  // namespace syk
