// Host driver of the batched OTOC: term tables and jobs of many realisations, launch-shape
// choice, the cut of the jobs into parts, one persistent launch, per-realisation
// averaging over vectors and normalisation.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <complex>
#include <functional>
#include <map>
#include <queue>
#include <vector>

#include "batch.hpp"

namespace syk {

namespace {

void majorana_form(int N, int n, uint32_t &x, uint32_t &z, int &w, int &top) {
    if (n == N - 1) {
        x = z = 0;
        w = 0;
        top = 1;
    } else {
        block_majorana(N, n, x, z, w);
        top = 0;
    }
}

int device_cus() {
    int dev = 0, cus = 0;
    SYK_HIP(hipGetDevice(&dev));
    SYK_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    return std::max(cus, 1);
}

// one block's terms as the kernel of `shape` reads them (see BatchTerm), and its run bounds
void add_block(const std::vector<BlockTerm> &bt, int L, const BatchVariant &shape, std::vector<BatchTerm> &terms,
               std::vector<uint32_t> &runs) {
    const int lch = std::min(L, shape.chb), lnt = __builtin_ctz(static_cast<unsigned>(shape.nt));
    const int rc = (1 << lch) / shape.nt, low = batch_low_bits(rc), n_runs = batch_runs(rc);
    const uint32_t lmask = (1u << low) - 1u, chmask = (1u << lch) - 1u, rmask = static_cast<uint32_t>(rc) - 1u;
    std::vector<std::pair<uint32_t, int>> order;        // (chunk, phase, low x bits, low z bits), term
    for (int a = 0; a < static_cast<int>(bt.size()); ++a) {
        const uint32_t xl = (bt[a].x >> lnt) & lmask, zl = (bt[a].z >> lnt) & lmask;
        const uint32_t run = (((bt[a].imag ? 1u : 0u) << low | xl) << low) | zl;
        order.push_back({(bt[a].x >> lch) * static_cast<uint32_t>(n_runs) + run, a});
    }
    std::stable_sort(order.begin(), order.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    size_t t = 0;
    for (uint32_t ch = 0; ch < (1u << (L - lch)); ++ch) {
        runs.push_back(static_cast<uint32_t>(t));
        for (int run = 0; run < n_runs; ++run) {
            while (t < order.size() && order[t].first == ch * static_cast<uint32_t>(n_runs) + static_cast<uint32_t>(run)) ++t;
            runs.push_back(static_cast<uint32_t>(t));
        }
    }
    for (const auto &o : order) {
        const BlockTerm &b = bt[o.second];
        const uint32_t zr = (b.z >> lnt) & rmask;
        uint32_t sg = 0;
        for (uint32_t h = 0; h <= (rmask >> low); ++h) sg |= (__builtin_popcount(h & (zr >> low)) & 1u) << h;
        terms.push_back(BatchTerm{(b.x & chmask & ~(lmask << lnt)) * 8u,
                                  (b.z & ((1u << lnt) - 1u)) | (b.z >> lch) << lnt, static_cast<float>(b.c), sg});
    }
}

// Lanczos steps of a propagation over |z| (estimate: the degree of the Chebyshev series of
// e^{z x} on a spectrum of half width r = 0.05 N)
double steps_of(double z, int N, double tol) {
    const double a = z * 0.05 * N / 2.0;
    double d = 3.0, err = 2.0;
    while (err > tol && d < 200.0) err *= a / (d++ - 2.0);
    return d;
}

// Cuts the jobs into parts for `slots` workgroups, most expensive first.  The makespan cannot fall below
// the mean load, and a part that takes longer than the mean holds up the end, so parts above a target cost
// are cut at t points; a cut repeats the incremental propagations before it, so of a few
// targets the one with the shortest estimated schedule is taken.
std::vector<BatchPart> make_parts(const std::vector<BatchJob> &jobs, const std::vector<double> &ts, double beta,
                                  double tol, int slots) {
    struct Cost {
        double start;                                   // r0 and r2
        std::vector<double> inc, full;                  // per t point: advancing r2 and l; r4 and r6
        double total;
    };
    const int nt = static_cast<int>(ts.size());
    std::map<std::pair<int, int>, Cost> costs;          // by (N, K)
    double total = 0.0, longest = 0.0;
    for (const BatchJob &j : jobs) {
        Cost &c = costs[{j.N, j.K}];
        if (c.inc.empty()) {
            // one step: K terms on 2^L amplitudes, vector passes and scalars worth about 12 more terms and
            // 4096 amplitudes (workgroup barriers, the small exponential)
            const double step = (j.K + 12.0) * ((1 << j.L) + 4096.0);
            c.start = step * (steps_of(beta / 8, j.N, tol) + steps_of(beta / 4, j.N, tol));
            c.total = c.start;
            for (int k = 0; k < nt; ++k) {
                const double dt = k ? ts[k] - ts[k - 1] : ts[0];
                c.inc.push_back(dt > 0.0 ? 2 * step * steps_of(dt, j.N, tol) : 0.0);
                c.full.push_back(2 * step * steps_of(std::hypot(beta / 4, ts[k]), j.N, tol));
                c.total += c.inc[k] + c.full[k];
            }
        }
        total += 2 * c.total;
        longest = std::max(longest, c.total);
    }
    auto cut = [&](double target) {
        std::vector<std::pair<double, BatchPart>> parts;
        for (int ji = 0; ji < static_cast<int>(jobs.size()); ++ji) {
            const Cost &c = costs.at({jobs[ji].N, jobs[ji].K});
            double before = c.start;                    // to reach t point k0
            for (int k0 = 0; k0 < nt;) {
                double cost = before;
                int k1 = k0;
                while (k1 < nt && (k1 == k0 || cost + c.inc[k1] + c.full[k1] <= target)) {
                    cost += c.inc[k1] + c.full[k1];
                    before += c.inc[k1++];
                }
                for (int A = 0; A < 2; ++A) parts.push_back({cost, BatchPart{ji, A, k0, k1}});
                k0 = k1;
            }
        }
        std::stable_sort(parts.begin(), parts.end(), [](const auto &a, const auto &b) { return a.first > b.first; });
        return parts;
    };
    auto makespan = [&](const std::vector<std::pair<double, BatchPart>> &parts) {
        std::priority_queue<double, std::vector<double>, std::greater<double>> ends;
        double last = 0.0;
        for (const auto &p : parts) {
            double t = p.first;
            if (static_cast<int>(ends.size()) >= slots) {
                t += ends.top();
                ends.pop();
            }
            ends.push(t);
            last = std::max(last, t);
        }
        return last;
    };
    auto best = cut(1e300);
    const double mean = total / slots;
    if (longest > 0.5 * mean) {
        double span = makespan(best);
        for (double f : {0.25, 0.35, 0.5, 0.7, 1.0, 1.4, 2.0, 3.0}) {
            auto p = cut(f * std::max(mean, longest / nt));
            const double s = makespan(p);
            if (s < span) {
                span = s;
                best = std::move(p);
            }
        }
    }
    std::vector<BatchPart> out;
    for (const auto &p : best) out.push_back(p.second);
    return out;
}

}  // namespace

void otoc_batch(const syk_batch_item *items, int n_items, const double *t, int nt, const syk_batch_opts &o,
                double *F_raw, double *F_norm, double *F_imag, syk_batch_stats &st, hipStream_t s) {
    const auto t_start = std::chrono::steady_clock::now();
    std::vector<double> ts(t, t + nt);
    const bool prepend = ts[0] != 0.0;
    if (prepend) ts.insert(ts.begin(), 0.0);
    const int ntt = static_cast<int>(ts.size());

    int lmax = 0;
    for (int r = 0; r < n_items; ++r) lmax = std::max(lmax, items[r].N / 2 - 1);
    // eligible launch shapes
    std::vector<int> elig;
    const auto &vars = batch_variants();
    for (int v = 0; v < static_cast<int>(vars.size()); ++v) {
        bool ok = true;
        for (int r = 0; r < n_items && ok; ++r) ok = batch_variant_supports(vars[v], items[r].N / 2 - 1);
        if (ok) elig.push_back(v);
    }
    if (elig.empty()) fail(SYK_EUNSUPPORTED, "no batched launch shape serves this mix of block sizes");
    if (o.variant >= 0 && std::find(elig.begin(), elig.end(), o.variant) == elig.end())
        fail(SYK_EINVAL, "requested batch variant does not serve this mix of block sizes");

    // Launch shape: the widest workgroups (the longest parts end soonest) that still hold four
    // amplitudes per thread of the largest block; below that the workgroup's fixed costs per step weigh
    // more than its width.  Kernel times of the eligible shapes (1024, 512, 256 threads), beta = 5, four t
    // points: 64 realisations x 4 states, N 24-32: 40.6, 70.2 ms; N = 28: 22.6, 22.2, 30.5 ms; N = 24: 10.1, 8.2,
    // 7.6 ms (the rule takes 512 threads); 256 x 2 at N = 20: -, 7.3, 5.7 ms.
    int chosen = o.variant;
    if (chosen < 0) {
        chosen = elig.back();
        for (auto v = elig.rbegin(); v != elig.rend(); ++v)
            if ((1 << lmax) >= 4 * vars[*v].nt) chosen = *v;
    }
    const BatchVariant &shape = vars[chosen];

    // term tables and jobs
    std::vector<BatchTerm> terms;
    std::vector<uint32_t> runs;
    std::vector<BatchJob> jobs;
    for (int r = 0; r < n_items; ++r) {
        const syk_batch_item &it = items[r];
        Hamiltonian h;
        build_hamiltonian(h, it.N, it.k, it.seed, it.ensemble);
        BatchJob jb{};
        jb.L = h.L;
        jb.N = h.N;
        jb.K = h.K;
        for (int blk = 0; blk < 2; ++blk) {
            jb.term_off[blk] = static_cast<uint32_t>(terms.size());
            jb.run_off[blk] = static_cast<uint32_t>(runs.size());
            add_block(h.block_terms[blk], h.L, shape, terms, runs);
        }
        majorana_form(it.N, it.i, jb.wx, jb.wz, jb.ww, jb.w_top);
        majorana_form(it.N, it.j, jb.vx, jb.vz, jb.vw, jb.v_top);
        jb.beta = o.beta;
        for (int v = 0; v < o.nvec; ++v) {
            jb.base = splitmix_mix(it.state_seed + static_cast<uint64_t>(v + 1) * 0x9E3779B97F4A7C15ULL);
            jobs.push_back(jb);
        }
    }
    const int n_jobs = static_cast<int>(jobs.size());

    const int slots = device_cus() * shape.occ;
    const std::vector<BatchPart> parts = make_parts(jobs, ts, o.beta, o.tol, slots);
    int grid = std::min<int>(static_cast<int>(parts.size()), slots);

    BatchParams p{};
    p.n_parts = static_cast<int>(parts.size());
    p.nt = ntt;
    p.m = o.m;
    p.tol = o.tol;
    p.max_substeps = o.max_substeps > 0 ? o.max_substeps : 20000;
    p.vec_stride = std::max<uint64_t>(1ULL << lmax, 64);
    p.slot_stride = static_cast<uint64_t>(p.m + 5) * p.vec_stride;

    // the thread's cached workspace holds everything (the call synchronises before it returns)
    DeviceBuffer &ws = thread_workspace(0);
    size_t need = 0;
    auto piece = [&](size_t bytes) {
        const size_t at = need;
        need += (bytes + 255) & ~static_cast<size_t>(255);
        return at;
    };
    const size_t n_F = static_cast<size_t>(n_jobs) * 2 * ntt * 2;
    const size_t at_jobs = piece(jobs.size() * sizeof(BatchJob)), at_parts = piece(parts.size() * sizeof(BatchPart));
    const size_t at_runs = piece(runs.size() * sizeof(uint32_t));
    const size_t at_terms = piece(terms.size() * sizeof(BatchTerm)), at_ts = piece(ts.size() * sizeof(double));
    const size_t at_F = piece(n_F * sizeof(double)), at_res = piece(parts.size() * sizeof(BatchResult));
    const size_t at_counter = piece(sizeof(unsigned));
    // The slots' vectors last.  A few jobs cut into many parts ask for more slots than there are jobs;
    // where memory is short fewer serve them all (a workgroup takes parts until none is left).
    const size_t at_ws = need, per_slot = p.slot_stride * sizeof(float2);
    for (;;) {
        try {
            ws.ensure(at_ws + static_cast<size_t>(grid) * per_slot);
            break;
        } catch (const Error &e) {
            if (e.status != SYK_ENOMEM || grid == 1) throw;
            grid = (grid + 1) / 2;
        }
    }
    char *base = ws.ptr();
    auto put = [&](size_t at, const auto &v) {
        if (!v.empty())
            SYK_HIP(hipMemcpyAsync(base + at, v.data(), v.size() * sizeof(v[0]), hipMemcpyHostToDevice, s));
        return base + at;
    };
    p.jobs = reinterpret_cast<const BatchJob *>(put(at_jobs, jobs));
    p.parts = reinterpret_cast<const BatchPart *>(put(at_parts, parts));
    p.terms = reinterpret_cast<const BatchTerm *>(put(at_terms, terms));
    p.runs = reinterpret_cast<const uint32_t *>(put(at_runs, runs));
    p.ts = reinterpret_cast<const double *>(put(at_ts, ts));
    p.F = reinterpret_cast<double *>(base + at_F);
    p.results = reinterpret_cast<BatchResult *>(base + at_res);
    p.counter = reinterpret_cast<unsigned *>(base + at_counter);
    p.ws = reinterpret_cast<float2 *>(base + at_ws);
    SYK_HIP(hipMemsetAsync(p.counter, 0, sizeof(unsigned), s));
    hipEvent_t e0, e1;
    SYK_HIP(hipEventCreate(&e0));
    SYK_HIP(hipEventCreate(&e1));
    std::vector<double> F(n_F);
    std::vector<BatchResult> res(parts.size());
    float ms = 0.0f;
    try {
        SYK_HIP(hipEventRecord(e0, s));
        launch_otoc_batch(shape, p, grid, s);
        SYK_HIP(hipEventRecord(e1, s));
        SYK_HIP(hipEventSynchronize(e1));
        SYK_HIP(hipEventElapsedTime(&ms, e0, e1));
        SYK_HIP(hipMemcpyAsync(F.data(), p.F, F.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        SYK_HIP(hipMemcpyAsync(res.data(), p.results, res.size() * sizeof(BatchResult), hipMemcpyDeviceToHost, s));
        SYK_HIP(hipStreamSynchronize(s));
    } catch (...) {
        ignore_status(hipEventDestroy(e0));
        ignore_status(hipEventDestroy(e1));
        throw;
    }
    ignore_status(hipEventDestroy(e0));
    ignore_status(hipEventDestroy(e1));
    st.variant = chosen;
    st.slots = grid;
    st.kernel_ms = ms;
    st.tuned_ms[0] = st.tuned_ms[1] = st.tuned_ms[2] = -1.0;
    st.matvecs = 0;
    std::vector<long long> substeps(jobs.size(), 0);
    for (size_t i = 0; i < parts.size(); ++i) {
        st.matvecs += res[i].matvecs;
        substeps[parts[i].job] += res[i].substeps;
        if (res[i].status == SYK_ENOTCONV || substeps[parts[i].job] > p.max_substeps)
            fail(SYK_ENOTCONV, "batched Krylov propagation did not converge");
        if (res[i].status == SYK_ENUMERIC) fail(SYK_ENUMERIC, "non-finite value in a batched job");
        if (res[i].status != 0) fail(SYK_EUNSUPPORTED, "batched job with an unsupported block size");
    }
    // per realisation: mean over vectors, normalised by t = 0
    const int off = prepend ? 1 : 0;
    for (int r = 0; r < n_items; ++r) {
        std::vector<std::complex<double>> acc(ntt, 0.0);
        for (int v = 0; v < o.nvec; ++v) {
            const double *u = F.data() + static_cast<size_t>(r * o.nvec + v) * 2 * ntt * 2, *d = u + 2 * ntt;
            for (int k = 0; k < ntt; ++k)
                acc[k] += std::complex<double>(u[2 * k] + d[2 * k], u[2 * k + 1] + d[2 * k + 1]);
        }
        for (auto &a : acc) a /= static_cast<double>(o.nvec);
        const double f0 = acc[0].real();
        for (int k = 0; k < nt; ++k) {
            const auto f = acc[k + off];
            if (F_raw) F_raw[static_cast<size_t>(r) * nt + k] = f.real();
            if (F_imag) F_imag[static_cast<size_t>(r) * nt + k] = f.imag();
            if (F_norm) F_norm[static_cast<size_t>(r) * nt + k] = f.real() / f0;
        }
    }
    st.n_jobs = n_jobs;
    st.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
}

}  // namespace syk
