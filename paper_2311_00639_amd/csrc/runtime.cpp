// Host runtime of libsyk: error reporting, device term tables, device workspaces.
#include <algorithm>
#include <cstring>
#include <map>
#include <thread>

#include "apply_plan.hpp"
#include "internal.hpp"

namespace syk {

[[noreturn]] void fail(syk_status s, const std::string &msg) { throw Error{s, msg}; }

void hip_check(hipError_t e, const char *what) {
    if (e == hipSuccess) return;
    if (e == hipErrorOutOfMemory) fail(SYK_ENOMEM, std::string(what) + ": out of device memory");
    fail(SYK_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// ------------------------------------------------------------------ device tables
void *DeviceSlab::take(size_t bytes, const char *what) {
    const size_t b = (std::max<size_t>(bytes, 1) + 255) & ~static_cast<size_t>(255);
    if (base == nullptr || b > size - used)
        fail(SYK_ENOMEM, std::string(what) + ": " + std::to_string(b) + " bytes do not fit in the " +
                             std::to_string(size - used) + " left of this request's device region");
    void *p = base + used;
    used += b;
    return p;
}

static void free_tables(DeviceTables &t) {
    if (t.in_slab) {
        t = DeviceTables{};
        return;
    }
    ignore_status(hipFree(t.mem));
    t = DeviceTables{};
}

int gather_groups(const std::vector<BlockTerm> &terms) {
    if (terms.size() < 1024) {               // few: cheaper than a bit per mask
        std::vector<uint32_t> xs;
        for (const BlockTerm &t : terms) xs.push_back(t.x);
        std::sort(xs.begin(), xs.end());
        return static_cast<int>(std::unique(xs.begin(), xs.end()) - xs.begin());
    }
    uint32_t top = 0;
    for (const BlockTerm &t : terms) top |= t.x;
    std::vector<uint64_t> seen((static_cast<size_t>(top) >> 6) + 1, 0);
    int n = 0;
    for (const BlockTerm &t : terms) {
        const uint64_t bit = 1ULL << (t.x & 63u);
        n += (seen[t.x >> 6] & bit) == 0;
        seen[t.x >> 6] |= bit;
    }
    return n;
}

// the terms' indices by x mask, then phase (real first), otherwise in the terms' order: a radix
// sort, as comparing 27405 terms took most of the first apply at N = 30
static std::vector<int> order_by_mask(const std::vector<BlockTerm> &bt) {
    std::vector<int> a(bt.size()), b(bt.size());
    uint32_t top = 0;
    for (size_t i = 0; i < bt.size(); ++i) {
        a[i] = static_cast<int>(i);
        top |= bt[i].x;
    }
    auto key = [&](int i) { return (static_cast<uint64_t>(bt[i].x) << 1) | (bt[i].imag ? 1u : 0u); };
    constexpr int kBits = 8;
    for (int sh = 0; sh == 0 || ((static_cast<uint64_t>(top) << 1) >> sh) != 0; sh += kBits) {
        size_t at[(1 << kBits) + 1] = {};
        for (int i : a) ++at[((key(i) >> sh) & ((1 << kBits) - 1)) + 1];
        for (int k = 0; k < 1 << kBits; ++k) at[k + 1] += at[k];
        for (int i : a) b[at[(key(i) >> sh) & ((1 << kBits) - 1)]++] = i;
        a.swap(b);
    }
    return a;
}

// One allocation and one copy for the pieces of a block's tables (each 256-byte aligned): three
// of each were most of the first apply of a dense block.
namespace {
class TableImage {
  public:
    template <typename U>
    size_t add(const std::vector<U> &v) {
        const size_t at = bytes_.size();
        bytes_.resize((at + std::max<size_t>(v.size(), 1) * sizeof(U) + 255) & ~static_cast<size_t>(255));
        if (!v.empty()) std::memcpy(bytes_.data() + at, v.data(), v.size() * sizeof(U));
        return at;
    }
    char *upload(DeviceTables &t, DeviceSlab *slab) {
        if (slab)
            t.mem = static_cast<char *>(slab->take(bytes_.size(), "term tables"));
        else
            SYK_HIP(hipMalloc(reinterpret_cast<void **>(&t.mem), bytes_.size()));
        SYK_HIP(hipMemcpy(t.mem, bytes_.data(), bytes_.size(), hipMemcpyHostToDevice));
        return t.mem;
    }

  private:
    std::vector<char> bytes_;
};
}  // namespace

bool Hamiltonian::grouped() {
    std::lock_guard<std::mutex> g(dev_mu);
    if (grouped_ < 0)
        grouped_ = L >= kDenseMinL && L <= kDenseMaxL &&
                   K >= kDenseTermsPerMask * static_cast<int64_t>(gather_groups(block_terms[0]));
    return grouped_ != 0;
}

template <typename T>
bool Hamiltonian::tiled() {
    if (L < kTiledMinL) return false;
    if ((2ULL * sizeof(T) << L) > kGatherBytes && !grouped()) return true;
    int d = 0;
    if (hipGetDevice(&d) != hipSuccess) d = 0;       // host-only queries: plans of device 0
    std::lock_guard<std::mutex> g(dev_mu);
    return pinned.count({sizeof(T) == 8 ? 1 : 0, d}) != 0;
}
template bool Hamiltonian::tiled<float>();
template bool Hamiltonian::tiled<double>();

// the grouped form of a block's terms (see DenseTerms)
static void dense_steps(const std::vector<BlockTerm> &bt, std::vector<uint32_t> &head, std::vector<uint32_t> &z,
                        std::vector<double> &c) {
    std::vector<uint32_t> hdr;
    head.assign(kDenseHead, 0u);
    uint32_t *cut = head.data(), *first = head.data() + kDenseSlices + 1;
    static_assert(2 * kDenseSlices + 1 <= kDenseHead, "table head");
    const std::vector<int> order = order_by_mask(bt);
    struct Group {
        size_t lo, mid, hi;
        size_t steps() const { return 2 * ((std::max(mid - lo, hi - mid) + 3) / 4); }
    };
    std::vector<Group> groups;
    size_t total = 0;
    for (size_t i = 0; i < order.size();) {
        Group g{i, i, i};
        while (g.hi < order.size() && bt[order[g.hi]].x == bt[order[i]].x) {
            if (!bt[order[g.hi]].imag) g.mid = g.hi + 1;
            ++g.hi;
        }
        groups.push_back(g);
        total += g.steps();
        i = g.hi;
    }
    size_t gi = 0, done = 0;
    for (int q = 0; q < kDenseSlices; ++q) {
        cut[q] = static_cast<uint32_t>(hdr.size());
        first[q] = gi < groups.size() ? bt[order[groups[gi].lo]].x : 0u;
        // whole groups up to this slice's share of the steps
        const size_t until = total * (q + 1) / kDenseSlices;
        while (gi < groups.size() && (done < until || q == kDenseSlices - 1)) {
            const Group &g = groups[gi++];
            done += g.steps();
            for (size_t p = 0; p < g.steps(); p += 2)
                for (int ph = 0; ph < 2; ++ph) {
                    const size_t lo = (ph ? g.mid : g.lo) + 2 * p, hi = ph ? g.hi : g.mid;
                    hdr.push_back(0u);
                    for (size_t u = lo; u < lo + 4; ++u) {
                        z.push_back(u < hi ? bt[order[u]].z : 0u);
                        c.push_back(u < hi ? bt[order[u]].c : 0.0);
                    }
                }
            hdr[hdr.size() - 2] = kDenseEnd | (gi < groups.size() ? bt[order[groups[gi].lo]].x : 0u);
        }
        while ((hdr.size() - cut[q]) % kDenseChunk != 0) {
            hdr.push_back(0u);
            z.insert(z.end(), 4, 0u);
            c.insert(c.end(), 4, 0.0);
        }
    }
    cut[kDenseSlices] = static_cast<uint32_t>(hdr.size());
    head.insert(head.end(), hdr.begin(), hdr.end());
}

const DeviceTables &Hamiltonian::tables(int blk) {
    int dev = 0;
    SYK_HIP(hipGetDevice(&dev));
    const bool dense = grouped();
    std::lock_guard<std::mutex> g(dev_mu);
    for (int b = 0; b < 2; ++b)
        if (static_cast<int>(this->dev[b].size()) <= dev) this->dev[b].resize(dev + 1);
    DeviceTables &t = this->dev[blk][dev];
    if (t.K) return t;
    const auto &bt = block_terms[blk];
    DeviceTables nt;
    nt.in_slab = slab != nullptr;
    nt.K = static_cast<uint32_t>(K);
    TableImage img;
    try {
        if (dense) {
            std::vector<uint32_t> head, z;
            std::vector<double> c;
            dense_steps(bt, head, z, c);
            // the 64-amplitude tiles of small blocks sum in 64 bits, whatever the vectors' type
            std::vector<DenseTerm<float>> d32(L > kDenseRowL32 ? z.size() : 0);
            std::vector<DenseTerm<double>> d64(z.size());
            for (size_t i = 0; i < d32.size(); ++i) d32[i] = {z[i], static_cast<float>(c[i])};
            for (size_t i = 0; i < z.size(); ++i) d64[i] = {z[i], 0u, c[i]};
            const size_t oh = img.add(head), o32 = img.add(d32), o64 = img.add(d64);
            char *m = img.upload(nt, slab);
            nt.head = reinterpret_cast<uint32_t *>(m + oh);
            nt.d32 = reinterpret_cast<DenseTerm<float> *>(m + o32);
            nt.d64 = reinterpret_cast<DenseTerm<double> *>(m + o64);
        } else {
            std::vector<GatherTerm<float>> r32(K);
            std::vector<GatherTerm<double>> r64(K);
            // by phase, then by the lowest bit of the x mask, otherwise in the terms' order
            uint32_t i = 0;
            for (uint32_t kind = 0; kind < 4; ++kind) {
                for (const BlockTerm &b : bt) {
                    if ((b.imag ? 2u : 0u) + (b.x & 1u) != kind) continue;
                    r32[i] = {b.x, b.z, static_cast<float>(b.c), 0u};
                    r64[i] = {b.x, b.z, b.c};
                    ++i;
                }
                if (kind < 3) nt.cut[kind] = i;
            }
            const size_t o32 = img.add(r32), o64 = img.add(r64);
            char *m = img.upload(nt, slab);
            nt.r32 = reinterpret_cast<GatherTerm<float> *>(m + o32);
            nt.r64 = reinterpret_cast<GatherTerm<double> *>(m + o64);
        }
    } catch (...) {
        free_tables(nt);
        throw;
    }
    t = nt;
    return t;
}

template <typename T>
static GatherTerms<T> gather_terms(const DeviceTables &t) {
    GatherTerms<T> g;
    if constexpr (sizeof(T) == 4)
        g.rec = t.r32;
    else
        g.rec = t.r64;
    g.K = t.K;
    for (int i = 0; i < 3; ++i) g.cut[i] = t.cut[i];
    return g;
}

template <typename T>
static int apply_gather(Hamiltonian &h, const int (&blks)[2], int nblk, const T *x, T *y, int nvec, uint64_t ld,
                        hipStream_t s, const LanczosFuse<T> *lf = nullptr) {
    const uint32_t n = 1u << h.L;
    const DeviceTables *tb[2] = {&h.tables(blks[0]), &h.tables(blks[nblk - 1])};
    if (tb[0]->head) return launch_apply_dense<T>(tb, nblk, x, y, n, nvec, ld, s, lf);
    const GatherTerms<T> g[2] = {gather_terms<T>(*tb[0]), gather_terms<T>(*tb[1])};
    return launch_apply_gather<T>(g, nblk, x, y, n, nvec, ld, s, lf);
}

template <>
const std::vector<TiledVariant> &tiled_variants<float>() {
    static const std::vector<TiledVariant> v = {{13, 3, 2, 1, 1, 0, 0}, {13, 3, 1, 0, 2, 0, 0}, {12, 3, 2, 1, 2, 0, 0},
                                                {12, 2, 4, 3, 1, 0, 0}, {13, 3, 2, 1, 1, 1, 0}, {13, 3, 2, 1, 1, 0, 1},
                                                {13, 3, 2, 1, 1, 0, 2}, {12, 3, 2, 1, 2, 0, 1}, {13, 3, 2, 1, 1, 2, 0},
                                                {13, 3, 2, 1, 1, 2, 1}, {13, 3, 2, 1, 1, 2, 2}, {11, 2, 2, 1, 2, 2, 0},
                                                {10, 2, 2, 1, 4, 2, 0}, {11, 2, 2, 1, 2, 2, 1}, {12, 3, 2, 1, 2, 2, 2},
                                                {12, 2, 2, 1, 2, 2, 2}, {12, 3, 2, 1, 2, 2, 1}};
    return v;
}
template <>
const std::vector<TiledVariant> &tiled_variants<double>() {
    static const std::vector<TiledVariant> v = {{12, 2, 2, 1, 1, 0, 0}, {12, 2, 1, 0, 2, 0, 0}, {11, 2, 2, 1, 2, 0, 0},
                                                {11, 1, 4, 3, 1, 0, 0}, {12, 2, 2, 1, 1, 1, 0}, {12, 2, 2, 1, 1, 0, 1},
                                                {12, 2, 2, 1, 1, 0, 2}, {11, 2, 2, 1, 2, 0, 1}, {12, 2, 2, 1, 1, 2, 0},
                                                {12, 2, 2, 1, 1, 2, 1}, {12, 2, 2, 1, 1, 2, 2}, {11, 2, 2, 1, 2, 2, 0},
                                                {10, 2, 2, 1, 4, 2, 0}, {11, 2, 2, 1, 2, 2, 1}, {11, 2, 2, 1, 2, 2, 2},
                                                {11, 1, 2, 1, 2, 2, 2}, {10, 1, 2, 1, 4, 2, 2}};
    return v;
}
// Before (or without) autotuning: the first of a preference order (control-block records, four, two,
// one tile per workgroup, then the next smaller tile at two workgroups per CU) whose grid still
// has >= 256 workgroups, else the variant with the most workgroups.  All variants at k = 2, 4, 8: the
// choice is within 6% of the fastest from N = 40 to 48; the smaller tile (2^11) against the smallest (2^10) at
// N = 42, complex64, k = 4: 46.8 / 49.0 us.
template <typename T>
int default_variant(int L) {
    const auto &v = tiled_variants<T>();
    for (int pref : {10, 9, 8, 11}) {
        const TiledVariant &tv = v.at(pref);
        if (L >= tv.bt + tv.w + 8) return pref;
    }
    int best = 0;
    for (int i = 1; i < static_cast<int>(v.size()); ++i)
        if (v[i].bt + v[i].w < v[best].bt + v[best].w) best = i;
    return best;
}
template int default_variant<float>(int);
template int default_variant<double>(int);

template <typename T>
const ApplyPlan &Hamiltonian::plan(int blk, int rot, int variant) {
    int d = 0;
    SYK_HIP(hipGetDevice(&d));
    const int prec = sizeof(T) == 8 ? 1 : 0;
    const TiledVariant &tv = tiled_variants<T>().at(variant);
    std::lock_guard<std::mutex> g(dev_mu);
    ApplyPlan &p = plans[std::make_tuple(blk, prec, d, rot, variant)];
    if (p.pi) return p;
    HostPlan hp = build_host_plan(block_terms[blk], L, tv.bt, tv.rb, tv.nbuf, tv.pf, rot, 2 * sizeof(T),
                                  resident_bits(tv), tv.sr, tv.w);
    upload_plan(hp, tv.bt, tv.rb, p, slab, tv.sr, 2 * sizeof(T));
    p.variant = variant;
    return p;
}
template const ApplyPlan &Hamiltonian::plan<float>(int, int, int);
template const ApplyPlan &Hamiltonian::plan<double>(int, int, int);

template <typename T>
int Hamiltonian::internal_rotation(int variant) {
    if (L < kTiledMinL) return 0;
    const int prec = sizeof(T) == 8 ? 1 : 0;
    const TiledVariant &tv = tiled_variants<T>().at(variant);     // throws for an unknown variant
    std::lock_guard<std::mutex> g(dev_mu);
    auto it = rotation.find({prec, variant});
    if (it == rotation.end())
        it = rotation.emplace(std::make_pair(prec, variant), choose_rotation(block_terms[0], L, tv.bt, resident_bits(tv),
                                                                              tv.w)).first;
    return it->second;
}
template int Hamiltonian::internal_rotation<float>(int);
template int Hamiltonian::internal_rotation<double>(int);

template <typename T>
int Hamiltonian::variant() {
    int d = 0;
    if (hipGetDevice(&d) != hipSuccess) d = 0;       // host-only queries: nothing tuned yet
    std::lock_guard<std::mutex> g(dev_mu);
    auto it = tuned.find({sizeof(T) == 8 ? 1 : 0, d});
    return it == tuned.end() ? default_variant<T>(L) : it->second;
}
template int Hamiltonian::variant<float>();
template int Hamiltonian::variant<double>();

template <typename T>
bool served_tiled(Hamiltonian &h, int rot) {
    if (rot != 0 && h.L < kTiledMinL) fail(SYK_EDEVICE, "rotated layouts are only planned for tiled blocks");
    return rot != 0 || h.tiled<T>();
}
template bool served_tiled<float>(Hamiltonian &, int);
template bool served_tiled<double>(Hamiltonian &, int);

template <typename T>
void apply_block(Hamiltonian &h, int blk, int rot, const T *x, T *y, int nvec, uint64_t ld, hipStream_t s) {
    if (served_tiled<T>(h, rot)) {
        launch_apply_tiled<T>(h.plan<T>(blk, rot, h.variant<T>()), x, y, nvec, ld, s);
    } else {
        apply_gather<T>(h, {blk, blk}, 1, x, y, nvec, ld, s);
    }
}

template <typename T>
void apply_full(Hamiltonian &h, const T *x, T *y, int nvec, uint64_t ld, hipStream_t s) {
    const uint64_t nb = 1ULL << h.L;
    if (h.tiled<T>()) {
        apply_block<T>(h, SYK_BLOCK_U, 0, x, y, nvec, ld, s);
        apply_block<T>(h, SYK_BLOCK_D, 0, x + 2 * nb, y + 2 * nb, nvec, ld, s);
    } else {
        apply_gather<T>(h, {SYK_BLOCK_U, SYK_BLOCK_D}, 2, x, y, nvec, ld, s);
    }
}
template void apply_full<float>(Hamiltonian &, const float *, float *, int, uint64_t, hipStream_t);
template void apply_full<double>(Hamiltonian &, const double *, double *, int, uint64_t, hipStream_t);
template void apply_block<float>(Hamiltonian &, int, int, const float *, float *, int, uint64_t, hipStream_t);
template void apply_block<double>(Hamiltonian &, int, int, const double *, double *, int, uint64_t, hipStream_t);

template <typename T>
int apply_block_lanczos(Hamiltonian &h, int blk, int rot, bool tiled, const T *x, T *y, const LanczosFuse<T> &lf,
                        hipStream_t s) {
    if (!tiled) {
        return apply_gather<T>(h, {blk, blk}, 1, x, y, 1, 1ULL << h.L, s, &lf);
    }
    const ApplyPlan &pl = h.plan<T>(blk, rot, h.variant<T>());
    if (pl.n_wg > lanczos_partials_max(h.L)) fail(SYK_EDEVICE, "partials buffer too small");
    launch_apply_tiled<T>(pl, x, y, 1, 1ULL << h.L, s, &lf);
    return static_cast<int>(pl.n_wg);
}
template int apply_block_lanczos<float>(Hamiltonian &, int, int, bool, const float *, float *,
                                        const LanczosFuse<float> &, hipStream_t);
template int apply_block_lanczos<double>(Hamiltonian &, int, int, bool, const double *, double *,
                                         const LanczosFuse<double> &, hipStream_t);

// Step j of one launch reads three vectors per term where two launches read one, and adds up three sums
// before its first term.  That costs less than a launch (about 4 us from one dependent launch to the
// next) while the further reads stay below 16 MB.  Two launches / one, a propagation of 12 steps in
// complex128: N = 16 151 / 136 us, N = 24 154 / 147 us (6 MB), N = 26 155 / 148 us (14 MB), N = 28 k = 2 153 / 152 us
// (15 MB), N = 26 k = 8 161 / 162 us (27 MB), N = 28 k = 4 155 / 157 us (29 MB) and k = 8 162 / 174 us (59 MB); of 10 steps in
// complex64: N = 20 133 / 121 us, N = 28 k = 2 135 / 128 us (7 MB), N = 26 k = 8 141 / 142 us (14 MB), N = 28 k = 4 137 / 134
// us (15 MB) and k = 8 143 / 148 us (29 MB).
template <typename T>
bool one_launch_steps(Hamiltonian &h) {
    return h.L <= 13 && !h.grouped() && 2.0 * h.K * static_cast<double>(1u << h.L) * 2 * sizeof(T) <= 16e6;
}
template bool one_launch_steps<float>(Hamiltonian &);
template bool one_launch_steps<double>(Hamiltonian &);

template <typename T>
int apply_step(Hamiltonian &h, int blk, const LanczosStep<T> &st, hipStream_t s) {
    return launch_lanczos_step<T>(gather_terms<T>(h.tables(blk)), st, 1u << h.L, s);
}
template int apply_step<float>(Hamiltonian &, int, const LanczosStep<float> &, hipStream_t);
template int apply_step<double>(Hamiltonian &, int, const LanczosStep<double> &, hipStream_t);

// Time the compiled variants of the tiled kernel on this Hamiltonian (block U, each in
// its own planned layout; force: every one, also if the handle is tuned already) and keep the
// fastest for the current device.  x, y: scratch device vectors of 2^L amplitudes.
template <typename T>
int autotune(Hamiltonian &h, T *x, T *y, hipStream_t s, bool force, std::vector<float> *times) {
    if (h.L < kTiledMinL) return -1;
    int dev = 0;
    SYK_HIP(hipGetDevice(&dev));
    if (!force) {
        std::lock_guard<std::mutex> g(h.dev_mu);
        auto it = h.tuned.find({sizeof(T) == 8 ? 1 : 0, dev});
        if (it != h.tuned.end()) return it->second;
    }
    const auto &vars = tiled_variants<T>();
    // On the way to an OTOC only the variants that can win are planned and timed: those with control
    // blocks whose workgroup holds the most amplitudes that still leave 512 workgroups, or more (or within
    // a factor two of the widest).  Of all 17, the fastest was one of these at every N from 40 to 56, k = 2, 4
    // and 8; at N = 52, complex64, that is 4 variants and 0.13 s against 0.36 s.
    int widest = 0;
    for (const TiledVariant &tv : vars) widest = std::max(widest, tv.bt + tv.w);
    widest = std::min(widest - 1, h.L - 9);
    const uint64_t n = 1ULL << h.L;
    const int np = reduction_blocks(n);
    double *part = nullptr;
    SYK_HIP(hipMalloc(reinterpret_cast<void **>(&part), (np + 1) * sizeof(double)));
    hipEvent_t e0, e1;
    SYK_HIP(hipEventCreate(&e0));
    SYK_HIP(hipEventCreate(&e1));
    int best = default_variant<T>(h.L);
    float best_ms = 1e30f;
    if (times) times->assign(vars.size(), -1.0f);
    try {
        launch_haar_raw<T>(1, 0, h.L - 1, 0, x, x + n, part, np, s);     // any finite data
        for (int v = 0; v < static_cast<int>(vars.size()); ++v) {
            if (vars[v].bt + vars[v].w + 3 > h.L) continue;              // needs >= 8 workgroups
            if (!force && (vars[v].sr != 2 || vars[v].bt + vars[v].w < widest)) continue;
            const ApplyPlan &pl = h.plan<T>(0, h.internal_rotation<T>(v), v);
            launch_apply_tiled<T>(pl, x, y, 1, n, s);                    // warm-up
            SYK_HIP(hipEventRecord(e0, s));
            for (int k = 0; k < 3; ++k) launch_apply_tiled<T>(pl, x, y, 1, n, s);
            SYK_HIP(hipEventRecord(e1, s));
            SYK_HIP(hipEventSynchronize(e1));
            float ms = 0.0f;
            SYK_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (times) (*times)[v] = ms / 3.0f;
            if (ms < best_ms) {
                best_ms = ms;
                best = v;
            }
        }
    } catch (...) {
        ignore_status(hipEventDestroy(e0));
        ignore_status(hipEventDestroy(e1));
        ignore_status(hipFree(part));
        throw;
    }
    ignore_status(hipEventDestroy(e0));
    ignore_status(hipEventDestroy(e1));
    ignore_status(hipFree(part));
    std::lock_guard<std::mutex> g(h.dev_mu);
    h.tuned[{sizeof(T) == 8 ? 1 : 0, dev}] = best;
    return best;
}
template int autotune<float>(Hamiltonian &, float *, float *, hipStream_t, bool, std::vector<float> *);
template int autotune<double>(Hamiltonian &, double *, double *, hipStream_t, bool, std::vector<float> *);

Hamiltonian::~Hamiltonian() {
    int cur = 0;
    bool have = hipGetDevice(&cur) == hipSuccess;
    for (int b = 0; b < 2; ++b) {
        for (size_t d = 0; d < dev[b].size(); ++d)
            if (dev[b][d].K) {
                if (have) ignore_status(hipSetDevice(static_cast<int>(d)));
                free_tables(dev[b][d]);
            }
    }
    for (auto &kv : plans)
        if (kv.second.pi) {
            if (have) ignore_status(hipSetDevice(std::get<2>(kv.first)));
            free_plan(kv.second);
        }
    if (have) ignore_status(hipSetDevice(cur));
}

// ------------------------------------------------------------------ workspaces
DeviceBuffer::~DeviceBuffer() { release(); }

void DeviceBuffer::ensure(size_t bytes) {
    if (bytes <= n_) return;
    if (!owned_)
        fail(SYK_ENOMEM, "workspace needs " + std::to_string(bytes) + " bytes, its caller-owned region holds " +
                             std::to_string(n_));
    release();
    void *p = nullptr;
    const hipError_t e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        ignore_status(hipGetLastError());        // reported here, not by the next launch's check too
        hip_check(e, "hipMalloc of a workspace");
    }
    p_ = static_cast<char *>(p);
    n_ = bytes;
}

void DeviceBuffer::release() {
    if (p_ && owned_) ignore_status(hipFree(p_));
    p_ = nullptr;
    n_ = 0;
    owned_ = true;
}

void DeviceBuffer::adopt(void *p, size_t bytes) {
    release();
    p_ = static_cast<char *>(p);
    n_ = bytes;
    owned_ = false;
}

namespace {
struct WsKey {
    int dev;
    std::thread::id tid;
    int slot;
    bool operator<(const WsKey &o) const {
        if (dev != o.dev) return dev < o.dev;
        if (tid != o.tid) return tid < o.tid;
        return slot < o.slot;
    }
};
std::mutex ws_mu;
std::map<WsKey, DeviceBuffer> *ws_map() {
    static auto *m = new std::map<WsKey, DeviceBuffer>();   // never destroyed: no HIP calls at exit
    return m;
}
}  // namespace

DeviceBuffer &thread_workspace(int slot) {
    int dev = 0;
    SYK_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(ws_mu);
    return (*ws_map())[WsKey{dev, std::this_thread::get_id(), slot}];
}

void release_thread_workspaces() {
    int dev = 0;
    SYK_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(ws_mu);
    auto *m = ws_map();
    for (auto it = m->begin(); it != m->end();) {
        if (it->first.dev == dev && it->first.tid == std::this_thread::get_id())
            it = m->erase(it);
        else
            ++it;
    }
}

}  // namespace syk
