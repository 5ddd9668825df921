// Internal declarations of libsyk shared by the host sources and the HIP kernels.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstddef>
#include <map>
#include <mutex>
#include <set>
#include <tuple>
#include <string>
#include <vector>

#include "../../include/syk.h"

namespace syk {

// ------------------------------------------------------------------ errors
struct Error {
    syk_status status;
    std::string msg;
};
[[noreturn]] void fail(syk_status s, const std::string &msg);
void hip_check(hipError_t e, const char *what);
#define SYK_HIP(call) ::syk::hip_check((call), #call)
// Cleanup paths (destructors, unwinding after an error): a failure to release a resource
// cannot be reported from there, so its status is dropped on purpose.
inline void ignore_status(hipError_t) {}

// ------------------------------------------------------------------ terms
// One term of Eq. (1) on one parity block, reduced for the kernels:
//   (J/4) i^p X^x Z^z acting as  y[m] += c * i^{imag} * (-1)^{popc(m & z)} * x[m ^ x]
// where the sign (-1)^{popc(x & z)} of reading the Z bits from the source index m ^ x has
// been folded into c together with the real sign of i^p; imag = p odd.
struct BlockTerm {
    uint32_t x, z;
    double c;
    bool imag;
};

// A region of device memory handed out front to back in 256-byte aligned pieces; nothing
// in it is freed piece by piece (its owner returns the region as a whole).
struct DeviceSlab {
    char *base = nullptr;
    size_t size = 0, used = 0;
    // next piece of `bytes`; ENOMEM naming `what` when the region is exhausted
    void *take(size_t bytes, const char *what);
};

// One term of the gather kernels (16 bytes in either precision): y[m] += c (-1)^{popc(m & z)}
// x[m ^ x], times i for the i-phase terms, which follow the real-phase ones.
template <typename T> struct GatherTerm;
template <> struct GatherTerm<float> {
    uint32_t x, z;
    float c;
    uint32_t pad;
};
template <> struct GatherTerm<double> {
    uint32_t x, z;
    double c;
};
template <typename T>
struct GatherTerms {
    const GatherTerm<T> *rec = nullptr;
    uint32_t K = 0;
    uint32_t cut[3] = {0, 0, 0};             // ends of (real, even x), (real, odd x), (i-phase, even x)
};

// Terms of the grouped gather kernel: groups of equal x mask, cut into steps of four terms of
// one phase, a real and an i-phase step in turn (padded with zero coefficients).  hdr[s] of the
// real step s is zero but for the last pair of a group: kDenseEnd and in bits 0..27 the next
// group's x mask.
// The steps are dealt to kDenseSlices slices of whole groups, slice q holding steps
// [cut[q], cut[q + 1]), a multiple of kDenseChunk (padded with empty steps); first[q] is the
// x mask of its first group.  The header table starts with cut (kDenseSlices + 1 words) and
// first (kDenseSlices), the step headers follow at word kDenseHead.
constexpr int kDenseSlices = 16, kDenseChunk = 16, kDenseHead = 64;
constexpr uint32_t kDenseEnd = 1u << 31;
template <typename T> struct DenseTerm;
template <> struct DenseTerm<float> {
    uint32_t z;
    float c;
};
template <> struct DenseTerm<double> {
    uint32_t z, pad;
    double c;
};
template <typename T>
struct DenseTerms {
    const uint32_t *head = nullptr;
    const DenseTerm<T> *rec = nullptr;       // four per step
};

struct DeviceTables {            // per device, per block: the gather kernels' term tables
    bool in_slab = false;        // carved from a DeviceSlab: not freed by the library
    char *mem = nullptr;         // holds what the pointers below point into
    GatherTerm<float> *r32 = nullptr;
    GatherTerm<double> *r64 = nullptr;
    uint32_t K = 0, cut[3] = {0, 0, 0};
    // the grouped form, for blocks that use it (null otherwise)
    uint32_t *head = nullptr;
    DenseTerm<float> *d32 = nullptr;
    DenseTerm<double> *d64 = nullptr;
};
// Blocks whose terms share x masks this often or more (terms per mask) use the grouped form,
// from one 64-amplitude tile up to 2^22 amplitudes, where the gathers still come from the
// 256 MB last-level cache.  Dense SYK, grouped / best tiled variant, complex64 and complex128: N = 38 0.73 / 8.2
// and 1.21 / 10.6 ms, N = 42 3.9 / 17 and 6.3 / 25 ms, N = 46 (2^22) 20.7 / 88 and 35 / 155 ms.  It is four times as
// fast at the limit and would be beyond it; larger dense blocks stay with the tiled kernel,
// which they had, until they are tested here.
constexpr int kDenseTermsPerMask = 4;
constexpr int kDenseMinL = 6, kDenseMaxL = 22;
// complex64 blocks up to this size take 64-amplitude tiles (complex128: one more)
constexpr int kDenseRowL32 = 14;

// distinct x masks of a block's terms: the groups the gather kernel loads once each
int gather_groups(const std::vector<BlockTerm> &terms);

// Compiled variant of the tiled apply_H kernel: tiles of 2^bt amplitudes, 2^rb per
// thread, nbuf LDS partner buffers (nbuf - 1 copies in flight; 1 = copy, then compute),
// pf extra partner entries at the end of the group list, occ workgroups resident per CU
// (the planner's XCD-resident subspace has dimension 5 + log2(occ)); sr = 1: each term's
// register permutation and register signs select a compiled code path (4-dword term
// records), sr = 0: they are read from the term record (4 + 2 * 2^rb dwords), sr = 2: each
// partner step's records sit in a 64-dword control block that a wave holds in one VGPR
// and reads with readlane (no scalar memory loads in the term loop; two buffers); each
// workgroup keeps 2^w output tiles in registers and streams the union of their partner
// tiles once.
struct TiledVariant {
    int bt, rb, nbuf, pf, occ, sr, w;   // w: each workgroup holds 2^w output tiles
};
inline int resident_bits(const TiledVariant &v) { return 5 + (v.occ >= 4 ? 2 : v.occ >= 2 ? 1 : 0); }
template <typename T>
const std::vector<TiledVariant> &tiled_variants();
// variant used before (or without) autotuning, for blocks of 2^L amplitudes
template <typename T>
int default_variant(int L);
// smallest block (in qubits) that the tiled kernel can serve
constexpr int kTiledMinL = 18;
// Blocks that fit the 4 MiB L2 of one XCD are gathered straight from there.  Gather against tiled
// apply at k = 4: 2^18 amplitudes 11.2 / 25.7 us in complex64 and 19.5 / 33.8 us in complex128 (4 MiB), 2^19
// amplitudes 21.5 / 29.8 us in complex64 (4 MiB) and 47 / 41 us in complex128 (8 MiB), 2^20 amplitudes
// 50 / 42 us in complex64 (8 MiB).
constexpr uint64_t kGatherBytes = 4ULL << 20;

// bit rotations within L bits: layout rotation s stores qubit (b + s) mod L at index bit b
uint32_t rotr_bits(uint32_t v, int s, int L);
uint32_t rotl_bits(uint32_t v, int s, int L);

struct ApplyPlan {
    bool in_slab = false;            // device arrays carved from a DeviceSlab: not freed by the library
    int bt = 0, rb = 0, rot = 0, variant = 0, w = 0;
    uint32_t n_tiles = 0;            // output tiles
    uint32_t n_wg = 0;               // workgroups (n_tiles >> w)
    uint32_t hvec[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // tiles of a workgroup: t0 ^ hvec[i], i < 2^w
    uint32_t *tile_map = nullptr;    // n_wg: blockIdx -> t0
    int n_pi = 0;
    uint32_t *pi = nullptr;          // n_pi + pf partner offsets (partner tile t0 ^ pi)
    uint32_t *ranges = nullptr;      // n_pi * 2^w * 3 term ranges (first, mid, end)
    uint32_t *meta = nullptr;        // K + 1 term records (see apply_tiled.hip)
    float *c32 = nullptr;
    double *c64 = nullptr;
};

// Optional epilogue of apply_H for Lanczos step j, where the basis is stored unnormalised:
// slot i holds u_i with n_i = ||u_i|| (so v_i = u_i / n_i and beta_i = n_{i+1}); slot 0 is the start
// vector itself.  With x = u_j (vcur) the epilogue forms
//   y = H v_j - beta_{j-1} v_{j-1} = H u_j / n_j - (n_j / n_{j-1}) u_{j-1}
// (vprev = u_{j-1}, null for j = 0) and one partial sum of Re <v_j, y> per workgroup at
// partials[blockIdx.x].  norm2[i] = n_i^2 (device) holds n_{j-1}, and n_j too where the tiled kernel
// runs; the gather kernels take n_j^2 as the sum of the n_parts partials at norm_parts (left by the pass
// that wrote u_j) and workgroup 0 writes it to norm2[j] and to norm2_host.
template <typename T>
struct LanczosFuse {
    const T *vprev = nullptr;
    const T *vcur = nullptr;
    double *norm2 = nullptr;           // device, indexed by basis slot
    int j = 0;
    double *partials = nullptr;
    const double *norm_parts = nullptr;
    int n_parts = 0;
    double *norm2_host = nullptr;      // pinned host memory, the slot of n_j^2
};

// One launch per Lanczos step (small sparse blocks).  Step j forms u_j wherever it reads it, from
// g = H u_{j-1}, u1 = u_{j-1}, u2 = u_{j-2} and the sums over them that step j - 1 left (three per workgroup:
// ||u_{j-1}||^2, Re <u_{j-1}, g>, Re <u_{j-1}, u_{j-2}>), writes u_j (j >= 1) and H u_j, and leaves its own sums.
// Step 0 reads u_0 as g.
template <typename T>
struct LanczosStep {
    const T *g = nullptr, *u1 = nullptr, *u2 = nullptr;
    T *u = nullptr, *gout = nullptr;
    const double *parts = nullptr;
    int np = 0, j = 0;
    double *out = nullptr;                            // 3 per workgroup
    double *norm2 = nullptr, *alpha = nullptr;        // device, indexed by step
    double *norm2_host = nullptr, *alpha_host = nullptr;   // pinned slots of step j - 1
    double *next_host = nullptr;                      // close: the slot of ||u_j||^2
};

// ------------------------------------------------------------------ host-side model
uint64_t splitmix_mix(uint64_t z);

struct Hamiltonian {
    int N = 0, L = 0, K = 0;
    double k = 0, p = 0, sigma = 0, sum_J2 = 0;
    double c_max = 0;                  // largest |c| of the block terms
    uint64_t seed = 0;
    int ensemble = 0;                  // -1: a general operator (syk_op_to_hamiltonian)
    bool hermitian = true;
    std::vector<int32_t> ijkl;         // 4K, sorted subsets
    std::vector<double> J;             // K
    std::vector<uint64_t> xmask, zmask;
    std::vector<int8_t> phase[2];      // U, D
    std::vector<BlockTerm> block_terms[2];   // kernel order: real first, then imaginary
    int n_real[2] = {0, 0};

    // where device tables and plans come from: hipMalloc (null) or a slab that outlives the
    // handle (the request engine carves each request's tables from its arena)
    DeviceSlab *slab = nullptr;
    std::mutex dev_mu;
    std::vector<DeviceTables> dev[2];  // indexed by device ordinal
    // plans keyed by (block, double?, device, rotation, variant)
    std::map<std::tuple<int, int, int, int, int>, ApplyPlan> plans;
    std::map<std::pair<int, int>, int> rotation;               // (double?, variant) -> planned rotation
    std::map<std::pair<int, int>, int> tuned;                   // (double?, device) -> variant
    std::set<std::pair<int, int>> pinned;                       // those of them chosen by syk_select_variant, until syk_autotune
    // whether the tiled kernel serves the block on the current device: blocks of at least
    // 2^kTiledMinL amplitudes, except, unless a tiled variant is pinned, those that fit an L2
    // (kGatherBytes) and dense ones that the grouped gather kernel serves
    template <typename T>
    bool tiled();
    bool grouped();                       // the terms share x masks often enough for the grouped form
    int grouped_ = -1;                    // cached grouped(): -1 not yet known
    const DeviceTables &tables(int blk);
    template <typename T>
    const ApplyPlan &plan(int blk, int rot, int variant);
    template <typename T>
    int internal_rotation(int variant);   // layout used inside Krylov/OTOC runs (0 if not tiled)
    template <typename T>
    int variant();                        // tuned variant on the current device, else the default
    ~Hamiltonian();
};

void build_hamiltonian(Hamiltonian &h, int N, double k, uint64_t seed, int ensemble = SYK_ENSEMBLE_EXACT_K);

// canonical Pauli string i^w X^x Z^z of block Majorana A_n (0 <= n <= N-2) on L qubits
void block_majorana(int N, int n, uint32_t &x, uint32_t &z, int &w);

// ------------------------------------------------------------------ device workspace
class DeviceBuffer {
  public:
    DeviceBuffer() = default;
    ~DeviceBuffer();
    DeviceBuffer(const DeviceBuffer &) = delete;
    DeviceBuffer &operator=(const DeviceBuffer &) = delete;
    void ensure(size_t bytes);
    void release();
    // use caller-owned device memory of `bytes` instead of allocating: ensure() then never
    // allocates (ENOMEM beyond `bytes`) and release() only forgets the pointer
    void adopt(void *p, size_t bytes);
    char *ptr() const { return p_; }
    size_t size() const { return n_; }

  private:
    char *p_ = nullptr;
    size_t n_ = 0;
    bool owned_ = true;
};

// per-(device, thread) cached workspace used by the convenience entry points
DeviceBuffer &thread_workspace(int slot);

// whether the tiled kernel serves vectors in layout rotation `rot`: any rotated layout (the gather kernels
// know the standard one only), and the standard one where Hamiltonian::tiled() says so
template <typename T>
bool served_tiled(Hamiltonian &h, int rot);
// y = H_blk x on the device: tiled kernel for large blocks, gather kernels otherwise
template <typename T>
void apply_block(Hamiltonian &h, int blk, int rot, const T *x, T *y, int nvec, uint64_t ld, hipStream_t s);
// the same on both blocks of the full space (U, then D at element offset 2^L), layout 0
template <typename T>
void apply_full(Hamiltonian &h, const T *x, T *y, int nvec, uint64_t ld, hipStream_t s);
// y = H_blk x with the fused Lanczos epilogue; returns the number of partials written (one per
// workgroup).  tiled: served_tiled() as it was when the run began (a variant pinned or forgotten by
// another thread must not change who adds the partials up)
template <typename T>
int apply_block_lanczos(Hamiltonian &h, int blk, int rot, bool tiled, const T *x, T *y, const LanczosFuse<T> &lf,
                        hipStream_t s);
// whether one launch per Lanczos step serves the block (apply_step)
template <typename T>
bool one_launch_steps(Hamiltonian &h);
// Lanczos step st.j of a block; returns the number of workgroups (triples of sums in st.out)
template <typename T>
int apply_step(Hamiltonian &h, int blk, const LanczosStep<T> &st, hipStream_t s);
template <typename T>
void launch_lanczos_close(const LanczosStep<T> &st, uint32_t n, hipStream_t s);
template <typename T>
int launch_lanczos_step(const GatherTerms<T> &tb, const LanczosStep<T> &st, uint32_t n, hipStream_t s);
// upper bound on the partials apply_block_lanczos writes for a block of 2^L amplitudes (tiled:
// one per tile of 2^10 or more; gather: at most 512 workgroups below the tiled size, and at
// most one per 256 amplitudes above it)
inline uint64_t lanczos_partials_max(int L) {
    return L >= kTiledMinL ? 1ULL << (L > kDenseMaxL ? L - 10 : L - 8) : 512;
}
// time the tiled-kernel variants and keep the fastest; returns it (-1: block not tiled)
template <typename T>
int autotune(Hamiltonian &h, T *x, T *y, hipStream_t s, bool force, std::vector<float> *times = nullptr);

// ------------------------------------------------------------------ kernels (HIP side)
// All launchers enqueue on `s` and never synchronise.
// gather kernels over nblk blocks side by side (2: U, then D at element offset n); with lf (one
// block, one vector) the Lanczos epilogue.  Return the workgroups launched per vector and block.
template <typename T>
int launch_apply_gather(const GatherTerms<T> (&tb)[2], int nblk, const T *x, T *y, uint32_t n, int nvec, uint64_t ld,
                        hipStream_t s, const LanczosFuse<T> *lf = nullptr);
template <typename T>
int launch_apply_dense(const DeviceTables *const (&tb)[2], int nblk, const T *x, T *y, uint32_t n, int nvec,
                       uint64_t ld, hipStream_t s, const LanczosFuse<T> *lf = nullptr);
// psi in layout rotation `rot`: index p holds standard amplitude rotl(p, rot)
template <typename T>
void launch_haar_raw(uint64_t state_seed, int v, int L, int rot, T *psi_U, T *psi_D, double *partials, int n_part,
                     hipStream_t s);
template <typename T>
void launch_scale_pair(T *a, T *b, uint64_t n, const double *inv_norm_dev, hipStream_t s);
template <typename T>
void launch_majorana(uint32_t x, uint32_t z, int w, double sre, double sim, const T *src, T *dst, uint64_t n,
                     hipStream_t s);
// partial reductions: out[b] for b < n_part, each (re, im) or (sum) in double
template <typename T>
void launch_dot_partials(const T *a, const T *b, uint64_t n, double *partials, int n_part, hipStream_t s);
template <typename T>
void launch_norm2_partials(const T *a, uint64_t n, double *partials, int n_part, hipStream_t s);
// reduce `n_part` partials of width `width` into dst[0..width) (single workgroup, fixed order)
void launch_reduce_partials(const double *partials, int n_part, int width, double *dst, hipStream_t s);

// Lanczos building blocks (scalars live on the device, see krylov.cpp)
template <typename T>
void launch_lanczos_orth1(T *w, const T *vprev, const T *vcur, const double *beta_prev, uint64_t n,
                          double *partials, int n_part, hipStream_t s);
template <typename T>
void launch_lanczos_orth2(T *w, const T *vcur, const double *alpha, uint64_t n, double *partials, int n_part,
                          hipStream_t s);
template <typename T>
void launch_lanczos_normalize(T *w, const double *beta, uint64_t n, hipStream_t s);
// The scalars of the fused path are summed over per-workgroup partials in a fixed order (256
// threads striding the partials, then lanes, then waves), wherever the sum is formed, and each is also
// stored to a slot of pinned host memory.
// dst = dst_host = sum of n_part partials
void launch_publish_sum(const double *partials, int n_part, double *dst, double *dst_host, hipStream_t s);
// u_{j+1} = w - (alpha_j / n_j) u_j in place on w (v = u_j, n_j^2 = norm2[j]), and n_part partials of
// ||u_{j+1}||^2.  a_parts > 0: alpha_j is the sum of a_parts partials at a_part, which every workgroup
// forms (workgroup 0 stores it to alpha and alpha_host); 0: alpha_j is read from alpha.
template <typename T>
void launch_lanczos_residual(T *w, const T *v, double *alpha, double *alpha_host, const double *a_part, int a_parts,
                             const double *norm2, int j, uint64_t n, double *partials, int n_part, hipStream_t s);
// the sum of many partials in two stages (stage: 512 doubles), published as launch_publish_sum
void launch_publish_sum2(const double *partials, int n_part, double *stage, double *dst, double *dst_host,
                         hipStream_t s);
template <typename T>
void launch_scale_copy(const T *src, T *dst, uint64_t n, double scale, hipStream_t s);
// out = coef[0] v0 + sum_{k >= 1} coef[k] basis_k (complex coefficients); out may equal v0
template <typename T>
void launch_combine(const T *v0, const T *basis, uint64_t stride, int nb, const double *coef_dev, T *out, uint64_t n,
                    hipStream_t s);
// the same for nb <= kCombineArgs vectors with the coefficients (host) passed by value
constexpr int kCombineArgs = 64;
template <typename T>
void launch_combine_args(const T *v0, const T *basis, uint64_t stride, int nb, const double *coef, T *out, uint64_t n,
                         hipStream_t s);
// subtract projections: w -= sum_k c_k v_k with c_k = <v_k, w> taken from coef_dev (complex)
template <typename T>
void launch_subtract_proj(T *w, const T *basis, uint64_t stride, int nb, const double *coef_dev, uint64_t n,
                          hipStream_t s);
template <typename T>
void launch_multi_dot_partials(const T *basis, uint64_t stride, int nb, const T *w, uint64_t n, double *partials,
                               int n_part, hipStream_t s);

int reduction_blocks(uint64_t n);   // number of partials the reduction launchers produce
// this device's copy of the library's fixed device scratch (at least n_doubles doubles;
// EINVAL beyond its size); looked up once per device, never allocated
double *fixed_scratch(size_t n_doubles);
size_t fixed_scratch_doubles();

}  // namespace syk
