// Batched OTOC (one persistent launch over many small-N realisations and random vectors).
#pragma once

#include <vector>

#include "internal.hpp"

namespace syk {

constexpr int kMaxKrylov = 60;          // largest Krylov dimension of the batched path

// One term of a block as the kernel reads it, for a launch shape of NT threads and LDS chunks of
// CH amplitudes; thread t holds amplitudes t + NT r of a chunk, r < RC = CH / NT.  The host sorts the
// terms into runs by partner chunk, phase and the lowest `low` register bits (two, or all where RC
// < 4) of x and of z, so that each run's registers and signs are known to the compiled code up
// to the higher register bits, which the record holds.
struct BatchTerm {
    uint32_t xb;                        // x inside the chunk times 8 bytes, its low register bits cleared
    uint32_t zt;                        // z: thread bits, then chunk bits
    float c;                            // coefficient, the parity of x & z folded in
    uint32_t sg;                        // bit h: sign of the registers with higher bits h
};
constexpr int batch_low_bits(int rc) { return rc >= 4 ? 2 : rc >= 2 ? 1 : 0; }
// runs per partner chunk: (phase, low x bits, low z bits), z fastest; the table holds runs + 1 bounds
constexpr int batch_runs(int rc) { return 2 << (2 * batch_low_bits(rc)); }

// one job: a realisation and one Haar vector
struct BatchJob {
    int L, N, K, pad;
    uint32_t term_off[2];               // first term of block U / D in BatchParams::terms
    uint32_t wx, wz;                    // W = chi_i block form (x, z, phase i^ww), w_top: i == N - 1
    int ww, w_top;
    uint32_t vx, vz;                    // V = chi_j
    int vw, v_top;
    uint64_t base;                      // Haar generator base of this vector
    double beta;
    uint32_t run_off[2];                // block U / D in BatchParams::runs: bounds by partner chunk
};

// One part of a job, the unit a workgroup takes: the chain that starts in parity block A, for the
// t points [k0, k1).  A part with k0 > 0 repeats the incremental propagations up to k0 (in the same
// steps, so its results do not depend on the split); stats count them in the part that owns them.
struct BatchPart {
    int job, A, k0, k1;
};

// what a part reports
struct BatchResult {
    long long matvecs;
    int substeps, status;               // status: 0, SYK_ENOTCONV, SYK_ENUMERIC, SYK_EUNSUPPORTED
};

struct BatchParams {
    const BatchJob *jobs;
    const BatchPart *parts;
    int n_parts;
    const BatchTerm *terms;
    const uint32_t *runs;               // run bounds, indices into a block's terms
    const double *ts;                   // t grid (t[0] = 0)
    int nt;
    int m;                              // Krylov dimension
    double tol;
    int max_substeps;                   // per part, over all propagations
    float2 *ws;                         // per slot: (m + 5) vectors of vec_stride amplitudes
    uint64_t slot_stride, vec_stride;   // in amplitudes
    double *F;                          // per job and block A: nt complex (re, im)
    unsigned *counter;                  // next part; zero at launch
    BatchResult *results;               // per part
};

// launch shape: threads per workgroup, LDS staging chunk 2^chb amplitudes, workgroups per CU
struct BatchVariant {
    int nt, chb, occ;
};
const std::vector<BatchVariant> &batch_variants();
bool batch_variant_supports(const BatchVariant &v, int L);
void launch_otoc_batch(const BatchVariant &v, const BatchParams &p, int grid, hipStream_t s);

// the whole batched request (arguments checked by the caller); synchronises s
void otoc_batch(const syk_batch_item *items, int n_items, const double *t, int nt, const syk_batch_opts &o,
                double *F_raw, double *F_norm, double *F_imag, syk_batch_stats &st, hipStream_t s);

}  // namespace syk
