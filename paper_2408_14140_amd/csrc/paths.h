// paths.h -- host-side entry points of the plain and batched loops.
#pragma once

#include "ibx_internal.h"

namespace ibx {

void desired_velocity(const ib_particles* p, const ib_markers* m, ib_prec prec, void* Ud,
                      hipStream_t st);

// Deterministic sum (fixed chunking and tree) of v[0..n) into *out (sqrt if asked).
void sum_to(const double* v, int64_t n, double* part, double* out, bool do_sqrt, hipStream_t st);
size_t sum_partials(int64_t n);
size_t field_elems(const Grid& g);

void plain_spread(const Grid& g, int P, ib_prec prec, const ib_markers* m, const ib_buckets* b,
                  const void* F, void* f, double scale, int use_dv, hipStream_t st);

size_t plain_workspace(const Grid& g, ib_prec prec, int64_t nl);
int plain_multidirect(const Grid& g, int P, ib_prec prec, const ib_particles* p,
                      const ib_markers* m, const ib_buckets* b, int ns, double dt,
                      const void* u0, void* ustar, void* f, void* F, double* resid, void* Fhist,
                      void* ws, size_t ws_bytes, hipStream_t st);

struct BatchedCfg {
    int bw;        // markers per interpolation work item (= threads per workgroup)
    int ncu;       // compute units of the device
    int wgs_s;     // cap on resident spreading workgroups per CU (0 = as many as fit)
    int masks;     // G slot row masks: zero rows neither stored nor loaded
    int txw;       // x extent of an interpolation work tile: 8 (one tile) or 16 (FP32)
    Profiler* prof;  // nullable: per-kernel event timing
    int products = 0;  // FP32: spread by matrix products (FP64 always does)
};

size_t batched_workspace(const Grid& g, ib_prec prec, int64_t nl, const BatchedCfg& cfg);
int batched_multidirect(const Grid& g, int P, ib_prec prec, const BatchedCfg& cfg,
                        const ib_particles* p, const ib_markers* m, const ib_buckets* b, int ns,
                        double dt, const void* u0, void* ustar, void* f, void* F, double* resid,
                        void* Fhist, void* ws, size_t ws_bytes, hipStream_t st, int f_acc = 0);

// The adjoint on the loop's tile kernels: records and work lists once per call,
// then a step at a time.  Grids with fewer than 16 cells on an axis, or boxes above
// 512, are not supported (tile_adjoint_supported).
bool tile_adjoint_supported(const Grid& g);
size_t tile_adjoint_workspace(const Grid& g, ib_prec prec, int64_t nl);
int tile_adjoint_setup(const Grid& g, int P, ib_prec prec, const BatchedCfg& cfg,
                       const ib_particles* p, const ib_markers* m, const ib_buckets* b, void* ws,
                       size_t ws_bytes, hipStream_t st);
// One step m of the reverse sweep (backward.hip), steps in order from ns: Ui = J a_f,
// a_F += (dV/h^3) Ui, a_Ud += a_F/dt, Ub = -a_F/dt, gu0 += a_u = J^T Ub on every
// valid covered cell, and gX += both position gradients.  af (the field, box layout)
// is given for the first step; later ones take a_f = dt a_u from the step before,
// which the workspace holds.  Fm = F^m, Fp = F^(m-1) (null for m = 1); marker
// arrays [nl][3] in marker order.
int tile_adjoint_step(const Grid& g, int P, ib_prec prec, const BatchedCfg& cfg,
                      const ib_markers* m, const ib_buckets* b, double dt, const void* af,
                      const void* Fm, const void* Fp, const void* u0, void* Ui, void* aF,
                      double* aUd, void* Ub, void* gu0, double* gX, void* ws, size_t ws_bytes,
                      hipStream_t st);

// Particle-by-particle order of the loop, run level by level (sequential.hip).
constexpr int SEQ_MAX_LEVELS = 4096;
size_t sequential_workspace(const ib_level* lv, const Grid& g, ib_prec prec, int32_t np,
                            int64_t nl, const BatchedCfg& cfg);
int sequential_multidirect(const ib_level* lv, const Grid& g, int P, ib_prec prec,
                           const BatchedCfg& cfg, const ib_particles* p, const ib_markers* m,
                           int ns, double dt, const int32_t* level, int32_t nlevels,
                           const void* u0, void* ustar, void* f, void* F, int32_t* flag,
                           void* ws, size_t ws_bytes, hipStream_t st);

}  // namespace ibx

namespace ibx {
size_t backward_workspace(const Grid& g, ib_prec prec, int64_t nl);
int multidirect_backward(const Grid& g, int P, ib_prec prec, const BatchedCfg& cfg,
                         const ib_particles* p,
                         const ib_markers* m, const ib_buckets* b, int ns, double dt,
                         const void* u0, const void* Fhist, const void* gus, const void* gf,
                         const void* gF, void* gu0, double* gup, double* gom, double* gX,
                         void* ws, size_t ws_bytes, hipStream_t st);
}  // namespace ibx
