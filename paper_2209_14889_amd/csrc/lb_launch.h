// Host-callable launch wrappers of the liblb kernels (defined in lb_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "lb_common.h"

namespace lbk {

// message returned by lb_last_error() on this thread
void set_last_error(const char *msg);

// nmax: nodes of the largest body
hipError_t launch_ib(bool advance, int nbodies, int ntiles, int nmax, hipStream_t st, const SimDev *sims, BodyDev *bodies,
                     const int2 *blk, int cur, const int *d_t, int *d_status);
// walls: the variant with wall handling (needed when any simulation of the launch has walls);
// pol: the variant with the polarization field (needed unless P is zero in every simulation);
// any_body: the variant for launches with bodies;
// cus: the device's compute units (work-groups of the first round are dealt to them in turn)
hipError_t launch_fused(int T, bool fp16, bool walls, bool pol, bool any_body, int grid, hipStream_t st, const SimDev *sims,
                        const BodyDev *bodies, const WorkItem *items, int n_items, int cur, int *d_t, int cus);
// the same step with short items as tiles, one work-group per item (T: 64, 128 or 256)
hipError_t launch_tile(int T, bool fp16, bool walls, bool pol, hipStream_t st, const SimDev *sims, const BodyDev *bodies,
                       const WorkItem *items, int n_items, int cur, int *d_t);
// resident fused work-groups per compute unit for work-group size T
int fused_blocks_per_cu(int T, bool fp16, bool walls, bool pol, bool any_body);
hipError_t launch_multipass(bool fp16, int nblocks, hipStream_t st, const SimDev *sims, const BodyDev *bodies,
                            const SiteBlock *blk, int cur, int *d_t);
// the planes of `mask` (bits 0 .. 9 in the order of lb_read_fields), packed into out
constexpr unsigned kReadForce = 0x306u;   // those that need the force density: vx, vy, fpx, fpy
constexpr unsigned kReadPops = 0x007u;    // those that need the populations: rho, vx, vy
hipError_t launch_readout(bool fp16, int nblocks, int block0, hipStream_t st, const SimDev *sims,
                          const BodyDev *bodies, const SiteBlock *blk, int cur, unsigned mask, float *out);
hipError_t launch_sums(bool fp16, int sim, int nblocks, hipStream_t st, const SimDev *sims, int cur, double *partial,
                       double *out, double check_mass, int *d_status);
// body observables of bodies body0 .. body0+nbodies-1, 6 doubles each into out
hipError_t launch_body_force(hipStream_t st, const SimDev *sims, const BodyDev *bodies, int body0, int nbodies, int cur,
                             double *out);
// streaming device-to-device copy (bytes a multiple of 16, 16-byte aligned pointers)
hipError_t launch_stream_copy(hipStream_t st, const void *src, void *dst, size_t bytes);
hipError_t launch_pack(bool fp16, hipStream_t st, const float *src, void *dst, size_t n, float scale);

}  // namespace lbk
