// HIP kernels of one coupled TLED + Pennes time step for CDNA4 (gfx950).
//
// Two variants share the element physics of device_math.h:
//   two-pass: element kernel (one thread per element) writes its npe nodal
//     (force, heat) contributions; node kernel (one thread per node) sums its
//     incident contributions in a fixed order and advances the node;
//   fused patch: one workgroup per patch of contiguous elements stages the
//     patch nodes in LDS, computes the elements, assembles and advances the
//     patch-interior nodes in LDS, and writes partial sums for the nodes it
//     shares with other patches; a shared-node kernel finishes those.
// No atomics in the assembly; every sum has a fixed order, so a run is
// bitwise reproducible.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "step_math.h"

#include <hip/hip_ext.h>

// Launch with optional timing: with a start/stop event pair the events are taken
// by the dispatch itself (hipExtLaunchKernelGGL), so no extra packets sit
// between kernels and the elapsed time is the kernel's own duration.
#define TLED_LAUNCH(ev, kern, grid, block, lds, stream, ...)                                              \
    do {                                                                                                  \
        if (ev) hipExtLaunchKernelGGL(kern, grid, block, lds, stream, (ev)->start, (ev)->stop, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(kern, grid, block, lds, stream, __VA_ARGS__);                             \
    } while (0)


namespace tled {

// Runs after a step's node updates (only when the dose is enabled, so the
// solver kernels carry no trace of it).
__global__ __launch_bounds__(kBlock) void dose_kernel(const float4 *__restrict__ nu4, int nn,
                                                      double2 *__restrict__ dose, DoseParams q) {
    const int a = int(blockIdx.x) * kBlock + int(threadIdx.x);
    if (a < nn) add_thermal_dose(dose, q, size_t(a), nu4[a].w);
}

// ---------------------------------------------------------------- two-pass kernels

template <int NP, bool MON, int MODE>
__global__ __launch_bounds__(kBlock) void t4_element_kernel(
    const int4 *__restrict__ conn, const float4 *__restrict__ g0, const float4 *__restrict__ g1,
    const float4 *__restrict__ g2, const float4 *__restrict__ nu4, float *__restrict__ theta,
    float4 *__restrict__ out, int ne, KMat m, unsigned *__restrict__ status, double *__restrict__ part,
    const float4 *__restrict__ aniso) {
    __shared__ double shd[kBlock / 64];
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int e = blk * kBlock + threadIdx.x;
    float psi = 0.f;
    bool nf = false, inv = false;
    if (e < ne) {
        const int4 c = conn[e];
        float4 u[4] = {nu4[c.x], nu4[c.y], nu4[c.z], nu4[c.w]};
        float th[6 * NP + 1];
        load_theta(theta, ne, e, NP, th);
        ElemResultT4 r;
        t4_compute<NP, MODE>(MON, m, u, t4_geo_planes(g0[e], g1[e], g2[e]), th, r, aniso, e);
        store_theta(theta, ne, e, NP, th);
#pragma unroll
        for (int k = 0; k < 4; ++k) out[4 * size_t(e) + k] = r.o[k];
        psi = r.psiV;
        nf = r.nonfinite;
        inv = r.inverted;
    }
    raise_flags(status, nf, inv);
    if (MON) {
        double s = block_sum<kBlock>(double(psi), shd);
        if (threadIdx.x == 0) part[blk] = s;
    }
}

template <int NP, bool MON, int MODE>
__global__ __launch_bounds__(kBlock) void h8_element_kernel(
    const int4 *__restrict__ conn0, const int4 *__restrict__ conn1, const float4 *__restrict__ g0,
    const float4 *__restrict__ g1, const float4 *__restrict__ g2, const float4 *__restrict__ hg0,
    const float4 *__restrict__ hg1, const float4 *__restrict__ hg2, const float *__restrict__ khg,
    const float4 *__restrict__ nu4, float *__restrict__ theta, float4 *__restrict__ out, int ne, KMat m,
    unsigned *__restrict__ status, double *__restrict__ part, const float4 *__restrict__ aniso) {
    __shared__ double shd[kBlock / 64];
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int e = blk * kBlock + threadIdx.x;
    float psi = 0.f;
    bool nf = false, inv = false;
    if (e < ne) {
        const int4 ca = conn0[e], cb = conn1[e];
        float4 u[8] = {nu4[ca.x], nu4[ca.y], nu4[ca.z], nu4[ca.w], nu4[cb.x], nu4[cb.y], nu4[cb.z], nu4[cb.w]};
        float th[6 * NP + 1];
        load_theta(theta, ne, e, NP, th);
        ElemResultH8 r;
        h8_compute<NP, MODE>(MON, m, u, h8_geo_planes(g0[e], g1[e], g2[e], hg0[e], hg1[e], hg2[e], khg[e]), th, r,
                            aniso, e);
        store_theta(theta, ne, e, NP, th);
#pragma unroll
        for (int k = 0; k < 8; ++k) out[8 * size_t(e) + k] = r.o[k];
        psi = r.psiV;
        nf = r.nonfinite;
        inv = r.inverted;
    }
    raise_flags(status, nf, inv);
    if (MON) {
        double s = block_sum<kBlock>(double(psi), shd);
        if (threadIdx.x == 0) part[blk] = s;
    }
}

template <bool MON>
__global__ __launch_bounds__(kBlock) void node_kernel(
    const int *__restrict__ rowptr, const int *__restrict__ inc, const float4 *__restrict__ out,
    float4 *__restrict__ nu4, float4 *__restrict__ nv4, const float4 *__restrict__ nth,
    const uint8_t *__restrict__ mask, const float *__restrict__ Vl, int nn, NodeParams p,
    const long long *__restrict__ step_base, int j, unsigned *__restrict__ status, double *__restrict__ part) {
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int a = blk * kBlock + threadIdx.x;
    const float src = source_switch(p, step_base, j);
    NodeMon mo{0.0, -INFINITY, INFINITY, 0.0};
    bool nf = false;
    if (a < nn) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        const int k1 = rowptr[a + 1];
        for (int k = rowptr[a]; k < k1; ++k) {
            const float4 o = out[inc[k]];
            acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
        }
        NodeNew r = node_advance(p, nu4[a], nv4[a], nth[a], mask[a], acc, src);
        nu4[a] = r.u;
        nv4[a] = r.v;
        nf = r.nonfinite;
        if (MON) node_monitor(p, r, Vl[a], mo);
    }
    raise_flags(status, nf, false);
    if (MON) write_node_partials<kBlock>(mo, part, blk, shd, shf);
}

// ---------------------------------------------------------------- fused patch kernels

// One workgroup per patch (a launch covers the first gridDim.x patches).
// H8 with precomputed geometry: compiled for four waves per SIMD (at most 128
// VGPRs, a few values spilled), which its LDS footprint allows; 3 waves per SIMD
// at 144 VGPRs otherwise.  Rebuilding the geometry needs the staged coordinates
// in LDS, which leave room for three workgroups per CU only.
template <int NPE, int NP, bool MON, int BS, bool GEOX, bool BATCH, int MODE, bool FUSED = false>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(NPE == 8 && !GEOX ? 4 : 1)))
void patch_kernel(PatchArgs A, int j) {
    extern __shared__ float4 lds[];
    __shared__ double shd[BS / 64];
    __shared__ float shf[BS / 64];
    patch_work<NPE, NP, MON, BS, GEOX, BATCH, MODE, false, FUSED>(A, xcd_block(blockIdx.x, gridDim.x), j, lds, shd,
                                                                  shf);
}

// Batch scenarios still running at `step`: the union positions run in order of
// descending end step, so they are the first m positions with pos_end > step.
__device__ __forceinline__ int running_positions(const PatchArgs &A, long long step) {
    int lo = 0, hi = A.n_pos;   // first position whose end step is <= step
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (A.pos_end[mid] > step) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Persistent form of the batch patch kernel: launched with the workgroups that
// are resident at once, which walk the step's patches (all patches at a monitor
// step, where finished ones write neutral monitor partials; else only those of
// the scenarios still running: their count for the step was left by the
// previous step's shared-node kernel in the slot of the step's parity, so one
// captured graph serves every step).  The workgroups of XCD x (dispatch is
// round-robin over the XCDs) take the x-th eighth of the patches in a strided
// walk, so that neighbouring patches, which share nodes, stay in one L2.  The
// assignment is static: pulling patches one by one from device-wide counters
// measured 3.8 times slower (every pull is an atomic on one of a few
// addresses, served in order at the coherence point of the XCDs).  No
// workgroup waits for another.
template <int NPE, int NP, bool MON, bool GEOX>
__global__ __launch_bounds__(kBlock) void patch_queue_kernel(PatchArgs A, int j) {
    extern __shared__ float4 lds[];
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    const long long step = *A.step_base + j;
    const int n = MON ? A.n_patches : int(A.qcount[2 * (step & 1)]);
    const int G = int(gridDim.x), x = int(blockIdx.x) % kNumXcd, i = int(blockIdx.x) / kNumXcd;
    const int gx = G / kNumXcd + (x < G % kNumXcd ? 1 : 0);          // workgroups on XCD x
    const int lo = int((long long)n * x / kNumXcd), hi = int((long long)n * (x + 1) / kNumXcd);
    for (int pid = lo + i; pid < hi; pid += gx)
        patch_work<NPE, NP, MON, kBlock, GEOX, true, kTi, true>(A, pid, j, lds, shd, shf);
}

template <bool MON, bool BATCH>
__global__ __launch_bounds__(kBlock) void shared_node_kernel(PatchArgs A, int j) {
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int s = blk * kBlock + threadIdx.x;
    NodeMon mo{0.0, -INFINITY, INFINITY, 0.0};
    bool nf = false;
    const int sc = (BATCH && s < A.n_shared) ? A.shared_scen[s] : 0;
    const long long step = *A.step_base + j;
    if (s < A.n_shared && (!BATCH || step < A.scen_end[sc])) {
        const NodeParams p = A.np[sc];
        const float src = (step >= p.n_on && step < p.n_off) ? 1.0f : 0.0f;
        const int a = A.n_interior + s;
        const float4 u0 = A.su_in[s], v0 = A.sv_in[s], th = A.nth[a];   // independent of the partials
        const unsigned mk = A.mask[a];
        const float4 acc = sum_node_partials(A.partial, A.srow[s], A.srow[s + 1]);
        NodeNew r = node_advance(p, u0, v0, th, mk, acc, src);
        A.nu4[a] = r.u;
        A.nv4[a] = r.v;
        nf = r.nonfinite;
        if (MON) node_monitor(p, r, A.Vl[a], mo);
    }
    raise_flags(A.status, nf, false);
    if (MON) write_node_partials<kBlock>(mo, A.part_node + 4 * size_t(A.n_patches), blk, shd, shf);
}

// Shared-node kernel of the persistent schedule: a fixed grid strides over the
// shared nodes of the scenarios still running (all of them at a monitor step),
// counted on the device; block 0 also counts the next step's running patches
// and shared nodes.
template <bool MON>
__global__ __launch_bounds__(kBlock) void shared_node_queue_kernel(PatchArgs A, int j) {
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    const long long step = *A.step_base + j;
    const int64_t n = MON ? int64_t(A.n_shared) : int64_t(A.qcount[2 * (step & 1) + 1]);
    // the running scenarios' patch and shared-node counts of the next step, into
    // the other parity's slots (read by the next step's kernels only)
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const int m = running_positions(A, step + 1);
        long long *nx = A.qcount + 2 * ((step + 1) & 1);
        nx[0] = m ? A.pos_patch_hi[m - 1] : 0;
        nx[1] = m ? A.pos_shared_hi[m - 1] : 0;
    }
    NodeMon mo{0.0, -INFINITY, INFINITY, 0.0};
    bool nf = false;
    for (int64_t s = int64_t(blockIdx.x) * kBlock + threadIdx.x; s < n; s += int64_t(gridDim.x) * kBlock) {
        const int sc = A.shared_scen[s];
        if (step >= A.scen_end[sc]) continue;
        const NodeParams p = A.np[sc];
        const float src = (step >= p.n_on && step < p.n_off) ? 1.0f : 0.0f;
        const int64_t a = A.n_interior + s;
        const float4 u0 = A.nu4[a], v0 = A.nv4[a], th = A.nth[a];
        const unsigned mk = A.mask[a];
        const float4 acc = sum_node_partials(A.partial, A.srow[s], A.srow[s + 1]);
        NodeNew r = node_advance(p, u0, v0, th, mk, acc, src);
        A.nu4[a] = r.u;
        A.nv4[a] = r.v;
        nf |= r.nonfinite;
        if (MON) node_monitor(p, r, A.Vl[a], mo);
    }
    raise_flags(A.status, nf, false);
    if (MON) write_node_partials<kBlock>(mo, A.part_node + 4 * size_t(A.n_patches), int(blockIdx.x), shd, shf);
}

// ---------------------------------------------------------------- monitors

__global__ __launch_bounds__(kBlock) void finish_kernel(const double *__restrict__ part_elem, int n_elem_parts,
                                                        const double *__restrict__ part_node, int n_node_parts,
                                                        long long *step_base, int k, const unsigned *status,
                                                        DevMonitors *mon, unsigned *sync, unsigned *done) {
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    finish_monitors(part_elem, n_elem_parts, part_node, n_node_parts, step_base, k, status, mon, shd, shf);
    if (sync && threadIdx.x == 0) count_chunk(sync, done);
}

// ---------------------------------------------------------------- launchers

namespace {
template <int NP, int MODE>
void launch_t4_element_a(bool mon, const TwoPassArgs &a, const KMat &m, hipStream_t s, const LaunchTiming *ev) {
    dim3 grid((a.ne + kBlock - 1) / kBlock);
    if (mon)
        TLED_LAUNCH(ev, (t4_element_kernel<NP, true, MODE>), grid, dim3(kBlock), 0, s, a.conn4, a.g0, a.g1, a.g2,
                    a.nu4, a.theta, a.out, a.ne, m, a.status, a.part_elem, a.aniso);
    else
        TLED_LAUNCH(ev, (t4_element_kernel<NP, false, MODE>), grid, dim3(kBlock), 0, s, a.conn4, a.g0, a.g1, a.g2,
                    a.nu4, a.theta, a.out, a.ne, m, a.status, a.part_elem, a.aniso);
}
template <int NP, int MODE>
void launch_h8_element_a(bool mon, const TwoPassArgs &a, const KMat &m, hipStream_t s, const LaunchTiming *ev) {
    dim3 grid((a.ne + kBlock - 1) / kBlock);
    if (mon)
        TLED_LAUNCH(ev, (h8_element_kernel<NP, true, MODE>), grid, dim3(kBlock), 0, s, a.conn4, a.conn4b, a.g0, a.g1,
                    a.g2, a.hg0, a.hg1, a.hg2, a.khg, a.nu4, a.theta, a.out, a.ne, m, a.status, a.part_elem, a.aniso);
    else
        TLED_LAUNCH(ev, (h8_element_kernel<NP, false, MODE>), grid, dim3(kBlock), 0, s, a.conn4, a.conn4b, a.g0,
                    a.g1, a.g2, a.hg0, a.hg1, a.hg2, a.khg, a.nu4, a.theta, a.out, a.ne, m, a.status, a.part_elem,
                    a.aniso);
}
// The anisotropy plane is present exactly when the orthotropic expansion or the tensor conduction is on.
template <int NP>
void launch_t4_element(bool mon, const TwoPassArgs &a, const KMat &m, hipStream_t s, const LaunchTiming *ev) {
    if (a.aniso) launch_t4_element_a<NP, kOrtho>(mon, a, m, s, ev);
    else launch_t4_element_a<NP, kTi>(mon, a, m, s, ev);
}
template <int NP>
void launch_h8_element(bool mon, const TwoPassArgs &a, const KMat &m, hipStream_t s, const LaunchTiming *ev) {
    if (a.aniso) launch_h8_element_a<NP, kOrtho>(mon, a, m, s, ev);
    else launch_h8_element_a<NP, kTi>(mon, a, m, s, ev);
}

// occ != nullptr: report the resident workgroups per CU of the instantiation
// instead of launching it.
template <int NPE, int NP, int BS, bool GEOX, bool BATCH, int MODE, bool FUSED = false>
void launch_patch_g(bool mon, const PatchArgs &a, int j, size_t lds, hipStream_t s, int *occ,
                    const LaunchTiming *ev) {
    if (occ) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                occ, reinterpret_cast<const void *>(&patch_kernel<NPE, NP, false, BS, GEOX, BATCH, MODE, FUSED>),
                BS, lds) != hipSuccess)
            *occ = -1;
        return;
    }
    dim3 grid(a.n_patches);
    if (mon)
        TLED_LAUNCH(ev, (patch_kernel<NPE, NP, true, BS, GEOX, BATCH, MODE, FUSED>), grid, dim3(BS), lds, s, a, j);
    else
        TLED_LAUNCH(ev, (patch_kernel<NPE, NP, false, BS, GEOX, BATCH, MODE, FUSED>), grid, dim3(BS), lds, s, a, j);
}

// Batches run with 256-thread workgroups only; so do single problems with the
// orthotropic expansion or the tensor conduction (a.mode kOrtho).  The fused form
// exists for single problems with the geometry rebuilt from coordinates, 256 threads
// and no anisotropy plane (the library enables it only then).  512-thread workgroups
// and the persistent batch kernel serve every other mode with kTi.
template <int NPE, int NP, int BS, bool GEOX, bool BATCH, bool FUSED>
void launch_patch_m(bool mon, const PatchArgs &a, int j, size_t lds, hipStream_t s, int *occ, const LaunchTiming *ev) {
    if (a.mode == kIso) launch_patch_g<NPE, NP, BS, GEOX, BATCH, kIso, FUSED>(mon, a, j, lds, s, occ, ev);
    else launch_patch_g<NPE, NP, BS, GEOX, BATCH, kTi, FUSED>(mon, a, j, lds, s, occ, ev);
}

template <int NPE, int NP>
void launch_patch_np(bool mon, bool geox, int bs, bool batch, const PatchArgs &a, int j, size_t lds,
                     hipStream_t s, int *occ, const LaunchTiming *ev, bool fused) {
    if (fused) {
        launch_patch_m<NPE, NP, 256, true, false, true>(mon, a, j, lds, s, occ, ev);
    } else if (a.mode == kOrtho && !batch) {
        if (geox) launch_patch_g<NPE, NP, 256, true, false, kOrtho, false>(mon, a, j, lds, s, occ, ev);
        else launch_patch_g<NPE, NP, 256, false, false, kOrtho, false>(mon, a, j, lds, s, occ, ev);
    } else if (batch) {
        if (geox) launch_patch_m<NPE, NP, 256, true, true, false>(mon, a, j, lds, s, occ, ev);
        else launch_patch_m<NPE, NP, 256, false, true, false>(mon, a, j, lds, s, occ, ev);
    } else if (NPE == 4 && bs == 512) {
        if constexpr (NPE == 4) {   // 512-thread workgroups exist for T4 only
            if (geox) launch_patch_g<NPE, NP, 512, true, false, kTi, false>(mon, a, j, lds, s, occ, ev);
            else launch_patch_g<NPE, NP, 512, false, false, kTi, false>(mon, a, j, lds, s, occ, ev);
        }
    } else {
        if (geox) launch_patch_m<NPE, NP, 256, true, false, false>(mon, a, j, lds, s, occ, ev);
        else launch_patch_m<NPE, NP, 256, false, false, false>(mon, a, j, lds, s, occ, ev);
    }
}
}  // namespace

void launch_element(int npe, int np, bool mon, const TwoPassArgs &a, const KMat &m, hipStream_t s,
                    const LaunchTiming *ev) {
    if (a.ne == 0) return;
    if (npe == 4) {
        switch (np) {
            case 0: launch_t4_element<0>(mon, a, m, s, ev); break;
            case 1: launch_t4_element<1>(mon, a, m, s, ev); break;
            case 2: launch_t4_element<2>(mon, a, m, s, ev); break;
            case 3: launch_t4_element<3>(mon, a, m, s, ev); break;
            default: launch_t4_element<4>(mon, a, m, s, ev); break;
        }
    } else {
        switch (np) {
            case 0: launch_h8_element<0>(mon, a, m, s, ev); break;
            case 1: launch_h8_element<1>(mon, a, m, s, ev); break;
            case 2: launch_h8_element<2>(mon, a, m, s, ev); break;
            case 3: launch_h8_element<3>(mon, a, m, s, ev); break;
            default: launch_h8_element<4>(mon, a, m, s, ev); break;
        }
    }
}

void launch_dose(const float4 *nu4, int nn, double2 *dose, const DoseParams &q, hipStream_t s) {
    if (nn > 0) hipLaunchKernelGGL(dose_kernel, dim3((nn + kBlock - 1) / kBlock), dim3(kBlock), 0, s, nu4, nn, dose, q);
}

void launch_node(bool mon, const TwoPassArgs &a, const NodeParams &p, int j, hipStream_t s, const LaunchTiming *ev) {
    dim3 grid((a.nn + kBlock - 1) / kBlock);
    if (mon)
        TLED_LAUNCH(ev, (node_kernel<true>), grid, dim3(kBlock), 0, s, a.rowptr, a.inc, a.out, a.nu4, a.nv4, a.nth,
                    a.mask, a.Vl, a.nn, p, a.step_base, j, a.status, a.part_node);
    else
        TLED_LAUNCH(ev, (node_kernel<false>), grid, dim3(kBlock), 0, s, a.rowptr, a.inc, a.out, a.nu4, a.nv4, a.nth,
                    a.mask, a.Vl, a.nn, p, a.step_base, j, a.status, a.part_node);
}

namespace {
void patch_dispatch(int npe, int np, bool mon, bool geox, int bs, bool batch, const PatchArgs &a, int j,
                    hipStream_t s, int *occ, const LaunchTiming *ev, bool fused) {
    const size_t lds = patch_lds_bytes(npe, geox, a);
    if (npe == 4) {
        switch (np) {
            case 0: launch_patch_np<4, 0>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 1: launch_patch_np<4, 1>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 2: launch_patch_np<4, 2>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 3: launch_patch_np<4, 3>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            default: launch_patch_np<4, 4>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
        }
    } else {
        switch (np) {
            case 0: launch_patch_np<8, 0>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 1: launch_patch_np<8, 1>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 2: launch_patch_np<8, 2>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            case 3: launch_patch_np<8, 3>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
            default: launch_patch_np<8, 4>(mon, geox, bs, batch, a, j, lds, s, occ, ev, fused); break;
        }
    }
}
}  // namespace

void launch_patch(int npe, int np, bool mon, bool geox, int bs, bool batch, const PatchArgs &a, int j,
                  hipStream_t s, const LaunchTiming *ev, bool fused) {
    patch_dispatch(npe, np, mon, geox, bs, batch, a, j, s, nullptr, ev, fused);
}

namespace {
// occ != nullptr: report resident workgroups per CU instead of launching.
template <int NPE, int NP, bool GEOX>
void launch_queue_g(bool mon, const PatchArgs &a, int j, int grid, size_t lds, hipStream_t s, int *occ,
                    const LaunchTiming *ev) {
    if (occ) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                occ, reinterpret_cast<const void *>(&patch_queue_kernel<NPE, NP, false, GEOX>), kBlock, lds) !=
            hipSuccess)
            *occ = -1;
        return;
    }
    if (mon) TLED_LAUNCH(ev, (patch_queue_kernel<NPE, NP, true, GEOX>), dim3(grid), dim3(kBlock), lds, s, a, j);
    else TLED_LAUNCH(ev, (patch_queue_kernel<NPE, NP, false, GEOX>), dim3(grid), dim3(kBlock), lds, s, a, j);
}
template <int NPE>
void queue_np(int np, bool mon, bool geox, const PatchArgs &a, int j, int grid, size_t lds, hipStream_t s, int *occ,
              const LaunchTiming *ev) {
#define TLED_QNP(NPV)                                                            \
    if (geox) launch_queue_g<NPE, NPV, true>(mon, a, j, grid, lds, s, occ, ev);  \
    else launch_queue_g<NPE, NPV, false>(mon, a, j, grid, lds, s, occ, ev);
    switch (np) {
        case 0: TLED_QNP(0) break;
        case 1: TLED_QNP(1) break;
        case 2: TLED_QNP(2) break;
        case 3: TLED_QNP(3) break;
        default: TLED_QNP(4) break;
    }
#undef TLED_QNP
}
}  // namespace

void launch_patch_queue(int npe, int np, bool mon, bool geox, const PatchArgs &a, int j, int grid, hipStream_t s,
                        const LaunchTiming *ev) {
    const size_t lds = patch_lds_bytes(npe, geox, a);
    if (npe == 4) queue_np<4>(np, mon, geox, a, j, grid, lds, s, nullptr, ev);
    else queue_np<8>(np, mon, geox, a, j, grid, lds, s, nullptr, ev);
}

int patch_queue_occupancy(int npe, int np, bool geox, const PatchArgs &a) {
    int occ = 0;
    const size_t lds = patch_lds_bytes(npe, geox, a);
    if (npe == 4) queue_np<4>(np, false, geox, a, 0, 1, lds, nullptr, &occ, nullptr);
    else queue_np<8>(np, false, geox, a, 0, 1, lds, nullptr, &occ, nullptr);
    return occ;
}

void launch_shared_nodes_queue(bool mon, const PatchArgs &a, int j, int grid, hipStream_t s, const LaunchTiming *ev) {
    if (mon) TLED_LAUNCH(ev, (shared_node_queue_kernel<true>), dim3(grid), dim3(kBlock), 0, s, a, j);
    else TLED_LAUNCH(ev, (shared_node_queue_kernel<false>), dim3(grid), dim3(kBlock), 0, s, a, j);
}

int patch_occupancy(int npe, int np, bool geox, int bs, bool batch, const PatchArgs &a, bool fused) {
    int occ = 0;
    patch_dispatch(npe, np, false, geox, bs, batch, a, 0, nullptr, &occ, nullptr, fused);
    return occ;
}

void launch_shared_nodes(bool mon, bool batch, const PatchArgs &a, int j, hipStream_t s, const LaunchTiming *ev) {
    const int nb = int((a.n_shared + kBlock - 1) / kBlock);
    if (nb == 0) return;
    dim3 grid(nb);
    if (batch) {
        if (mon) TLED_LAUNCH(ev, (shared_node_kernel<true, true>), grid, dim3(kBlock), 0, s, a, j);
        else TLED_LAUNCH(ev, (shared_node_kernel<false, true>), grid, dim3(kBlock), 0, s, a, j);
    } else {
        if (mon) TLED_LAUNCH(ev, (shared_node_kernel<true, false>), grid, dim3(kBlock), 0, s, a, j);
        else TLED_LAUNCH(ev, (shared_node_kernel<false, false>), grid, dim3(kBlock), 0, s, a, j);
    }
}

// One block per scenario: max T and the lumped volume at or above T_abl (fixed-order reduction).
__global__ __launch_bounds__(kBlock) void scenario_monitor_kernel(const float4 *__restrict__ nu4,
                                                                  const float *__restrict__ Vl,
                                                                  const long long *__restrict__ ranges,
                                                                  const NodeParams *__restrict__ np, float T_abl,
                                                                  double *__restrict__ out) {
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    const int sc = blockIdx.x;
    const float T0 = np[sc].T0;
    float tmax = -INFINITY;
    double vol = 0.0;
    for (int r = 0; r < 2; ++r) {
        const long long lo = ranges[4 * sc + 2 * r], hi = ranges[4 * sc + 2 * r + 1];
        for (long long a = lo + threadIdx.x; a < hi; a += kBlock) {
            const float T = T0 + nu4[a].w;
            tmax = fmaxf(tmax, T);
            if (T >= T_abl) vol += double(Vl[a]);
        }
    }
    vol = block_sum<kBlock>(vol, shd);
    tmax = block_max<kBlock>(tmax, shf);
    if (threadIdx.x == 0) {
        out[2 * sc] = tmax;
        out[2 * sc + 1] = vol;
    }
}

void launch_scenario_monitors(const float4 *nu4, const float *Vl, const long long *ranges, const NodeParams *np,
                              int n_scen, float T_abl, double *out, hipStream_t s) {
    if (n_scen <= 0) return;
    hipLaunchKernelGGL(scenario_monitor_kernel, dim3(n_scen), dim3(kBlock), 0, s, nu4, Vl, ranges, np, T_abl, out);
}

void launch_finish(const double *part_elem, int n_elem_parts, const double *part_node, int n_node_parts,
                   long long *step_base, int k, const unsigned *status, DevMonitors *mon, unsigned *sync,
                   unsigned *done, hipStream_t s) {
    hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(kBlock), 0, s, part_elem, n_elem_parts, part_node, n_node_parts,
                       step_base, k, status, mon, sync, done);
}

size_t patch_lds_bytes(int npe, bool geox, const PatchArgs &a) {
    return sizeof(float4) * ((geox ? 2 : 1) * size_t(a.max_nodes) + size_t(a.max_elems) * npe);
}

}  // namespace tled

// ---------------------------------------------------------------- field export

namespace tled {

__global__ __launch_bounds__(kBlock) void export_fields_kernel(const float4 *__restrict__ nu4,
                                                               const int *__restrict__ new2old, int nn, float T0,
                                                               float *__restrict__ u_dst, float *__restrict__ T_dst) {
    const int a = blockIdx.x * kBlock + threadIdx.x;
    if (a >= nn) return;
    const float4 u = nu4[a];
    const int o = new2old[a];
    if (u_dst) {
        u_dst[3 * size_t(o)] = u.x;
        u_dst[3 * size_t(o) + 1] = u.y;
        u_dst[3 * size_t(o) + 2] = u.z;
    }
    if (T_dst) T_dst[o] = T0 + u.w;
}

void launch_export_fields(const float4 *nu4, const int *new2old, int nn, float T0, float *u_dst, float *T_dst,
                          hipStream_t s) {
    if (nn == 0) return;
    hipLaunchKernelGGL(export_fields_kernel, dim3((nn + kBlock - 1) / kBlock), dim3(kBlock), 0, s, nu4, new2old, nn,
                       T0, u_dst, T_dst);
}

}  // namespace tled
