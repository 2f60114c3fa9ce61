// Whole chunks of time steps in one kernel, for problems whose patches are all
// resident on the GPU at once.
//
// A small or medium problem spends its step on the two launches of the patch and
// shared-node kernels and on staging state that has not left the chip's reach: the
// 6000-tet cube takes 7.9 us per step for 0.1 us of arithmetic and traffic.  Here
// every patch has a workgroup of its own that keeps its nodes in LDS and its Prony
// state in registers for k steps, and exchanges the partial sums of the nodes it
// shares with other patches through memory, every step.
//
// Exchange.  A partial is one 16-byte store and one 16-byte load per reader, both past
// the XCDs' L2 caches (sc1).  There is no flag and no second round trip: each 32-bit
// word says by itself whether it has been written, because its slot holds kEmpty (a NaN
// that no partial keeps) until then, so nothing is assumed of a 16-byte access beyond
// whole 32-bit words.  Slots come in three buffers, step j uses buffer j mod 3, and a
// patch empties its own slots: at the start of step j those of step j + 1, which held
// step j - 2.  All readers are done with them, since each has published step j - 1 after
// reading step j - 2, and this patch has read what they published; and they see the
// empty slot before they look for step j + 1, since it is complete (a wait on the
// stores, behind the element work) before this patch publishes step j, which they
// read first.  The first chunk step finds all slots empty: every workgroup empties its
// own before the meeting below.  (With four 8-byte words (value, step) per partial, the
// 83k-tet ellipsoid took 33 us per step, bound by the requests; 6.6 us like this.)
//
// Waiting.  A workgroup waits for others, so all must be resident.  Before the first
// step they meet: the last to arrive decides GO; one that has waited meet_ticks decides
// ABORT, and whichever came first holds for all (one compare-and-swap).
// After ABORT every workgroup returns with the state untouched, and the finish kernel,
// which ends every chunk, does the chunk's steps with those of its workgroups that have
// come to run within 20 us (at least one, so it is right whatever else occupies the GPU):
// they walk the patches and the shared nodes of a step together and meet twice per step.
// From then on a chunk waits 0.1 ms at most, until one goes; nothing is asked of the host,
// which may have enqueued any number of chunks by then.  (With the steps in a single
// workgroup a chunk of 50 steps of the 83k-tet ellipsoid took 208 ms, 2.5 ms like this,
// and every chunk waited meet_ticks anew.)  After GO each wait is for a workgroup
// that runs, and that itself waits only for partials of earlier steps or of the same
// step written before its own wait; a bound on the polls stays as a guard.
//
// What is left per step (in chunks of 50, against the per-step launches: 6000-tet cube
// 4.4 and 7.9 us, 83k-tet ellipsoid 6.6 and 9.2, 27^3 H8 6.5 and 9.5) is a chain: one
// element's dependent arithmetic, two passes over LDS slots and one trip of a partial from
// store to load past the L2 caches, which is longer with more workgroups.  No unit is busy:
// vector instructions issue in 16 % of the cube's cycles and 28 % of the ellipsoid's.
//
// Bits.  The element, node and summation code is that of the patch kernels, in the
// same order, so a chunk gives the same bits either way.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.h"
#include "step_math.h"

namespace tled {

namespace {

constexpr unsigned kGo = 1, kAbort = 2;
constexpr int kMeetGroups = 16, kMeetStride = 32;   // words of 4 bytes: 128-byte lines
// Words of ResidentArgs::sync, each on a line of its own.  The meeting: the decision, groups
// that are complete, arrivals per group; cleared by the finish kernel.  Its team after
// ABORT: workgroups that joined (and kClosed), team size, arrivals at its barriers; cleared
// by the next chunk's resident kernel.  kImpatient: the last chunk gave up.  kEnded: chunks
// that have ended.
constexpr int kDecision = 0, kGroups = kMeetStride, kArrivals = 2 * kMeetStride,
              kJoined = kArrivals + kMeetGroups * kMeetStride, kTeam = kJoined + kMeetStride,
              kBarrier = kTeam + kMeetStride, kImpatient = kBarrier + kMeetStride,
              kEnded = kImpatient + kMeetStride;
static_assert(kEnded == kResidentEnded && kEnded + kMeetStride == kResidentSyncWords, "one line per word");
constexpr unsigned kClosed = 1u << 31;
constexpr long long kShortTicks = 10000, kTeamTicks = 2000;   // 0.1 ms and 20 us of the 100 MHz clock
constexpr unsigned kMaxPolls = 1u << 21;     // seconds; only a defect reaches it
constexpr unsigned kEmpty = 0xffffffffu, kQuietNan = 0x7fc00000u;
constexpr int kSc1 = 16;                     // cache policy of the buffer accesses: agent scope

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// The exchange buffer as a buffer resource (the accesses are bounds-checked by the
// hardware) and its slots: buffer b, partial position pos.
struct Slots {
    __amdgpu_buffer_rsrc_t rsrc;
    int n;
    __device__ Slots(void *p, int n_entries)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, 48 * n_entries, 0x00027000)), n(n_entries) {}
    __device__ __forceinline__ int at(int b, int pos) const { return 16 * (b * n + pos); }
    __device__ __forceinline__ void put(u32x4 v, int b, int pos) const {
        __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, at(b, pos), 0, kSc1);
    }
    __device__ __forceinline__ u32x4 get(int b, int pos) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, at(b, pos), 0, kSc1);
    }
};

// Waits until this wavefront's stores are complete.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ unsigned get_word(const unsigned *w) {
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_word(unsigned *w, unsigned v) {
    __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arrival at the meeting, thread 0: workgroup b of G counts itself in its group's word
// (kMeetGroups words on lines of their own, since arrivals at one address are served one
// after the other); each group's last counts the group, and the last group decides (with
// no patience at all: to give up).
__device__ __forceinline__ void arrive(unsigned *sync, unsigned b, unsigned G, long long ticks) {
    const unsigned g = b % kMeetGroups, groups = min(G, unsigned(kMeetGroups));
    const unsigned size = G / kMeetGroups + (g < G % kMeetGroups ? 1 : 0);
    if (__hip_atomic_fetch_add(&sync[kArrivals + kMeetStride * g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 < size)
        return;
    if (__hip_atomic_fetch_add(&sync[kGroups], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 < groups) return;
    unsigned undecided = 0;
    if (__hip_atomic_compare_exchange_strong(&sync[kDecision], &undecided, ticks > 0 ? kGo : kAbort, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        put_word(sync + kImpatient, 0);
}

// Whether the launch's workgroups are all resident (the same answer for each), thread 0.
__device__ __forceinline__ bool decided_go(unsigned *sync, long long ticks) {
    const long long t0 = wall_clock64();
    unsigned d;
    while ((d = get_word(sync + kDecision)) == 0) {
        const long long t = wall_clock64() - t0;
        if (t >= ticks || (t >= kShortTicks && get_word(sync + kImpatient))) {
            unsigned undecided = 0;
            __hip_atomic_compare_exchange_strong(&sync[kDecision], &undecided, kAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        } else {
            __builtin_amdgcn_s_sleep(2);
        }
    }
    return d == kGo;
}

__device__ __forceinline__ unsigned full(float v) {
    const unsigned u = __float_as_uint(v);
    return u == kEmpty ? kQuietNan : u;
}

// Sum of the n partials from position k0 in buffer b, mine being the one at position
// own, once all are there: the additions of sum_node_partials.  lost: the guard on the
// polls has been reached.
__device__ __forceinline__ float4 collect(const Slots &x, int b, int k0, int n, int own, float4 mine, bool &lost) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    const u32x4 me = {__float_as_uint(mine.x), __float_as_uint(mine.y), __float_as_uint(mine.z), __float_as_uint(mine.w)};
    for (int k = 0; k < n; k += 4) {
        u32x4 w[4];
        unsigned polls = 0;
        bool ok;
        do {
            asm volatile("" ::: "memory");     // load again in every round
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                w[q] = k0 + k + q == own ? me : u32x4{0u, 0u, 0u, 0u};
                if (k + q < n && k0 + k + q != own) w[q] = x.get(b, k0 + k + q);
            }
            ok = true;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k0 + k + q != own)
                    ok = ok && w[q].x != kEmpty && w[q].y != kEmpty && w[q].z != kEmpty && w[q].w != kEmpty;
        } while (!ok && !lost && ++polls < kMaxPolls);
        lost = lost || !ok;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc.x += __uint_as_float(w[q].x);
            acc.y += __uint_as_float(w[q].y);
            acc.z += __uint_as_float(w[q].z);
            acc.w += __uint_as_float(w[q].w);
        }
    }
    return acc;
}

// Sum of a local node's element slots [k, k1) in LDS, in order as in the patch kernels,
// eight loads in flight: the wave waits for its longest run (24 slots for an interior
// node of a Kuhn mesh), so the latency of a load per slot or four is what counts.
// Past the end a slot of zeros is added, which changes no sum (none is -0).
__device__ __forceinline__ float4 gather(const float4 *lout, int k, int k1, int zero) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (; k < k1; k += 8) {
        float4 o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = lout[k + q < k1 ? k + q : zero];
#pragma unroll
        for (int q = 0; q < 8; ++q) { acc.x += o[q].x; acc.y += o[q].y; acc.z += o[q].z; acc.w += o[q].w; }
    }
    return acc;
}

// Geometry of an element kept in registers when a thread has one element; with two T4
// elements rebuilt every step from the patch's coordinates in LDS (13 registers per
// element against 41 instructions).
constexpr bool lds_coords(int npe, int ept) { return npe == 4 && ept > 1; }

// One workgroup per patch, EPT elements per thread, k steps (fewer where the patch's
// scenario ends).  LDS per local node: (u, dT), (v, B), thermal constants, and
// {slots [x & 0xffff, x >> 16), partial position or -1, first partial, partial count |
// mask << 16}; then the element slots.  T4: 128 VGPRs at most, for four workgroups per
// CU.  H8: 58.6 KB of LDS for 256 elements let two workgroups share a CU anyway, so the
// registers of two (at 128 it spilled some 140 values).
template <int NPE, int NP, int EPT, int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(NPE == 8 ? 2 : 4))) void resident_kernel(
    PatchArgs A, ResidentArgs R, int k) {
    extern __shared__ float4 lds[];
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    __shared__ bool go;
    const Slots x(R.xbuf, R.n_entries);
    {   // empty this patch's slots; complete before the meeting
        const int p0 = xcd_block(blockIdx.x, gridDim.x);
        for (int q = A.shared_begin[p0] + int(threadIdx.x); q < A.shared_begin[p0 + 1]; q += kBlock)
            for (int b = 0; b < 3; ++b) x.put(u32x4{kEmpty, kEmpty, kEmpty, kEmpty}, b, A.ppos[q]);
        if (blockIdx.x == 0 && threadIdx.x == 0) {   // the finish kernel of the chunk before is through
            put_word(R.sync + kJoined, 0);
            put_word(R.sync + kTeam, 0);
            put_word(R.sync + kBarrier, 0);
        }
        stores_done();
        __syncthreads();
        if (threadIdx.x == 0) arrive(R.sync, blockIdx.x, gridDim.x, R.meet_ticks);
    }
    constexpr bool COORDS = lds_coords(NPE, EPT);
    const int pid = xcd_block(blockIdx.x, gridDim.x), t = threadIdx.x;
    const int sc = A.patch_scen[pid];
    const KMat m = A.km[sc];
    const NodeParams p = A.np[sc];
    const long long base = *A.step_base, end = A.scen_end[sc];
    const int kk = int(min((long long)k, max(end - base, 0LL)));
    const int e0 = A.elem_begin[pid], e1 = A.elem_begin[pid + 1];
    const int ib = A.int_begin[pid], nint = A.int_begin[pid + 1] - ib;
    const int sb = A.shared_begin[pid], nloc = nint + A.shared_begin[pid + 1] - sb;
    float4 *ln = lds, *lv = ln + A.max_nodes, *lt = lv + A.max_nodes;
    int4 *li = reinterpret_cast<int4 *>(lt + A.max_nodes);
    float4 *lxyz = lt + 2 * A.max_nodes;
    float4 *lout = lxyz + (COORDS ? A.max_nodes : 0);
    const int zero = NPE * A.max_elems;        // a slot of zeros after the element slots
    if (t == 0) lout[zero] = make_float4(0.f, 0.f, 0.f, 0.f);
    // Nodes to threads: the shared ones from thread 0, the interior ones from the next
    // wavefront on, so that the two kinds of work run side by side
    const int nsh = nloc - nint, nshp = (nsh + 63) & ~63;
    const float *gx = NPE == 4 ? A.lX + 3 * size_t(A.lx_begin[pid]) : nullptr;
    const uint16_t *lrow = A.lrow + A.lrow_begin[pid];
    for (int l = t; l < nloc; l += kBlock) {
        const bool interior = l < nint;
        const int q = sb + l - nint;
        const int a = interior ? ib + l : A.shared_ids[q];
        const int2 kr = interior ? make_int2(0, 0) : R.srange[q];
        ln[l] = A.nu4[a];
        lv[l] = A.nv4[a];
        lt[l] = A.nth[a];
        li[l] = make_int4(int(lrow[l]) | (int(lrow[l + 1]) << 16), interior ? -1 : A.ppos[q], kr.x,
                          (kr.y - kr.x) | (int(A.mask[a]) << 16));
        if (COORDS) lxyz[l] = make_float4(gx[3 * l], gx[3 * l + 1], gx[3 * l + 2], 0.f);
    }
    // elements: Prony state, and with one element per thread its T4 geometry and the node
    // and slot numbers
    float th[EPT][6 * NP + 1];
    GeoT4 geo;
    GeoH8 geo8;
    ushort4 ca{}, cb{}, pa{}, pb{};
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = e0 + t + it * kBlock;
        if (e < e1) {
            load_theta(A.theta, A.ne, e, NP, th[it]);
            if (EPT == 1) {
                const ushort4 *cn = reinterpret_cast<const ushort4 *>(A.lconn), *ps = reinterpret_cast<const ushort4 *>(A.lpos);
                ca = cn[NPE / 4 * e];
                pa = ps[NPE / 4 * e];
                if (NPE == 8) {
                    cb = cn[2 * e + 1];
                    pb = ps[2 * e + 1];
                    geo8 = h8_geo_planes(A.g0[e], A.g1[e], A.g2[e], A.hg0[e], A.hg1[e], A.hg2[e], A.khg[e]);
                } else {
                    const int c[4] = {ca.x, ca.y, ca.z, ca.w};
                    float4 x[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = make_float4(gx[3 * c[i]], gx[3 * c[i] + 1], gx[3 * c[i] + 2], 0.f);
                    geo = t4_geo_coords(x, A.fib[e]);
                }
            }
        }
    }
    // the others' decision, behind the loads above
    if (t == 0) go = decided_go(R.sync, R.meet_ticks);
    __syncthreads();
    if (!go) return;
    // The loads above are complete from here on, for the compiler too: with one left that it
    // may still have to wait for, it waits inside the loop, every step, and there for the
    // step's stores as well (6000-tet cube 4.4 us per step, 4.0 like this).
    __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0)
    float psi = 0.f;
    bool nf = false, inv = false, lost = false;
    int b = 0;                                 // j mod 3
    for (int j = 0; j < kk; ++j) {
        const bool mon = j == k - 1;
        const int next = b == 2 ? 0 : b + 1;
        if (j >= 2)                            // the first two steps after the meeting find theirs empty
            for (int l = nint + t; l < nloc; l += kBlock) x.put(u32x4{kEmpty, kEmpty, kEmpty, kEmpty}, next, li[l].y);
#pragma unroll
        for (int it = 0; it < EPT; ++it) {
            const int e = e0 + t + it * kBlock;
            if (e < e1) {
                if (NPE == 4) {
                    const ushort4 c = EPT == 1 ? ca : reinterpret_cast<const ushort4 *>(A.lconn)[e];
                    const ushort4 ps = EPT == 1 ? pa : reinterpret_cast<const ushort4 *>(A.lpos)[e];
                    const float4 u[4] = {ln[c.x], ln[c.y], ln[c.z], ln[c.w]};
                    GeoT4 g;
                    if (COORDS) {
                        const float4 x[4] = {lxyz[c.x], lxyz[c.y], lxyz[c.z], lxyz[c.w]};
                        g = t4_geo_coords(x, A.fib[e]);
                    } else {
                        g = geo;
                    }
                    ElemResultT4 r;
                    t4_compute<NP, MODE>(mon, m, u, g, th[it], r, nullptr, e);
                    lout[ps.x] = r.o[0];
                    lout[ps.y] = r.o[1];
                    lout[ps.z] = r.o[2];
                    lout[ps.w] = r.o[3];
                    psi += r.psiV;
                    nf |= r.nonfinite;
                    inv |= r.inverted;
                } else {
                    const float4 u[8] = {ln[ca.x], ln[ca.y], ln[ca.z], ln[ca.w], ln[cb.x], ln[cb.y], ln[cb.z], ln[cb.w]};
                    ElemResultH8 r;
                    h8_compute<NP, MODE>(mon, m, u, geo8, th[it], r, nullptr, e);
                    lout[pa.x] = r.o[0];
                    lout[pa.y] = r.o[1];
                    lout[pa.z] = r.o[2];
                    lout[pa.w] = r.o[3];
                    lout[pb.x] = r.o[4];
                    lout[pb.y] = r.o[5];
                    lout[pb.z] = r.o[6];
                    lout[pb.w] = r.o[7];
                    psi += r.psiV;
                    nf |= r.nonfinite;
                    inv |= r.inverted;
                }
            }
        }
        __syncthreads();
        // shared nodes publish
        const float src = (base + j >= p.n_on && base + j < p.n_off) ? 1.0f : 0.0f;
        stores_done();
        for (int l = nint + t; l < nloc; l += kBlock) {
            const int4 q = li[l];
            const int k0 = q.x & 0xffff;
            const float4 v = gather(lout, k0, int(unsigned(q.x) >> 16), zero);
            x.put(u32x4{full(v.x), full(v.y), full(v.z), full(v.w)}, b, q.y);
            lout[k0] = v;                      // this thread's own slots: read again when the partials are summed
        }
        // interior nodes advance while the partials travel
        for (int i = t; i < nshp + nint; i += kBlock) {
            const int l = i - nshp;
            if (l < 0) continue;
            const int4 q = li[l];
            const float4 acc = gather(lout, q.x & 0xffff, int(unsigned(q.x) >> 16), zero);
            const NodeNew r = node_advance(p, ln[l], lv[l], lt[l], unsigned(q.w) >> 16, acc, src);
            ln[l] = r.u;
            lv[l] = r.v;
            nf |= r.nonfinite;
            if (R.hist) R.hist[size_t(j) * R.nn + ib + l] = r.u.w;
        }
        // Not too early: a poll that comes before its partials costs a whole round trip, and
        // polls delay the stores they wait for.  With many workgroups the first poll waits
        // until this one's own partials are through and a little longer, with few it goes out
        // at once.  us per step, at once / waiting: T4 with 47 workgroups 4.14 / 4.41, 81 4.15 /
        // 4.36, 102 4.71 / 4.70, 126 4.73 / 4.70, 159 4.50 / 4.28, 203 5.08 / 4.74, 431 6.96 /
        // 5.50, 650 8.51 / 6.47, 1018 10.1 / 7.3; two elements per thread with 68 6.32 / 6.68,
        // 135 6.71 / 7.01, 201 7.12 / 6.73, 448 11.2 / 10.2.  H8, where a step is longer, loses
        // little by either: 77 6.34 / 6.92, 154 6.46 / 6.79, 250 7.10 / 7.13, 489 9.34 / 9.32.
        if (gridDim.x > 128) {
            __builtin_amdgcn_s_sleep(16);
            stores_done();
            __builtin_amdgcn_s_sleep(4);
        }
        for (int l = nint + t; l < nloc; l += kBlock) {
            const int4 q = li[l];
            const float4 acc = collect(x, b, q.z, q.w & 0xffff, q.y, lout[q.x & 0xffff], lost);
            const NodeNew r = node_advance(p, ln[l], lv[l], lt[l], unsigned(q.w) >> 16, acc, src);
            ln[l] = r.u;
            lv[l] = r.v;
            nf |= r.nonfinite;
            if (R.hist && q.y == q.z) R.hist[size_t(j) * R.nn + A.shared_ids[sb + l - nint]] = r.u.w;
        }
        __syncthreads();
        b = next;
    }
    // state back to memory: interior nodes, and the shared nodes whose first partial is this patch's
    NodeMon mo{0.0, -INFINITY, INFINITY, 0.0};
    const bool ran_last = kk == k;
    for (int l = t; l < nloc; l += kBlock) {
        const int4 q = li[l];
        if (l >= nint && q.y != q.z) continue;
        const int a = l < nint ? ib + l : A.shared_ids[sb + l - nint];
        const NodeNew r{ln[l], lv[l], false};
        A.nu4[a] = r.u;
        A.nv4[a] = r.v;
        if (ran_last) node_monitor(p, r, A.Vl[a], mo);
    }
#pragma unroll
    for (int it = 0; it < EPT; ++it) {
        const int e = e0 + t + it * kBlock;
        if (e < e1) store_theta(A.theta, A.ne, e, NP, th[it]);
    }
    raise_flags(A.status, nf || lost, inv);
    const double s = block_sum<kBlock>(double(psi), shd);
    if (t == 0) A.part_elem[pid] = s;
    write_node_partials<kBlock>(mo, A.part_node, pid, shd, shf);
    if (blockIdx.x == 0 && t == 0) {   // the finish kernel's entry for shared nodes: counted with their patches here
        double *pp = A.part_node + 4 * size_t(gridDim.x);
        pp[0] = 0.0; pp[1] = -INFINITY; pp[2] = INFINITY; pp[3] = 0.0;
    }
}

// Barrier of the finish kernel's team of W running workgroups; n counts it.  The fences,
// one wavefront's for its whole workgroup, make each workgroup's stores visible to the
// others' loads after it.  lost: the guard on the polls has been reached.
__device__ __forceinline__ void team_barrier(unsigned *arrivals, unsigned W, unsigned &n, bool &lost) {
    stores_done();
    __syncthreads();
    ++n;
    if (threadIdx.x == 0) {
        __threadfence();
        __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned polls = 0;
        while (get_word(arrivals) < n * W && !lost) {
            __builtin_amdgcn_s_sleep(2);
            lost = ++polls >= kMaxPolls;
        }
        __threadfence();
    }
    __syncthreads();
}

// Joins the team that does the steps of a chunk that gave up, thread 0: this workgroup's
// number in it and its size, which the first to come fixes when all have come or after
// kTeamTicks.  False: too late.
__device__ __forceinline__ bool join_team(unsigned *sync, unsigned all, unsigned &number, unsigned &size) {
    number = __hip_atomic_fetch_add(&sync[kJoined], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (number & kClosed) return false;
    if (number == 0) {
        const long long t0 = wall_clock64();
        while (get_word(sync + kJoined) < all && wall_clock64() - t0 < kTeamTicks) __builtin_amdgcn_s_sleep(2);
        size = __hip_atomic_fetch_or(&sync[kJoined], kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        put_word(sync + kTeam, size);
    } else {
        while ((size = get_word(sync + kTeam)) == 0) __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// Ends a chunk of k steps over the first G patches: after ABORT does the steps, with the
// workgroups that run, then the monitor record, the step counter and the next launch's
// meeting words.  After GO there is work for the first workgroup only.
template <int NPE, int NP>
__global__ __launch_bounds__(kBlock) void resident_finish_kernel(PatchArgs A, ResidentArgs R, int k, int G,
                                                                 long long *step_base, DevMonitors *mon) {
    extern __shared__ float4 lds[];
    __shared__ double shd[kBlock / 64];
    __shared__ float shf[kBlock / 64];
    __shared__ unsigned number, size;
    __shared__ bool joined;
    // neither kGo nor kAbort: everything has been done and the word cleared
    const unsigned decision = uniform_int(reinterpret_cast<const int *>(R.sync + kDecision));
    if (decision != kAbort && (decision != kGo || blockIdx.x != 0)) return;
    const bool aborted = decision == kAbort;
    unsigned W = 1;
    if (aborted) {
        if (threadIdx.x == 0) joined = join_team(R.sync, gridDim.x, number, size);
        __syncthreads();
        if (!joined) return;
        const unsigned me = __builtin_amdgcn_readfirstlane(number);
        W = __builtin_amdgcn_readfirstlane(size);
        unsigned barriers = 0;
        bool lost = false;
        const long long base = *A.step_base;
        for (int j = 0; j < k; ++j) {
            const bool last = j == k - 1;
            for (int pid = int(me); pid < G; pid += int(W)) {
                if (last) patch_work<NPE, NP, true, kBlock, NPE == 4, true, kTi, true>(A, pid, j, lds, shd, shf);
                else patch_work<NPE, NP, false, kBlock, NPE == 4, true, kTi, true>(A, pid, j, lds, shd, shf);
                __syncthreads();
                if (R.hist)
                    for (int a = A.int_begin[pid] + int(threadIdx.x); a < A.int_begin[pid + 1]; a += kBlock)
                        R.hist[size_t(j) * R.nn + a] = A.nu4[a].w;
            }
            team_barrier(R.sync + kBarrier, W, barriers, lost);
            NodeMon mo{0.0, -INFINITY, INFINITY, 0.0};
            bool nf = false;
            const long long step = base + j;
            for (int s = int(me) * kBlock + int(threadIdx.x); s < A.n_shared; s += int(W) * kBlock) {
                const int sc = A.shared_scen[s];
                if (step >= A.scen_end[sc]) continue;
                const NodeParams p = A.np[sc];
                const float src = (step >= p.n_on && step < p.n_off) ? 1.0f : 0.0f;
                const int a = A.n_interior + s;
                const float4 acc = sum_node_partials(A.partial, A.srow[s], A.srow[s + 1]);
                const NodeNew r = node_advance(p, A.nu4[a], A.nv4[a], A.nth[a], A.mask[a], acc, src);
                A.nu4[a] = r.u;
                A.nv4[a] = r.v;
                nf |= r.nonfinite;
                if (R.hist) R.hist[size_t(j) * R.nn + a] = r.u.w;
                node_monitor(p, r, A.Vl[a], mo);
            }
            raise_flags(A.status, nf || lost, false);
            if (last) write_node_partials<kBlock>(mo, A.part_node, G + int(me), shd, shf);
            team_barrier(R.sync + kBarrier, W, barriers, lost);
        }
        if (me != 0) return;
    }
    finish_monitors(A.part_elem, G, A.part_node, G + int(W), step_base, k, A.status, mon, shd, shf);
    __syncthreads();
    if (threadIdx.x < kJoined / kMeetStride) put_word(R.sync + kMeetStride * threadIdx.x, 0);
    if (threadIdx.x == 0) {
        if (aborted) {
            A.status[1] += 1;
            put_word(R.sync + kImpatient, 1);
        }
        count_chunk(R.sync, R.done);
    }
}

// Thermal dose of a chunk from its temperature history, step by step as dose_kernel.
// Apart from the steps: the FP64 powers of the dose would cost the resident kernel
// some 40 registers, and here every node has a thread.
__global__ __launch_bounds__(kBlock) void dose_history_kernel(const float *__restrict__ hist, int nn, int k,
                                                              double2 *__restrict__ dose, DoseParams q) {
    const int a = int(blockIdx.x) * kBlock + int(threadIdx.x);
    if (a < nn)
        for (int j = 0; j < k; ++j) add_thermal_dose(dose, q, size_t(a), hist[size_t(j) * nn + a]);
}

// occ != nullptr: resident workgroups per CU instead of a launch.
template <int NPE, int NP, int EPT, int MODE>
void launch_one(const PatchArgs &a, const ResidentArgs &r, int k, size_t lds, hipStream_t s, int *occ) {
    if (occ) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                occ, reinterpret_cast<const void *>(&resident_kernel<NPE, NP, EPT, MODE>), kBlock, lds) != hipSuccess)
            *occ = -1;
        return;
    }
    hipLaunchKernelGGL((resident_kernel<NPE, NP, EPT, MODE>), dim3(a.n_patches), dim3(kBlock), lds, s, a, r, k);
}

template <int NPE, int NP, int EPT>
void launch_mode(const PatchArgs &a, const ResidentArgs &r, int k, size_t lds, hipStream_t s, int *occ) {
    if (a.mode == kIso) launch_one<NPE, NP, EPT, kIso>(a, r, k, lds, s, occ);
    else launch_one<NPE, NP, EPT, kTi>(a, r, k, lds, s, occ);
}

template <int NPE, int NP>
void launch_np(const PatchArgs &a, const ResidentArgs &r, int k, size_t lds, hipStream_t s, int *occ) {
    if constexpr (NPE == 4 && NP <= kResidentMaxProny2) {
        if (a.max_elems > kBlock) return launch_mode<NPE, NP, 2>(a, r, k, lds, s, occ);
    }
    launch_mode<NPE, NP, 1>(a, r, k, lds, s, occ);
}

template <int NPE>
void launch_npe(int np, const PatchArgs &a, const ResidentArgs &r, int k, size_t lds, hipStream_t s, int *occ) {
    switch (np) {
        case 0: launch_np<NPE, 0>(a, r, k, lds, s, occ); break;
        case 1: launch_np<NPE, 1>(a, r, k, lds, s, occ); break;
        case 2: launch_np<NPE, 2>(a, r, k, lds, s, occ); break;
        case 3: launch_np<NPE, 3>(a, r, k, lds, s, occ); break;
        default: launch_np<NPE, 4>(a, r, k, lds, s, occ); break;
    }
}

template <int NPE>
void finish_npe(int np, const PatchArgs &a, const ResidentArgs &r, int k, long long *step_base, DevMonitors *mon,
                hipStream_t s) {
    const size_t lds = patch_lds_bytes(NPE, NPE == 4, a);
#define TLED_RF(NPV)                                                                                              \
    hipLaunchKernelGGL((resident_finish_kernel<NPE, NPV>), dim3(std::min(a.n_patches, r.team)), dim3(kBlock), lds, s, a, r, \
                       k, a.n_patches, step_base, mon)
    switch (np) {
        case 0: TLED_RF(0); break;
        case 1: TLED_RF(1); break;
        case 2: TLED_RF(2); break;
        case 3: TLED_RF(3); break;
        default: TLED_RF(4); break;
    }
#undef TLED_RF
}

}  // namespace

size_t resident_lds_bytes(int npe, const PatchArgs &a) {
    const int ept = npe == 4 && a.max_elems > kBlock ? 2 : 1;
    return sizeof(float4) * ((lds_coords(npe, ept) ? 5 : 4) * size_t(a.max_nodes) + size_t(a.max_elems) * npe + 1);
}

int resident_occupancy(int npe, int np, const PatchArgs &a) {
    int occ = 0;
    const size_t lds = resident_lds_bytes(npe, a);
    if (npe == 4) launch_npe<4>(np, a, ResidentArgs{}, 0, lds, nullptr, &occ);
    else launch_npe<8>(np, a, ResidentArgs{}, 0, lds, nullptr, &occ);
    return occ;
}

void launch_resident(int npe, int np, const PatchArgs &a, const ResidentArgs &r, int k, long long *step_base,
                     DevMonitors *mon, double2 *dose, const DoseParams &dq, hipStream_t s) {
    const size_t lds = resident_lds_bytes(npe, a);
    if (npe == 4) {
        launch_npe<4>(np, a, r, k, lds, s, nullptr);
        finish_npe<4>(np, a, r, k, step_base, mon, s);
    } else {
        launch_npe<8>(np, a, r, k, lds, s, nullptr);
        finish_npe<8>(np, a, r, k, step_base, mon, s);
    }
    if (r.hist)
        hipLaunchKernelGGL(dose_history_kernel, dim3((r.nn + kBlock - 1) / kBlock), dim3(kBlock), 0, s, r.hist, r.nn, k,
                           dose, dq);
}

}  // namespace tled
