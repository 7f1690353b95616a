// mesh.hip -- voxels -> robot: largest component, nodes, springs, initial state.
//
// One workgroup builds one robot in LDS (Sec. II-A: masses on voxel corners;
// springs on the 12 edges, 12 face diagonals and 4 body diagonals of every kept
// voxel).  All integer decisions use integer arithmetic or integer LDS
// atomics, so the result is independent of thread timing.
#include "internal.h"

// No contraction of a*b + c into FMAs in this file: the spring parameters are
// sums of separately rounded per-voxel products, which the step kernels that
// rebuild them from voxels repeat operation by operation.
#pragma clang fp contract(off)

namespace sr {

namespace {

struct BuildArgs {
    const RobotInfo *robots;
    RobotInfo *robots_out;
    const uint8_t *cls;
    const float *w;
    uint8_t *kept;
    Planes pl;
    SpringIndex ix;
    float4 *x0, *x, *v;
    int32_t *slot_node;
    uint8_t *bad_class, *diverged;
    float k_class[5], ac_cos[5], ac_sin[5];
    float a_class[5], phi_class[5];  // for weight-scaled actuation
    int weight_act;
    float dash2m;  // 2 m zeta_spring^2: a voxel spring's dashpot is sqrt(dash2m k_c w)
    float voxel_len;
};

// A kept voxel's contributions to each of its springs (parallel-sum rule):
// x = k_c w, y = k_c w amp cos(ph), z = k_c w amp sin(ph), w = its dashpot.
// Separately rounded operations (contraction is off in this file), so that a
// spring's sums can be rebuilt bit for bit from these per-voxel values.
__device__ float4 voxel_terms(const BuildArgs &A, int kc, float wv) {
    const float kw = A.k_class[kc] * wv;
    float cz, sz;
    if (A.weight_act) {
        // amplitude w a_c and phase w phi_c (Table II maxima times the weight)
        const float amp = wv * A.a_class[kc], ph = wv * A.phi_class[kc];
        cz = amp * cosf(ph);
        sz = amp * sinf(ph);
    } else {
        cz = A.ac_cos[kc];
        sz = A.ac_sin[kc];
    }
    return make_float4(kw, kw * cz, kw * sz, sqrtf(A.dash2m * kw));
}

// q / x for q < 2^16 / x (mul = 65536 / x + 1): the arrays here have at most
// 2744 entries and x <= 14
__device__ __forceinline__ int div_small(int q, int mul) { return (q * mul) >> 16; }

template <bool FULL>
struct TermT {
    typedef float2 T;
};
template <>
struct TermT<true> {
    typedef float4 T;
};
__device__ __forceinline__ void term_store(float2 &d, float4 v) { d = make_float2(v.x, v.y); }
__device__ __forceinline__ void term_store(float4 &d, float4 v) { d = v; }
__device__ __forceinline__ float4 term_load(float2 v) { return make_float4(v.x, v.y, 0.f, 0.f); }
__device__ __forceinline__ float4 term_load(float4 v) { return v; }

// Voxels sit in LDS on the grid padded by one empty layer, (n + 2)^3 cells, so
// neighbour reads need no bounds checks; a padded id orders voxels as the plain
// one does.  The lattice's slots are cut into runs of 64 in slot order, one
// wave each, and the canonical node and spring ids are ordered prefix sums over
// the runs.
// FULL: the population has actuation phases or dashpots, whose planes (kbe,
// kd) are then written too; without, they keep the zeros of pop_create (with
// every class phase zero the sums of k_c w a sin(phi) are exact zeros).
// What bounds it: for thousands of robots the HBM writes, 180 B a slot (spring
// ids, k L0 and neighbour lists, 390 B more, are rebuilt by the few kernels
// that need them); for a few robots the chain of barriers (component labels
// take 5 to 15 rounds).  Each voxel's terms are formed once, not once for each
// of its 28 springs.  Measured against one 1024-thread workgroup per robot that
// wrote all of those: 4096 robots of 10^3 1350 -> 186 us (5.3 TB/s), 1024
// uneven robots 348 -> 40 us, 30 of 5^3 41 -> 10 us.
// BT 256 for grids up to 6^3 (216 voxels): larger workgroups only add waves to
// every barrier there.
template <int BT, int MAXN, bool FULL>
__global__ __launch_bounds__(BT) void k_build_mesh(BuildArgs A) {
    constexpr int MAXP = (MAXN + 2) * (MAXN + 2) * (MAXN + 2);
    constexpr int RUNS = ((MAXN + 1) * (MAXN + 1) * (MAXN + 1) + 63) / 64;
    constexpr int W = BT / 64, RPW = (RUNS + W - 1) / W;
    static_assert(RUNS <= 64, "one wave scans the runs");
    typedef typename TermT<FULL>::T VT;
    __shared__ int lab[MAXP];
    __shared__ VT vt[MAXP];
    __shared__ uint8_t cl[MAXP];
    __shared__ unsigned long long pmask[RUNS];  // present slots of each run
    __shared__ int rspr[RUNS], nbase[RUNS], sbase[RUNS];
    __shared__ int flag[3];
    __shared__ unsigned bestkey;
    __shared__ int zlow;
    int *const cnt = reinterpret_cast<int *>(vt);  // component sizes, before the terms

    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RobotInfo ri = A.robots[r];
    const int n = ri.n, N = n + 1, P = n + 2, np = P * P * P, SL = ri.slots, runs = (SL + 63) / 64;
    const int mulP = 65536 / P + 1, mulN = 65536 / N + 1;
    const int absent = 0x7fffffff;

    // 1. classes; out-of-range classes are reported and treated as empty
    for (int q = tid; q < np; q += BT) {
        const int t = div_small(q, mulP), k = div_small(t, mulP), j = t - P * k, i = q - P * t;
        int c = 0;
        if (i >= 1 && i <= n && j >= 1 && j <= n && k >= 1 && k <= n) {
            c = A.cls[ri.vox_base + (i - 1) + n * ((j - 1) + n * (k - 1))];
            if (c > 4) { A.bad_class[r] = 1; c = 0; }
        }
        cl[q] = (uint8_t)c;
        lab[q] = c ? q : absent;
        cnt[q] = 0;
    }
    if (tid < 3) flag[tid] = 0;
    if (tid == 0) bestkey = 0u;
    __syncthreads();

    // 2. face-connected components by min-label propagation; a label is always a
    // voxel of the component, and a smaller one also goes to the voxel the old
    // label names.  The fixed point is the smallest voxel id of each component.
    for (int it = 0;; ++it) {
        if (tid == 0) flag[(it + 1) % 3] = 0;
        for (int q = tid; q < np; q += BT) {
            if (!cl[q]) continue;
            const int own = lab[q];
            int m = min(min(own, min(lab[q - 1], lab[q + 1])),
                        min(min(lab[q - P], lab[q + P]), min(lab[q - P * P], lab[q + P * P])));
            m = min(m, lab[m]);
            if (m < own) {
                atomicMin(&lab[q], m);
                atomicMin(&lab[own], m);
                flag[it % 3] = 1;
            }
        }
        __syncthreads();
        if (flag[it % 3] == 0) break;
    }

    // 3. component sizes (a wave adds the voxels that share its first label at
    // once); the largest wins, ties to the smallest root id
    for (int q0 = 0; q0 < np; q0 += BT) {
        const int q = q0 + tid;
        const bool on = q < np && cl[q] != 0;
        const int L = on ? lab[q] : absent;
        const unsigned long long act = __ballot(on);
        if (act) {
            const int lead = __ffsll(act) - 1;
            const int first = __shfl(L, lead, 64);
            const unsigned long long same = __ballot(on && L == first);
            if (lane == lead) atomicAdd(&cnt[first], __popcll(same));
            if (on && L != first) atomicAdd(&cnt[L], 1);
        }
    }
    __syncthreads();
    for (int q = tid; q < np; q += BT)
        if (cl[q] && lab[q] == q) atomicMax(&bestkey, ((unsigned)cnt[q] << 16) | (unsigned)(0xffff - q));
    __syncthreads();
    const int best = bestkey ? 0xffff - (int)(bestkey & 0xffff) : -1;
    for (int q = tid; q < np; q += BT) {
        const int t = div_small(q, mulP), k = div_small(t, mulP), j = t - P * k, i = q - P * t;
        const int c = (cl[q] && lab[q] == best) ? cl[q] : 0;
        float4 terms = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i >= 1 && i <= n && j >= 1 && j <= n && k >= 1 && k <= n) {
            const int vox = ri.vox_base + (i - 1) + n * ((j - 1) + n * (k - 1));
            A.kept[vox] = (uint8_t)c;
            if (c) terms = voxel_terms(A, c, A.w[vox]);
        }
        cl[q] = (uint8_t)c;
        term_store(vt[q], terms);
    }
    __syncthreads();

    // 4. nodes are the lattice points touching a kept voxel, springs join two of
    // them along the 13 forward directions through at least one kept voxel, and
    // the kept voxels holding both ends add up in parallel (fixed order)
    const float L0e = A.voxel_len, L0f = A.voxel_len * sqrtf(2.0f), L0b = A.voxel_len * sqrtf(3.0f);
    const int pbase = NDIR * ri.slot_base;
    unsigned masks[RPW];
    int before[RPW];  // springs of the run's earlier slots
#pragma unroll
    for (int e = 0; e < RPW; ++e) {
        const int u = wave + e * W, s = 64 * u + lane;
        masks[e] = 0;
        before[e] = 0;
        if (u >= runs) continue;
        unsigned occ = 0, mask = 0;
        if (s < SL) {
            const int t = div_small(s, mulN), c = div_small(t, mulN), b = t - N * c, a = s - N * t;
            const int low = a + P * (b + P * c);  // padded id of voxel (a - 1, b - 1, c - 1)
            float4 V[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int q = low + (i & 1) + P * ((i >> 1) & 1) + P * P * (i >> 2);
                V[i] = term_load(vt[q]);
                occ |= (cl[q] ? 1u : 0u) << i;
            }
#pragma unroll
            for (int d = 0; d < NDIR; ++d) {
                unsigned through = 0;
                float ks = 0.f, zr = 0.f, zi = 0.f, cd = 0.f;
#pragma unroll
                for (int i = 0; i < vox_cnt(d); ++i) {
                    const int v = vox_idx(d, i);
                    through |= occ >> v & 1u;
                    ks += V[v].x;
                    zr += V[v].y;
                    if (FULL) zi += V[v].z;
                    if (FULL) cd += V[v].w;
                }
                mask |= through << d;
                const float L0 = dir_len2(d) == 1 ? L0e : dir_len2(d) == 2 ? L0f : L0b;
                const int pi = pbase + d * SL + s;
                A.pl.k[pi] = ks;
                A.pl.kal[pi] = zr * L0;
                if (FULL) A.pl.kbe[pi] = zi * L0;
                if (FULL && A.pl.kd) A.pl.kd[pi] = cd;
            }
            // the voxel whose lowest corner is this slot, for kernels that rebuild
            // spring parameters from voxels (zero where there is no kept voxel)
            A.pl.vkp[ri.slot_base + s] = V[7];
        }
        const unsigned long long pres = __ballot(occ != 0);
        int inc = __popc(mask);
        const int own = inc;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        masks[e] = mask;
        before[e] = inc - own;
        if (lane == 63) {
            pmask[u] = pres;
            rspr[u] = inc;
        }
    }
    __syncthreads();
    // 5. canonical ids: nodes by slot, springs by (slot, direction)
    if (wave == 0) {
        const bool on = lane < runs;
        const unsigned long long pm = on ? pmask[lane] : 0ull;
        const int own_n = __popcll(pm), own_s = on ? rspr[lane] : 0;
        int in = own_n, is = own_s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int tn = __shfl_up(in, o, 64), ts = __shfl_up(is, o, 64);
            if (lane >= o) {
                in += tn;
                is += ts;
            }
        }
        if (on) {
            nbase[lane] = in - own_n;
            sbase[lane] = is - own_s;
        }
        const unsigned long long some = __ballot(pm != 0);
        if (lane == (some ? __ffsll(some) - 1 : 0))  // the lowest node's layer
            zlow = some ? div_small(div_small(64 * lane + __ffsll(pm) - 1, mulN), mulN) : 0;
        if (lane == 63) {
            RobotInfo o = ri;
            o.M = in;
            o.S = is;
            A.robots_out[r] = o;
            A.diverged[r] = 0;
        }
    }
    __syncthreads();
    // 6. index and initial state: lattice positions with the lowest node on
    // z = 0.  An absent lattice point sits far outside the robot (2e4 m plus its
    // lattice offset, beyond the 1e4 m ghost slots): the step kernels evaluate
    // every stencil spring, and an absent one (zero parameters) then never meets
    // a zero length.
    const int zc = zlow;
#pragma unroll
    for (int e = 0; e < RPW; ++e) {
        const int u = wave + e * W, s = 64 * u + lane;
        if (u >= runs || s >= SL) continue;
        const int t = div_small(s, mulN), c = div_small(t, mulN), b = t - N * c, a = s - N * t;
        const unsigned long long pm = pmask[u];
        const bool here = pm >> lane & 1ull;
        const float far = here ? 0.f : 2e4f;
        const float4 p = make_float4(far + A.voxel_len * a, far + A.voxel_len * b, far + A.voxel_len * (c - zc),
                                     here ? 1.f : 0.f);
        const int g = ri.slot_base + s;
        A.x0[g] = p;
        A.x[g] = p;
        A.v[g] = make_float4(0.f, 0.f, 0.f, 0.f);
        A.slot_node[g] = here ? nbase[u] + __popcll(pm & ((1ull << lane) - 1ull)) : -1;
        A.ix.base[g] = sbase[u] + before[e];
        A.ix.mask[g] = (uint16_t)masks[e];
    }
}

// Node and spring offsets of every robot (prefix sums over robots), the first
// robot with an out-of-range class (-1: none), and the step counter back to
// zero; the same numbers go to pinned host memory, so the host has them once
// the stream is synchronised, without a copy.
__global__ __launch_bounds__(1024) void k_finish_build(const RobotInfo *robots, int R, uint8_t *bad_class,
                                                       int64_t *mass_off, int64_t *spring_off, int64_t *step,
                                                       int64_t *host) {
    __shared__ int64_t tm[16], ts[16];
    __shared__ int bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) bad = INT32_MAX;
    __syncthreads();
    const int per = (R + 1023) / 1024, r0 = min(tid * per, R), r1 = min(r0 + per, R);
    int64_t m = 0, s = 0;
    for (int r = r0; r < r1; ++r) {
        m += robots[r].M;
        s += robots[r].S;
        if (bad_class[r]) {
            atomicMin(&bad, r);
            bad_class[r] = 0;
        }
    }
    int64_t im = m, is = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t a = __shfl_up(im, o, 64), b = __shfl_up(is, o, 64);
        if (lane >= o) {
            im += a;
            is += b;
        }
    }
    if (lane == 63) {
        tm[wave] = im;
        ts[wave] = is;
    }
    __syncthreads();
    int64_t om = im - m, os = is - s;
    for (int q = 0; q < wave; ++q) {
        om += tm[q];
        os += ts[q];
    }
    for (int r = r0; r < r1; ++r) {
        mass_off[r] = host[1 + r] = om;
        spring_off[r] = host[2 + R + r] = os;
        om += robots[r].M;
        os += robots[r].S;
    }
    if (r0 < R && r1 == R) {
        mass_off[R] = host[1 + R] = om;
        spring_off[R] = host[2 + 2 * R] = os;
    }
    if (tid == 0) {
        host[0] = bad == INT32_MAX ? -1 : bad;
        *step = 0;
    }
}

}  // namespace

hipError_t launch_build_mesh(const RobotInfo *robots, int R, int max_side, bool full, const sr_sim_params &p,
                             const uint8_t *cls, const float *w, uint8_t *kept, Planes pl, SpringIndex ix,
                             float4 *x0, float4 *x, float4 *v, int32_t *slot_node, uint8_t *bad_class,
                             uint8_t *diverged, hipStream_t st) {
    BuildArgs A;
    A.robots = robots;
    A.robots_out = const_cast<RobotInfo *>(robots);
    A.cls = cls;
    A.w = w;
    A.kept = kept;
    A.pl = pl;
    A.ix = ix;
    A.x0 = x0;
    A.x = x;
    A.v = v;
    A.slot_node = slot_node;
    A.bad_class = bad_class;
    A.diverged = diverged;
    for (int c = 0; c < 5; ++c) {
        A.k_class[c] = p.k_class[c];
        A.ac_cos[c] = (float)((double)p.a_class[c] * cos((double)p.phi_class[c]));
        A.ac_sin[c] = (float)((double)p.a_class[c] * sin((double)p.phi_class[c]));
        A.a_class[c] = p.a_class[c];
        A.phi_class[c] = p.phi_class[c];
    }
    A.weight_act = (p.flags & SR_WEIGHT_ACTUATION) != 0;
    A.dash2m = (float)(2.0 * (double)p.mass * (double)p.zeta_spring * (double)p.zeta_spring);
    A.voxel_len = p.voxel_len;
    if (max_side <= 6)
        hipLaunchKernelGGL((full ? k_build_mesh<256, 6, true> : k_build_mesh<256, 6, false>), dim3(R), dim3(256), 0,
                           st, A);
    else
        hipLaunchKernelGGL((full ? k_build_mesh<512, SR_MAX_SIDE, true> : k_build_mesh<512, SR_MAX_SIDE, false>),
                           dim3(R), dim3(512), 0, st, A);
    return hipGetLastError();
}

hipError_t launch_finish_build(const RobotInfo *robots, int R, uint8_t *bad_class, int64_t *mass_off,
                               int64_t *spring_off, int64_t *step, int64_t *host, hipStream_t st) {
    hipLaunchKernelGGL(k_finish_build, dim3(1), dim3(1024), 0, st, robots, R, bad_class, mass_off, spring_off, step,
                       host);
    return hipGetLastError();
}

}  // namespace sr
