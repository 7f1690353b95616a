// ga.hip -- one GA generation over a population of genomes (Sec. II-C, Table I):
// elites by rank, two k-tournaments per child, uniform crossover, per-gene
// Gaussian mutation, every random decision drawn from Philox-4x64-10 at the
// counter (generation, child, purpose, block) with key (seed, 0).
#include <cmath>

#include "internal.h"

namespace sr {

namespace {

// Philox-4x64 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11): per round,
// words 0 and 2 are multiplied by the two round multipliers; the high halves
// are xored with the other words and the key, the low halves move over; the
// key is bumped by the two Weyl constants between rounds.
struct U64x4 {
    uint64_t w[4];
};

// 64 x 64 -> 128 bit product in four 32 x 32 + 64 bit multiply-adds; no partial
// sum overflows
__device__ __forceinline__ void mul128(uint64_t a, uint64_t b, uint64_t &hi, uint64_t &lo) {
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p = (uint64_t)a0 * b0;
    const uint64_t m = (uint64_t)a1 * b0 + (p >> 32);
    const uint64_t q = (uint64_t)a0 * b1 + (uint32_t)m;
    hi = (uint64_t)a1 * b1 + (m >> 32) + (q >> 32);
    lo = (q << 32) | (uint32_t)p;
}

__device__ __forceinline__ U64x4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                               uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    const uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += W0;
            k1 += W1;
        }
        uint64_t hi0, lo0, hi1, lo1;
        mul128(M0, c0, hi0, lo0);
        mul128(M1, c2, hi1, lo1);
        const uint64_t y0 = hi1 ^ c1 ^ k0, y2 = hi0 ^ c3 ^ k1;
        c0 = y0;
        c1 = lo1;
        c2 = y2;
        c3 = lo0;
    }
    U64x4 r;
    r.w[0] = c0;
    r.w[1] = c1;
    r.w[2] = c2;
    r.w[3] = c3;
    return r;
}

enum { PUR_TOUR_A = 0, PUR_TOUR_B = 1, PUR_CX = 2, PUR_CX_MASK = 3, PUR_MUT = 4, PUR_GAUSS = 5 };

struct GAArgs {
    const float *fit;
    const float *gin;
    float *gout;
    int P, L, E, k;
    uint64_t p_cross_thr, p_mut_thr;
    float sigma;
    uint64_t seed, gen;
    int32_t *dec;
};

// a is better than b: larger fitness (NaN counts as -inf), ties to the lower index
__device__ __forceinline__ bool better(const float *fit, int a, int b) {
    float fa = fit[a], fb = fit[b];
    if (fa != fa) fa = -INFINITY;
    if (fb != fb) fb = -INFINITY;
    if (fa != fb) return fa > fb;
    return a < b;
}

// One launch does the whole generation; a workgroup is one of two kinds.
//
// Children: nch workgroups per child slot c >= E, each making `chunk`
// consecutive genes.  Bound by the integer multiplies of Philox (one block per
// four genes for the mutation flags), not by memory.  What it is built around:
//  - the child's few shared draws (both tournaments, the crossover flag, the
//    chunk's crossover mask) are one Philox evaluation with a draw block per
//    lane of wave 0, repeated per workgroup, beside the mutation draws of the
//    other waves;
//  - a gene mutates with probability p_mut, so almost every wave holds a
//    mutating gene but few lanes do: mutating genes are listed in LDS and the
//    Gaussian step (a Philox block, and log, sqrt and cos in FP64) runs over
//    the dense list.  The list's order does not matter, every entry draws from
//    its own counter;
//  - genes pass through LDS, so that loads and stores are coalesced for any
//    genome length and alignment;
//  - the chunks spread a child over several CUs, for small populations.
// Measured against a workgroup per child with the Gaussian step inside the
// gene loop and a separate elite launch: 30 genomes of 8710 genes 84 -> 9.5 us,
// 4096 394 -> 141 us (285 MB of genomes: 56 us at the copy rate), of which 94
// without mutations.  Chunks of 2048 genes instead of 3072 cost 163 us instead
// of 137 (the shared draws are per workgroup), cos(2 pi u) instead of cospi 13 us
// (its registers for large arguments), __umul64hi instead of mul128 10 us.
//
// Elites: a workgroup per individual ranks it against the population and, if
// it is among the E best, copies its genome unchanged to slot rank.
constexpr int GB = 256;     // threads per workgroup
constexpr int GCH = 3072;   // most genes per workgroup
constexpr int GMASK = GCH / 256;

__device__ void ga_elite(const GAArgs &A, int i) {
    __shared__ int part[GB / 64];
    int cnt = 0;
    for (int j = threadIdx.x; j < A.P; j += GB) cnt += better(A.fit, j, i) ? 1 : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = cnt;
    __syncthreads();
    const int rank = part[0] + part[1] + part[2] + part[3];
    if (rank >= A.E) return;
    const float *src = A.gin + (size_t)i * A.L;
    float *dst = A.gout + (size_t)rank * A.L;
    for (int q = threadIdx.x; q < A.L; q += GB) dst[q] = src[q];
    if (threadIdx.x == 0 && A.dec) {
        A.dec[3 * rank] = i;
        A.dec[3 * rank + 1] = i;
        A.dec[3 * rank + 2] = 0;
    }
}

// winner of a tournament whose draw blocks are words[4 b .. 4 b + 3]; wave 0
// only, candidate t on lane t.  `better` is a total order, so the fold's shape
// does not matter.
__device__ int tournament(const GAArgs &A, const uint64_t *words) {
    const int lane = threadIdx.x & 63;
    const uint64_t hi = words[lane < A.k ? lane : 0] >> 32;
    int win = (int)((hi * (uint64_t)A.P) >> 32);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int other = __shfl_xor(win, o, 64);
        if (better(A.fit, other, win)) win = other;
    }
    return win;
}

__global__ __launch_bounds__(GB) void k_ga_children(GAArgs A, int chunk, int nch, int64_t first) {
    const int64_t kids = (int64_t)(A.P - A.E) * nch, wg = first + blockIdx.x;
    if (wg >= kids) {
        ga_elite(A, (int)(wg - kids));
        return;
    }
    __shared__ float vals[GCH];
    __shared__ uint16_t list[GCH];
    // wave 0's draw blocks: 16 + 16 of the tournaments, the crossover flag, the mask
    __shared__ uint64_t words[4 * (33 + GMASK)];
    __shared__ int sh[4];
    const int tid = threadIdx.x;
    const int c = A.E + (int)(wg / nch);
    const int g0 = (int)(wg % nch) * chunk;
    const int len = A.L - g0 < chunk ? A.L - g0 : chunk;
    if (tid == 0) sh[3] = 0;
    if (tid < 33 + GMASK) {
        const int b = tid < 16 ? tid : tid < 32 ? tid - 16 : tid == 32 ? 0 : (g0 >> 8) + tid - 33;
        const int pur = tid < 16 ? PUR_TOUR_A : tid < 32 ? PUR_TOUR_B : tid == 32 ? PUR_CX : PUR_CX_MASK;
        const U64x4 r = philox4x64_10(A.gen, (uint64_t)c, (uint64_t)pur, (uint64_t)b, A.seed, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) words[4 * tid + q] = r.w[q];
    }
    __syncthreads();
    if (tid < 64) {
        const int a = tournament(A, words), b = tournament(A, words + 64);
        if (tid == 0) {
            sh[0] = a;
            sh[1] = b;
            sh[2] = words[4 * 32] < A.p_cross_thr;
            if (A.dec && g0 == 0) {
                A.dec[3 * c] = a;
                A.dec[3 * c + 1] = b;
                A.dec[3 * c + 2] = sh[2] ? 2 : 1;
            }
        }
    }
    // one draw block gives the mutation words of four consecutive genes
    for (int q0 = 4 * tid; q0 < len; q0 += 4 * GB) {
        const U64x4 mut = philox4x64_10(A.gen, (uint64_t)c, PUR_MUT, (uint64_t)((g0 + q0) >> 2), A.seed, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q0 + q < len && mut.w[q] < A.p_mut_thr) list[atomicAdd(&sh[3], 1)] = (uint16_t)(q0 + q);
    }
    __syncthreads();
    const bool cx = sh[2] != 0;
    const float *ga = A.gin + (size_t)sh[0] * A.L + g0, *gb = A.gin + (size_t)sh[1] * A.L + g0;
    for (int q = tid; q < len; q += GB) {
        const bool fromB = cx && ((words[4 * 33 + (q >> 6)] >> (q & 63)) & 1ULL);
        vals[q] = fromB ? gb[q] : ga[q];
    }
    __syncthreads();
    for (int i = tid; i < sh[3]; i += GB) {
        // Box-Muller from two 53-bit uniforms, u1 in (0, 1], u2 in [0, 1)
        const int q = list[i], g = g0 + q;
        const U64x4 z = philox4x64_10(A.gen, (uint64_t)c, PUR_GAUSS, (uint64_t)(g >> 1), A.seed, 0);
        const uint64_t z0 = (g & 1) ? z.w[2] : z.w[0], z1 = (g & 1) ? z.w[3] : z.w[1];
        const double u1 = ((double)(z0 >> 11) + 1.0) * 0x1.0p-53;
        const double u2 = (double)(z1 >> 11) * 0x1.0p-53;
        const double nz = sqrt(-2.0 * log(u1)) * cospi(2.0 * u2);
        vals[q] = (float)((double)vals[q] + (double)A.sigma * nz);
    }
    __syncthreads();
    float *out = A.gout + (size_t)c * A.L + g0;
    for (int q = tid; q < len; q += GB) out[q] = vals[q];
}

}  // namespace

hipError_t launch_ga(const float *fit, const float *gin, float *gout, int P, int L, int E, int k, uint64_t pc,
                     uint64_t pm, float sigma, uint64_t seed, uint64_t gen, int32_t *dec, hipStream_t st) {
    GAArgs A;
    A.fit = fit;
    A.gin = gin;
    A.gout = gout;
    A.P = P;
    A.L = L;
    A.E = E;
    A.k = k;
    A.p_cross_thr = pc;
    A.p_mut_thr = pm;
    A.sigma = sigma;
    A.seed = seed;
    A.gen = gen;
    A.dec = dec;
    // chunks of equal length, a multiple of 256 genes (one crossover-mask block):
    // as few as GCH allows, more for populations that would not fill 256 CUs
    // four times, but no shorter than 1024
    const int few = (L + GCH - 1) / GCH, most = (L + 1023) / 1024, fill = 1024 / P;
    const int parts = fill < few ? few : fill > most ? most : fill;
    const int chunk = ((L + parts - 1) / parts + 255) / 256 * 256, nch = (L + chunk - 1) / chunk;
    const int64_t total = (int64_t)(P - E) * nch + P, per = 1 << 23;  // a grid holds less than 2^32 threads
    for (int64_t first = 0; first < total; first += per) {
        const unsigned grid = (unsigned)(total - first < per ? total - first : per);
        hipLaunchKernelGGL(k_ga_children, dim3(grid), dim3(GB), 0, st, A, chunk, nch, first);
    }
    return hipGetLastError();
}

}  // namespace sr
