// query.hip -- genome MLP over every robot's voxel grid (Sec. II-B Eq. (1), Sec. II-C).
//
// For voxel (i,j,k) of an n^3 grid the query point is v = ((i+1/2)/n, (j+1/2)/n, (k+1/2)/n);
// gamma(v) = [cos(2 pi B v), sin(2 pi B v)] (32 + 32 entries), h1 = tanh(W1 gamma + b1),
// h2 = tanh(W2 h1 + b2), o = W3 h2 + b3; the class is argmax o[0..4] (lowest id on ties) and
// the weight is sigmoid(o[5]).
#include "internal.h"

namespace sr {

namespace {

constexpr int QB = 512;  // threads per workgroup: 8 waves, each 16 voxels (a tile) at a time
constexpr int QTAB_ROBOTS = 128;  // populations from which the encoding is tabulated
constexpr int OFF_W1 = 0, OFF_B1 = 4096, OFF_W2 = 4160, OFF_B2 = 8256, OFF_W3 = 8320, OFF_B3 = 8704;

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// entry q of the encoding at v: cos and sin of 2 pi b_q . v, taken as
// pi * (2 b_q . v) so the angle scaling is exact
__device__ __forceinline__ void encode(const float *b, float vx, float vy, float vz, float &cs, float &sn) {
    const float t = 2.0f * fmaf(b[2], vz, fmaf(b[1], vy, b[0] * vx));
    sincospif(t, &sn, &cs);
}

// Query point of voxel v of an n^3 grid
__device__ __forceinline__ float3 query_point(int v, int n, float inv) {
    return make_float3(((v % n) + 0.5f) * inv, (((v / n) % n) + 0.5f) * inv, ((v / (n * n)) + 0.5f) * inv);
}

// The encoding depends on the grid side and the voxel only, not on the robot:
// for populations of QTAB_ROBOTS robots or more one launch first writes it for
// every side present, in the order a query lane reads it (16 values of one
// voxel's lane quarter side by side), and the query kernels load it, one tile
// ahead, instead of computing 8 sin/cos pairs per lane and tile.  Below that the
// extra launch costs more than it saves.  Build from genomes without / with the
// table, us, FP32 then BF16: 128 robots of 5^3 35.0 / 36.7, 34.2 / 35.6; of 8^3 50.6 /
// 50.9, 42.3 / 42.7; of 10^3 75.0 / 74.0, 56.9 / 55.5; of 4^3 to 12^3 92.0 / 90.6, 70.0 /
// 67.0; 64 of 8^3 40.4 / 43.0, 36.8 / 38.1; 256 of 8^3 70.7 / 68.3, 55.0 / 52.4; 512 of
// 10^3 184 / 170, 120 / 106.
struct QueryTable {
    int base[SR_MAX_SIDE + 2];  // first table voxel of side n; base[SR_MAX_SIDE + 1]: all
};

template <bool BF>
__global__ __launch_bounds__(256) void k_encode(QueryTable tab, const float *B, void *out) {
    const int e = blockIdx.x * 256 + threadIdx.x, v = e / SR_PE_M, q = e % SR_PE_M;
    if (v >= tab.base[SR_MAX_SIDE + 1]) return;
    int n = 1;
    while (v >= tab.base[n + 1]) ++n;
    const float3 p = query_point(v - tab.base[n], n, 1.0f / (float)n);
    float cs, sn;
    encode(B + 3 * q, p.x, p.y, p.z, cs, sn);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int f = q + 32 * h;
        const float val = h ? sn : cs;
        if constexpr (BF)  // feature 16 m + 4 kq + i
            static_cast<unsigned short *>(out)[(v * 4 + ((f >> 2) & 3)) * 16 + 4 * (f >> 4) + (f & 3)] = f2bf(val);
        else  // feature 4 b + kq
            static_cast<float *>(out)[(v * 4 + (f & 3)) * 16 + (f >> 2)] = val;
    }
}

// ---------------------------------------------------------------- FP32 MFMA form
// Activations are kept transposed (features x voxels), one wave handles 16
// voxels, and each layer is D = W H^T on v_mfma_f32_16x16x4_f32: lane l of A
// holds row l%16 and k = l/16, lane l of B column l%16 and k = l/16, lane l of
// D column l%16 and rows 4(l/16)..+3.  The instruction accumulates its four
// products as FMAs in ascending k on top of C (measured against an fmaf chain:
// no mismatch in 2 million results, zeros and denormals among them), so with
// the bias as the first C and K-steps in ascending order the sums are those of
// the scalar loop a = b_i; a = fma(W_ij, h_j, a), bit for bit.
// D row 4 kq + i of output block m is given weight row 16 m + 4 i + kq: then
// register i of lane quarter kq holds feature 4 (4 m + i) + kq, which is the B
// operand of K-step 4 m + i of the next layer, and activations never leave
// registers.
// The fragments of K-steps 4 c .. 4 c + 3 of a lane are one 16-byte LDS read.
// Bound by the tanh and sin/cos of every feature (about 1400 VALU instructions
// a tile of 16 voxels) and 144 matrix instructions of 32 cycles; four waves a
// SIMD hide the latencies of both, so the fragments are read from LDS for every
// tile instead of held in registers (with them in registers, two waves a SIMD,
// 1.23 ms instead of 1.07 at 4096 robots of 10^3).
// Measured against one voxel per thread with weights broadcast from LDS, which
// the LDS reads bound: 4096 robots of 10^3 2.26 -> 1.07 ms (66 TFLOP/s of the
// MLP's products), 30 robots of 5^3 63 -> 14 us.  With the encoding from the
// table 0.94 ms: 1.16 M cycles of matrix instructions and 0.94 M of VALU issue
// per SIMD, which add up to the 2.06 M it takes; on this card FP32 matrix
// instructions do not run beside VALU ones of the same SIMD.
constexpr int FRAG3 = 2 * 4 * 4 * 64;  // first fragment quad of the output layer
constexpr int NFRAG = FRAG3 + 4 * 64;

template <bool TAB>
__global__ __launch_bounds__(QB) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_query_fp32(
    const RobotInfo *robots, const float *genomes, const float *B, uint8_t *cls, float *w, int tiles, QueryTable tab,
    const float4 *enc) {
    __shared__ float4 Ws[NFRAG];  // [layer][m][c][lane], then [c][lane] of the output layer
    __shared__ float bias[64 + 64 + 16];
    __shared__ float Bs[3 * SR_PE_M];
    const int r = blockIdx.x, part = blockIdx.y;
    const RobotInfo ri = robots[r];
    const int n = ri.n, nv = n * n * n;
    if (part * tiles * 16 >= nv) return;
    const float *g = genomes + (size_t)r * SR_GENOME_LEN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int col = lane & 15, kq = lane >> 4;  // voxel column and k of this lane
    {
        float *Wf = reinterpret_cast<float *>(Ws);
        for (int q = tid; q < 64 * 64; q += QB) {
            const int row = q >> 6, j = q & 63;
            // row 16 m + 4 i + kq' is A row 4 kq' + i of block m; feature j is k = j % 4 of K-step j / 4
            const int at = ((row >> 4) * 4 + (j >> 4)) * 64 + (j & 3) * 16 + 4 * (row & 3) + ((row >> 2) & 3);
            Wf[4 * at + ((j >> 2) & 3)] = g[OFF_W1 + q];
            Wf[4 * (at + 4 * 4 * 64) + ((j >> 2) & 3)] = g[OFF_W2 + q];
        }
        for (int q = tid; q < 16 * 64; q += QB) {
            const int row = q >> 6, j = q & 63;  // rows in their own order
            Wf[4 * (FRAG3 + (j >> 4) * 64 + (j & 3) * 16 + row) + ((j >> 2) & 3)] = q < 6 * 64 ? g[OFF_W3 + q] : 0.f;
        }
        for (int q = tid; q < 64; q += QB) {
            bias[q] = g[OFF_B1 + q];
            bias[64 + q] = g[OFF_B2 + q];
        }
        if (tid < 16) bias[128 + tid] = tid < 6 ? g[OFF_B3 + tid] : 0.f;
        for (int q = tid; q < 3 * SR_PE_M; q += QB) Bs[q] = B[q];
    }
    __syncthreads();

    const float inv = 1.0f / (float)n;
    const int vend = min(nv, (part + 1) * tiles * 16);
    const int first = (part * tiles + (tid >> 6)) * 16;
    float4 next[TAB ? 4 : 1];  // the next tile's encoding
    auto fetch = [&](int v0) {
        const int v = v0 + col < nv ? v0 + col : nv - 1;
#pragma unroll
        for (int c = 0; c < (TAB ? 4 : 0); ++c) next[c] = enc[((tab.base[n] + v) * 4 + kq) * 4 + c];
    };
    fetch(first);
    for (int v0 = first; v0 < vend; v0 += QB / 4) {
        const int vid = v0 + col;
        // the tile loop must not hoist the fragments and biases into registers
        int at = lane, bq = kq;
        __asm__ volatile("" : "+v"(at), "+v"(bq));
        float h[16];
        if constexpr (TAB) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                h[4 * c] = next[c].x;
                h[4 * c + 1] = next[c].y;
                h[4 * c + 2] = next[c].z;
                h[4 * c + 3] = next[c].w;
            }
            fetch(v0 + QB / 4);
        } else {
            const float3 p = query_point(vid < nv ? vid : nv - 1, n, inv);
#pragma unroll
            for (int b = 0; b < 8; ++b) encode(Bs + 3 * (4 * b + bq), p.x, p.y, p.z, h[b], h[8 + b]);
        }
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            f32x4 acc[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[m][i] = bias[64 * layer + 16 * m + 4 * i + bq];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float4 f[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) f[m] = Ws[((layer * 4 + m) * 4 + c) * 64 + at];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const float a = e == 0 ? f[m].x : e == 1 ? f[m].y : e == 2 ? f[m].z : f[m].w;
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, h[4 * c + e], acc[m], 0, 0, 0);
                    }
            }
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) h[4 * m + i] = tanhf(acc[m][i]);
        }
        // output layer: rows 0..5 of a 16-row block, in their own order
        f32x4 acc;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = bias[128 + 4 * bq + i];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float4 f = Ws[FRAG3 + c * 64 + at];
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f.x, h[4 * c], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f.y, h[4 * c + 1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f.z, h[4 * c + 2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f.w, h[4 * c + 3], acc, 0, 0, 0);
        }
        // lane col (kq = 0) holds o0..o3, lane col + 16 (kq = 1) holds o4, o5
        const float o4 = __shfl(acc[0], col + 16, 64);
        const float o5 = __shfl(acc[1], col + 16, 64);
        if (kq == 0 && vid < nv) {
            const float o[5] = {acc[0], acc[1], acc[2], acc[3], o4};
            int best = 0;
#pragma unroll
            for (int q = 1; q < 5; ++q)
                if (o[q] > o[best]) best = q;
            cls[ri.vox_base + vid] = (uint8_t)best;
            w[ri.vox_base + vid] = 1.0f / (1.0f + expf(-o5));
        }
    }
}

// ---------------------------------------------------------------- BF16 MFMA form
// Activations are kept transposed (features x voxels), so each layer is
// D = W H^T with the weights as the MFMA A operand and the activations as B.
// gfx950's v_mfma_f32_16x16x32_bf16: lane l of A holds row l%16 and eight
// values of k, lane l of B column l%16 and the same eight k, lane l of D
// column l%16 and rows 4(l/16)..+3.  A contraction may number its k in any
// order that A and B share; here k = 8 kq + j (kq = l/16, j = 0..7) of K-block
// b is feature 32 b + 16 (j/4) + 4 kq + j%4.  Then the D fragments of output
// blocks 2b and 2b + 1, side by side, are exactly the B fragment of K-block b
// of the next layer, so activations never leave registers, and a lane's A
// fragment is two 8-byte runs of one weight row.  One wave handles 16 voxels.
// Weights are staged in LDS as BF16 (round to nearest even) in fragment order:
// a lane's fragment is one 16-byte read.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// activations to BF16: the hardware's rounding (v_cvt_pk_bf16_f32) gives f2bf's
// bits on every number (checked over all 2^32 encodings)
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4 pack4(float a, float b, float c, float d) {
    const bf16x4 r = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    return __builtin_bit_cast(s16x4, r);
}

__device__ __forceinline__ bf16x8 cat8(s16x4 lo, s16x4 hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Bound by the tanh (and, without the table, sin/cos) of every feature on the
// VALU.  The work of a
// small population's robot is split over workgroups like the FP32 form's.
// Measured with the table, fragment-order weights, 8 waves a SIMD and hardware
// rounding to BF16 against row-order weights in registers: 1024 uneven robots 237
// -> 151 us, 256 robots of 8^3 42 -> 21 us.
constexpr int BFRAG3 = 2 * 4 * 2 * 64;  // first fragment of the output layer
constexpr int BNFRAG = BFRAG3 + 2 * 64;

template <bool TAB>
__global__ __launch_bounds__(QB) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_query_bf16(
    const RobotInfo *robots, const float *genomes, const float *B, uint8_t *cls, float *w, int tiles, QueryTable tab,
    const uint4 *enc) {
    __shared__ uint4 Ws[BNFRAG];  // [layer][m][K-block][lane], then [K-block][lane] of the output layer
    __shared__ float bias[64 + 64 + 6];
    __shared__ float Bs[3 * SR_PE_M];
    const int r = blockIdx.x, part = blockIdx.y;
    const RobotInfo ri = robots[r];
    const int n = ri.n, nv = n * n * n;
    if (part * tiles * 16 >= nv) return;
    const float *g = genomes + (size_t)r * SR_GENOME_LEN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int col = lane & 15, kq = lane >> 4;  // voxel column and k quarter of this lane
    {
        unsigned short *Wb = reinterpret_cast<unsigned short *>(Ws);
        // feature 32 b + 16 h + 4 kq' + i is entry 4 h + i of K-block b's lane quarter kq'
        auto place = [](int frag, int row, int j) {
            return 8 * ((frag + (j >> 5)) * 64 + ((j >> 2) & 3) * 16 + (row & 15)) + 4 * ((j >> 4) & 1) + (j & 3);
        };
        for (int q = tid; q < 64 * 64; q += QB) {
            const int row = q >> 6, j = q & 63;
            Wb[place(2 * (row >> 4), row, j)] = f2bf(g[OFF_W1 + q]);
            Wb[place(2 * (4 + (row >> 4)), row, j)] = f2bf(g[OFF_W2 + q]);
        }
        for (int q = tid; q < 16 * 64; q += QB)
            Wb[place(2 * 8, q >> 6, q & 63)] = q < 6 * 64 ? f2bf(g[OFF_W3 + q]) : 0;
        for (int q = tid; q < 64; q += QB) {
            bias[q] = g[OFF_B1 + q];
            bias[64 + q] = g[OFF_B2 + q];
        }
        if (tid < 6) bias[128 + tid] = g[OFF_B3 + tid];
        for (int q = tid; q < 3 * SR_PE_M; q += QB) Bs[q] = B[q];
    }
    __syncthreads();

    const float inv = 1.0f / (float)n;
    const int vend = min(nv, (part + 1) * tiles * 16);
    const int first = (part * tiles + (tid >> 6)) * 16;
    uint4 next[TAB ? 2 : 1];  // the next tile's encoding
    auto fetch = [&](int v0) {
        const int v = v0 + col < nv ? v0 + col : nv - 1;
#pragma unroll
        for (int c = 0; c < (TAB ? 2 : 0); ++c) next[c] = enc[((tab.base[n] + v) * 4 + kq) * 2 + c];
    };
    fetch(first);
    for (int v0 = first; v0 < vend; v0 += QB / 4) {
        const int vid = v0 + col;
        // the tile loop must not hoist the fragments and biases into registers
        int at = lane, bq = kq;
        __asm__ volatile("" : "+v"(at), "+v"(bq));
        // gamma(v) in 16-feature blocks (features 16 m + 4 kq + i of voxel `col`):
        // blocks 0, 1 are cos(2 pi b_q . v) and blocks 2, 3 sin of the same q
        s16x4 H[4];
        if constexpr (TAB) {
            H[0] = __builtin_bit_cast(s16x4, make_uint2(next[0].x, next[0].y));
            H[1] = __builtin_bit_cast(s16x4, make_uint2(next[0].z, next[0].w));
            H[2] = __builtin_bit_cast(s16x4, make_uint2(next[1].x, next[1].y));
            H[3] = __builtin_bit_cast(s16x4, make_uint2(next[1].z, next[1].w));
            fetch(v0 + QB / 4);
        } else {
            const float3 p = query_point(vid < nv ? vid : nv - 1, n, inv);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                float cs[4], sn[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) encode(Bs + 3 * (16 * m + 4 * bq + i), p.x, p.y, p.z, cs[i], sn[i]);
                H[m] = pack4(cs[0], cs[1], cs[2], cs[3]);
                H[m + 2] = pack4(sn[0], sn[1], sn[2], sn[3]);
            }
        }
        // two tanh layers
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            const float *bb = bias + 64 * layer;
            const bf16x8 b0 = cat8(H[0], H[1]), b1 = cat8(H[2], H[3]);
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) {
                const uint4 *f = Ws + 2 * (4 * layer + mb) * 64 + at;
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[0]), b0, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[64]), b1, acc, 0, 0, 0);
                const int f0 = 16 * mb + 4 * bq;
                H[mb] = pack4(tanhf(acc[0] + bb[f0]), tanhf(acc[1] + bb[f0 + 1]), tanhf(acc[2] + bb[f0 + 2]),
                              tanhf(acc[3] + bb[f0 + 3]));
            }
        }
        // output layer: rows 0..5 of a 16-row block
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Ws[BFRAG3 + at]), cat8(H[0], H[1]),
                                                      acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Ws[BFRAG3 + 64 + at]),
                                                      cat8(H[2], H[3]), acc, 0, 0, 0);
        // lane col (kq = 0) holds o0..o3, lane col + 16 (kq = 1) holds o4, o5
        const float o4 = __shfl(acc[0], col + 16, 64);
        const float o5 = __shfl(acc[1], col + 16, 64);
        if (kq == 0 && vid < nv) {
            float o[5] = {acc[0] + bias[128], acc[1] + bias[129], acc[2] + bias[130], acc[3] + bias[131],
                          o4 + bias[132]};
            int best = 0;
#pragma unroll
            for (int q = 1; q < 5; ++q)
                if (o[q] > o[best]) best = q;
            cls[ri.vox_base + vid] = (uint8_t)best;
            w[ri.vox_base + vid] = 1.0f / (1.0f + expf(-(o5 + bias[133])));
        }
    }
}

}  // namespace

size_t query_table_bytes(const RobotInfo *robots, int R) {
    bool side[SR_MAX_SIDE + 1] = {};
    for (int r = 0; r < R; ++r) side[robots[r].n] = true;
    size_t vox = 0;
    for (int n = 1; n <= SR_MAX_SIDE; ++n) vox += side[n] ? n * n * n : 0;
    return R < QTAB_ROBOTS ? 0 : vox * 64 * sizeof(float);
}

hipError_t launch_query(const RobotInfo *robots, int R, uint32_t sides, const float *genomes, const float *B,
                        int precision, void *table, uint8_t *cls, float *w, hipStream_t st) {
    QueryTable tab;
    int vox = 0, max_side = 1;
    for (int n = 0; n <= SR_MAX_SIDE; ++n) {
        tab.base[n] = vox;
        if (!(sides >> n & 1u)) continue;
        vox += n * n * n;
        max_side = n;
    }
    tab.base[SR_MAX_SIDE + 1] = vox;
    const bool bf = precision == SR_QUERY_BF16;
    if (table) {
        const dim3 grid((vox * SR_PE_M + 255) / 256);
        if (bf) hipLaunchKernelGGL(k_encode<true>, grid, dim3(256), 0, st, tab, B, table);
        else hipLaunchKernelGGL(k_encode<false>, grid, dim3(256), 0, st, tab, B, table);
    }
    // tiles of 16 voxels per workgroup: a multiple of its 8 waves, as many as
    // still leave two workgroups for each of 256 CUs, so that the weights' way
    // into LDS is shared by many tiles (1024 uneven robots in BF16: 151 us with
    // a workgroup per robot, 166 us with four for the largest).  When workgroups of
    // 4 tiles still have a CU each, half their waves only stage weights and no
    // SIMD runs two tiles in turn.
    const int maxt = (max_side * max_side * max_side + 15) / 16;
    const int64_t want = (int64_t)R * maxt / (512 * 8);
    const int tiles = (int64_t)R * ((maxt + 3) / 4) <= 256 ? 4 : 8 * (int)(want < 1 ? 1 : want > 16 ? 16 : want);
    // robots in the grid's x: y ends at 65535, and a population of small robots may be larger
    const dim3 grid(R, (maxt + tiles - 1) / tiles);
    if (bf)
        hipLaunchKernelGGL((table ? k_query_bf16<true> : k_query_bf16<false>), grid, dim3(QB), 0, st, robots, genomes,
                           B, cls, w, tiles, tab, static_cast<const uint4 *>(table));
    else
        hipLaunchKernelGGL((table ? k_query_fp32<true> : k_query_fp32<false>), grid, dim3(QB), 0, st, robots, genomes,
                           B, cls, w, tiles, tab, static_cast<const float4 *>(table));
    return hipGetLastError();
}

}  // namespace sr
