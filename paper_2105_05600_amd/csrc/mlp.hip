// The learned PST proposal network: forward, Gaussian-NLL backward and Adam,
// with BF16 matrix-core (MFMA) GEMMs and FP32 accumulation.
//
// Parameters live in one caller-owned float32 buffer laid out
// [W1 (in x hid), b1 (hid), W2 (hid x hid), b2 (hid), W3 (hid x out), b3 (out)]
// (row-vector convention, y = x W + b); gradients and Adam moments use the
// same layout.  Operands are rounded to BF16 (round to nearest even) as the
// GEMM tiles are staged in LDS; products accumulate in FP32.
#include <algorithm>

#include "common.h"

namespace rose {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ inline float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ inline float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

enum { EPI_STORE = 0, EPI_BIAS_GELU = 1, EPI_BIAS = 2, EPI_GELU_GRAD = 3 };

struct GemmArgs {
    int32_t M, N, K;
    const float* A;
    int64_t sam, sak;  // A(m, k) = A[m * sam + k * sak]
    const float* B;
    int64_t sbk, sbn;  // B(k, n) = B[k * sbk + n * sbn]
    float* C;
    int64_t ldc;       // C(m, n) = C[m * ldc + n]
    const float* bias; // EPI_BIAS*, length N
    float* H;          // EPI_BIAS_GELU: GELU(C), same layout as C
    const float* Z;    // EPI_GELU_GRAD: pre-activations, same layout as C
    int32_t mode;
    int32_t span;  // k that the operands' buffers reach (set by the launch)
};

// Products: C = A B with binary32 operands rounded to bfloat16 on their way
// into LDS and gfx950's double-K v_mfma_f32_32x32x16_bf16.  Every output
// element is one chain of these instructions over ascending k whatever the
// kernel and tile, so a product's bits do not depend on which one runs it.
// Operand layout: lane l holds A[l % 32][8 (l / 32) .. +7] and
// B[8 (l / 32) .. +7][l % 32]; the 16 accumulators of lane l are
// D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32].
//
// An LDS tile holds rows of kc bfloat16 (kc a multiple of 32) in 16-byte
// chunks of 8 consecutive k, the unit that is written (one chunk per lane
// from 8 binary32 values) and read back as an MFMA operand.  Within its row
// chunk c of row r lies at c ^ (r mod 8), or with 4 chunks per row at
// c ^ ((r / 2) mod 4): 8 lanes that touch the same chunk of 8 consecutive
// rows then touch 8 different groups of banks.
template <int KC>
__device__ inline int chunk_at(int row, int c) {
    return row * (KC / 8) + (c ^ (KC == 32 ? (row >> 1) & 3 : row & 7));
}

// How an operand lies in memory, as rows (m or n) by k.
enum { LD_K = 0,     // k contiguous (through pointers also backwards): two 16-byte loads per chunk, lanes along k
       LD_ROW = 1 }; // any other strides: 8 loads per chunk, lanes along the rows

struct OpView {
    const float* p;
    int64_t srow, sk;
    int32_t rows, K;
};

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef f32x4_t f32x4u_t __attribute__((aligned(4)));  // 16-byte loads need 4-byte alignment only

// the 8 values of row r at k .. k + 7 (0 past the matrix)
template <int LD>
__device__ inline void load_chunk(const OpView& o, int r, int k, float (&v)[8]) {
    if (r < o.rows && k + 8 <= o.K) {
        const float* q = o.p + r * o.srow + k * o.sk;
        if constexpr (LD == LD_K) {
            const bool back = o.sk < 0;
            const float* first = back ? q - 7 : q;
            const f32x4_t a = *(const f32x4u_t*)first, b = *(const f32x4u_t*)(first + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = back ? b[3 - e] : a[e];
                v[4 + e] = back ? a[3 - e] : b[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = q[e * o.sk];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (r < o.rows && k + e < o.K) ? o.p[r * o.srow + (k + e) * o.sk] : 0.0f;
    }
}

// The same through a raw buffer that starts at the tile's first row: a
// 32-bit offset per chunk, held for the whole product, plus a wave-uniform
// offset of the k-step.  kNoRow marks a chunk past the last row: at or past
// the buffer's size with every k-step added, it reads 0.  The launch keeps
// every offset of a tile (rows and `span` k together) below kNoRow; where that
// is not all of K (FAR), the buffers' start moves on every `span` k.  That is
// a kernel of its own: the moving start costs the others 5 % (2048^3: 61 us
// against 58).
constexpr uint32_t kNoRow = 0x80000000u;

__device__ inline __amdgpu_buffer_rsrc_t tile_buffer(const OpView& o, int row0, int k0) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(o.p + (row0 * o.srow + k0 * o.sk)), (short)0, (int)kNoRow,
                                             0x00020000);
}

template <int LD>
__device__ inline void load_chunk(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t k_bytes, uint32_t sk_bytes,
                                  float (&v)[8]) {
    if constexpr (LD == LD_K) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(b, (int)(off + 16 * h), (int)k_bytes, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = __uint_as_float(a[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, (int)(k_bytes + e * sk_bytes), 0));
    }
}

// a chunk of which only the first `left` values are inside the matrix
__device__ inline void load_chunk_tail(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t k_bytes, uint32_t sk_bytes,
                                       int left, float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
        v[e] = __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(b, (int)(e < left ? off : kNoRow), (int)(k_bytes + e * sk_bytes), 0));
}

// 8 binary32 values as a chunk of 8 bfloat16 (round to nearest even)
__device__ inline bf16x8_t to_chunk(const float (&v)[8]) {
    bf16x8_t c;
#pragma unroll
    for (int e = 0; e < 8; ++e) c[e] = (__bf16)v[e];
    return c;
}

__device__ inline void epilogue(const GemmArgs& g, const f32x16_t& acc, int mt, int nt, int lane) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = mt + 8 * (i / 4) + 4 * (lane >> 5) + (i % 4);
        const int n = nt + (lane & 31);
        if (m >= g.M || n >= g.N) continue;
        const int64_t o = m * g.ldc + n;
        const float v = acc[i];
        if (g.mode == EPI_STORE) {
            g.C[o] = v;
        } else if (g.mode == EPI_BIAS_GELU) {
            const float z = v + g.bias[n];
            g.C[o] = z;
            g.H[o] = gelu_f(z);
        } else if (g.mode == EPI_BIAS) {
            g.C[o] = v + g.bias[n];
        } else {
            g.C[o] = v * gelu_grad_f(g.Z[o]);
        }
    }
}

// Large products: a BM x BN tile per workgroup, WM x WN of it per wavefront.
// Bound by the binary32 operands on their way from L2 into the CU: a k-step
// of 32 moves (BM + BN) 128 bytes for BM BN 64 flops, which at 64 B per
// clock is as long as its matrix instructions take with 256 x 256.  The next
// step's values are loaded into registers before this step's matrix
// instructions and written to the other LDS buffer after them (one barrier
// per step).  4096^3 with 256 x 256: 0.219 ms, 627 TFLOP/s (1.74 ms, 79
// TFLOP/s, with one 64 x 64 tile, 4-byte loads and no load ahead).
template <int BM, int BN, int WM, int WN, int LA, int LB, bool FAR>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void k_gemm_tile(GemmArgs g) {
    constexpr int kThreads = (BM / WM) * (BN / WN) * 64, KC = 32, TM = WM / 32, TN = WN / 32;
    constexpr int CA = BM * (KC / 8) / kThreads, CB = BN * (KC / 8) / kThreads;  // chunks per thread
    __shared__ bf16x8_t As[2][BM * (KC / 8)];
    __shared__ bf16x8_t Bs[2][BN * (KC / 8)];
    // XCD x (workgroup index mod 8) takes a contiguous run of the tile list,
    // which goes down 4 tile rows before it moves to the next column: the
    // tiles in flight on an XCD share their operands in its L2
    const int nt = (g.N + BN - 1) / BN, mt = (g.M + BM - 1) / BM, total = nt * mt;
    int t;
    {
        const int b = blockIdx.x, x = b & 7, per = total >> 3, rem = total & 7;
        t = x * per + min(x, rem) + (b >> 3);
    }
    const int band = t / (4 * nt), rows_in = min(4, mt - 4 * band), in = t - band * 4 * nt;
    const int m0 = (4 * band + in % rows_in) * BM, n0 = (in / rows_in) * BN;
    const OpView A{g.A, g.sam, g.sak, g.M, g.K}, B{g.B, g.sbn, g.sbk, g.N, g.K};
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    float va[CA][8], vb[CB][8];
    const uint32_t ska = 4u * (uint32_t)g.sak, skb = 4u * (uint32_t)g.sbk;
    uint32_t oa[CA], ob[CB];
#pragma unroll
    for (int q = 0; q < CA; ++q) {
        const int e = tid + q * kThreads, r = LA == LD_ROW ? e % BM : e / 4, c = LA == LD_ROW ? e / BM : e % 4;
        oa[q] = m0 + r < g.M ? 4u * (uint32_t)g.sam * r + 8u * ska * c : kNoRow;
    }
#pragma unroll
    for (int q = 0; q < CB; ++q) {
        const int e = tid + q * kThreads, r = LB == LD_ROW ? e % BN : e / 4, c = LB == LD_ROW ? e / BN : e % 4;
        ob[q] = n0 + r < g.N ? 4u * (uint32_t)g.sbn * r + 8u * skb * c : kNoRow;
    }
    __amdgpu_buffer_rsrc_t ra = tile_buffer(A, m0, 0), rb = tile_buffer(B, n0, 0);
    int kbase = 0;  // the buffers' k
    auto fetch = [&](int k0) {
        if (FAR && k0 - kbase >= g.span) {
            ra = tile_buffer(A, m0, kbase = k0);
            rb = tile_buffer(B, n0, kbase);
        }
        const int kr = FAR ? k0 - kbase : k0;
        if (k0 + KC <= g.K) {
#pragma unroll
            for (int q = 0; q < CA; ++q) load_chunk<LA>(ra, oa[q], kr * ska, ska, va[q]);
#pragma unroll
            for (int q = 0; q < CB; ++q) load_chunk<LB>(rb, ob[q], kr * skb, skb, vb[q]);
        } else {  // the last, partial step
#pragma unroll
            for (int q = 0; q < CA; ++q) {
                const int e = tid + q * kThreads, c = LA == LD_ROW ? e / BM : e % 4;
                load_chunk_tail(ra, oa[q], kr * ska, ska, g.K - k0 - 8 * c, va[q]);
            }
#pragma unroll
            for (int q = 0; q < CB; ++q) {
                const int e = tid + q * kThreads, c = LB == LD_ROW ? e / BN : e % 4;
                load_chunk_tail(rb, ob[q], kr * skb, skb, g.K - k0 - 8 * c, vb[q]);
            }
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int q = 0; q < CA; ++q) {
            const int e = tid + q * kThreads, r = LA == LD_ROW ? e % BM : e / 4, c = LA == LD_ROW ? e / BM : e % 4;
            As[buf][chunk_at<KC>(r, c)] = to_chunk(va[q]);
        }
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const int e = tid + q * kThreads, r = LB == LD_ROW ? e % BN : e / 4, c = LB == LD_ROW ? e / BN : e % 4;
            Bs[buf][chunk_at<KC>(r, c)] = to_chunk(vb[q]);
        }
    };
    fetch(0);
    stage(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < g.K; k0 += KC, buf ^= 1) {
        const bool more = k0 + KC < g.K;
        if (more) fetch(k0 + KC);
#pragma unroll
        for (int kk = 0; kk < KC / 16; ++kk) {
            bf16x8_t a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = As[buf][chunk_at<KC>(wm + 32 * i + (lane & 31), 2 * kk + (lane >> 5))];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = Bs[buf][chunk_at<KC>(wn + 32 * j + (lane & 31), 2 * kk + (lane >> 5))];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (more) stage(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) epilogue(g, acc[i][j], m0 + wm + 32 * i, n0 + wn + 32 * j, lane);
}

// Small products (the network's): one 32 x 32 tile per workgroup, so that
// also a few rows or columns spread over the chip.  Bound by the latency of
// the loads: the 8 wavefronts together fetch kSmallK columns of both
// operands at once, two such stages ahead of the matrix instructions, and wavefront 0 runs the chain of
// matrix instructions over them.  One row through the network: 16 us for its
// three products (127 us with 64 x 64 tiles and 38 dependent loads per
// product); a 1024-sample training step 103 us (809 us).
// BUF: through the raw buffers of the tile kernels (a 32-bit offset per chunk);
// otherwise (strides past their range) through plain pointers.
constexpr int kSmallK = 256;
template <int LA, int LB, bool BUF, bool FAR>
__global__ __launch_bounds__(512) void k_gemm_small(GemmArgs g) {
    constexpr int KC = kSmallK, CH = 32 * (KC / 8) / 512;  // chunks per thread and operand
    __shared__ bf16x8_t As[2][32 * (KC / 8)];
    __shared__ bf16x8_t Bs[2][32 * (KC / 8)];
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    const OpView A{g.A, g.sam, g.sak, g.M, g.K}, B{g.B, g.sbn, g.sbk, g.N, g.K};
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    f32x16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    float va[2][CH][8], vb[2][CH][8];
    auto at = [&](int ld, int q, int* r, int* c) {
        const int e = tid + q * 512;
        *r = ld == LD_ROW ? e % 32 : e / (KC / 8);
        *c = ld == LD_ROW ? e / 32 : e % (KC / 8);
    };
    const uint32_t ska = 4u * (uint32_t)g.sak, skb = 4u * (uint32_t)g.sbk;
    uint32_t oa[CH], ob[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        int r, c;
        at(LA, q, &r, &c);
        oa[q] = m0 + r < g.M ? 4u * (uint32_t)g.sam * r + 8u * ska * c : kNoRow;
        at(LB, q, &r, &c);
        ob[q] = n0 + r < g.N ? 4u * (uint32_t)g.sbn * r + 8u * skb * c : kNoRow;
    }
    __amdgpu_buffer_rsrc_t ra = tile_buffer(A, m0, 0), rb = tile_buffer(B, n0, 0);
    int kbase = 0;  // the buffers' k
    auto fetch = [&](int k0, float (&va)[CH][8], float (&vb)[CH][8]) {
        const bool full = k0 + KC <= g.K;
        if (FAR && k0 - kbase >= g.span) {
            ra = tile_buffer(A, m0, kbase = k0);
            rb = tile_buffer(B, n0, kbase);
        }
        const int kr = FAR ? k0 - kbase : k0;
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            int r, c;
            at(LA, q, &r, &c);
            if constexpr (!BUF) load_chunk<LA>(A, m0 + r, k0 + 8 * c, va[q]);
            else if (full) load_chunk<LA>(ra, oa[q], kr * ska, ska, va[q]);
            else load_chunk_tail(ra, oa[q], kr * ska, ska, g.K - k0 - 8 * c, va[q]);
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            int r, c;
            at(LB, q, &r, &c);
            if constexpr (!BUF) load_chunk<LB>(B, n0 + r, k0 + 8 * c, vb[q]);
            else if (full) load_chunk<LB>(rb, ob[q], kr * skb, skb, vb[q]);
            else load_chunk_tail(rb, ob[q], kr * skb, skb, g.K - k0 - 8 * c, vb[q]);
        }
    };
    fetch(0, va[0], vb[0]);
    if (KC < g.K) fetch(KC, va[1], vb[1]);
    for (int k0 = 0; k0 < g.K; k0 += 2 * KC) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // the stage at k0 + h KC, register set and LDS buffer h
            const int ks = k0 + h * KC;
            if (ks >= g.K) break;
            int r, c;
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                at(LA, q, &r, &c);
                As[h][chunk_at<KC>(r, c)] = to_chunk(va[h][q]);
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                at(LB, q, &r, &c);
                Bs[h][chunk_at<KC>(r, c)] = to_chunk(vb[h][q]);
            }
            // the other buffer's readers (wavefront 0, one stage back) passed
            // this barrier after their reads, so two buffers need one barrier
            __syncthreads();
            if (ks + 2 * KC < g.K) fetch(ks + 2 * KC, va[h], vb[h]);
            if (wave == 0) {
                // 8 instructions' operands at a time, so that the chain does
                // not wait for LDS between them (past K the chunks hold zeros)
                const int steps = min(KC / 16, (g.K - ks + 15) / 16);
                for (int kb = 0; kb < steps; kb += 8) {
                    bf16x8_t a[8], b[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        a[e] = As[h][chunk_at<KC>(lane & 31, 2 * (kb + e) + (lane >> 5))];
                        b[e] = Bs[h][chunk_at<KC>(lane & 31, 2 * (kb + e) + (lane >> 5))];
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[e], b[e], acc, 0, 0, 0);
                }
            }
        }
    }
    if (wave == 0) epilogue(g, acc, m0, n0, lane);
}

// Gaussian NLL per sample and its gradient w.r.t. the 12 outputs (scaled by
// 1/B); one block of one thread per sample (and per 1024 of them) adds the
// per-sample losses in a fixed order: each thread its own, the wavefront by
// butterfly, one wavefront the 16 partial sums.
constexpr int kNllThreads = 1024;
__global__ __launch_bounds__(kNllThreads) void k_nll(const float* out, const float* Y, int32_t B, float* dout,
                                                     float* loss) {
    __shared__ double part[kNllThreads / 64];
    double s = 0.0;
    const float invB = 1.0f / (float)B;
    for (int b = threadIdx.x; b < B; b += kNllThreads) {
        double lb = 0.0;
        float o[12], y[6];
#pragma unroll
        for (int d = 0; d < 12; ++d) o[d] = out[b * 12 + d];
#pragma unroll
        for (int d = 0; d < 6; ++d) y[d] = Y[b * 6 + d];
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            const float mu = o[d], ls = o[6 + d];
            const float r = y[d] - mu;
            const float inv = expf(-2.0f * ls);
            lb += (double)(0.5f * r * r * inv + ls);
            dout[b * 12 + d] = -r * inv * invB;
            dout[b * 12 + 6 + d] = (1.0f - r * r * inv) * invB;
        }
        s += lb;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double t = wave_sum(threadIdx.x < kNllThreads / 64 ? part[threadIdx.x] : 0.0);
        if (threadIdx.x == 0) *loss = (float)(t / (double)B);
    }
}

// column sums (bias gradients): a workgroup per 64 columns; wave w of its
// 16 sums rows w, w + 16, ... of its lane's column (each row read as one
// coalesced 64-column segment, 16 of them loaded before they are added: the
// kernel waits for memory, not for its 64 additions), then one lane per column adds the 16
// partial sums in wave order (a fixed order: deterministic)
constexpr int kColsumWaves = 16;
__global__ __launch_bounds__(1024) void k_colsum(const float* X, int32_t rows, int32_t cols, float* out) {
    __shared__ float part[kColsumWaves][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (c < cols) {
        int r = w;
        for (; r + 15 * kColsumWaves < rows; r += 16 * kColsumWaves) {
            float x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) x[q] = X[(int64_t)(r + q * kColsumWaves) * cols + c];
#pragma unroll
            for (int q = 0; q < 16; ++q) s += x[q];
        }
        for (; r < rows; r += kColsumWaves) s += X[(int64_t)r * cols + c];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && c < cols) {
        float t = 0.0f;
        for (int k = 0; k < kColsumWaves; ++k) t += part[k][lane];
        out[c] = t;
    }
}

__global__ __launch_bounds__(256) void k_adam(int64_t n, float* p, const float* gr, float* m, float* v, float lr,
                                             float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = gr[i];
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// How many k (a multiple of a kernel's k-step ks, or all K) the offsets of an
// operand's tile of `rows` rows reach with 31 bits, a step and a chunk past
// the last k included; 0: not even one step.
static int32_t tile_span(int64_t srow, int64_t sk, int32_t rows, int32_t ks, int32_t K) {
    if (srow < 0 || sk < 0 || srow >= (1 << 29) || sk >= (1 << 29)) return 0;
    const int64_t left = ((int64_t)kNoRow - 1) / 4 - rows * srow;
    const int32_t past = std::min(ks, K) + 8;
    if (left < past * sk) return 0;
    const int64_t k = sk > 0 ? left / sk - past : K;
    return k >= K ? K : (int32_t)(k / ks * ks);
}

// Kernel by output size and K (rows and columns contiguous in memory, us):
//   4096^2 x 4096  256: 210, 128: 264, 64: 420, small: 1052   (256 tiles of 256)
//   4096 x 2048 x 4096  256: 183, 128: 112, 64: 206
//   2048 x 1024 x 2048  128: 58, 64: 38, small: 78             (128 tiles of 128)
//   1024^2 x 1024  128: 29, 64: 17, small: 23                  (256 tiles of 64)
//   512^2 x 2048  64: 27, small: 20; 1024 x 256 x 1216  64: 18, small: 15
//   4096^2 x 128  256: 41, 128: 33, 64: 23 (few k-steps: the stores count,
//   and more workgroups overlap them with other tiles' products)
//   between these, K = 2048, 256 / 128 / 64:  2048^2 107 / 59 / 58 (K = 512:
//   48 / 24 / 19), 3072 x 2048 107 / 60 / 78, 4096 x 3072 108 / 98 / 152, 3584^2
//   108 / 119 / 152, 4352 x 4096 213 / 142 / 208, 4608^2 213 / 172 / 244
// so a wider tile is taken once it leaves (almost) every CU a workgroup.  The
// last round of workgroups is not looked at: just past 256 tiles of 256 the
// 128-square tile would be the faster one, at 256 tiles of 128 the 64-square.
template <int LA, int LB>
static void launch_gemm(GemmArgs g, hipStream_t s) {
    auto tiles = [&](int t) { return (int64_t)((g.M + t - 1) / t) * ((g.N + t - 1) / t); };
    auto reach = [&](int rows, int ks) {
        g.span = std::min(tile_span(g.sam, g.sak, std::min(rows, g.M), ks, g.K),
                          tile_span(g.sbn, g.sbk, std::min(rows, g.N), ks, g.K));
        return g.span > 0;
    };
    auto go = [&](auto near, auto far, dim3 blocks, int threads) {
        hipLaunchKernelGGL(g.span < g.K ? far : near, blocks, dim3(threads), 0, s, g);
    };
    const dim3 small((g.N + 31) / 32, (g.M + 31) / 32);
    if (g.K >= 512 && tiles(256) >= 192 && reach(256, 32))
        go(&k_gemm_tile<256, 256, 128, 64, LA, LB, false>, &k_gemm_tile<256, 256, 128, 64, LA, LB, true>,
           dim3((unsigned)tiles(256)), 512);
    else if (g.K >= 512 && tiles(128) >= 256 && reach(128, 32))
        go(&k_gemm_tile<128, 128, 64, 64, LA, LB, false>, &k_gemm_tile<128, 128, 64, 64, LA, LB, true>,
           dim3((unsigned)tiles(128)), 256);
    else if (tiles(64) >= 192 && reach(64, 32))
        go(&k_gemm_tile<64, 64, 32, 32, LA, LB, false>, &k_gemm_tile<64, 64, 32, 32, LA, LB, true>,
           dim3((unsigned)tiles(64)), 256);
    else if (reach(32, kSmallK))
        go(&k_gemm_small<LA, LB, true, false>, &k_gemm_small<LA, LB, true, true>, small, 512);
    else {  // row pitches of 64 MB or more, and negative strides
        const bool ka = g.sak == 1 || g.sak == -1, kb = g.sbk == 1 || g.sbk == -1;
        auto plain = kb ? (ka ? &k_gemm_small<LD_K, LD_K, false, false> : &k_gemm_small<LD_ROW, LD_K, false, false>)
                        : (ka ? &k_gemm_small<LD_K, LD_ROW, false, false> : &k_gemm_small<LD_ROW, LD_ROW, false, false>);
        hipLaunchKernelGGL(plain, small, dim3(512), 0, s, g);
    }
}

static rose_status gemm(int M, int N, int K, const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbk,
                        int64_t sbn, float* C, int64_t ldc, int mode, const float* bias, float* H, const float* Z,
                        hipStream_t s) {
    GemmArgs g{M, N, K, A, sam, sak, B, sbk, sbn, C, ldc, bias, H, Z, mode, K};
    if (sak == 1) sbk == 1 ? launch_gemm<LD_K, LD_K>(g, s) : launch_gemm<LD_K, LD_ROW>(g, s);
    else sbk == 1 ? launch_gemm<LD_ROW, LD_K>(g, s) : launch_gemm<LD_ROW, LD_ROW>(g, s);
    ROSE_CHECK_HIP(hipGetLastError());
    return ROSE_OK;
}

}  // namespace rose

struct rose_mlp {
    int32_t in, hid, out, max_batch;
    float *Z1, *H1, *Z2, *H2, *Y, *dY, *dZ2, *dZ1, *dH;
};

using namespace rose;

namespace {
struct Offs {
    int64_t W1, b1, W2, b2, W3, b3, total;
};
Offs offsets(int in, int hid, int out) {
    Offs o;
    o.W1 = 0;
    o.b1 = o.W1 + (int64_t)in * hid;
    o.W2 = o.b1 + hid;
    o.b2 = o.W2 + (int64_t)hid * hid;
    o.W3 = o.b2 + hid;
    o.b3 = o.W3 + (int64_t)hid * out;
    o.total = o.b3 + out;
    return o;
}
}  // namespace

extern "C" {

int64_t rose_mlp_param_count(int32_t in_dim, int32_t hidden, int32_t out_dim) {
    if (in_dim < 1 || hidden < 1 || out_dim != 12) return 0;
    return offsets(in_dim, hidden, out_dim).total;
}

rose_status rose_mlp_create(int32_t in_dim, int32_t hidden, int32_t out_dim, int32_t max_batch, rose_mlp** out) {
    clear_error();
    ROSE_REQUIRE(out != nullptr, ROSE_E_ARG, "rose_mlp_create: NULL output");
    *out = nullptr;
    ROSE_REQUIRE(in_dim >= 1 && in_dim <= 65536 && hidden >= 1 && hidden <= 4096 && out_dim == 12 &&
                     max_batch >= 1 && max_batch <= 65536,
                 ROSE_E_SHAPE, "rose_mlp_create: sizes out of range (out_dim must be 12)");
    rose_mlp* m = (rose_mlp*)calloc(1, sizeof(rose_mlp));
    ROSE_REQUIRE(m != nullptr, ROSE_E_DEVICE, "rose_mlp_create: out of host memory");
    m->in = in_dim;
    m->hid = hidden;
    m->out = out_dim;
    m->max_batch = max_batch;
    const size_t bh = sizeof(float) * (size_t)max_batch * hidden;
    const size_t bo = sizeof(float) * (size_t)max_batch * out_dim;
    float** bufs_h[] = {&m->Z1, &m->H1, &m->Z2, &m->H2, &m->dZ2, &m->dZ1, &m->dH};
    bool ok = true;
    for (float** b : bufs_h) ok = ok && hipMalloc((void**)b, bh) == hipSuccess;
    ok = ok && hipMalloc((void**)&m->Y, bo) == hipSuccess && hipMalloc((void**)&m->dY, bo) == hipSuccess;
    if (!ok) {
        rose_mlp_destroy(m);
        set_error("rose_mlp_create: hipMalloc failed");
        return ROSE_E_DEVICE;
    }
    *out = m;
    return ROSE_OK;
}

rose_status rose_mlp_destroy(rose_mlp* m) {
    clear_error();
    if (!m) return ROSE_OK;
    (void)hipDeviceSynchronize();
    float* bufs[] = {m->Z1, m->H1, m->Z2, m->H2, m->Y, m->dY, m->dZ2, m->dZ1, m->dH};
    for (float* b : bufs)
        if (b) (void)hipFree(b);
    free(m);
    return ROSE_OK;
}

static rose_status mlp_forward_impl(rose_mlp* m, const float* P, const float* X, int32_t B, float* out,
                                    hipStream_t s) {
    const Offs o = offsets(m->in, m->hid, m->out);
    rose_status st;
    if ((st = gemm(B, m->hid, m->in, X, m->in, 1, P + o.W1, m->hid, 1, m->Z1, m->hid, EPI_BIAS_GELU, P + o.b1,
                   m->H1, nullptr, s)) != ROSE_OK)
        return st;
    if ((st = gemm(B, m->hid, m->hid, m->H1, m->hid, 1, P + o.W2, m->hid, 1, m->Z2, m->hid, EPI_BIAS_GELU, P + o.b2,
                   m->H2, nullptr, s)) != ROSE_OK)
        return st;
    return gemm(B, m->out, m->hid, m->H2, m->hid, 1, P + o.W3, m->out, 1, out, m->out, EPI_BIAS, P + o.b3, nullptr,
                nullptr, s);
}

rose_status rose_mlp_forward(rose_mlp* m, const float* params_dev, const float* X_dev, int32_t B, float* out_dev,
                             hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(m && params_dev && X_dev && out_dev, ROSE_E_ARG, "rose_mlp_forward: NULL argument");
    ROSE_REQUIRE(B >= 1 && B <= m->max_batch, ROSE_E_SHAPE, "rose_mlp_forward: batch %d out of [1, %d]", B,
                 m->max_batch);
    return mlp_forward_impl(m, params_dev, X_dev, B, out_dev, s);
}

rose_status rose_mlp_loss_grad(rose_mlp* m, const float* params_dev, const float* X_dev, const float* Y_dev,
                               int32_t B, float* grads_dev, float* loss_dev, hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(m && params_dev && X_dev && Y_dev && grads_dev && loss_dev, ROSE_E_ARG,
                 "rose_mlp_loss_grad: NULL argument");
    ROSE_REQUIRE(B >= 1 && B <= m->max_batch, ROSE_E_SHAPE, "rose_mlp_loss_grad: batch %d out of [1, %d]", B,
                 m->max_batch);
    const Offs o = offsets(m->in, m->hid, m->out);
    const float* P = params_dev;
    float* G = grads_dev;
    rose_status st;
    if ((st = mlp_forward_impl(m, P, X_dev, B, m->Y, s)) != ROSE_OK) return st;
    hipLaunchKernelGGL(k_nll, dim3(1), dim3(kNllThreads), 0, s, m->Y, Y_dev, B, m->dY, loss_dev);
    ROSE_CHECK_HIP(hipGetLastError());
    const int hid = m->hid, in = m->in, out = m->out;
    // dW3 = H2^T dY ; db3 = colsum(dY)
    if ((st = gemm(hid, out, B, m->H2, 1, hid, m->dY, out, 1, G + o.W3, out, EPI_STORE, nullptr, nullptr, nullptr,
                   s)) != ROSE_OK)
        return st;
    hipLaunchKernelGGL(k_colsum, dim3((out + 63) / 64), dim3(64 * kColsumWaves), 0, s, m->dY, B, out, G + o.b3);
    // dZ2 = (dY W3^T) * gelu'(Z2)
    if ((st = gemm(B, hid, out, m->dY, out, 1, P + o.W3, 1, out, m->dZ2, hid, EPI_GELU_GRAD, nullptr, nullptr, m->Z2,
                   s)) != ROSE_OK)
        return st;
    // dW2 = H1^T dZ2 ; db2
    if ((st = gemm(hid, hid, B, m->H1, 1, hid, m->dZ2, hid, 1, G + o.W2, hid, EPI_STORE, nullptr, nullptr, nullptr,
                   s)) != ROSE_OK)
        return st;
    hipLaunchKernelGGL(k_colsum, dim3((hid + 63) / 64), dim3(64 * kColsumWaves), 0, s, m->dZ2, B, hid, G + o.b2);
    // dZ1 = (dZ2 W2^T) * gelu'(Z1)
    if ((st = gemm(B, hid, hid, m->dZ2, hid, 1, P + o.W2, 1, hid, m->dZ1, hid, EPI_GELU_GRAD, nullptr, nullptr, m->Z1,
                   s)) != ROSE_OK)
        return st;
    // dW1 = X^T dZ1 ; db1
    if ((st = gemm(in, hid, B, X_dev, 1, in, m->dZ1, hid, 1, G + o.W1, hid, EPI_STORE, nullptr, nullptr, nullptr,
                   s)) != ROSE_OK)
        return st;
    hipLaunchKernelGGL(k_colsum, dim3((hid + 63) / 64), dim3(64 * kColsumWaves), 0, s, m->dZ1, B, hid, G + o.b1);
    ROSE_CHECK_HIP(hipGetLastError());
    return ROSE_OK;
}

rose_status rose_mlp_adam(int64_t n, float* params_dev, const float* grads_dev, float* m_dev, float* v_dev,
                          int32_t step, float lr, float beta1, float beta2, float eps, hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(params_dev && grads_dev && m_dev && v_dev, ROSE_E_ARG, "rose_mlp_adam: NULL argument");
    ROSE_REQUIRE(n >= 1 && step >= 1, ROSE_E_ARG, "rose_mlp_adam: n >= 1 and step >= 1 required");
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, params_dev, grads_dev, m_dev,
                       v_dev, lr, beta1, beta2, eps, c1, c2);
    ROSE_CHECK_HIP(hipGetLastError());
    return ROSE_OK;
}

rose_status rose_gemm_bf16(int32_t M, int32_t N, int32_t K, const float* A_dev, int64_t sam, int64_t sak,
                           const float* B_dev, int64_t sbk, int64_t sbn, float* C_dev, int64_t ldc, hipStream_t s) {
    clear_error();
    ROSE_REQUIRE(A_dev && B_dev && C_dev, ROSE_E_ARG, "rose_gemm_bf16: NULL argument");
    ROSE_REQUIRE(M >= 1 && N >= 1 && K >= 1 && M <= 65536 && N <= 65536 && K <= 65536, ROSE_E_SHAPE,
                 "rose_gemm_bf16: sizes out of range");
    return gemm(M, N, K, A_dev, sam, sak, B_dev, sbk, sbn, C_dev, ldc, EPI_STORE, nullptr, nullptr, nullptr, s);
}

}  // extern "C"
