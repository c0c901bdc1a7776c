// float32 projection GEMM C = A B^T (A [M, K] activations, B [N, K] weights) for float32 models,
// on the float32 matrix instructions (16x16x4: float32 products and sums).
//
// What bounds it at the sizes a float32 model has (d 256, a few hundred rows): latency.  So many
// small workgroups, no staging and few dependent steps: a 256-thread workgroup takes a 32 x 32
// tile, each of its 4 wavefronts a quarter of K (in steps of 16, the steps dealt round-robin), with
// its operands loaded straight into the lanes that multiply them and kDepth steps in flight; the
// four quarters are added through LDS in wavefront order.  An element's sum does not depend on M
// or on the tile's place, so packed and padded batches agree bit for bit.
// Measured (us; 64 x 64 tiles on the vector units with a barrier per 16 columns before -> now):
// 384 rows, N 768, K 256: 24 -> 8; N 256, K 688: 67 -> 7; 4096 rows, N = K = 4096:
// 2237 -> 1977.
//
// Epilogues: store; residual add; SwiGLU over gate/up rows interleaved in blocks of 16 (a tile's 32
// weight rows are the gate and up rows of 16 features); QKV with RoPE at the restart positions and
// the cache UNPACK (a tile's rows are 16 dims of a head and their rotate-half partners).
//
// K of at most 64 over more tiles than the chip holds at once: a wavefront per tile (below).  4096 x 4096
// with 64 x 64 tiles on the vector units -> with a workgroup per tile -> now: K 16 20 -> 34 -> 20 us, K 64
// 43 -> 120 -> 41; K 128 74 -> 121 -> 73.
#include "device.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace {

constexpr int TB = 32, TK = 16, NT = 256, kDepth = 4;

// Row m of a tile, weight rows c .. c + 3 of its two blocks of 16 (first rows n0, n1) in v; t: the
// tile's index along N; old: C's values (load_old), read before the products.
template <int EPI>
__device__ __forceinline__ void load_old(f32x4 (&old)[2], int m, int n0, int n1, int c, const float* __restrict__ C,
                                         int64_t ldc, int M, int N, int vec) {
    if constexpr (EPI == ppk::kResidual) {
        if (!vec || m >= M) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int n = (i ? n1 : n0) + c;
            if (n + 4 <= N) old[i] = *reinterpret_cast<const f32x4*>(C + m * ldc + n);
        }
    }
}
template <int EPI>
__device__ __forceinline__ void finish(f32x4 (&v)[2], const f32x4 (&old)[2], int m, int n0, int n1, int t, int c,
                                       float* __restrict__ C, int64_t ldc, int M, int N, int vec, const ppk::QkvOut& qo,
                                       int D) {
    if (m >= M) return;
    if constexpr (EPI == ppk::kSwiGLU) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = silu(v[0][e]) * v[1][e];
        *reinterpret_cast<f32x4*>(C + m * ldc + t * 16 + c) = o;
    } else if constexpr (EPI == ppk::kQkvRope) {
        const int head = n0 / D, i0 = n0 % D + c;
        const int kind = head < qo.H ? 0 : (head < qo.H + qo.Hkv ? 1 : 2);   // q, k, v
        if (kind < 2) {
            const float2* cs = qo.table + int64_t(qo.slot_pos[m]) * (D / 2) + i0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = v[0][e], y = v[1][e];
                v[0][e] = rope_lo(x, y, cs[e].x, cs[e].y);
                v[1][e] = rope_hi_step(x, y, cs[e].x, cs[e].y);
            }
        }
        const int row = kind == 0 ? m : qo.slot_kv[m];
        if (row < 0) return;   // a pad slot has no cache row
        float* dst = kind == 0 ? static_cast<float*>(qo.q) + row * qo.ldq + head * D
                               : static_cast<float*>(kind == 1 ? qo.kc : qo.vc) + row * qo.ldkv +
                                     (head - qo.H - (kind == 2 ? qo.Hkv : 0)) * D;
        *reinterpret_cast<f32x4*>(dst + i0) = v[0];
        *reinterpret_cast<f32x4*>(dst + i0 + D / 2) = v[1];
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int n = (i ? n1 : n0) + c;
            float* p = C + m * ldc + n;
            if (vec && n + 4 <= N) {   // vec: C's rows are 16-byte aligned
                f32x4 o = v[i];
                if constexpr (EPI == ppk::kResidual) o += old[i];
                *reinterpret_cast<f32x4*>(p) = o;
            } else {
                for (int e = 0; e < 4 && n + e < N; ++e) p[e] = EPI == ppk::kResidual ? p[e] + v[i][e] : v[i][e];
            }
        }
    }
}

// How a tile's K is taken (the sum's order, and so its bits, are the same in all three):
// kLong   a workgroup per tile, at least kDepth steps for each of its wavefronts
// kMid    the same with fewer steps, no loads for the ones that are not there (clamped to the last
//         step, four times the bytes: 4096 x 4096, K 64: 120 us, 46 without them)
// 1 .. 4  K of so many steps, a wavefront per tile, its quarters (a step each) added in the
//         same order; no LDS, few registers
constexpr int kLong = 0, kMid = -1;

template <int EPI, int STEPS>
__global__ __launch_bounds__(NT) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda,
                                                      const float* __restrict__ B, int64_t ldb,
                                                      float* __restrict__ C, int64_t ldc, int M, int N, int K,
                                                      int vec, ppk::QkvOut qo, int D) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, q4 = lane >> 4, c = 4 * q4;
    const int tiles_n = (N + TB - 1) / TB;
    int m0, t;
    if constexpr (STEPS > 0) {   // the workgroup's four tiles: 2 x 2
        const int pairs_n = (tiles_n + 1) / 2;
        m0 = (blockIdx.x / pairs_n * 2 + (wave >> 1)) * TB;
        t = blockIdx.x % pairs_n * 2 + (wave & 1);
        if (m0 >= M || t >= tiles_n) return;
    } else {
        m0 = blockIdx.x / tiles_n * TB;
        t = blockIdx.x % tiles_n;
    }
    // first weight row of the tile's two blocks of 16
    int n0 = t * TB, n1 = n0 + 16;
    if constexpr (EPI == ppk::kQkvRope) {
        const int per_head = D / TB;
        n0 = t / per_head * D + t % per_head * 16;
        n1 = n0 + D / 2;
    }
    // lane l supplies row l % 16 of each block at columns 4 (l / 16) .. + 3 of a step: 16 rows x
    // 64 bytes a load; rows past the matrix read its last row (never stored)
    const float* a[2];
    const float* b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a[i] = A + int64_t(min(m0 + 16 * i + lr, M - 1)) * lda + c;
        b[i] = B + int64_t(min((i ? n1 : n0) + lr, N - 1)) * ldb + c;
    }
    constexpr int kSlots = STEPS > 0 ? STEPS : kDepth;
    f32x4 ra[kSlots][2], rb[kSlots][2];
    // step s of K into slot u (in range; with the clamp the long form is 2% faster: 4096 x 4096 x 1024
    // 530 and 518 us)
    auto issue = [&](int u, int s) {
        const int k = TK * (STEPS == kLong ? min(s, K / TK - 1) : s);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ra[u][i] = *reinterpret_cast<const f32x4*>(a[i] + k);
            rb[u][i] = *reinterpret_cast<const f32x4*>(b[i] + k);
        }
    };
    auto multiply = [&](int u, f32x4 (&acc)[2][2]) {   // [weight block][activation block]
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(rb[u][i][e], ra[u][j][e], acc[i][j], 0, 0, 0);
    };
    if constexpr (STEPS > 0) {
#pragma unroll
        for (int u = 0; u < STEPS; ++u) issue(u, u);
        f32x4 old[2][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) load_old<EPI>(old[j], m0 + 16 * j + lr, n0, n1, c, C, ldc, M, N, vec);
        f32x4 sum[2][2] = {};
        multiply(0, sum);
#pragma unroll
        for (int u = 1; u < 4; ++u) {
            f32x4 acc[2][2] = {};
            if (u < STEPS) multiply(u < STEPS ? u : 0, acc);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) sum[i][j] += acc[i][j];
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            f32x4 v[2] = {sum[0][j], sum[1][j]};
            finish<EPI>(v, old[j], m0 + 16 * j + lr, n0, n1, t, c, C, ldc, M, N, vec, qo, D);
        }
    } else {
        __shared__ f32x4 red[4][4][64];
        const int steps = K / TK;
        const int n_mine = (steps - wave + 3) / 4;   // may be 0 where K < 64
        if constexpr (STEPS == kLong) {
#pragma unroll
            for (int u = 0; u < kDepth; ++u) issue(u, wave + 4 * u);
        } else {
#pragma unroll
            for (int u = 0; u < kDepth; ++u)
                if (u < n_mine) issue(u, wave + 4 * u);
        }
        f32x4 old[2];
        if (STEPS == kMid && wave < 2) load_old<EPI>(old, m0 + 16 * wave + lr, n0, n1, c, C, ldc, M, N, vec);
        f32x4 acc[2][2] = {};
        for (int s0 = 0; s0 < n_mine; s0 += kDepth) {
#pragma unroll
            for (int u = 0; u < kDepth; ++u) {
                if (s0 + u < n_mine) multiply(u, acc);
                if (s0 + u + kDepth < n_mine) issue(u, wave + 4 * (s0 + u + kDepth));
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) red[wave][2 * i + j][lane] = acc[i][j];
        __syncthreads();
        // wavefront w < 2 finishes activation block w
        if (wave >= 2) return;
        f32x4 v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            v[i] = red[0][2 * i + wave][lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) v[i] += red[w][2 * i + wave][lane];
        }
        if constexpr (STEPS == kLong) load_old<EPI>(old, m0 + 16 * wave + lr, n0, n1, c, C, ldc, M, N, vec);
        finish<EPI>(v, old, m0 + 16 * wave + lr, n0, n1, t, c, C, ldc, M, N, vec, qo, D);
    }
}

template <int EPI>
void launch(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int M, int N, int K,
            const ppk::QkvOut& qo, int D, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    const int64_t tiles = int64_t((N + TB - 1) / TB) * ((M + TB - 1) / TB);
    const int vec = ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    // A wavefront per tile past four workgroups' worth of tiles on every CU (us, a workgroup per tile and a
    // wavefront: 288 tiles, K 64: 6.2 and 7.0; 1024 tiles: 7.6 and 7.7; 2048: 10.8 and 10.1; 16384, K 16: 31
    // and 20)
    const int steps = K / TK;
    const unsigned one = static_cast<unsigned>(tiles);
    const unsigned four = static_cast<unsigned>(int64_t((N + 2 * TB - 1) / (2 * TB)) * ((M + 2 * TB - 1) / (2 * TB)));
#define PP_LAUNCH(STEPS, BLOCKS) \
    gemm_f32_kernel<EPI, STEPS><<<BLOCKS, NT, 0, s>>>(A, lda, B, ldb, C, ldc, M, N, K, vec, qo, D)
    switch (steps >= 4 * kDepth ? kLong : steps <= 4 && tiles > 1024 ? steps : kMid) {
        case 1: PP_LAUNCH(1, four); break;
        case 2: PP_LAUNCH(2, four); break;
        case 3: PP_LAUNCH(3, four); break;
        case 4: PP_LAUNCH(4, four); break;
        case kMid: PP_LAUNCH(kMid, one); break;
        default: PP_LAUNCH(kLong, one); break;
    }
#undef PP_LAUNCH
}

}  // namespace

namespace ppk {

void gemm_f32(int epi, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int M,
              int N, int K, hipStream_t s) {
    const QkvOut none{};
    switch (epi) {
        case kResidual: return launch<kResidual>(A, lda, B, ldb, C, ldc, M, N, K, none, 0, s);
        case kSwiGLU: return launch<kSwiGLU>(A, lda, B, ldb, C, ldc, M, N, K, none, 0, s);
        default: return launch<kStore>(A, lda, B, ldb, C, ldc, M, N, K, none, 0, s);
    }
}

void qkv_rope_f32(const float* A, int64_t lda, const float* B, int64_t ldb, int M, int K, int D, const QkvOut& out,
                  hipStream_t s) {
    launch<kQkvRope>(A, lda, B, ldb, nullptr, 0, M, (out.H + 2 * out.Hkv) * D, K, out, D, s);
}

}  // namespace ppk
