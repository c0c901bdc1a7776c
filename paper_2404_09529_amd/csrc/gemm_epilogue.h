// Element-wise arithmetic of the projection GEMMs' epilogues, shared by the kernels of every
// tile size so that a result does not depend on which of them computed it (the packed and the
// padded layout of a batch take different ones and agree bit for bit).
#pragma once
#include "argmax.h"
#include "device.h"
#include "kernels.h"

// The epilogue of one wavefront's NB x MB blocks, stored straight from the registers.  In block
// (i, j) lane l holds activation row mb + 16 j + l % 16 and 4 consecutive weight rows of block i,
// 4 (l / 16) + 0..3.  The wavefront is the wn-th along N of a tile whose first weight row is n0;
// its weight rows are n0 + 16 NB wn + 16 i + .., except for QKV with fewer than 128 rows per
// wavefront: blocks 0 .. NB / 2 - 1 are then dims wn 8 NB + 16 i + .. from n0 of a head and
// blocks NB / 2 .. their rotate-half partners, 64 dims further.
template <int EPI, int NB, int MB>
__device__ __forceinline__ void epilogue_direct(f32x4 (&acc)[NB][MB], void* __restrict__ Cv, int64_t ldc, int M, int mb,
                                                int n0, int wn, int lane, const ppk::QkvOut& qo) {
    const int lr = lane & 15, g = lane >> 4;
    const int nb0 = n0 + wn * 16 * NB;
    // block row j's accumulators leave the accumulation registers here, one block row at a time
    // (all at once they would need as many vector registers)
    auto take = [&](int j, f32x4 (&c)[NB]) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if constexpr (NB * MB >= 16) asm volatile("" : "+a"(acc[i][j]) : : "memory");
            c[i] = acc[i][j];
        }
    };
    if constexpr (EPI == ppk::kPartial) {
        float* C = static_cast<float*>(Cv) + nb0 + 4 * g;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int m = mb + 16 * j + lr;
            f32x4 a[NB];
            take(j, a);
            if (m < M) {
#pragma unroll
                for (int i = 0; i < NB; ++i) *reinterpret_cast<f32x4*>(C + int64_t(m) * ldc + 16 * i) = a[i];
            }
        }
    } else if constexpr (EPI == ppk::kResidual) {
        float* C = static_cast<float*>(Cv) + nb0 + 4 * g;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int m = mb + 16 * j + lr;
            float* row = C + int64_t(min(m, M - 1)) * ldc;
            f32x4 c[NB], a[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) c[i] = *reinterpret_cast<const f32x4*>(row + 16 * i);
            take(j, a);
            if (m < M) {
#pragma unroll
                for (int i = 0; i < NB; ++i) *reinterpret_cast<f32x4*>(row + 16 * i) = a[i] + c[i];
            }
        }
    } else if constexpr (EPI == ppk::kQkvRope) {
        constexpr int NH = NB / 2;
        const int head = n0 >> 7;                   // of the tile; a wavefront of 128 rows is one head
        const int hw = 16 * NB >= 128 ? head + wn : head;
        const int dim0 = 16 * NB >= 128 ? 0 : (n0 & 127) + wn * 16 * NH;
        const int kind = hw < qo.H ? 0 : (hw < qo.H + qo.Hkv ? 1 : 2);   // q, k, v
        bf16* base = kind == 0 ? static_cast<bf16*>(qo.q) + hw * 128
                               : static_cast<bf16*>(kind == 1 ? qo.kc : qo.vc) +
                                     (hw - qo.H - (kind == 2 ? qo.Hkv : 0)) * 128;
        const int64_t ld = kind == 0 ? qo.ldq : qo.ldkv;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int m = mb + 16 * j + lr, mc = min(m, M - 1);
            const int kv = kind > 0 ? qo.slot_kv[mc] : m;
            const int dst = m < M ? kv : -1;
            f32x4 a[NB];
            take(j, a);
            const float2* cs = qo.table + int64_t(qo.slot_pos[mc]) * 64 + dim0 + 4 * g;
#pragma unroll
            for (int i = 0; i < NH; ++i) {
                bf16x4 lo, hi;
                if (kind < 2) {
                    const f32x4 t0 = *reinterpret_cast<const f32x4*>(cs + 16 * i);
                    const f32x4 t1 = *reinterpret_cast<const f32x4*>(cs + 16 * i + 2);
                    const float cv[4] = {t0[0], t0[2], t1[0], t1[2]};
                    const float sv[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = a[i][e], y = a[i + NH][e];
                        lo[e] = static_cast<bf16>(rope_lo(x, y, cv[e], sv[e]));
                        hi[e] = static_cast<bf16>(rope_hi(x, y, cv[e], sv[e]));
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        lo[e] = static_cast<bf16>(a[i][e]);
                        hi[e] = static_cast<bf16>(a[i + NH][e]);
                    }
                }
                if (dst >= 0) {
                    bf16* p = base + int64_t(dst) * ld + dim0 + 16 * i + 4 * g;
                    *reinterpret_cast<bf16x4*>(p) = lo;
                    *reinterpret_cast<bf16x4*>(p + 64) = hi;
                }
            }
        }
    } else {
        bf16* C = static_cast<bf16*>(Cv) + (EPI == ppk::kSwiGLU ? nb0 / 2 : nb0) + 4 * g;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int m = mb + 16 * j + lr;
            f32x4 a[NB];
            take(j, a);
            if (m >= M) continue;
            bf16* row = C + int64_t(m) * ldc;
            if constexpr (EPI == ppk::kSwiGLU) {   // block 2 k: 16 gate rows, 2 k + 1: the matching up rows
#pragma unroll
                for (int k = 0; k < NB / 2; ++k) {
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = static_cast<bf16>(silu_rcp(a[2 * k][e]) * a[2 * k + 1][e]);
                    *reinterpret_cast<bf16x4*>(row + 16 * k) = v;
                }
            } else {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = static_cast<bf16>(a[i][e]);
                    *reinterpret_cast<bf16x4*>(row + 16 * i) = v;
                }
            }
        }
    }
}

// kLogits: the wavefront's columns are one block of 128 vocabulary rows (NB = 8); rows past the
// vocabulary V are not reported.
struct LogitsOut {
    float* logits;   // [k, V] or null
    ArgMax* part;    // [k, n_blocks]
    int V, n_blocks;
    int vec;         // every row of logits is 16-byte aligned
};
template <int MB>
__device__ __forceinline__ void epilogue_logits(f32x4 (&acc)[8][MB], int k, int mb, int n0, int lane,
                                                const LogitsOut& lo) {
    const int lr = lane & 15, g = lane >> 4;
    if (n0 >= lo.V) return;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int m = mb + 16 * j + lr;
        f32x4 a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            asm volatile("" : "+a"(acc[i][j]) : : "memory");
            a[i] = acc[i][j];
        }
        float bv = -INFINITY;
        int bi = INT32_MAX;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int n = n0 + 16 * i + 4 * g;
            if (lo.logits && lo.vec && m < k && n < lo.V)
                *reinterpret_cast<f32x4*>(lo.logits + int64_t(m) * lo.V + n) = a[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (n + e >= lo.V) continue;
                if (lo.logits && !lo.vec && m < k) lo.logits[int64_t(m) * lo.V + n + e] = a[i][e];
                if (better(a[i][e], n + e, bv, bi)) { bv = a[i][e]; bi = n + e; }
            }
        }
        // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same prompt
#pragma unroll
        for (int x = 16; x < 64; x <<= 1) {
            const float ov = __shfl_xor(bv, x);
            const int oi = __shfl_xor(bi, x);
            if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if (g == 0 && m < k) lo.part[int64_t(m) * lo.n_blocks + n0 / 128] = ArgMax{bv, bi};
    }
}
