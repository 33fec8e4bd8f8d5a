// gfx950 kernels of the many-row passes: prefill blocks (row embedding, GEMMs, causal attention) and
// the drafter update's logits GEMM.
//
// Every output of a prefill block has its arithmetic fixed by the matrix and the row alone: a GEMM output
// accumulates its K chunks in increasing order, one MFMA per chunk, whatever tile, wave or launch shape
// it sits in, and a query row's softmax runs over its 64-key chunks in increasing order.  A prompt's
// keys, values and logits therefore do not depend on its batch, on how its rows are cut into blocks or
// on the launch shape chosen for them.  The update's logits (EPI_LOGITS) make no such promise: where few
// rows or few tiles select it, K is summed in parts (kUpdateParts), elsewhere in one chain, so a replay
// row's last bits depend on how many rows the ring holds and on the number of compute units.
#include "kernels.h"

#include <hip/hip_ext.h>

#include <algorithm>

#include "device.h"
#include "ring.h"

// Multiplies and adds fuse only where fmaf is written: otherwise the compiler picks which product of
// a sum to fuse separately in every launch shape's instance, and a row would differ in its last bit.
#pragma clang fp contract(off)

namespace dvi {

namespace {

// Wait until at most VM vector-memory operations of this wave are in flight and (LGKM0) every LDS
// read has returned.  gfx9 s_waitcnt immediate: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8.
template <int VM, bool LGKM0>
__device__ __forceinline__ void wait_mem() {
    static_assert(VM >= 0 && VM < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (0x7 << 4) | ((LGKM0 ? 0x0 : 0xf) << 8));
}
__device__ __forceinline__ void barrier() {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ float sumsq4(float a, float b, float c, float d) {
    return fmaf(d, d, fmaf(c, c, fmaf(b, b, a * a)));
}

// ------------------------------------------------------------------------------------------
// Rows of a prefill block
// ------------------------------------------------------------------------------------------
// Row m of the block is row t0 + m of the prompts laid end to end: sequence b with starts[b] <= t <
// starts[b + 1], position t - starts[b].  rowmap[m] = (b, position); h = E[token] (fp32), its partial
// sums of squares per 16 columns, and hg = dtype(h * g) (FM) for the first layer's folded RMSNorm.
// Bound by the stores (h and hg, 6 bytes per element in bf16): every thread holds EPL consecutive columns,
// so loads and stores are 16 bytes wide (2048 rows of the 7B shape: 60 us with 2-byte accesses).
template <DType T>
__global__ void __launch_bounds__(256) embed_rows_kernel(const void *emb, const int32_t *ids, const int32_t *starts,
                                                         int B, int t0, int d, float *h, float *ss, void *hg,
                                                         const float *g, int2 *rowmap) {
    typedef typename St<T>::type E;
    constexpr int EPL = 16 / (int)sizeof(E);
    const int m = blockIdx.x, t = t0 + m;
    int b = 0;
    while (b + 1 < B && starts[b + 1] <= t) ++b;  // uniform
    if (threadIdx.x == 0) rowmap[m] = make_int2(b, t - starts[b]);
    const uint4 *row = (const uint4 *)((const E *)emb + (size_t)ids[t] * d);
    for (int q = threadIdx.x; q < d / EPL; q += 256) {
        const uint4 raw = row[q];
        float v[EPL];
        unpack_frag<T>(raw, v);
        float s = 0.f;
        float gv[EPL];
#pragma unroll
        for (int e = 0; e < EPL; e += 4) {
            *(float4 *)(h + (size_t)m * d + q * EPL + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
            const float4 g4 = *(const float4 *)(g + q * EPL + e);
            gv[e] = v[e] * g4.x;
            gv[e + 1] = v[e + 1] * g4.y;
            gv[e + 2] = v[e + 2] * g4.z;
            gv[e + 3] = v[e + 3] * g4.w;
            s += sumsq4(v[e], v[e + 1], v[e + 2], v[e + 3]);
        }
        *(uint4 *)((E *)hg + fm_index<T>(m, q * EPL, d)) = pack_frag_cvt<T>(gv);
        // 16 columns are 16 / EPL neighbouring threads, in one wave (d is a multiple of 16)
#pragma unroll
        for (int o = 1; o < 16 / EPL; o <<= 1) s += __shfl_xor(s, o);
        if (q % (16 / EPL) == 0) ss[(size_t)m * (d / 16) + q * EPL / 16] = s;
    }
}

// Each sequence's last prompt row of a block (its folded-norm input and partial sums of squares) to
// row b of compact buffers.  Workgroup b.
template <DType T>
__global__ void __launch_bounds__(256) gather_last_kernel(const void *hg, const float *ss, int d, int nps, LastRows lr,
                                                          void *dst, float *ss_dst) {
    typedef typename St<T>::type E;
    constexpr int EPL = 16 / (int)sizeof(E);
    const int b = blockIdx.x, r = lr.src[b];
    if (r < 0) return;  // uniform across the workgroup
    for (int k = threadIdx.x * EPL; k < d; k += 256 * EPL)
        *(uint4 *)((E *)dst + fm_index<T>(b, k, d)) = *(const uint4 *)((const E *)hg + fm_index<T>(r, k, d));
    for (int k = threadIdx.x; k < nps; k += 256) ss_dst[(size_t)b * nps + k] = ss[(size_t)r * nps + k];
}

// ------------------------------------------------------------------------------------------
// 1/rms of a token from its partial sums of squares, by the four lanes l, l ^ 16, l ^ 32, l ^ 48 (l =
// token % 16): lane quarter q adds the groups of four partials q, q + 4, ... in order, and the
// quarters are added as (0 + 1) + (2 + 3).  One code path for every launch shape, so every GEMM of a
// row scales it by the same value.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float token_inv_rms(const float *ss, int nparts, int d, float eps, int q) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (nparts % 4 == 0) {  // uniform; rows are then 16-byte aligned
#pragma unroll 8
        for (int i = 4 * q; i < nparts; i += 16) {
            const float4 v = *(const float4 *)(ss + i);
            s0 += v.x;
            s1 += v.y;
            s2 += v.z;
            s3 += v.w;
        }
    } else {
        for (int i = 4 * q; i < nparts; i += 16) {
            s0 += ss[i];
            if (i + 1 < nparts) s1 += ss[i + 1];
            if (i + 2 < nparts) s2 += ss[i + 2];
            if (i + 3 < nparts) s3 += ss[i + 3];
        }
    }
    return 1.0f / sqrtf(quad_rows_sum((s0 + s1) + (s2 + s3)) / (float)d + eps);
}

// 16 tokens per wave.
__global__ void __launch_bounds__(64) rms_rows_kernel(const float *ss, int ld_ss, int nparts, int K, float eps, int M,
                                                      float *out) {
    const int lane = threadIdx.x, m = blockIdx.x * 16 + (lane & 15);
    const float v = token_inv_rms(ss + (size_t)min(m, M - 1) * ld_ss, nparts, K, eps, lane >> 4);
    if (lane < 16 && m < M) out[m] = v;
}

// ------------------------------------------------------------------------------------------
// Epilogues.  A wave holds tiles t0 .. t0 + RT - 1 (16 features each) of token groups g0 .. g0 + XG - 1
// in the MFMA output layout: acc[t][g][j] is feature 16 (t0 + t) + 4 (l / 16) + j of token 16 (g0 + g)
// + l % 16.  The same operations per output as the decode GEMM's epilogue; the operands of the next
// token group are requested while one is computed, and every store is as wide as a lane's values lie
// together: 16, 8 or 4 bytes, but one element in the value cache, which runs along the tokens (8 x 2048
// prefill, 7B: the K = 4096 GEMMs spent 24-48 us per tile round in per-element epilogues).
// sc[g]: 1/rms of the lane's token.
// ------------------------------------------------------------------------------------------
template <DType T, int N>
__device__ __forceinline__ void store_n(typename St<T>::type *p, const float (&v)[N]) {
    static_assert(N == 2 || N == 4, "width");
    if constexpr (T == DType::BF16) {
        if constexpr (N == 4)
            *(uint2 *)p = uint2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
        else
            *(uint32_t *)p = pack2bf(v[0], v[1]);
    } else {
        if constexpr (N == 4)
            *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
        else
            *(float2 *)p = make_float2(v[0], v[1]);
    }
}

template <DType T, int RT, int XG>
__device__ __forceinline__ void resid_epilogue(const GemmArgs &a, int t0, int g0, const f32x4 (&acc)[RT][XG]) {
    typedef typename St<T>::type E;
    const int lane = threadIdx.x & 63, l16 = lane & 15, G4 = lane >> 4, NT = a.N / 16;
    float4 hv[2][RT], gn[RT];
    auto load = [&](int g, float4 (&o)[RT]) {
        const float *hp = a.H + (size_t)min(16 * (g0 + g) + l16, a.M - 1) * a.ldh + 4 * G4;
#pragma unroll
        for (int t = 0; t < RT; ++t) o[t] = *(const float4 *)(hp + 16 * min(t0 + t, NT - 1));
    };
    load(0, hv[0]);
#pragma unroll
    for (int t = 0; t < RT; ++t) gn[t] = *(const float4 *)(a.g_next + 16 * min(t0 + t, NT - 1) + 4 * G4);
#pragma unroll
    for (int g = 0; g < XG; ++g) {
        if (g + 1 < XG) load(g + 1, hv[(g + 1) & 1]);
        const int m = 16 * (g0 + g) + l16;
        float *hp = a.H + (size_t)m * a.ldh + 4 * G4;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int nt = t0 + t;
            const float4 h4 = hv[g & 1][t];
            const float v[4] = {h4.x + acc[t][g][0], h4.y + acc[t][g][1], h4.z + acc[t][g][2], h4.w + acc[t][g][3]};
            const float s = quad_rows_sum(sumsq4(v[0], v[1], v[2], v[3]));
            if (m < a.M && nt < NT) {
                *(float4 *)(hp + 16 * nt) = make_float4(v[0], v[1], v[2], v[3]);
                if (G4 == 0) a.ss_out[(size_t)m * a.ld_ss_out + nt] = s;
                const float x[4] = {v[0] * gn[t].x, v[1] * gn[t].y, v[2] * gn[t].z, v[3] * gn[t].w};
                store_n<T, 4>((E *)a.hg_out + fm_index<T>(m * a.hg_rs + a.hg_off, nt * 16 + 4 * G4, a.N), x);
            }
        }
    }
}

template <DType T, int RT, int XG>
__device__ __forceinline__ void swiglu_epilogue(const GemmArgs &a, int t0, int g0, const f32x4 (&acc)[RT][XG],
                                                const float (&sc)[XG]) {
    typedef typename St<T>::type E;
    const int lane = threadIdx.x & 63, l16 = lane & 15, G4 = lane >> 4, NT = a.N / 16;
#pragma unroll
    for (int g = 0; g < XG; ++g) {
        const int m = 16 * (g0 + g) + l16;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int nt = t0 + t;
            float x[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const float gt = acc[t][g][2 * p] * sc[g], up = acc[t][g][2 * p + 1] * sc[g];
                x[p] = gt / (1.0f + expf(-gt)) * up;
            }
            if (m < a.M && nt < NT) store_n<T, 2>((E *)a.A + fm_index<T>(m, 8 * nt + 2 * G4, a.N / 2), x);
        }
    }
}

// The wave's tiles lie in one head (RT divides a head's hd / 16 tiles and t0).
template <DType T, int RT, int XG>
__device__ __forceinline__ void qkv_epilogue(const GemmArgs &a, int t0, int g0, const f32x4 (&acc)[RT][XG],
                                             const float (&sc)[XG]) {
    typedef typename St<T>::type E;
    const int lane = threadIdx.x & 63, l16 = lane & 15, G4 = lane >> 4;
    if (t0 >= a.N / 16) return;  // uniform; N / 16 is a multiple of RT
    const int tph = a.hd / 16, half = a.hd / 2, head = t0 / tph, tt = t0 - head * tph;
    const bool isq = head < a.n_heads, rot = head < a.n_heads + a.n_kv;
    const int kvh = head - a.n_heads - (rot ? 0 : a.n_kv);
    constexpr int kc = (T == DType::BF16) ? 32 : 16;
    int2 bp[XG];  // (sequence, position)
#pragma unroll
    for (int g = 0; g < XG; ++g) bp[g] = a.rowmap[min(16 * (g0 + g) + l16, a.M - 1)];
    if (rot) {
        float4 cs[2][RT];  // (cos, sin) of the lane's two pairs
        auto load = [&](int g, float4 (&o)[RT]) {
            const float4 *rp = (const float4 *)(a.rope + (size_t)bp[g].y * half + 8 * tt + 2 * G4);
#pragma unroll
            for (int t = 0; t < RT; ++t) o[t] = rp[4 * t];
        };
        load(0, cs[0]);
#pragma unroll
        for (int g = 0; g < XG; ++g) {
            if (g + 1 < XG) load(g + 1, cs[(g + 1) & 1]);
            const int m = 16 * (g0 + g) + l16, kk = bp[g].y % CK;
            float *q = a.Q + ((size_t)m * a.n_heads + head) * a.hd + 8 * tt + 2 * G4;
            E *kb = (E *)a.Kc + (((size_t)bp[g].x * a.n_kv + kvh) * a.s_max + (size_t)(bp[g].y - kk)) * a.hd;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const float4 c4 = cs[g & 1][t];
                const float c[2] = {c4.x, c4.z}, s[2] = {c4.y, c4.w};
                float lo[2], hi[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const float x0 = acc[t][g][2 * p] * sc[g], x1 = acc[t][g][2 * p + 1] * sc[g];
                    lo[p] = fmaf(x0, c[p], -(x1 * s[p]));
                    hi[p] = fmaf(x0, s[p], x1 * c[p]);
                }
                if (m >= a.M) continue;
                if (isq) {
                    *(float2 *)(q + 8 * t) = make_float2(lo[0], lo[1]);
                    *(float2 *)(q + 8 * t + half) = make_float2(hi[0], hi[1]);
                } else {
                    const int j = 8 * (tt + t) + 2 * G4;
                    store_n<T, 2>(kb + kv_key_offset(kc, a.hd, kk, j), lo);
                    store_n<T, 2>(kb + kv_key_offset(kc, a.hd, kk, j + half), hi);
                }
            }
        }
    } else {
#pragma unroll
        for (int g = 0; g < XG; ++g) {
            if (16 * (g0 + g) + l16 >= a.M) continue;
            const int kk = bp[g].y % CK;
            E *vb = (E *)a.Vc + (((size_t)bp[g].x * a.n_kv + kvh) * a.s_max + (size_t)(bp[g].y - kk)) * a.hd;
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int j = 8 * (tt + t) + 2 * G4 + p;
                    St<T>::store(vb, kv_val_offset(kc, a.hd, kk, j), acc[t][g][2 * p] * sc[g]);
                    St<T>::store(vb, kv_val_offset(kc, a.hd, kk, j + half), acc[t][g][2 * p + 1] * sc[g]);
                }
        }
    }
}

// Drafter-update logits: z = acc + gamma * A_s u.  The LoRA term is a product over the rank on fp32
// MFMAs in steps of 16 ranks (lane quarter q holds ranks 4 q .. 4 q + 3 of the step, one MFMA per e):
// one 16-byte load per tile and per token group instead of a gather per rank and output.  No argmax
// partials, no sampling (the update asks for neither).
__device__ __forceinline__ float4 rank_slice(const float *row, int c, int r) {
    if (r % 4 == 0) return c < r ? *(const float4 *)(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);  // r uniform
    return make_float4(c < r ? row[c] : 0.f, c + 1 < r ? row[c + 1] : 0.f, c + 2 < r ? row[c + 2] : 0.f,
                       c + 3 < r ? row[c + 3] : 0.f);
}

template <DType T, int RT, int XG>
__device__ __forceinline__ void logits_epilogue(const GemmArgs &a, int t0, int g0, const f32x4 (&acc)[RT][XG]) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, G4 = lane >> 4, NT = a.N / 16;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int nt = t0 + t;
        const float *Ar = a.lora_A + ((size_t)min(nt, NT - 1) * 16 + l16) * a.r;
        f32x4 s[XG];
#pragma unroll
        for (int g = 0; g < XG; ++g) s[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < a.r; c0 += 16) {
            const float4 av = rank_slice(Ar, c0 + 4 * G4, a.r);
#pragma unroll
            for (int g = 0; g < XG; ++g) {
                const float4 uv =
                    rank_slice(a.lora_u + (size_t)min(16 * (g0 + g) + l16, a.M - 1) * a.r, c0 + 4 * G4, a.r);
                s[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, uv.x, s[g], 0, 0, 0);
                s[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, uv.y, s[g], 0, 0, 0);
                s[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, uv.z, s[g], 0, 0, 0);
                s[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, uv.w, s[g], 0, 0, 0);
            }
        }
#pragma unroll
        for (int g = 0; g < XG; ++g) {
            const int m = 16 * (g0 + g) + l16;
            if (m < a.M && nt < NT)
                *(float4 *)(a.Z + (size_t)m * a.N + nt * 16 + 4 * G4) =
                    make_float4(fmaf(a.gamma, s[g][0], acc[t][g][0]), fmaf(a.gamma, s[g][1], acc[t][g][1]),
                                fmaf(a.gamma, s[g][2], acc[t][g][2]), fmaf(a.gamma, s[g][3], acc[t][g][3]));
        }
    }
}

template <DType T, int EPI, int RT, int XG>
__device__ __forceinline__ void rows_epilogue(const GemmArgs &a, int t0, int g0, const f32x4 (&acc)[RT][XG],
                                              const float (&sc)[XG]) {
    if constexpr (EPI == EPI_RESID) resid_epilogue<T, RT, XG>(a, t0, g0, acc);
    else if constexpr (EPI == EPI_SWIGLU) swiglu_epilogue<T, RT, XG>(a, t0, g0, acc, sc);
    else if constexpr (EPI == EPI_QKV) qkv_epilogue<T, RT, XG>(a, t0, g0, acc, sc);
    else logits_epilogue<T, RT, XG>(a, t0, g0, acc);
}

// ------------------------------------------------------------------------------------------
// Many-row GEMM.  Workgroup tile: 16 XG tokens x 16 RT WV features, WV waves; each wave owns RT
// feature tiles for all the tile's tokens.  A wave's weight fragments are its own, so they go from
// memory straight into its registers (WD chunks in flight); the token fragments, which all waves
// need, go through an LDS ring of NS stages of CPS chunks by direct-to-LDS copies, one barrier per
// stage.  Staging both operands in LDS, as the kernel before did, needed 172 bytes of LDS traffic per
// clock at full MFMA rate against the 128 it has; this split needs 80.
// 128 x 256 tiles of four waves, four feature tiles each (128 accumulators, 236 registers), leave room
// for two workgroups on a compute unit, so one's epilogue runs under the other's MFMAs; each fragment
// read from LDS feeds four MFMAs.  With PIPE the fragments of the next chunk are read before the
// products of the current one, across the stage barrier too: read two at a time just before their use,
// as the compiler places them, every pair stalled both waves of a SIMD for the LDS latency.  7B shapes,
// 8192 rows, in sequence and so at the clock this load settles at: gate/up 1212 -> 1189 us, QKV 778 ->
// 741, out-proj and down 985 -> 929 against eight waves of two feature tiles without PIPE; 512 rows: QKV
// 78 -> 73, out-proj and down 128 -> 117.  256 x 256 tiles (1254, 769, 968 us) and more bytes in flight
// change little.  Gate/up takes 1211 us with expf and a division in its epilogue, 1220 TFLOP/s (the
// library's 8192 cubed product reaches 1470).
// Workgroups are numbered so that each XCD (workgroup id mod 8) takes a contiguous range of tiles,
// in strips of kStrip feature blocks with the token tile major: the tiles that run together on an
// XCD form a near-square, which reads the fewest bytes into its L2 (gate/up, 8192 rows: 1167 ->
// 1238 TFLOP/s against feature block major).
// ------------------------------------------------------------------------------------------
constexpr int kStrip = 8;

// The update's logits of up to 64 rows, and of any rows in gemm_few_kernel, are sums over K in four
// interleaved parts (chunk mod 4); every block of chunks the parts are added as a tree and the block's
// sum to the total, so that no chain of additions is longer than 8 chunks of a part (the ring) or 6
// (gemm_few_kernel).  The decode GEMM, which had these shapes before, splits K over its waves, in chains
// of 16 chunks at K = 4096; four parts over all of K were chains of 32, and A_s after an update of 16 rows
// was 15% further from 64 bits (1.30e-6 -> 1.50e-6).
// Where one token tile covers the rows, these launches read every weight once, non-temporally, as the
// decode GEMM does: between two updates the decode steps have streamed gigabytes, and ordinary loads of a
// head that is not in the last-level cache cost 20 to 50 us more and leave nothing of the ring's rows
// there.  An update at V = 32000, d = 4096 with cold caches: 8 rows 212 -> 170 us (172 with the decode
// GEMM), 48 rows 219 -> 179 (225); with the head still cached from the update before 159 -> 161 and 169 ->
// 172.
constexpr int kUpdateParts = 4;
constexpr int kRingBlock = 4;  // turns of the ring's weight registers per block (8 chunks each)
template <int N, int RT, int XG>
__device__ __forceinline__ void zero_parts(f32x4 (&acc)[N][RT][XG]) {
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int g = 0; g < XG; ++g) acc[q][t][g] = (f32x4){0.f, 0.f, 0.f, 0.f};
}
template <int N, int RT, int XG>
__device__ __forceinline__ void fold_parts(f32x4 (&acc)[N][RT][XG], f32x4 (&sum)[1][RT][XG]) {
    static_assert(N == 4, "parts");
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int g = 0; g < XG; ++g)
            sum[0][t][g] = sum[0][t][g] + ((acc[0][t][g] + acc[1][t][g]) + (acc[2][t][g] + acc[3][t][g]));
    zero_parts(acc);
}

// CPS chunks per stage, NS stages of the ring, WD chunks of weights in flight.
template <DType T, int EPI, int WV, int RT, int XG, int CPS, int NS, int WD, int MINW, bool PIPE, int NACC>
__global__ void __launch_bounds__(64 * WV, MINW) gemm_rows_kernel(GemmArgs a, int tok_tiles, int blocks, int total) {
    constexpr int PX = CPS * XG / WV;        // copies per wave and stage
    constexpr int UN = WD > CPS ? WD / CPS : 1;  // stages per turn of the weight ring
    static_assert(PX * WV == CPS * XG && UN * CPS == WD && WD % NACC == 0 && (!PIPE || (WD % 2 == 0 && NACC == 1)), "stage and ring shapes");
    __shared__ __align__(1024) uint4 ring[NS][CPS * XG][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KT = a.K / ((T == DType::BF16) ? 32 : 16), NT = a.N / 16, NG = (a.M + 15) / 16;
    const int per = (total + 7) / 8, j = blockIdx.x >> 3, tl = (blockIdx.x & 7) * per + j;
    if (j >= per || tl >= total) return;  // uniform across the workgroup (before any barrier)
    const int strip = tl / (kStrip * tok_tiles), r = tl - strip * kStrip * tok_tiles;
    const int width = min(kStrip, blocks - strip * kStrip), ti = r / width;
    const int g0 = ti * XG, t0 = (strip * kStrip + r - ti * width) * (RT * WV) + wave * RT;
    // the copies of this wave: fragment f = wave * PX + i of a stage is chunk f / XG, token group f % XG;
    // groups, tiles and chunks past the end repeat the last one (never stored, or never multiplied)
    const uint8_t *xsrc[PX];
    int xchunk[PX];
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        const int f = wave * PX + i;
        xchunk[i] = f / XG;
        xsrc[i] = (const uint8_t *)a.X + (size_t)min(g0 + f % XG, NG - 1) * KT * 1024;
    }
    const uint32_t ring0 = lds_addr(&ring[0][0][0]), lane16 = 16 * lane;
    auto copy_stage = [&](int st, int s) {
#pragma unroll
        for (int i = 0; i < PX; ++i)
            copy_1k(ring0 + (uint32_t)(st * (CPS * XG) + wave * PX + i) * 1024, lane16,
                    xsrc[i] + (size_t)min(s * CPS + xchunk[i], KT - 1) * 1024);
    };
    const uint4 *wsrc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) wsrc[t] = (const uint4 *)a.W + (size_t)min(t0 + t, NT - 1) * KT * 64;
    uint4 w[WD][RT];
    auto load_w = [&](int k, uint4 (&wf)[RT]) {
        const size_t o = (size_t)min(k, KT - 1) * 64;
#pragma unroll
        for (int t = 0; t < RT; ++t) wf[t] = NACC > 1 ? ld_stream(wsrc[t] + o + lane) : (wsrc[t] + o)[lane];
    };
    f32x4 acc[NACC][RT][XG], sum[1][RT][XG];
    zero_parts(acc);
    if constexpr (NACC > 1) zero_parts(sum);
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) copy_stage(st, st);
#pragma unroll
    for (int k = 0; k < WD; ++k) load_w(k, w[k]);
    constexpr int kYoung = ring_wait_count(CPS, NS, WD, RT, PX, PIPE);
    const int KS = KT / CPS;  // KT is a multiple of CPS
    if constexpr (PIPE) {
        auto read_x = [&](int st, int c, uint4 (&xf)[XG]) {
#pragma unroll
            for (int g = 0; g < XG; ++g) xf[g] = ring[st][c * XG + g][lane];
        };
        uint4 x[2][XG];  // token fragments: the chunk being multiplied and the one after it
        int st = 0;
        wait_mem<kYoung, true>();
        barrier();
        copy_stage(NS - 1, NS - 1);
        read_x(0, 0, x[0]);
        for (int s0 = 0; s0 < KS; s0 += UN) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int s = s0 + u;
                if (UN > 1 && s >= KS) break;  // uniform
#pragma unroll
                for (int c = 0; c < CPS; ++c) {
                    const int q = u * CPS + c;
                    if (c + 1 < CPS) {
                        read_x(st, c + 1, x[(q + 1) & 1]);
                    } else {
                        // this wave's copies of stage s + 1 have landed and its reads of stage s have
                        // returned; past the barrier that holds for every wave, so stage s + 1 can be read
                        // and the slot of stage s overwritten (stages past the end repeat the last chunk
                        // and are not multiplied)
                        const int next = st + 1 == NS ? 0 : st + 1;
                        wait_mem<kYoung, true>();
                        barrier();
                        copy_stage(st, s + NS);
                        read_x(next, 0, x[(q + 1) & 1]);
                        st = next;
                    }
                    __builtin_amdgcn_sched_barrier(0);  // the reads above go out before these products
                    uint4(&wf)[RT] = w[q % WD];
#pragma unroll
                    for (int g = 0; g < XG; ++g)
#pragma unroll
                        for (int t = 0; t < RT; ++t) {
                            f32x4 &o = acc[q % NACC][t][g];
                            o = St<T>::mma(wf[t], x[q & 1][g], o);
                        }
                    load_w(s * CPS + c + WD, wf);
                }
            }
        }
    } else {
        int st = 0;
        for (int s0 = 0; s0 < KS; s0 += UN) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int s = s0 + u;
                if (UN > 1 && s >= KS) break;  // uniform
                // this wave's copies of stage s have landed and its reads of stage s - 1 have returned;
                // past the barrier that holds for every wave, so stage s can be read and the slot of
                // stage s - 1 overwritten
                wait_mem<kYoung, true>();
                barrier();
                copy_stage(st == 0 ? NS - 1 : st - 1, s + NS - 1);
                const uint4 *b = &ring[st][0][lane];
#pragma unroll
                for (int c = 0; c < CPS; ++c) {
                    uint4(&wf)[RT] = w[(u * CPS + c) % WD];
#pragma unroll
                    for (int g = 0; g < XG; ++g) {
                        const uint4 xf = b[(c * XG + g) * 64];
#pragma unroll
                        for (int t = 0; t < RT; ++t) {
                            f32x4 &o = acc[(u * CPS + c) % NACC][t][g];
                            o = St<T>::mma(wf[t], xf, o);
                        }
                    }
                    load_w(s * CPS + c + WD, wf);
                }
                st = st + 1 == NS ? 0 : st + 1;
            }
            if constexpr (NACC > 1)
                if (s0 / UN % kRingBlock == kRingBlock - 1) fold_parts(acc, sum);  // uniform
        }
    }
    wait_mem<0, true>();  // no copy may land after the workgroup has given its LDS back
    float sc[XG];
#pragma unroll
    for (int g = 0; g < XG; ++g)
        sc[g] = a.ss_in != nullptr ? a.sinv_rows[min(16 * (g0 + g) + (lane & 15), a.M - 1)] : 1.0f;
    if constexpr (NACC > 1) {
        fold_parts(acc, sum);
        rows_epilogue<T, EPI, RT, XG>(a, t0, g0, sum[0], sc);
    } else {
        rows_epilogue<T, EPI, RT, XG>(a, t0, g0, acc[0], sc);
    }
}

// Few rows, or few tiles: one wave per feature tile and XG token groups, both operands straight into
// registers through rings of SW weight and SX token chunks.  Nothing is shared between waves, so the
// wave's serial chain of MFMAs (one per chunk and group) never waits for a barrier.  Bound by what
// one compute unit can stream (about 50 GB/s of cold lines).  1/rms of the tokens is computed here,
// under the operand stream.  1B shapes, 37 rows, against the LDS-staged kernel before (16 workgroups
// for 2048 features): out-proj 38 -> 8 us, down 120 -> 17, QKV 41 -> 9.
template <DType T, int EPI, int XG, int SW, int SX, bool ONCE>
__global__ void __launch_bounds__(64) gemm_few_kernel(GemmArgs a, int gb) {
    static_assert(SW % SX == 0, "ring depths");
    const int lane = threadIdx.x;
    const int KT = a.K / ((T == DType::BF16) ? 32 : 16), NG = (a.M + 15) / 16;
    // the gb waves of a tile sit on one XCD (workgroup id mod 8) and share its weights there
    const int i = blockIdx.x >> 3, nt = i / gb * 8 + (blockIdx.x & 7), g0 = (i % gb) * XG;
    if (nt >= a.N / 16) return;
    const uint4 *wsrc = (const uint4 *)a.W + (size_t)nt * KT * 64, *xsrc[XG];
#pragma unroll
    for (int g = 0; g < XG; ++g) xsrc[g] = (const uint4 *)a.X + (size_t)min(g0 + g, NG - 1) * KT * 64;
    uint4 w[SW], x[SX][XG];
    auto load_w = [&](int k, uint4 &wf) {
        const uint4 *p = wsrc + (size_t)min(k, KT - 1) * 64 + lane;
        wf = ONCE ? ld_stream(p) : *p;
    };
    auto load_x = [&](int k, uint4 (&xf)[XG]) {
#pragma unroll
        for (int g = 0; g < XG; ++g) xf[g] = (xsrc[g] + (size_t)min(k, KT - 1) * 64)[lane];
    };
    constexpr int kAcc = EPI == EPI_LOGITS ? kUpdateParts : 1;
    static_assert(SW % kAcc == 0, "parts of a turn");
    f32x4 acc[kAcc][1][XG], sum[1][1][XG];
    zero_parts(acc);
    if constexpr (kAcc > 1) zero_parts(sum);
#pragma unroll
    for (int k = 0; k < SW; ++k) load_w(k, w[k]);
#pragma unroll
    for (int k = 0; k < SX; ++k) load_x(k, x[k]);
    float sc[XG];
#pragma unroll
    for (int g = 0; g < XG; ++g)
        sc[g] = a.ss_in != nullptr ? token_inv_rms(a.ss_in + (size_t)min(16 * (g0 + g) + (lane & 15), a.M - 1) * a.ld_ss_in,
                                                   a.K / 16, a.K, a.eps, lane >> 4)
                                   : 1.0f;
    int k = 0;
    for (; k + SW <= KT; k += SW) {
#pragma unroll
        for (int i = 0; i < SW; ++i) {
#pragma unroll
            for (int g = 0; g < XG; ++g) acc[i % kAcc][0][g] = St<T>::mma(w[i], x[i % SX][g], acc[i % kAcc][0][g]);
            load_w(k + SW + i, w[i]);
            load_x(k + SX + i, x[i % SX]);
        }
        if constexpr (kAcc > 1) fold_parts(acc, sum);
    }
#pragma unroll
    for (int i = 0; i < SW; ++i)
        if (k + i < KT) {  // uniform
#pragma unroll
            for (int g = 0; g < XG; ++g) acc[i % kAcc][0][g] = St<T>::mma(w[i], x[i % SX][g], acc[i % kAcc][0][g]);
            load_x(k + SX + i, x[i % SX]);
        }
    if constexpr (kAcc > 1) {
        fold_parts(acc, sum);
        rows_epilogue<T, EPI, 1, XG>(a, nt, g0, sum[0], sc);
    } else {
        rows_epilogue<T, EPI, 1, XG>(a, nt, g0, acc[0], sc);
    }
}

template <typename... P, typename... Q>
void launch_ev(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t s, const LaunchEvents &ev, const Q &...args) {
    if (ev.start || ev.stop)
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev.start, ev.stop, 0, args...);
    else
        kernel<<<grid, block, 0, s>>>(args...);
}

template <DType T, int EPI, int WV, int RT, int XG, int CPS, int NS, int WD, int MINW, bool PIPE, int NACC = 1>
void launch_rows(const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    const int tok = (a.M + 16 * XG - 1) / (16 * XG), blk = (a.N / 16 + RT * WV - 1) / (RT * WV), total = tok * blk;
    if (a.ss_in != nullptr)
        rms_rows_kernel<<<(a.M + 15) / 16, 64, 0, s>>>(a.ss_in, a.ld_ss_in, a.K / 16, a.K, a.eps, a.M, a.sinv_rows);
    launch_ev(gemm_rows_kernel<T, EPI, WV, RT, XG, CPS, NS, WD, MINW, PIPE, NACC>, dim3(8 * ((total + 7) / 8)), dim3(64 * WV),
              s, ev, a, tok, blk, total);
}

template <DType T, int EPI, int XG, int SW, int SX, bool ONCE = false>
void launch_few(const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    const int NT = a.N / 16, gb = ((a.M + 15) / 16 + XG - 1) / XG;
    launch_ev(gemm_few_kernel<T, EPI, XG, SW, SX, ONCE>, dim3((NT + 7) / 8 * 8 * gb), dim3(64), s, ev, a, gb);
}

// Launch shape (times: weights cold, as inside a model).
// One token group: a wave per tile.  Up to 64 rows of a wide matrix: 64 x 64 tiles (7B gate/up at 37
// rows 44 us, a wave per tile 59; QKV 31 against 34).  Up to 64 rows of a narrow one: a wave per tile
// and as many token groups as still put a wave on every compute unit, for a wave streams at most what
// one compute unit can (1B down at 37 rows: 22 us as 128 waves, 17 us as 256, 45 us as 64 x 64 tiles).
// Beyond, the largest tile that gives three quarters of the compute units a workgroup: a smaller tile
// reads more bytes per product, but idle compute units cost more (7B out-proj at 512 rows: 78 us as 64
// workgroups of 128 x 256, 34 us as 256 of 64 x 128; gate/up there 104 us as 344 of 128 x 256, 110 us
// as 688 of 128 x 128).  A grid of at most one workgroup per compute unit takes the whole unit: deeper
// rings, 256 registers (out-proj at 2048 rows 82 -> 72 us, QKV at 512 rows 84 -> 73 us; with two
// workgroups per unit that costs 20%: gate/up 104 -> 123 us).  PIPE where its second set of fragments
// fits and was the faster: eight waves of one feature tile keep the plain loop (1024 rows, 7B: 2104 us a
// prefill of four layers, 2168 as four piped waves of two tiles; 200 rows 1043 against 1188), as do the
// 64 x 64 tiles (1B, 37 rows: 1111 against 1144 us).  When not even 64 x 64 tiles fill the
// chip, a wave per tile and four groups again (1B down at 200 rows 45 -> 38 us).  A K of an odd number
// of chunks takes one-chunk stages.
template <DType T, int EPI>
void gemm_rows_t(const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    const int NT = a.N / 16, KT = a.K / pack_kc(T), NG = (a.M + 15) / 16, cu = compute_units();
    constexpr int NACC = EPI == EPI_LOGITS ? kUpdateParts : 1;
    const long want = (long)cu * 3 / 4;
    auto wgs = [&](int rows, int feats) { return (long)((a.M + rows - 1) / rows) * ((a.N + feats - 1) / feats); };
    if (NG == 1) return launch_few<T, EPI, 1, 24, 12, EPI == EPI_LOGITS>(a, s, ev);
    if (a.M <= 64 && NT > 2 * cu && KT % 2 == 0) return launch_rows<T, EPI, 4, 1, 4, 2, 4, 8, 2, false, NACC>(a, s, ev);
    if (a.M <= 64 || wgs(64, 64) < want) {
        const int xg = (int)std::min<long>(4, std::max<long>(1, (long)NT * NG / cu));
        if (xg == 1) return launch_few<T, EPI, 1, 24, 12>(a, s, ev);
        if (xg == 2) return launch_few<T, EPI, 2, 24, 12>(a, s, ev);
        if (NG == 3) return launch_few<T, EPI, 3, 16, 8>(a, s, ev);
        return launch_few<T, EPI, 4, 16, 8>(a, s, ev);
    }
    if (KT % 2) return launch_rows<T, EPI, 8, 2, 8, 1, 7, 2, 4, false>(a, s, ev);
    if (wgs(128, 256) > cu) return launch_rows<T, EPI, 4, 4, 8, 2, 4, 2, 2, true>(a, s, ev);
    if (wgs(128, 256) >= want) return launch_rows<T, EPI, 8, 2, 8, 2, 8, 8, 2, true>(a, s, ev);
    if (wgs(128, 128) > cu) return launch_rows<T, EPI, 8, 1, 8, 2, 4, 8, 4, false>(a, s, ev);
    if (wgs(128, 128) >= want) return launch_rows<T, EPI, 8, 1, 8, 2, 8, 16, 2, false>(a, s, ev);
    if (wgs(64, 128) >= want && KT % 4 == 0) return launch_rows<T, EPI, 4, 2, 4, 4, 4, 8, 2, true>(a, s, ev);
    if (wgs(64, 128) >= want) return launch_rows<T, EPI, 8, 1, 4, 2, 6, 16, 4, false>(a, s, ev);
    return launch_rows<T, EPI, 4, 1, 4, 2, 4, 8, 2, false>(a, s, ev);
}

template <DType T>
void gemm_rows_epi(Epi e, const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    switch (e) {
        case EPI_RESID: gemm_rows_t<T, EPI_RESID>(a, s, ev); break;
        case EPI_QKV: gemm_rows_t<T, EPI_QKV>(a, s, ev); break;
        case EPI_SWIGLU: gemm_rows_t<T, EPI_SWIGLU>(a, s, ev); break;
        default: gemm_rows_t<T, EPI_LOGITS>(a, s, ev); break;
    }
}

// ------------------------------------------------------------------------------------------
// Causal attention of a prefill block, flash-style: online softmax over 64-key chunks in increasing
// order, no partials in memory.  A workgroup takes 16 QG WV consecutive rows of the R = rows * G that
// read one kv head in one segment (row r: position p0 + r / G, head kvh * G + r % G); wave w has QG
// groups of 16 rows.  Both products are computed transposed, so that nothing has to change lanes:
//   S^T = K Q^T   A = key fragments (16 keys), B = query fragments: the lane holds keys 4 (l / 16) + j
//                 of query row l % 16, so a row's maximum and sum are in-lane but for two swaps, and
//                 its running maximum, sum and rescale factor are one register each;
//   O^T = V^T P^T A = value fragments, B = P^T.  In bf16 a B fragment holds eight keys 8 (l / 16) + e
//                 per lane; the lanes read their key rows in the order that makes the two 16-key
//                 tiles of a 32-key step give exactly those eight, so P goes from the softmax into
//                 the product without leaving its lane (the kernel before wrote it to LDS and read
//                 it back in A layout, and every wave streamed every chunk for 16 rows only).
// The chunk's keys and values are copied to LDS once per workgroup, one chunk ahead.  Rows past a
// chunk's positions mask it whole and keep their state exactly.
// 7B, 8 x 2048 tokens, per layer: 1135 us (121 TFLOP/s) before.
// ------------------------------------------------------------------------------------------
template <DType T, int HD, int QG, int WV>
__global__ void __launch_bounds__(64 * WV, HD * (int)sizeof(typename St<T>::type) > 256 ? 1 : 2) flash_prefill_kernel(FlashArgs a) {
    typedef typename St<T>::type E;
    constexpr int KC = (T == DType::BF16) ? 32 : 16, EPL = KC / 4;
    constexpr int DS = HD / KC;       // head-dim steps of S
    constexpr int KS = CK / KC;       // key steps of O
    constexpr int DT = HD / 16;       // head-dim tiles of O
    constexpr int TPK = KC / 16;      // 16-key tiles per key step
    constexpr int NF = CK * HD * (int)sizeof(E) / 1024;  // 1 KiB fragments of a chunk's keys (or values)
    __shared__ __align__(1024) uint4 kv[2][2 * NF][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int kvh = blockIdx.y, sg = blockIdx.z;
    const int b = a.seg_b[sg], p0 = a.seg_pos[sg], row0 = a.seg_row[sg], n = a.seg_len[sg];
    const int G = a.n_heads / a.n_kv, R = n * G;
    const int wg0 = (gridDim.x - 1 - blockIdx.x) * (16 * QG * WV);  // the longest rows first
    if (wg0 >= R) return;  // uniform across the workgroup
    const int r0 = wg0 + 16 * QG * w;
    const int nch = (p0 + min(wg0 + 16 * QG * WV - 1, R - 1) / G) / CK + 1;  // chunks the workgroup reads
    const int my_nch = r0 < R ? (p0 + min(r0 + 16 * QG - 1, R - 1) / G) / CK + 1 : 0;
    const size_t base = ((size_t)b * a.n_kv + kvh) * a.s_max * HD;
    const uint8_t *kc = (const uint8_t *)((const E *)a.Kc + base), *vc = (const uint8_t *)((const E *)a.Vc + base);
    const uint32_t lds0 = lds_addr(&kv[0][0][0]), lane16 = 16 * lane;
    auto copy_chunk = [&](int ch) {
        const uint32_t dst = lds0 + (uint32_t)(ch & 1) * (2 * NF * 1024);
#pragma unroll
        for (int i = 0; i < 2 * NF / WV; ++i) {
            const int f = w + WV * i;  // fragments 0 .. NF - 1: keys, then values
            copy_1k(dst + f * 1024, lane16, (f < NF ? kc + (size_t)f * 1024 : vc + (size_t)(f - NF) * 1024) + (size_t)ch * (NF * 1024));
        }
    };
    static_assert(2 * NF % WV == 0, "copies per wave");
    copy_chunk(0);
    // query fragments, pre-scaled by nothing: rounded to the storage type as the keys are
    uint4 qf[QG][DS];
    int rpos[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        const int r = r0 + 16 * g + l16, rr = min(r, R - 1), i = rr / G;
        rpos[g] = r < R ? p0 + i : -1;
        const float4 *q = (const float4 *)(a.Q + ((size_t)(row0 + i) * a.n_heads + kvh * G + rr - i * G) * HD + EPL * lg);
#pragma unroll
        for (int st = 0; st < DS; ++st) {
            float v[EPL];
#pragma unroll
            for (int e = 0; e < EPL; e += 4) {
                const float4 t = q[(st * KC + e) / 4];
                v[e] = t.x;
                v[e + 1] = t.y;
                v[e + 2] = t.z;
                v[e + 3] = t.w;
            }
            qf[g][st] = pack_frag_cvt<T>(v);
        }
    }
    f32x4 O[QG][DT];
    float m_run[QG], l_run[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        m_run[g] = -INFINITY;
        l_run[g] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) O[g][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const float sl = a.scale * 1.44269504088896341f;  // scores in units of log2
    // the lane's key row of tile h of a key step: in bf16, row r of tile h is key 8 (r / 4) + 4 h + r % 4
    // of the step, found in fragment (key / 16), slot key % 16 + 16 lg
    int koff[TPK];
#pragma unroll
    for (int h = 0; h < TPK; ++h) {
        const int key = TPK == 2 ? 8 * (l16 >> 2) + 4 * h + (l16 & 3) : l16;
        koff[h] = (key >> 4) * (DS * 64) + (key & 15) + 16 * lg;
    }
    const int nwritten = p0 + n;  // cache positions holding keys and values
    for (int ch = 0; ch < nch; ++ch) {
        wait_mem<0, true>();
        barrier();  // chunk ch is in LDS; every wave is done with the buffer of chunk ch - 1
        if (ch + 1 < nch) copy_chunk(ch + 1);
        if (ch >= my_nch) continue;  // uniform across the wave: all its keys lie past the wave's rows
        const uint4 *kb = &kv[ch & 1][0][0], *vb = &kv[ch & 1][NF][0];
        const int kbase = ch * CK;
        f32x4 S[QG][KS][TPK];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int h = 0; h < TPK; ++h) {
#pragma unroll
                for (int g = 0; g < QG; ++g) S[g][ks][h] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < DS; ++st) {
                    const uint4 kf = kb[(ks * TPK * DS + st) * 64 + koff[h]];
#pragma unroll
                    for (int g = 0; g < QG; ++g) S[g][ks][h] = St<T>::mma(kf, qf[g][st], S[g][ks][h]);
                }
            }
        // key of S[g][ks][h][j]: kbase + ks KC + (bf16: 8 lg + 4 h, fp32: 4 lg) + j
        const bool diag = kbase + CK - 1 > p0 + r0 / G;  // uniform: some row of the wave masks keys
        uint4 pf[QG][KS];
#pragma unroll
        for (int g = 0; g < QG; ++g) {
            if (diag) {
                const int lim = rpos[g] - kbase;  // keys 0 .. lim of the chunk are seen
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int h = 0; h < TPK; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (ks * KC + 4 * TPK * lg + 4 * h + j > lim) S[g][ks][h][j] = -INFINITY;
            }
            float mx = -INFINITY;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int h = 0; h < TPK; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) mx = fmaxf(mx, S[g][ks][h][j]);
            mx = quad_rows_max(mx);
            const float mnew = fmaxf(m_run[g], mx * sl);
            const float mref = mnew == -INFINITY ? 0.f : mnew;  // rows with no key yet: all weights zero
            const float alpha = __builtin_amdgcn_exp2f(m_run[g] - mref);
            float ps = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                float p[EPL];
#pragma unroll
                for (int h = 0; h < TPK; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        p[4 * h + j] = __builtin_amdgcn_exp2f(fmaf(S[g][ks][h][j], sl, -mref));
                        ps += p[4 * h + j];
                    }
                pf[g][ks] = pack_frag_cvt<T>(p);
            }
            l_run[g] = fmaf(l_run[g], alpha, ps);  // this lane's keys; the four lanes of a row add up at the end
            m_run[g] = mnew;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) O[g][dt] *= alpha;
        }
        // values of positions not yet written may hold anything: they enter as zeros
        const int nk = nwritten - kbase;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                uint4 vf = vb[(dt * KS + ks) * 64 + lane];
                if (nk < CK) vf = mask_keys<T>(vf, ks * KC + EPL * lg, nk);  // uniform
#pragma unroll
                for (int g = 0; g < QG; ++g) O[g][dt] = St<T>::mma(vf, pf[g][ks], O[g][dt]);
            }
    }
    // the lane holds head dims 16 dt + 4 lg + j of row l16 of each group
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        const int r = r0 + 16 * g + l16;
        const float inv = 1.0f / quad_rows_sum(l_run[g]);
        if (r >= R) continue;
        const int i = r / G, head = kvh * G + r - i * G;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const float v[4] = {O[g][dt][0] * inv, O[g][dt][1] * inv, O[g][dt][2] * inv, O[g][dt][3] * inv};
            store_n<T, 4>((E *)a.O + fm_index<T>(row0 + i, head * HD + 16 * dt + 4 * lg, a.n_heads * HD), v);
        }
    }
}

// Two groups of 16 rows per wave halve the LDS reads per product; with fewer than one workgroup per
// compute unit that way, one group per wave spreads the rows over twice as many workgroups.
template <DType T, int HD>
void flash_t(const FlashArgs &a, hipStream_t s, const LaunchEvents &ev) {
    const int G = a.n_heads / a.n_kv;
    long wg2 = 0;
    int longest = 0;
    for (int i = 0; i < a.n_seg; ++i) {
        wg2 += (a.seg_len[i] * G + 127) / 128 * a.n_kv;
        longest = a.seg_len[i] > longest ? a.seg_len[i] : longest;
    }
    if (wg2 >= compute_units())
        launch_ev(flash_prefill_kernel<T, HD, 2, 4>, dim3((longest * G + 127) / 128, a.n_kv, a.n_seg), dim3(256), s, ev, a);
    else
        launch_ev(flash_prefill_kernel<T, HD, 1, 4>, dim3((longest * G + 63) / 64, a.n_kv, a.n_seg), dim3(256), s, ev, a);
}

}  // namespace

void launch_gemm_rows(DType t, Epi e, const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    if (t == DType::BF16) gemm_rows_epi<DType::BF16>(e, a, s, ev);
    else gemm_rows_epi<DType::F32>(e, a, s, ev);
}

void launch_flash_prefill(DType t, const FlashArgs &a, hipStream_t s, const LaunchEvents &ev) {
    if (t == DType::BF16) {
        if (a.hd == 128) flash_t<DType::BF16, 128>(a, s, ev);
        else flash_t<DType::BF16, 64>(a, s, ev);
    } else {
        if (a.hd == 128) flash_t<DType::F32, 128>(a, s, ev);
        else flash_t<DType::F32, 64>(a, s, ev);
    }
}

void launch_embed_rows(DType t, const void *emb, const int32_t *ids, const int32_t *starts, int B, int t0, int M, int d,
                       float *h, float *ss, void *hg, const float *g, int2 *rowmap, hipStream_t s) {
    if (t == DType::BF16)
        embed_rows_kernel<DType::BF16><<<M, 256, 0, s>>>(emb, ids, starts, B, t0, d, h, ss, hg, g, rowmap);
    else
        embed_rows_kernel<DType::F32><<<M, 256, 0, s>>>(emb, ids, starts, B, t0, d, h, ss, hg, g, rowmap);
}

void launch_gather_last(DType t, const void *hg, const float *ss, int d, int nps, int B, const LastRows &lr, void *dst,
                        float *ss_dst, hipStream_t s) {
    if (t == DType::BF16) gather_last_kernel<DType::BF16><<<B, 256, 0, s>>>(hg, ss, d, nps, lr, dst, ss_dst);
    else gather_last_kernel<DType::F32><<<B, 256, 0, s>>>(hg, ss, d, nps, lr, dst, ss_dst);
}

}  // namespace dvi
