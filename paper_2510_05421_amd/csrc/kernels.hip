// gfx950 (CDNA4) kernels for the DVI self-speculative decode step.
//
// Every reduction of the decode step has a fixed order that depends only on the operand shape
// (K, head dim, vocabulary, chunk size), never on how many tokens are processed together.  Any
// token's result is therefore the same whether it is computed alone (one draft token) or inside
// a verify block: that is what makes the committed keys and values bitwise independent of which
// drafts were proposed, and the speculative output identical to plain greedy decoding on the
// same engine.  (Prompt tokens always go through the kernels of prefill.hip, in both runs.)
#include "kernels.h"

#include <hip/hip_ext.h>

#include <math.h>

#include "device.h"

namespace dvi {

// ------------------------------------------------------------------------------------------
// weight packing
// ------------------------------------------------------------------------------------------
template <DType T>
__global__ void pack_kernel(PackSrc srcs, const int32_t *prow, int N, int K, void *dst) {
    typedef typename St<T>::type E;
    const int KC = (T == DType::BF16) ? 32 : 16, EPL = KC / 4;
    const int KT = K / KC;
    const size_t nfrag = (size_t)(N / 16) * KT * 64;
    for (size_t f = (size_t)blockIdx.x * blockDim.x + threadIdx.x; f < nfrag; f += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(f & 63);
        const size_t tile = f >> 6;
        const int nt = (int)(tile / KT), kt = (int)(tile % KT);
        const int32_t code = prow[nt * 16 + (lane & 15)];
        const E *src = (const E *)srcs.src[code >> 24] + (size_t)(code & 0xffffff) * K + kt * KC + (lane >> 4) * EPL;
        E *d = (E *)dst + f * EPL;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d[e] = src[e];
    }
}

void launch_pack(DType t, PackSrc srcs, const int32_t *prow, int N, int K, void *dst, hipStream_t s) {
    if (t == DType::BF16)
        pack_kernel<DType::BF16><<<2048, 256, 0, s>>>(srcs, prow, N, K, dst);
    else
        pack_kernel<DType::F32><<<2048, 256, 0, s>>>(srcs, prow, N, K, dst);
}

// ------------------------------------------------------------------------------------------
// Skinny-M weight-streaming GEMM:  Y[m][n] = sum_k X[m][k] W[n][k],  M <= 64.
//
// One workgroup owns RT bands of 16 output features (packed tile rows) for all M tokens.
// Its waves split the K range into contiguous pieces (split fixed by K and the wave count,
// which depends only on the matrix shape), each wave streaming 1 KiB weight fragments straight
// into MFMA A operands; tokens are the MFMA B operand (16 per group, MG groups).  The per-wave
// partial tiles are summed in wave order through LDS and tile t's epilogue runs on wave t.
// Output layout of a 16x16 MFMA tile: lane l holds rows 4*(l/16)+j (j = 0..3) of column
// l % 16, i.e. features nt*16 + 4*(l/16) + j of token 16*g + (l % 16).
//
// RMSNorm is folded in: when ss_in is given, X holds dtype(h * g) and row m of the result
// is scaled by 1/sqrt(mean(h[m]^2) + eps), reduced from the partial sums of squares that the
// producing epilogue wrote.  RMSNorm(h) W^T = (h*g) W^T / rms(h), so no separate pass over h.
// ------------------------------------------------------------------------------------------
// The gate/up shape at 33-64 tokens (up to three tiles) runs under a register bound that fits two
// workgroups per compute unit (see the ring below).
template <int MG, int EPI, int RT, int WMAX>
constexpr bool gemm_two_per_cu() {
    return MG >= 3 && WMAX == 8 && EPI == EPI_SWIGLU && RT <= 3;
}

template <DType T, int MG, int EPI, int RT, int WMAX>
__global__ void __launch_bounds__(64 * WMAX, (gemm_two_per_cu<MG, EPI, RT, WMAX>() ? 4 : 1)) gemm_kernel(GemmArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int nt0 = blockIdx.x * RT;
    // the last workgroup may hold fewer than RT tiles: tiles past N / 16 load nothing and store
    // nothing (their MFMAs run on zeros)
    const int nvalid = RT == 1 ? 1 : min(RT, a.N / 16 - nt0);
    const int KC = (T == DType::BF16) ? 32 : 16;
    const int KT = a.K / KC;
    const int c0 = (wave * KT) / nw, c1 = ((wave + 1) * KT) / nw;
    // A wave takes its chunks in a rotated order, c0 + rot .. c1 - 1 then c0 .. c0 + rot - 1.
    // Without it every workgroup streams the same offset of its tile at the same time, and that
    // lockstep costs bandwidth (down projection at one row, measured alone: 19.5 -> 17.5 us).
    // rot depends only on the 12-tile group of the tile (one group holds whole workgroups of 1,
    // 2, 3 or 4 tiles), so a tile's chunk order, and its rounding, is the same at every M.
    const int rot = (nt0 / 12) % (c1 - c0);
    const size_t es = (T == DType::BF16) ? 2 : 4;
    const uint4 *wp = (const uint4 *)a.W + (size_t)nt0 * KT * 64 + lane;
    const size_t tile_stride = (size_t)KT * 64;

    const uint4 *xp[MG];
    bool xv[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g) {
        const int m = 16 * g + (lane & 15);
        xv[g] = m < a.M;
        xp[g] = (const uint4 *)a.X + (size_t)g * KT * 64 + lane;   // FM block (g, chunk 0)
    }
    f32x4 acc[RT][MG];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int g = 0; g < MG; ++g) acc[t][g] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // Requested ahead of the weight stream (their latency then hides under it): the folded
    // norm's partial sums of this wave's first token (K <= 5120), and the operands of the tile
    // whose epilogue this wave will run.  Decode shapes only (up to 32 tokens); larger M keeps
    // its registers for the accumulators and loads these after the stream.
    constexpr bool kEarly = MG <= 2;
    constexpr int SSP = 5;
    const int nparts = a.K / 16;
    const bool ss_early = kEarly && a.ss_in != nullptr && wave < a.M && nparts <= 64 * SSP;
    float ssv[SSP];
    if (ss_early) {
        const float *src = a.ss_in + (size_t)wave * a.ld_ss_in;
#pragma unroll
        for (int k = 0; k < SSP; ++k) ssv[k] = src[min(lane + 64 * k, nparts - 1)];
    }
    EpiOperands<MG> pre;
    if (kEarly && wave < nvalid) epilogue_prefetch<MG, EPI>(a, nt0 + wave, pre);

    // Each activation fragment feeds RT weight tiles.  Loads go through a ring of S stages,
    // stage st holding chunk c + st: once a stage's MFMAs have issued it is refilled with the
    // chunk S ahead, so S - 1 chunks are always in flight while one is multiplied (the same
    // registers as double-buffering S/2 chunks, with more of them in flight).  Chunks are
    // accumulated in the wave's rotated order whatever S is.  At 33-64 rows, gate/up workgroups
    // of up to three tiles take two stages under a register bound (128, the launch bound above)
    // that fits two workgroups per compute unit instead of one (7B, 64 rows: 62.9 -> 52.7 us);
    // the other epilogues, and four tiles, spill under that bound (the head at 64 rows: 86 ->
    // 145 us) and keep four stages.
    constexpr int S = gemm_two_per_cu<MG, EPI, RT, WMAX>() ? 2 : 4;
    uint4 w[S][RT], x[S][MG];
    auto fetch = [&](int cb, uint4 (&wf)[RT], uint4 (&xf)[MG]) {
        const bool in = cb < c1;
        const int cr = cb + rot - (cb + rot >= c1 ? c1 - c0 : 0);  // the chunk step cb - c0 reads
        const uint4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < RT; ++t) wf[t] = (in && t < nvalid) ? ld_stream(wp + t * tile_stride + (size_t)cr * 64) : zero;
#pragma unroll
        for (int g = 0; g < MG; ++g) xf[g] = (in && xv[g]) ? ld_stream(xp[g] + (size_t)cr * 64) : zero;
    };
#pragma unroll
    for (int st = 0; st < S; ++st) fetch(c0 + st, w[st], x[st]);
    if (kEarly && wave < nvalid) epilogue_prefetch_rope<MG, EPI>(a, nt0 + wave, pre);
    for (int c = c0; c < c1; c += S) {
#pragma unroll
        for (int st = 0; st < S; ++st) {
            if (c + st < c1) {  // uniform across the wave
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int g = 0; g < MG; ++g) acc[t][g] = St<T>::mma(w[st][t], x[st][g], acc[t][g]);
            }
            fetch(c + S + st, w[st], x[st]);
        }
    }

    // Per-wave partial tiles are summed in wave order; tile t's sum lands in wave t, which
    // then runs that tile's epilogue.
    __shared__ f32x4 red[RT][WMAX][64];
    __shared__ float sinv[64];
    // Past 32 tokens the epilogue operands, and the partial sums of the folded norm for several
    // rows at a time (all eight of a wave, or two under the register bound), are requested
    // together once the ring's registers are free: a row at a time would cost a memory round trip
    // per row (eight per wave at 64 tokens).  Same summation order as inv_rms.
    constexpr int RPW = 8;  // rows per wave when 8 waves cover 64 tokens
    constexpr int RB = gemm_two_per_cu<MG, EPI, RT, WMAX>() ? 2 : RPW;
    if (!kEarly && wave < nvalid) {
        epilogue_prefetch<MG, EPI>(a, nt0 + wave, pre);
        epilogue_prefetch_rope<MG, EPI>(a, nt0 + wave, pre);
    }
    if (a.ss_in != nullptr) {
        if (!kEarly && nw * RPW >= a.M && nparts <= 64 * SSP) {
#pragma unroll 1
            for (int r0 = 0; r0 < RPW; r0 += RB) {
                float sv[RB][SSP];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const float *src = a.ss_in + (size_t)min(wave + nw * (r0 + r), a.M - 1) * a.ld_ss_in;
#pragma unroll
                    for (int k = 0; k < SSP; ++k) sv[r][k] = src[min(lane + 64 * k, nparts - 1)];
                }
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int m = wave + nw * (r0 + r);
                    if (m < a.M) {  // uniform across the wave
                        const float v = inv_rms_regs<SSP>(sv[r], nparts, a.K, a.eps);
                        if (lane == 0) sinv[m] = v;
                    }
                }
            }
        } else {
            for (int m = wave; m < a.M; m += nw) {
                const float v = (m == wave && ss_early)
                                    ? inv_rms_regs<SSP>(ssv, nparts, a.K, a.eps)
                                    : inv_rms_loop(a.ss_in + (size_t)m * a.ld_ss_in, nparts, a.K, a.eps);
                if (lane == 0) sinv[m] = v;
            }
        }
    }
    f32x4 mine[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g) {
#pragma unroll
        for (int t = 0; t < RT; ++t) red[t][wave][lane] = acc[t][g];
        __syncthreads();
        if (wave < RT) {
            f32x4 sum = red[wave][0][lane];
            for (int w2 = 1; w2 < nw; ++w2) sum += red[wave][w2][lane];
            mine[g] = sum;
        }
        __syncthreads();
    }
    if (wave >= nvalid) return;
    gemm_epilogue<T, MG, EPI>(a, nt0 + wave, mine, sinv, pre);
}

// ------------------------------------------------------------------------------------------
// Decode GEMM at 33-64 tokens with the K pieces spread over workgroups.  Each output gets exactly
// gemm_kernel's arithmetic: K cut into the same w pieces (w from (N, K)), each piece accumulated
// from zero in the tile's rotated chunk order, the pieces added in order 0..w-1, then the same
// epilogue.  Only the placement differs.  Workgroup (tile group g, piece p) of 16 waves takes
// piece p of 16 consecutive tiles, one per wave, and loads piece p's activation fragments (every
// token group: 4 KiB per chunk at 64 tokens) into LDS once for all 16 waves; gemm_kernel instead
// has every workgroup read the activations of all its pieces for its 1-3 tiles, which at 64
// tokens crosses from L2 4x the weight bytes (out-proj, down).  Each wave writes its partial tile;
// gemm_fold_kernel adds the pieces in order and runs the epilogue.  Workgroup id = g * w + p, so
// with w = 16 the workgroups of one piece share an XCD and its L2 copy of the piece.
// ------------------------------------------------------------------------------------------
constexpr int kSplitTiles = 16;   // tiles (one per wave) of a split workgroup
constexpr int kSplitXPer = 8;     // activation fragments per wave: at most 128 per piece (128 KiB LDS)

template <DType T, int MG>
__global__ void __launch_bounds__(64 * kSplitTiles) gemm_split_kernel(GemmArgs a, int w) {
    extern __shared__ uint4 xs[];  // fragment (chunk c - c0, group g) at (c - c0) * MG + g, 64 lanes each
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blockIdx.x % w, nt = (blockIdx.x / w) * kSplitTiles + wave;
    const bool tv = nt < a.N / 16;  // uniform across the wave
    const int KT = a.K / ((T == DType::BF16) ? 32 : 16);
    const int c0 = (p * KT) / w, c1 = ((p + 1) * KT) / w, nc = c1 - c0;
    const uint4 zero = {0u, 0u, 0u, 0u};
    // the piece's activation fragments, all requested before the first weight load; rows past M
    // are zero (as gemm_kernel's lanes that load nothing)
    const int nfrag = nc * MG;
    uint4 xr[kSplitXPer];
#pragma unroll
    for (int q = 0; q < kSplitXPer; ++q) {
        const int f = wave + kSplitTiles * q, c = f / MG, g = f - c * MG;
        xr[q] = (f < nfrag && 16 * g + (lane & 15) < a.M)
                    ? ld_stream((const uint4 *)a.X + ((size_t)g * KT + c0 + c) * 64 + lane)
                    : zero;
    }
    // the tile's weights through a ring of S chunk steps, in the rotated order
    const int rot = (nt / 12) % nc;
    const uint4 *wp = (const uint4 *)a.W + (size_t)nt * KT * 64 + lane;
    constexpr int S = 4;
    uint4 wr[S];
    auto wfetch = [&](int st) {
        int c = st + rot;
        if (c >= nc) c -= nc;
        return (tv && st < nc) ? ld_stream(wp + (size_t)(c0 + c) * 64) : zero;
    };
#pragma unroll
    for (int st = 0; st < S; ++st) wr[st] = wfetch(st);
#pragma unroll
    for (int q = 0; q < kSplitXPer; ++q) {
        const int f = wave + kSplitTiles * q;
        if (f < nfrag) xs[f * 64 + lane] = xr[q];
    }
    __syncthreads();
    f32x4 acc[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g) acc[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nc; s0 += S) {
#pragma unroll
        for (int st = 0; st < S; ++st) {
            if (s0 + st < nc) {  // uniform
                int c = s0 + st + rot;
                if (c >= nc) c -= nc;
#pragma unroll
                for (int g = 0; g < MG; ++g) acc[g] = St<T>::mma(wr[st], xs[(c * MG + g) * 64 + lane], acc[g]);
            }
            wr[st] = wfetch(s0 + st + S);
        }
    }
    if (!tv) return;
    f32x4 *dst = (f32x4 *)a.kpart + ((size_t)nt * w + p) * MG * 64 + lane;
#pragma unroll
    for (int g = 0; g < MG; ++g) dst[g * 64] = acc[g];
}

// The pieces of each tile added in order 0..W-1 (P0 + P1, then + P2, ...: gemm_kernel's
// wave-order sum), then the tile's epilogue.  Workgroup nt holds tile nt, wave g its token group g
// (the epilogue treats token groups independently); 1/rms of every token as gemm_kernel computes
// it for more than 32 tokens.  All W pieces of a group are requested before the first add.
template <DType T, int EPI, int W>
__global__ void __launch_bounds__(256) gemm_fold_kernel(GemmArgs a, int mg) {
    __shared__ float sinv[64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6, nt = blockIdx.x;
    if (a.ss_in != nullptr)
        for (int m = g; m < a.M; m += 4) {
            const float v = inv_rms(a.ss_in + (size_t)m * a.ld_ss_in, a.K / 16, a.K, a.eps);
            if (lane == 0) sinv[m] = v;
        }
    __syncthreads();
    if (g >= mg) return;  // uniform across the wave
    EpiOperands<1> pre;
    epilogue_prefetch<1, EPI>(a, nt, pre, 16 * g);
    const f32x4 *src = (const f32x4 *)a.kpart + ((size_t)nt * W * mg + g) * 64 + lane;
    f32x4 v[W];
#pragma unroll
    for (int p = 0; p < W; ++p) v[p] = src[(size_t)p * mg * 64];
    f32x4 mine[1] = {v[0]};
#pragma unroll
    for (int p = 1; p < W; ++p) mine[0] = mine[0] + v[p];
    epilogue_prefetch_rope<1, EPI>(a, nt, pre);
    gemm_epilogue<T, 1, EPI>(a, nt, mine, sinv + 16 * g, pre, 16 * g);
}

// Launch shape of a weight matrix, a function of (N, K) only, never of M: RT 16-row tiles
// per workgroup (activations reused across them) and the K split over the workgroup's waves.
// Since neither depends on M, every output's summation order is the same for every call on
// that matrix (batch invariance).
struct GemmShape {
    int rt, waves;
};
static GemmShape gemm_shape(int N, int K, int KC, int M) {
    const int tiles = N / 16, chunks = K / KC, mg = (M + 15) / 16;
    // K split, from the matrix only: the most waves per workgroup (up to 16) that keep the whole
    // grid resident at once (8 waves per SIMD x 4 SIMDs x 256 CUs), and at least 8 (more loads in
    // flight per tile beats residency for the widest matrices), with >= 4 chunks per wave.
    int w = 1;
    while (w < 16 && ((long)tiles * (2 * w) <= 8192 || w < 8) && chunks / (2 * w) >= 4) w *= 2;
    // tiles per workgroup: more when there are more token groups to reuse each weight tile on
    // (16-wave workgroups have 128 registers per lane and keep one tile)
    int rt = 1;
    if (w <= 8) {
        if (mg >= 3 && tiles % 4 == 0) rt = 4;
        else if (mg >= 2 && tiles % 2 == 0) rt = 2;
        while (rt > w) rt >>= 1;
        // Workgroups this wide hold one compute unit's share of registers per 8 waves, so the
        // grid runs in rounds of (CUs x 8 / w) workgroups: take 3 tiles instead of 4 when that
        // needs fewer tile-rounds (the last workgroup may hold fewer).  QKV at 7B: 256
        // workgroups, one full round, instead of 192; gate/up: 2 rounds of 3 instead of 4.
        if (rt == 4) {
            const long slots = (long)compute_units() * 8 / w;
            auto cost = [&](int r) { return (((tiles + r - 1) / r + slots - 1) / slots) * r; };
            if (cost(3) < cost(4)) rt = 3;
        }
    }
    return {rt, w};
}

template <typename Arg>
static void launch_timed(void (*kernel)(Arg), dim3 grid, dim3 block, hipStream_t s, const LaunchEvents &ev,
                         const Arg &a) {
    if (ev.start || ev.stop)  // either may be null: one interval can span several launches
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev.start, ev.stop, 0, a);
    else
        kernel<<<grid, block, 0, s>>>(a);
}
// the same with a second argument and dynamic LDS
template <typename Arg, typename Arg2>
static void launch_timed(void (*kernel)(Arg, Arg2), dim3 grid, dim3 block, hipStream_t s, const LaunchEvents &ev,
                         const Arg &a, Arg2 b, size_t lds) {
    if (ev.start || ev.stop)
        hipExtLaunchKernelGGL(kernel, grid, block, lds, s, ev.start, ev.stop, 0, a, b);
    else
        kernel<<<grid, block, lds, s>>>(a, b);
}

template <DType T, int EPI, int RT, int WMAX>
static void gemm_dispatch_mg(const GemmArgs &a, dim3 grid, dim3 block, hipStream_t s, const LaunchEvents &ev) {
    const int mg = (a.M + 15) / 16;
    switch (mg) {
        case 1: launch_timed(gemm_kernel<T, 1, EPI, RT, WMAX>, grid, block, s, ev, a); break;
        case 2: launch_timed(gemm_kernel<T, 2, EPI, RT, WMAX>, grid, block, s, ev, a); break;
        case 3: launch_timed(gemm_kernel<T, 3, EPI, RT, WMAX>, grid, block, s, ev, a); break;
        default: launch_timed(gemm_kernel<T, 4, EPI, RT, WMAX>, grid, block, s, ev, a); break;
    }
}

template <DType T, int RT, int WMAX>
static void gemm_dispatch_epi(Epi e, const GemmArgs &a, dim3 grid, dim3 block, hipStream_t s,
                              const LaunchEvents &ev) {
    switch (e) {
        case EPI_RESID: gemm_dispatch_mg<T, EPI_RESID, RT, WMAX>(a, grid, block, s, ev); break;
        case EPI_QKV: gemm_dispatch_mg<T, EPI_QKV, RT, WMAX>(a, grid, block, s, ev); break;
        case EPI_SWIGLU: gemm_dispatch_mg<T, EPI_SWIGLU, RT, WMAX>(a, grid, block, s, ev); break;
        default: gemm_dispatch_mg<T, EPI_LOGITS, RT, WMAX>(a, grid, block, s, ev); break;
    }
}

template <DType T>
static void gemm_dispatch(Epi e, const GemmArgs &a, GemmShape sh, hipStream_t s, const LaunchEvents &ev) {
    dim3 grid((a.N / 16 + sh.rt - 1) / sh.rt), block(64 * sh.waves);
    if (sh.waves > 8) {
        gemm_dispatch_epi<T, 1, 16>(e, a, grid, block, s, ev);
        return;
    }
    switch (sh.rt) {
        case 4: gemm_dispatch_epi<T, 4, 8>(e, a, grid, block, s, ev); break;
        case 3: gemm_dispatch_epi<T, 3, 8>(e, a, grid, block, s, ev); break;
        case 2: gemm_dispatch_epi<T, 2, 8>(e, a, grid, block, s, ev); break;
        default: gemm_dispatch_epi<T, 1, 8>(e, a, grid, block, s, ev); break;
    }
}

// The split launch applies to matrices of 16 K pieces (one tile per 16-wave workgroup in
// gemm_kernel, whose activation reads at 64 tokens are 4x the weight bytes) whose piece of 64
// tokens' activations fits the LDS of one split workgroup.  In the 7B batch-8 verify (64 rows)
// out-proj and down went from 21.7 + 47.3 us to 47 us for both, split and fold launches
// included.  Matrices of 8 pieces keep gemm_kernel, whose three tiles per workgroup read the
// activations 1.3x the weight bytes: there the partial tiles' round trip through memory costs
// more than it saves (gate/up 59 -> 71 us, QKV 40 -> 55 us, head 75 -> 95 us).
static bool split_fits(const GemmShape &sh, int K, int KC, int mg) {
    const int KT = K / KC, ncmax = (KT + sh.waves - 1) / sh.waves;
    return sh.waves == 16 && ncmax * mg <= kSplitTiles * kSplitXPer;
}

size_t gemm_split_bytes(DType t, int N, int K) {
    const GemmShape sh = gemm_shape(N, K, pack_kc(t), 64);
    if (!split_fits(sh, K, pack_kc(t), 4)) return 0;
    return (size_t)(N / 16) * sh.waves * 4 * 1024;
}

template <DType T, int EPI>
static void launch_split(const GemmArgs &a, const GemmShape &sh, hipStream_t s, const LaunchEvents &ev) {
    const int NT = a.N / 16, mg = (a.M + 15) / 16, KT = a.K / pack_kc(T);
    const int ncmax = (KT + sh.waves - 1) / sh.waves;
    LaunchEvents e1 = ev, e2 = ev;  // one interval around both launches
    e1.stop = nullptr;
    e2.start = nullptr;
    const dim3 g1((NT + kSplitTiles - 1) / kSplitTiles * sh.waves), b1(64 * kSplitTiles);
    const size_t lds = (size_t)ncmax * mg * 1024;
    if (mg == 3) launch_timed(gemm_split_kernel<T, 3>, g1, b1, s, e1, a, sh.waves, lds);
    else launch_timed(gemm_split_kernel<T, 4>, g1, b1, s, e1, a, sh.waves, lds);
    launch_timed(gemm_fold_kernel<T, EPI, 16>, dim3(NT), dim3(256), s, e2, a, mg, 0);
}

template <DType T>
static void launch_split_epi(Epi e, const GemmArgs &a, const GemmShape &sh, hipStream_t s, const LaunchEvents &ev) {
    switch (e) {
        case EPI_RESID: launch_split<T, EPI_RESID>(a, sh, s, ev); break;
        case EPI_QKV: launch_split<T, EPI_QKV>(a, sh, s, ev); break;
        case EPI_SWIGLU: launch_split<T, EPI_SWIGLU>(a, sh, s, ev); break;
        default: launch_split<T, EPI_LOGITS>(a, sh, s, ev); break;
    }
}

bool launch_gemm(DType t, Epi e, const GemmArgs &a, hipStream_t s, const LaunchEvents &ev) {
    if (a.M > 64) return false;
    const GemmShape sh = gemm_shape(a.N, a.K, pack_kc(t), a.M);
    if (a.kpart != nullptr && a.M > 32 && split_fits(sh, a.K, pack_kc(t), (a.M + 15) / 16)) {
        if (t == DType::BF16)
            launch_split_epi<DType::BF16>(e, a, sh, s, ev);
        else
            launch_split_epi<DType::F32>(e, a, sh, s, ev);
        return true;
    }
    if (t == DType::BF16)
        gemm_dispatch<DType::BF16>(e, a, sh, s, ev);
    else
        gemm_dispatch<DType::F32>(e, a, sh, s, ev);
    return true;
}

// ------------------------------------------------------------------------------------------
// Embedding gather (first layer input) and the draft-head preparation
// ------------------------------------------------------------------------------------------
// Row m = b*c + i takes token tok[b*tok_stride + i]: h = E[token] (fp32), its partial sums of
// squares per 16 columns, and hg = dtype(h * g) for the first layer's folded RMSNorm.  Thread t
// holds columns 1024*kb + 4t .. +3 (d <= 8192); every load of the row is issued before the first
// use (addresses clamped into the row, values of columns past d zeroed).
template <DType T>
__global__ void __launch_bounds__(256) embed_kernel(const void *emb, const int32_t *tok, int tok_stride, int c, int d,
                                                    float *h, int ldh, float *ss, int ld_ss, void *hg, const float *g) {
    constexpr int KB = 8;
    const int m = blockIdx.x;
    const int b = m / c, i = m - b * c;
    const size_t row = (size_t)tok[(size_t)b * tok_stride + i] * d;
    float v[KB][4];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int col = min(kb * 1024 + 4 * (int)threadIdx.x, d - 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[kb][j] = St<T>::load(emb, row + col + j);
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        if (kb * 1024 >= d) break;  // uniform
        const int col = kb * 1024 + 4 * threadIdx.x;
        const bool ok = col < d;
        if (!ok)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[kb][j] = 0.f;
        const float s = sumsq16(v[kb], 1);
        if (ok) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                h[(size_t)m * ldh + col + j] = v[kb][j];
                St<T>::store(hg, fm_index<T>(m, col + j, d), v[kb][j] * g[col + j]);
            }
            if ((threadIdx.x & 3) == 0) ss[(size_t)m * ld_ss + col / 16] = s;
        }
    }
}

void launch_embed(DType t, const void *emb, const int32_t *tok, int tok_stride, int B, int c, int d, float *h, int ldh,
                  float *ss, int ld_ss, void *hg, const float *g, hipStream_t s) {
    if (t == DType::BF16)
        embed_kernel<DType::BF16><<<B * c, 256, 0, s>>>(emb, tok, tok_stride, c, d, h, ldh, ss, ld_ss, hg, g);
    else
        embed_kernel<DType::F32><<<B * c, 256, 0, s>>>(emb, tok, tok_stride, c, d, h, ldh, ss, ld_ss, hg, g);
}

// Draft head input: xhat = dtype(RMSNorm(h; g)) (the row the replay buffer logs and the head
// GEMM reads) and the LoRA projection u[c] = sum_i B_s[c][i] xhat[i].  Workgroup (c, m).
template <DType T>
__global__ void __launch_bounds__(256) head_prep_kernel(const float *__restrict__ h, int ldh,
                                                        const float *__restrict__ ss, int ld_ss,
                                                        const float *__restrict__ g, int d, float eps,
                                                        const float *__restrict__ Bm, int r, void *xhat, int ldx,
                                                        void *xfm, float *u) {
    // Thread t holds float4 columns t + 256k (d <= 8192); the row, gain and B_s row are
    // requested together (addresses clamped, columns past d skipped), then used.
    constexpr int KQ = 8;
    __shared__ float red[4];
    const int c = blockIdx.x, m = blockIdx.y;
    const int n4 = d / 4;
    const float4 *h4 = (const float4 *)(h + (size_t)m * ldh), *g4 = (const float4 *)g;
    const float4 *b4 = (const float4 *)(Bm + (size_t)c * d);
    float4 hv[KQ], gv[KQ], bv[KQ];
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
        const int q = min((int)threadIdx.x + 256 * k, n4 - 1);
        hv[k] = h4[q];
        gv[k] = g4[q];
        bv[k] = b4[q];
    }
    const float inv = inv_rms(ss + (size_t)m * ld_ss, d / 16, d, eps);
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
        const int q = threadIdx.x + 256 * k;
        if (q < n4) {
            const float hk[4] = {hv[k].x, hv[k].y, hv[k].z, hv[k].w};
            const float gk[4] = {gv[k].x, gv[k].y, gv[k].z, gv[k].w};
            const float bk[4] = {bv[k].x, bv[k].y, bv[k].z, bv[k].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x = hk[j] * inv * gk[j];
                if (T == DType::BF16) x = bf2f(f2bf(x));
                if (c == 0) {
                    St<T>::store(xhat, (size_t)m * ldx + 4 * q + j, x);
                    St<T>::store(xfm, fm_index<T>(m, 4 * q + j, d), x);
                }
                acc += bk[j] * x;
            }
        }
    }
    acc = block_sum256(acc, red);
    if (threadIdx.x == 0) u[(size_t)m * r + c] = acc;
}

void launch_head_prep(DType t, const float *h, int ldh, const float *ss, int ld_ss, const float *g, int M, int d,
                      float eps, const float *Bm, int r, void *xhat, int ldx, void *xfm, float *u, hipStream_t s) {
    if (M <= 0) return;
    dim3 grid(r, M);
    if (t == DType::BF16)
        head_prep_kernel<DType::BF16><<<grid, 256, 0, s>>>(h, ldh, ss, ld_ss, g, d, eps, Bm, r, xhat, ldx, xfm, u);
    else
        head_prep_kernel<DType::F32><<<grid, 256, 0, s>>>(h, ldh, ss, ld_ss, g, d, eps, Bm, r, xhat, ldx, xfm, u);
}

// ------------------------------------------------------------------------------------------
// Block-causal attention against the KV cache, on MFMA: split over 64-key chunks at absolute
// positions (attn_chunk), then a merge of every row's chunks in chunk order (merge_fold).
// ------------------------------------------------------------------------------------------
// One group of up to 64 chunks of a row's merge (lane = chunk for the statistics; lane holds
// head dims PER*lane .. PER*lane + PER-1 of the outputs): the group's maximum and the rescaled sums come from wave reductions with
// a fixed tree, and the partial outputs are folded in chunk order.  All NB chunks' loads are
// unconditional (addresses clamped to the group's last chunk, weights of clamped lanes zero, so
// they add zeros) and issued before the arithmetic that needs them: one round trip per group.
// NB only sets how many loads are in flight; the sum is the same for every NB >= cn.
// The arithmetic of one group, on values already loaded: my_m, my_l of chunk `lane` and the
// output partials ov[u] of chunk u for the lane's head dims.  Every merge path runs this code,
// so they give the same bits.
template <int HD, int NB>
__device__ __forceinline__ void merge_fold(float my_m, float my_l, const float (&ov)[NB][HD / 64], int cn, int lane,
                                           float &Mr, float &L, float (&o)[HD / 64]) {
    constexpr int PER = HD / 64;
    const float gm = wave_max(lane < cn ? my_m : -INFINITY);
    const float Mn = fmaxf(Mr, gm);
    const float rs = expf(Mr - Mn);  // 0 on the first group
    const float scl = lane < cn ? expf(my_m - Mn) : 0.f;
    L = L * rs + wave_sum(my_l * scl);
#pragma unroll
    for (int q = 0; q < PER; ++q) o[q] *= rs;
    Mr = Mn;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const float sc = lane_f32(scl, u);  // zero for chunks past cn
#pragma unroll
        for (int q = 0; q < PER; ++q) o[q] += ov[u][q] * sc;
    }
}

// One group from the partials in memory (coherent loads, all in flight together).
template <int HD, int NB>
__device__ __forceinline__ void merge_group(__amdgpu_buffer_rsrc_t mlr, __amdgpu_buffer_rsrc_t por, size_t slot,
                                            int cn, int lane, float &Mr, float &L, float (&o)[HD / 64]) {
    constexpr int PER = HD / 64;
    const size_t sl = slot + min(lane, cn - 1);
    const float my_m = ld_coherent_f32(mlr, (uint32_t)(sl * 8)), my_l = ld_coherent_f32(mlr, (uint32_t)(sl * 8 + 4));
    float ov[NB][PER];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const uint32_t off = (uint32_t)(((slot + min(u, cn - 1)) * HD + PER * lane) * 4);
        if (PER == 2) {
            const float2 v = ld_coherent_f32x2(por, off);
            ov[u][0] = v.x;
            ov[u][PER - 1] = v.y;
        } else {
            ov[u][0] = ld_coherent_f32(por, off);
        }
    }
    merge_fold<HD, NB>(my_m, my_l, ov, cn, lane, Mr, L, o);
}

// Head dim of position p of a chunk's partial output (the lane-major order the chunk waves
// write: position l16 * HD/16 + dt holds head dim 16 dt + l16).
template <int HD>
__device__ __forceinline__ int part_dim(int p) {
    return 16 * (p % (HD / 16)) + p / (HD / 16);
}

// Output of one merged row: lane holds slot positions PER*lane .. +PER-1.
template <DType T, int HD>
__device__ __forceinline__ void store_row(const AttnArgs &a, int m, int h, int lane, const float (&o)[HD / 64],
                                          float L) {
#pragma unroll
    for (int q = 0; q < HD / 64; ++q)
        St<T>::store(a.O, fm_index<T>(m, h * HD + part_dim<HD>((HD / 64) * lane + q), a.n_heads * HD), o[q] / L);
}

// Merge of one query row m of head h over its ncr chunks (one wave), then the row's output.
template <DType T, int HD>
__device__ __forceinline__ void merge_row(const AttnArgs &a, int m, int h, int ncr, int lane) {
    const __amdgpu_buffer_rsrc_t mlr = coherent_rsrc(a.part_ml), por = coherent_rsrc(a.part_o);
    const size_t slot0 = ((size_t)m * a.n_heads + h) * a.chunk_stride;
    float Mr = -INFINITY, L = 0.f, o[HD / 64];
#pragma unroll
    for (int q = 0; q < HD / 64; ++q) o[q] = 0.f;
    for (int c0 = 0; c0 < ncr; c0 += 64) {
        const int cn = min(64, ncr - c0);
        if (cn <= 8)
            merge_group<HD, 8>(mlr, por, slot0 + c0, cn, lane, Mr, L, o);
        else if (cn <= 16)
            merge_group<HD, 16>(mlr, por, slot0 + c0, cn, lane, Mr, L, o);
        else if (cn <= 32)
            merge_group<HD, 32>(mlr, por, slot0 + c0, cn, lane, Mr, L, o);
        else
            merge_group<HD, 64>(mlr, por, slot0 + c0, cn, lane, Mr, L, o);
    }
    store_row<T, HD>(a, m, h, lane, o, L);
}

// One wave's 64-key chunk ch of (sequence b, kv head kvh), nk of its keys in the cache.
// Keys are cut into 64-position chunks at absolute positions; the query rows that read this kv
// head (c tokens x n_heads/n_kv grouped heads) are taken 16 at a time as the MFMA row dimension:
//   S = Q K^T      A = query fragments, B = key fragments read straight from the key cache's
//                  fragment-major block of the chunk;
//   softmax        per row over the chunk's 64 keys: max, p = exp(s - max), sum (fixed tree);
//   O = P V        P goes through the wave's LDS tile Ps into A-operand layout; B = value
//                  fragments read straight from the value cache's block.
// Row at position p sees keys 0..p (block-causal); keys past a row's position, or past the
// cached length, are masked before the max and multiply as zeros.  Each row's unnormalised
// output, max and sum go to sink(row, head dim, value, with_stats, max, sum).  Rows are
// independent MFMA rows and the chunk arithmetic depends only on positions, so a row's result
// is the same whichever other rows share its block.
//
// The pieces below are shared by both chunk routines (all loads first for many query tiles;
// values after the scores for one tile), so every launch shape gives the same bits.
template <DType T, int HD>
struct AttnTile {
    typedef typename St<T>::type E;
    static constexpr int KC = (T == DType::BF16) ? 32 : 16;  // reduction depth of one fragment step
    static constexpr int EPL = KC / 4;                        // elements per lane per step
    static constexpr int DS = HD / KC;                        // head-dim steps of S = Q K^T
    static constexpr int KS = CK / KC;                        // key steps of O = P V
    static constexpr int DT = HD / 16;                        // 16-wide head-dim tiles of O
    static constexpr int PST = CK + 16 / (int)sizeof(E);      // padded LDS row of P (elements)
    typedef float4 QRaw[DS][EPL / 4];
    typedef uint4 KFrag[4][DS];
    typedef uint4 VFrag[DT][KS];

    // Query fragments of one 16-row tile: row r0 + l16, head dims step*KC + EPL*lg .. +EPL.
    // Rows past R read row R-1 and are zeroed when packed.
    static __device__ __forceinline__ void load_q(const AttnArgs &a, int b, int kvh, int r0, QRaw &qraw) {
        const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
        const int G = a.n_heads / a.n_kv, R = a.c * G;
        const int rr = min(r0 + l16, R - 1);
        const int i = rr / G, gi = rr - i * G;
        const float4 *qrow =
            (const float4 *)(a.Q + ((size_t)(b * a.c + i) * a.n_heads + kvh * G + gi) * HD + EPL * lg);
#pragma unroll
        for (int st = 0; st < DS; ++st)
#pragma unroll
            for (int e4 = 0; e4 < EPL / 4; ++e4) qraw[st][e4] = qrow[(st * KC) / 4 + e4];
    }
    // Every position of a 64-key chunk lies inside the cache row (the row length is a multiple of
    // 64), so the fragment loads are unconditional.  Keys at or past nk (not yet written, or past
    // the block) get score -inf, whatever they hold, so key fragments need no mask.
    // Key fragments: tile t holds keys 16t + l16; head dims step*KC + EPL*lg .. +EPL.  The
    // cache block is fragment-major (kv_key_offset), so fragment (t, step) is 1 KiB at
    // (t * DS + step) KiB and each load is contiguous across the wave.
    static __device__ __forceinline__ void load_k(const AttnArgs &a, int b, int kvh, int ch, KFrag &kf) {
        const int lane = threadIdx.x & 63;
        const uint4 *blk =
            (const uint4 *)((const E *)a.Kc + (((size_t)b * a.n_kv + kvh) * a.s_max + (size_t)ch * CK) * HD) + lane;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int st = 0; st < DS; ++st) kf[t][st] = blk[(t * DS + st) * 64];
    }
    // Value fragments: tile dt holds head dim 16 dt + l16; keys step*KC + EPL*lg .. +EPL, at
    // fragment dt * KS + step of the block (kv_val_offset).
    static __device__ __forceinline__ void load_v(const AttnArgs &a, int b, int kvh, int ch, VFrag &vf) {
        const int lane = threadIdx.x & 63;
        const uint4 *blk =
            (const uint4 *)((const E *)a.Vc + (((size_t)b * a.n_kv + kvh) * a.s_max + (size_t)ch * CK) * HD) + lane;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) vf[dt][ks] = blk[(dt * KS + ks) * 64];
    }
    static __device__ __forceinline__ void pack_q(const QRaw &qraw, int r0, int R, uint4 (&qf)[DS]) {
        const bool ok = r0 + ((threadIdx.x & 63) & 15) < R;
#pragma unroll
        for (int st = 0; st < DS; ++st) {
            float v[EPL];
#pragma unroll
            for (int e4 = 0; e4 < EPL / 4; ++e4) {
                const float4 q4 = qraw[st][e4];
                v[4 * e4 + 0] = ok ? q4.x : 0.f;
                v[4 * e4 + 1] = ok ? q4.y : 0.f;
                v[4 * e4 + 2] = ok ? q4.z : 0.f;
                v[4 * e4 + 3] = ok ? q4.w : 0.f;
            }
            qf[st] = pack_frag<T>(v);
        }
    }
    // S: lane holds rows r0 + 4 lg + j, key 16 t + l16
    static __device__ __forceinline__ void scores(const uint4 (&qf)[DS], const KFrag &kf, f32x4 (&S)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            S[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < DS; ++st) S[t] = St<T>::mma(qf[st], kf[t][st], S[t]);
        }
    }
    // Softmax over the chunk, P through LDS, O = P V, and the row outputs of one tile.  Values of
    // keys at or past nk have probability zero, but 0 * (NaN or inf) is not, so they are zeroed
    // as they enter the product (after the softmax, so value loads may still be in flight).
    template <typename Sink>
    static __device__ __forceinline__ void finish(const AttnArgs &a, int ch, int len0, int nk, int r0, f32x4 (&S)[4],
                                                  const VFrag &vf, E (*Ps)[PST], Sink &&sink) {
        const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
        const int kbase = ch * CK;
        const int G = a.n_heads / a.n_kv, R = a.c * G;
        float rmax[4], rsum[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (r0 + j >= R) {  // no lane holds a row here (uniform): zero weights, nothing stored
#pragma unroll
                for (int t = 0; t < 4; ++t) S[t][j] = 0.f;
                rmax[j] = -INFINITY;
                rsum[j] = 0.f;
                continue;
            }
            const int r = r0 + 4 * lg + j;
            const int i = r / G;
            const int nvalid = r < R ? min(nk, len0 + i + 1 - kbase) : 0;
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float sv = (16 * t + l16 < nvalid) ? S[t][j] * a.scale : -INFINITY;
                S[t][j] = sv;
                mx = fmaxf(mx, sv);
            }
            mx = row16_max(mx);
            float ps = 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float pv = (mx == -INFINITY) ? 0.f : exp_fast(S[t][j] - mx);
                S[t][j] = pv;
                ps += pv;
            }
            ps = row16_sum(ps);
            rmax[j] = mx;
            rsum[j] = ps;
        }
        // P -> LDS (row-major, dtype), then read back as A fragments
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) St<T>::store(&Ps[4 * lg + j][0], 16 * t + l16, S[t][j]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint4 pf[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) pf[ks] = *(const uint4 *)&Ps[l16][ks * KC + EPL * lg];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // O: lane holds rows r0 + 4 lg + j, head dim 16 dt + l16
        // A chunk whose 64 keys are all written (every chunk but a sequence's last) needs no mask.
        const bool full = nk >= CK;
        f32x4 O[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            O[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                O[dt] = St<T>::mma(pf[ks], full ? vf[dt][ks] : mask_keys<T>(vf[dt][ks], ks * KC + EPL * lg, nk), O[dt]);
        }
        // row 4 lg + j's output: head dims 16 dt + l16, dt = 0..DT-1, in this lane
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = r0 + 4 * lg + j;
            if (r < R && rmax[j] != -INFINITY) {
                float v[DT];
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) v[dt] = O[dt][j];
                sink(r, v, l16 == 0, rmax[j], rsum[j]);
            }
        }
    }
};

// Any number of query tiles (grouped heads): the first query tile and the chunk's key and
// value fragments are all requested before any of them is used; further tiles follow one by one.
template <DType T, int HD, typename Sink>
__device__ __forceinline__ void attn_chunk(const AttnArgs &a, int b, int kvh, int ch, int len0, int nk,
                                           typename St<T>::type (*Ps)[AttnTile<T, HD>::PST], Sink &&sink) {
    typedef AttnTile<T, HD> A;
    const int G = a.n_heads / a.n_kv, R = a.c * G;
    typename A::QRaw qraw;
    typename A::KFrag kf;
    typename A::VFrag vf;
    A::load_q(a, b, kvh, 0, qraw);
    A::load_k(a, b, kvh, ch, kf);
    A::load_v(a, b, kvh, ch, vf);
    // keep every load above in flight before the first use of any of them
    __builtin_amdgcn_sched_barrier(0);
    for (int r0 = 0; r0 < R; r0 += 16) {
        // a tile whose last row sits before this chunk has no keys here (a block over a chunk's edge)
        if (len0 + min(R - 1, r0 + 15) / G < ch * CK) continue;  // uniform across the wave
        if (r0 > 0) A::load_q(a, b, kvh, r0, qraw);
        uint4 qf[A::DS];
        A::pack_q(qraw, r0, R, qf);
        f32x4 S[4];
        A::scores(qf, kf, S);
        A::finish(a, ch, len0, nk, r0, S, vf, Ps, sink);
    }
}

// At most 16 query rows (one tile): the values are requested once the scores have consumed the
// keys, so keys and values are never live together (117 instead of 222 registers at head dim
// 128 in bf16: four waves per SIMD instead of two), and the value loads overlap the softmax.
template <DType T, int HD, typename Sink>
__device__ __forceinline__ void attn_chunk1(const AttnArgs &a, int b, int kvh, int ch, int len0, int nk,
                                            typename St<T>::type (*Ps)[AttnTile<T, HD>::PST], Sink &&sink) {
    typedef AttnTile<T, HD> A;
    const int R = a.c * (a.n_heads / a.n_kv);
    uint4 qf[A::DS];
    f32x4 S[4];
    {
        typename A::QRaw qraw;
        typename A::KFrag kf;
        A::load_q(a, b, kvh, 0, qraw);
        A::load_k(a, b, kvh, ch, kf);
        __builtin_amdgcn_sched_barrier(0);
        A::pack_q(qraw, 0, R, qf);
        A::scores(qf, kf, S);
    }
    __builtin_amdgcn_sched_barrier(0);
    typename A::VFrag vf;
    A::load_v(a, b, kvh, ch, vf);
    __builtin_amdgcn_sched_barrier(0);
    A::finish(a, ch, len0, nk, 0, S, vf, Ps, sink);
}

// Split-KV decode attention on MFMA: wave w of workgroup x owns chunk WPB x + w of one
// (sequence, kv head).  With MERGE, each chunk's (max, sum, unnormalised output) is published
// with agent-scope relaxed stores, and a per-(sequence, kv head) counter then tells the
// workgroup that finishes last, and that one merges every row's chunks in chunk order, reading
// them back with coherent (sc1) loads: no cache writeback, and the loads stay in flight together.
// Without MERGE the partials go out with plain stores for attn_merge_kernel, the next launch on
// the stream (7B, batch 8, 2048-token prompts, 64-row verify: 3.451 -> 3.353 ms against sc1
// write-through stores).
// ONE (at most 16 query rows per kv head, every decode shape but grouped heads over 16 rows)
// takes attn_chunk1, whose lower register count lets more waves stay resident.
template <DType T, int HD, int WPB, bool MERGE, bool ONE = false>
__global__ void __launch_bounds__(64 * WPB, (ONE && T == DType::BF16) ? 3 : 1) attn_kernel(AttnArgs a) {
    typedef typename St<T>::type E;
    constexpr int PST = CK + 16 / (int)sizeof(E);        // padded LDS row of P (elements)
    __shared__ __align__(16) E Ps[WPB][16][PST];
    __shared__ int is_last;

    const int kvh = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int len0 = a.lens[b] + a.pos_off;
    const int pmax = len0 + a.c - 1;
    const int nch = pmax / CK + 1;
    if (WPB * (int)blockIdx.x >= nch) return;  // uniform across the workgroup
    const int ch = WPB * blockIdx.x + w;
    const int G = a.n_heads / a.n_kv;
    const int R = a.c * G;
    if (ch < nch) {  // uniform across the wave
        // A row's partial output goes to its slot lane-major: the lane holding head dims
        // 16 dt + l16 (dt = 0..HD/16-1) writes them contiguously at l16 * HD/16 (part_dim maps a
        // slot position back to its head dim).
        const __amdgpu_buffer_rsrc_t por = coherent_rsrc(a.part_o);
        auto sink = [&](int r, const float (&v)[HD / 16], bool stats, float mx, float sm) {
            const int i = r / G, gi = r - i * G;
            const size_t slot = ((size_t)(b * a.c + i) * a.n_heads + kvh * G + gi) * a.chunk_stride + ch;
            const uint32_t off = (uint32_t)((slot * HD + (size_t)(lane & 15) * (HD / 16)) * 4);
            if (MERGE) {  // read back in this launch by another workgroup
#pragma unroll
                for (int q = 0; q < HD / 16; q += 4)
                    st_coherent_f32x4(por, off + 4 * q, v[q], v[q + 1], v[q + 2], v[q + 3]);
                if (stats) {
                    st_agent(a.part_ml + slot * 2 + 0, mx);
                    st_agent(a.part_ml + slot * 2 + 1, sm);
                }
            } else {  // read by the next launch: the kernel boundary orders them, plain stores suffice
#pragma unroll
                for (int q = 0; q < HD / 16; q += 4)
                    *(float4 *)((char *)a.part_o + off + 4 * q) = make_float4(v[q], v[q + 1], v[q + 2], v[q + 3]);
                if (stats) *(float2 *)(a.part_ml + slot * 2) = make_float2(mx, sm);
            }
        };
        if (ONE)
            attn_chunk1<T, HD>(a, b, kvh, ch, len0, min(CK, pmax + 1 - ch * CK), Ps[w], sink);
        else
            attn_chunk<T, HD>(a, b, kvh, ch, len0, min(CK, pmax + 1 - ch * CK), Ps[w], sink);
    }

    // Without MERGE, attn_merge_kernel merges in a launch of its own and this workgroup is done.
    if (!MERGE) return;
    // The workgroup that finishes last for (b, kv head) merges every row's chunks.  Ordering:
    // every wave's partial stores complete, then the workgroup barrier, then thread 0's counter
    // update, an agent-scope release read-modify-write that publishes the workgroup's partials
    // (ordered before it by the barrier).  Only the workgroup that reads the final count follows
    // it with an agent-scope acquire fence, synchronising with every earlier release of the
    // counter; the barrier below orders that before all of its threads' merge loads.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nwg = (nch + WPB - 1) / WPB;
        const int old = __hip_atomic_fetch_add(a.counters + (size_t)(b * a.n_kv + kvh) * kCounterStride, 1, __ATOMIC_RELEASE,
                                               __HIP_MEMORY_SCOPE_AGENT);
        is_last = (old == nwg - 1);
        if (is_last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __hip_atomic_store(a.counters + (size_t)(b * a.n_kv + kvh) * kCounterStride, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (!is_last) return;
    for (int row = w; row < R; row += WPB) {
        const int i = row / G, gi = row - i * G;
        merge_row<T, HD>(a, b * a.c + i, kvh * G + gi, (len0 + i) / CK + 1, lane);
    }
}

// The whole attention of short contexts (at most WPB chunks, at most 16 query rows per kv head) in one
// workgroup per (sequence, kv head): wave w takes chunk w, the partials stay in LDS, and the waves merge
// the rows there.  Same chunk and merge arithmetic as attn_kernel (merge_fold over eight chunks, those
// past the row's repeated with weight zero).  What it saves is the handoff: at one row the partials'
// way through memory, the counter and the reload took about half of attn_kernel's time, at more than
// four rows a launch of its own.  Bound by the latency of one chain: queries and keys, then values.
template <DType T, int HD, int WPB>
__global__ void __launch_bounds__(64 * WPB) attn_local_kernel(AttnArgs a) {
    typedef typename St<T>::type E;
    constexpr int PST = CK + 16 / (int)sizeof(E), PER = HD / 64, NB = 8;
    static_assert(WPB <= NB, "one merge group");
    __shared__ __align__(16) E Ps[WPB][16][PST];
    __shared__ __align__(16) float po[WPB][16][HD];
    __shared__ float2 ml[WPB][16];
    const int kvh = blockIdx.x, b = blockIdx.y;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int len0 = a.lens[b] + a.pos_off, pmax = len0 + a.c - 1, nch = pmax / CK + 1;
    const int G = a.n_heads / a.n_kv, R = a.c * G;
    if (w < nch) {  // uniform across the wave; nch <= WPB
        auto sink = [&](int r, const float (&v)[HD / 16], bool stats, float mx, float sm) {
            float *o = &po[w][r][(lane & 15) * (HD / 16)];
#pragma unroll
            for (int q = 0; q < HD / 16; q += 4) *(float4 *)(o + q) = make_float4(v[q], v[q + 1], v[q + 2], v[q + 3]);
            if (stats) ml[w][r] = make_float2(mx, sm);
        };
        attn_chunk1<T, HD>(a, b, kvh, w, len0, min(CK, pmax + 1 - w * CK), Ps[w], sink);
    }
    __syncthreads();
    for (int row = w; row < R; row += WPB) {
        const int i = row / G, gi = row - i * G, cn = (len0 + i) / CK + 1;  // cn <= nch
        const float2 st = ml[min(lane, cn - 1)][row];
        float ov[NB][PER], Mr = -INFINITY, L = 0.f, o[PER];
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int q = 0; q < PER; ++q) ov[u][q] = po[min(u, cn - 1)][row][PER * lane + q];
#pragma unroll
        for (int q = 0; q < PER; ++q) o[q] = 0.f;
        merge_fold<HD, NB>(st.x, st.y, ov, cn, lane, Mr, L, o);
        store_row<T, HD>(a, b * a.c + i, kvh * G + gi, lane, o, L);
    }
}

// The merge as a launch of its own: one wave per (query row, head), all at once.
template <DType T, int HD>
__global__ void __launch_bounds__(256) attn_merge_kernel(AttnArgs a) {
    const int lane = threadIdx.x & 63;
    const int gw = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (gw >= a.B * a.c * a.n_heads) return;  // uniform across the wave
    const int m = gw / a.n_heads, h = gw - m * a.n_heads;
    const int b = m / a.c, i = m - b * a.c;
    merge_row<T, HD>(a, m, h, (a.lens[b] + a.pos_off + i) / CK + 1, lane);
}

template <DType T, int HD>
static void launch_attention_t(const AttnArgs &a, hipStream_t s, const LaunchEvents &ev) {
    // One wave per 64-key chunk, four chunks per workgroup: the workgroup that finishes last
    // merges with four waves.  Each workgroup publishes its partials with one agent-scope release
    // (an L2 writeback), so four chunks per workgroup also beat one: 7B draft token 1.502 ->
    // 1.478 ms with one query row per kv head, against 1.468 ms with the ordering left to cache
    // policy bits (a relaxed counter), which the memory model does not guarantee.  A large grid, or
    // more query rows per kv head than the last workgroup has waves (verify blocks of 6 or more,
    // grouped-head verify), merges in a second launch instead, one wave per row:
    // otherwise every workgroup would wait for its partial stores before counting itself done,
    // and the last merges would run at the kernel's tail, each wave merging several rows one
    // after another (6 rows: 17.1 -> 16.0 us, 20 rows: 18.6 -> 15.7 us with the second launch).
    const int rows = a.c * (a.n_heads / a.n_kv);
    const AttnRoute route = attn_route(T, HD, rows, a.n_chunks, (long)a.n_kv * a.B, compute_units());
    if (route == ATTN_LOCAL4) {
        launch_timed(attn_local_kernel<T, HD, 4>, dim3(a.n_kv, a.B), dim3(256), s, ev, a);
    } else if (route == ATTN_LOCAL8) {
        launch_timed(attn_local_kernel<T, HD, 8>, dim3(a.n_kv, a.B), dim3(512), s, ev, a);
    } else if (route == ATTN_TWO_LAUNCHES) {
        const int all_rows = a.B * a.c * a.n_heads;
        LaunchEvents e1 = ev, e2 = ev;  // one interval around both launches
        e1.stop = nullptr;
        e2.start = nullptr;
        if (rows <= 16)  // one query tile (attn_chunk1)
            launch_timed(attn_kernel<T, HD, 4, false, true>, dim3((a.n_chunks + 3) / 4, a.n_kv, a.B), dim3(256), s, e1,
                         a);
        else
            launch_timed(attn_kernel<T, HD, 4, false>, dim3((a.n_chunks + 3) / 4, a.n_kv, a.B), dim3(256), s, e1, a);
        launch_timed(attn_merge_kernel<T, HD>, dim3((all_rows + 3) / 4), dim3(256), s, e2, a);
    } else {
        launch_timed(attn_kernel<T, HD, 4, true, true>, dim3((a.n_chunks + 3) / 4, a.n_kv, a.B), dim3(256), s, ev, a);
    }
}

void launch_attention(DType t, const AttnArgs &a, hipStream_t s, const LaunchEvents &ev) {
    if (t == DType::BF16) {
        if (a.hd == 128) launch_attention_t<DType::BF16, 128>(a, s, ev);
        else launch_attention_t<DType::BF16, 64>(a, s, ev);
    } else {
        if (a.hd == 128) launch_attention_t<DType::F32, 128>(a, s, ev);
        else launch_attention_t<DType::F32, 64>(a, s, ev);
    }
}

// ------------------------------------------------------------------------------------------
// argmax over tile partials
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) argmax_kernel(const float *pv, const int32_t *pi, int ntiles, int32_t *out,
                                                     int out_stride, const int32_t *forced, int32_t *flags) {
    __shared__ float sv[4];
    __shared__ int si[4], sb[4];
    const int m = blockIdx.x;
    float best = -INFINITY;
    int bidx = 0x3fffffff, bad = 0;
    // Eight partials per thread are requested before the first comparison.  The winner (largest
    // value, lowest index among equals) does not depend on the order they are compared in;
    // slots past ntiles compare as (-inf, no index) and change nothing.
    constexpr int U = 8;
    for (int t0 = threadIdx.x; t0 < ntiles; t0 += 256 * U) {
        float v[U];
        int code[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = t0 + 256 * k;
            v[k] = t < ntiles ? pv[(size_t)m * ntiles + t] : -INFINITY;
            code[k] = t < ntiles ? pi[(size_t)m * ntiles + t] : 0x3fffffff;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int idx = code[k] & 0x3fffffff;
            bad |= (code[k] >> 30) & 1;
            if (v[k] > best || (v[k] == best && idx < bidx)) {
                best = v[k];
                bidx = idx;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(bidx, o);
        bad |= __shfl_xor(bad, o);
        if (ov > best || (ov == best && oi < bidx)) {
            best = ov;
            bidx = oi;
        }
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sv[w] = best;
        si[w] = bidx;
        sb[w] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k) {
            if (sv[k] > best || (sv[k] == best && si[k] < bidx)) {
                best = sv[k];
                bidx = si[k];
            }
            bad |= sb[k];
        }
        if (bidx >= 0x3fffffff) bad = 1, bidx = 0;
        out[(size_t)m * out_stride] = forced ? forced[(size_t)m * out_stride] : bidx;
        if (bad) atomicOr(flags, 1);
    }
}

void launch_argmax(const float *pv, const int32_t *pi, int M, int ntiles, int32_t *out, int out_stride,
                   const int32_t *forced, int32_t *flags, hipStream_t s) {
    if (M > 0) argmax_kernel<<<M, 256, 0, s>>>(pv, pi, ntiles, out, out_stride, forced, flags);
}

// ------------------------------------------------------------------------------------------
// Commit: longest agreeing prefix, length advance (the rollback), pending token, replay log.
// One wave; lane b owns sequence b (batch <= 64).  m_b is the number of leading agreements of
// drafts and targets, read off the lane's mismatch bits.  The replay rows of every sequence get
// consecutive ring slots in sequence order from a wave prefix sum of the per-sequence row
// counts.  A step that logs more rows than the ring holds keeps its last ring_rows rows, the ones
// that would survive logging the rows one by one, so no two rows share a slot.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) commit_kernel(CommitArgs a) {
    const int lane = threadIdx.x, b = lane, k = a.k_spec;
    const bool act = b < a.B;
    if (a.flags[0] != 0) {  // non-finite logits: nothing is committed
        if (act) {
            for (int i = 0; i < k; ++i) a.tokens_out[(size_t)b * k + i] = -1;
            a.n_out[b] = 0;
            a.m_out[b] = 0;
        }
        if (lane == 0) a.copy_list[0] = 0;
        return;
    }
    const int next = a.ring_state[0], valid = a.ring_state[1];
    int m = 0, rows = 0, prev0 = 0;
    const int32_t *dr = a.drafts + (size_t)b * k;
    if (act) {
        const int32_t *tg = a.targets + (size_t)b * k;
        uint32_t miss = 1u << k;  // bit i: draft i disagrees (bit k stops the count)
        for (int i = 0; i < k; ++i) miss |= (uint32_t)(dr[i] != tg[i]) << i;
        m = __builtin_ctz(miss);
        const int lim = a.max_new ? max(a.max_new[b], 0) : k;
        const int n = min(min(m + 1, k), lim);
        prev0 = a.pending[b];
        for (int i = 0; i < k; ++i) a.tokens_out[(size_t)b * k + i] = i < n ? tg[i] : -1;
        a.lens[b] += n;
        if (n > 0) a.pending[b] = tg[n - 1];
        a.n_out[b] = n;
        a.m_out[b] = m;
        if (a.max_new && a.max_new_dec) a.max_new[b] = lim - n;
        rows = (lim > 0 && a.ring_rows > 0) ? min(m + 1, k) : 0;
    }
    // inclusive prefix sum of the row counts over the lanes (sequence order)
    int incl = rows;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    const int total = __shfl(incl, 63);
    const int first_kept = a.ring_rows > 0 ? max(total - a.ring_rows, 0) : total;
    for (int i = 1; i <= rows; ++i) {
        const int g = incl - rows + i - 1;  // row index within this step, in sequence order
        if (g < first_kept) continue;
        const int slot = (next + g) % a.ring_rows;
        a.ring_a[slot] = dr[i - 1];
        a.ring_r[slot] = (int8_t)(i <= m ? 1 : 0);
        a.ring_i[slot] = i;
        a.ring_prev[slot] = i == 1 ? prev0 : dr[i - 2];
        a.ring_fresh[slot] = 1;
        const int e = g - first_kept;
        a.copy_list[1 + 2 * e] = b * k + i - 1;
        a.copy_list[2 + 2 * e] = slot;
    }
    if (lane == 0) {
        a.copy_list[0] = total - first_kept;
        if (a.ring_rows > 0) {
            a.ring_state[0] = (next + total) % a.ring_rows;
            a.ring_state[1] = min(valid + total, a.ring_rows);
        }
        a.rng_step[0] += 1;
    }
}

void launch_commit(const CommitArgs &a, hipStream_t s) { commit_kernel<<<1, 64, 0, s>>>(a); }

// Copy of the listed rows into their ring slots: row e of the list goes src -> slot, its state
// row (row_bytes) and logits row (V floats), each split over gridDim.y blocks in 16-byte steps.
__device__ __forceinline__ void copy16(uint8_t *__restrict__ dst, const uint8_t *__restrict__ src, size_t bytes) {
    const size_t step = (size_t)gridDim.y * blockDim.x * 16;
#pragma unroll 4
    for (size_t k = ((size_t)blockIdx.y * blockDim.x + threadIdx.x) * 16; k < bytes; k += step)
        *(uint4 *)(dst + k) = *(const uint4 *)(src + k);
}

__global__ void __launch_bounds__(256) ring_copy_kernel(const int32_t *cl, const uint8_t *hk, int row_bytes,
                                                        const float *vl, int V, uint8_t *rh, float *rl) {
    const int e = blockIdx.x;
    if (e >= cl[0]) return;
    const int src = cl[1 + 2 * e], slot = cl[2 + 2 * e];
    copy16(rh + (size_t)slot * row_bytes, hk + (size_t)src * row_bytes, (size_t)row_bytes);
    copy16((uint8_t *)(rl + (size_t)slot * V), (const uint8_t *)(vl + (size_t)src * V), (size_t)V * 4);
}

void launch_ring_copy(const int32_t *cl, int max_rows, const void *hk_hat, int d, int es, const float *vlogits, int V,
                      void *ring_h, float *ring_logits, hipStream_t s) {
    // row_bytes = d * es and V * 4 are multiples of 16 (d and V are multiples of 16)
    if (max_rows > 0)
        ring_copy_kernel<<<dim3(max_rows, 8), 256, 0, s>>>(cl, (const uint8_t *)hk_hat, d * es, vlogits, V,
                                                           (uint8_t *)ring_h, ring_logits);
}

// ------------------------------------------------------------------------------------------
// Drafter update (Section 3.4).  Forward logits use the MFMA GEMM (EPI_LOGITS with LoRA);
// these kernels turn them into the loss gradient and the LoRA-factor gradients.
// ------------------------------------------------------------------------------------------
// What the update needs of the replay rows before its GEMM, in one launch (the three parts do not
// depend on each other and none fills the chip; as launches of their own: counts 2.5, u 15, FM copy 8
// us at 256 rows of d = 5120): workgroups 0 .. n r - 1 the projections u[m][c] = sum_i B_s[c][i] x[m][i]
// of row m = id / r, rank c = id % r; the next n the row's copy into the FM layout; the last the row
// counts (all, accepted, fresh, fresh and accepted; integer sums, exact in any order).  Bound by the
// L2 reads of x and B_s (each workgroup of the first part streams a row of both), so 16-byte loads.
template <DType T>
__global__ void __launch_bounds__(256) upd_prep_kernel(UpdateArgs u, float *counts) {
    typedef typename St<T>::type E;
    constexpr int EPL = 16 / (int)sizeof(E);
    __shared__ float red[4];
    const int id = blockIdx.x, nq = u.d / EPL;
    if (id < u.n * u.rank) {
        const int m = id / u.rank, c = id - m * u.rank;
        const uint4 *x = (const uint4 *)((const E *)u.Hh + (size_t)m * u.d);
        const float *bm = u.Bm + (size_t)c * u.d;
        float acc = 0.f;
        for (int q = threadIdx.x; q < nq; q += 256) {
            float xv[EPL];
            unpack_frag<T>(x[q], xv);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc += bm[q * EPL + e] * xv[e];
        }
        acc = block_sum256(acc, red);
        if (threadIdx.x == 0) u.u[id] = acc;
    } else if (id < u.n * (u.rank + 1)) {
        const int m = id - u.n * u.rank;
        const uint4 *x = (const uint4 *)((const E *)u.Hh + (size_t)m * u.d);
        for (int q = threadIdx.x; q < nq; q += 256) *(uint4 *)((E *)u.xfm + fm_index<T>(m, q * EPL, u.d)) = x[q];
    } else if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int na = 0, nf = 0, nfa = 0;
        for (int i = lane; i < u.n; i += 64) {
            const bool acc = u.r[i] != 0, fr = u.fresh[i] != 0;
            na += acc;
            nf += fr;
            nfa += acc && fr;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            na += __shfl_xor(na, o);
            nf += __shfl_xor(nf, o);
            nfa += __shfl_xor(nfa, o);
        }
        if (lane == 0) {
            counts[0] = (float)u.n;
            counts[1] = (float)na;
            counts[2] = (float)nf;
            counts[3] = (float)nfa;
        }
    }
}

// Row i: p = softmax(z), q = softmax(l/tau); KL, entropy, log p(a); then overwrite z with
// g = alpha p (log p - log q - KL) + beta (p - e_a) + eps p (log p + H).  One 1024-thread
// workgroup per row; the row maxima first, then the normalisers as sums of exp(x - max).
__device__ __forceinline__ float block_sum1024(float v, float *lds16) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds16[w] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += lds16[k];
    return s;
}
__device__ __forceinline__ float block_max1024(float v, float *lds16) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds16[w] = v;
    __syncthreads();
    float s = -INFINITY;
#pragma unroll
    for (int k = 0; k < 16; ++k) s = fmaxf(s, lds16[k]);
    return s;
}

// The row kernel (see above): thread t takes entries v = t + 1024 e in order; the first NE of them
// (e < NE) are read once into registers and serve every pass, any beyond 1024 NE are read from
// memory in each pass (7B ring of 256 rows: 54.8 -> 36.5 us).  The maxima come before the sums,
// so no running rescale and no branch per entry, and the exponentials (arguments <= 0) take the
// hardware exp2 (36.5 -> 23.1 us); the gradients stay within a few 1e-6 of the oracle.
template <int NE>
__global__ void __launch_bounds__(1024) upd_rows_kernel(UpdateArgs u, const float *counts) {
    __shared__ float red[16];
    const int i = blockIdx.x;
    float *z = u.Z + (size_t)i * u.V;
    const float *lg = u.logits + (size_t)i * u.V;
    const float itau = 1.0f / u.tau;
    const int tail = threadIdx.x + 1024 * NE;  // first entry read from memory in every pass
    float zr[NE], qr[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int v = min((int)threadIdx.x + 1024 * e, u.V - 1);  // entries past V are never used
        zr[e] = z[v];
        qr[e] = lg[v] * itau;
    }
    // both distributions' maxima over the row, then their sums of exp(x - max)
    float mz = -INFINITY, mq = -INFINITY;
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if ((int)threadIdx.x + 1024 * e < u.V) {
            mz = fmaxf(mz, zr[e]);
            mq = fmaxf(mq, qr[e]);
        }
    for (int v = tail; v < u.V; v += 1024) {
        mz = fmaxf(mz, z[v]);
        mq = fmaxf(mq, lg[v] * itau);
    }
    const float Mz = block_max1024(mz, red), Mq = block_max1024(mq, red);
    float sz = 0.f, sq = 0.f;
    if (Mz > -INFINITY && Mq > -INFINITY) {  // uniform; logits are finite
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if ((int)threadIdx.x + 1024 * e < u.V) {
                sz += exp_fast(zr[e] - Mz);
                sq += exp_fast(qr[e] - Mq);
            }
        for (int v = tail; v < u.V; v += 1024) {
            sz += exp_fast(z[v] - Mz);
            sq += exp_fast(lg[v] * itau - Mq);
        }
    }
    sz = block_sum1024(sz, red);
    sq = block_sum1024(sq, red);
    const float lz = Mz + logf(sz), lq = Mq + logf(sq);
    float kl = 0.f, ent = 0.f;
    auto klent = [&](float zv, float qv) {
        const float lp = zv - lz, lqv = qv - lq;
        const float p = exp_fast(lp);
        kl += p * (lp - lqv);
        ent -= p * lp;
    };
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if ((int)threadIdx.x + 1024 * e < u.V) klent(zr[e], qr[e]);
    for (int v = tail; v < u.V; v += 1024) klent(z[v], lg[v] * itau);
    kl = block_sum1024(kl, red);
    ent = block_sum1024(ent, red);
    const int ai = u.a[i];
    const float lpa = z[ai] - lz;
    const float n = counts[0], na = counts[1], nf = counts[2];
    const float ri = (float)u.r[i], fi = (float)u.fresh[i];
    const float alpha = u.c_kl / n;
    const float beta = u.c_ce * ri / fmaxf(na, 1.f) + u.c_pg * (ri - u.baseline) * fi / fmaxf(nf, 1.f);
    const float eps = u.c_ent / n;
    __syncthreads();  // every thread has read z[ai] before it is overwritten
    auto grad = [&](int v, float zv, float qv) {
        const float lp = zv - lz, lqv = qv - lq;
        const float p = exp_fast(lp);
        z[v] = alpha * p * (lp - lqv - kl) + beta * (p - (v == ai ? 1.f : 0.f)) + eps * p * (lp + ent);
    };
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int v = (int)threadIdx.x + 1024 * e;
        if (v < u.V) grad(v, zr[e], qr[e]);
    }
    for (int v = tail; v < u.V; v += 1024) grad(v, z[v], lg[v] * itau);
    if (threadIdx.x == 0) {
        float *st = u.row_stats + (size_t)i * 8;
        st[0] = kl;
        st[1] = ent;
        st[2] = lpa;
        st[3] = alpha * kl - beta * lpa - eps * ent;
    }
}

// The loss and its terms, summed over the ring rows by one wave, lane l adding rows l, l + 64, ...
// in order, then the fixed wave tree.
__device__ __forceinline__ void upd_loss(const UpdateArgs &u, const float *counts) {
    const int lane = threadIdx.x & 63;
    float loss = 0.f, kl = 0.f, ent = 0.f, ce = 0.f, pg = 0.f;
    for (int i = lane; i < u.n; i += 64) {
        const float *st = u.row_stats + (size_t)i * 8;
        loss += st[3];
        kl += st[0];
        ent += st[1];
        ce -= (float)u.r[i] * st[2];
        pg -= ((float)u.r[i] - u.baseline) * (float)u.fresh[i] * st[2];
    }
    loss = wave_sum(loss);
    kl = wave_sum(kl);
    ent = wave_sum(ent);
    ce = wave_sum(ce);
    pg = wave_sum(pg);
    if (lane != 0) return;
    u.loss_out[0] = loss;
    u.loss_out[1] = kl / counts[0];
    u.loss_out[2] = ce / fmaxf(counts[1], 1.f);
    u.loss_out[3] = pg / fmaxf(counts[2], 1.f);
    u.loss_out[4] = ent / counts[0];
    u.loss_out[5] = counts[0];
    u.loss_out[6] = counts[1];
    u.loss_out[7] = counts[2];
    u.loss_out[8] = counts[3];
}

// Rows rb .. rb + 255 of the ranks c0 .. c0 + 15 of a row-major [n][rank] matrix into LDS, 16
// floats per row, zero past the rank and past n (so the readers need no guards).
__device__ __forceinline__ void stage_rank_slice(float (&dst)[256][16], const float *src, int n, int rank, int rb,
                                                 int c0, int nthreads) {
    for (int e = threadIdx.x; e < 256 * 16; e += nthreads) {
        const int row = e >> 4, c = e & 15, i = rb + row;
        dst[row][c] = (i < n && c0 + c < rank) ? src[(size_t)i * rank + c0 + c] : 0.f;
    }
}

// dA[v][c] = gamma sum_i g[i][v] u[i][c] and du[i][c] = gamma sum_v A_s[v][c] g[i][v], g = dL/dz
// (the rows of Z after upd_rows_kernel), for the 16 ranks c0 .. c0 + 15: two contractions over g on
// fp32 MFMAs (16 ranks x 16 columns, four terms of the sum each).  A workgroup takes kGradV = 128
// vocabulary entries; wave w takes the 16-row blocks w, w + 8, ...  A block of g is read twice, once
// with the rows and once with the vocabulary as the MFMA's summed index, both times 16 bytes a lane
// and all in flight together; the second reading hits the caches, so memory still carries g once.  A
// wave keeps its dA sums over its blocks (the eight waves are added in order through LDS); a block's
// du sums go to du_part[b][i][16], and upd_du_sum_kernel adds the workgroups' shares.  V is a multiple
// of 16, as every vocabulary here.  Bound by the latency of one block's loads and then by memory; with
// vector fmas and a 64-lane reduction per row it was bound by those: 256 rows of V = 32000 28.9 -> 19.5 us
// (the whole update, at d = 5120, 258 -> 249), 48 rows 14.1 -> 12.4.
constexpr int kGradWaves = 8;

__global__ void __launch_bounds__(64 * kGradWaves) upd_grad_kernel(UpdateArgs u, int c0) {
    __shared__ float red[kGradWaves][kGradV][17];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    const int b = blockIdx.x, v0 = b * kGradV;
    const int rc = min(16, u.rank - c0), cc = c0 + min(l16, rc - 1);
    constexpr int VB = kGradV / 16, VH = kGradV / 64;
    // A_s[v][c0 + l16] of the lane's summed entries v = v0 + 16 m + 4 q4 + j
    float as[VB][4];
#pragma unroll
    for (int m = 0; m < VB; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int v = v0 + 16 * m + 4 * q4 + j;
            const float t = u.A[(size_t)min(v, u.V - 1) * u.rank + cc];
            as[m][j] = (v < u.V && l16 < rc) ? t : 0.f;
        }
    f32x4 dA[VH][4];  // [h][t][j]: rank 4 q4 + j, entry v0 + 64 h + 4 l16 + t
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int t = 0; t < 4; ++t) dA[h][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int ib = 16 * w; ib < u.n; ib += 16 * kGradWaves) {
        float4 gr[4][VH], gv[VB];  // rows ib + 4 s + q4, entries 64 h + 4 l16 ..; row ib + l16, entries 16 m + 4 q4 ..
        float uv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const size_t i = (size_t)min(ib + 4 * s + q4, u.n - 1);
#pragma unroll
            for (int h = 0; h < VH; ++h)
                gr[s][h] = *(const float4 *)(u.Z + i * u.V + min(v0 + 64 * h + 4 * l16, u.V - 4));
            uv[s] = u.u[i * u.rank + cc];
        }
#pragma unroll
        for (int m = 0; m < VB; ++m)
            gv[m] = *(const float4 *)(u.Z + (size_t)min(ib + l16, u.n - 1) * u.V + min(v0 + 16 * m + 4 * q4, u.V - 4));
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool row = ib + 4 * s + q4 < u.n;  // rows past n enter as zeros
            const float uc = (row && l16 < rc) ? uv[s] : 0.f;
#pragma unroll
            for (int h = 0; h < VH; ++h) {
                const float4 g = gr[s][h];
                dA[h][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(uc, row ? g.x : 0.f, dA[h][0], 0, 0, 0);
                dA[h][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(uc, row ? g.y : 0.f, dA[h][1], 0, 0, 0);
                dA[h][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(uc, row ? g.z : 0.f, dA[h][2], 0, 0, 0);
                dA[h][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(uc, row ? g.w : 0.f, dA[h][3], 0, 0, 0);
            }
        }
        // 32 products of four terms, added as a tree: chained through the accumulators, 32 terms in a row,
        // they were 1.6 times as far from the exact sum
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 du[VB];
#pragma unroll
        for (int m = 0; m < VB; ++m) {
            const bool in = v0 + 16 * m + 4 * q4 < u.V;  // entries past V enter as zeros
            const float4 g = gv[m];
            const f32x4 d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[m][0], in ? g.x : 0.f, zero, 0, 0, 0);
            const f32x4 d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[m][1], in ? g.y : 0.f, zero, 0, 0, 0);
            const f32x4 d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[m][2], in ? g.z : 0.f, zero, 0, 0, 0);
            const f32x4 d3 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[m][3], in ? g.w : 0.f, zero, 0, 0, 0);
            du[m] = (d0 + d1) + (d2 + d3);
        }
#pragma unroll
        for (int o = 1; o < VB; o <<= 1)
#pragma unroll
            for (int m = 0; m < VB; m += 2 * o) du[m] = du[m] + du[m + o];
        const f32x4 t = du[0];  // ranks 4 q4 .. + 3 of row ib + l16
        if (ib + l16 < u.n)
            *(float4 *)(u.du_part + ((size_t)b * u.n + ib + l16) * 16 + 4 * q4) = make_float4(t[0], t[1], t[2], t[3]);
    }
#pragma unroll
    for (int h = 0; h < VH; ++h)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[w][64 * h + 4 * l16 + t][4 * q4 + j] = dA[h][t][j];
    __syncthreads();
    for (int e = threadIdx.x; e < kGradV * 16; e += 64 * kGradWaves) {
        const int vv = e >> 4, c = e & 15, v = b * kGradV + vv;
        if (c >= rc || v >= u.V) continue;
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < kGradWaves; ++k) t += red[k][vv][c];
        u.dA[(size_t)v * u.rank + c0 + c] = u.gamma * t;
    }
}

// du[i][c0 + c] = gamma * (sum of the nb workgroups' shares du_part[b][i][c]).  One workgroup
// per row; thread (j, c) adds the shares of workgroups [j P, (j + 1) P) in order (P = ceil(nb /
// 16)), then the sixteen partial sums are added in order.  Workgroup n, in the first pass, sums the
// loss over the rows.
__global__ void __launch_bounds__(256) upd_du_sum_kernel(UpdateArgs u, int c0, int nb, const float *counts) {
    __shared__ float part[16][17];
    if ((int)blockIdx.x == u.n) {  // one more workgroup in the first pass
        if (threadIdx.x < 64) upd_loss(u, counts);
        return;
    }
    const int i = blockIdx.x, c = threadIdx.x & 15, j = threadIdx.x >> 4;
    const int per = (nb + 15) / 16, b0 = min(nb, j * per), b1 = min(nb, b0 + per);
    float t = 0.f;
    for (int bb = b0; bb < b1; ++bb) t += u.du_part[((size_t)bb * u.n + i) * 16 + c];
    part[j][c] = t;
    __syncthreads();
    if (j == 0 && c < min(16, u.rank - c0)) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += part[k][c];
        u.du[(size_t)i * u.rank + c0 + c] = u.gamma * sum;
    }
}

// dB[c][k] = sum_i du[i][c] h[i][k] for the 16 ranks c0 .. c0 + 15: lane = k (64 per wave); per
// block of up to 256 rows the block's du slice goes to LDS and the eight waves take an eighth of its
// rows each, eight rows' loads of h in flight.  The eight waves' sums are added in order
// through LDS.  h is read once per pass.
template <DType T>
__global__ void __launch_bounds__(512) upd_dB_kernel(UpdateArgs u, int c0) {
    __shared__ float red[8][64][17];
    __shared__ __align__(16) float ds[256][16];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = blockIdx.x * 64 + lane, kk = min(k, u.d - 1);
    const int rc = min(16, u.rank - c0);
    float acc[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[c] = 0.f;
    for (int rb = 0; rb < u.n; rb += 256) {
        __syncthreads();  // every wave is done with the previous block's slice
        stage_rank_slice(ds, u.du, u.n, u.rank, rb, c0, 512);
        __syncthreads();
        const int rpw = (min(256, u.n - rb) + 7) / 8;  // rows per wave
        const int i0 = min(u.n, rb + rpw * w), i1 = min(u.n, i0 + rpw);
        for (int ib = i0; ib < i1; ib += 8) {
            float hv[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) hv[q] = St<T>::load(u.Hh, (size_t)min(ib + q, i1 - 1) * u.d + kk);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int i = ib + q;
                if (i < i1) {  // uniform
                    const float4 *dr = (const float4 *)ds[i - rb];
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4) {
                        const float4 t = dr[c4];
                        acc[4 * c4] += t.x * hv[q];
                        acc[4 * c4 + 1] += t.y * hv[q];
                        acc[4 * c4 + 2] += t.z * hv[q];
                        acc[4 * c4 + 3] += t.w * hv[q];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) red[w][lane][c] = acc[c];
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 16; e += 512) {
        const int c = e >> 6, kl = e & 63, ko = blockIdx.x * 64 + kl;
        if (c >= rc || ko >= u.d) continue;
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) t += red[q][kl][c];
        u.dB[(size_t)(c0 + c) * u.d + ko] = t;
    }
}

void launch_update_forward(DType t, const UpdateArgs &u, hipStream_t s) {
    float *counts = u.loss_out + 12;
    const int prep = u.n * (u.rank + 1) + 1;
    if (t == DType::BF16)
        upd_prep_kernel<DType::BF16><<<prep, 256, 0, s>>>(u, counts);
    else
        upd_prep_kernel<DType::F32><<<prep, 256, 0, s>>>(u, counts);
    GemmArgs g{};
    g.W = u.W;
    g.X = u.xfm;
    g.M = u.n;
    g.N = u.V;
    g.K = u.d;
    g.Z = u.Z;
    g.lora_A = u.A;
    g.lora_u = u.u;
    g.r = u.rank;
    g.gamma = u.gamma;
    launch_gemm_rows(t, EPI_LOGITS, g, s);
    if (u.V <= 4096)
        upd_rows_kernel<4><<<u.n, 1024, 0, s>>>(u, counts);
    else
        upd_rows_kernel<32><<<u.n, 1024, 0, s>>>(u, counts);
}

void launch_update_backward(DType t, const UpdateArgs &u, hipStream_t s) {
    const int nb = grad_parts(u.V);
    for (int c0 = 0; c0 < u.rank; c0 += 16) {  // 16 ranks per pass over g
        upd_grad_kernel<<<nb, 64 * kGradWaves, 0, s>>>(u, c0);
        upd_du_sum_kernel<<<u.n + (c0 == 0), 256, 0, s>>>(u, c0, nb, u.loss_out + 12);
    }
    for (int c0 = 0; c0 < u.rank; c0 += 16) {
        if (t == DType::BF16)
            upd_dB_kernel<DType::BF16><<<(u.d + 63) / 64, 512, 0, s>>>(u, c0);
        else
            upd_dB_kernel<DType::F32><<<(u.d + 63) / 64, 512, 0, s>>>(u, c0);
    }
}

// The end of an update in one launch (as two Adam launches, two gradient copies and the flag reset:
// 20 us of launches for 4 us of memory traffic): thread i takes element i of A_s, then of B_s, then
// clears ring flag i - nA - nB.
__global__ void __launch_bounds__(256) upd_finish_kernel(FinishArgs f) {
    long i = (long)blockIdx.x * 256 + threadIdx.x;
    const bool isA = i < f.nA;
    if (!isA) i -= f.nA;
    if (!isA && i >= f.nB) {
        i -= f.nB;
        if (i < f.ring_rows) f.fresh[i] = 0;
        return;
    }
    const float gi = (isA ? f.gA : f.gB)[i];
    float *out = isA ? f.outA : f.outB;
    if (out != nullptr) out[i] = gi;
    if (f.lr == 0.f) return;
    float *m = isA ? f.mA : f.mB, *v = isA ? f.vA : f.vB, *p = isA ? f.A : f.B;
    const float mi = f.b1 * m[i] + (1.f - f.b1) * gi;
    const float vi = f.b2 * v[i] + (1.f - f.b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - f.lr * (mi / f.c1) / (sqrtf(vi / f.c2) + f.eps);
}

void launch_update_finish(FinishArgs f, int step, hipStream_t s) {
    f.c1 = 1.f - powf(f.b1, (float)step);
    f.c2 = 1.f - powf(f.b2, (float)step);
    const long n = f.nA + f.nB + f.ring_rows;
    upd_finish_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(f);
}

// ------------------------------------------------------------------------------------------
// Streaming-read reference (measurement): the HBM read rate the decode GEMMs' load pattern can
// reach.  Each lane streams 16-byte non-temporal loads, eight in flight, over a grid-stride range.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) stream_read_kernel(const uint4 *buf, size_t n16, uint32_t *sink) {
    constexpr int U = 8;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    uint32_t acc = 0;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + (U - 1) * stride < n16; i += U * stride) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ld_stream(buf + i + u * stride);
#pragma unroll
        for (int u = 0; u < U; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < n16; i += stride) {
        const uint4 v = ld_stream(buf + i);
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9e3779b9u) sink[0] = acc;
}

void launch_stream_read(const void *buf, size_t bytes, uint32_t *sink, hipStream_t s, const LaunchEvents &ev) {
    // eight 256-lane workgroups per compute unit
    const int grid = compute_units() * 8;
    if (ev.start || ev.stop)
        hipExtLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, s, ev.start, ev.stop, 0,
                              (const uint4 *)buf, bytes / 16, sink);
    else
        stream_read_kernel<<<grid, 256, 0, s>>>((const uint4 *)buf, bytes / 16, sink);
}

}  // namespace dvi
