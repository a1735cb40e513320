// Forward pass of Gated Slot Attention, chunkwise (paper: Eq. (gsa), Eq. (gsa-2pass),
// Appendix A Eqs. (gla-chunk-gate)/(gla-chunk), Algorithm 1 forward).
//
// Both slot memories decay with the same gate and are written with the same
// intensity, so they are carried as ONE memory S = [Kt | Vt] of shape
// [m x (d_k+d_v)].  Kernels of one forward call:
//
//   gate_kernel +     (gsa_scan.hip) one workgroup per (sequence, head, column slice of S)
//   scan_kernel       walks the chunks in order, keeps its slice of S in matrix-core
//                     accumulators and writes the memory at the START of every chunk to the
//                     workspace (the only sequential part; column slices are independent).
//   chunk_fwd_kernel  one workgroup per (chunk, head): pass-1 scores z (inter-chunk term from
//                     the stored memory + gated intra-chunk term), softmax over the slots in
//                     registers, and the two small matrices of pass 2: p*exp(G) [C x m] and
//                     the pair weights A2 [C x C].  z and p never round-trip HBM except for
//                     the z the backward needs.
//                     o = (p e^G) Vt_start + A2 V, the wide contraction, follows in the same kernel
//                     (gsa_wide.h) in bf16 where that is the faster form (the rule stands at the launch).
//   apply_kernel      (gsa_apply.hip) the wide contraction where it does not (also: fp32, feature map,
//                     output epilogue).
#include "gsa_chunk.h"
#include "gsa_launch.h"
#include "gsa_wide.h"

namespace gsa {

// ---------------------------------------------------------------------------------------
// Packed form: build the chunk table from the device-side sequence offsets.
// ---------------------------------------------------------------------------------------
// width: workgroups per chunk of an unsegmented scan (0: the scans are not segmented, segbase is not needed).
__global__ void prepare_kernel(const int32_t *__restrict__ cu, int n_seqs, int T, int kChunk, int chunk_slots,
                               int seg_chunks, int width, bool f32, int m, int32_t *__restrict__ table, int32_t *__restrict__ seqtab,
                               int32_t *__restrict__ segbase)
{
    __shared__ int total;
    if (threadIdx.x == 0) {
        int c0 = 0, prev_end = 0, longest = 0;
        for (int s = 0; s < n_seqs; ++s) {
            int b = min(max(cu[s], prev_end), T);
            int e = min(max(cu[s + 1], b), T);
            const int nch = (e - b + kChunk - 1) / kChunk;
            seqtab[4 * s + 0] = c0;
            seqtab[4 * s + 1] = nch;
            seqtab[4 * s + 2] = b;
            seqtab[4 * s + 3] = e - b;
            longest = max(longest, nch);
            c0 += nch;
            prev_end = e;
        }
        if (width) {   // scan segments (gsa_scan.hip); an empty sequence still has one
            if (scan_unsegmented(f32, m, longest, (long long)c0 * width)) seg_chunks = max(longest, 1);   // one per sequence
            int nsegs = 0;
            for (int s = 0; s < n_seqs; ++s) {
                segbase[s] = nsegs;
                nsegs += max(1, (seqtab[4 * s + 1] + seg_chunks - 1) / seg_chunks);
            }
            segbase[n_seqs] = nsegs;
            segbase[n_seqs + 1] = seg_chunks;
        }
        total = c0;
    }
    __syncthreads();
    // one chunk slot per thread and pass: its sequence is the last one whose first chunk is <= the slot
    // (a sequence without tokens shares its first-chunk index with its successor, so it is never the last)
    const int used = min(total, chunk_slots);
    for (int c = threadIdx.x; c < used; c += blockDim.x) {
        int lo = 0, hi = n_seqs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (seqtab[4 * mid + 0] <= c) lo = mid; else hi = mid - 1;
        }
        const int j = c - seqtab[4 * lo + 0];
        table[4 * c + 0] = lo;
        table[4 * c + 1] = seqtab[4 * lo + 2] + j * kChunk;
        table[4 * c + 2] = min(kChunk, seqtab[4 * lo + 3] - j * kChunk);
        table[4 * c + 3] = j;
    }
    for (int c = total + threadIdx.x; c < chunk_slots; c += blockDim.x) {
        table[4 * c + 0] = 0; table[4 * c + 1] = 0; table[4 * c + 2] = 0; table[4 * c + 3] = 0;
    }
}

hipError_t launch_prepare(const Plan &pl, const Work &w, hipStream_t st)
{
    if (!pl.cu_seqlens) return hipSuccess;
    KernelTimer kt(kSlotPrepare, st);
    hipLaunchKernelGGL(prepare_kernel, dim3(1), dim3(256), 0, st, pl.cu_seqlens, pl.n_seqs, pl.T, pl.chunk,
                       pl.chunk_slots, pl.seg_chunks, pl.max_seg > 1 ? pl.H * ((pl.d_k + pl.d_v) / 64) : 0, pl.dtype == 0, pl.m,
                       w.table, w.seqtab, w.segbase);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Chunk kernel of the forward: scores, softmax, pass-2 weights.
//
// Gates, contraction over the head dimension (HeadContraction), and behind it no barrier: everything stays in the registers
// of the wave that owns the 16-token row block.  B=8, T=2048, H=4, m=64, bf16, without the wide contraction: the register tiles took
// d=512 66 -> 56 us and d=128 43 -> 31 us against a form that kept gates, scores and weights as fp32 LDS tiles (eight barriers).
// With 128 workgroups (one sequence of 2048 tokens, d=512, 18.6 us of a workgroup) 2.1 us go to the gates, 5.6 to the contraction, 1.8
// to scores, softmax and pairs, 7.5 to the eight units of the wide contraction; with the chip full the launch is bound by its bytes.
// ---------------------------------------------------------------------------------------
// WIDE: the wide contraction follows in the same kernel, small matrices in LDS.
template <typename T, int M, bool WIDE> struct ChunkFwdLds {
    static constexpr int C = Geo<T>::C;
    static constexpr int PAD = Atom<T>::kPad;
    static constexpr int KM = (M < 32) ? 32 : M;   // slots padded to the contraction depth of the apply kernel
    static constexpr int ldn = M + PAD, ldt = C + PAD;
    static constexpr size_t oVn = 0;                                  // Vn [C][ldn]
    static constexpr size_t oVt = oVn + sizeof(T) * C * ldn;          // Vt [M][ldt]
    static constexpr size_t oRb = oVt + sizeof(T) * M * ldt;          // Rb [C/16][M] fp32
    // behind the gate tiles: the buffers of the contraction; in their place gated_rows' scratch of every wave, then the
    // buffers of the wide contraction; A2 and p*exp(G) behind what scratch a slower wave may still use
    static constexpr size_t oBuf = oRb + sizeof(float) * (C / 16) * M;
    static constexpr size_t szVp = sizeof(T) * kPrivate<T, M> * (C / 16), szWide = WIDE ? 2 * Wide<M>::szBuf : 0;
    static constexpr size_t oMat = oBuf + (szVp > szWide ? szVp : szWide);
    static constexpr size_t oEx = oMat + (WIDE ? Wide<M>::szTok + Wide<M>::szSlot : 0);   // rows of o on their way out
    static constexpr size_t end = oEx + (WIDE ? Wide<M>::szEx : 0);
    static constexpr size_t endC = oBuf + HeadContraction<T, M, C, 0, 0>::kBytes;
    static constexpr size_t bytes = end > endC ? end : endC;
    static_assert(sizeof(T) == 2 || 2 * bytes <= 160 * 1024, "two workgroups on a CU");
};

// GEN: the general form (write intensities from `sin` when it is not NULL; opts: read-out in the low
// byte).  PHI (with GEN): the feature map on q and k.
template <typename T, int M, bool GEN, bool PHI, bool WIDE>
__global__ __launch_bounds__(Geo<T>::NT, (M > 64 ? 1 : 2)) void chunk_fwd_kernel(ChunkMap cm, int H, int d_k, float scale,
                                                               const T *__restrict__ q, const T *__restrict__ k,
                                                               const float *__restrict__ g,
                                                               const T *__restrict__ S, StateLayout lay,
                                                               float *__restrict__ z_saved, T *__restrict__ tA,
                                                               T *__restrict__ tP, const float *__restrict__ sin,
                                                               int opts, float gate_tau, int d_v,
                                                               const T *__restrict__ v, T *__restrict__ o)
{
    using L = ChunkFwdLds<T, M, WIDE>;
    const int readout = opts & kReadoutMask;
    constexpr int C = Geo<T>::C;
    constexpr int MI = M / 16, CI = C / 16, KM = L::KM;
    extern __shared__ __align__(16) unsigned char smem[];
    T *Vn = reinterpret_cast<T *>(smem + L::oVn), *Vt = reinterpret_cast<T *>(smem + L::oVt);
    float *Rb = reinterpret_cast<float *>(smem + L::oRb);

    ChunkInfo ci;
    int cid, h;
    chunk_order(cm, H, true, cid, h);   // the forward scan has just written the last chunks
    if (!chunk_lookup(cm, cid, ci)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    const size_t tokh = (size_t)ci.tok0 * H + h;
    const size_t ch = (size_t)cid * H + h;
    const T *Kn = S + ch * lay.stride + lay.oK;      // key memory at chunk start (tiled)
    const int rowb = 16 * w, t = rowb + r;            // this wave's row block, this lane's token

    // ---- pass 1: z = scale * (inter + gated intra), Eq. (gla-chunk) with the gate on the slot side.  The gates are
    // evaluated while the first operands of the contraction are on their way.
    f32x4 p[MI];
    typename Atom<T>::Frag16 a[CI], alo[CI];
    BlockGates<M, GEN> bg;
    bg.load(g + tokh * M, (size_t)H * M, ci.len, rowb, lane, (GEN && sin) ? sin + tokh * M : nullptr, gate_tau);
    __builtin_amdgcn_sched_barrier(0);
    {
        // q, k and the key memory are not read again by this forward call: all three hinted
        HeadContraction<T, M, C, kHintX | kHintY | kHintSt, PHI ? (kHintX | kHintY) : 0> hc(q + tokh * d_k, k + tokh * d_k, (size_t)H * d_k, d_k, Kn, ci.len, tid);
        bg.template finish<T>(ci.len, rowb, lane);
        bg.template write_tiles<T>(Vn, L::ldn, Vt, L::ldt, Rb, rowb, lane);
        hc.finish(p, a, alo, smem + L::oBuf, lane, w);
    }
    gated_rows<T, M, C, GEN>(p, a, alo, bg, Vt, L::ldt, Rb, reinterpret_cast<T *>(smem + L::oBuf) + w * kPrivate<T, M>, lane, w);
    // ---- softmax over the slots, in registers
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) p[ni] *= scale;
    if (z_saved && t < ci.len) {
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
            *reinterpret_cast<f32x4 *>(z_saved + (tokh + (size_t)t * H) * M + ni * 16 + g4) = p[ni];
    }
    if (!GEN || readout == kReadSoftmax) {
        softmax_slots<M>(p);
    } else {   // element-wise read-out (ablations of Section 4)
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) p[ni][j] = readout_value(readout, p[ni][j]);
    }
    // ---- pass-2 pair weights A2[t][r] = sum_i p_t[i] s_r[i] exp(G_t[i] - G_r[i]), r <= t: row t of this wave's
    // block, one column block after the other, nearest first; `p` walks its reference backwards with them and
    // ends as the inter-chunk weights p * exp(G)
    T *mA = tA + ch * C * C, *mP = tP + ch * C * KM;
    typedef Wide<M> W;
    typename W::Stage sa, sb;
    const T *const Vs = S + ch * lay.stride + lay.oV, *const vt = v + tokh * d_v;
    T *const ot = o + tokh * d_v;
    auto unit = [=](int i) {   // columns 64*i .. of o; i is uniform over the workgroup
        return typename W::Unit{(const bf16_t *)(Vs + (size_t)64 * i * M), (const bf16_t *)(vt + 64 * i), (bf16_t *)(ot + 64 * i), (size_t)H * d_v,
                                (const bf16_t *)(smem + L::oMat), (const bf16_t *)(smem + L::oMat + W::szTok)};
    };
    const int units = d_v / 64;
    if constexpr (WIDE) {   // the first two units' tiles land during what follows
        mA = reinterpret_cast<T *>(smem + L::oMat);
        mP = reinterpret_cast<T *>(smem + L::oMat + W::szTok);
        W::fetch(sa, unit(0), ci.len, tid);
        W::fetch(sb, unit(min(1, units - 1)), ci.len, tid);
    }
    auto dA = [&](int col) { return mA + (WIDE ? W::template at<C>(t, col) : t * C + col); };
    auto dP = [&](int col) { return mP + (WIDE ? W::template at<KM>(t, col) : t * KM + col); };
    f32x4 diag = {0.f, 0.f, 0.f, 0.f};
    if (bg.kind == kPairs) diag = pair_tile_exact<M, GEN>(p, bg, lane);
    if (bg.kind == kHalf) diag = pair_tile_half<T, M, GEN>(p, bg, lane);
#pragma unroll
    for (int ni = 0; ni < MI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) p[ni][j] *= bg.walk_gate(ni, j);
#pragma unroll
    for (int b = CI - 1; b >= 0; --b) {
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        if (b <= w) {   // wave-uniform
            if (b == w && bg.kind != kNarrow) {
                x = diag;   // p is already at the start of the block
            } else {
                x = pair_tile<T, M>(p, Vn, L::ldn, b, lane);
#pragma unroll
                for (int ni = 0; ni < MI; ++ni) p[ni] *= *reinterpret_cast<const f32x4 *>(Rb + b * M + ni * 16 + g4);
            }
            if (b == w) {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = g4 + j <= r ? x[j] : 0.f;
            }
        }
        store_frag16<T>(dA(b * 16 + g4), x);
    }
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) store_frag16<T>(dP(ni * 16 + g4), p[ni]);
    if (M < KM) store_frag16<T>(dP(M + g4), f32x4{0.f, 0.f, 0.f, 0.f});   // the padded slot columns
    // ---- pass 2: o = A2 V + (p * exp(G)) Vt_start (B=8, T=2048, H=4, d=512, m=64: 57 us and a kernel of its own of 40 us -> 86 us)
    if constexpr (WIDE) {
        __syncthreads();   // the small matrices are whole, and the tiles they were made from are dead
        if (ci.len == C) W::template walk<true>(unit, units, sa, sb, smem + L::oBuf, smem + L::oEx, ci.len, tid);
        else W::template walk<false>(unit, units, sa, sb, smem + L::oBuf, smem + L::oEx, ci.len, tid);
    }
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
template <typename T, int M>
static hipError_t launch_fwd_tm(const Plan &pl, const Work &w, const void *q, const void *k, const void *v,
                                const float *g, const float *K0, const float *V0, void *o, float *z_saved, float *KT,
                                float *VT, hipStream_t st)
{
    const ChunkMap cm = make_chunk_map(pl, w);
    GSA_HIP_TRY(launch_gates(pl, w, g, pl.s_in, pl.gate_tau, st));
    {
        // kept for the backward: also the memories after the last token, as the recomputation would leave them
        const ScanIo io = {k, v, K0, V0, KT, VT, pl.keep ? w.SF : nullptr, false, pl.phi != 0, pl.phi != 0};
        GSA_HIP_TRY(launch_scan(pl, w, io, st));
    }
    // bf16 without the feature map and the output epilogue: the wide contraction follows in the chunk kernel.  Its
    // workgroup then walks the d_v/64 units one after the other, which takes longer than a kernel of its own where the walk
    // is long and few (chunk, head) pairs leave the chip idle.  Time of the forward call with the contraction inside over
    // that with a kernel of its own, 16 to 128 slots, d_k = d_v or 64:
    //   up to 9 units: 0.77 to 1.02 at 8 to 2048 pairs (d = 128, 64 slots, 1024 pairs: 73 us instead of 80)
    //   10 to 16 units: 1.2 to 1.03 at 8 to 64 pairs; equal at 144 pairs, with 128 slots at 96; 0.87 to 0.99 beyond
    //   more than 12 units and 512 pairs: 0.95 to 1.14 up to 64 slots (d_v = 1024)
    const int64_t pairs = (int64_t)pl.chunk_slots * pl.H;
    const bool wide = sizeof(T) == 2 && !pl.phi && !pl.act_out && !pl.act_ssq &&
                      (pl.d_v <= 576 || pairs >= (M > 64 ? 96 : 144)) && (pl.d_v <= 768 || pairs <= 512);
    {
        constexpr bool kWide = sizeof(T) == 2;
        auto kern = pl.phi          ? chunk_fwd_kernel<T, M, true, true, false>
                    : pl.general() ? (wide ? chunk_fwd_kernel<T, M, true, false, kWide> : chunk_fwd_kernel<T, M, true, false, false>)
                                   : (wide ? chunk_fwd_kernel<T, M, false, false, kWide> : chunk_fwd_kernel<T, M, false, false, false>);
        const size_t lds = wide ? ChunkFwdLds<T, M, kWide>::bytes : ChunkFwdLds<T, M, false>::bytes;
        GSA_HIP_TRY(allow_lds(kern, lds));
        dim3 grid(pl.chunk_slots, pl.H);
        KernelTimer kt(kSlotChunkFwd, st);
        hipLaunchKernelGGL(kern, grid, dim3(Geo<T>::NT), lds, st, cm, pl.H, pl.d_k, pl.scale, (const T *)q,
                           (const T *)k, g, (const T *)w.S, pl.lay, z_saved, (T *)w.tA, (T *)w.tP, pl.s_in,
                           pl.opts(), pl.gate_tau, pl.d_v, (const T *)v, (T *)o);
        GSA_HIP_TRY(hipGetLastError());
    }
    if (wide) return hipSuccess;
    ApplyIo io = {w.tA, w.tP, v, w.S, pl.lay.oV, pl.lay.stride, o, pl.d_v, pl.phi != 0, nullptr};
    io.act = pl.act_out;
    io.ssq = pl.act_ssq;
    return launch_apply(pl, w, &io, 1, kSlotApplyFwd, st);
}

template <typename T>
static hipError_t launch_fwd_t(const Plan &pl, const Work &w, const void *q, const void *k, const void *v,
                               const float *g, const float *K0, const float *V0, void *o, float *z_saved, float *KT,
                               float *VT, hipStream_t st)
{
    switch (pl.m) {
    case 16: return launch_fwd_tm<T, 16>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
    case 32: return launch_fwd_tm<T, 32>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
    case 128: return launch_fwd_tm<T, 128>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
    default: return launch_fwd_tm<T, 64>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
    }
}

hipError_t launch_fwd(const Plan &pl, const Work &w, const void *q, const void *k, const void *v, const float *g,
                      const float *K0, const float *V0, void *o, float *z_saved, float *KT, float *VT, hipStream_t st)
{
    if (pl.tokens == 0) return hipSuccess;
    GSA_HIP_TRY(launch_prepare(pl, w, st));
    if (pl.dtype == 0) return launch_fwd_t<float>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
    return launch_fwd_t<bf16_t>(pl, w, q, k, v, g, K0, V0, o, z_saved, KT, VT, st);
}

}  // namespace gsa
