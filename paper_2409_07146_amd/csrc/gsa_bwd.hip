// Backward pass of Gated Slot Attention, chunkwise (paper: Algorithm 1 backward;
// gradients derived from Eq. (gsa), not transcribed from the listing).
//
// Per sequence and head, with S = [Kt | Vt] the joint slot memory, G the chunk-local
// cumulative log gate, s = 1 - exp(g), p = softmax(z):
//
//   dp_t[i] = <Vt_t[i], dO_t>                       (same gated contraction as pass 1)
//   dz_t    = p_t * (dp_t - <p_t, dp_t>)
//   E       = gradient of the loss w.r.t. the memory at the END of a chunk, through later
//             chunks only; carried backwards by  E' = Diag(exp G_C) E + (w * exp G)^T x
//             with (w, x) = (scale*dz, q) on the key columns and (p, dO) on the value columns
//   Bm[t,r] = sum_i dz_t[i] s_r[i] exp(G_t[i]-G_r[i]),  A2[t,r] likewise with p_t   (r <= t)
//   dq = scale * ((dz*exp G) Kt_start + Bm K)        (the scale is folded into the small matrices)
//   dk = scale * Bm^T Q + (s*exp(G_C-G)) E_k          dv = A2^T dO + (s*exp(G_C-G)) E_v
//   ds_r[i] = exp(G_C-G_r)[i] <E[i], [k_r|v_r]> + sum_{t>=r} exp(G_t-G_r)[i] (scale dz_t[i] <q_t,k_r> + p_t[i] <dO_t,v_r>)
//   dGam_t = z_t dz_t + p_t dp_t - s_t ds_t          (gradient w.r.t. the cumulative log gate)
//   dg_j   = sum_{t>=j, same chunk} dGam_t + <E[i], S_end[i]> - exp(g_j) ds_j
//
// The last line replaces the sequence-long reversed cumulative sum of Algorithm 1 by a
// chunk-local one: the sum of dGam over all later chunks equals the row-wise inner product
// of the chunk-end memory with its gradient, which both scans already hold.  That keeps
// rounding errors from accumulating along the sequence (measured: summing the chunk totals
// instead costs about a third more error on dg with bf16 memories).
//
// Kernels of one backward call: gate + forward scan (gsa_scan.hip; recompute the chunk-start
// memories, since nothing but z was saved by the forward), chunk_dz (chunk-parallel: dp, dz,
// weights of the reverse scan), reverse scan (gsa_scan.hip: E), chunk_intra (chunk-parallel:
// Bm, A2, ds, dg and, in bf16, dq, dk, dv from them: gsa_wide.h), or apply (gsa_apply.hip: dq,
// dk, dv from matrices in memory; the rule stands at the launch).
#include "gsa_chunk.h"
#include "gsa_launch.h"
#include "gsa_wide.h"

namespace gsa {

// ---------------------------------------------------------------------------------------
// dz kernel: the forward's chunk kernel with (dO, v, value memory) for (q, k, key memory) and the softmax
// backward behind it, in the same register tiles (B=8, T=2048, H=4, d=512, m=64, bf16: 69 -> 62 us)
// ---------------------------------------------------------------------------------------
template <typename T, int M> struct DzLds {
    static constexpr int C = Geo<T>::C;
    static constexpr int PAD = Atom<T>::kPad;
    static constexpr int ldt = C + PAD, ldx = 16 + PAD;
    static constexpr size_t oVt = 0;                                  // Vt [M][ldt]
    static constexpr size_t oRb = oVt + sizeof(T) * M * ldt;          // Rb [C/16][M] fp32
    static constexpr size_t oX = oRb + sizeof(float) * (C / 16) * M;  // per wave: [kRows][ldx], transposing scratch
    static constexpr int kRows = 2 * M + (sizeof(T) == 2 ? 2 : 1) * C;   // the products' roundings leave a rest in bf16
    static constexpr size_t szX = sizeof(T) * kRows * ldx;
    static_assert(kRows * ldx >= kPrivate<T, M>, "gated_rows' scratch");
    static constexpr size_t end = oX + szX * (C / 16), endC = oX + HeadContraction<T, M, C, 0, 0>::kBytes;   // the contraction's buffers go first
    static constexpr size_t bytes = end > endC ? end : endC;
};

// GEN: the general form (write intensities from `sin` when it is not NULL; opts: read-out in the low
// byte).  PHI (with GEN): the feature map on v.
template <typename T, int M, bool GEN, bool PHI>
__global__ __launch_bounds__(Geo<T>::NT, (M > 64 ? 1 : 2)) void chunk_dz_kernel(ChunkMap cm, int H, int d_v, float scale,
                                                              const T *__restrict__ v, const T *__restrict__ dO,
                                                              const float *__restrict__ g, const float *__restrict__ z,
                                                              const T *__restrict__ S, StateLayout lay,
                                                              float *__restrict__ dz, float *__restrict__ dgf,
                                                              T *__restrict__ Wr, T *__restrict__ tAvT, T *__restrict__ tAvLo,
                                                              const float *__restrict__ sin, int opts,
                                                              float gate_tau)
{
    using L = DzLds<T, M>;
    const int readout = opts & kReadoutMask;
    constexpr int C = Geo<T>::C;
    constexpr int MI = M / 16, CI = C / 16;
    extern __shared__ __align__(16) unsigned char smem[];
    T *Vt = reinterpret_cast<T *>(smem + L::oVt);
    float *Rb = reinterpret_cast<float *>(smem + L::oRb);

    ChunkInfo ci;
    int cid, h;
    chunk_order(cm, H, true, cid, h);   // the forward scan has just written the last chunks
    if (!chunk_lookup(cm, cid, ci)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    const size_t tokh = (size_t)ci.tok0 * H + h;
    const size_t ch = (size_t)cid * H + h;
    const T *Vn = S + ch * lay.stride + lay.oV;      // value memory at chunk start (tiled)
    const int rowb = 16 * w, t = rowb + r;            // this wave's row block, this lane's token
    const bool live = t < ci.len;
    const size_t row = (tokh + (size_t)min(t, ci.len - 1) * H) * M + g4;   // clamped; nothing is stored past len

    f32x4 dp[MI], zv[MI];
    typename Atom<T>::Frag16 a[CI], alo[CI];
    BlockGates<M, GEN> bg;
    bg.load(g + tokh * M, (size_t)H * M, ci.len, rowb, lane, (GEN && sin) ? sin + tokh * M : nullptr, gate_tau);
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) zv[ni] = *reinterpret_cast<const f32x4 *>(z + row + ni * 16);
    __builtin_amdgcn_sched_barrier(0);
    {
        // dO is hinted; v and the chunk-start value memory are read again by chunk_intra and stay cached
        HeadContraction<T, M, C, kHintX, PHI ? kHintY : 0> hc(dO + tokh * d_v, v + tokh * d_v, (size_t)H * d_v, d_v, Vn, ci.len, tid);
        bg.template finish<T>(ci.len, rowb, lane);
        bg.template write_tiles<T>(nullptr, 0, Vt, L::ldt, Rb, rowb, lane);
        hc.finish(dp, a, alo, smem + L::oX, lane, w);
    }
    T *X = reinterpret_cast<T *>(smem + L::oX + (size_t)w * L::szX);   // this wave's scratch
    gated_rows<T, M, C, GEN>(dp, a, alo, bg, Vt, L::ldt, Rb, X, lane, w);
    // slope*(dp - pdp) is dz: p and <p,dp> for the softmax, f'(z) and 0 for an element-wise read-out
    f32x4 p[MI], slope[MI];
    float pdp = 0.f;
    if (!GEN || readout == kReadSoftmax) {
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) p[ni] = zv[ni];
        softmax_slots<M>(p);
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            slope[ni] = p[ni];
#pragma unroll
            for (int j = 0; j < 4; ++j) sum[j] += p[ni][j] * dp[ni][j];
        }
        pdp = slots_sum((sum[0] + sum[1]) + (sum[2] + sum[3]));
    } else {
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                p[ni][j] = readout_value(readout, zv[ni][j]);
                slope[ni][j] = readout_slope(readout, zv[ni][j]);
            }
    }
    // dz, dgf for the intra kernel; gate-weighted transposes (scale*dz*exp G, p*exp G) for the reverse scan and
    // the causally masked (dO_t . v_r), transposed, for the intra kernel's ds contraction.  The three are
    // token-fastest in memory: this wave's 16 tokens of every row meet in its own piece of LDS first.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // gated_rows has read what it kept there
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        f32x4 pre = {1.f, 1.f, 1.f, 1.f};   // exp of the cumulative log gate before the block
#pragma unroll
        for (int b = 0; b < CI - 1; ++b)
            if (b < w) pre *= *reinterpret_cast<const f32x4 *>(Rb + b * M + ni * 16 + g4);
        f32x4 dzv, dgv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float x = live ? slope[ni][j] * (dp[ni][j] - pdp) : 0.f;
            const float eg = __expf(bg.L[ni][j]) * pre[j];
            dzv[j] = x;
            dgv[j] = zv[ni][j] * x + p[ni][j] * dp[ni][j];
            const int i = ni * 16 + g4 + j;
            X[i * L::ldx + r] = from_f32<T>(scale * x * eg);
            X[(M + i) * L::ldx + r] = from_f32<T>(live ? p[ni][j] * eg : 0.f);
        }
        if (live) {
            *reinterpret_cast<f32x4 *>(dz + row + ni * 16) = dzv;
            *reinterpret_cast<f32x4 *>(dgf + row + ni * 16) = dgv;
        }
    }
#pragma unroll
    for (int b = 0; b < CI; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            X[(2 * M + b * 16 + g4 + j) * L::ldx + r] = a[b][j];
            // dp carries what the rounding of the products left behind; ds has to as well, so that the errors of the two
            // cancel in dg (bf16, rel-L2 from the fp64 recurrence: 3.1e-3 where only one does)
            if (sizeof(T) == 2) X[(2 * M + C + b * 16 + g4 + j) * L::ldx + r] = alo[b][j];
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // The scan weights in fragment order: 16 slots, a piece of the tokens next to each other in a run of 256 bytes.
    T *dW = Wr + ch * 2 * M * C, *dAv = tAvT + ch * C * C + rowb, *dLo = tAvLo + ch * C * C + rowb;
    constexpr int PV = 16 / sizeof(T), PT = 16 / PV;   // pieces of a row's 16 tokens
#pragma unroll
    for (int u = 0; u < 2 * M * PT / kWave; ++u) {
        const int idx = lane + u * kWave, rr = idx / (16 * PT) * 16 + (idx & 15), c = idx / 16 % PT * PV;
        const f32x4 x = *reinterpret_cast<const f32x4 *>(X + rr * L::ldx + c);
        *reinterpret_cast<f32x4 *>(dW + (rr / M) * M * C + frag_order<T, C / 32>(rr % M, rowb + c)) = x;
    }
#pragma unroll
    for (int u = 0; u < 2 * (L::kRows - 2 * M) / kWave; ++u) {
        const int idx = lane + u * kWave, rr = idx >> 1, c8 = (idx & 1) * 8;
        Raw8<T> x;
        x.load(X + (2 * M + rr) * L::ldx + c8);
        x.store((rr < C ? dAv + (size_t)rr * C : dLo + (size_t)(rr - C) * C) + c8);
    }
}

// ---------------------------------------------------------------------------------------
// Intra-chunk gradient kernel.
// ---------------------------------------------------------------------------------------
// By value: a conditional expression over variables selects their addresses, which keeps them in memory.
template <typename P> __device__ __forceinline__ P pick(bool c, P x, P y) { return c ? x : y; }

// WIDE: the wide contractions follow in the same kernel, small matrices in LDS.
template <typename T, int M, bool WIDE> struct IntraLds {
    static constexpr int C = Geo<T>::C;
    static constexpr int PAD = Atom<T>::kPad;
    static constexpr int KM = (M < 32) ? 32 : M;
    static constexpr int ldn = M + PAD, ldt = C + PAD;
    static constexpr size_t oVn = 0;                                  // Vn [C][ldn]
    static constexpr size_t oUd = oVn + sizeof(T) * C * ldn;          // Ud [M][ldt]
    static constexpr size_t oUp = oUd + sizeof(T) * M * ldt;          // Up [M][ldt]
    static constexpr size_t tiles = oUp + sizeof(T) * M * ldt;
    // Rb, Rd, Rr, dGam totals: [C/16][M] fp32 each, and the carry [M], behind the first buffer of the wide contractions
    // (they are read until that buffer has been written)
    static constexpr size_t oRb = (WIDE && tiles < Wide<M>::szBuf) ? Wide<M>::szBuf : tiles;
    static constexpr size_t oCarry = oRb + 4 * sizeof(float) * (C / 16) * M;
    static constexpr size_t endR = oCarry + sizeof(float) * M;
    static constexpr bool kTwo = sizeof(T) == 2 || M < 64;   // registers for two steps at a time (see walk_steps), gates and scores
    // the buffers of the contractions; later Bm, Bm^T, A2^T, scale*dz*exp(G), s*exp(G_C-G)
    // fp32 with 128 slots: one buffer, in the place of the tiles (without kTwo they are written when the contractions have ended), so that
    // two workgroups fit a CU: 8 x 2048 tokens, 4 heads, d = 512 726 -> 574 us, d = 64 225 -> 152.  With 64 slots two fit as
    // it is, and more make no difference on the whole: d = 128 117 -> 105 us, d = 512 354 -> 362, d = 640 417 -> 440.
    static constexpr bool kTight = sizeof(T) == 4 && M > 64;
    static constexpr size_t oMat = kTight ? 0 : (WIDE && endR < 2 * Wide<M>::szBuf) ? 2 * Wide<M>::szBuf : endR;
    static constexpr size_t oK = sizeof(T) * C * StepTile<T>::KS, oE = 2 * oK, szBuf = oE + sizeof(T) * M * StepTile<T>::KS;   // q, k or v, E
    static constexpr size_t szMat = WIDE ? 3 * Wide<M>::szTok + 2 * Wide<M>::szSlot : 0;
    static constexpr size_t oEx = oMat + szMat;   // rows of the outputs on their way out
    static constexpr size_t szAll = szMat + (WIDE ? Wide<M>::szEx : 0);
    static constexpr size_t szC = (kTight ? 1 : 2) * szBuf, endC = oMat + (szAll > szC ? szAll : szC);
    static constexpr size_t bytes = endC > endR ? endC : endR;
    static_assert(!(kTight && kTwo) && (sizeof(T) == 2 || 2 * bytes <= 160 * 1024), "two workgroups on a CU");
};

template <typename T> struct IntraArgs {
    const T *q, *k, *v;
    const float *g, *z, *dz, *dgf;
    const T *S, *SF, *E;
    StateLayout lay;
    const T *tAvT, *tAvLo;   // bf16: product and rest
    float *dg;
    T *tB, *tBT, *tA2T, *tDZe, *tSbe;   // for the apply kernel (not WIDE)
    const T *dO;                        // WIDE
    T *dq, *dk, *dv;                    // WIDE
    const float *sin;   // general form: write intensities, or NULL
    float *ds;          // general form: their gradient (with sin)
    int readout;
    float gate_tau;     // general form: > 0 when g holds gate logits
};

template <typename T, int M, bool GEN, bool PHI, bool WIDE>
__global__ __launch_bounds__(Geo<T>::NT, (M > 64 ? 1 : 2)) void chunk_intra_kernel(ChunkMap cm, int H, int d_k, int d_v, float scale,
                                                                 IntraArgs<T> a)
{
    using L = IntraLds<T, M, WIDE>;
    constexpr int C = Geo<T>::C;
    constexpr int MI = M / 16, CI = C / 16, KM = L::KM;
    constexpr int NB = CI + MI;
    extern __shared__ __align__(16) unsigned char smem[];
    T *Vn = reinterpret_cast<T *>(smem + L::oVn), *Ud = reinterpret_cast<T *>(smem + L::oUd), *Up = reinterpret_cast<T *>(smem + L::oUp);
    float *Rb = reinterpret_cast<float *>(smem + L::oRb), *Rd = Rb + CI * M, *Rr = Rd + CI * M, *Tot = Rr + CI * M;
    float *carry = reinterpret_cast<float *>(smem + L::oCarry);   // [M]

    ChunkInfo ci;
    int cid, h;
    chunk_order(cm, H, false, cid, h);   // the reverse scan has just written the first chunks
    if (!chunk_lookup(cm, cid, ci)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    const size_t tokh = (size_t)ci.tok0 * H + h;
    const size_t ch = (size_t)cid * H + h;
    const T *EK = a.E + ch * a.lay.stride + a.lay.oK;        // memory gradient at chunk end
    const T *EV = a.E + ch * a.lay.stride + a.lay.oV;
    int chunk0, nch, stok0, sntok;
    seq_lookup(cm, ci.seq, chunk0, nch, stok0, sntok);
    const T *SendK, *SendV;                                  // memory at chunk end
    if (ci.idx + 1 < nch) {
        const T *rec = a.S + (ch + H) * a.lay.stride;        // = start of the next chunk
        SendK = rec + a.lay.oK;
        SendV = rec + a.lay.oV;
    } else {
        const T *rec = a.SF + ((size_t)ci.seq * H + h) * a.lay.stride;
        SendK = rec + a.lay.oK;
        SendV = rec + a.lay.oV;
    }
    const T *AvT = a.tAvT + ch * C * C;
    const int rowb = 16 * w;
    const int t = rowb + r;                                  // this lane's token
    const bool live = t < ci.len;
    const size_t row = (tokh + (size_t)min(t, ci.len - 1) * H) * M + g4;   // clamped; nothing is stored past len
    f32x4 ds[MI], p[MI], wd[MI];                             // X, later ds; z, later p; dz, later scale*dz
    typename Atom<T>::Frag16 fa[CI], fav[CI], favlo[CI];                // (q_t . k_r) and (dO_t . v_r), masked: operands of contractions over t
    BlockGates<M, GEN> bg;
    const bool given = GEN && a.sin != nullptr;   // write intensities are an input of their own
    bg.load(a.g + tokh * M, (size_t)H * M, ci.len, rowb, lane, given ? a.sin + tokh * M : nullptr, GEN ? a.gate_tau : 0.f);
    __builtin_amdgcn_sched_barrier(0);
    // ---- phase 1: contractions over the head dimension (see StepTile)
    //   A[t][r] = q_t . k_r (r <= t),  X[r][i] = <E[i], [k_r | v_r]>,  carry[i] = <E[i], S_end[i]>
    // Wave w keeps the tiles of its own tokens as r: A as D[t][r] for the row blocks of t from w on, X as D[slot][r].  The
    // carry is the product of two tiles of the same layout, piece by piece in the registers they arrive in: the chunk-end
    // memory does not go through LDS.
    // Non-temporal loads for what is read here for the last time (v, the chunk-end memories, and q where the wide
    // contractions run on their own); k and E are read again, by this kernel or by the apply kernel right after it.
    f32x4 dgl[MI];   // z*dz + p*dp of this lane's token
    constexpr bool kTwo = L::kTwo;
    auto gates = [&] {   // the write-intensity tile Vn is for the pair weights of other waves
        bg.template finish<T>(ci.len, rowb, lane);
        bg.template write_tiles<T>(Vn, L::ldn, nullptr, 0, Rb, rowb, lane);
    };
    auto load_scores = [&] {
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            p[ni] = *reinterpret_cast<const f32x4 *>(a.z + row + ni * 16);
            wd[ni] = *reinterpret_cast<const f32x4 *>(a.dz + row + ni * 16);
        }
    };
    {
        using Tile = StepTile<T>;
        constexpr int NT = Geo<T>::NT;
        typedef StepRows<T, C, NT, false, !WIDE> RQ;
        typedef StepRows<T, C, NT, false, false> RK;
        typedef StepRows<T, C, NT, false, true> RV;
        typedef StepRows<T, M, NT, true, false> RE;
        typedef StepRows<T, M, NT, true, true> RS;
        const RQ rq(a.q + tokh * d_k, (size_t)H * d_k, ci.len, tid);
        const RK rk(a.k + tokh * d_k, (size_t)H * d_k, ci.len, tid);
        const RV rv(a.v + tokh * d_v, (size_t)H * d_v, ci.len, tid);
        const RE rek(EK, 0, 0, tid), rev(EV, 0, 0, tid);
        const RS rsk(SendK, 0, 0, tid), rsv(SendV, 0, 0, tid);
        typename RQ::Stage sq[2];
        typename RK::Stage sk[2];
        typename RE::Stage se[2];
        typename RS::Stage ss[2];
        StepSums<T, NB> sums;   // [row blocks of t (causal) | slot blocks]
        float cpart[RE::V];   // this thread's share of the carry of its pieces' slots
#pragma unroll
        for (int v = 0; v < RE::V; ++v) cpart[v] = 0.f;
        auto add_carry = [&](const typename RE::Stage &e, const typename RS::Stage &s) {
#pragma unroll
            for (int v = 0; v < RE::V; ++v)
#pragma unroll
                for (int j = 0; j < Tile::PV; ++j) cpart[v] += to_f32(e.x[v][j]) * to_f32(s.x[v][j]);
        };
        const int nk = d_k / Tile::KS, nv = d_v / Tile::KS;
        unsigned char *buf = smem + L::oMat;
        auto fetch_k = [&](auto u, int step) {
            constexpr int U = decltype(u)::value;
            rq.fetch(sq[U], step);
            rk.fetch(sk[U], step);
            rek.fetch(se[U], step);
            rsk.fetch(ss[U], step);
        };
        fetch_k(std::integral_constant<int, 0>{}, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kTwo) fetch_k(std::integral_constant<int, 1>{}, min(1, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kTwo) {
            gates();   // while the first operands are on their way
            __builtin_amdgcn_sched_barrier(0);
        }
        // key half: A = Q K^T, X += K E_k^T
        walk_steps<kTwo>(
            nk, fetch_k,
            [&](auto u, int step) {
                constexpr int U = decltype(u)::value;
                unsigned char *at = buf + U * L::szBuf;
                if (step < nk) add_carry(se[U], ss[U]);
                rq.template put<PHI>(reinterpret_cast<T *>(at), sq[U], tid);
                rk.template put<PHI>(reinterpret_cast<T *>(at + L::oK), sk[U], tid);
                rek.put(reinterpret_cast<T *>(at + L::oE), se[U], tid);
            },
            [&](int b) {
                f32x4(&acc)[NB] = sums.step();
                const T *Q = reinterpret_cast<const T *>(buf + b * L::szBuf), *K = reinterpret_cast<const T *>(buf + b * L::szBuf + L::oK);
                const T *E = reinterpret_cast<const T *>(buf + b * L::szBuf + L::oE);
#pragma unroll
                for (int f = 0; f < Tile::F; ++f) {
                    const typename Atom<T>::Frag x = Tile::frag(K, rowb, f, lane);
#pragma unroll
                    for (int ni = 0; ni < MI; ++ni) Atom<T>::mma(acc[CI + ni], Tile::frag(E, 16 * ni, f, lane), x);
#pragma unroll
                    for (int cb = 0; cb < CI; ++cb)
                        if (cb >= w) Atom<T>::mma(acc[cb], Tile::frag(Q, 16 * cb, f, lane), x);   // wave-uniform
                }
                sums.done();
            });
        if constexpr (kTwo) {
            load_scores();   // land during the value half
            __builtin_amdgcn_sched_barrier(0);
        }
        // value half: X += V E_v^T
        typename RV::Stage sv[2];
        auto fetch_v = [&](auto u, int step) {
            constexpr int U = decltype(u)::value;
            rv.fetch(sv[U], step);
            rev.fetch(se[U], step);
            rsv.fetch(ss[U], step);
        };
        fetch_v(std::integral_constant<int, 0>{}, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kTwo) fetch_v(std::integral_constant<int, 1>{}, min(1, nv - 1));
        __builtin_amdgcn_sched_barrier(0);
        walk_steps<kTwo>(
            nv, fetch_v,
            [&](auto u, int step) {
                constexpr int U = decltype(u)::value;
                unsigned char *at = buf + U * L::szBuf;
                if (step < nv) add_carry(se[U], ss[U]);
                rv.template put<PHI>(reinterpret_cast<T *>(at + L::oK), sv[U], tid);
                rev.put(reinterpret_cast<T *>(at + L::oE), se[U], tid);
            },
            [&](int b) {
                f32x4(&acc)[NB] = sums.step();
                const T *V = reinterpret_cast<const T *>(buf + b * L::szBuf + L::oK), *E = reinterpret_cast<const T *>(buf + b * L::szBuf + L::oE);
#pragma unroll
                for (int f = 0; f < Tile::F; ++f) {
                    const typename Atom<T>::Frag x = Tile::frag(V, rowb, f, lane);
#pragma unroll
                    for (int ni = 0; ni < MI; ++ni) Atom<T>::mma(acc[CI + ni], Tile::frag(E, 16 * ni, f, lane), x);
                }
                sums.done();
            });
#pragma unroll
        for (int v = 0; v < RE::V; ++v) {   // eight neighbouring threads hold the pieces of one slot
            float x = cpart[v];
            x += __shfl_xor(x, 1, 64);
            x += __shfl_xor(x, 2, 64);
            x += __shfl_xor(x, 4, 64);
            const int idx = tid + v * NT;
            if (idx % Tile::PR == 0 && idx < RE::N) carry[idx / Tile::PR] = x;   // read behind the barrier of phase 2e
        }
#pragma unroll
        for (int b = 0; b < CI; ++b) {
            f32x4 x = sums.sum[b];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = (b > w || (b == w && g4 + j >= r)) ? x[j] : 0.f;
            fa[b] = to_frag16<T>(x);
        }
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) ds[ni] = sums.sum[CI + ni];
    }
    // what the rest of phase 2 needs from global memory
    if constexpr (!kTwo) {
        load_scores();
        gates();
    }
#pragma unroll
    for (int b = 0; b < CI; ++b) {
        const size_t off = (size_t)t * C + max(b, w) * 16 + g4;
        fav[b] = Atom<T>::load16(AvT + off);
        if (sizeof(T) == 2) favlo[b] = Atom<T>::load16(a.tAvLo + ch * C * C + off);
    }
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) dgl[ni] = *reinterpret_cast<const f32x4 *>(a.dgf + row + ni * 16);
    __builtin_amdgcn_sched_barrier(0);
    // ---- phase 2: p and scale*dz in D[slot][token] tiles of this wave's block.  The other waves need of them the tiles
    // U = (scale*dz | p) * exp(L_t - ref) for ds.
    // ref lies halfway down the block's decay, so that neither U nor exp(ref - L_r) leaves fp32's range by
    // more than e^40; a kPairs block is referenced to its start, which serves the earlier blocks, and its own pairs are
    // evaluated one by one.
    const bool unsafe = bg.kind == kPairs;
    if (!GEN || a.readout == kReadSoftmax) {
        softmax_slots<M>(p);
    } else {
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) p[ni][j] = readout_value(a.readout, p[ni][j]);
    }
    const float half = unsafe ? 0.f : 0.5f;   // ref = half * tot
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        f32x4 rd, rr;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[ni][j] = live ? p[ni][j] : 0.f;
            wd[ni][j] = live ? scale * wd[ni][j] : 0.f;
            const float ref = half * bg.tot[ni][j], e = __expf(bg.L[ni][j] - ref);
            const int i = ni * 16 + g4 + j;
            Ud[i * L::ldt + t] = from_f32<T>(wd[ni][j] * e);
            Up[i * L::ldt + t] = from_f32<T>(p[ni][j] * e);
            rd[j] = __expf(bg.tot[ni][j] - ref);
            rr[j] = __expf(ref);
        }
        if (r == 0) {
            *reinterpret_cast<f32x4 *>(Rd + w * M + ni * 16 + g4) = rd;
            *reinterpret_cast<f32x4 *>(Rr + w * M + ni * 16 + g4) = rr;
        }
    }
    // (the rests of the products lie where Bm^T goes below: every wave has its own before any wave writes)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __syncthreads();
    // ---- phase 2a: ds for the tokens r of block w: the sum over later tokens walks from the chunk's end (where
    // it is the inter-chunk term) to the start of each block, ds <- ds * exp(tot) + U_b A_b
#pragma unroll
    for (int b = CI - 1; b >= 0; --b) {
        if (b < w || (b == w && unsafe)) continue;   // wave-uniform
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            ds[ni] *= *reinterpret_cast<const f32x4 *>(Rd + b * M + ni * 16 + g4);
            Atom<T>::mma16(ds[ni], Atom<T>::load16(Ud + (ni * 16 + r) * L::ldt + b * 16 + g4), fa[b]);
            const typename Atom<T>::Frag16 up = Atom<T>::load16(Up + (ni * 16 + r) * L::ldt + b * 16 + g4);
            Atom<T>::mma16(ds[ni], up, fav[b]);
            if (sizeof(T) == 2) Atom<T>::mma16(ds[ni], up, favlo[b]);
            if (b > w) ds[ni] *= *reinterpret_cast<const f32x4 *>(Rr + b * M + ni * 16 + g4);
        }
    }
#pragma unroll
    for (int ni = 0; ni < MI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) ds[ni][j] *= __expf((unsafe ? 1.f : 0.5f) * bg.tot[ni][j] - bg.L[ni][j]);
    f32x4 exb = {0.f, 0.f, 0.f, 0.f}, exa = {0.f, 0.f, 0.f, 0.f};   // diagonal pair weights of a block that is not kNarrow
    if (unsafe) {
        typename Atom<T>::Frag16 ownA = fa[0], ownAv = fav[0], ownLo = favlo[0];
#pragma unroll
        for (int b = 0; b < CI; ++b)
            if (b == w) { ownA = fa[b]; ownAv = fav[b]; ownLo = favlo[b]; }
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int tt = 4 * q + c, src = (lane & 48) | tt;
                const float x = __shfl(to_f32(ownA[c]), 16 * q + r, 64), y = __shfl(sizeof(T) == 2 ? to_f32(ownAv[c]) + to_f32(ownLo[c]) : to_f32(ownAv[c]), 16 * q + r, 64);   // zero for t < r
#pragma unroll
                for (int ni = 0; ni < MI; ++ni)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float Lt = __shfl(bg.L[ni][j], src, 64);
                        const float d = __shfl(wd[ni][j], src, 64), pt = __shfl(p[ni][j], src, 64);
                        ds[ni][j] += (x * d + y * pt) * __expf(fminf(Lt - bg.L[ni][j], 0.f));
                    }
            }
        exb = pair_tile_exact<M, GEN>(wd, bg, lane);
        exa = pair_tile_exact<M, GEN>(p, bg, lane);
    }
    if (bg.kind == kHalf) {
        for (int u = 0; u < 2; ++u) {   // one body for both: two of them cost registers (three spilled at m = 64)
            f32x4 wt[MI];
#pragma unroll
            for (int ni = 0; ni < MI; ++ni) wt[ni] = u ? p[ni] : wd[ni];
            const f32x4 x = pair_tile_half<T, M, GEN>(wt, bg, lane);
            if (u) exa = x;
            else exb = x;
        }
    }
    // ---- phase 2b: the gate gradient inside the block, and the block's total for the earlier ones
    f32x4 dg[MI];
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        f32x4 sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float x = live ? dgl[ni][j] - bg.s[ni][j] * ds[ni][j] : 0.f;
            sum[j] = row16_suffix_sum(x);
            // tied: d(1 - e^g)/dg = -e^g = -(1 - s)
            dg[ni][j] = given ? sum[j] : sum[j] - (1.f - bg.s[ni][j]) * ds[ni][j];
        }
        if (r == 0) *reinterpret_cast<f32x4 *>(Tot + w * M + ni * 16 + g4) = sum;
        if (GEN && given && live) *reinterpret_cast<f32x4 *>(a.ds + row + ni * 16) = ds[ni];
    }
    // ---- phase 2c: the slot-side operand of dk and dv, s*exp(G_C - G)
    // (the five small matrices stay in LDS when the wide contractions follow here)
    T *mB = a.tB + ch * C * C, *mBT = a.tBT + ch * C * C, *mA2T = a.tA2T + ch * C * C, *mD = a.tDZe + ch * C * KM, *mS = a.tSbe + ch * C * KM;
    if constexpr (WIDE) {
        mB = reinterpret_cast<T *>(smem + L::oMat);
        mBT = mB + C * C;
        mA2T = mBT + C * C;
        mD = mA2T + C * C;
        mS = mD + C * KM;
    }
    typedef Wide<M> W;
    auto tok_at = [](int row, int col) { return WIDE ? W::template at<C>(row, col) : row * C + col; };
    auto slot_at = [](int row, int col) { return WIDE ? W::template at<KM>(row, col) : row * KM + col; };
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        f32x4 y;
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = bg.s[ni][j] * __expf(bg.tot[ni][j] - bg.L[ni][j]);
#pragma unroll
        for (int b = 1; b < CI; ++b)
            if (b > w) y *= *reinterpret_cast<const f32x4 *>(Rb + b * M + ni * 16 + g4);
        store_frag16<T>(mS + slot_at(t, ni * 16 + g4), y);
    }
    if (M < KM) store_frag16<T>(mS + slot_at(t, M + g4), f32x4{0.f, 0.f, 0.f, 0.f});   // the padded slot columns
    typename W::Stage sa, sb;
    const int nk = d_k / 64, units = 2 * nk + d_v / 64;
    const T *const SK = a.S + ch * a.lay.stride + a.lay.oK;
    const T *const tk0 = a.k + tokh * d_k, *const tk1 = a.q + tokh * d_k, *const tk2 = a.dO + tokh * d_v;
    T *const to0 = a.dq + tokh * d_k, *const to1 = a.dk + tokh * d_k, *const to2 = a.dv + tokh * d_v;
    auto unit = [=](int i) {   // i is uniform over the workgroup
        const bool isq = i < nk, isv = i >= 2 * nk;
        const int c = 64 * (isq ? i : isv ? i - 2 * nk : i - nk), d = isv ? d_v : d_k;
        const T *slot = pick(isq, SK, pick(isv, EV, EK)), *tok = pick(isq, tk0, pick(isv, tk2, tk1));
        T *out = pick(isq, to0, pick(isv, to2, to1));
        return typename W::Unit{(const bf16_t *)(slot + (size_t)c * M), (const bf16_t *)(tok + c), (bf16_t *)(out + c), (size_t)H * d,
                                (const bf16_t *)pick(isq, mB, pick(isv, mA2T, mBT)), (const bf16_t *)pick(isq, mD, mS)};
    };
    if constexpr (WIDE) {   // the first two units' tiles land during the rest of phase 2
        W::fetch(sa, unit(0), ci.len, tid);
        W::fetch(sb, unit(1), ci.len, tid);
    }
    // ---- phase 2d: Bm (both orientations) and A2^T, row t of this wave's block, one column block after the
    // other as in the forward; `wd` ends as the slot-side operand of dq, scale*dz*exp(G)
#pragma unroll
    for (int ni = 0; ni < MI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float e = bg.walk_gate(ni, j);
            wd[ni][j] *= e;
            p[ni][j] *= e;
        }
#pragma unroll
    for (int b = CI - 1; b >= 0; --b) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 xb = zero, xbt = zero, xat = zero;   // D[r][t]; D[t][r]
        if (b == w && bg.kind != kNarrow) {   // weights are already at the start of the block
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mBT[tok_at(b * 16 + g4 + j, t)] = from_f32<T>(exb[j]);
                mA2T[tok_at(b * 16 + g4 + j, t)] = from_f32<T>(exa[j]);
            }
            store_frag16<T>(mB + tok_at(t, b * 16 + g4), exb);
            continue;
        }
        if (b <= w) {   // wave-uniform
            pair_tiles<T, M>(wd, p, Vn, L::ldn, b, lane, xb, xbt, xat);
#pragma unroll
            for (int ni = 0; ni < MI; ++ni) {
                const f32x4 e = *reinterpret_cast<const f32x4 *>(Rb + b * M + ni * 16 + g4);
                wd[ni] *= e;
                p[ni] *= e;
            }
            if (b == w) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xb[j] = g4 + j <= r ? xb[j] : 0.f;
                    xbt[j] = g4 + j >= r ? xbt[j] : 0.f;
                    xat[j] = g4 + j >= r ? xat[j] : 0.f;
                }
            }
        }
        store_frag16<T>(mB + tok_at(t, b * 16 + g4), xb);
        store_frag16<T>(mBT + tok_at(b * 16 + r, rowb + g4), xbt);
        store_frag16<T>(mA2T + tok_at(b * 16 + r, rowb + g4), xat);
    }
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) store_frag16<T>(mD + slot_at(t, ni * 16 + g4), wd[ni]);
    if (M < KM) store_frag16<T>(mD + slot_at(t, M + g4), f32x4{0.f, 0.f, 0.f, 0.f});
    // ---- phase 2e: dg = (suffix sum of dGam inside the chunk) + carry - exp(g) ds
    __syncthreads();   // the other blocks' totals
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        f32x4 off = *reinterpret_cast<const f32x4 *>(carry + ni * 16 + g4);
#pragma unroll
        for (int b = 1; b < CI; ++b)
            if (b > w) off += *reinterpret_cast<const f32x4 *>(Tot + b * M + ni * 16 + g4);
        f32x4 x = dg[ni] + off;
        if (GEN && a.gate_tau > 0.f) {   // gate logits in g: the gradient goes on to the logit
            const f32x4 u = *reinterpret_cast<const f32x4 *>(a.g + row + ni * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] *= log_gate_slope(u[j], a.gate_tau);
        }
        if (live) *reinterpret_cast<f32x4 *>(a.dg + row + ni * 16) = x;
    }
    // ---- phase 3: dq, dk, dv (B=8, T=2048, H=4, d=512, m=64: 131 us and a kernel of its own of 102 us -> 200 us)
    if constexpr (WIDE) {
        if (ci.len == C) W::template walk<true>(unit, units, sa, sb, smem, smem + L::oEx, ci.len, tid);
        else W::template walk<false>(unit, units, sa, sb, smem, smem + L::oEx, ci.len, tid);
    }
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
template <typename T, int M>
static hipError_t launch_bwd_tm(const Plan &pl, const Work &w, const void *q, const void *k, const void *v,
                                const float *g, const float *K0, const float *V0, const float *z, const void *dO,
                                const float *dKT, const float *dVT, void *dq, void *dk, void *dv, float *dg,
                                float *dK0, float *dV0, hipStream_t st)
{
    const ChunkMap cm = make_chunk_map(pl, w);
    // 1. recompute the chunk-start memories (and the memories after the last token), unless the forward
    // call left them in this workspace (Section 4, "Efficiency": the kernel without recomputation)
    if (!pl.keep) {
        GSA_HIP_TRY(launch_gates(pl, w, g, pl.s_in, pl.gate_tau, st));
        const ScanIo io = {k, v, K0, V0, nullptr, nullptr, w.SF, false, pl.phi != 0, pl.phi != 0};
        GSA_HIP_TRY(launch_scan(pl, w, io, st));
    }
    dim3 grid(pl.chunk_slots, pl.H);
    // 2. dp, dz and the weights of the reverse scan
    {
        auto kern = !pl.general() ? chunk_dz_kernel<T, M, false, false>
                    : pl.phi     ? chunk_dz_kernel<T, M, true, true>
                                 : chunk_dz_kernel<T, M, true, false>;
        const size_t lds = DzLds<T, M>::bytes;
        GSA_HIP_TRY(allow_lds(kern, lds));
        KernelTimer kt(kSlotChunkDz, st);
        hipLaunchKernelGGL(kern, grid, dim3(Geo<T>::NT), lds, st, cm, pl.H, pl.d_v, pl.scale, (const T *)v,
                           (const T *)dO, g, z, (const T *)w.S, pl.lay, w.dz, w.dgf, (T *)w.Wr, (T *)w.tAvT,
                           (T *)w.tBT, pl.s_in,
                           pl.opts(), pl.gate_tau);
        GSA_HIP_TRY(hipGetLastError());
    }
    // 3. reverse scan of the memory gradient
    {
        const ScanIo io = {q, dO, dKT, dVT, dK0, dV0, nullptr, true, pl.phi != 0, false};
        GSA_HIP_TRY(launch_scan(pl, w, io, st));
    }
    // 4. everything chunk-local, and in bf16 without the feature map the wide contractions as well.  One workgroup
    // then walks all 64-column units of its (chunk, head), which takes longer than a kernel of its own where few
    // pairs are left to fill the chip.  Time of the backward call with them inside over that without, 64 slots: d = 512 (24
    // units) 1.18 at 8 pairs, 1.08 at 64, 1.02 at 96, 0.94 at 256, 0.92 from 1024 on; d = 1024 (48 units) 1.30, 1.13, 1.08,
    // 0.98, 0.96; d = 128 (6 units) 0.97, 0.95, 0.96, 0.92, 0.90.  With 128 slots 1 to 4 per cent lower throughout (one
    // workgroup per CU holds the 125.5 KB, the kernel it replaces reads everything again); with 16 and 32 slots the same up to
    // d = 512 and 0.96 to 1.04 above.
    const int64_t pairs = (int64_t)pl.chunk_slots * pl.H;
    const bool wide = sizeof(T) == 2 && !pl.phi && pairs >= 4 * (2 * pl.d_k + pl.d_v) / 64;
    {
        constexpr bool kWide = sizeof(T) == 2;
        auto kern = pl.phi          ? chunk_intra_kernel<T, M, true, true, false>
                    : pl.general() ? (wide ? chunk_intra_kernel<T, M, true, false, kWide> : chunk_intra_kernel<T, M, true, false, false>)
                                   : (wide ? chunk_intra_kernel<T, M, false, false, kWide> : chunk_intra_kernel<T, M, false, false, false>);
        const size_t lds = wide ? IntraLds<T, M, sizeof(T) == 2>::bytes : IntraLds<T, M, false>::bytes;
        GSA_HIP_TRY(allow_lds(kern, lds));
        IntraArgs<T> a;
        a.q = (const T *)q; a.k = (const T *)k; a.v = (const T *)v;
        a.g = g; a.z = z; a.dz = w.dz; a.dgf = w.dgf;
        a.S = (const T *)w.S; a.SF = (const T *)w.SF; a.E = (const T *)w.E;
        a.lay = pl.lay;
        a.tAvT = (const T *)w.tAvT;
        a.tAvLo = (const T *)w.tBT;
        a.dO = (const T *)dO;
        a.dq = (T *)dq; a.dk = (T *)dk; a.dv = (T *)dv;
        a.dg = dg;
        a.tB = (T *)w.tA; a.tBT = (T *)w.tBT; a.tA2T = (T *)w.tA2T; a.tDZe = (T *)w.tP; a.tSbe = (T *)w.tSbe;
        a.sin = pl.s_in; a.ds = pl.ds_out; a.readout = pl.readout; a.gate_tau = pl.gate_tau;
        KernelTimer kt(kSlotChunkIntra, st);
        hipLaunchKernelGGL(kern, grid, dim3(Geo<T>::NT), lds, st, cm, pl.H, pl.d_k, pl.d_v, pl.scale, a);
        GSA_HIP_TRY(hipGetLastError());
    }
    if (wide) return hipSuccess;
    // 5. dq, dk, dv (with the feature map: through its slope at the raw q, k, v)
    const bool phi = pl.phi != 0;
    const ApplyIo io[3] = {
        {w.tA, w.tP, k, w.S, pl.lay.oK, pl.lay.stride, dq, pl.d_k, phi, phi ? q : nullptr},
        {w.tBT, w.tSbe, q, w.E, pl.lay.oK, pl.lay.stride, dk, pl.d_k, phi, phi ? k : nullptr},
        {w.tA2T, w.tSbe, dO, w.E, pl.lay.oV, pl.lay.stride, dv, pl.d_v, false, phi ? v : nullptr},
    };
    return launch_apply(pl, w, io, 3, kSlotApplyBwd, st);
}

template <typename T>
static hipError_t launch_bwd_t(const Plan &pl, const Work &w, const void *q, const void *k, const void *v,
                               const float *g, const float *K0, const float *V0, const float *z, const void *dO,
                               const float *dKT, const float *dVT, void *dq, void *dk, void *dv, float *dg, float *dK0,
                               float *dV0, hipStream_t st)
{
    switch (pl.m) {
    case 16: return launch_bwd_tm<T, 16>(pl, w, q, k, v, g, K0, V0, z, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
    case 32: return launch_bwd_tm<T, 32>(pl, w, q, k, v, g, K0, V0, z, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
    case 128: return launch_bwd_tm<T, 128>(pl, w, q, k, v, g, K0, V0, z, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
    default: return launch_bwd_tm<T, 64>(pl, w, q, k, v, g, K0, V0, z, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
    }
}

hipError_t launch_bwd(const Plan &pl, const Work &w, const void *q, const void *k, const void *v, const float *g,
                      const float *K0, const float *V0, const float *z_saved, const void *dO, const float *dKT,
                      const float *dVT, void *dq, void *dk, void *dv, float *dg, float *dK0, float *dV0,
                      hipStream_t st)
{
    if (pl.tokens == 0) return hipSuccess;
    if (!pl.keep) GSA_HIP_TRY(launch_prepare(pl, w, st));
    if (pl.dtype == 0)
        return launch_bwd_t<float>(pl, w, q, k, v, g, K0, V0, z_saved, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
    return launch_bwd_t<bf16_t>(pl, w, q, k, v, g, K0, V0, z_saved, dO, dKT, dVT, dq, dk, dv, dg, dK0, dV0, st);
}

}  // namespace gsa
