// The sequential part of Gated Slot Attention: carrying the joint slot memory S = [Kt | Vt]
// (forward) and its gradient E (backward) across chunks (paper, Appendix A,
// Eq. (gla-chunk-gate); Algorithm 1, the two "for n" loops).
//
// Both recurrences have the same shape,
//     acc <- Diag(dec_n) acc + W_n X_n          W_n [m x C] gate-weighted, X_n [C x columns]
// with a snapshot of acc taken BEFORE the update of chunk n.  Forward: W = s*exp(G_C-G),
// X = [k | v], snapshots = memory at chunk start.  Reverse: W = scale*dz*exp(G) (key
// columns) or p*exp(G) (value columns), X = [q | dO], snapshots = memory gradient at chunk
// end.  Nothing in W depends on acc, so the weights are produced by chunk-parallel kernels
// (gate_kernel here, chunk_dz_kernel for the reverse scan) and the sequential loop only
// copies tiles, multiplies and stores:
//
//   * one workgroup per (sequence, head, column slice); the slice of acc lives in MFMA
//     accumulators for the whole sequence;
//   * the operands of the next chunks are prefetched into registers while one is multiplied.  Every access to memory is
//     by whole lines: the weights come in fragment order (see frag_order), the token rows go through LDS as they lie
//     and are read back by the transposing LDS load, snapshots are put together in LDS;
//   * snapshots are one contiguous block per workgroup and chunk (the records are tiled by column slice for this).
//     With the chip full the launch is bound by these bytes: 8 x 2048 tokens, 4 heads, d = 512, 64 slots, 285 MB in 53 us; loads
//     and stores of this pattern alone, without arithmetic, take 43;
//   * workgroups that share (sequence, head) — and therefore W and dec — are mapped to
//     the same XCD so those re-reads hit its L2.
#include "gsa_chunk.h"
#include "gsa_launch.h"

namespace gsa {

// ---------------------------------------------------------------------------------------
// Gate weights of the forward scan (chunk-parallel).
//
// Everything stays in the registers of the thread that owns a slot's tokens; only the partial sums of the
// partitions meet in LDS.  A thread takes eight tokens, one 16-byte piece of the weights in bf16: the more waves share the
// evaluation of the gates, the better it hides its own latency.  With 256 threads whatever the slots: 128 slots, 4 x 1000
// tokens, 4 heads, 8.8 us instead of 7.0 (with the event), with gate logits 7 us more for the call; 64 slots the same.
// ---------------------------------------------------------------------------------------
template <typename T, int M> constexpr int kGateThreads = M * Geo<T>::C / 8;
template <typename T, int M, bool GEN>
__global__ __launch_bounds__((kGateThreads<T, M>)) void gate_kernel(ChunkMap cm, int H, const float *__restrict__ g,
                                                                  const float *__restrict__ sin, float gate_tau,
                                                                  T *__restrict__ Wf, float *__restrict__ dec)
{
    constexpr int C = Geo<T>::C, NT = kGateThreads<T, M>;
    typedef GatePrep<M, NT, C, GEN> Gates;
    constexpr int P = Gates::P, TP = Gates::TP;   // a thread owns one slot and TP consecutive tokens
    static_assert(TP == 8, "one operand's worth of tokens");
    __shared__ float tot[NT];
    ChunkInfo ci;
    if (!chunk_lookup(cm, blockIdx.x, ci)) return;
    const int h = blockIdx.y, tid = threadIdx.x, i = tid % M, part = tid / M;
    const size_t ch = (size_t)blockIdx.x * H + h;
    const size_t goff = ((size_t)ci.tok0 * H + h) * M;
    Gates gp;
    gp.load(g + goff, (size_t)H * M, ci.len, tid, (GEN && sin) ? sin + goff : nullptr, gate_tau);
    float x[TP], w[TP], behind[TP], own = 0.f;   // behind: decay of this thread's own later tokens
#pragma unroll
    for (int tt = TP - 1; tt >= 0; --tt) {
        gp.token(x[tt], w[tt], tt, part * TP + tt < ci.len);
        behind[tt] = own;
        own += x[tt];
    }
    tot[part * M + i] = own;
    __syncthreads();
    float after = 0.f;   // decay of the chunk behind the token: G_C - G_t
#pragma unroll
    for (int pp = P - 1; pp > 0; --pp) after += pp > part ? tot[pp * M + i] : 0.f;
    // fp32: two sums, the shorter chains of roundings (16 slots, 500 tokens: error of the memories 9.9e-8 against 10.0e-8 with one)
#pragma unroll
    for (int tt = TP - 1; tt >= 0; --tt) {
        w[tt] *= __expf(sizeof(T) == 4 ? after + behind[tt] : after);
        if (sizeof(T) != 4) after += x[tt];
    }
    if (sizeof(T) == 4) after += own;
    T *W = Wf + ch * M * C;   // in fragment order: a slot's neighbours write next to it
    if constexpr (sizeof(T) == 2) {
        store8<T>(W + frag_order<T, C / 32>(i, part * TP), w);
    } else {
        store4(W + frag_order<T, C / 32>(i, part * TP), w[0], w[1], w[2], w[3]);
        store4(W + frag_order<T, C / 32>(i, part * TP + 4), w[4], w[5], w[6], w[7]);
    }
    if (part == 0) dec[ch * M + i] = __expf(after);
}

// ---------------------------------------------------------------------------------------
// The scan.
// ---------------------------------------------------------------------------------------
template <typename T> struct ScanArgs {
    const T *W;            // [chunk][H][parts], [M][C] in fragment order
    int w_parts;           // 1 (forward) or 2 (reverse: key part, value part)
    const float *dec;      // [chunk][H][M]
    const T *xk, *xv;      // token tensors feeding the key / value columns
    bool phi_k, phi_v;     // feature map on xk / xv on their way into LDS
    const float *initK, *initV;   // [n_seqs][H][M][d] or NULL
    T *snap;               // one record per (chunk, head)
    StateLayout lay;       // layout of every record
    float *outK, *outV;    // [n_seqs][H][M][d] or NULL: acc after the last chunk
    T *outJ;               // one record per (sequence, head), or NULL: the same, element type T
    // long sequences cut into segments (modes 1 and 2 of the kernel):
    int seg_chunks;        // chunks per segment (packed: as the prepare kernel decided, behind seg_base)
    int max_seg;           // segments per sequence the grid provides for
    float *sumY;           // [n_seqs][max_seg][H][M][d_k+d_v]   what a segment adds, from a zero start
    float *sumD;           // [n_seqs][max_seg][H][slices][M]    its total decay
};

// Shape of a scan workgroup: four waves that share out the slots (WS), then the columns (WC); a wave holds MI x NI tiles.
// (Eight waves, of two column tiles each with 64 slots, load the weights twice: 8 x 2048 tokens, 4 heads, d = 512 64 us
// against 56; 32 slots 47 against 44.)
template <typename T, int M> struct ScanGeo {
    static constexpr int C = Geo<T>::C, NS = kSnapTile, NW = 4, NT = NW * kWave;
    static constexpr int WS = M < 64 ? M / 16 : 4, WC = NW / WS, MI = M / (16 * WS), NI = NS / (16 * WC);
};

template <typename T, int M> struct ScanLds {
    using G = ScanGeo<T, M>;
    // Per parity of the chunk's position in the walk, one written while the other is read: the token tile [C][NS] as it lies
    // in memory (TokRows), and the snapshot tile, which leaves in whole lines one step later, behind the step's barrier.
    // (Straight from the registers a store takes 16 bytes or 32 of each of many lines: d = 512, 64 slots, 512 workgroups 62 us
    // against 57; 32 slots 57 against 47; 128 workgroups 31 against 30.)
    static constexpr size_t szX = sizeof(T) * G::C * G::NS;
    static constexpr int ldx = G::NS + Atom<T>::kPad;
    static constexpr size_t oSn = szX, szSn = sizeof(T) * M * ldx;
    static constexpr size_t set = oSn + szSn, bytes = 2 * set;
};

// Matrix-core operands from a token tile that lies in LDS as it lies in memory ([token][column]), and the columns they
// leave a lane with.  frags: the A operands X^T of one depth-32 step for a wave's NI column tiles; after the product, a
// lane's accumulators hold 4*NI consecutive columns from 4*NI*(l/16) on, group g of four by get / set.
//   bf16: the transposing LDS load hands a lane four tokens of one column; which columns is the lane's choice.
//   fp32: there is no such load for 32 bits, and none is needed: a lane's NI tiles are dealt NI consecutive columns of a row.
template <typename T, int NS, int NI> struct TokRows;
template <int NS, int NI> struct TokRows<bf16_t, NS, NI> {
    static_assert(NS == TrTile<NI>::kCols && (NI == 1 || NI == 2 || NI == 4), "columns per lane");
    typedef bf16x8 Piece;   // 16 bytes of one row
    __device__ static __forceinline__ void put(bf16_t *X, int row, int p, const Piece &x) { TrTile<NI>::put(X, row, p, x); }
    uint32_t off[NI];   // where this lane reads, per column tile
    __device__ __forceinline__ TokRows(int wcol, int lane)
    {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) off[ni] = TrTile<NI>::lane_off((wcol >> 2) + NI * (lane & 3) + ni, lane);
    }
    __device__ __forceinline__ void frags(bf16x8 (&f)[NI], const bf16_t *X, int k0) const
    {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) f[ni] = TrTile<NI>::frag(X + k0 * NS + off[ni]);
    }
    __device__ static __forceinline__ f32x4 get(const f32x4 (&acc)[NI], int g) { return acc[g]; }
    __device__ static __forceinline__ void set(f32x4 (&acc)[NI], int g, const f32x4 &x) { acc[g] = x; }
};
template <int NS, int NI> struct TokRows<float, NS, NI> {
    static_assert(NI == 1 || NI == 2 || NI == 4, "columns per lane");
    typedef f32x4 Piece;
    __device__ static __forceinline__ void put(float *X, int row, int p, const Piece &x) { *reinterpret_cast<f32x4 *>(X + row * NS + p * 4) = x; }
    uint32_t off;
    __device__ __forceinline__ TokRows(int wcol, int lane) : off(8 * (lane >> 4) * NS + wcol + NI * (lane & 15)) {}
    __device__ __forceinline__ void frags(f32x8 (&f)[NI], const float *X, int k0) const
    {
        typedef float vec __attribute__((ext_vector_type(NI)));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const vec x = *reinterpret_cast<const vec *>(X + (k0 + e) * NS + off);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) f[ni][e] = x[ni];
        }
    }
    // matrix row rho = 4*(l/16) + j of tile ni is column NI*rho + ni
    __device__ static __forceinline__ f32x4 get(const f32x4 (&acc)[NI], int g)
    {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = acc[(4 * g + e) % NI][(4 * g + e) / NI];
        return x;
    }
    __device__ static __forceinline__ void set(f32x4 (&acc)[NI], int g, const f32x4 &x)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[(4 * g + e) % NI][(4 * g + e) / NI] = x[e];
    }
};

// MODE 0: one workgroup walks a whole sequence.  A sequence of many chunks leaves the chip waiting on
// that one chain, so long sequences are cut into segments of seg_chunks chunks and walked in two
// launches: MODE 1 walks every segment but the last of the walk from a zero start, without snapshots,
// and leaves what the segment adds (sumY) and its total decay (sumD); MODE 2 walks every segment for
// real, starting from the memory its predecessors leave behind, which it gets by running the
// recurrence over their summaries (at most max_seg - 1 steps of an element-wise update).
//
// AHEAD: chunks whose loads are in flight while one multiplies (the rule stands at the launch).
template <typename T, int M, bool REVERSE, int MODE, int AHEAD>
__global__ __launch_bounds__((ScanGeo<T, M>::NT), 2) void scan_kernel(ChunkMap cm, int H, int d_k, int d_v,
                                                                                    int n_seqs, ScanArgs<T> a)
{
    using L = ScanLds<T, M>;
    using G = ScanGeo<T, M>;
    constexpr int C = G::C, NS = G::NS, NT = G::NT, MI = G::MI, NI = G::NI;
    using R = TokRows<T, NS, NI>;
    typedef typename R::Piece Piece;
    constexpr int PV = 16 / sizeof(T), PR = NS / PV, XV = C * PR / NT;   // elements per piece, pieces per row, pieces per thread
    static_assert(XV * NT == C * PR && NT % PR == 0, "whole pieces per thread, all in one column group");
    extern __shared__ __align__(16) unsigned char smem[];
    auto XT = [&](int b) { return reinterpret_cast<T *>(smem + b * L::set); };

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15;
    const int D = d_k + d_v;
    const int nsl = D / NS;
    // XCD-aware placement: consecutive workgroup ids go round-robin over the 8 XCDs.  The slices of one
    // (sequence, head, segment) share W and dec, so a whole group of slices is put on one XCD (one L2),
    // and successive groups on successive XCDs (the segments of a long sequence, of which a packed
    // batch may hold few, then spread over the whole chip).
    const int nseg_grid = (MODE == 0) ? 1 : a.max_seg;
    const int ngroups = H * n_seqs * nseg_grid;
    int slice, group;
    if ((ngroups & 7) == 0) {
        const int x = blockIdx.x & 7, t = blockIdx.x >> 3;
        slice = t % nsl;
        group = (t / nsl) * 8 + x;
    } else {
        slice = blockIdx.x % nsl;
        group = blockIdx.x / nsl;
    }
    // A group is (segment of a sequence, head), heads fastest.  The segments are numbered densely,
    // sequence after sequence; a packed batch has fewer of them than the grid provides for (their
    // number is only known on the device), and the surplus sits at the end of the numbering, so the
    // real ones are spread evenly over the XCDs.
    const int h = group % H, dense = group / H;
    int s, seg;
    if (MODE == 0) {
        s = dense; seg = 0;
    } else if (cm.seg_base) {
        if (dense >= cm.seg_base[n_seqs]) return;   // uniform over the workgroup
        int lo = 0, hi = n_seqs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (cm.seg_base[mid] <= dense) lo = mid; else hi = mid - 1;
        }
        s = lo; seg = dense - cm.seg_base[lo];
    } else {
        s = dense / nseg_grid; seg = dense % nseg_grid;
    }
    const int col0 = slice * NS;
    const bool isK = col0 < d_k;
    const T *src = isK ? a.xk : a.xv;
    const bool phi = isK ? a.phi_k : a.phi_v;
    const int dsrc = isK ? d_k : d_v;
    const int c0 = isK ? col0 : col0 - d_k;
    const size_t wpart = (a.w_parts == 2 && !isK) ? (size_t)M * C : 0;

    int chunk0, nch_seq, tok0, ntok;
    seq_lookup(cm, s, chunk0, nch_seq, tok0, ntok);
    // acc[mi]: slot slot0 + 16*mi, columns lcol + 4*g .. +3 of the slice in group g
    const int slot0 = (wave % G::WS) * MI * 16 + r, wcol = (wave / G::WS) * 16 * NI, lcol = wcol + (lane >> 4) * 4 * NI;
    const R rows_of(wcol, lane);
    // the chunks this workgroup walks: [first, first + nch) of the sequence
    int first = 0, nch = nch_seq, nseg = 1;
    if (MODE != 0) {
        const int seg_chunks = cm.seg_base ? cm.seg_base[n_seqs + 1] : a.seg_chunks;
        nseg = max(1, (nch_seq + seg_chunks - 1) / seg_chunks);
        first = seg * seg_chunks;
        nch = min(seg_chunks, nch_seq - first);
        const int last_of_walk = REVERSE ? 0 : nseg - 1;
        if (seg >= nseg || (MODE == 1 && seg == last_of_walk)) return;   // uniform over the workgroup
        if (nch_seq == 0) nch = 0;   // a sequence without tokens still hands its initial memory through (MODE 2)
    }
    const bool starts_walk = (MODE == 0) || seg == (REVERSE ? nseg - 1 : 0);
    const bool ends_walk = (MODE == 0) || seg == (REVERSE ? 0 : nseg - 1);

    f32x4 acc[MI][NI];
    {
        const float *S0 = isK ? a.initK : a.initV;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int g = 0; g < NI; ++g) {
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                R::set(acc[mi], g, (MODE != 1 && S0) ? *reinterpret_cast<const f32x4 *>(
                                                           S0 + (((size_t)s * H + h) * M + slot0 + 16 * mi) * dsrc + c0 + lcol + 4 * g)
                                                     : zero);
            }
        if (MODE == 2 && !starts_walk) {
            // the memory at the start of this segment: the recurrence over the summaries of the segments
            // walked before it, acc <- Diag(sumD) acc + sumY, in walk order
            const int npre = REVERSE ? nseg - 1 - seg : seg;
#pragma unroll 2
            for (int u = 0; u < npre; ++u) {
                const int sg = REVERSE ? nseg - 1 - u : u;
                const size_t rec = ((size_t)s * a.max_seg + sg) * H + h;
                const float *Y = a.sumY + rec * M * D + col0;
                const float *Dd = a.sumD + (rec * nsl + slice) * M;
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) {
                    const float dd = Dd[slot0 + 16 * mi];
#pragma unroll
                    for (int g = 0; g < NI; ++g)
                        R::set(acc[mi], g, dd * R::get(acc[mi], g) +
                                               *reinterpret_cast<const f32x4 *>(Y + (size_t)(slot0 + 16 * mi) * D + lcol + 4 * g));
                }
            }
        }
        // Let these loads land before the loop's prefetches are issued: otherwise the first use of the
        // accumulator inside the loop has to wait for "everything older", which the compiler can only
        // express as "everything", and that would drain the prefetches in every iteration.
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0) only
    }
    float dprod[MI];   // MODE 1: product of the chunk decays, slots as in acc
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) dprod[mi] = 1.f;

    // Operands of one chunk, in registers: the weights are matrix-core operands as they lie in memory, the token rows wait
    // there for their turn in LDS.  The loads of AHEAD chunks are in flight while one multiplies: a step takes a
    // fraction of the memory latency, and the chain over the chunks is the only sequential part of the method.
    struct Weights {
        typename Atom<T>::Frag w[C / 32][MI];
        float dec[MI];
    };
    struct Tokens {
        Piece x[XV];
        int len;
    };
    // Bases are uniform and advance from chunk to chunk, lanes add 32-bit byte offsets.  Positions past the end of the walk
    // repeat the last chunk, so that refills can be issued unconditionally (a refill under a branch makes the number of
    // loads in flight unknown to the compiler, which then waits for all of them wherever it needs one).
    const int n0 = first + (REVERSE ? nch - 1 : 0);   // first chunk of the walk
    constexpr int dir = REVERSE ? -1 : 1;
    const int64_t dW = (int64_t)dir * H * a.w_parts * (M * C * (int)sizeof(T)), dD = (int64_t)dir * H * (M * (int)sizeof(float));
    const int64_t dX = (int64_t)dir * C * H * dsrc * (int)sizeof(T), dS = dir * (int64_t)H * a.lay.stride;
    const size_t ch0 = (size_t)(chunk0 + n0) * H + h;
    const char *wp = reinterpret_cast<const char *>(a.W + ch0 * a.w_parts * M * C + wpart), *dp = reinterpret_cast<const char *>(a.dec + ch0 * M);
    const char *xp = reinterpret_cast<const char *>(src + ((size_t)(tok0 + n0 * C) * H + h) * dsrc + c0);
    static_assert(NS == kSnapTile, "one workgroup owns one tile of the record");
    auto tile_of = [&](T *rec) { return rec + (isK ? a.lay.oK : a.lay.oV) + (size_t)(c0 / kSnapTile) * (M * kSnapTile); };   // contiguous [M][NS]
    T *sp = tile_of(a.snap + ch0 * a.lay.stride);   // where the next snapshot goes
    int wleft = nch - 1, xleft = nch - 1;   // chunks the weights and the tokens can still move on
    const uint32_t wtile = (wave % G::WS) * MI * (C / 32), doff = (uint32_t)slot0 * sizeof(float);
    const uint32_t xstep = (uint32_t)H * dsrc * sizeof(T), xcol = (tid % PR) * 16;
    auto fetch_w = [&](Weights &st) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            st.dec[mi] = *reinterpret_cast<const float *>(dp + (doff + 64 * mi));
#pragma unroll
            for (int ks = 0; ks < C / 32; ++ks)
                st.w[ks][mi] = load_frag_order(reinterpret_cast<const T *>(wp) + (wtile + mi * (C / 32) + ks) * 512, lane);
        }
        const bool more = wleft > 0;
        wp += more ? dW : 0;
        dp += more ? dD : 0;
        --wleft;
    };
    int xn = n0;
    auto fetch_x = [&](Tokens &st) {
        st.len = min(C, ntok - xn * C);
#pragma unroll
        for (int v = 0; v < XV; ++v) {
            const int row0 = min(v * (NT / PR) + wave * (kWave / PR), st.len - 1);   // uniform over the wave
            static_assert(kWave / PR <= kLaneRows, "rows of a wave");
            const uint32_t row = min(tid / PR + v * (NT / PR), st.len - 1) - row0;
            st.x[v] = __builtin_nontemporal_load(reinterpret_cast<const Piece *>(xp + (size_t)row0 * xstep + (row * xstep + xcol)));
        }
        const bool more = xleft > 0;
        xp += more ? dX : 0;
        xn += more ? dir : 0;
        --xleft;
    };
    auto tokens_to_lds = [&](const Tokens &st, int b) {
#pragma unroll
        for (int v = 0; v < XV; ++v) {
            const int row = tid / PR + v * (NT / PR);
            const f32x4 none = {0.f, 0.f, 0.f, 0.f};   // missing rows are zero
            Piece x = __builtin_bit_cast(Piece, row < st.len ? __builtin_bit_cast(f32x4, st.x[v]) : none);
            if (phi) {   // uniform over the workgroup
#pragma unroll
                for (int e = 0; e < PV; ++e) x[e] = from_f32<T>(swish_value(to_f32(x[e])));
            }
            R::put(XT(b), row, tid % PR, x);
        }
    };
    // The accumulator on its way to a record, in two halves: what a lane holds goes to the tile of a set, and from there
    // (behind a barrier) to this workgroup's tile of the record.
    auto gather = [&](int b) {
        T *X = reinterpret_cast<T *>(smem + b * L::set + L::oSn) + slot0 * L::ldx + lcol;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            if constexpr (NI == 1) {
                const f32x4 x = R::get(acc[mi], 0);
                store4(X + mi * 16 * L::ldx, x[0], x[1], x[2], x[3]);
            } else {
#pragma unroll
                for (int g = 0; g < NI; g += 2) {
                    const f32x4 x = R::get(acc[mi], g), y = R::get(acc[mi], g + 1);
                    const float v[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
                    store8<T>(X + mi * 16 * L::ldx + 4 * g, v);
                }
            }
    };
    auto send = [&](T *tile, int b) {
        const T *X = reinterpret_cast<const T *>(smem + b * L::set + L::oSn);
        constexpr int N = M * PR;
#pragma unroll
        for (int u = 0; u < (N + NT - 1) / NT; ++u) {
            const int idx = min(tid + u * NT, N - 1);
            const f32x4 x = *reinterpret_cast<const f32x4 *>(X + (idx / PR) * L::ldx + (idx % PR) * PV);   // clamped: the read is not under the branch
            if (N % NT == 0 || tid + u * NT < N) *reinterpret_cast<f32x4 *>(tile + (uint32_t)idx * PV) = x;   // read back by the next kernel: cached
        }
    };
    // The walk, software-pipelined with ONE barrier per chunk.  At the top of step `it` LDS set it%2
    // holds the token rows of chunk `it` (written during the previous step).  The step
    //   - sends the memory the previous step gathered, and gathers the accumulator, which chunk `it` starts from,
    //   - applies S <- Diag(dec) S + W X,
    //   - writes the token rows of chunk it+1 into the other set,
    // and the caller refills the registers that became free, so only the accumulator update lies on the chain from one
    // chunk to the next.
    // The walk is rounded up to whole trips of AHEAD steps: steps past its end (real = false) update and store nothing.
    // (Their store is switched off lane by lane and not by a branch, for the same reason as the refills.)
    int lane_nch = nch;
    asm("" : "+v"(lane_nch));
    auto step = [&](const Weights &op, const Tokens &nx, int it, int b) {   // b = it % 2, a constant where it is called
        typename Atom<T>::Frag bf[C / 32][NI];
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) rows_of.frags(bf[ks], XT(b), ks * 32);
        if constexpr (MODE != 1) {
            if (it > 0 && it <= lane_nch) send(sp - dS, b ^ 1);
            gather(b);
            sp += dS;
        }
        if (it < nch) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                if (MODE == 1) dprod[mi] *= op.dec[mi];
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) acc[mi][ni] *= op.dec[mi];
            }
#pragma unroll
            for (int ks = 0; ks < C / 32; ++ks)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) Atom<T>::mma(acc[mi][ni], bf[ks][ni], op.w[ks][mi]);
        }
        tokens_to_lds(nx, b ^ 1);
    };
    // (the scheduling fences keep the compiler from hoisting a refill above the reads of its registers: it would
    // then load into other registers and copy them back at the end of the trip, which means waiting for loads that
    // were only just issued)
    if (nch > 0) {
        Weights op[AHEAD];
        Tokens tk[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            fetch_x(tk[u]);
            __builtin_amdgcn_sched_barrier(0);   // in the order of their use, as in the loop
            fetch_w(op[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
        tokens_to_lds(tk[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_x(tk[0]);
        __syncthreads();
        int it = 0;
        do {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {   // every position keeps its own registers
                step(op[u], tk[(u + 1) % AHEAD], it + u, u & 1);
                __builtin_amdgcn_sched_barrier(0);
                fetch_w(op[u]);
                fetch_x(tk[(u + 1) % AHEAD]);
                __syncthreads();
            }
            it += AHEAD;
        } while (it < nch);
        if constexpr (MODE != 1) {
            if (it == nch) send(sp - dS, (AHEAD - 1) & 1);
        }
    }
    if (MODE == 1) {   // what this segment adds and how much it decays, for its successors
        const size_t rec = ((size_t)s * a.max_seg + seg) * H + h;
        float *Y = a.sumY + rec * M * D + col0;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int g = 0; g < NI; ++g)
                *reinterpret_cast<f32x4 *>(Y + (size_t)(slot0 + 16 * mi) * D + lcol + 4 * g) = R::get(acc[mi], g);
        if (lcol == 0) {   // one lane per slot
            float *Dd = a.sumD + (rec * nsl + slice) * M;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) Dd[slot0 + 16 * mi] = dprod[mi];
        }
        return;
    }
    if (!ends_walk) return;
    // accumulator after the last chunk
    float *ST = isK ? a.outK : a.outV;
    if (ST) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int g = 0; g < NI; ++g)
                *reinterpret_cast<f32x4 *>(ST + (((size_t)s * H + h) * M + slot0 + 16 * mi) * dsrc + c0 + lcol + 4 * g) = R::get(acc[mi], g);
    }
    if (a.outJ) {
        __syncthreads();   // the last snapshot may still be on its way out of the set
        gather(0);
        __syncthreads();
        send(tile_of(a.outJ + ((size_t)s * H + h) * a.lay.stride), 0);
    }
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
template <typename T, int M>
static hipError_t launch_gates_tm(const Plan &pl, const Work &w, const float *g, const float *sin, float tau,
                                  hipStream_t st)
{
    const ChunkMap cm = make_chunk_map(pl, w);
    KernelTimer kt(kSlotGates, st);
    if (sin || tau > 0.f)
        hipLaunchKernelGGL((gate_kernel<T, M, true>), dim3(pl.chunk_slots, pl.H), dim3(kGateThreads<T, M>), 0, st, cm, pl.H, g,
                           sin, tau, (T *)w.Wf, w.dec);
    else
        hipLaunchKernelGGL((gate_kernel<T, M, false>), dim3(pl.chunk_slots, pl.H), dim3(kGateThreads<T, M>), 0, st, cm, pl.H, g,
                           sin, 0.f, (T *)w.Wf, w.dec);
    return hipGetLastError();
}

hipError_t launch_gates(const Plan &pl, const Work &w, const float *g, const float *sin, float tau, hipStream_t st)
{
#define GSA_GATES(T)                                                   \
    switch (pl.m) {                                                    \
    case 16: return launch_gates_tm<T, 16>(pl, w, g, sin, tau, st);         \
    case 32: return launch_gates_tm<T, 32>(pl, w, g, sin, tau, st);         \
    case 128: return launch_gates_tm<T, 128>(pl, w, g, sin, tau, st);       \
    default: return launch_gates_tm<T, 64>(pl, w, g, sin, tau, st);         \
    }
    if (pl.dtype == 0) { GSA_GATES(float) }
    GSA_GATES(bf16_t)
#undef GSA_GATES
}

template <typename T, int M, bool REVERSE, int MODE>
static hipError_t run_scan_mode(const Plan &pl, const ChunkMap &cm, const ScanArgs<T> &a, int slot, hipStream_t st)
{
    using G = ScanGeo<T, M>;
    const int total = (pl.d_k + pl.d_v) / G::NS * pl.H * pl.n_seqs * (MODE == 0 ? 1 : a.max_seg);
    // Prefetch depth: with at most one workgroup per CU the launch waits for the chain and its loads (8 x 2048 tokens, 4
    // heads, d = 128, 64 slots, 128 workgroups: 27.5 us four chunks ahead, 30.0 two; d = 512, 4 sequences, 256 workgroups:
    // 31.2 and 32.6); with more, more loads in flight only get into the way of the stores (512 workgroups: 57 and 56).  With 128
    // slots (256 workgroups 26.5 and 25.4) and for fp32 from 64 on (registers): two.
    constexpr int kDeep = M > 64 || (sizeof(T) == 4 && M > 32) ? 2 : 4;
    // (A packed batch may walk its sequences whole, see scan_unsegmented: what counts is how many workgroups that takes.)
    auto kern = total / (MODE != 0 && pl.cu_seqlens ? a.max_seg : 1) <= 256 ? scan_kernel<T, M, REVERSE, MODE, kDeep>
                                                                             : scan_kernel<T, M, REVERSE, MODE, 2>;
    constexpr size_t lds = ScanLds<T, M>::bytes;
    GSA_HIP_TRY(allow_lds(kern, lds));
    KernelTimer kt(slot, st);
    hipLaunchKernelGGL(kern, dim3(total), dim3(G::NT), lds, st, cm, pl.H, pl.d_k, pl.d_v, pl.n_seqs, a);
    return hipGetLastError();
}

template <typename T, int M, bool REVERSE>
static hipError_t run_scan(const Plan &pl, const ChunkMap &cm, const ScanArgs<T> &a, hipStream_t st)
{
    const int slot = REVERSE ? kSlotScanBwd : kSlotScanFwd;
    if (a.max_seg <= 1) return run_scan_mode<T, M, REVERSE, 0>(pl, cm, a, slot, st);
    GSA_HIP_TRY((run_scan_mode<T, M, REVERSE, 1>(pl, cm, a, kSlotScanSummary, st)));
    return run_scan_mode<T, M, REVERSE, 2>(pl, cm, a, slot, st);
}

template <typename T, int M>
static hipError_t launch_scan_tm(const Plan &pl, const Work &w, const ScanIo &io, hipStream_t st)
{
    const ChunkMap cm = make_chunk_map(pl, w);
    ScanArgs<T> a;
    a.W = static_cast<const T *>(io.reverse ? w.Wr : w.Wf);
    a.w_parts = io.reverse ? 2 : 1;
    a.dec = w.dec;
    a.xk = static_cast<const T *>(io.xk);
    a.xv = static_cast<const T *>(io.xv);
    a.phi_k = io.phi_k;
    a.phi_v = io.phi_v;
    a.initK = io.initK;
    a.initV = io.initV;
    a.snap = static_cast<T *>(io.reverse ? w.E : w.S);
    a.lay = pl.lay;
    a.outK = io.outK;
    a.outV = io.outV;
    a.outJ = static_cast<T *>(io.outJ);
    a.seg_chunks = pl.seg_chunks;
    a.max_seg = pl.max_seg;
    a.sumY = w.sumY;
    a.sumD = w.sumD;
    // 64-column slices: several workgroups per CU, so that their dependent chains overlap
    if (io.reverse) return run_scan<T, M, true>(pl, cm, a, st);
    return run_scan<T, M, false>(pl, cm, a, st);
}

hipError_t launch_scan(const Plan &pl, const Work &w, const ScanIo &io, hipStream_t st)
{
#define GSA_SCAN(T)                                                   \
    switch (pl.m) {                                                   \
    case 16: return launch_scan_tm<T, 16>(pl, w, io, st);             \
    case 32: return launch_scan_tm<T, 32>(pl, w, io, st);             \
    case 128: return launch_scan_tm<T, 128>(pl, w, io, st);             \
    default: return launch_scan_tm<T, 64>(pl, w, io, st);             \
    }
    if (pl.dtype == 0) { GSA_SCAN(float) }
    GSA_SCAN(bf16_t)
#undef GSA_SCAN
}

}  // namespace gsa
