// Chunk-level device routines shared by the forward output kernel and the backward
// kernels: the gated "scores" contraction that both GLA passes of GSA reduce to.
//
// Gate handling (paper, Appendix A: the chunkwise form divides by cumulative decays,
// which overflows; GLA's remedy is a secondary chunking).  Here rows of a chunk are
// grouped in blocks of 16 tokens, one wave per block, and every gate factor is relative
// to a block's own start or end (see BlockGates).  Factors between different blocks are
// all <= 1; inside the diagonal block one factor grows with the decay across 16 tokens.
// If that decay exceeds e^80 for some slot (alpha < 0.007 sustained over a block; not
// reachable with the paper's sigmoid^(1/8) gates) the diagonal block is evaluated pair by
// pair with the unfactored exponent instead.
//
// Orientation: the per-token slot vectors (scores, read weights, their gradients) are kept
// in matrix-core tiles D[slot][token]: lane l holds token l%16 of the wave's row block and
// slots 16*ni + 4*(l/16) + j.  Three things follow.  Such a tile, rounded to the I/O type, IS
// the operand of a contraction over the slots, and a tile D[r][t] of pair products IS the
// operand of a contraction over r, so neither goes through LDS.  A sum over the slots of a
// token is a sum over a lane's own registers and two shuffles.  And a cumulative sum over the
// tokens of a block runs over 16 neighbouring lanes (DPP row shifts), with no barrier.
#pragma once
#include <type_traits>

#include "gsa_common.h"

namespace gsa {

// ----------------------------------------------------------------------------
// Contractions over the head dimension.  A workgroup walks the columns in steps of 128 bytes per row; the tiles of a step
// ([rows][128 bytes]) come from memory in whole lines, every thread taking 16-byte pieces, wait in registers for their turn
// and lie in one of two LDS buffers while the waves read them as depth-32 operands, wave w for the tokens of row block w.
// One barrier per step.  What this replaces: every wave took a share of the columns for all row blocks, with its operands
// straight from memory (16 bytes of each of 16 rows per quarter of a load, four times the address unit's time) and the
// partial sums exchanged through LDS.  Forward chunk kernel, 64 slots, 8 x 2048 tokens, 4 heads: d = 128 41.4 -> 36.0 us, d = 512 86 -> 82; one
// sequence of 2048, d = 512 26.7 -> 22.6; 128 slots, 4 x 1000 tokens 41 -> 36; intra-chunk gradients, d = 128 77 -> 68, d = 512 201 -> 198.
// ----------------------------------------------------------------------------
template <typename T> struct StepTile {
    static constexpr int KS = 128 / sizeof(T), PV = 16 / sizeof(T), PR = 8;   // columns per step, elements per piece, pieces per row
    static constexpr int F = KS / 32;                                         // depth-32 operands per step
    typedef T Piece __attribute__((ext_vector_type(16 / sizeof(T))));
    // Pieces are XOR-swizzled so that the same piece of 16 rows lies in all banks.
    __device__ static __forceinline__ void put(T *tile, int row, int p, const Piece &x)
    {
        *reinterpret_cast<Piece *>(tile + row * KS + ((p ^ ((row >> 1) & 7)) * PV)) = x;
    }
    // operand f of rows row0 .. row0+15 (row0 a multiple of 16)
    __device__ static __forceinline__ typename Atom<T>::Frag frag(const T *tile, int row0, int f, int lane)
    {
        const int r = lane & 15, g = lane >> 4, s = r >> 1;
        const T *row = tile + (row0 + r) * KS;
        if constexpr (sizeof(T) == 2) {
            return Atom<T>::load(row + (((f * 4 + g) ^ s) * PV));
        } else {
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(row + (((2 * g) ^ s) * PV)), hi = *reinterpret_cast<const f32x4 *>(row + (((2 * g + 1) ^ s) * PV));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
};

// One operand of such a walk: ROWS rows of a token tensor (rows `ld` elements apart, those past the end of a ragged
// chunk read as copies of its last row: they stay finite and only ever produce rows of the result that are not stored or
// that meet zero weights), or of one part of a memory snapshot (SNAP, tiled as StateLayout describes).
// HINT: loads carry the non-temporal hint (for what the caller knows nobody reads again soon).
template <typename T, int ROWS, int NT, bool SNAP, bool HINT> struct StepRows {
    using Tile = StepTile<T>;
    typedef typename Tile::Piece Piece;
    static constexpr int N = ROWS * Tile::PR, V = (N + NT - 1) / NT;   // pieces, pieces per thread
    struct Stage { Piece x[V]; };
    const char *base[V];   // uniform over the wave: the first row of its piece v
    uint32_t off[V];       // bytes from there; kLaneRows, which the host checks
    __device__ __forceinline__ StepRows(const T *p, size_t ld, int len, int tid)
    {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int idx = min(tid + v * NT, N - 1), row = idx / Tile::PR;
            const int row0 = SNAP ? 0 : min(v * (NT / Tile::PR) + __builtin_amdgcn_readfirstlane(tid >> 6) * (kWave / Tile::PR), len - 1);
            static_assert(kWave / Tile::PR <= kLaneRows, "rows of a wave");
            base[v] = reinterpret_cast<const char *>(p) + (size_t)row0 * ld * sizeof(T);
            off[v] = SNAP ? (uint32_t)(row * kSnapTile * (int)sizeof(T) + (idx % Tile::PR) * 16)
                          : (uint32_t)(min(row, len - 1) - row0) * (uint32_t)(ld * sizeof(T)) + (idx % Tile::PR) * 16;
        }
    }
    __device__ __forceinline__ void fetch(Stage &st, int step) const
    {
        const size_t at = (SNAP ? (size_t)(step / (kSnapTile / Tile::KS)) * (ROWS * kSnapTile * sizeof(T)) + (size_t)(step % (kSnapTile / Tile::KS)) * 128
                                     : (size_t)step * 128);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const Piece *q = reinterpret_cast<const Piece *>(base[v] + at + off[v]);
            if (HINT) st.x[v] = __builtin_nontemporal_load(q);
            else st.x[v] = *q;
        }
    }
    // PHI: with the feature map applied on the way
    template <bool PHI = false> __device__ __forceinline__ void put(T *tile, const Stage &st, int tid) const
    {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int idx = tid + v * NT;
            Piece x = st.x[v];
            if (PHI) {
#pragma unroll
                for (int e = 0; e < Tile::PV; ++e) x[e] = from_f32<T>(swish_value(to_f32(x[e])));
            }
            if (N % NT == 0 || idx < N) Tile::put(tile, idx / Tile::PR, idx % Tile::PR, x);
        }
    }
};

// The walk over n steps, two at a time, so that 256 bytes of a row are asked for together (one step at a time, two ahead: forward,
// 8 x 2048 tokens, 4 heads, d = 512, 64 slots 92 us instead of 82).  fetch(u, step): loads of a step into register stage u; put(u,
// step): stage u, which holds that step, to LDS buffer u; multiply(b): the products of buffer b.  The caller has issued the loads of
// the first two steps (past the end: of the last one again) and has the buffers free; the walk ends with a barrier.
// PAIRS = false: one step at a time, stage and buffer 0 only, where two do not fit.
template <bool PAIRS = true, typename Fetch, typename Put, typename Multiply>
__device__ __forceinline__ void walk_steps(int n, Fetch &&fetch, Put &&put, Multiply &&multiply)
{
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    for (int it = 0;; it += 2) {
        put(even, it);
        if constexpr (PAIRS) put(odd, it + 1);
        __builtin_amdgcn_sched_barrier(0);   // a refill stays behind the reads of its registers
        if (it + (PAIRS ? 2 : 1) < n) {   // uniform over the grid
            fetch(even, it + (PAIRS ? 2 : 1));
            if constexpr (PAIRS) fetch(odd, min(it + 3, n - 1));
        }
        __syncthreads();
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);   // operands of both at a time would not fit the registers
        if constexpr (PAIRS) {
            if (it + 1 < n) multiply(1);
        }
        __syncthreads();
        if constexpr (!PAIRS) {
            if (it + 1 >= n) return;
            put(even, it + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (it + 2 < n) fetch(even, it + 2);
            __syncthreads();
            multiply(0);
            __syncthreads();
        }
        if (it + 2 >= n) return;
    }
}

// Accumulators of such a walk: step(), the products of one step, done().  fp32 sums every step on its own: the longer a chain of
// roundings, the larger its error.  With one chain over all columns dq is 2.92e-7 from the fp64 recurrence (m = 32, 700 tokens, d_k = 192).
template <typename T, int N> struct StepSums {
    static constexpr bool kSplit = sizeof(T) == 4;
    f32x4 sum[N], part[kSplit ? N : 1];
    __device__ __forceinline__ StepSums()
    {
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ auto step() -> f32x4 (&)[N]
    {
        if constexpr (kSplit) {
#pragma unroll
            for (int i = 0; i < N; ++i) part[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            return part;
        } else {
            return sum;
        }
    }
    __device__ __forceinline__ void done()
    {
        if constexpr (kSplit) {
#pragma unroll
            for (int i = 0; i < N; ++i) sum[i] += part[i];
        }
    }
};

// ----------------------------------------------------------------------------
// Row shifts inside the 16 lanes that share l/16 (DPP; lanes without a source read zero).
// ----------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ float dpp_or_zero(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_prefix_sum(float x)   // inclusive, over lanes l%16 = 0 .. own
{
    x += dpp_or_zero<0x111>(x);   // row_shr:1, 2, 4, 8
    x += dpp_or_zero<0x112>(x);
    x += dpp_or_zero<0x114>(x);
    x += dpp_or_zero<0x118>(x);
    return x;
}
__device__ __forceinline__ float row16_suffix_sum(float x)   // inclusive, over lanes own .. l%16 = 15
{
    x += dpp_or_zero<0x101>(x);   // row_shl:1, 2, 4, 8
    x += dpp_or_zero<0x102>(x);
    x += dpp_or_zero<0x104>(x);
    x += dpp_or_zero<0x108>(x);
    return x;
}
__device__ __forceinline__ float row16_last(float x) { return dpp_or_zero<0x15f>(x); }   // row_newbcast:15

// Sum / maximum over the slots of a token: over the four lanes that share l%16, after the lane's own registers.
__device__ __forceinline__ float slots_sum(float x)
{
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float slots_max(float x)
{
    x = fmaxf(x, __shfl_xor(x, 16, 64));
    return fmaxf(x, __shfl_xor(x, 32, 64));
}

// Softmax over the slots of every token of the block, in place (D[slot][token] tiles).
template <int M> __device__ __forceinline__ void softmax_slots(f32x4 (&p)[M / 16])
{
    float mx = p[0][0];
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};   // four short chains
#pragma unroll
    for (int ni = 0; ni < M / 16; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) mx = fmaxf(mx, p[ni][j]);
    mx = slots_max(mx);
#pragma unroll
    for (int ni = 0; ni < M / 16; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) { p[ni][j] = __expf(p[ni][j] - mx); sum[j] += p[ni][j]; }
    const float inv = 1.f / slots_sum((sum[0] + sum[1]) + (sum[2] + sum[3]));
#pragma unroll
    for (int ni = 0; ni < M / 16; ++ni) p[ni] *= inv;
}

// D tile -> depth-16 operand of the same lane (rows 4*(l/16)+j become contraction indices).
template <typename T> __device__ __forceinline__ typename Atom<T>::Frag16 to_frag16(const f32x4 &x)
{
    typename Atom<T>::Frag16 f;
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = from_f32<T>(x[j]);
    return f;
}
// What that rounding left behind, as a second operand: a contraction with both carries the tile to twice the
// I/O type's precision (bf16; nothing is left behind in fp32, and the second product is not issued).
template <typename T> __device__ __forceinline__ typename Atom<T>::Frag16 rest_frag16(const f32x4 &x, const typename Atom<T>::Frag16 &f)
{
    f32x4 y;
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // of an infinity nothing: its sum with a NaN would lose the sign
        const float h = to_f32(f[j]);
        y[j] = fabsf(h) < __builtin_inff() ? x[j] - h : 0.f;
    }
    return to_frag16<T>(y);
}
template <typename T> __device__ __forceinline__ void store_frag16(T *p, const f32x4 &x)
{
    store4(p, x[0], x[1], x[2], x[3]);
}

// ----------------------------------------------------------------------------
// Gates of one wave's row block (16 tokens, all slots), in D[slot][token] registers.
//   L[ni][j]   = sum over the block's tokens up to and including t of g       (block-local, inclusive)
//   tot[ni][j] = the same over the whole block (equal in the 16 lanes of a row)
//   kind       = how far the block's widest slot decays (wave-uniform), which decides how its own pairs are weighted
//   s[ni][j]   = write intensity, 0 on rows past the end of the chunk
// What other waves need of them goes to LDS once (write_tiles): the write-intensity tile referenced to
// the END of its block,
//   V[r][i] = s_r[i] * exp(tot[i] - L_r[i])  <= 1,
// in both orientations (Vn[token][slot], Vt[slot][token]), and the decay across the block Rb[b][i] =
// exp(tot[i]).  The weight between a token t of block w and a token r of block b <= w is then
//   exp(G_t - G_r) s_r = exp(L_t - tot_w) * (product of Rb over the blocks b+1 .. w) * V[r]
// no operand of a gated contraction needs an exponential of its own, and no exponential is evaluated twice.  The
// diagonal block (b = w) depends on its kind:
//   kNarrow (bf16, down to e^-40): as above, exp(L_t - tot) * V[r].
//   kHalf (down to e^-80; fp32: always): referenced halfway by the wave that owns it, exp(L_t - tot/2) * s_r exp(tot/2 - L_r),
//   with operands of its own.  Neither factor leaves e^+-40 then, and what they multiply may lie anywhere in fp32's range
//   but its outer 17 orders of magnitude; referenced to the end, weights above 6e3 overflowed at e^-80 and products below
//   1e-4 underflowed.  (Tokens of later blocks are all behind the decay: what underflows there is far below their own
//   block's terms.)  fp32 takes it for the smaller exponents: the error of dq is 2.56e-7 instead of 2.94e-7 (m = 32, 700
//   tokens, d_k = 192).
//   kPairs (wider): the block's own pairs are evaluated one by one with the unfactored exponent.
// ----------------------------------------------------------------------------
enum BlockKind { kNarrow = 0, kHalf = 1, kPairs = 2 };
template <int M, bool GEN> struct BlockGates {
    static constexpr int MI = M / 16;
    f32x4 L[MI], s[MI], tot[MI];
    int kind = kNarrow;
    bool given = false;
    float tau = 0.f;
    // Issues the loads (rows clamped into the chunk); may be called well before finish().
    __device__ __forceinline__ void load(const float *g, size_t gld, int len, int rowb, int lane, const float *sin,
                                         float gate_tau)
    {
        const size_t off = (size_t)min(rowb + (lane & 15), len - 1) * gld + (lane >> 4) * 4;
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) L[ni] = *reinterpret_cast<const f32x4 *>(g + off + ni * 16);
        if (GEN) tau = gate_tau;
        if (GEN && sin) {   // uniform over the grid
            given = true;
#pragma unroll
            for (int ni = 0; ni < MI; ++ni) s[ni] = *reinterpret_cast<const f32x4 *>(sin + off + ni * 16);
        }
    }
    template <typename T> __device__ __forceinline__ void finish(int len, int rowb, int lane)
    {
        const bool live = rowb + (lane & 15) < len;
        float least = 0.f;
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x = L[ni][j];
                if (GEN && tau > 0.f) x = log_gate_from_logit(x, tau);
                x = live ? floor_gate(x) : 0.f;
                const float sx = (GEN && given) ? s[ni][j] : -expm1f(x);
                s[ni][j] = live ? sx : 0.f;
                x = row16_prefix_sum(x);
                L[ni][j] = x;
                tot[ni][j] = row16_last(x);
                least = fminf(least, tot[ni][j]);
            }
        kind = __any(least < -kExpClamp) ? kPairs : (sizeof(T) == 4 || __any(least < -0.5f * kExpClamp)) ? kHalf : kNarrow;
    }
    // exp(L_t - ref) with ref the block's end where its diagonal uses the shared tile, else its start
    __device__ __forceinline__ float walk_gate(int ni, int j) const { return __expf(kind == kNarrow ? L[ni][j] - tot[ni][j] : L[ni][j]); }
    // kHalf: the two factors of the diagonal
    __device__ __forceinline__ float half_read(int ni, int j) const { return __expf(L[ni][j] - 0.5f * tot[ni][j]); }
    __device__ __forceinline__ float half_write(int ni, int j) const { return s[ni][j] * __expf(0.5f * tot[ni][j] - L[ni][j]); }
    template <typename T>
    __device__ __forceinline__ void write_tiles(T *Vn, int ldn, T *Vt, int ldt, float *Rb, int rowb, int lane) const
    {
        const int r = lane & 15, g4 = (lane >> 4) * 4;
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            f32x4 v, e;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = s[ni][j] * __expf(tot[ni][j] - L[ni][j]);
                e[j] = __expf(tot[ni][j]);
            }
            if (Vn) store_frag16<T>(Vn + (rowb + r) * ldn + ni * 16 + g4, v);
            if (Vt) {
#pragma unroll
                for (int j = 0; j < 4; ++j) Vt[(ni * 16 + g4 + j) * ldt + rowb + r] = from_f32<T>(v[j]);
            }
            if (r == 0) *reinterpret_cast<f32x4 *>(Rb + (rowb / 16) * M + ni * 16 + g4) = e;
        }
    }
};

// One gated pass whose gate sits on the slot side (pass 1 of Eq. (gsa-2pass) with X=q, Y=k, St=Kt; its
// mirror in the backward with X=dO, Y=v, St=Vt), first part: the contractions over the head dimension.
//   a[cb][.]  = D[r][t] tile of X_t . Y_r for this wave's row block t and the row blocks cb <= w of r,
//               rounded to T and causally masked: an operand of contractions over r; alo[cb]: the rest
//   run[ni]   = D[slot][t] tile of <X_t, St[slot]>
// X, Y: [len][d] rows in global memory (row stride ldx elements); St: one part of a memory snapshot
// (M slots, d columns, tiled as StateLayout describes).  d must be a multiple of 64.
// HINT: which operands are loaded with the non-temporal hint (kHintX | kHintY | kHintSt).
// PHI: which of X, Y get the feature map on their way into LDS (kHintX | kHintY bits).
// buf: LDS, kBytes, free from the start.  begin() issues the first loads, before which the caller issues its own and behind
// which it does what needs no operand of the contraction (gates); finish() is for all threads of the workgroup and ends
// with a barrier.
constexpr int kHintX = 1, kHintY = 2, kHintSt = 4;
template <typename T, int M, int C, int HINT, int PHI> struct HeadContraction {
    using Tile = StepTile<T>;
    static constexpr int NT = Geo<T>::NT, MI = M / 16, CI = C / 16, NB = CI + MI;
    static constexpr size_t oY = sizeof(T) * C * Tile::KS, oS = 2 * oY, szBuf = oS + sizeof(T) * M * Tile::KS;
    // Two steps at a time (see walk_steps), one for fp32 with 128 slots: a second buffer leaves one workgroup on a CU
    // instead of two (8 x 2048 tokens, 4 heads, d = 512 forward 324 us against 205; d = 256, 16384 tokens 206 against 118).
    static constexpr bool kTwo = sizeof(T) == 2 || M < 128;
    static constexpr size_t kBytes = (kTwo ? 2 : 1) * szBuf;
    typedef StepRows<T, C, NT, false, (HINT & kHintX) != 0> RX;
    typedef StepRows<T, C, NT, false, (HINT & kHintY) != 0> RY;
    typedef StepRows<T, M, NT, true, (HINT & kHintSt) != 0> RS;
    RX rx;
    RY ry;
    RS rs;
    typename RX::Stage sx[2];
    typename RY::Stage sy[2];
    typename RS::Stage ss[2];
    int n, tid;
    __device__ __forceinline__ void fetch(int u, int step)
    {
        rx.fetch(sx[u], step);
        ry.fetch(sy[u], step);
        rs.fetch(ss[u], step);
    }
    __device__ __forceinline__ HeadContraction(const T *X, const T *Y, size_t ldx, int d, const T *St, int len, int tid_)
        : rx(X, ldx, len, tid_), ry(Y, ldx, len, tid_), rs(St, 0, 0, tid_), n(d / Tile::KS), tid(tid_)
    {
#pragma unroll
        for (int u = 0; u < (kTwo ? 2 : 1); ++u) {
            fetch(u, min(u, n - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ void finish(f32x4 (&run)[MI], typename Atom<T>::Frag16 (&a)[CI], typename Atom<T>::Frag16 (&alo)[CI],
                                           unsigned char *buf, int lane, int w)
    {
        const int r = lane & 15, g4 = (lane >> 4) * 4;
        StepSums<T, NB> sums;
        walk_steps<kTwo>(
            n, [&](auto u, int step) { fetch(decltype(u)::value, step); },
            [&](auto u, int) {
                constexpr int U = decltype(u)::value;
                unsigned char *p = buf + U * szBuf;
                rx.template put<(PHI & kHintX) != 0>(reinterpret_cast<T *>(p), sx[U], tid);
                ry.template put<(PHI & kHintY) != 0>(reinterpret_cast<T *>(p + oY), sy[U], tid);
                rs.put(reinterpret_cast<T *>(p + oS), ss[U], tid);
            },
            [&](int b) {
                f32x4(&acc)[NB] = sums.step();
                const T *X = reinterpret_cast<const T *>(buf + b * szBuf), *Y = reinterpret_cast<const T *>(buf + b * szBuf + oY);
                const T *S = reinterpret_cast<const T *>(buf + b * szBuf + oS);
#pragma unroll
                for (int f = 0; f < Tile::F; ++f) {
                    const typename Atom<T>::Frag x = Tile::frag(X, 16 * w, f, lane);
#pragma unroll
                    for (int ni = 0; ni < MI; ++ni) Atom<T>::mma(acc[CI + ni], Tile::frag(S, 16 * ni, f, lane), x);
#pragma unroll
                    for (int cb = 0; cb < CI; ++cb)
                        if (cb <= w) Atom<T>::mma(acc[cb], Tile::frag(Y, 16 * cb, f, lane), x);   // wave-uniform
                }
                sums.done();
            });
#pragma unroll
        for (int cb = 0; cb < CI; ++cb) {
            f32x4 x = sums.sum[cb];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = (cb < w || (cb == w && g4 + j <= r)) ? x[j] : 0.f;
            a[cb] = to_frag16<T>(x);
            alo[cb] = rest_frag16<T>(x, a[cb]);
        }
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) run[ni] = sums.sum[CI + ni];
    }
};

// Second part: the gated sum itself, from the tiles of HeadContraction and of BlockGates::write_tiles (which
// must be visible to all waves).  Vp: LDS, kPrivate<T, M> elements of this wave's own.
//   run[ni][j] <- exp(G_t[i]) * <X_t, St[i]>  +  sum_{r<=t} <X_t, Y_r> s_r[i] exp(G_t[i]-G_r[i])
// `run` walks its reference from the chunk start (where it is the inter-chunk term) to the end of this
// wave's block, one block at a time: run <- run * Rb[b] + V_b^T a_b.  (To its start where the diagonal is not kNarrow.)
template <typename T, int M> constexpr int kPrivate = M * (16 + Atom<T>::kPad);
template <typename T, int M, int C, bool GEN>
__device__ __forceinline__ void gated_rows(f32x4 (&run)[M / 16], const typename Atom<T>::Frag16 (&a)[C / 16],
                                           const typename Atom<T>::Frag16 (&alo)[C / 16],
                                           const BlockGates<M, GEN> &bg, const T *Vt, int ldt,
                                           const float *Rb, T *Vp, int lane, int w)
{
    constexpr int MI = M / 16, CI = C / 16;
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    typename Atom<T>::Frag16 own = a[0], rest = alo[0];
#pragma unroll
    for (int b = 0; b < CI; ++b) {
        if (b > w) continue;   // wave-uniform
        own = a[b];
        rest = alo[b];
        if (b == w && bg.kind != kNarrow) continue;
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            run[ni] *= *reinterpret_cast<const f32x4 *>(Rb + b * M + ni * 16 + g4);
            const typename Atom<T>::Frag16 v = Atom<T>::load16(Vt + (ni * 16 + r) * ldt + b * 16 + g4);
            Atom<T>::mma16(run[ni], v, a[b]);
            if (sizeof(T) == 2) Atom<T>::mma16(run[ni], v, alo[b]);
        }
    }
#pragma unroll
    for (int ni = 0; ni < MI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) run[ni][j] *= bg.walk_gate(ni, j);
    if (bg.kind == kHalf) {
        constexpr int ldp = 16 + Atom<T>::kPad;
#pragma unroll
        for (int ni = 0; ni < MI; ++ni)
#pragma unroll
            for (int j = 0; j < 4; ++j) Vp[(ni * 16 + g4 + j) * ldp + r] = from_f32<T>(bg.half_write(ni, j));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int ni = 0; ni < MI; ++ni) {
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
            const typename Atom<T>::Frag16 v = Atom<T>::load16(Vp + (ni * 16 + r) * ldp + g4);
            Atom<T>::mma16(x, v, own);
            if (sizeof(T) == 2) Atom<T>::mma16(x, v, rest);
#pragma unroll
            for (int j = 0; j < 4; ++j) run[ni][j] += x[j] * bg.half_read(ni, j);
        }
    }
    if (bg.kind == kPairs) {   // the diagonal block pair by pair
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int rr = 4 * q + c;
                const float x = sizeof(T) == 2 ? to_f32(own[c]) + to_f32(rest[c]) : to_f32(own[c]);
                const float av = __shfl(x, 16 * q + r, 64);   // zero for rr > t
#pragma unroll
                for (int ni = 0; ni < MI; ++ni)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float Lr = __shfl(bg.L[ni][j], (lane & 48) | rr, 64), sr = __shfl(bg.s[ni][j], (lane & 48) | rr, 64);
                        run[ni][j] += av * sr * __expf(fminf(bg.L[ni][j] - Lr, 0.f));
                    }
            }
    }
}

// Pair weights of this wave's row block w against row block b <= w, with the slots contracted in registers:
//   out[j] = sum_i wt[i] V[r][i],   D[r][t]
// wt: D[slot][t] tiles referenced to the END of block b.  Entries with r > t are returned as computed.
template <typename T, int M>
__device__ __forceinline__ f32x4 pair_tile(const f32x4 (&wt)[M / 16], const T *Vn, int ldn, int b, int lane)
{
    constexpr int MI = M / 16;
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ni = 0; ni < MI; ++ni)
        Atom<T>::mma16(acc, Atom<T>::load16(Vn + (b * 16 + r) * ldn + ni * 16 + g4), to_frag16<T>(wt[ni]));
    return acc;
}

// The same for two sets of weights: x1 in D[r][t]; x1t, x2t in D[t][r].
template <typename T, int M>
__device__ __forceinline__ void pair_tiles(const f32x4 (&w1)[M / 16], const f32x4 (&w2)[M / 16], const T *Vn, int ldn,
                                           int b, int lane, f32x4 &x1, f32x4 &x1t, f32x4 &x2t)
{
    constexpr int MI = M / 16;
    const int r = lane & 15, g4 = (lane >> 4) * 4;
#pragma unroll
    for (int ni = 0; ni < MI; ++ni) {
        const typename Atom<T>::Frag16 v = Atom<T>::load16(Vn + (b * 16 + r) * ldn + ni * 16 + g4);
        const typename Atom<T>::Frag16 f = to_frag16<T>(w1[ni]);
        Atom<T>::mma16(x1, v, f);
        Atom<T>::mma16(x1t, f, v);
        Atom<T>::mma16(x2t, to_frag16<T>(w2[ni]), v);
    }
}

// The diagonal tile D[r][t] of the pair weights of a kHalf block, zero for r > t.  wt: ungated D[slot][t] weights.
template <typename T, int M, bool GEN>
__device__ __forceinline__ f32x4 pair_tile_half(const f32x4 (&wt)[M / 16], const BlockGates<M, GEN> &bg, int lane)
{
    const int r = lane & 15, g4 = (lane >> 4) * 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ni = 0; ni < M / 16; ++ni) {
        f32x4 v, x;
#pragma unroll
        for (int j = 0; j < 4; ++j) { v[j] = bg.half_write(ni, j); x[j] = wt[ni][j] * bg.half_read(ni, j); }
        Atom<T>::mma16(acc, to_frag16<T>(v), to_frag16<T>(x));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = g4 + j <= r ? acc[j] : 0.f;
    return acc;
}

// The diagonal tile D[r][t] of the pair weights without factoring: sum_i wt[i] s_r[i] exp(L_t[i] - L_r[i]) for
// r <= t, else 0.  wt: ungated D[slot][t] weights.
template <int M, bool GEN>
__device__ __forceinline__ f32x4 pair_tile_exact(const f32x4 (&wt)[M / 16], const BlockGates<M, GEN> &bg, int lane)
{
    constexpr int MI = M / 16;
    const int r = lane & 15, g = lane >> 4;
    f32x4 out = {0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int rr = 4 * q + c;
            float sum = 0.f;
#pragma unroll
            for (int ni = 0; ni < MI; ++ni)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float Lr = __shfl(bg.L[ni][j], (lane & 48) | rr, 64), sr = __shfl(bg.s[ni][j], (lane & 48) | rr, 64);
                    sum += wt[ni][j] * sr * __expf(fminf(bg.L[ni][j] - Lr, 0.f));
                }
            sum = slots_sum(sum);
            if (q == g) out[c] = rr <= r ? sum : 0.f;
        }
    return out;
}

// The eight slots i0 .. i0+7 a lane contributes to a contraction over the (padded) slot axis,
// and whether they exist: with M < KM the padding lanes re-read the last eight real slots and
// are masked, so that no LDS read sits under a per-lane branch.
template <int M, int KM> struct SlotSpan {
    int i0;
    bool live;
    __device__ __forceinline__ SlotSpan(int k) : i0((M < KM) ? min(k, M - 8) : k), live((M >= KM) || (k < M)) {}
};

// Stores a C x ncols tile held in LDS (Os, row stride ldo) to global rows of `ld` elements,
// 8 elements per thread, rows >= len skipped.  NTS: with the non-temporal hint (final outputs).
template <typename T, bool NTS = false>
__device__ __forceinline__ void store_tile(T *dst, size_t ld, const T *Os, int ldo, int rows, int ncols, int len,
                                           int tid, int nthreads)
{
    const int vpr = ncols >> 3;
    for (int idx = tid; idx < rows * vpr; idx += nthreads) {
        const int t = idx / vpr, c = (idx - t * vpr) << 3;
        if (t >= len) continue;
        const T *s = Os + t * ldo + c;
        T *d = dst + (size_t)t * ld + c;
        if (NTS) {
            __builtin_nontemporal_store(*reinterpret_cast<const f32x4 *>(s), reinterpret_cast<f32x4 *>(d));
            if (sizeof(T) == 4) __builtin_nontemporal_store(*reinterpret_cast<const f32x4 *>(s + 4), reinterpret_cast<f32x4 *>(d + 4));
        } else {
            *reinterpret_cast<f32x4 *>(d) = *reinterpret_cast<const f32x4 *>(s);
            if (sizeof(T) == 4) *reinterpret_cast<f32x4 *>(d + 4) = *reinterpret_cast<const f32x4 *>(s + 4);
        }
    }
}

}  // namespace gsa
