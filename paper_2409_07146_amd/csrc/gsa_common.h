// Device-side building blocks shared by the libgsa kernels (gfx950 / CDNA4, wave64).
//
// Everything here is written in terms of one matrix-core atom: a 16x16 fp32
// accumulator tile updated with a depth-32 contraction.  For bf16 operands that
// is one v_mfma_f32_16x16x32_bf16; for fp32 operands it is eight
// v_mfma_f32_16x16x4_f32.  Both take their operands as fragments of 8 consecutive
// k per lane, so every kernel is written once and instantiated for both element
// types.  Where the contraction index runs fastest a fragment is read as it lies (LDS tiles,
// or memory in fragment order); bf16 tiles that lie the other way go through
// the transposing LDS load (TrTile).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gsa_layout.h"

namespace gsa {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

constexpr int kWave = 64;
constexpr int kSub = 16;            // row block inside a chunk sharing one gate reference
constexpr float kGateFloor = -30.f; // log-gates below this are treated as this
constexpr float kExpClamp = 80.f;   // largest exponent a factored gate may carry in fp32

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return (bf16_t)x; }

// ----------------------------------------------------------------------------
// Matrix-core atom.
//   A fragment: lane l holds A[row = l%16][k = 8*(l/16) + e], e = 0..7
//   B fragment: lane l holds B[k = 8*(l/16) + e][col = l%16]
//   D tile    : lane l holds D[row = 4*(l/16) + j][col = l%16], j = 0..3
// ----------------------------------------------------------------------------
template <typename T> struct Atom;

template <> struct Atom<bf16_t> {
    typedef bf16x8 Frag;
    static constexpr int kPad = 8;  // elements of padding that keep rows 16-byte aligned
    __device__ static __forceinline__ Frag load(const bf16_t *p) { return *reinterpret_cast<const Frag *>(p); }
    __device__ static __forceinline__ Frag zero() { Frag f; for (int e = 0; e < 8; ++e) f[e] = (bf16_t)0.f; return f; }
    __device__ static __forceinline__ void mma(f32x4 &c, const Frag &a, const Frag &b) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    // depth-16 form: lane l holds row l%16 and the four contraction indices 4*(l/16) .. +3
    typedef bf16x4 Frag16;
    __device__ static __forceinline__ Frag16 load16(const bf16_t *p) { return *reinterpret_cast<const Frag16 *>(p); }
    __device__ static __forceinline__ void mma16(f32x4 &c, const Frag16 &a, const Frag16 &b) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
    }
};

template <> struct Atom<float> {
    typedef f32x8 Frag;
    static constexpr int kPad = 4;
    __device__ static __forceinline__ Frag load(const float *p) {
        const f32x4 lo = *reinterpret_cast<const f32x4 *>(p);
        const f32x4 hi = *reinterpret_cast<const f32x4 *>(p + 4);
        Frag f;
        f[0] = lo[0]; f[1] = lo[1]; f[2] = lo[2]; f[3] = lo[3];
        f[4] = hi[0]; f[5] = hi[1]; f[6] = hi[2]; f[7] = hi[3];
        return f;
    }
    __device__ static __forceinline__ Frag zero() { Frag f; for (int e = 0; e < 8; ++e) f[e] = 0.f; return f; }
    __device__ static __forceinline__ void mma(f32x4 &c, const Frag &a, const Frag &b) {
        // instruction e contracts k = {e, 8+e, 16+e, 24+e}: lane group l/16 supplies k = 8*(l/16)+e
#pragma unroll
        for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    }
    // depth-16 form: lane l holds row l%16 and the four contraction indices 4*(l/16) .. +3
    typedef f32x4 Frag16;
    __device__ static __forceinline__ Frag16 load16(const float *p) { return *reinterpret_cast<const Frag16 *>(p); }
    __device__ static __forceinline__ void mma16(f32x4 &c, const Frag16 &a, const Frag16 &b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    }
};

// Fragment order: a matrix [rows][32*steps] kept for one reader, as that reader's depth-32 operands (tile after tile of 16
// rows, step after step), so that a fragment load of a wave is one contiguous kilobyte.  From an array of rows the
// same load takes 16 bytes of each of 16 rows per quarter of the wave, and the address unit works line by line: four times as long.
template <typename T, int STEPS> __device__ __forceinline__ uint32_t frag_order(int row, int k)   // k % (16 / sizeof(T)) = 0: start of a 16-byte piece
{
    constexpr int PV = 16 / sizeof(T);
    const int lane = (row & 15) + 16 * ((k & 31) >> 3);
    return (uint32_t)(((row >> 4) * STEPS + (k >> 5)) * 512 + ((k & 7) / PV) * (kWave * PV) + lane * PV);
}
__device__ __forceinline__ bf16x8 load_frag_order(const bf16_t *tile, uint32_t lane) { return *reinterpret_cast<const bf16x8 *>(tile + lane * 8); }
__device__ __forceinline__ f32x8 load_frag_order(const float *tile, uint32_t lane)
{
    const f32x4 lo = *reinterpret_cast<const f32x4 *>(tile + lane * 4), hi = *reinterpret_cast<const f32x4 *>(tile + 256 + lane * 4);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Chunk geometry per element type: one wave per 16-token row block.  fp32 tiles are
// twice as large in LDS, so the fp32 path uses half the chunk.
template <typename T> struct Geo {
    static constexpr int C = (sizeof(T) == 2) ? 64 : 32;   // tokens per chunk
    static constexpr int NW = C / kSub;                    // waves per workgroup
    static constexpr int NT = NW * kWave;                  // threads per workgroup
};
inline int chunk_of_dtype(int dtype) { return dtype == 0 ? Geo<float>::C : Geo<bf16_t>::C; }

template <int MI, int NI> __device__ __forceinline__ void zero_acc(f32x4 (&acc)[MI][NI])
{
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
}

template <typename T> __device__ __forceinline__ void store8(T *dst, const float (&v)[8]);
template <> __device__ __forceinline__ void store8<bf16_t>(bf16_t *dst, const float (&v)[8]) {
    bf16x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (bf16_t)v[e];
    *reinterpret_cast<bf16x8 *>(dst) = x;
}
template <> __device__ __forceinline__ void store8<float>(float *dst, const float (&v)[8]) {
    *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4 *>(dst + 4) = f32x4{v[4], v[5], v[6], v[7]};
}

// Non-temporal forms (load_nt / store_nt below, the builtins elsewhere): for data a kernel touches once and
// nobody reads again soon.  Such traffic then streams through the caches instead of displacing lines
// that the co-resident workgroups or the next kernel still want.  They are on the decode memories, the apply
// kernel's wide operands and outputs, the scans' token tiles, the outputs of the wide contractions, and those
// operands of the chunk kernels that nobody reads again (said where they are loaded); not on the scans'
// snapshots, which the next kernel reads.
// Eight elements held as loaded (no conversion): the unit of register prefetching.
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
    bf16x8 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const bf16x8 *>(p); }
    __device__ __forceinline__ void store(bf16_t *p) const { *reinterpret_cast<bf16x8 *>(p) = v; }
    __device__ __forceinline__ void load_nt(const bf16_t *p) { v = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(p)); }
    __device__ __forceinline__ void store_nt(bf16_t *p) const { __builtin_nontemporal_store(v, reinterpret_cast<bf16x8 *>(p)); }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (bf16_t)0.f;
    }
    __device__ __forceinline__ bf16_t get(int e) const { return v[e]; }
    __device__ __forceinline__ void set(int e, bf16_t x) { v[e] = x; }
    __device__ __forceinline__ void keep(bool live) {   // zero unless live, by register select
        bf16x8 z;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (bf16_t)0.f;
        v = live ? v : z;
    }
};
template <> struct Raw8<float> {
    f32x4 lo, hi;
    __device__ __forceinline__ void load(const float *p) {
        lo = *reinterpret_cast<const f32x4 *>(p);
        hi = *reinterpret_cast<const f32x4 *>(p + 4);
    }
    __device__ __forceinline__ void store(float *p) const {
        *reinterpret_cast<f32x4 *>(p) = lo;
        *reinterpret_cast<f32x4 *>(p + 4) = hi;
    }
    __device__ __forceinline__ void load_nt(const float *p) {
        lo = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
        hi = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p + 4));
    }
    __device__ __forceinline__ void store_nt(float *p) const {
        __builtin_nontemporal_store(lo, reinterpret_cast<f32x4 *>(p));
        __builtin_nontemporal_store(hi, reinterpret_cast<f32x4 *>(p + 4));
    }
    __device__ __forceinline__ void zero() { lo = f32x4{0.f, 0.f, 0.f, 0.f}; hi = lo; }
    __device__ __forceinline__ float get(int e) const { return e < 4 ? lo[e] : hi[e - 4]; }
    __device__ __forceinline__ void set(int e, float x) { if (e < 4) lo[e] = x; else hi[e - 4] = x; }
    __device__ __forceinline__ void keep(bool live) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        lo = live ? lo : z;
        hi = live ? hi : z;
    }
};

// four consecutive elements of one row, from fp32
__device__ __forceinline__ void store4(bf16_t *p, float a, float b, float c, float d)
{
    bf16x4 x;
    x[0] = (bf16_t)a; x[1] = (bf16_t)b; x[2] = (bf16_t)c; x[3] = (bf16_t)d;
    *reinterpret_cast<bf16x4 *>(p) = x;
}
__device__ __forceinline__ void store4(float *p, float a, float b, float c, float d)
{
    *reinterpret_cast<f32x4 *>(p) = f32x4{a, b, c, d};
}

// ----------------------------------------------------------------------------
// Chunk map: which tokens a chunk covers.  Batch form: arithmetic.  Packed form:
// a table the prepare kernel writes into the workspace.
// ----------------------------------------------------------------------------
struct ChunkMap {
    const int32_t *table;   // packed: [4 * n_chunk_slots] = {seq, tok0, len, index in seq}; batch: NULL
    const int32_t *seq_tab; // packed: [4 * n_seqs] = {first chunk id, number of chunks, first token, tokens}
    const int32_t *seg_base; // packed, scans in segments: [n_seqs + 1] running count of scan segments before each sequence, chunks per segment
    int32_t T;              // batch: tokens per sequence
    int32_t chunk;          // tokens per chunk (C in Appendix A)
    int32_t chunks_per_seq; // batch: ceil(T / chunk)
    int32_t n_chunk_slots;  // upper bound on the number of chunks (grid size)
};

struct ChunkInfo { int seq, tok0, len, idx; };

__device__ __forceinline__ bool chunk_lookup(const ChunkMap &cm, int c, ChunkInfo &ci)
{
    if (cm.table) {
        ci.seq = cm.table[4 * c + 0];
        ci.tok0 = cm.table[4 * c + 1];
        ci.len = cm.table[4 * c + 2];
        ci.idx = cm.table[4 * c + 3];
        return ci.len > 0;
    }
    ci.seq = c / cm.chunks_per_seq;
    ci.idx = c - ci.seq * cm.chunks_per_seq;
    const int off = ci.idx * cm.chunk;
    ci.tok0 = ci.seq * cm.T + off;
    ci.len = min(cm.chunk, cm.T - off);
    return true;
}

// Which (chunk, head) a workgroup of a chunk-parallel kernel takes, for a grid of
// (n_chunk_slots, H) workgroups dispatched x-fastest.  Workgroups are handed out so that all
// sequences and heads advance through their chunks together, newest_first = from the last chunk
// of every sequence backwards: a kernel that follows a scan then starts on the snapshots the scan
// wrote last, which are the ones still sitting in the memory-side cache.
__device__ __forceinline__ void chunk_order(const ChunkMap &cm, int H, bool newest_first, int &chunk, int &head)
{
    const int b = blockIdx.y * gridDim.x + blockIdx.x;
    if (cm.table) {
        const int c = b / H;
        head = b - c * H;
        chunk = newest_first ? cm.n_chunk_slots - 1 - c : c;
        return;
    }
    const int n = cm.chunks_per_seq, per = (cm.n_chunk_slots / n) * H;   // per: (sequence, head) pairs
    const int rank = b / per, rem = b - rank * per;
    const int seq = rem / H;
    head = rem - seq * H;
    chunk = seq * n + (newest_first ? n - 1 - rank : rank);
}

// First chunk id, number of chunks and first token of sequence s.
__device__ __forceinline__ void seq_lookup(const ChunkMap &cm, int s, int &chunk0, int &nchunks, int &tok0, int &ntok)
{
    if (cm.seq_tab) {
        chunk0 = cm.seq_tab[4 * s + 0];
        nchunks = cm.seq_tab[4 * s + 1];
        tok0 = cm.seq_tab[4 * s + 2];
        ntok = cm.seq_tab[4 * s + 3];
    } else {
        chunk0 = s * cm.chunks_per_seq;
        nchunks = cm.chunks_per_seq;
        tok0 = s * cm.T;
        ntok = cm.T;
    }
}

// ----------------------------------------------------------------------------
// Gates (Algorithm 1, chunk_cumsum, plus the write intensity).
// ----------------------------------------------------------------------------
// (the maximum that keeps a NaN; fmaxf would turn it into the floor)
__device__ __forceinline__ float floor_gate(float x) { return __builtin_elementwise_maximum(x, kGateFloor); }

// log gate from a gate logit: logsigmoid(u) / tau = -(log(1 + exp(-|u|)) + max(-u, 0)) / tau, and its slope
__device__ __forceinline__ float log_gate_from_logit(float u, float tau)
{
    return -(log1pf(__expf(-fabsf(u))) + fmaxf(-u, 0.f)) / tau;
}
__device__ __forceinline__ float log_gate_slope(float u, float tau) { return 1.f / ((1.f + __expf(u)) * tau); }

// Gates of one slot's run of tokens in a chunk-wide layout: thread tid owns slot tid % M and the C / P tokens
// from (tid / M) * C / P on.  Log gates are floored at kGateFloor, rows past the end of the chunk are g = 0, s = 0.
// GEN: the general form, in which the write intensity may come from an array of its own
// (sin: [len][M] fp32, same layout as g; NULL = 1 - exp(g) as above), and the array g may hold gate
// LOGITS u instead of log gates: with tau > 0 the log gate is logsigmoid(u) / tau, the layer's gate
// alpha = sigmoid(W x)^(1/tau) of Section 3.3 (tau = 0: g is the log gate itself).
template <int M, int NT, int C, bool GEN = false> struct GatePrep {
    static constexpr int P = NT / M;     // token partitions
    static constexpr int TP = C / P;     // tokens per partition
    static_assert(NT % M == 0 && C % P == 0, "slots and tokens split evenly over the threads");
    float gv[TP];
    float sv[GEN ? TP : 1];
    bool given = false;
    float tau = 0.f;
    // Issues the loads (rows clamped into the chunk).
    __device__ __forceinline__ void load(const float *g, size_t gld, int len, int tid, const float *sin = nullptr,
                                         float gate_tau = 0.f)
    {
        if (GEN) tau = gate_tau;
        const int i = tid % M, part = tid / M;
#pragma unroll
        for (int tt = 0; tt < TP; ++tt) gv[tt] = g[(size_t)min(part * TP + tt, len - 1) * gld + i];
        if (GEN && sin) {   // uniform over the grid
            given = true;
#pragma unroll
            for (int tt = 0; tt < (GEN ? TP : 1); ++tt) sv[tt] = sin[(size_t)min(part * TP + tt, len - 1) * gld + i];
        }
    }
    // Log gate and write intensity of this thread's token tt (0 and 0 past the end of the chunk).
    __device__ __forceinline__ void token(float &x, float &sx, int tt, bool live) const
    {
        float graw = gv[tt];
        if (GEN && tau > 0.f) graw = log_gate_from_logit(graw, tau);
        x = live ? floor_gate(graw) : 0.f;
        sx = -expm1f(x);   // as in the decode step: a memory is handed from one to the other
        if (GEN && given) sx = sv[GEN ? tt : 0];
        sx = live ? sx : 0.f;
    }
};

// ----------------------------------------------------------------------------
// Read-outs: how the slot scores z become the read weights p.  Softmax over the slots is the
// method's own (Eq. (gsa)); the element-wise ones are the ablations of Section 4 (no softmax,
// Swish, ReLU, ReLU squared).  Values match gsa_readout in the C header.
// ----------------------------------------------------------------------------
enum Readout { kReadSoftmax = 0, kReadIdentity = 1, kReadSwish = 2, kReadRelu = 3, kReadRelu2 = 4 };

__device__ __forceinline__ float readout_value(int ro, float z)
{
    const float sg = 1.f / (1.f + __expf(-z)), zp = fmaxf(z, 0.f);
    return ro == kReadIdentity ? z : ro == kReadSwish ? z * sg : ro == kReadRelu ? zp : zp * zp;
}
__device__ __forceinline__ float readout_slope(int ro, float z)
{
    const float sg = 1.f / (1.f + __expf(-z));
    return ro == kReadIdentity ? 1.f : ro == kReadSwish ? sg + z * sg * (1.f - sg) : ro == kReadRelu ? (z > 0.f ? 1.f : 0.f)
                                                                                               : 2.f * fmaxf(z, 0.f);
}

// ----------------------------------------------------------------------------
// Feature map on q, k, v (Section 3.3: the layer feeds phi(W x) with phi = Swish into the operator).
// With the option on, the q, k, v arguments hold the raw projections and every kernel applies
// phi(x) = x sigmoid(x) to what it has just loaded, in registers: the values are rounded to the I/O
// type once more (they are matrix-core operands), and dq, dk, dv leave multiplied by the slope at
// the raw value.  The arithmetic runs under the loads that are still in flight, which is what makes
// this cheaper than a pass of its own over the three tensors.
// ----------------------------------------------------------------------------
__device__ __forceinline__ float swish_value(float x) { return x * __builtin_amdgcn_rcpf(1.f + __expf(-x)); }
__device__ __forceinline__ float swish_slope(float x)
{
    const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-x));
    return sg * (1.f + x * (1.f - sg));
}

// Loads in this library are never placed under a data-dependent branch (the compiler would have to wait for
// each one before leaving the branch, which serialises them): callers clamp the row index into
// the valid range so the load is always legal, and rows past the end are zeroed by a register
// select -- or left as finite duplicates of the last row where they only ever meet zero weights.

// ----------------------------------------------------------------------------
// Transposed token tile in LDS: XT[c][t] for c < ncols, t < C, row stride C + kPad,
// with the 8-token blocks of row c XOR-swizzled by (c/8) so that the transposing writes
// (one thread owns two adjacent tokens of 8 consecutive columns) spread over all banks
// and fragment reads stay 16-byte aligned.
// ----------------------------------------------------------------------------
template <int C> __device__ __forceinline__ int xt_off(int c, int t, int ld)
{
    constexpr int NB = C / 8;
    return c * ld + ((((t >> 3) ^ (c >> 3)) & (NB - 1)) << 3) + (t & 7);
}

// ----------------------------------------------------------------------------
// bf16 tile [rows][64 columns] in LDS as it lies in memory, read by the transposing LDS load, which hands a lane four
// consecutive rows of one column.  Rows are 128 bytes.  Their 8-byte pieces are XOR-swizzled so that the 32 lanes of half a
// transposing load (eight rows, four pieces each, STEP pieces apart) touch every bank once.
// ----------------------------------------------------------------------------
template <int STEP> struct TrTile {
    static constexpr int kCols = 64;
    static constexpr int B0 = STEP == 1 ? 2 : 0, B1 = STEP == 4 ? 1 : 3;   // the two address bits of a piece that STEP leaves free
    __device__ static __forceinline__ int swz(int row) { return (((row >> 1) & 1) << B0) | (((row >> 3) & 1) << B1); }
    __device__ static __forceinline__ void put(bf16_t *tile, int row, int cg, bf16x8 x)
    {
        const int f = swz(row);
        const bf16x8 y = __builtin_shufflevector(x, x, 4, 5, 6, 7, 0, 1, 2, 3);
        *reinterpret_cast<bf16x8 *>(tile + row * kCols + ((cg ^ (f >> 1)) << 3)) = (B0 == 0 && (f & 1)) ? y : x;
    }
    // Eight rows of one column: lane l of 16 gets element l%4 of the piece (of four columns) that lane l/4 of the 16
    // names, so each lane names the piece for lanes 4*(l%4) .. +3.  lane_off: where a lane of the wave reads, relative to the
    // first of 32 rows; frag: rows 8*(l/16) .. +7 from there.  (The swizzle of a row is that of the row 4, 16 or 32 further.)
    __device__ static __forceinline__ uint32_t lane_off(int piece, int lane)
    {
        const int row = 8 * (lane >> 4) + ((lane & 15) >> 2);
        return (uint32_t)(row * kCols + ((piece ^ swz(row)) << 2));
    }
    __device__ static __forceinline__ bf16x8 frag(const bf16_t *p)
    {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * kCols));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// Token tile held in registers between the global load and the transposing LDS write.
// The tile is C tokens x NCOLS columns; thread (tid) owns row pairs and 8-column groups.
template <typename T, int C, int NCOLS, int NT> struct TokTile {
    static constexpr int NVEC = (C / 2) * (NCOLS / 8);          // (row pair, column group) items
    static constexpr int PER = (NVEC + NT - 1) / NT;
    Raw8<T> a[PER], b[PER];
    bool la[PER], lb[PER];   // whether the row really exists (else it is written as zeros)
    // src: row 0 of the tile, column 0 of the slice; rows >= len read as zero; columns >= ncols skipped.
    // Only issues the loads: the masking of missing rows is left to store_transposed, so that nothing
    // here waits for the data (a select right after the load would stall the wave for the full memory
    // latency before it could issue anything else).
    template <bool NTL = false>
    __device__ __forceinline__ void load(const T *src, size_t gld, int len, int ncols, int tid)
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            int idx = tid + NT * u;
            const bool in = idx < NVEC;
            idx = in ? idx : 0;
            const int rp = idx / (NCOLS / 8);
            int cg = idx - rp * (NCOLS / 8);
            const bool ok = in && cg * 8 < ncols;
            cg = ok ? cg : 0;
            const int r0 = min(2 * rp, len - 1), r1 = min(2 * rp + 1, len - 1);
            if (NTL) { a[u].load_nt(src + (size_t)r0 * gld + cg * 8); b[u].load_nt(src + (size_t)r1 * gld + cg * 8); }
            else { a[u].load(src + (size_t)r0 * gld + cg * 8); b[u].load(src + (size_t)r1 * gld + cg * 8); }
            la[u] = ok && 2 * rp < len;
            lb[u] = ok && 2 * rp + 1 < len;
        }
    }
    // The same for a column slice of one part of a memory snapshot (C slots, all present; the part is
    // tiled by kSnapTile columns): col0 = first column of the slice.
    template <bool NTL = false>
    __device__ __forceinline__ void load_snapshot(const T *part, int col0, int ncols, int tid)
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            int idx = tid + NT * u;
            const bool in = idx < NVEC;
            idx = in ? idx : 0;
            const int rp = idx / (NCOLS / 8);
            int cg = idx - rp * (NCOLS / 8);
            const bool ok = in && cg * 8 < ncols;
            cg = ok ? cg : 0;
            const T *p = part + snap_col<C>(col0 + cg * 8);
            if (NTL) { a[u].load_nt(p + (2 * rp) * kSnapTile); b[u].load_nt(p + (2 * rp + 1) * kSnapTile); }
            else { a[u].load(p + (2 * rp) * kSnapTile); b[u].load(p + (2 * rp + 1) * kSnapTile); }
            la[u] = lb[u] = ok;
        }
    }
    // PHI: with the feature map applied on the way (see swish_value)
    template <bool PHI = false>
    __device__ __forceinline__ void store_transposed(T *XT, int ld, int ncols, int tid) const
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = tid + NT * u;
            const int rp = idx / (NCOLS / 8), cg = idx - rp * (NCOLS / 8);
            if (idx < NVEC && cg * 8 < ncols) {
                Raw8<T> x = a[u], y = b[u];
                x.keep(la[u]);
                y.keep(lb[u]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // two 2-byte stores: measured faster here than one packed 4-byte store
                    T *dst = XT + xt_off<C>(cg * 8 + e, 2 * rp, ld);
                    dst[0] = PHI ? from_f32<T>(swish_value((float)x.get(e))) : x.get(e);
                    dst[1] = PHI ? from_f32<T>(swish_value((float)y.get(e))) : y.get(e);
                }
            }
        }
    }
};

}  // namespace gsa
