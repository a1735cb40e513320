// The wide contractions of a chunk inside the kernel that made its small matrices (bf16).
//
//     out[C x cols] = A_tok[C x C] X[C x cols]  +  A_slot[C x m] St[m x cols]
//
// is what apply_kernel evaluates from small matrices in global memory, one workgroup per column slice.  Here one
// workgroup walks all 64-column units of all outputs of its (chunk, head), with the small matrices in LDS:
// they never leave the chip, and what the same workgroup has read just before (q, k, the memory gradient) comes
// from the caches.  Both operands of a unit are [rows][64 columns] tiles, stored in LDS as they are and read
// by the transposing LDS load, which hands a lane four consecutive rows of one column; tiles of the unit after
// next are in flight while a unit multiplies, and there is one barrier per unit.
#pragma once
#include "gsa_common.h"

namespace gsa {

template <int M> struct Wide {
    static constexpr int C = Geo<bf16_t>::C, NT = Geo<bf16_t>::NT;
    static constexpr int KM = (M < 32) ? 32 : M;              // slot rows, padded with zeros to the contraction depth
    static constexpr int kCols = TrTile<2>::kCols;
    static constexpr size_t szBuf = sizeof(bf16_t) * (KM + C) * kCols;   // slot tile, token tile
    static constexpr size_t szTok = sizeof(bf16_t) * C * C, szSlot = sizeof(bf16_t) * C * KM;   // A_tok [C][C], A_slot [C][KM]
    static constexpr size_t szEx = sizeof(bf16_t) * C * kCols;   // the rows of a unit on their way out, 16 per wave
    // Element (row, col) of a matrix with rows of K elements: 16-byte pieces are XOR-swizzled so that the same piece of 16
    // rows lies in all banks (no padding: with 64 slots chunk_intra's LDS is exactly half of a CU's).
    template <int K> __device__ static __forceinline__ int at(int row, int col)
    {
        constexpr int R = K < 128 ? 128 / K : 1;   // rows per 256 bytes
        return row * K + ((((col >> 3) ^ (row / R)) & (K / 8 - 1)) << 3) + (col & 7);
    }
    static constexpr int SV = KM * kCols / 8 / NT, XV = C * kCols / 8 / NT;
    static_assert(SV * NT * 8 == KM * kCols && XV * NT * 8 == C * kCols, "whole 16-byte pieces per thread");

    // Fragment of column tile ni: lane l gets column 32*(ni/2) + 8*((l%16)/4) + 4*(ni%2) + l%4 and the rows k0 +
    // 8*(l/16) .. +7, so that a lane of the product D[column][token] holds columns 32*(ni/2) + 8*(l/16) + 4*(ni%2) + j:
    // two runs of eight, and the four lanes that share a token store 64 bytes in a row.
    __device__ static __forceinline__ bf16x8 frag(const bf16_t *tile, int k0, int ni, int lane)
    {
        return TrTile<2>::frag(tile + k0 * kCols + TrTile<2>::lane_off(8 * (ni >> 1) + 2 * (lane & 3) + (ni & 1), lane));
    }
    struct Stage { bf16x8 s[SV], x[XV]; };
    // One unit: tile `slot` is [M][64] contiguous, rows of `tok` and `out` are `ld` elements apart.
    struct Unit { const bf16_t *slot, *tok; bf16_t *out; size_t ld; const bf16_t *At, *As; };

    __device__ static __forceinline__ void fetch(Stage &st, const Unit &u, int len, int tid)
    {
#pragma unroll
        for (int v = 0; v < SV; ++v) {
            const int idx = tid + NT * v;
            st.s[v] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(u.slot + (size_t)(M < KM ? min(idx, M * 8 - 1) : idx) * 8));
        }
#pragma unroll
        for (int v = 0; v < XV; ++v) {
            const int idx = tid + NT * v;
            st.x[v] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(u.tok + (size_t)min(idx >> 3, len - 1) * u.ld + (idx & 7) * 8));
        }
    }
    __device__ static __forceinline__ void to_lds(const Stage &st, bf16_t *buf, int len, int tid)
    {
        const bf16x8 zero = Atom<bf16_t>::zero();
#pragma unroll
        for (int v = 0; v < SV; ++v) {
            const int idx = tid + NT * v;
            TrTile<2>::put(buf, idx >> 3, idx & 7, (M < KM && idx >= M * 8) ? zero : st.s[v]);
        }
#pragma unroll
        for (int v = 0; v < XV; ++v) {
            const int idx = tid + NT * v;
            TrTile<2>::put(buf + KM * kCols, idx >> 3, idx & 7, (idx >> 3) < len ? st.x[v] : zero);   // missing rows are zero
        }
    }
    // This wave's 16 tokens of one unit.  FULL: every token of the chunk exists (the store is then unconditional,
    // which keeps the number of memory operations in flight known).
    template <bool FULL>
    __device__ static __forceinline__ void multiply(const Unit &u, const bf16_t *buf, bf16_t *ex, int len, int rowb, int lane)
    {
        const int r = lane & 15, g = lane >> 4;
        f32x4 acc[4];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[ni] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k0 = 0; k0 < KM; k0 += 32) {
            const bf16x8 a = Atom<bf16_t>::load(u.As + at<KM>(rowb + r, k0 + 8 * g));
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) Atom<bf16_t>::mma(acc[ni], frag(buf, k0, ni, lane), a);
        }
#pragma unroll
        for (int k0 = 0; k0 < C; k0 += 32) {
            const bf16x8 a = Atom<bf16_t>::load(u.At + at<C>(rowb + r, k0 + 8 * g));
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) Atom<bf16_t>::mma(acc[ni], frag(buf + KM * kCols, k0, ni, lane), a);
        }
        // The wave's 16 rows meet in LDS of its own and leave in whole lines.  (Straight from the registers a store takes 16 bytes of
        // each of 16 rows per quarter of the wave: 8 x 2048 tokens, 4 heads, 64 slots, d = 512 forward 82.3 -> 80.1 us, d = 640 98.7 -> 92.8 and
        // intra-chunk gradients 254 -> 241; 32 slots 73.5 -> 70.8 and 153 -> 148.)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 y;
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = (bf16_t)acc[2 * h + (j >> 2)][j & 3];
            *reinterpret_cast<bf16x8 *>(ex + at<kCols>(r, 32 * h + 8 * g)) = y;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = 8 * h + (lane >> 3);
            const bf16x8 y = *reinterpret_cast<const bf16x8 *>(ex + at<kCols>(row, (lane & 7) * 8));
            if (FULL || rowb + row < len)
                __builtin_nontemporal_store(y, reinterpret_cast<bf16x8 *>(u.out + (size_t)(rowb + row) * u.ld + (lane & 7) * 8));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // All units, unit(i) for i in [0, n).  sa, sb: units 0 and 1 as fetched by the caller.  smem: two buffers of szBuf;
    // out: szEx;
    // the first must be free, the second is first written behind a barrier.  The small matrices must be in
    // LDS (a barrier follows the first write of a tile).  All threads of the workgroup must call it.
    template <bool FULL, typename F>
    __device__ static __forceinline__ void walk(F &&unit, int n, Stage &sa, Stage &sb, unsigned char *smem, unsigned char *out, int len, int tid)
    {
        const int lane = tid & 63, rowb = 16 * __builtin_amdgcn_readfirstlane(tid >> 6);
        bf16_t *const ex = reinterpret_cast<bf16_t *>(out) + rowb * kCols;
        bf16_t *b0 = reinterpret_cast<bf16_t *>(smem), *b1 = reinterpret_cast<bf16_t *>(smem + szBuf);
        to_lds(sa, b0, len, tid);
        __builtin_amdgcn_sched_barrier(0);
        fetch(sa, unit(min(2, n - 1)), len, tid);
        __syncthreads();
        // the refills are unconditional (past the end they repeat the last unit)
        auto step = [&](Stage &nx, int i, bf16_t *cur, bf16_t *next) {
            multiply<FULL>(unit(i), cur, ex, len, rowb, lane);
            to_lds(nx, next, len, tid);
            __builtin_amdgcn_sched_barrier(0);
            fetch(nx, unit(min(i + 3, n - 1)), len, tid);
            __syncthreads();
        };
        int i = 0;
        for (; i + 1 < n; i += 2) {
            step(sb, i, b0, b1);
            step(sa, i + 1, b1, b0);
        }
        if (i < n) multiply<FULL>(unit(i), b0, ex, len, rowb, lane);
    }
};

}  // namespace gsa
