// The FP32 direction's matrix-core operands: their places in the workspace and
// the packing of the particles' rows, which the median's Gram form reads too.
#ifndef STAMP_OPERANDS32_H
#define STAMP_OPERANDS32_H

#include "common.h"

namespace stamp {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

struct View32 {  // one problem's FP32 matrix-core workspace
    const float* ctr;
    float* xr;   // [npad][4 ks]: row i, lane group q holds coordinates q ks .. q ks + ks - 1
    float* nrm;  // [npad]: |x_i|^2
    float* vt;   // [npad / 16][ot][16 columns n][16 rows j]: X[j][16 o + n] at 16 n + j of tile (j/16, o)
    float* part; // [splits32][16 ot][npad]
    __bf16* xs3; // split form: [npad][3][32], row i's part p at (3 i + p) 32 (slot 31: -|x_i|^2 / 2's part)
    __bf16* vs3; // split form: part p of V at p npad 16 ot, as [npad / 32][16 ot][32] in MFMA k order
    const SelState* sel;
};

__device__ __forceinline__ View32 view32(const SvgdLayout& L, char* base) {
    View32 v;
    v.ctr = reinterpret_cast<const float*>(base + L.ctr_off);
    v.xr = reinterpret_cast<float*>(base + L.x32_off);
    v.nrm = reinterpret_cast<float*>(base + L.n32_off);
    v.vt = reinterpret_cast<float*>(base + L.v32_off);
    v.part = reinterpret_cast<float*>(base + L.part_off);
    v.xs3 = reinterpret_cast<__bf16*>(base + L.xs3_off);
    v.vs3 = reinterpret_cast<__bf16*>(base + L.vs3_off);
    v.sel = sel_state(base, L.sel_off);
    return v;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// Two values as packed BF16 pairs (element 0 in the low half): one
// conversion, and the pair's values back in FP32 by shift and mask.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf16x2));
}
__device__ __forceinline__ float pair_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float pair_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// v[u] = hi[u] + mid[u] + lo[u] for eight values (BF16 parts; the two
// differences are exact in FP32)
__device__ __forceinline__ void split3(const float (&v)[8], bf16x8& hi, bf16x8& mid, bf16x8& lo) {
    u4v h, m, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        h[q] = bf16_pair(v[2 * q], v[2 * q + 1]);
        const float ra = v[2 * q] - pair_lo(h[q]), rb = v[2 * q + 1] - pair_hi(h[q]);
        m[q] = bf16_pair(ra, rb);
        l[q] = bf16_pair(ra - pair_lo(m[q]), rb - pair_hi(m[q]));
    }
    hi = __builtin_bit_cast(bf16x8, h);
    mid = __builtin_bit_cast(bf16x8, m);
    lo = __builtin_bit_cast(bf16x8, l);
}

// ---- operands: 64 rows per 256 threads, lane group q = threadIdx.x / 64 takes
// the coordinates l = 4 s + q (its MFMA lane group's values), so a thread's
// stores of xr are contiguous and its loop is a quarter of the dimension.
// The centred rows and their norms come first (the median's Gram form reads
// them); X = [-(2/h) x | 1 | 0] needs h and comes after the median.
// In split form the rows are also written as three BF16 parts (thread (r, q)
// the coordinates 8 q .. 8 q + 7 of row r, as the MFMA lane group q reads
// them), which the median's Gram form and the contraction both read.  The
// spare slot 31 (d <= 31) holds e_i = -|x_i|^2 / 2's parts: as a column
// operand against (1, 0, 0) in the row operand's slot, the contraction's Gram
// adds e_j itself; the median's row operand zeroes the slot.
template <int GROUPS = 1>
__device__ void pack32_x_rows(int N, int d, int ks, int row0, const float* __restrict__ theta, const View32& v,
                              bool parts) {
    __shared__ float parts4[GROUPS][4][64];
    const int r = threadIdx.x & 63, q = (threadIdx.x >> 6) & 3, grp = threadIdx.x >> 8;
    float(&part)[4][64] = parts4[GROUPS == 1 ? 0 : grp];
    const int i = row0 + 64 * grp + r;
    const int kd = 4 * ks;
    float nrm = 0.0f;
    for (int s = 0; s < ks; ++s) {
        const int l = 4 * s + q;
        const float x = (i < N && l < d) ? theta[(int64_t)l * N + i] - v.ctr[l] : 0.0f;
        nrm = fmaf(x, x, nrm);
        v.xr[(int64_t)i * kd + q * ks + s] = x;
    }
    part[q][r] = nrm;
    __syncthreads();
    if (q == 0) v.nrm[i] = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
    __syncthreads();
    if (parts) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int l = 8 * q + u;
            x[u] = (i < N && l < d) ? theta[(int64_t)l * N + i] - v.ctr[l] : 0.0f;
        }
        if (q == 3) x[7] = -0.5f * ((part[0][r] + part[1][r]) + (part[2][r] + part[3][r]));
        bf16x8 p0, p1, p2;
        split3(x, p0, p1, p2);
        __bf16* o = v.xs3 + (int64_t)i * 96 + 8 * q;
        *reinterpret_cast<bf16x8*>(o) = p0;
        *reinterpret_cast<bf16x8*>(o + 32) = p1;
        *reinterpret_cast<bf16x8*>(o + 64) = p2;
    }
}

}  // namespace
}  // namespace stamp

#endif  // STAMP_OPERANDS32_H
