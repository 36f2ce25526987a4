// Element-level building blocks shared by the AxLocal kernels (internal header): work-group
// shapes per order and the one-dimensional D-contractions.
#pragma once

#include "ax_internal.h"

namespace ax {

// GEO_TRIL: trilinear with the per-node scale lam = 0.125 w / det(8J) read from memory (the
// partial recomputation of Sec. 4.2.2): no determinant and no division in the kernel.
// GEO_HELM: the trilinear Helmholtz operator with merged scalar factors (Sec. 4.2.1): per node
// Lambda2 = lam * lambda0 scales adj(K) and Lambda3 = gwj * lambda1 the mass term.
enum { GEO_TRI = 0, GEO_PARA = 1, GEO_STORED = 2, GEO_TRIL = 3, GEO_HELM = 4 };

constexpr bool is_trilinear(int geo) { return geo == GEO_TRI || geo == GEO_TRIL || geo == GEO_HELM; }

// ---- Launch variants chosen at run time (the tuning table, ax_tune_set) ----
//
// Tuning kinds: one table entry per (order, kind, precision).
enum { TUNE_TRI = 0, TUNE_PARA = 1, TUNE_STORED = 2, TUNE_PARTIAL = 3, TUNE_HELM = 4, TUNE_BATCHED = 5,
       TUNE_KINDS = 6 };
constexpr int tune_kind_of(int geo)
{
    return geo == GEO_TRI ? TUNE_TRI : geo == GEO_PARA ? TUNE_PARA : geo == GEO_STORED ? TUNE_STORED
         : geo == GEO_TRIL ? TUNE_PARTIAL : TUNE_HELM;
}

// Shape of the per-item kernels (one element per N1^2 lanes, several elements per work-group):
// variant 0 is a 256-lane work-group holding floor(256 / N1^2) elements (at most 64); variant 1
// is the alternative the tuner may pick: half the work-group for N1 <= 8 (smaller groups, cheaper
// barriers), a larger group for N1 = 9, 10 and a tighter one for N1 = 11..13 (fewer idle lanes:
// at N1 = 12 the 256-lane group leaves 112 lanes idle, a 192-lane group 48).  N1 >= 14 has no
// alternative.
struct ItemShape {
    int epb, block;
};
constexpr ItemShape item_shape(int N1, int v)
{
    if (v == 1) {
        switch (N1) {
        case 2: return {32, 128};
        case 3: return {14, 128};
        case 4: return {8, 128};
        case 5: return {5, 128};
        case 6: return {5, 192};
        case 7: return {2, 128};
        case 8: return {2, 128};
        case 9: return {4, 384};
        case 10: return {3, 320};
        case 11: return {1, 128};
        case 12: return {1, 192};
        case 13: return {1, 192};
        default: break;
        }
    }
    return {256 / (N1 * N1) > 64 ? 64 : (256 / (N1 * N1) < 1 ? 1 : 256 / (N1 * N1)), 256};
}
constexpr bool item_has_alt(int N1) { return N1 >= 2 && N1 <= 13; }

// Register budget of the single-mesh per-item kernel, as waves per SIMD: the default (FP32 full
// form five waves except at N1 = 13, otherwise no limit beyond two) and the alternative (one wave
// more where the default is two, one fewer where it is five).
constexpr int item_waves(int N1, bool fp32, bool partial, int alt)
{
    const int d = (fp32 && !partial && N1 != 13) ? 5 : 2;
    return alt ? (d == 2 ? 3 : 4) : d;
}

// Which kernel runs when the tuning table says "auto" (measured on gfx950, GDOF/s at 2^24 nodes,
// tile against per-item kernel).  The tile kernel (FP64 N1 = 6: 200 against 190; 9: 203, 177; 10:
// 181, 161; FP32 9: 304, 305; 13: 274, 274; 15: 279, 268; partial form 13: 286, 282) except FP64
// N1 = 7, full form: the per-item kernel is that order's documented default, kept although the tile
// kernel is now the faster one there (us at 2^22.9, 2^23.6 and 2^24 nodes: 41.6, 59.7, 79.3 against
// 41.9, 63.1, 86.2); the table's kernel field selects it.
constexpr bool item_default(int N1, int geo, bool fp32) { return geo == GEO_TRI && !fp32 && N1 == 7; }

// Orders with a batched tile kernel (the single-mesh tile body walking the batch's work list):
// FP64 up to N1 = 7, FP32 up to N1 = 10.  At FP64 N1 >= 8 the kernel spills (N1 = 8: 464-496
// bytes of scratch with the tables resident, read through the constant address space or reloaded
// per row, whether or not the item descriptors are re-read at each use; 45 against 214 GDOF/s for
// the per-item kernel on sixteen order-7 meshes of 512 to 32768 elements, 8 columns).
constexpr bool batched_tile_available(int N1, bool fp32) { return fp32 ? N1 <= 10 : N1 <= 7; }

// Register budget of the batched per-order kernels: FP32 fits five waves per SIMD.
#ifndef AX_BATCH_MINW_F32
#define AX_BATCH_MINW_F32 5
#endif
constexpr int batch_waves(bool fp32) { return fp32 ? AX_BATCH_MINW_F32 : 2; }

// Orders with a per-item kernel: the full trilinear form for every order, the partial form from
// N1 = 9.
constexpr bool item_available(int N1, int geo)
{
    return (geo == GEO_TRI && N1 >= 2 && N1 <= 16) || (geo == GEO_TRIL && N1 >= 9 && N1 <= 16);
}

// Element shape of order N1 - 1.
template <int N1>
struct Shape {
    static constexpr int NT = N1 * N1;                        // lanes per element
    static constexpr int NP = N1 * N1 * N1;                   // nodes per element
    // elements per work-group: fill (nearly) whole waves while keeping LDS modest
    static constexpr int EPB = N1 == 2 ? 16 : N1 == 3 ? 7 : N1 == 4 ? 4 : N1 == 5 ? 5
                             : N1 == 6 ? 7 : N1 == 7 ? 5 : N1 == 9 ? 3 : N1 == 10 ? 3
                             : N1 == 11 ? 2 : 1;
    // the alternative elements-per-group the tuner may pick (same as EPB where there is none)
    static constexpr int EPB_ALT = N1 == 2 ? 32 : N1 == 3 ? 14 : N1 == 4 ? 8 : N1 == 5 ? 10
                                 : N1 == 6 ? 14 : N1 == 7 ? 10 : N1 == 8 ? 2 : N1 <= 11 ? 1 : EPB;
    static constexpr int BLOCK = ((EPB * NT + 63) / 64) * 64;
};

// LDS layout of a work-group: EPB elements of order N1 - 1, two fields each of
// WB-byte values, node (i, j, k) at word i + SJ j + SK k of a field, SJ = N1.
//
// The LDS serves 128 bytes per clock, G = 128 / WB lanes at a time, without a conflict when their
// words differ modulo G.  Home columns (lane i + N1 j) are consecutive words, also across elements:
// the element stride ST continues the sequence modulo G.  The r-pencils (j, k) and s-pencils (i, k)
// may be owned by any lanes, so they are dealt out such that every G lanes start at words that
// differ modulo G (make()); with a few words of padding per slice that works out almost
// perfectly at every order: 0-7 % above the conflict-free cycles (N1 = 2, 4: 27 %) where rows
// padded to an odd number of words with pencils in lane order cost 7-77 % (77 % at N1 = 6).
// Measured with those the conflicts took 0.21 of the kernel at N1 = 6 and 0.19 at N1 = 10 (FP64
// trilinear).
// N1 = 8 (slices of 64 + 2 words, 64 + 4 in FP32) moves its r-pencils as 16-byte accesses: lanes
// take them k-fastest, so 8 lanes k = 0..7 start at banks 4 bytes x 2 k (FP32: 8 j + 4 k) and
// cover all; the s-pencils are assigned so that each group of 16 lanes takes the slices k and
// k + 4 (FP32: 32 lanes, the even or the odd slices), which cover the banks too.
constexpr int tile_slice_pad(int N1, int WB)
{
    constexpr int p8[17] = {0, 0, 1, 6, 3, 4, 5, 4, 2, 1, 3, 4, 3, 0, 1, 0, 1};
    constexpr int p4[17] = {0, 0, 1, 22, 3, 4, 3, 4, 4, 3, 9, 4, 1, 0, 3, 1, 5};
    return WB == 8 ? p8[N1] : p4[N1];
}

template <int N1, int EPB, int WB>
struct TileLds {
    static constexpr int NT = N1 * N1, SJ = N1, SK = NT + tile_slice_pad(N1, WB), G = 128 / WB;
    static constexpr bool V16 = N1 == 8;  // r-pencils start on 16-byte boundaries
    static constexpr int FS = N1 == 8 ? 8 * SK : (N1 - 1) * SK + NT;
    static constexpr int ST = EPB == 1 || N1 == 8 ? 2 * FS : 2 * FS + ((NT - 2 * FS) % G + G) % G;
    static constexpr int WORDS = (EPB - 1) * ST + 2 * FS;
    static constexpr int LANES = EPB * NT;
    static_assert(WORDS <= 0xffff, "pencil offsets are 16-bit words");
    static __device__ __forceinline__ constexpr int pos(int i, int j, int k) { return k * SK + j * SJ + i; }

    // first word of the r-pencil and of the s-pencil each lane owns
    struct Pencils {
        uint16_t r[LANES], s[LANES];
    };
    // `w`: the pencils' first words in any order; on return every G of them differ modulo G as far
    // as possible (each group takes one pencil from every residue class, fullest classes first)
    static constexpr void deal(uint16_t* w)
    {
        uint16_t c[G][LANES] = {};
        int n[G] = {}, left = LANES;
        for (int q = 0; q < LANES; ++q) c[w[q] % G][n[w[q] % G]++] = w[q];
        for (int q = 0; q < LANES;) {
            const int need = left < G ? left : G;
            bool used[G] = {};
            for (int t = 0; t < need; ++t) {
                int best = -1;
                for (int r = 0; r < G; ++r)
                    if (!used[r] && n[r] > 0 && (best < 0 || n[r] > n[best])) best = r;
                if (best < 0)
                    for (int r = 0; r < G; ++r)
                        if (n[r] > 0 && (best < 0 || n[r] > n[best])) best = r;
                used[best] = true;
                w[q++] = c[best][--n[best]];
                --left;
            }
        }
    }
    static constexpr Pencils make()
    {
        Pencils p{};
        for (int e = 0; e < EPB; ++e)
            for (int l = 0; l < NT; ++l) {
                int ra = l % N1, rb = l / N1, sa = l % N1, sb = l / N1;
                if (N1 == 8) {
                    ra = l / N1;
                    rb = l % N1;
                    sb = WB == 8 ? ((l >> 3) & 1) * 4 + (l >> 4) : 2 * ((l >> 3) & 3) + (l >> 5);
                }
                p.r[e * NT + l] = (uint16_t)(e * ST + ra * SJ + rb * SK);
                p.s[e * NT + l] = (uint16_t)(e * ST + sa + sb * SK);
            }
        if (N1 != 8) {
            deal(p.r);
            deal(p.s);
        }
        return p;
    }
    static constexpr Pencils pencils = make();
};

// An r-pencil: contiguous words, moved as 16-byte accesses where the layout aligns them.
template <typename L, int N1, typename T>
__device__ __forceinline__ void rpencil_read(const T* F, T* p)
{
    if constexpr (L::V16) {
        constexpr int W = 16 / sizeof(T);  // values per 16-byte access
        typedef T v16 __attribute__((ext_vector_type(W)));
        const v16* q = reinterpret_cast<const v16*>(F);
#pragma unroll
        for (int m = 0; m < N1 / W; ++m) {
            const v16 v = q[m];
#pragma unroll
            for (int u = 0; u < W; ++u) p[W * m + u] = v[u];
        }
    } else {
#pragma unroll
        for (int n = 0; n < N1; ++n) p[n] = F[n];
    }
}

template <typename L, int N1, typename T>
__device__ __forceinline__ void rpencil_write(T* F, const T* o)
{
    if constexpr (L::V16) {
        constexpr int W = 16 / sizeof(T);
        typedef T v16 __attribute__((ext_vector_type(W)));
        v16* q = reinterpret_cast<v16*>(F);
#pragma unroll
        for (int m = 0; m < N1 / W; ++m) {
            v16 v;
#pragma unroll
            for (int u = 0; u < W; ++u) v[u] = o[W * m + u];
            q[m] = v;
        }
    } else {
#pragma unroll
        for (int a = 0; a < N1; ++a) F[a] = o[a];
    }
}

// Waves per SIMD the register allocation of the prefetching (tile) kernel must allow, by its form and,
// for the trilinear forms, by whether it is the single-column kernel (`one`) or keeps the factor
// coefficients between columns (17 values more).  Chosen by timing every budget on every form (2^23.6
// nodes; in brackets the time against one wave more or, where given, fewer).
//   FP64: four to N1 = 8 and three above (natural use 110-168 VGPRs).  One fewer for the Helmholtz form
// at N1 = 4 (0.89), 7 (0.90; columns 0.88) and 8 (late_prefetch), and for its columns at N1 = 11 (0.84,
// 26 spills at three); two for it from N1 = 13 and for columns at 12 (184-224 VGPRs; at three 1.2 to 2.3
// times the time); two at N1 = 15, whose LDS admits no third group (stored factors 0.92, trilinear
// columns 0.91, partial 0.88), and at 16; stored factors there at one, whose LDS still admits two groups, so
// that the compiler holds a column's 96 factor loads in flight (248 VGPRs, 168 at two: 0.92 with two columns).
// At N1 = 10, 12, 13 and 14 some forms spill 4 to 19 at three and are no slower.
//   FP32: five (96 VGPRs); four for the trilinear form to N1 = 12 (single columns at N1 = 4 and 8 fit
// five: 0.97, 0.97 to 1.0; at N1 = 10 five spills 8 and is 1-3 % faster from 2^23.6 nodes, 6 % slower below
// 2^22), the Helmholtz form, stored factors at N1 = 8 (0.96; two columns 0.89) and partial columns at N1 = 2
// (0.81), 8 (0.70, 22 spills at five) and 11 (0.87); three for columns of the Helmholtz form at N1 = 11 and
// 12 (0.83) and the partial one at 12 (0.89).
constexpr int tile_waves(int N1, int geo, bool fp32, bool one)
{
    if (fp32) {
        if (!one && ((geo == GEO_HELM && (N1 == 11 || N1 == 12)) || (geo == GEO_TRIL && N1 == 12))) return 3;
        if (geo == GEO_HELM || (geo == GEO_STORED && N1 == 8)) return 4;
        if (geo == GEO_TRI) return N1 <= 12 && !(one && (N1 == 4 || N1 == 8)) ? 4 : 5;
        return !one && geo == GEO_TRIL && (N1 == 2 || N1 == 8 || N1 == 11) ? 4 : 5;
    }
    if (geo == GEO_HELM) return N1 >= 13 || (!one && N1 >= 11) ? 2 : N1 == 4 || N1 >= 7 ? 3 : 4;
    return N1 <= 8 ? 4 : N1 <= 14 ? 3 : geo == GEO_STORED && N1 == 16 ? 1 : 2;
}

// Coefficient sources of the contractions.  CoefResident reads the basis tables as they are
// (kernel arguments: the compiler keeps every coefficient it needs in scalar registers).
// CoefReload reads them through a pointer into the kernel-argument segment that is made opaque
// before each output row, so only one row of coefficients is live in scalar registers at a time
// (scalar loads from the scalar cache): for orders whose tables do not fit the scalar register
// file, where keeping them resident would spill them into vector-register lanes.
template <typename T>
struct CoefResident {
    static constexpr bool kByRow = false;
    const Basis<T>& b;
    __device__ __forceinline__ CoefResident row() const { return *this; }
    __device__ __forceinline__ T D(int q) const { return b.D[q]; }
    template <int H>
    __device__ __forceinline__ void rows(int a, T* p, T* m) const
    {
#pragma unroll
        for (int n = 0; n < H; ++n) {
            p[n] = b.P[a * H + n];
            m[n] = b.M[a * H + n];
        }
    }
    __device__ __forceinline__ T P(int q) const { return b.P[q]; }
    __device__ __forceinline__ T M(int q) const { return b.M[q]; }
    __device__ __forceinline__ T Cm(int q) const { return b.Cm[q]; }
    __device__ __forceinline__ T Rm(int q) const { return b.Rm[q]; }
};

template <typename KA>
using KargPtr = const __attribute__((address_space(4))) KA*;

// The tables behind a constant-address-space pointer (the kernel-argument segment, or a device
// table that the kernel only reads), which keeps the loads on the scalar unit.
template <typename T>
struct CoefReload {
    static constexpr bool kByRow = true;  // transposed contractions walk the tables by rows
    KargPtr<Basis<T>> k;
    __device__ __forceinline__ CoefReload row() const
    {
        KargPtr<Basis<T>> q = k;
        asm volatile("" : "+s"(q));
        return CoefReload{q};
    }
    __device__ __forceinline__ T D(int q) const { return k->D[q]; }
    __device__ __forceinline__ T Cm(int q) const { return k->Cm[q]; }
    __device__ __forceinline__ T Rm(int q) const { return k->Rm[q]; }
    __device__ __forceinline__ double xi(int q) const { return k->xi[q]; }
    __device__ __forceinline__ double w(int q) const { return k->w[q]; }
    // row a of the H by H tables P and M
    template <int H>
    __device__ __forceinline__ void rows(int a, T* p, T* m) const
    {
        copy_row<H>(&k->P[a * H], p);
        copy_row<H>(&k->M[a * H], m);
    }
    // in whole vectors, which run on into the next row or table (one scalar load of 16 or 32 bytes each)
    template <int H>
    static __device__ __forceinline__ void copy_row(KargPtr<T> q, T* r)
    {
        constexpr int V = sizeof(T) == 4 && H > 4 ? 8 : 4;
        typedef T vec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
#pragma unroll
        for (int c = 0; c < H; c += V) {
            if (H - c > V / 2) {
                const vec v = *(KargPtr<vec>)(q + c);
#pragma unroll
                for (int n = 0; n < V; ++n)
                    if (c + n < H) r[c + n] = v[n];
            } else {
#pragma unroll
                for (int n = c; n < H; ++n) r[n] = q[n];
            }
        }
    }
};

// Basis tables in device memory read through the constant address space and left to the
// compiler to keep in scalar registers or reload (loads there are invariant, so it can
// rematerialise them under register pressure instead of spilling): the resident tables of a
// kernel that receives them by pointer.
template <typename T>
struct CoefConst {
    static constexpr bool kByRow = false;
    KargPtr<Basis<T>> k;
    __device__ __forceinline__ CoefConst row() const { return *this; }
    __device__ __forceinline__ T D(int q) const { return k->D[q]; }
    template <int H>
    __device__ __forceinline__ void rows(int a, T* p, T* m) const
    {
#pragma unroll
        for (int n = 0; n < H; ++n) {
            p[n] = k->P[a * H + n];
            m[n] = k->M[a * H + n];
        }
    }
    __device__ __forceinline__ T P(int q) const { return k->P[q]; }
    __device__ __forceinline__ T M(int q) const { return k->M[q]; }
    __device__ __forceinline__ T Cm(int q) const { return k->Cm[q]; }
    __device__ __forceinline__ T Rm(int q) const { return k->Rm[q]; }
};

// ---- FP64 contractions with row-broadcast coefficients ----
//
// The even-odd blocks of an order do not fit the scalar register file from N1 = 10 on (2 H^2
// doubles against about 50), so scalar sources reload them row by row: scalar loads in every
// contraction whose waits also drain the LDS counter, and lane spills of what stays resident.
// A vector register instead holds 16 coefficients, one per lane of each 16-lane row, and
// v_fmac_f64 takes one of them for the whole row as a row_newbcast operand: the tables of N1 = 16
// are 8 such registers, no scalar load is left in the loop, and the multiply-add issues at the
// full FP64 rate (measured over 8 independent chains: 72.4 TF/s with a row-broadcast operand,
// 73.3 with a scalar one; FP32 halves its rate with one, so FP32 keeps the scalar sources).
// Every lane of the wave must be active: a broadcast reads the lanes of its own row.
//
// Coefficient q of an order: P[a][n] at a H + n, M[a][n] at H^2 + a H + n, then Cm[a], Rm[n];
// register q / 16, lane q % 16.
template <int N1>
struct DppCoef {
    static constexpr int H = N1 / 2;
    static constexpr int P0 = 0, M0 = H * H, C0 = 2 * H * H, R0 = C0 + H;
    static constexpr int COUNT = 2 * H * H + (N1 % 2 ? 2 * H : 0);
    static constexpr int REGS = (COUNT + 15) / 16;
    double r[REGS];
};

// Loads this lane's coefficients from the tables in global or constant memory.
template <int N1, typename B>
__device__ __forceinline__ void dpp_coef_init(const B& bs, int lane, DppCoef<N1>& k)
{
    using K = DppCoef<N1>;
    const int l = lane & 15;
#pragma unroll
    for (int g = 0; g < K::REGS; ++g) {
        const int q = 16 * g + l;
        double v = 0.0;
        if (q < K::M0) v = bs.P[q];
        else if (q < K::C0) v = bs.M[q - K::M0];
        else if (q < K::COUNT) v = q < K::R0 ? bs.Cm[q - K::C0] : bs.Rm[q - K::R0];
        k.r[g] = v;
    }
}

// e += sum over T terms of coefficient EQ(i) times ue[i], o likewise: the two chains interleaved.
// The s_nop covers the two wait states a row-broadcast read needs after a vector write of its
// register (the compiler may have just copied a coefficient there).
#define AX_DPP_FMAC(acc, c, x, l) "v_fmac_f64_dpp " acc ", " c ", " x " row_newbcast:" l " row_mask:0xf bank_mask:0xf\n\t"

template <int T, int EQ0, int ES, int OQ0, int OS, typename K>
__device__ __forceinline__ void dpp_terms(const K& k, const double* ue, const double* uo, double& e, double& o)
{
    static_assert(T >= 1 && T <= 4, "terms per block");
#define AX_EC(i) "v"(k.r[(EQ0 + (i) * ES) / 16])
#define AX_OC(i) "v"(k.r[(OQ0 + (i) * OS) / 16])
#define AX_EL(i) "n"((EQ0 + (i) * ES) % 16)
#define AX_OL(i) "n"((OQ0 + (i) * OS) % 16)
    if constexpr (T == 1)
        asm("s_nop 1\n\t" AX_DPP_FMAC("%0", "%2", "%4", "%6") AX_DPP_FMAC("%1", "%3", "%5", "%7")
            : "+v"(e), "+v"(o)
            : AX_EC(0), AX_OC(0), "v"(ue[0]), "v"(uo[0]), AX_EL(0), AX_OL(0));
    else if constexpr (T == 2)
        asm("s_nop 1\n\t" AX_DPP_FMAC("%0", "%2", "%6", "%10") AX_DPP_FMAC("%1", "%3", "%7", "%11")
            AX_DPP_FMAC("%0", "%4", "%8", "%12") AX_DPP_FMAC("%1", "%5", "%9", "%13")
            : "+v"(e), "+v"(o)
            : AX_EC(0), AX_OC(0), AX_EC(1), AX_OC(1), "v"(ue[0]), "v"(uo[0]), "v"(ue[1]), "v"(uo[1]), AX_EL(0),
              AX_OL(0), AX_EL(1), AX_OL(1));
    else if constexpr (T == 3)
        asm("s_nop 1\n\t" AX_DPP_FMAC("%0", "%2", "%8", "%14") AX_DPP_FMAC("%1", "%3", "%9", "%15")
            AX_DPP_FMAC("%0", "%4", "%10", "%16") AX_DPP_FMAC("%1", "%5", "%11", "%17")
            AX_DPP_FMAC("%0", "%6", "%12", "%18") AX_DPP_FMAC("%1", "%7", "%13", "%19")
            : "+v"(e), "+v"(o)
            : AX_EC(0), AX_OC(0), AX_EC(1), AX_OC(1), AX_EC(2), AX_OC(2), "v"(ue[0]), "v"(uo[0]), "v"(ue[1]),
              "v"(uo[1]), "v"(ue[2]), "v"(uo[2]), AX_EL(0), AX_OL(0), AX_EL(1), AX_OL(1), AX_EL(2), AX_OL(2));
    else
        asm("s_nop 1\n\t" AX_DPP_FMAC("%0", "%2", "%10", "%18") AX_DPP_FMAC("%1", "%3", "%11", "%19")
            AX_DPP_FMAC("%0", "%4", "%12", "%20") AX_DPP_FMAC("%1", "%5", "%13", "%21")
            AX_DPP_FMAC("%0", "%6", "%14", "%22") AX_DPP_FMAC("%1", "%7", "%15", "%23")
            AX_DPP_FMAC("%0", "%8", "%16", "%24") AX_DPP_FMAC("%1", "%9", "%17", "%25")
            : "+v"(e), "+v"(o)
            : AX_EC(0), AX_OC(0), AX_EC(1), AX_OC(1), AX_EC(2), AX_OC(2), AX_EC(3), AX_OC(3), "v"(ue[0]), "v"(uo[0]),
              "v"(ue[1]), "v"(uo[1]), "v"(ue[2]), "v"(uo[2]), "v"(ue[3]), "v"(uo[3]), AX_EL(0), AX_OL(0), AX_EL(1),
              AX_OL(1), AX_EL(2), AX_OL(2), AX_EL(3), AX_OL(3));
#undef AX_EC
#undef AX_OC
#undef AX_EL
#undef AX_OL
}

// one chain: m += coefficient MQ times x
template <int MQ, typename K>
__device__ __forceinline__ void dpp_term(const K& k, double x, double& m)
{
    asm("s_nop 1\n\t" AX_DPP_FMAC("%0", "%1", "%2", "%3") : "+v"(m) : "v"(k.r[MQ / 16]), "v"(x), "n"(MQ % 16));
}

// terms N0..H-1 of one output row, four at a time (coefficients EQ0 + n ES and OQ0 + n OS)
template <int H, int N0, int EQ0, int ES, int OQ0, int OS, typename K>
__device__ __forceinline__ void dpp_row(const K& k, const double* ue, const double* uo, double& e, double& o)
{
    if constexpr (N0 < H) {
        constexpr int T = H - N0 >= 4 ? 4 : H - N0;
        dpp_terms<T, EQ0 + N0 * ES, ES, OQ0 + N0 * OS, OS>(k, ue + N0, uo + N0, e, o);
        dpp_row<H, N0 + T, EQ0, ES, OQ0, OS>(k, ue, uo, e, o);
    }
}

// Orders whose first coefficient of every row also fits the scalar registers (4 H doubles): the
// row's chains then start with a product instead of a cleared accumulator.
template <int N1>
constexpr bool dpp_scalar_start() { return N1 <= 9; }

template <int N1, bool TRANS, int A, typename B>
__device__ __forceinline__ void dpp_rows(const DppCoef<N1>& k, const B& bs, const double* in, const double* ue,
                                         const double* uo, double* out)
{
    using K = DppCoef<N1>;
    constexpr int H = K::H, N = N1 - 1;
    if constexpr (A < H) {
        constexpr int S = dpp_scalar_start<N1>() ? 1 : 0;
        double e = 0.0, o = 0.0;
        if constexpr (S == 1) {
            e = (TRANS ? bs.M[A] : bs.P[A * H]) * ue[0];
            o = (TRANS ? bs.P[A] : bs.M[A * H]) * uo[0];
        }
        if constexpr (TRANS)
            dpp_row<H, S, K::M0 + A, H, K::P0 + A, H>(k, ue, uo, e, o);
        else
            dpp_row<H, S, K::P0 + A * H, 1, K::M0 + A * H, 1>(k, ue, uo, e, o);
        if constexpr (N1 % 2 == 1) dpp_term<(TRANS ? K::R0 : K::C0) + A>(k, in[H], e);
        out[A] = e + o;
        out[N - A] = o - e;
        dpp_rows<N1, TRANS, A + 1>(k, bs, in, ue, uo, out);
    }
}

template <int N1, bool TRANS, int A>
__device__ __forceinline__ void dpp_middle(const DppCoef<N1>& k, const double* uo, double& m)
{
    using K = DppCoef<N1>;
    if constexpr (A < K::H) {
        dpp_term<(TRANS ? K::C0 : K::R0) + A>(k, uo[A], m);
        dpp_middle<N1, TRANS, A + 1>(k, uo, m);
    }
}

// contract_eo (below) in FP64 with row-broadcast coefficients: the same operations in the same
// order, so the same bits.
template <int N1, bool TRANS, typename B>
__device__ __forceinline__ void contract_dpp(const DppCoef<N1>& k, const B& bs, const double* in, double* out)
{
    constexpr int H = N1 / 2, N = N1 - 1;
    double ue[H], uo[H];
#pragma unroll
    for (int n = 0; n < H; ++n) {
        ue[n] = in[n] + in[N - n];
        uo[n] = in[n] - in[N - n];
    }
    double m = 0.0;
    if constexpr (N1 % 2 == 1) dpp_middle<N1, TRANS, 0>(k, uo, m);
    dpp_rows<N1, TRANS, 0>(k, bs, in, ue, uo, out);
    if constexpr (N1 % 2 == 1) out[H] = m;
}

// Basis member `bs` of the kernel's single by-value argument struct KA.
template <typename T, typename KA>
__device__ __forceinline__ CoefReload<T> karg_coefs()
{
    const KargPtr<KA> ka = (KargPtr<KA>)__builtin_amdgcn_kernarg_segment_ptr();
    return CoefReload<T>{&ka->bs};
}

// A device pointer that every lane shares (moved to scalar registers), viewed in the constant
// address space.
template <typename T>
__device__ __forceinline__ KargPtr<T> as_constant(const T* p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (KargPtr<T>)(uintptr_t)(lo | (hi << 32));
}

// out[a] = sum_n D[a][n] in[n]   (TRANS: out[a] = sum_n D[n][a] in[n])
template <int N1, bool TRANS, typename T, typename C>
__device__ __forceinline__ void contract_full(const C& src, const T* in, T* out)
{
#pragma unroll
    for (int a = 0; a < N1; ++a) {
        const C c = src.row();
        T acc = T(0);
#pragma unroll
        for (int n = 0; n < N1; ++n) acc = fma(c.D(TRANS ? n * N1 + a : a * N1 + n), in[n], acc);
        out[a] = acc;
    }
}

// The same contraction for a centro-antisymmetric D by its even-odd split (H = N1/2 squared
// blocks P and M, see Basis): with ue[n] = in[n] + in[N-n], uo[n] = in[n] - in[N-n],
//   e[a] = sum_n P[a][n] ue[n],  o[a] = sum_n M[a][n] uo[n],  out[a] = e + o,  out[N-a] = o - e.
// D^T is centro-antisymmetric too, with blocks M^T and P^T.  2 H^2 FMAs instead of N1^2, and
// half as many distinct coefficients.
template <int N1, bool TRANS, typename T, typename C>
__device__ __forceinline__ void contract_eo(const C& src, const T* in, T* out)
{
    constexpr int H = N1 / 2, N = N1 - 1;
    T ue[H], uo[H];
#pragma unroll
    for (int n = 0; n < H; ++n) {
        ue[n] = in[n] + in[N - n];
        uo[n] = in[n] - in[N - n];
    }
    if constexpr (TRANS && C::kByRow) {
        // all outputs advance by one row of the tables at a time: a row is contiguous, a column
        // takes one scalar load per coefficient.  Each sum has its terms in the order it has below.
        T e[H], o[H];
#pragma unroll
        for (int a = 0; a < H; ++a) e[a] = o[a] = T(0);
#pragma unroll
        for (int n = 0; n < H; ++n) {
            T p[H], m[H];
            src.row().template rows<H>(n, p, m);
#pragma unroll
            for (int a = 0; a < H; ++a) {
                e[a] = fma(m[a], ue[n], e[a]);
                o[a] = fma(p[a], uo[n], o[a]);
            }
        }
        const C c = src.row();
#pragma unroll
        for (int a = 0; a < H; ++a) {
            if constexpr (N1 % 2 == 1) e[a] = fma(c.Rm(a), in[H], e[a]);
            out[a] = e[a] + o[a];
            out[N - a] = o[a] - e[a];
        }
    } else {
#pragma unroll
        for (int a = 0; a < H; ++a) {
            const C c = src.row();
            T e = T(0), o = T(0), p[H], m[H];
            if constexpr (!TRANS) c.template rows<H>(a, p, m);
#pragma unroll
            for (int n = 0; n < H; ++n) {
                if constexpr (TRANS) {
                    p[n] = c.M(n * H + a);
                    m[n] = c.P(n * H + a);
                }
                e = fma(p[n], ue[n], e);
                o = fma(m[n], uo[n], o);
            }
            if constexpr (N1 % 2 == 1) e = fma(TRANS ? c.Rm(a) : c.Cm(a), in[H], e);
            out[a] = e + o;
            out[N - a] = o - e;
        }
    }
    if constexpr (N1 % 2 == 1) {
        const C c = src.row();
        T m = T(0);
#pragma unroll
        for (int n = 0; n < H; ++n) m = fma(TRANS ? c.Cm(n) : c.Rm(n), uo[n], m);
        out[H] = m;
    }
    // the products are formed here: moved under the condition of their use by the compiler they
    // would leave the loads behind, and all rows of the tables in registers
    if constexpr (C::kByRow) {
#pragma unroll
        for (int a = 0; a < N1; ++a) asm volatile("" : "+v"(out[a]));
    }
}

template <int N1, bool TRANS, bool EO, typename T, typename C>
__device__ __forceinline__ void contract(const C& src, const T* in, T* out)
{
    if constexpr (EO)
        contract_eo<N1, TRANS>(src, in, out);
    else
        contract_full<N1, TRANS>(src, in, out);
}

}  // namespace ax
