// Helpers of the kernels: tile order, neighbour offsets, population slots and the four
// storage formats.
#pragma once

#include <cstddef>
#include <type_traits>

#include "adjoint.hpp"
#include "lattice.hpp"
#include "params.hpp"
#include "physics.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// helpers



// 1/x: exact in FP64, the hardware reciprocal (1 ulp) in FP32
template <class C>
__device__ __forceinline__ C rcp(C x) {
    if constexpr (std::is_same<C, double>::value) return 1.0 / x;
    else return __builtin_amdgcn_rcpf(x);
}

// Work-groups are handed to the 8 XCDs of the chip round-robin by linear id.
// Remap so that XCD j owns the contiguous range of tiles [j N / 8, (j + 1) N / 8):
// tiles that share phi-halo cache lines then run on the same XCD and meet in
// its L2 instead of each fetching the lines from memory.
__device__ __forceinline__ int xcd_tile(int w, int n) {
    constexpr int kXcd = 8;
    const int base = n / kXcd, rem = n % kXcd;
    const int j = w % kXcd, local = w / kXcd;
    return j < rem ? j * (base + 1) + local : rem * (base + 1) + (j - rem) * base + local;
}

// periodic wrap / mirror ghost of a coordinate in [-1, n]
__device__ __forceinline__ int map_coord(int c, int n, int wall) {
    if (c < 0) return wall ? 0 : n - 1;
    if (c >= n) return wall ? n - 1 : 0;
    return c;
}

// index offsets of the six axis neighbours of node (x, y, z), periodic wrap folded in
struct Nbr {
    int xp, xm, yp, ym, zp, zm;
};

__device__ __forceinline__ Nbr neighbours(int x, int y, int z, const KParams& P) {
    const int nxny = P.nx * P.ny;
    Nbr n;
    n.xp = (x + 1 < P.nx) ? 1 : 1 - P.nx;
    n.xm = (x > 0) ? -1 : P.nx - 1;
    n.yp = (y + 1 < P.ny) ? P.nx : (1 - P.ny) * P.nx;
    n.ym = (y > 0) ? -P.nx : (P.ny - 1) * P.nx;
    n.zp = (z + 1 < P.nz) ? nxny : (1 - P.nz) * nxny;
    n.zm = (z > 0) ? -nxny : (P.nz - 1) * nxny;
    return n;
}

// offset of the node x - e that a population moving along e arrives from (pull)
template <int EX, int EY, int EZ>
__device__ __forceinline__ int pull_offset(const Nbr& n) {
    int d = 0;
    if constexpr (EX > 0) d += n.xm;
    if constexpr (EX < 0) d += n.xp;
    if constexpr (EY > 0) d += n.ym;
    if constexpr (EY < 0) d += n.yp;
    if constexpr (EZ > 0) d += n.zm;
    if constexpr (EZ < 0) d += n.zp;
    return d;
}

// A 32-bit byte offset the optimiser may not widen to 64 bits (an empty asm with a
// register operand, no instruction).  Base (SGPR) + this offset selects the
// `global_* voffset, saddr` form instead of a 64-bit per-lane address.
__device__ __forceinline__ unsigned voff(unsigned byte_offset) {
    asm("" : "+v"(byte_offset));
    return byte_offset;
}

// index offsets of the axis neighbours for the phi stencil: periodic wrap, or the
// node itself beyond a wall (mirror ghost of a half-way wall)
__device__ __forceinline__ Nbr stencil_neighbours(int x, int y, int z, const KParams& P) {
    const int nxny = P.nx * P.ny;
    Nbr n;
    n.xp = (x + 1 < P.nx) ? 1 : (P.wall_x ? 0 : 1 - P.nx);
    n.xm = (x > 0) ? -1 : (P.wall_x ? 0 : P.nx - 1);
    n.yp = (y + 1 < P.ny) ? P.nx : (P.wall_y ? 0 : (1 - P.ny) * P.nx);
    n.ym = (y > 0) ? -P.nx : (P.wall_y ? 0 : (P.ny - 1) * P.nx);
    n.zp = (z + 1 < P.nz) ? nxny : (P.wall_z ? 0 : (1 - P.nz) * nxny);
    n.zm = (z > 0) ? -nxny : (P.wall_z ? 0 : (P.nz - 1) * nxny);
    return n;
}

// offset of the node x + e
template <int EX, int EY, int EZ>
__device__ __forceinline__ int push_offset(const Nbr& n) {
    return pull_offset<-EX, -EY, -EZ>(n);
}

// does the pull of a population moving along z-component EZ at a node on the low
// (zlo) or high (zhi) z wall plane cross the wall?  Then it bounces back: the node's
// own population of the opposite direction (Section 4.2.4, half-way bounce-back).
template <int EZ>
__device__ __forceinline__ bool zbounce(bool zlo, bool zhi) {
    if constexpr (EZ > 0) return zlo;
    else if constexpr (EZ < 0) return zhi;
    else return false;
}

// ---------------------------------------------------------------------------
// population storage

// slot bookkeeping of one lattice family: f, g, then NC composition fields (hA, hB,
// and hC with three compositions); rest slots (k = 0) are f_0, g_0, hA_0, hB_0 (, hC_0)
template <int QF, int QS, int NC = 2>
struct Slots {
    static constexpr int G0 = QF, A0 = QF + QS, B0 = QF + 2 * QS, C0 = QF + 3 * QS, N = QF + (1 + NC) * QS;
    __host__ __device__ static constexpr bool rest(int s) {
        return (QF > 0 && s == 0) || s == G0 || s == A0 || s == B0 || (NC >= 3 && s == C0);
    }
    __host__ __device__ static constexpr int rest_before(int s) {
        return (QF > 0 && s > 0 ? 1 : 0) + (s > G0 ? 1 : 0) + (s > A0 ? 1 : 0) + (s > B0 ? 1 : 0) +
               (NC >= 3 && s > C0 ? 1 : 0);
    }
    __host__ __device__ static constexpr int field(int s) {
        return s < G0 ? 0 : (s < A0 ? 1 : (s < B0 ? 2 : (s < C0 ? 3 : 4)));
    }
};

// byte offset of slot S in a copy (moving slots take stride_m bytes, rest slots stride_r)
template <class SLOTS, int S>
__device__ __forceinline__ unsigned long long slot_offset(const KParams& P) {
    constexpr int rb = SLOTS::rest_before(S);
    return (unsigned long long)(S - rb) * P.stride_m + (unsigned long long)rb * P.stride_r;
}

// where a reader finds X_k(x) (slot S = direction k of lattice L of a field): slot S at
// the pull source x - e_k, or the node's own slot of opp(k) when that crosses a z wall
// (zbounce).  Returns the slot base in `base`'s copy and the node index in t.
template <class SLOTS, class L, int S, int K>
__device__ __forceinline__ const char* pull_src(const char* base, const KParams& P, int z, unsigned idx,
                                                const Nbr& nb, unsigned& t) {
    if (zbounce<L::ez(K)>(P.wall_z && z == 0, P.wall_z && z == P.nz - 1)) {
        t = idx;
        return base + slot_offset<SLOTS, S - K + L::opp(K)>(P);
    }
    t = unsigned(int(idx) + pull_offset<L::ex(K), L::ey(K), L::ez(K)>(nb));
    return base + slot_offset<SLOTS, S>(P);
}

// load one population at node idx and decode it to the compute type
// NT: a non-temporal load, for data no other work-group reads
template <class T, bool NT>
__device__ __forceinline__ T ld_raw(const T* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <int PREC, bool REST, bool NT = false>
__device__ __forceinline__ typename Stor<PREC>::C ld_at(const char* slot, unsigned idx, float wref,
                                                        float inv_scale) {
    if constexpr (PREC == P64) {
        return ld_raw<double, NT>(reinterpret_cast<const double*>(slot + idx * 8u));
    } else if constexpr (PREC == P32 || REST) {
        return ld_raw<float, NT>(reinterpret_cast<const float*>(slot + idx * 4u));
    } else {
        const unsigned short bits = ld_raw<unsigned short, NT>(reinterpret_cast<const unsigned short*>(slot + idx * 2u));
        if constexpr (PREC == P16) return fmaf(__half2float(__ushort_as_half(bits)), inv_scale, wref);
        else return float(__builtin_bit_cast(__bf16, bits)) + wref;  // BF16: no scale
    }
}

// decode the low / high 16 bits of a word as a moving 16-bit population (the words of
// the packed LDS ring); the same arithmetic as ld_at
template <int PREC>
__device__ __forceinline__ float dec_lo(unsigned w, float wref, float inv_scale) {
    if constexpr (PREC == P16) return fmaf(__half2float(__ushort_as_half((unsigned short)(w & 0xffffu))), inv_scale, wref);
    else return __builtin_bit_cast(float, w << 16) + wref;
}
template <int PREC>
__device__ __forceinline__ float dec_hi(unsigned w, float wref, float inv_scale) {
    if constexpr (PREC == P16) return fmaf(__half2float(__ushort_as_half((unsigned short)(w >> 16))), inv_scale, wref);
    else return __builtin_bit_cast(float, w & 0xffff0000u) + wref;
}

// 16-bit encoding of one moving population: d = (v - w_k ref) 2^s in FP16, or v - w_k ref
// in BF16 (its exponent range is FP32's, so it takes no scale), rounded to nearest even
template <int PREC>
__device__ __forceinline__ float enc_d(float v, float wref, float scale) {
    if constexpr (PREC == P16) return (v - wref) * scale;
    else return v - wref;
}

// encode and store one population (initialisation and population access: plain stores, the
// shifted rows of a pull layout start inside lines)
template <int PREC, bool REST>
__device__ __forceinline__ void st_at(char* slot, unsigned idx, float wref, float scale,
                                      typename Stor<PREC>::C v) {
    if constexpr (PREC == P64) {
        *reinterpret_cast<double*>(slot + idx * 8u) = v;
    } else if constexpr (PREC == P32 || REST) {
        *reinterpret_cast<float*>(slot + idx * 4u) = float(v);
    } else {
        const float d = enc_d<PREC>(v, wref, scale);
        unsigned short bits;
        if constexpr (PREC == P16) bits = __half_as_ushort(__float2half_rn(d));
        else bits = __builtin_bit_cast(unsigned short, __bf16(d));  // round to nearest even
        *reinterpret_cast<unsigned short*>(slot + idx * 2u) = bits;
    }
}

// store, returning the value the slot now decodes to (16-bit moving populations:
// the rounded value; otherwise v itself)
template <int PREC, bool REST>
__device__ __forceinline__ typename Stor<PREC>::C st_at_r(char* slot, unsigned idx, float wref, float scale,
                                                           float inv_scale, typename Stor<PREC>::C v) {
    if constexpr (PREC == P64 || PREC == P32 || REST) {
        st_at<PREC, REST>(slot, idx, wref, scale, v);
        return v;
    } else {
        const float d = enc_d<PREC>(v, wref, scale);
        unsigned short bits;
        float back;
        if constexpr (PREC == P16) {
            const __half hd = __float2half_rn(d);
            bits = __half_as_ushort(hd);
            back = __half2float(hd) * inv_scale;
        } else {
            const __bf16 bd = __bf16(d);  // round to nearest even
            bits = __builtin_bit_cast(unsigned short, bd);
            back = float(bd);
        }
        *reinterpret_cast<unsigned short*>(slot + idx * 2u) = bits;
        return back + wref;
    }
}

// encode a moving 16-bit population; returns its rounding residue in the encoded domain,
// d - round(d): (value - stored value) is that times 2^-s (FP16) or itself (BF16)
template <int PREC>
__device__ __forceinline__ float enc_res(float wref, float scale, float v, unsigned short& bits) {
    static_assert(PREC == P16 || PREC == PB16, "16-bit formats only");
    const float d = enc_d<PREC>(v, wref, scale);
    float back;
    if constexpr (PREC == P16) {
        const __half hd = __float2half_rn(d);
        bits = __half_as_ushort(hd);
        back = __half2float(hd);
    } else {
        const __bf16 bd = __bf16(d);  // round to nearest even
        bits = __builtin_bit_cast(unsigned short, bd);
        back = float(bd);
    }
    return d - back;
}

// encode two moving 16-bit populations of one field (the same reference w_k ref) with one
// packed conversion (round to nearest even): the bits of va in the low half; dev receives
// the sum of their stored deviations in the encoded domain
template <int PREC>
__device__ __forceinline__ unsigned enc2_dev(float wref, float scale, float va, float vb, float& dev) {
    static_assert(PREC == P16 || PREC == PB16, "16-bit formats only");
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 d = {enc_d<PREC>(va, wref, scale), enc_d<PREC>(vb, wref, scale)};
    unsigned bits;
    if constexpr (PREC == P16) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        const h2 r = __builtin_convertvector(d, h2);
        bits = __builtin_bit_cast(unsigned, r);
        dev = float(r.x) + float(r.y);
    } else {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        bits = __builtin_bit_cast(unsigned, __builtin_convertvector(d, b2));
        dev = __builtin_bit_cast(float, bits << 16) + __builtin_bit_cast(float, bits & 0xffff0000u);
    }
    return bits;
}

// store the stored form of one population: the 16 bits of a moving population, or the
// value itself (FP32 / FP64 storage, rest populations), as a step writes it.  STREAM: a non-temporal store, for
// whole 128-byte lines that nobody reads before the next step (256^3 FP32 1114 us a step
// against 1200 with plain stores, 512^3 BF16 5660 against 6200).  Rows that start inside a
// line take plain stores: L2 joins the parts of a line that neighbouring waves and rows
// write, a non-temporal store sends each part to memory by itself (297 x 182 x 133 BF16
// 472 us against 663, FP32 722 against 863)
template <bool STREAM, class V>
__device__ __forceinline__ void st_raw(char* slot, unsigned idx, V v) {
    V* p = reinterpret_cast<V*>(slot + idx * unsigned(sizeof(V)));
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

}  // namespace lbm
