// Device-side bit transpose of one "unit" (Bitshuffle, Section 4.2 of
// Masui et al.).  A block of n_B elements is the (n_B x 8E) bit matrix of
// its elements; bit b of element i (b = 8 * byte + bit, LSB first) goes to
// plane b, byte i / 8, bit i % 8.
//
// A lane transposes one unit in registers:
//   E = 1  : 128 elements, output 16 bytes of each of the 8 planes
//   E = 2  : 64 elements,  output 8 bytes of each of the 16 planes
//   E = 4c : 32 elements,  per 4-byte column one 32x32 transpose, output 4
//            bytes of each of the 8E planes
// Plane bytes of unit u sit at plane * (n_B / 8) + u * (G / 8), so the
// block's units must tile it exactly (n_B a multiple of G).
#pragma once

#include "bsg_internal.hpp"

namespace bsg {

template <int E> struct Unit {
    static constexpr int G = E == 1 ? 128 : (E == 2 ? 64 : 32); // elements
    static constexpr int IN_WORDS = G * E / 4;                  // input dwords
    static constexpr int PB = G / 8;                            // plane bytes per unit
    static constexpr int NC = E >= 4 ? E / 4 : 1;               // 32x32 transposes
};

// In-register forward transform.  in: the unit's raw element dwords
// (IN_WORDS).  out (same array): plane words; plane pl of the unit is
//   E = 1 : out[pl], out[pl+8], out[pl+16], out[pl+24]   (16 bytes)
//   E = 2 : out[pl], out[pl+16]                           (8 bytes)
//   E = 4c: out[32 * (pl / 32) + pl % 32]                 (4 bytes)
template <int E>
__device__ __forceinline__ void unit_forward(uint32_t (&w)[Unit<E>::IN_WORDS])
{
    if constexpr (E == 1) {
        uint32_t d[32];
        pack_e1(w, d);
        transpose32(d);
#pragma unroll
        for (int k = 0; k < 32; ++k) w[k] = d[k];
    } else if constexpr (E == 2) {
        uint32_t d[32];
        pack_e2(w, d);
        transpose32(d);
#pragma unroll
        for (int k = 0; k < 32; ++k) w[k] = d[k];
    } else {
        constexpr int NC = Unit<E>::NC;
        uint32_t o[Unit<E>::IN_WORDS];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint32_t a[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) a[i] = w[i * NC + c];
            transpose32(a);
#pragma unroll
            for (int b = 0; b < 32; ++b) o[32 * c + b] = a[b];
        }
#pragma unroll
        for (int k = 0; k < Unit<E>::IN_WORDS; ++k) w[k] = o[k];
    }
}

// Exact inverse of unit_forward (plane words in the layout above -> raw
// element dwords).
template <int E>
__device__ __forceinline__ void unit_inverse(uint32_t (&w)[Unit<E>::IN_WORDS])
{
    if constexpr (E == 1) {
        uint32_t d[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) d[k] = w[k];
        transpose32(d);
        unpack_e1(d, w);
    } else if constexpr (E == 2) {
        uint32_t d[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) d[k] = w[k];
        transpose32(d);
        unpack_e2(d, w);
    } else {
        constexpr int NC = Unit<E>::NC;
        uint32_t o[Unit<E>::IN_WORDS];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint32_t a[32];
#pragma unroll
            for (int b = 0; b < 32; ++b) a[b] = w[32 * c + b];
            transpose32(a);
#pragma unroll
            for (int i = 0; i < 32; ++i) o[i * NC + c] = a[i];
        }
#pragma unroll
        for (int k = 0; k < Unit<E>::IN_WORDS; ++k) w[k] = o[k];
    }
}

// Index of plane pl's first word within the unit's plane-word array, and
// the number of words per plane.
template <int E> struct PlaneWords {
    static constexpr int PER = Unit<E>::PB / 4; // 4, 2 or 1 words
    static constexpr int NPL = 8 * E;
    __device__ static constexpr int word(int pl, int q)
    {
        return E == 1 ? pl + 8 * q : (E == 2 ? pl + 16 * q : pl);
    }
};

// Load/store the unit's raw elements (16-byte aligned, IN_WORDS dwords).
template <int E>
__device__ __forceinline__ void load_unit(const uint8_t *p, uint32_t (&w)[Unit<E>::IN_WORDS])
{
    const uint4 *q = reinterpret_cast<const uint4 *>(p);
#pragma unroll
    for (int k = 0; k < Unit<E>::IN_WORDS / 4; ++k) {
        const uint4 v = q[k];
        w[4 * k] = v.x;
        w[4 * k + 1] = v.y;
        w[4 * k + 2] = v.z;
        w[4 * k + 3] = v.w;
    }
}
template <int E>
__device__ __forceinline__ void store_unit(uint8_t *p, const uint32_t (&w)[Unit<E>::IN_WORDS])
{
    uint4 *q = reinterpret_cast<uint4 *>(p);
#pragma unroll
    for (int k = 0; k < Unit<E>::IN_WORDS / 4; ++k)
        q[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
}

// Store / load the unit's plane bytes into a block laid out as planes of
// plane_bytes each (global or LDS; aligned to the plane chunk size).
template <int E>
__device__ __forceinline__ void store_planes(uint8_t *blk, int64_t plane_bytes, int64_t u,
                                             const uint32_t (&w)[Unit<E>::IN_WORDS])
{
    using PW = PlaneWords<E>;
#pragma unroll
    for (int pl = 0; pl < PW::NPL; ++pl) {
        uint8_t *dst = blk + pl * plane_bytes + u * Unit<E>::PB;
        if constexpr (PW::PER == 4)
            *reinterpret_cast<uint4 *>(dst) =
                make_uint4(w[PW::word(pl, 0)], w[PW::word(pl, 1)], w[PW::word(pl, 2)],
                           w[PW::word(pl, 3)]);
        else if constexpr (PW::PER == 2)
            *reinterpret_cast<uint2 *>(dst) = make_uint2(w[PW::word(pl, 0)], w[PW::word(pl, 1)]);
        else
            *reinterpret_cast<uint32_t *>(dst) = w[PW::word(pl, 0)];
    }
}
template <int E>
__device__ __forceinline__ void load_planes(const uint8_t *blk, int64_t plane_bytes, int64_t u,
                                            uint32_t (&w)[Unit<E>::IN_WORDS])
{
    using PW = PlaneWords<E>;
#pragma unroll
    for (int pl = 0; pl < PW::NPL; ++pl) {
        const uint8_t *src = blk + pl * plane_bytes + u * Unit<E>::PB;
        if constexpr (PW::PER == 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(src);
            w[PW::word(pl, 0)] = v.x;
            w[PW::word(pl, 1)] = v.y;
            w[PW::word(pl, 2)] = v.z;
            w[PW::word(pl, 3)] = v.w;
        } else if constexpr (PW::PER == 2) {
            const uint2 v = *reinterpret_cast<const uint2 *>(src);
            w[PW::word(pl, 0)] = v.x;
            w[PW::word(pl, 1)] = v.y;
        } else {
            w[PW::word(pl, 0)] = *reinterpret_cast<const uint32_t *>(src);
        }
    }
}

// 8 x 8 bit transpose: bit j of byte i of (lo, hi) goes to bit i of byte j.
__device__ __forceinline__ void transpose8(uint32_t &lo, uint32_t &hi)
{
    uint32_t t = (lo ^ (lo >> 7)) & 0x00AA00AAu;
    lo ^= t ^ (t << 7);
    t = (hi ^ (hi >> 7)) & 0x00AA00AAu;
    hi ^= t ^ (t << 7);
    t = (lo ^ (lo >> 14)) & 0x0000CCCCu;
    lo ^= t ^ (t << 14);
    t = (hi ^ (hi >> 14)) & 0x0000CCCCu;
    hi ^= t ^ (t << 14);
    t = (lo ^ (hi << 4)) & 0xF0F0F0F0u;
    lo ^= t;
    hi ^= t >> 4;
}

// Generic transpose of one block by a whole wavefront, any E, any n_B
// (multiple of 8) and any alignment: a lane takes byte k of 8 consecutive
// elements, whose 8 x 8 bits are byte g of the planes 8 k .. 8 k + 7 (several
// k at once where a block has fewer than 64 such groups).  A ballot per bit
// of every 64 elements took 48 us for 4 Mi 3-byte elements, this takes 11.
// ROWS: the bytes k a wavefront's lanes take at once, for elements of 16 bytes
// and more: its 8 x 8 lanes then read whole pieces of 64 neighbouring elements
// one after the other instead of the block's length once for every k.  (0: as
// many as the block leaves lanes for.)
template <int ROWS = 0>
__device__ __forceinline__ void block_forward_bits(const uint8_t *in, uint8_t *out, int64_t elems,
                                                   int64_t E)
{
    const int lane = threadIdx.x & 63;
    const int64_t pb = elems / 8;
    const auto byte_group = [&](int64_t k, int64_t g) {
        uint32_t b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = in[(8 * g + i) * E + k];
        uint32_t lo = b[0] | b[1] << 8 | b[2] << 16 | b[3] << 24;
        uint32_t hi = b[4] | b[5] << 8 | b[6] << 16 | b[7] << 24;
        transpose8(lo, hi);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            out[(8 * k + j) * pb + g] = (uint8_t)((j < 4 ? lo : hi) >> (8 * (j & 3)));
    };
    if constexpr (ROWS > 0) {
        constexpr int COLS = 64 / ROWS;
        for (int64_t g = lane % COLS; g < pb; g += COLS)
#pragma unroll 2
            for (int64_t k = lane / COLS; k < E; k += ROWS) byte_group(k, g);
    } else {
        const int rows = pb < 64 ? 64 / (int)pb : 1;
        const int k0 = rows > 1 ? lane / (int)pb : 0, g0 = lane - k0 * (int)pb;
        if (k0 >= rows) return;
        for (int64_t k = k0; k < E; k += rows) {
#pragma unroll 2
            for (int64_t g = g0; g < pb; g += 64) byte_group(k, g);
        }
    }
}

// A block whose elements are no whole number of units goes by groups of 8
// elements and, for E >= 4, columns of 4 of their bytes: byte g of 8 planes is
// the 8 x 8 bit matrix of one byte of the group's elements.  The elements (from
// a 16-byte aligned block) are moved as whole dwords, the plane bytes one by one.
template <int E> constexpr int group_columns() { return E >= 4 ? E / 4 : 1; }

// Column c of group g: the dwords of its elements (2 for E = 1, 4 for E = 2,
// else one of each of the 8 elements).
template <int E> constexpr int group_words() { return E == 1 ? 2 : E == 2 ? 4 : 8; }

template <int E, typename Int>
__device__ __forceinline__ void group_load(const uint8_t *__restrict__ in, Int g, int c,
                                           uint32_t (&w)[group_words<E>()])
{
    if constexpr (E == 1) {
        const uint2 v = reinterpret_cast<const uint2 *>(in)[g];
        w[0] = v.x;
        w[1] = v.y;
    } else if constexpr (E == 2 || E == 4) {
#pragma unroll
        for (int i = 0; i < E / 2; ++i) {
            const uint4 v = reinterpret_cast<const uint4 *>(in)[(E / 2) * g + i];
            w[4 * i] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    } else {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(in) + 8 * g * (E / 4) + c;
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = p[i * (E / 4)];
    }
}

// Those dwords to byte g of the column's planes.
template <int E, typename Int>
__device__ __forceinline__ void group_forward(const uint32_t (&w)[group_words<E>()], Int pb, Int g,
                                              int c, uint8_t *planes)
{
    constexpr int KB = E < 4 ? E : 4;
    uint32_t lo[KB], hi[KB];
    if constexpr (E == 1) {
        lo[0] = w[0];
        hi[0] = w[1];
    } else if constexpr (E == 2) {
        lo[0] = perm(w[1], w[0], 0x06040200u);
        lo[1] = perm(w[1], w[0], 0x07050301u);
        hi[0] = perm(w[3], w[2], 0x06040200u);
        hi[1] = perm(w[3], w[2], 0x07050301u);
    } else {
        byte_transpose4(w[0], w[1], w[2], w[3], lo[0], lo[1], lo[2], lo[3]);
        byte_transpose4(w[4], w[5], w[6], w[7], hi[0], hi[1], hi[2], hi[3]);
    }
    uint8_t *p = planes + 8 * KB * c * pb + g;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        transpose8(lo[k], hi[k]);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            p[(8 * k + j) * pb] = (uint8_t)((j < 4 ? lo[k] : hi[k]) >> (8 * (j & 3)));
    }
}

// And back, from the planes to the elements.  (Stored byte by byte the
// wavefront's stores fell 8 E bytes apart: 42 MB of 8-byte elements in blocks
// of 1008 took 200 us to decompress, this 44, a lane per element 78.)
template <int E, typename Int>
__device__ __forceinline__ void group_inverse(const uint8_t *planes, Int pb, Int g, int c,
                                              uint8_t *__restrict__ out)
{
    constexpr int KB = E < 4 ? E : 4;
    const uint8_t *p = planes + 8 * KB * c * pb + g;
    uint32_t lo[KB], hi[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        uint32_t b[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = p[(8 * k + j) * pb];
        lo[k] = b[0] | b[1] << 8 | b[2] << 16 | b[3] << 24;
        hi[k] = b[4] | b[5] << 8 | b[6] << 16 | b[7] << 24;
        transpose8(lo[k], hi[k]);
    }
    if constexpr (E == 1) {
        reinterpret_cast<uint2 *>(out)[g] = make_uint2(lo[0], hi[0]);
    } else if constexpr (E == 2) {
        reinterpret_cast<uint4 *>(out)[g] =
            make_uint4(perm(lo[1], lo[0], 0x05010400u), perm(lo[1], lo[0], 0x07030602u),
                       perm(hi[1], hi[0], 0x05010400u), perm(hi[1], hi[0], 0x07030602u));
    } else {
        uint32_t e[8];
        byte_transpose4(lo[0], lo[1], lo[2], lo[3], e[0], e[1], e[2], e[3]);
        byte_transpose4(hi[0], hi[1], hi[2], hi[3], e[4], e[5], e[6], e[7]);
        if constexpr (E == 4) {
            uint4 *o = reinterpret_cast<uint4 *>(out) + 2 * g;
            o[0] = make_uint4(e[0], e[1], e[2], e[3]);
            o[1] = make_uint4(e[4], e[5], e[6], e[7]);
        } else {
            uint32_t *o = reinterpret_cast<uint32_t *>(out) + 8 * g * (E / 4) + c;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i * (E / 4)] = e[i];
        }
    }
}

// The generic inverse: a lane per element,
// so that a wavefront's byte stores fall into neighbouring lines (with 8
// elements per lane 2 Mi 6-byte elements took 47 us instead of 37, and their
// decompression 53 instead of 30).
__device__ __forceinline__ void block_inverse_elements(const uint8_t *in, uint8_t *out,
                                                       int64_t elems, int64_t E)
{
    const int lane = threadIdx.x & 63;
    const int64_t pb = elems / 8;
    for (int64_t i = lane; i < elems; i += 64) {
        for (int64_t byte = 0; byte < E; ++byte) {
            uint32_t v = 0;
            for (int bit = 0; bit < 8; ++bit)
                v |= ((uint32_t)(in[(8 * byte + bit) * pb + i / 8] >> (i % 8)) & 1u) << bit;
            out[i * E + byte] = (uint8_t)v;
        }
    }
}

} // namespace bsg
