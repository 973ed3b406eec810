// Table lookup in registers: codes -> 16-bit table values, packed as matrix-core operands.
//
// A lane that keeps to ONE weight row can hold that row's whole table in eight registers, and
// v_perm_b32 looks four codes up at once: it picks four bytes out of eight by four byte selectors.
// The table is kept as two byte planes (low and high bytes of the entries); a plane of 16 entries is
// two halves of eight.  Selecting between the halves costs nothing: selectors 8 .. 15 of v_perm_b32
// yield constants or copies of a sign bit of its operands, so
//     perm(lower half, code) ^ perm(upper half, code ^ 8)
// is the wanted entry XOR a byte that depends on the code and on the OTHER half only; that byte is
// folded into the halves once per row (RowTable::load).  8 codes take 23 (4 bits: 5 to spread the
// nibbles over bytes in order, 2 for the upper half's selectors, 12 lookups, 4 to interleave the planes) vector instructions, no
// LDS traffic, no table in LDS to build and no bank conflicts.
#pragma once
#include "any4_device.h"

namespace any4 {

__device__ __forceinline__ uint32_t vperm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

template <int BITS> struct RowTable;

// 32-bit constants the decode steps use in every instruction
constexpr uint32_t kPairLo = 0x05010400u;      // bytes lo0 hi0 lo1 hi1 of two planes
constexpr uint32_t kPairHi = 0x07030602u;      // bytes lo2 hi2 lo3 hi3

// the two dwords of four 16-bit values from their byte planes
__device__ __forceinline__ void interleave(uint32_t lo, uint32_t hi, uint32_t& d0, uint32_t& d1) {
    d0 = vperm(hi, lo, kPairLo);
    d1 = vperm(hi, lo, kPairHi);
}

template <> struct RowTable<4> {
    uint32_t al[2], bl[2], ah[2], bh[2];       // low-byte plane: entries 0-7, 8-15; high-byte plane
    // the halves of a plane (each {entries 0-3, entries 4-7}) with the other half's by-products folded in:
    // as a selector, 8 + j reads for j = 0 .. 3 the sign of byte 2j + 1 of its operand pair, for j = 4 zero,
    // for j = 5 .. 7 all ones
    static __device__ __forceinline__ void fold(uint32_t (&a)[2], uint32_t (&b)[2]) {
        a[1] ^= 0xFFFFFF00u;
        b[1] ^= 0xFFFFFF00u;
        const uint32_t a1 = a[0] ^ vperm(b[1], 0u, 0x0B0A0C0Cu), b1 = b[0] ^ vperm(a[1], 0u, 0x0B0A0C0Cu);   // entries 2, 3
        const uint32_t a2 = a1 ^ vperm(0u, b1, 0x0C0C090Cu), b2 = b1 ^ vperm(0u, a1, 0x0C0C090Cu);          // entry 1
        a[0] = a2 ^ vperm(0u, b2, 0x0C0C0C08u);                                                             // entry 0
        b[0] = b2 ^ vperm(0u, a2, 0x0C0C0C08u);
    }
    // d: the row's 16 entries, two per dword
    __device__ __forceinline__ void load(const uint32_t (&d)[8]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            al[i] = vperm(d[2 * i + 1], d[2 * i], 0x06040200u);
            ah[i] = vperm(d[2 * i + 1], d[2 * i], 0x07050301u);
            bl[i] = vperm(d[2 * i + 5], d[2 * i + 4], 0x06040200u);
            bh[i] = vperm(d[2 * i + 5], d[2 * i + 4], 0x07050301u);
        }
        fold(al, bl);
        fold(ah, bh);
    }
    __device__ __forceinline__ void four(uint32_t v, uint32_t& d0, uint32_t& d1) const {
        const uint32_t u = v ^ 0x08080808u;
        interleave(vperm(al[1], al[0], v) ^ vperm(bl[1], bl[0], u), vperm(ah[1], ah[0], v) ^ vperm(bh[1], bh[0], u), d0, d1);
    }
    // codes 8 j + 4 s .. + 3 of the words w -> the four values in order
    template <int W> __device__ __forceinline__ void half(const uint32_t (&w)[W], int j, int s, uint32_t& d0, uint32_t& d1) const {
        const uint32_t e = w[j] & 0x0F0F0F0Fu, o = (w[j] >> 4) & 0x0F0F0F0Fu;     // codes 0 2 4 6 / 1 3 5 7
        four(vperm(o, e, s ? kPairHi : kPairLo), d0, d1);
    }
    // eight codes (a word) -> the eight values in order
    __device__ __forceinline__ void eight(const uint32_t (&w)[4], int j, uint32_t (&d)[4]) const {
        half(w, j, 0, d[0], d[1]);
        half(w, j, 1, d[2], d[3]);
    }
};

template <> struct RowTable<3> {
    uint32_t l[2], h[2];
    __device__ __forceinline__ void load(const uint32_t (&d)[4]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            l[i] = vperm(d[2 * i + 1], d[2 * i], 0x06040200u);
            h[i] = vperm(d[2 * i + 1], d[2 * i], 0x07050301u);
        }
    }
    // u: four codes in its low 12 bits, the bits above zero up to bit 15
    __device__ __forceinline__ void four(uint32_t u, uint32_t& d0, uint32_t& d1) const {
        const uint32_t p = (u | (u << 10)) & 0x003F003Fu;
        const uint32_t v = (p | (p << 5)) & 0x07070707u;
        interleave(vperm(l[1], l[0], v), vperm(h[1], h[0], v), d0, d1);
    }
    // (W = 2: the first 16 codes)
    template <int W> __device__ __forceinline__ void half(const uint32_t (&w)[W], int j, int s, uint32_t& d0, uint32_t& d1) const {
        const uint32_t f = j == 0 ? w[0] : j == 1 ? __builtin_amdgcn_alignbit(w[1], w[0], 24)
                         : j == 2 ? __builtin_amdgcn_alignbit(w[W - 1], w[1], 16) : w[W - 1] >> 8;
        four((s ? f >> 12 : f) & 0xFFFu, d0, d1);
    }
    __device__ __forceinline__ void eight(const uint32_t (&w)[3], int j, uint32_t (&d)[4]) const {
        half(w, j, 0, d[0], d[1]);
        half(w, j, 1, d[2], d[3]);
    }
};

template <> struct RowTable<2> {
    uint32_t t;                                // low bytes of the four entries
    uint32_t h;                                // high bytes
    __device__ __forceinline__ void load(const uint32_t (&d)[2]) {
        t = vperm(d[1], d[0], 0x06040200u);
        h = vperm(d[1], d[0], 0x07050301u);
    }
    // u: four codes in its low 8 bits, the bits above zero up to bit 19
    __device__ __forceinline__ void four(uint32_t u, uint32_t& d0, uint32_t& d1) const {
        const uint32_t p = (u | (u << 12)) & 0x000F000Fu;
        const uint32_t v = (p | (p << 6)) & 0x03030303u;
        interleave(vperm(t, t, v), vperm(h, h, v), d0, d1);
    }
    template <int W> __device__ __forceinline__ void half(const uint32_t (&w)[W], int j, int s, uint32_t& d0, uint32_t& d1) const {
        const uint32_t f = j & 1 ? w[j >> 1] >> 16 : w[j >> 1];
        four((s ? f >> 8 : f) & 0xFFu, d0, d1);
    }
    __device__ __forceinline__ void eight(const uint32_t (&w)[2], int j, uint32_t (&d)[4]) const {
        half(w, j, 0, d[0], d[1]);
        half(w, j, 1, d[2], d[3]);
    }
};

}  // namespace any4
