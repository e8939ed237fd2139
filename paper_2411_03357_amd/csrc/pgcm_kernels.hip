// HIP kernels for batched AES-GCM on gfx950 (MI355X).
//
// What is computed is the AES-GCM transform the paper's transport applies to every transfer
// (paper sections 2.2 and 4.1), i.e. FIPS-197 AES-256 in the GCM mode of NIST SP 800-38D with a
// 96-bit IV; the other two key lengths and other IV lengths are served by the same kernels
// (round count as a template parameter).  How:
//   * AES rounds read four 1 KiB round tables, each replicated 32 times in LDS so that lane l
//     always reads bank l % 32: table lookups never collide, whatever the data.  AddRoundKey is
//     folded into forming the next round's lookup addresses (one SDWA XOR per state byte).
//   * GHASH multiplies by fixed powers of H with 4-bit tables (Shoup).  The row power H^64 sits in
//     LDS and its thirty-two lookups are spread over the AES rounds; as an alternative, in the unit
//     kernel, the same multiplication runs on the matrix cores, as a product with a 128 x 128
//     matrix over GF(2) (GhashRowMatrix).  Sums over the 64 lanes are formed bit by bit from powers
//     of H themselves (GfWords).
//   * A wavefront walks rows of 64 blocks of one chunk, one block per lane, 16-byte coalesced loads
//     and stores, ciphertext hashed from registers.
// Which rows, and how their sums become tags, differs:
//   * burst_kernel: up to sixty-four rows a compute unit, in one launch: a call is as long as its chain of
//     dependent steps.
//   * swap_kernel: more than that, in one launch, in units of one size, where they are filled well enough
//     (eight rows or sixteen, some 26 to 32 MiB) or spans are not to be had.
//   * span_kernel: everything else, of one key or of several, in one launch: every wavefront of the
//     chip an equal share of all rows.
//   * small_kernel: many chunks of one row each, a wavefront per chunk.
//   * bulk_kernel, then fold kernels and final_kernel: chunks cut into units of one size, which the
//     wavefronts take in turn, each leaving 64 per-lane sums.  For what the others do not take: the
//     entry point with fixed buffers, chunks of more than 1 GiB, forced unit sizes, the matrix cores.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "pgcm_arrive.h"
#include "pgcm_kernels.h"

namespace pgcm {

// ------------------------------------------------------------------------------------------
// S-box, generated at compile time from its definition (FIPS-197 5.1.1): inverse in
// GF(2^8) mod x^8+x^4+x^3+x+1, then the affine map.
namespace {

constexpr uint8_t xtime(uint8_t a) { return (uint8_t)((a << 1) ^ ((a & 0x80) ? 0x1B : 0)); }

constexpr uint8_t mul8(uint8_t a, uint8_t b) {
    uint8_t p = 0;
    for (int i = 0; i < 8; ++i) {
        if (b & (1 << i)) p ^= a;
        a = xtime(a);
    }
    return p;
}

constexpr uint8_t inv8(uint8_t a) {
    // a^254: the inverse of every non-zero element, and 0 for 0
    uint8_t r = 1, s = a;
    for (int bit = 1; bit < 8; ++bit) {
        s = mul8(s, s);    // a^(2^bit)
        r = mul8(r, s);
    }
    return r;              // a^(2+4+...+128) = a^254
}

constexpr uint8_t rotl8(uint8_t v, int k) { return (uint8_t)((v << k) | (v >> (8 - k))); }

struct SboxTable {
    uint8_t v[256];
};

constexpr SboxTable make_sbox() {
    SboxTable t{};
    for (int x = 0; x < 256; ++x) {
        uint8_t b = inv8((uint8_t)x);
        t.v[x] = (uint8_t)(b ^ rotl8(b, 1) ^ rotl8(b, 2) ^ rotl8(b, 3) ^ rotl8(b, 4) ^ 0x63);
    }
    return t;
}

__device__ const SboxTable kSbox = make_sbox();
static_assert(make_sbox().v[0x00] == 0x63 && make_sbox().v[0x53] == 0xED, "S-box");

// ------------------------------------------------------------------------------------------
// GF(2^128) in GCM's bit order (SP 800-38D 6.3): bit 0 of a block is the top bit of byte 0.
__device__ __forceinline__ uint32_t bswap32(uint32_t v) { return __builtin_bswap32(v); }

// a ^ b ^ c in one instruction (gfx950's three-input bitwise op, truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
// a ^ (b & c) in one instruction, which the compiler makes of that expression only at the start of a chain:
// what sums over lanes bit by bit takes 95 instructions a bit instead of 153 (300 adapters both ways 168.5 ->
// 163.1 us, 2 MiB decrypted 9.04 -> 8.76, 64 chunks of 4 KiB both ways 13.3 -> 12.9)
__device__ __forceinline__ uint32_t xor_and(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x78);
}

__device__ __forceinline__ void block_xor(Block& a, const Block& b) {
    a.w[0] ^= b.w[0];
    a.w[1] ^= b.w[1];
    a.w[2] ^= b.w[2];
    a.w[3] ^= b.w[3];
}

// X * C from C's nibble table in global memory: 32 lookups of 16 bytes
__device__ Block gf_mul_table(const Block* __restrict__ tbl, const Block& x) {
    Block z{{0, 0, 0, 0}};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t byte = (x.w[i] >> (8 * k)) & 0xFF;
            uint32_t pos = 2 * (4 * i + k);
            block_xor(z, tbl[pos * 16 + (byte >> 4)]);
            block_xor(z, tbl[(pos + 1) * 16 + (byte & 15)]);
        }
    }
    return z;
}

// ------------------------------------------------------------------------------------------
// AES block encryption from tables in global memory (set-up, J0, not the bulk path)
__device__ __forceinline__ uint32_t byte_of(uint32_t w, int k) { return (w >> (8 * k)) & 0xFF; }

__device__ void aes_block_global(const KeyTables* __restrict__ kt, uint32_t s[4]) {
    const uint32_t* rk = kt->rk;
    const int nr = (int)kt->rounds;
    uint32_t a0 = s[0] ^ rk[0], a1 = s[1] ^ rk[1], a2 = s[2] ^ rk[2], a3 = s[3] ^ rk[3];
    for (int r = 1; r < nr; ++r) {
        uint32_t t0 = kt->te[0][byte_of(a0, 0)] ^ kt->te[1][byte_of(a1, 1)] ^
                      kt->te[2][byte_of(a2, 2)] ^ kt->te[3][byte_of(a3, 3)] ^ rk[4 * r + 0];
        uint32_t t1 = kt->te[0][byte_of(a1, 0)] ^ kt->te[1][byte_of(a2, 1)] ^
                      kt->te[2][byte_of(a3, 2)] ^ kt->te[3][byte_of(a0, 3)] ^ rk[4 * r + 1];
        uint32_t t2 = kt->te[0][byte_of(a2, 0)] ^ kt->te[1][byte_of(a3, 1)] ^
                      kt->te[2][byte_of(a0, 2)] ^ kt->te[3][byte_of(a1, 3)] ^ rk[4 * r + 2];
        uint32_t t3 = kt->te[0][byte_of(a3, 0)] ^ kt->te[1][byte_of(a0, 1)] ^
                      kt->te[2][byte_of(a1, 2)] ^ kt->te[3][byte_of(a2, 3)] ^ rk[4 * r + 3];
        a0 = t0, a1 = t1, a2 = t2, a3 = t3;
    }
    const uint8_t* S = kSbox.v;
    auto last = [&](uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
        return (uint32_t)S[byte_of(c0, 0)] | ((uint32_t)S[byte_of(c1, 1)] << 8) |
               ((uint32_t)S[byte_of(c2, 2)] << 16) | ((uint32_t)S[byte_of(c3, 3)] << 24);
    };
    s[0] = last(a0, a1, a2, a3) ^ rk[4 * nr + 0];
    s[1] = last(a1, a2, a3, a0) ^ rk[4 * nr + 1];
    s[2] = last(a2, a3, a0, a1) ^ rk[4 * nr + 2];
    s[3] = last(a3, a0, a1, a2) ^ rk[4 * nr + 3];
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Arithmetic on field elements held as words of coefficients (GfWords): x^0 is the top bit of the
// first word, so multiplying by x is a shift to the right.
namespace {

// x^128 = 1 + x + x^2 + x^7: folds `over`, coefficients x^128 .. x^159, back in; at most the first
// 25 of them may be set
__device__ __forceinline__ void gfw_fold_word(GfWords& v, uint32_t over) {
    v.a[0] ^= over ^ (over >> 1) ^ (over >> 2) ^ (over >> 7);
}

__device__ __forceinline__ void gfw_mul_x(GfWords& v) {
    const uint32_t over = 0u - (v.a[3] & 1u);
    v.a[3] = (v.a[3] >> 1) | (v.a[2] << 31);
    v.a[2] = (v.a[2] >> 1) | (v.a[1] << 31);
    v.a[1] = (v.a[1] >> 1) | (v.a[0] << 31);
    v.a[0] = (v.a[0] >> 1) ^ (over & 0xE1000000u);
}

// times x^8
__device__ __forceinline__ void gfw_mul_x8(GfWords& v) {
    const uint32_t over = v.a[3] << 24;
    v.a[3] = (v.a[3] >> 8) | (v.a[2] << 24);
    v.a[2] = (v.a[2] >> 8) | (v.a[1] << 24);
    v.a[1] = (v.a[1] >> 8) | (v.a[0] << 24);
    v.a[0] >>= 8;
    gfw_fold_word(v, over);
}

__device__ __forceinline__ Block gfw_to_block(const GfWords& v) {
    return Block{{bswap32(v.a[0]), bswap32(v.a[1]), bswap32(v.a[2]), bswap32(v.a[3])}};
}
__device__ __forceinline__ GfWords gfw_from_block(const Block& b) {
    return GfWords{{bswap32(b.w[0]), bswap32(b.w[1]), bswap32(b.w[2]), bswap32(b.w[3])}};
}

// bit by bit (SP 800-38D algorithm 1); used for set-up only
__device__ GfWords gfw_mul(const GfWords& x, GfWords y) {
    GfWords z{{0, 0, 0, 0}};
    for (int i = 0; i < 4; ++i) {
        for (int j = 31; j >= 0; --j) {
            const uint32_t m = 0u - ((x.a[i] >> j) & 1u);
            for (int k = 0; k < 4; ++k) z.a[k] ^= y.a[k] & m;
            gfw_mul_x(y);
        }
    }
    return z;
}

// coefficient x^i to x^(2 i), then reduced
__device__ GfWords gfw_square(const GfWords& x) {
    auto spread = [](uint32_t v) {  // sixteen coefficients to every other place of a word
        v &= 0xFFFFu;
        v = (v | (v << 8)) & 0x00FF00FFu;
        v = (v | (v << 4)) & 0x0F0F0F0Fu;
        v = (v | (v << 2)) & 0x33333333u;
        v = (v | (v << 1)) & 0x55555555u;
        return v << 1;
    };
    uint32_t r[8];
    for (int i = 0; i < 4; ++i) {
        r[2 * i] = spread(x.a[i] >> 16);
        r[2 * i + 1] = spread(x.a[i]);
    }
    const uint32_t* u = r + 4;  // coefficients from x^128 on, times 1 + x + x^2 + x^7
    GfWords z;
    for (int i = 0; i < 4; ++i) {
        const uint32_t before = i == 0 ? 0u : u[i - 1];
        z.a[i] = r[i] ^ u[i] ^ ((u[i] >> 1) | (before << 31)) ^ ((u[i] >> 2) | (before << 30)) ^
                 ((u[i] >> 7) | (before << 25));
    }
    gfw_fold_word(z, (u[3] << 31) ^ (u[3] << 30) ^ (u[3] << 25));
    return z;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Key set-up: key schedule (FIPS-197 5.2), round tables, H and everything made of its powers.
// One workgroup; `key_words` are the key bytes as nk = 4, 6 or 8 little-endian words.
// The serial part is one thread's (key schedule, E_K(0), thirty squarings) and runs from LDS; a
// nibble table is linear in the nibble, so only its 128 products with single coefficients are
// made, by shifting, and its 512 entries are sums of up to four of them.
__global__ __launch_bounds__(1024) void expand_key_kernel(KeyTables* __restrict__ kt,
                                                          const uint32_t* __restrict__ key_words,
                                                          uint32_t nk, uint4* __restrict__ clear,
                                                          uint32_t n_clear) {
    // H^(2^k), then H^3, H^12, H^48, H^96 and H^192; all but H^96 get a nibble table
    constexpr uint32_t kConstants = kNumPowers + kNumLanePowers + 2, kAt96 = kConstants - 2,
                       kAt192 = kConstants - 1;
    constexpr uint32_t kLevels = 8;  // nibble tables of H^1 .. H^128 kept in LDS as well
    __shared__ GfWords constants[kConstants];
    __shared__ Block basis[kConstants][128];  // x^b * constant, b = bit b % 32 of word b / 32
    __shared__ Block nibbles[kLevels][kNibbleTableEntries];
    __shared__ GfWords h_power[kDotBlocks + 2];
    __shared__ uint32_t te[4][256], rk[60];
    __shared__ uint8_t sbox[256];
    const uint32_t tid = threadIdx.x;

    for (uint32_t i = tid; i < n_clear; i += blockDim.x) clear[i] = make_uint4(0, 0, 0, 0);
    // round tables: te[0][x] = (2s, s, s, 3s) in bytes 0..3, te[r] = te[0] rotated left by 8r bits
    for (uint32_t x = tid; x < 256; x += blockDim.x) {
        uint32_t s = kSbox.v[x];
        uint32_t s2 = xtime((uint8_t)s), s3 = s2 ^ s;
        uint32_t t0 = s2 | (s << 8) | (s << 16) | (s3 << 24);
        sbox[x] = (uint8_t)s;
        te[0][x] = t0;
        te[1][x] = (t0 << 8) | (t0 >> 24);
        te[2][x] = (t0 << 16) | (t0 >> 16);
        te[3][x] = (t0 << 24) | (t0 >> 8);
        for (int r = 0; r < 4; ++r) kt->te[r][x] = te[r][x];
    }
    if (tid < 60) rk[tid] = tid < nk ? key_words[tid] : 0;
    __syncthreads();
    const uint32_t nr = nk + 6;
    if (tid == 0) {
        auto sub_word = [&](uint32_t w) {
            return (uint32_t)sbox[w & 0xFF] | ((uint32_t)sbox[(w >> 8) & 0xFF] << 8) |
                   ((uint32_t)sbox[(w >> 16) & 0xFF] << 16) | ((uint32_t)sbox[w >> 24] << 24);
        };
        uint32_t rcon = 1, t = rk[nk - 1];
        for (uint32_t i = nk; i < 4 * (nr + 1); ++i) {
            if (i % nk == 0) {
                t = sub_word((t >> 8) | (t << 24)) ^ rcon;  // RotWord on little-endian bytes
                rcon = xtime((uint8_t)rcon);
            } else if (nk > 6 && i % nk == 4) {
                t = sub_word(t);
            }
            t ^= rk[i - nk];
            rk[i] = t;
        }
        // H = E_K(0)
        uint32_t a[4] = {rk[0], rk[1], rk[2], rk[3]};
        for (uint32_t r = 1; r <= nr; ++r) {
            uint32_t n[4];
            for (int c = 0; c < 4; ++c) {
                const uint32_t x0 = byte_of(a[c], 0), x1 = byte_of(a[(c + 1) & 3], 1),
                               x2 = byte_of(a[(c + 2) & 3], 2), x3 = byte_of(a[(c + 3) & 3], 3);
                n[c] = r < nr ? te[0][x0] ^ te[1][x1] ^ te[2][x2] ^ te[3][x3]
                              : (uint32_t)sbox[x0] | ((uint32_t)sbox[x1] << 8) |
                                    ((uint32_t)sbox[x2] << 16) | ((uint32_t)sbox[x3] << 24);
                n[c] ^= rk[4 * r + c];
            }
            for (int c = 0; c < 4; ++c) a[c] = n[c];
        }
        const Block h{{a[0], a[1], a[2], a[3]}};
        kt->h = h;
        GfWords p = gfw_from_block(h);
        constants[0] = p;
        for (uint32_t k = 1; k < kNumPowers; ++k) {
            p = gfw_square(p);
            constants[k] = p;
        }
        kt->rounds = nr;
        for (int i = 0; i < 3; ++i) kt->pad_[i] = 0;
    }
    __syncthreads();
    if (tid < 60) kt->rk[tid] = rk[tid];
    if (tid < 64) {
        const uint32_t c = tid / 16, r = tid % 16;
        kt->column_keys[c][r] = r < 14 ? rk[4 * r + c] : r == 15 ? rk[4 * nr + c] : 0;
    }
    // H^3, H^12, H^48, H^96, H^192 = products of two neighbouring squares
    if (tid <= kNumLanePowers + 1) {
        const uint32_t first = tid < 3 ? 2 * tid : tid + 2;
        constants[kNumPowers + tid] = gfw_mul(constants[first], constants[first + 1]);
    }
    __syncthreads();

    // sixteen threads per constant, eight neighbouring coefficients each
    for (uint32_t e = tid; e < kConstants * 16; e += blockDim.x) {
        const uint32_t c = e / 16, byte = e % 16;
        GfWords p = constants[c];
        for (uint32_t i = 0; i < byte; ++i) gfw_mul_x8(p);
        for (int bit = 7; bit >= 0; --bit) {  // coefficient x^(8 byte + 7 - bit)
            basis[c][8 * byte + bit] = gfw_to_block(p);
            gfw_mul_x(p);
        }
    }
    __syncthreads();
    for (uint32_t e = tid; e < (kNumPowers + kNumLanePowers) * kNibbleTableEntries; e += blockDim.x) {
        const uint32_t c = e / kNibbleTableEntries, idx = e % kNibbleTableEntries;
        const uint32_t pos = idx / 16, val = idx % 16;
        const Block* from = &basis[c][8 * (pos / 2) + ((pos & 1) ? 0 : 4)];
        Block z{{0, 0, 0, 0}};
        for (int i = 0; i < 4; ++i)
            if (val & (1u << i)) block_xor(z, from[i]);
        if (c < kNumPowers)
            kt->ghash[c][idx] = z;
        else
            kt->ghash_lane[c - kNumPowers][idx] = z;
        if (c < kLevels) nibbles[c][idx] = z;
    }
    for (uint32_t idx = tid; idx < kNibbleTableEntries; idx += blockDim.x) {
        const Block* from = &basis[kAt192][8 * (idx / 32) + ((idx & 16) ? 0 : 4)];
        Block z{{0, 0, 0, 0}};
        for (int i = 0; i < 4; ++i)
            if (idx & (1u << i)) block_xor(z, from[i]);
        kt->ghash_rows3[idx] = z;
    }

    // Multiplication by H^64 with the bits of every operand quarter in a register of its own lane
    // half (part of the published tables)
    for (uint32_t e = tid; e < kRowMatrixWords; e += blockDim.x) {
        const uint32_t r = e % 4, lane = (e / 4) % 64, ks = (e / 256) % 2, mt = e / 512;
        // the operand row this lane holds, the product bit it makes, the operand quarter
        const uint32_t ml = lane % 32, h = lane / 32, reg = 4 * (ml / 8) + ml % 4;
        const uint32_t word = 2 * ((ml / 4) % 2) + mt / 2, bit = 16 * (reg / 8) + 8 * (mt % 2) + reg % 8;
        uint32_t v = 0;
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t in = 32 * r + 4 * j + 2 * ks + h;
            if ((basis[kRowPower][in].w[word] >> bit) & 1u) v |= 0x2u << (4 * j);  // 1.0 in e2m1
        }
        kt->row_matrix[e] = v;
    }
    // ... and those by H^64 and H^96 in the operand order of the unit kernel (see GhashRowMatrix)
    for (uint32_t e = tid; e < kHashImages * kRowMatrixWords; e += blockDim.x) {
        const uint32_t quarter = e % 4, lane = (e / 4) % 64, ks = (e / 256) % 2, mt = (e / 512) % 4,
                       m = e / kRowMatrixWords;
        const uint32_t ml = lane % 32, reg = 4 * (ml / 8) + ml % 4;
        const uint32_t word = 2 * (mt / 2) + (ml / 4) % 2, bit = 16 * (reg / 8) + 8 * (mt % 2) + reg % 8;
        // 2.0, 1.0, 0.5, 0.5 in e2m1 where the other operand has 0.5, 1.0, 2.0, 2.0
        const uint32_t one = quarter == 0 ? 4u : quarter == 1 ? 2u : 1u;
        uint32_t v = 0;
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t in = 32 * (2 * ks + lane / 32) + 4 * j + quarter;
            if ((basis[m == 0 ? kRowPower : kAt96][in].w[word] >> bit) & 1u) v |= one << (4 * j);
        }
        kt->hash_image[m][e % kRowMatrixWords] = v;
    }

    // H^1 .. H^257, doubling: H^(2^j + i) = H^i * H^(2^j)
    static_assert(kDotBlocks == 1u << kLevels, "and one more");
    if (tid == 0) h_power[1] = constants[0];
    __syncthreads();
    for (uint32_t j = 0; j < kLevels; ++j) {
        if (tid >= 1 && tid <= (1u << j)) {
            const Block b = gf_mul_table(nibbles[j], gfw_to_block(h_power[tid]));
            h_power[(1u << j) + tid] = gfw_from_block(b);
        }
        __syncthreads();
    }
    if (tid == 0)
        h_power[kDotBlocks + 1] =
            gfw_from_block(gf_mul_table(nibbles[0], gfw_to_block(h_power[kDotBlocks])));
    __syncthreads();
    for (uint32_t e = tid; e < kDotBlocks * 4; e += blockDim.x) {
        const uint32_t l = e / 4, t = kDotSlices / 4 * (e % 4);
        GfWords p = h_power[kDotBlocks + 1 - l];
        for (uint32_t i = 0; i < t; ++i) gfw_mul_x8(p);
        for (uint32_t i = t; i < t + kDotSlices / 4; ++i) {
            kt->dot[l / kRowBlocks][i % 4][i / 4][l % kRowBlocks] = p;
            gfw_mul_x8(p);
        }
    }
    // hop[d][k] likewise: k = 2^j + i from i with H^(2^(8 + d + j)), from its nibble table; and the
    // rows' hops
    auto one = [&](GfWords* first) { *first = GfWords{{0x80000000u, 0, 0, 0}}; };
    if (tid < kHopPowers) one(kt->hop[tid]);
    if (tid == kHopPowers) one(kt->row_hop);
    if (tid == kHopPowers + 1) one(kt->far_hop);
    auto next = [&](GfWords* table, uint32_t power, uint32_t j, uint32_t i) {
        const Block b = gf_mul_table(kt->ghash[power + j], gfw_to_block(table[i]));
        table[(1u << j) + i] = gfw_from_block(b);
    };
    for (uint32_t j = 0; j < kRowHopPower; ++j) {
        __syncthreads();
        const uint32_t tables = (1u << j) < kHopEntries ? kHopPowers + 2 : 1;
        for (uint32_t e = tid; e < tables << j; e += blockDim.x) {
            const uint32_t d = e >> j, i = e & ((1u << j) - 1);
            if (d == 0)
                next(kt->row_hop, kRowPower, j, i);
            else if (d == 1)
                next(kt->far_hop, kRowPower + kRowHopPower, j, i);
            else
                next(kt->hop[d - 2], kHopMinPower + d - 2, j, i);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Global memory.
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4* global_u128_cptr;
typedef __attribute__((address_space(1))) u32x4* global_u128_ptr;

// payload accesses go through global (not flat) instructions, so that waiting for LDS results
// never waits for them
__device__ __forceinline__ u32x4 global_read128(const uint8_t* p) {
    return *reinterpret_cast<global_u128_cptr>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ void global_write128(uint8_t* p, u32x4 v) {
    *reinterpret_cast<global_u128_ptr>(reinterpret_cast<uintptr_t>(p)) = v;
}
// ... and so do the single bytes of a ragged last block: one flat access anywhere in the row loop
// would make every wait in it a wait for everything
typedef __attribute__((address_space(1))) const uint8_t* global_u8_cptr;
__device__ __forceinline__ uint8_t global_read8(const uint8_t* p) {
    return *reinterpret_cast<global_u8_cptr>(reinterpret_cast<uintptr_t>(p));
}

// 16 bytes at any alignment
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef __attribute__((address_space(1))) const u32x4_any* global_u128_any_cptr;
typedef __attribute__((address_space(1))) u32x4_any* global_u128_any_ptr;
__device__ __forceinline__ Block global_read_block_any(const uint8_t* p) {
    const u32x4_any v = *reinterpret_cast<global_u128_any_cptr>(reinterpret_cast<uintptr_t>(p));
    return Block{{v.x, v.y, v.z, v.w}};
}
__device__ __forceinline__ void global_write_block_any(uint8_t* p, const Block& b) {
    const u32x4_any v = {b.w[0], b.w[1], b.w[2], b.w[3]};
    *reinterpret_cast<global_u128_any_ptr>(reinterpret_cast<uintptr_t>(p)) = v;
}

// Payload stores that go through to memory at once instead of staying dirty in this XCD's L2:
// for output that a wavefront on another XCD may overwrite later in the same kernel (the wipe of
// a rejected chunk), where two L2s holding different dirty versions of a line would leave it to
// chance which one memory keeps.
// In launches of a few rows a wavefront, encrypting ones write rows of whole lines like this as well (others, whose
// neighbours' parts of a line an L2 puts together, come to host memory 3 % later, 2 of 3 to 4 MB 144.7 us -> 149.0; of sweeps
// see sweep_through): what is left in the L2s is written back when a kernel ends, with nothing else going on (2 MiB 8.47 ->
// 8.23 us, 8 x 512 KiB both ways 24.1 -> 23.8, 28 MB in units 47.3 -> 46.3; but 64 x 4 KiB, in quads, 12.4 -> 12.5, and 2000
// chunks of 16 KiB to 8 MiB in spans 2815 -> 2833).
// (A store of more than 64 bits still reads its registers when the next instruction issues: the next
// two must not write them, and only in code of its own does the compiler see to that.)
__device__ __forceinline__ void global_write128_through(uint8_t* p, u32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void global_write128_through(uint8_t* base, uint32_t offset, u32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, %2 sc0 sc1\n\ts_nop 1"
                 : : "v"(offset), "v"(v), "s"(base) : "memory");
}

// Rows, which are counted back from the end of a chunk's nblk blocks, begin and end with lines of 128 bytes.
__device__ __forceinline__ bool rows_of_whole_lines(const uint8_t* dst, int64_t nblk) {
    return ((reinterpret_cast<uint64_t>(dst) + 16 * (uint64_t)nblk) & 127) == 0;
}

// n < 16 bytes at any alignment, zero-padded, and nothing behind them: pieces of 8, 4, 2 and 1 bytes as
// the bits of n say, all on their way at once.  (Byte by byte, each added to its word before the next
// was asked for, a ragged block took up to fifteen trips to memory one after the other.)
template <class T>
__device__ __forceinline__ T global_read_any(const uint8_t* p) {
    typedef T any __attribute__((aligned(1)));
    return *reinterpret_cast<__attribute__((address_space(1))) const any*>(
        reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ Block read_bytes(const uint8_t* p, uint32_t n) {
    asm volatile("" : "+v"(n));  // what is made of it is not to be kept from row to row
    uint64_t v8 = 0;
    uint32_t v4 = 0, v2 = 0, v1 = 0;
    if (n & 8) v8 = global_read_any<uint64_t>(p);
    if (n & 4) v4 = global_read_any<uint32_t>(p + (n & 8));
    if (n & 2) v2 = global_read_any<uint16_t>(p + (n & 12));
    if (n & 1) v1 = global_read8(p + (n & 14));
    const uint32_t last = (n & 2) ? v2 | v1 << 16 : v1;  // the up to three bytes of the last word
    const uint32_t from4 = (n & 4) ? v4 : last, then = (n & 4) ? last : 0;
    Block b;
    b.w[0] = (n & 8) ? (uint32_t)v8 : from4;
    b.w[1] = (n & 8) ? (uint32_t)(v8 >> 32) : then;
    b.w[2] = (n & 8) ? from4 : 0;
    b.w[3] = (n & 8) ? then : 0;
    return b;
}
// ... and written, to a 16-byte boundary
template <bool kThrough, class T>
__device__ __forceinline__ void global_write_piece(uint8_t* p, T v) {
    auto* const to = reinterpret_cast<__attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p));
    if constexpr (kThrough)
        __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else
        *to = v;
}
template <bool kThrough>
__device__ __forceinline__ void write_bytes(uint8_t* p, uint32_t n, uint32_t w0, uint32_t w1,
                                            uint32_t w2, uint32_t w3) {
    asm volatile("" : "+v"(n), "+v"(w0), "+v"(w1), "+v"(w2), "+v"(w3));
    if (n & 8) global_write_piece<kThrough>(p, (uint64_t)w0 | (uint64_t)w1 << 32);
    if (n & 8) w0 = w2, w1 = w3;  // what is behind that piece
    if (n & 4) global_write_piece<kThrough>(p + (n & 8), w0);
    const uint32_t last = (n & 4) ? w1 : w0;
    if (n & 2) global_write_piece<kThrough>(p + (n & 12), (uint16_t)last);
    if (n & 1) global_write_piece<kThrough>(p + (n & 14), (uint8_t)((n & 2) ? last >> 16 : last));
}

// block i of a byte string, zero-padded (SP 800-38D 6.4)
__device__ __forceinline__ Block padded_block(const uint8_t* p, uint32_t bytes, uint32_t i) {
    const uint32_t off = 16 * i, m = bytes - off;
    if (m >= 16) return global_read_block_any(p + off);
    return read_bytes(p + off, m);
}
}  // namespace

// ------------------------------------------------------------------------------------------
// GHASH state after the AAD of a chunk (SP 800-38D 6.4 over A || 0-pad), hashed serially with the
// table of H in global memory: meant for the short headers AAD is used for.  All lanes that call
// it with the same arguments compute the same value.
namespace {
__device__ Block aad_hash(const KeyTables* __restrict__ kt, const uint8_t* __restrict__ aad,
                          uint32_t aad_len) {
    Block y{{0, 0, 0, 0}};
    for (uint32_t off = 0; off < aad_len; off += 16) {
        const Block x = padded_block(aad, aad_len, off / 16);
        block_xor(y, x);
        y = gf_mul_table(kt->ghash[0], y);
    }
    return y;
}

// Pre-counter block of a chunk (SP 800-38D 7.1 step 2): IV || 0^31 1 for a 96-bit IV, else
// GHASH_H(IV || 0-pad || 0^64 || [8 |IV|]_64).  Same remark on lanes as above.
__device__ Block j0_from_iv(const KeyTables* __restrict__ kt, const uint8_t* __restrict__ iv,
                            uint32_t iv_len) {
    if (iv_len == 12) {
        Block j;
        __builtin_memcpy(j.w, iv, 12);  // at any alignment
        j.w[3] = 0x01000000u;  // be32(1)
        return j;
    }
    Block y = aad_hash(kt, iv, iv_len);
    const uint64_t bits = (uint64_t)iv_len * 8;
    y.w[2] ^= bswap32((uint32_t)(bits >> 32));
    y.w[3] ^= bswap32((uint32_t)bits);
    return gf_mul_table(kt->ghash[0], y);
}

// J0 of the batch's chunk number `chunk`: read from `j0` when the host had it hashed beforehand
// (IVs that are not 96 bits long), otherwise formed from the IV bytes, which sit at the chunk's
// place `index` in the caller's array.
__device__ __forceinline__ Block chunk_j0(const KeyTables* __restrict__ kt,
                                          const uint8_t* __restrict__ ivs,
                                          const Block* __restrict__ j0, uint32_t chunk,
                                          uint32_t index) {
    if (j0 != nullptr) return j0[chunk];
    return j0_from_iv(kt, ivs + (uint64_t)index * 12, 12);
}
}  // namespace

// One thread per chunk: J0 of IVs whose length is not 96 bits, for the kernels that follow.
__global__ __launch_bounds__(64) void j0_kernel(const KeyTables* __restrict__ kt,
                                                const ChunkDesc* __restrict__ chunks,
                                                const uint8_t* __restrict__ ivs, uint32_t iv_len,
                                                uint32_t nchunks, Block* __restrict__ j0) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nchunks) j0[i] = j0_from_iv(kt, ivs + (uint64_t)chunks[i].index * iv_len, iv_len);
}

// ------------------------------------------------------------------------------------------
// Rows.  LDS map of the kernels that walk units and spans (byte addresses):
//   [0, 16 KiB)          operands of the row hash: the matrix images of H^64 and H^96, or the nibble
//                        table of H^64 (entry offsets fit the 16-bit DS offset field)
//   [16 KiB, 80 KiB)     row x (256 B): te[0][x] in dwords 0..31, te[1][x] in dwords 32..63
//   [80 KiB, 144 KiB)    the same for te[2], te[3]
//   [144 KiB, 152 KiB)   every wavefront's second-round constants (see ctr_consts)
// A round-table lookup address is  pair << 16 | x << 8 | 4 * (lane % 32)  plus a constant DS
// offset, so lane l always reads bank l % 32: lookups never collide, whatever the data.
namespace {

constexpr uint32_t kLdsGhBytes = kNibbleTableEntries * 16;
constexpr uint32_t kLdsTeBase = kHashImages * kLdsGhBytes;
constexpr uint32_t kLdsTeBytes = 4 * 256 * 32 * 4;
// counter values that differ above their lowest byte and occur in one segment of a unit
constexpr uint32_t kCtrEntries = 32;
constexpr uint32_t kLdsCtrBase = kLdsTeBase + kLdsTeBytes;
constexpr uint32_t kLdsBytes = kLdsCtrBase + kWavesPerGroup * kCtrEntries * 16;

struct alignas(16) BulkLds {
    Block gh[kHashImages * kNibbleTableEntries];
    uint32_t te[kLdsTeBytes / 4];
    Block ctr[kWavesPerGroup * kCtrEntries];
    Block long_aad[kWavesPerGroup];  // see AadBlocks
    uint32_t rows_done[4];           // see Pace; the first word
};
static_assert(sizeof(BulkLds) == kLdsBytes + 16 * (kWavesPerGroup + 1) && offsetof(BulkLds, gh) == 0 &&
                  offsetof(BulkLds, te) == kLdsTeBase && offsetof(BulkLds, ctr) == kLdsCtrBase,
              "LDS map");

typedef __attribute__((address_space(3))) const uint32_t* lds_u32_ptr;
typedef __attribute__((address_space(3))) const u32x4* lds_u128_ptr;
typedef __attribute__((address_space(3))) u32x4* lds_u128_wptr;
// The AAD comes right before the ciphertext in what is hashed, so its blocks are given the numbers
// -n .. -1 and are hashed by the lanes that lie before the chunk's start: no multiplications of
// their own, where hashing 64 bytes ahead of block 0 from the table in memory takes some 5 us.
// AAD of more than kAadLaneBlocks blocks is meant to be rare: all but its last block is hashed
// first (long_hash), and the sum with that block stands in for "block -1".
constexpr uint32_t kAadLaneBlocks = 64;
__device__ __attribute__((noinline)) Block long_hash(const KeyTables* __restrict__ kt, const uint8_t* p,
                                                     uint32_t blocks, uint32_t lane);

struct AadBlocks {
    const uint8_t* bytes = nullptr;
    uint32_t len = 0, blocks = 0;
    uint32_t stand_in = 0;  // LDS address of what a long AAD has at block -1 (rare: no registers for it)

    __device__ __forceinline__ Block at(int64_t blk) const {
        Block b{{0, 0, 0, 0}};
        if (blocks > kAadLaneBlocks) {
            if (blk == -1) {
                const u32x4 v = *reinterpret_cast<lds_u128_ptr>(stand_in);
                b = Block{{v.x, v.y, v.z, v.w}};
            }
        } else if (blk >= -(int64_t)blocks) {
            b = padded_block(bytes, len, blocks + (uint32_t)(int32_t)blk);
        }
        return b;
    }
    // to be called by the wavefront that walks the blocks before block 0
    __device__ __forceinline__ void prepare(const KeyTables* __restrict__ kt, uint32_t lane) {
        if (__builtin_expect(blocks > kAadLaneBlocks, 0)) {
            Block y = long_hash(kt, bytes, blocks - 1, lane);
            const Block b = padded_block(bytes, len, blocks - 1);
            block_xor(y, b);
            const u32x4 v = {y.w[0], y.w[1], y.w[2], y.w[3]};
            *reinterpret_cast<lds_u128_wptr>(stand_in) = v;
        }
    }
};

// stand_in: LDS for this wavefront
__device__ __forceinline__ AadBlocks aad_blocks(const uint8_t* p, uint32_t len, const Block* stand_in) {
    AadBlocks a;
    a.bytes = p, a.len = len, a.blocks = (uint32_t)(((uint64_t)len + 15) / 16);
    a.stand_in = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)stand_in;
    return a;
}

// waits until every global load and store this wavefront has issued is complete (for a
// device-scope store: has reached memory)
__device__ __forceinline__ void wait_for_own_global_accesses() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// LDS byte address of a __shared__ object
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

__device__ __forceinline__ uint32_t lds_read32(uint32_t addr) {
    return *reinterpret_cast<lds_u32_ptr>(addr);
}
__device__ __forceinline__ u32x4 lds_read128(uint32_t addr) {
    return *reinterpret_cast<lds_u128_ptr>(addr);
}

__device__ __forceinline__ void lds_write128(uint32_t addr, u32x4 v) {
    *reinterpret_cast<lds_u128_wptr>(addr) = v;
}

// The round tables' place and replication in LDS.  A lookup address is bytes 0 and 2 of the lane's
// constants, the looked-up byte in between (so a row of 256 bytes per value), and a constant part
// in the instruction's offset field that selects the table and carries `base`, the LDS address of
// the kernel's tables (a link-time constant; a[] itself must stay free of it because byte 1 of a[]
// is rewritten every round).
// TeWide: 128 KiB, every entry 32 times, so that no lookups collide: 2 cycles each.
struct TeWide {
    static constexpr uint32_t kBase = kLdsTeBase, kPairs = 0x10000u, kLanes = 32;
    static constexpr uint32_t offset(int t) { return kBase + 128u * (t & 1); }
};
template <class Te, int T>
__device__ __forceinline__ uint32_t te_read(uint32_t a, uint32_t base) {
    return lds_read32(a + (base + Te::offset(T)));
}

// a.byte1 = rk.byte[KS] ^ v.byte[KV], every other byte of a kept: one SDWA instruction folds the
// AddRoundKey of a state byte into forming its next lookup address.
template <int KS, int KV>
__device__ __forceinline__ void key_xor_into_addr(uint32_t& a, uint32_t rk, uint32_t v) {
    static_assert(KS >= 0 && KS < 4 && KV >= 0 && KV < 4, "byte index");
    if constexpr (KS == 0 && KV == 0)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:BYTE_0" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 1 && KV == 1)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:BYTE_1" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 2 && KV == 2)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:BYTE_2" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 3 && KV == 3)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_3" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 3 && KV == 0)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_0" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 2 && KV == 1)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:BYTE_1" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 1 && KV == 2)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:BYTE_2" : "+v"(a) : "s"(rk), "v"(v));
    else if constexpr (KS == 0 && KV == 3)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:BYTE_3" : "+v"(a) : "s"(rk), "v"(v));
    else
        static_assert(KS == KV, "unsupported byte pairing");
}

// Sixteen lookup-address registers, one per state byte: a[j][k] serves byte k (row k) of column
// j and always reads table k.  Bytes 0 and 2 hold the lane's constants for the whole kernel;
// byte 1 is rewritten every round.
struct AesAddr {
    uint32_t a[4][4];
    // the last round key, in vector registers: the sixty key words and everything else a kernel
    // keeps in scalar registers do not fit them all, and one that is spilled costs a vector
    // instruction per use
    uint32_t last_key[4];
};

// last_round_key: the four words of round key Nr
template <class Te>
__device__ __forceinline__ void aes_addr_init(AesAddr& A, uint32_t lane) {
    const uint32_t lo = (lane & (Te::kLanes - 1)) * 4, hi = lo | Te::kPairs;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        A.a[j][0] = lo;
        A.a[j][1] = lo;
        A.a[j][2] = hi;
        A.a[j][3] = hi;
    }
}
template <class Te>
__device__ __forceinline__ void aes_addr_init(AesAddr& A, uint32_t lane,
                                              const uint32_t* __restrict__ last_round_key) {
    aes_addr_init<Te>(A, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        A.last_key[j] = last_round_key[j];
        asm volatile("" : "+v"(A.last_key[j]));  // a vector register, and kept there
    }
}

// What the first two rounds of a unit's counter blocks have in common.  The blocks differ in the
// counter word only, and within a segment of at most kSegmentRows rows the counter takes few values
// above its lowest byte.  The lowest byte reaches, in round 1, column 0 alone, whose other three
// lookups depend on the IV only: k0 is their sum.  In round 2 that column feeds one lookup of every
// column; the other three depend on the IV and the counter's upper bytes: their sums, four words,
// are kept in LDS for every upper value the segment meets (lane i of the wavefront forms the one
// i above the first).  So a block takes one lookup in round 1 and four in round 2 instead of
// sixteen each, for 27 lookups per segment and one 16-byte read per row; in most rows of longer pieces
// it takes none, see CtrClass.  The kernel is bound by
// LDS accesses and by the board's power together, and both go down: per row of 64 blocks 555 -> 532
// LDS cycles and 448 -> 432 vector instructions, 1.424 -> 1.389 ms for 4096 chunks of 320 KiB
// (AES-256, alternating on one box), against keeping only round 1's constant sums.
constexpr uint32_t kSegmentRows = 123;
static_assert(255 + (kSegmentRows + 1) * kRowBlocks <= 256 * kCtrEntries,
              "upper counter values of a segment of kSegmentRows rows, or one more");
struct CtrConsts {
    uint32_t k0;
    uint32_t q_addr;  // LDS address of the wavefront's entries
    // of the row at hand: this lane's block number in the segment plus the lowest byte of the
    // segment's first counter, so that its lowest byte is the counter's and rel >> 8 the number
    // of the upper counter value
    uint32_t rel;
};

// Rows four apart have the same lowest counter byte in a lane, and what round 2 makes of it, one lookup
// of every column, is then the same as well: it is kept in registers, for four classes of rows, and
// their rounds 1 and 2 take no lookup at all but that of q, fetched a row ahead.  Sixteen registers
// and four copies of a row's code, for 10 of 532 LDS cycles and, with the checks that rows within a
// piece do without, some 30 of 438 vector instructions: 4096 chunks of 320 KiB both ways 2658 -> 2592
// us, 2000 of 16 KiB to 8 MiB 2889 -> 2813 (alternating).  What binds is the board's power: without
// those 10 cycles alone it was 2.3 %, and taking the checks out as well gave next to nothing.
constexpr uint32_t kRowClasses = 4;
static_assert(kRowClasses * kRowBlocks == 256, "the lowest counter byte's period in rows");
struct CtrClass {
    uint32_t s[4];
};
struct CtrInner {
    const CtrClass& low;
    u32x4& q;
    uint32_t next;  // LDS address of the next row's q
};

// first_ctr: the counter of the segment's first block (the same in every lane)
__device__ __forceinline__ CtrConsts ctr_consts(const uint32_t* __restrict__ rk, uint32_t lane,
                                                uint32_t wave, uint32_t iv0, uint32_t iv1,
                                                uint32_t iv2, uint32_t first_ctr, uint32_t base) {
    using Te = TeWide;
    const uint32_t lo = (lane & 31) * 4, hi = lo | 0x10000u;
    auto at = [&](uint32_t w, int k, uint32_t lane_bytes) {
        return (((w >> (8 * k)) & 0xFFu) << 8) | lane_bytes;
    };
    const uint32_t upper = ((first_ctr >> 8) + lane) << 8;
    const uint32_t s0 = iv0 ^ rk[0], s1 = iv1 ^ rk[1], s2 = iv2 ^ rk[2],
                   s3 = bswap32(upper) ^ rk[3];
    CtrConsts c;
    c.k0 = xor3(te_read<Te, 0>(at(s0, 0, lo), base), te_read<Te, 1>(at(s1, 1, lo), base),
                te_read<Te, 2>(at(s2, 2, hi), base));
    const uint32_t u1 = xor3(te_read<Te, 0>(at(s1, 0, lo), base), te_read<Te, 1>(at(s2, 1, lo), base),
                             te_read<Te, 2>(at(s3, 2, hi), base)) ^
                        te_read<Te, 3>(at(s0, 3, hi), base) ^ rk[5];
    const uint32_t u2 = xor3(te_read<Te, 0>(at(s2, 0, lo), base), te_read<Te, 1>(at(s3, 1, lo), base),
                             te_read<Te, 2>(at(s0, 2, hi), base)) ^
                        te_read<Te, 3>(at(s1, 3, hi), base) ^ rk[6];
    const uint32_t u3 = xor3(te_read<Te, 0>(at(s3, 0, lo), base), te_read<Te, 1>(at(s0, 1, lo), base),
                             te_read<Te, 2>(at(s1, 2, hi), base)) ^
                        te_read<Te, 3>(at(s2, 3, hi), base) ^ rk[7];
    u32x4 q;
    q.x = xor3(te_read<Te, 1>(at(u1, 1, lo), base), te_read<Te, 2>(at(u2, 2, hi), base),
               te_read<Te, 3>(at(u3, 3, hi), base));
    q.y = xor3(te_read<Te, 0>(at(u1, 0, lo), base), te_read<Te, 1>(at(u2, 1, lo), base),
               te_read<Te, 2>(at(u3, 2, hi), base));
    q.z = xor3(te_read<Te, 0>(at(u2, 0, lo), base), te_read<Te, 1>(at(u3, 1, lo), base),
               te_read<Te, 3>(at(u1, 3, hi), base));
    q.w = xor3(te_read<Te, 0>(at(u3, 0, lo), base), te_read<Te, 2>(at(u1, 2, hi), base),
               te_read<Te, 3>(at(u2, 3, hi), base));
    c.q_addr = base + kLdsCtrBase + wave * (kCtrEntries * 16);
    if (lane < kCtrEntries) lds_write128(c.q_addr + lane * 16, q);
    // the wavefront's own later reads come after this write: LDS serves a wavefront in order
    asm volatile("" ::: "memory");
    c.rel = (first_ctr & 0xFFu) + lane;
    return c;
}

__device__ __forceinline__ uint32_t ctr_q_addr(const CtrConsts& C, uint32_t rel) {
    return C.q_addr + ((rel >> 8) << 4);
}

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// (v.byte[K]) & 0xF0: the table offset of a high nibble, in one instruction
template <int K>
__device__ __forceinline__ uint32_t nibble_offset(uint32_t v, uint32_t mask_f0) {
    uint32_t r;
    if constexpr (K == 0)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "s"(mask_f0), "v"(v));
    else if constexpr (K == 1)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "s"(mask_f0), "v"(v));
    else if constexpr (K == 2)
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "s"(mask_f0), "v"(v));
    else
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "s"(mask_f0), "v"(v));
    return r;
}

// The row hash.  An engine keeps a unit's hash state in four registers per lane, in a form of its
// own, from row to row: start() clears it, begin() prepares a row's multiplication, its parts
// ride along with the row's AES rounds, absorb() adds the row's ciphertext, home() leaves the
// unit's 64 lane sums as blocks.

// Y * H^64 in every lane, from the nibble table in LDS, cut into sixteen byte steps (two 16-byte
// lookups and eight XORs each) so that the steps can be spread over the AES rounds of the same
// row: the hash arithmetic then fills the time the wavefront would wait for round-table lookups.
struct GhashRowMul {
    static constexpr bool kMatrix = false, kTable = true;
    uint32_t table; // LDS address of the nibble table of H^64
    uint32_t w[4];  // the state, and the multiplicand
    uint32_t t;     // current word << 4: its byte k carries the low nibble of byte k
    uint32_t z0, z1, z2, z3;
    u32x4 ra, rb;

    __device__ __forceinline__ void start(uint32_t lds_table, uint32_t) {
        table = lds_table;
        w[0] = w[1] = w[2] = w[3] = 0;
    }
    __device__ __forceinline__ void begin() { z0 = z1 = z2 = z3 = 0; }
    template <int S>
    __device__ __forceinline__ void issue() {
        constexpr int i = S / 4, k = S % 4;
        constexpr uint32_t pos = 2 * S;
        const uint32_t f0 = 0xF0u;
        if constexpr (k == 0) t = w[i] << 4;
        ra = lds_read128(nibble_offset<k>(w[i], f0) + (table + pos * 256));
        rb = lds_read128(nibble_offset<k>(t, f0) + (table + (pos + 1) * 256));
    }
    __device__ __forceinline__ void consume() {
        z0 = xor3(z0, ra.x, rb.x);
        z1 = xor3(z1, ra.y, rb.y);
        z2 = xor3(z2, ra.z, rb.z);
        z3 = xor3(z3, ra.w, rb.w);
        // pin the running sums here: otherwise the optimizer moves the whole XOR chain to where
        // its result is used and keeps all thirty-two table entries alive until then
        asm volatile("" : "+v"(z0), "+v"(z1), "+v"(z2), "+v"(z3));
    }
    template <int S>
    __device__ __forceinline__ void step() {
        issue<S>();
        consume();
    }
    __device__ __forceinline__ void absorb(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
        w[0] = z0 ^ c0, w[1] = z1 ^ c1, w[2] = z2 ^ c2, w[3] = z3 ^ c3;
    }
    __device__ __forceinline__ void home(uint32_t y[4]) const {
        y[0] = w[0], y[1] = w[1], y[2] = w[2], y[3] = w[3];
    }
};

// The same on the matrix cores, with the two halves of a row folded together.  The state is, lane
// by lane, Z; a row turns it into
//     Z'[0..31] = C[0..31],     Z'[32..63] = C[32..63] + Z[32..63] * H^64 + Z[0..31] * H^96,
// which stands for the same sum of C(r, lane) * H^(64 * rows after r + 64 - lane) as a
// multiplication of all 64 lanes by H^64 would: lane l's blocks are moved one row and 32
// blocks on, to lane l + 32.  Only 32 products are left to be made per row, each a sum of two.
// Multiplication by a constant is linear over GF(2): product bit m is the parity of the number of
// bits k with M[m][k] = Z[k] = 1, and the matrix instruction counts those for 32 product bits of
// 32 columns at once when every bit is spread out to a 4-bit floating-point number.  Per row: 4
// product tiles x 2 factors x 2 instructions of depth 64.  Products are scaled down into the
// denormal range, where a float's pattern is the integer it counts in units of 2^-149 (the matrix
// pipeline keeps denormals, in its results and in the sum it continues from), and rows are
// scaled apart: result register i of a lane counts in units of 2^(i % 8), and the second tile of
// a pair shares the first one's registers, another 2^8 up.  So one register holds two counts
// whose lowest bits, the parities, sit at bits i % 8 and 8 + i % 8: one masked OR per register
// collects them, eight registers to a half word.  The two counts stay apart because neither
// reaches 256: a row of M that is all ones belongs to one constant only (bit m of x * h as a
// function of x is another one for every h), so both factors' rows could only be all ones
// with H^64 = H^96, that is H = 1 (or 0), whose matrix has single ones.
// No table lookups: the matrix images (16 KiB) are read from LDS, 16 bytes per lane and
// instruction.  Per row that leaves 467 LDS cycles of the 532 the nibble table needs and 3 % fewer
// cycles in all, but the matrix pipeline draws so much more power that the chip, at its limit
// of 1400 W under either engine, clocks at 2.15 instead of 2.23 GHz: 1.40 ms against 1.38 ms for
// 4096 chunks of 320 KiB.  So the table is the default.
//
// Operand layout of v_mfma_scale_f32_32x32x64_f8f6f4 with 4-bit operands: lane l holds row (or
// column) l % 32, depth elements 32 (l / 32) .. + 31, eight to a register, lowest nibble first;
// one scale (a power of two, biased by 127, in byte 0) per lane.  Result register i of lane l is
// row 8 (i / 4) + 4 (l / 32) + i % 4 of column l % 32.
// Depth element <-> bit of Z: slice s of the depth is words 2 s (lanes 0..31) and 2 s + 1 (lanes
// 32..63); register c of it holds bits 4 j + c, left where they are inside their nibble (worth 0.5,
// 1.0, 2.0; bit 3 would be the sign and is moved down one place), which the matrix entries make
// up for (2.0, 1.0, 0.5, 0.5).
// Product bit <-> row: tile pair p makes word 2 p in lanes 0..31 and word 2 p + 1 in lanes 32..63,
// register i of tile 2 p + f its bit 16 (i / 8) + 8 f + i % 8 (KeyTables::hash_image is laid out to
// match).  So a result comes in the very lanes in which the next row needs it as operand, and the
// state is kept like that: lo[s], hi[s] are words 2 s (lanes 0..31) and 2 s + 1 (lanes 32..63) of
// lanes 0..31 and of lanes 32..63; two swaps of lane halves bring a row's ciphertext there.
typedef int v8i32 __attribute__((ext_vector_type(8)));
typedef float v16f32 __attribute__((ext_vector_type(16)));

struct GhashRowMatrix {
    static constexpr bool kMatrix = true, kTable = false;
    uint32_t image;    // LDS address of this lane's first piece of the matrix images
    uint32_t scale_a;  // scale of this lane's matrix row in the first tile of a pair
    uint32_t scale_a2; // ... in the second
    uint32_t lo[2], hi[2];
    uint32_t q[2][2][4];  // [factor: hi with H^64, lo with H^96][slice][bits 4 j + c]
    uint32_t out[2];
    u32x4 a0, a1;
    v16f32 acc;

    // matrix rows are scaled to 2^-127 and up, the other operand to 2^-22
    static constexpr int kScaleB = 127 - 22;

    __device__ __forceinline__ void start(uint32_t lds_table, uint32_t lane) {
        image = lds_table + lane * 16;
        const uint32_t row = lane & 31, reg = 4 * (row / 8) + row % 4;
        scale_a = reg % 8;  // 2^(reg % 8 - 127)
        scale_a2 = scale_a + 8;
        lo[0] = lo[1] = hi[0] = hi[1] = 0;
    }
    __device__ __forceinline__ void begin() {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const uint32_t w = m == 0 ? hi[s] : lo[s];
                q[m][s][0] = w & 0x11111111u;
                q[m][s][1] = w & 0x22222222u;
                q[m][s][2] = w & 0x44444444u;
                q[m][s][3] = (w >> 1) & 0x44444444u;
            }
    }
    // Step I = 0 .. 7: chain I / 4 (a tile pair: eight instructions into one set of sums), tile
    // (I / 2) % 2 of it, factor I % 2; each in three parts that the caller spreads over an AES
    // round: the two matrix pieces are fetched, the first instruction starts or continues the
    // sums, the second (which has to wait for the first) follows.
    template <int I>
    __device__ __forceinline__ void load() {
        constexpr int piece = ((I % 2) * 4 + 2 * (I / 4) + (I / 2) % 2) * 2;
        a0 = lds_read128(image + piece * 1024);
        a1 = lds_read128(image + (piece + 1) * 1024);
    }
    template <int I, int S>
    __device__ __forceinline__ void product() {
        constexpr int m = I % 2, f = (I / 2) % 2;
        const u32x4 a = S == 0 ? a0 : a1;
        const v8i32 A = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
        const v8i32 B = {(int)q[m][S][0], (int)q[m][S][1], (int)q[m][S][2], (int)q[m][S][3],
                         0, 0, 0, 0};
        if constexpr (I % 4 == 0 && S == 0) {
            const v16f32 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                                 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                A, B, zero, 4, 4, 0, (int)(f == 0 ? scale_a : scale_a2), 0, kScaleB);
        } else {
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                A, B, acc, 4, 4, 0, (int)(f == 0 ? scale_a : scale_a2), 0, kScaleB);
        }
    }
    // the chain's thirty-two parities: registers 0..7 give the low half word, 8..15 the high
    template <int C>
    __device__ __forceinline__ void consume() {
        uint32_t l = __float_as_uint(acc[0]) & 0x0101u, h = __float_as_uint(acc[8]) & 0x0101u;
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            // (sum & mask) | collected, in one instruction (truth table 0xEA)
            const uint32_t mask = 0x0101u << i;
            l = __builtin_amdgcn_bitop3_b32(__float_as_uint(acc[i]), mask, l, 0xEA);
            h = __builtin_amdgcn_bitop3_b32(__float_as_uint(acc[8 + i]), mask, h, 0xEA);
        }
        out[C] = (h << 16) | l;
        // pinned here: otherwise the optimizer moves the whole chain to where its result is used
        asm volatile("" : "+v"(out[C]));
    }
    __device__ __forceinline__ void absorb(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
        // lanes 32..63 of the first word change places with lanes 0..31 of the second
        const auto r0 = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
        const auto r1 = __builtin_amdgcn_permlane32_swap(c2, c3, false, false);
        lo[0] = r0[0], hi[0] = r0[1] ^ out[0];
        lo[1] = r1[0], hi[1] = r1[1] ^ out[1];
    }
    __device__ __forceinline__ void home(uint32_t y[4]) const {
        const auto r0 = __builtin_amdgcn_permlane32_swap(lo[0], hi[0], false, false);
        const auto r1 = __builtin_amdgcn_permlane32_swap(lo[1], hi[1], false, false);
        y[0] = r0[0], y[1] = r0[1], y[2] = r1[0], y[3] = r1[1];
    }
};

// Rounds kFirst .. kRounds of AES with the row's GHASH multiplication G riding along; rk is
// wave-uniform (scalar registers).  Between rounds the state u0 .. u3 is carried without its round
// key: the key bytes are added while the next round's addresses are formed.
// The byte steps of a table hash from step 4 on are spread evenly over rounds 3 .. kRounds (one
// each for AES-256, one or two each for the shorter keys).
// On the matrix cores the multiplication is two chains of eight instructions instead: chain c is
// issued in rounds 4 c + 3 .. 4 c + 6 (two matrix pieces fetched ahead of each round's lookups,
// two instructions, one before and one after the round's sums) and its result packed in the
// middle of the round after, so that neither the fetch nor the matrix pipeline is waited for.
template <class Te, int kFirst, int kRounds, class Hash>
__device__ __forceinline__ void aes_rounds_lds(const uint32_t* __restrict__ rk, AesAddr& A,
                                               uint32_t u0, uint32_t u1, uint32_t u2, uint32_t u3,
                                               Hash& G, uint32_t base, uint32_t& o0, uint32_t& o1,
                                               uint32_t& o2, uint32_t& o3) {
    static_assert(kRounds >= 10, "eight pairs of matrix instructions in rounds 3 .. 10");
    static_for<kFirst, kRounds + 1>([&](auto round) __attribute__((always_inline)) {
        constexpr int r = decltype(round)::value;
        constexpr int step_begin = 4 + (12 * (r - 3)) / (kRounds - 2),
                      step_end = 4 + (12 * (r - 2)) / (kRounds - 2);
        static_assert(!Hash::kTable || step_end - step_begin == 1 || step_end - step_begin == 2,
                      "hash steps");
        const uint32_t* k = rk + 4 * (r - 1);
        if constexpr (Hash::kMatrix) {
            if constexpr (r <= 10) G.template load<r - 3>();
            __builtin_amdgcn_sched_barrier(0);
        }
        key_xor_into_addr<0, 0>(A.a[0][0], k[0], u0);
        key_xor_into_addr<1, 1>(A.a[0][1], k[0], u0);
        key_xor_into_addr<2, 2>(A.a[0][2], k[0], u0);
        key_xor_into_addr<3, 3>(A.a[0][3], k[0], u0);
        key_xor_into_addr<0, 0>(A.a[1][0], k[1], u1);
        key_xor_into_addr<1, 1>(A.a[1][1], k[1], u1);
        key_xor_into_addr<2, 2>(A.a[1][2], k[1], u1);
        key_xor_into_addr<3, 3>(A.a[1][3], k[1], u1);
        key_xor_into_addr<0, 0>(A.a[2][0], k[2], u2);
        key_xor_into_addr<1, 1>(A.a[2][1], k[2], u2);
        key_xor_into_addr<2, 2>(A.a[2][2], k[2], u2);
        key_xor_into_addr<3, 3>(A.a[2][3], k[2], u2);
        key_xor_into_addr<0, 0>(A.a[3][0], k[3], u3);
        key_xor_into_addr<1, 1>(A.a[3][1], k[3], u3);
        key_xor_into_addr<2, 2>(A.a[3][2], k[3], u3);
        key_xor_into_addr<3, 3>(A.a[3][3], k[3], u3);
        uint32_t t00 = te_read<Te, 0>(A.a[0][0], base), t11 = te_read<Te, 1>(A.a[1][1], base),
                 t22 = te_read<Te, 2>(A.a[2][2], base), t33 = te_read<Te, 3>(A.a[3][3], base);
        uint32_t t10 = te_read<Te, 0>(A.a[1][0], base), t21 = te_read<Te, 1>(A.a[2][1], base),
                 t32 = te_read<Te, 2>(A.a[3][2], base), t03 = te_read<Te, 3>(A.a[0][3], base);
        uint32_t t20 = te_read<Te, 0>(A.a[2][0], base), t31 = te_read<Te, 1>(A.a[3][1], base),
                 t02 = te_read<Te, 2>(A.a[0][2], base), t13 = te_read<Te, 3>(A.a[1][3], base);
        uint32_t t30 = te_read<Te, 0>(A.a[3][0], base), t01 = te_read<Te, 1>(A.a[0][1], base),
                 t12 = te_read<Te, 2>(A.a[1][2], base), t23 = te_read<Te, 3>(A.a[2][3], base);
        if constexpr (Hash::kMatrix) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (r == 7) G.template consume<0>();
            if constexpr (r == 11) G.template consume<1>();
            if constexpr (r <= 10) G.template product<r - 3, 0>();
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (Hash::kTable) G.template issue<step_begin>();
        if constexpr (r < kRounds) {
            u0 = xor3(t00, t11, t22) ^ t33;
            u1 = xor3(t10, t21, t32) ^ t03;
            u2 = xor3(t20, t31, t02) ^ t13;
            u3 = xor3(t30, t01, t12) ^ t23;
        } else {
            // last round, no MixColumns: S(x) is byte 1 of te[0], byte 2 of te[1], byte 0 of
            // te[2] and te[3]
            auto last = [&](uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, uint32_t key) {
                uint32_t lo = __builtin_amdgcn_perm(v0, v1, 0x0c0c0205u);  // [v0.b1, v1.b2, 0, 0]
                uint32_t hi = __builtin_amdgcn_perm(v2, v3, 0x00040c0cu);  // [0, 0, v2.b0, v3.b0]
                return xor3(lo, hi, key);
            };
            o0 = last(t00, t11, t22, t33, A.last_key[0]);
            o1 = last(t10, t21, t32, t03, A.last_key[1]);
            o2 = last(t20, t31, t02, t13, A.last_key[2]);
            o3 = last(t30, t01, t12, t23, A.last_key[3]);
        }
        if constexpr (Hash::kMatrix) {
            if constexpr (r <= 10) {
                __builtin_amdgcn_sched_barrier(0);  // after the round's sums, not before
                G.template product<r - 3, 1>();
            }
        }
        if constexpr (Hash::kTable) {
            G.consume();
            if constexpr (step_end - step_begin == 2) G.template step<step_begin + 1>();
        }
        // keep every round's hash step with its round: without this the compiler sinks the
        // hash XORs to the end of the block and spills the table entries they wait for
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (Hash::kMatrix && kRounds == 10) G.template consume<1>();
}

// E_K(J0[0..95] || be32(ctr)) for this lane's counter, in a row of a unit of several: rounds 1 and
// 2 from the unit's constants, with two byte steps of a table hash each.
template <int kRounds, class Hash>
__device__ __forceinline__ void aes_ctr_lds(const uint32_t* __restrict__ rk, AesAddr& A,
                                            const CtrConsts& C, Hash& G, uint32_t base,
                                            uint32_t& o0, uint32_t& o1, uint32_t& o2,
                                            uint32_t& o3) {
    using Te = TeWide;
    const u32x4 q = lds_read128(ctr_q_addr(C, C.rel));
    // round 1: the counter is the last word, big endian: its lowest byte is state byte 3
    key_xor_into_addr<3, 0>(A.a[3][3], rk[3], C.rel);
    uint32_t u0 = te_read<Te, 3>(A.a[3][3], base) ^ C.k0;
    if constexpr (Hash::kTable) {
        G.template step<0>();
        G.template step<1>();
    }
    // round 2: column 0 alone depends on the lowest counter byte
    key_xor_into_addr<0, 0>(A.a[0][0], rk[4], u0);
    key_xor_into_addr<1, 1>(A.a[0][1], rk[4], u0);
    key_xor_into_addr<2, 2>(A.a[0][2], rk[4], u0);
    key_xor_into_addr<3, 3>(A.a[0][3], rk[4], u0);
    u0 = te_read<Te, 0>(A.a[0][0], base) ^ q.x;
    const uint32_t u3 = te_read<Te, 1>(A.a[0][1], base) ^ q.w, u2 = te_read<Te, 2>(A.a[0][2], base) ^ q.z,
                   u1 = te_read<Te, 3>(A.a[0][3], base) ^ q.y;
    if constexpr (Hash::kTable) {
        G.template step<2>();
        G.template step<3>();
    }
    __builtin_amdgcn_sched_barrier(0);
    aes_rounds_lds<Te, 3, kRounds>(rk, A, u0, u1, u2, u3, G, base, o0, o1, o2, o3);
}

// round 2's lookups of the lowest counter byte of the row `row` behind the one at hand
__device__ __forceinline__ CtrClass ctr_class(const uint32_t* __restrict__ rk, AesAddr& A,
                                              const CtrConsts& C, uint32_t row, uint32_t base) {
    using Te = TeWide;
    CtrClass c;
    key_xor_into_addr<3, 0>(A.a[3][3], rk[3], C.rel + row * kRowBlocks);
    const uint32_t u0 = te_read<Te, 3>(A.a[3][3], base) ^ C.k0;
    key_xor_into_addr<0, 0>(A.a[0][0], rk[4], u0);
    key_xor_into_addr<1, 1>(A.a[0][1], rk[4], u0);
    key_xor_into_addr<2, 2>(A.a[0][2], rk[4], u0);
    key_xor_into_addr<3, 3>(A.a[0][3], rk[4], u0);
    c.s[0] = te_read<Te, 0>(A.a[0][0], base);
    c.s[3] = te_read<Te, 1>(A.a[0][1], base);
    c.s[2] = te_read<Te, 2>(A.a[0][2], base);
    c.s[1] = te_read<Te, 3>(A.a[0][3], base);
    return c;
}
// The same in a row of which every lane has a whole block, with its class's lookups made.
template <int kRounds, class Hash>
__device__ __forceinline__ void aes_ctr_lds(const uint32_t* __restrict__ rk, AesAddr& A,
                                            const CtrInner& C, Hash& G, uint32_t base,
                                            uint32_t& o0, uint32_t& o1, uint32_t& o2,
                                            uint32_t& o3) {
    const uint32_t u0 = C.low.s[0] ^ C.q.x, u1 = C.low.s[1] ^ C.q.y, u2 = C.low.s[2] ^ C.q.z,
                   u3 = C.low.s[3] ^ C.q.w;
    C.q = lds_read128(C.next);
    if constexpr (Hash::kTable) {
        G.template step<0>();
        G.template step<1>();
        G.template step<2>();
        G.template step<3>();
    }
    __builtin_amdgcn_sched_barrier(0);
    aes_rounds_lds<TeWide, 3, kRounds>(rk, A, u0, u1, u2, u3, G, base, o0, o1, o2, o3);
}

// One block, the same in every lane, by a wavefront that has nothing else to do; lane i of key_word has
// round key word i.
template <class Te>
__device__ __forceinline__ void aes_block_lds(uint32_t key_word, uint32_t rounds, uint32_t lane,
                                              uint32_t base, uint32_t (&u)[4]) {
    AesAddr A;
    aes_addr_init<Te>(A, lane);
    uint32_t t[4][4];
    auto lookups = [&](uint32_t r) __attribute__((always_inline)) {
        static_for<0, 4>([&](auto col) __attribute__((always_inline)) {
            constexpr int c = decltype(col)::value;
            const uint32_t k = __builtin_amdgcn_readlane(key_word, 4 * r + c);
            key_xor_into_addr<0, 0>(A.a[c][0], k, u[c]);
            key_xor_into_addr<1, 1>(A.a[c][1], k, u[c]);
            key_xor_into_addr<2, 2>(A.a[c][2], k, u[c]);
            key_xor_into_addr<3, 3>(A.a[c][3], k, u[c]);
        });
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            t[c][0] = te_read<Te, 0>(A.a[c][0], base);
            t[c][1] = te_read<Te, 1>(A.a[(c + 1) & 3][1], base);
            t[c][2] = te_read<Te, 2>(A.a[(c + 2) & 3][2], base);
            t[c][3] = te_read<Te, 3>(A.a[(c + 3) & 3][3], base);
        }
    };
#pragma unroll 1
    for (uint32_t r = 0; r + 1 < rounds; ++r) {
        lookups(r);
#pragma unroll
        for (int c = 0; c < 4; ++c) u[c] = xor3(t[c][0], t[c][1], t[c][2]) ^ t[c][3];
    }
    lookups(rounds - 1);
    // last round, no MixColumns: S(x) is byte 1 of te[0], byte 2 of te[1], byte 0 of te[2] and te[3]
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t lo = __builtin_amdgcn_perm(t[c][0], t[c][1], 0x0c0c0205u);
        const uint32_t hi = __builtin_amdgcn_perm(t[c][2], t[c][3], 0x00040c0cu);
        u[c] = xor3(lo, hi, __builtin_amdgcn_readlane(key_word, 4 * rounds + c));
    }
}

// Y * C from C's nibble table at LDS address `base`, on its own (not riding along with AES):
// the eight lookups of each word are issued together.
__device__ __forceinline__ void ghash_mul_lds(uint32_t base, uint32_t y[4]) {
    uint32_t z0 = 0, z1 = 0, z2 = 0, z3 = 0;
    const uint32_t f0 = 0xF0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = y[i], t = y[i] << 4;
        u32x4 e[8];
        e[0] = lds_read128(base + nibble_offset<0>(w, f0) + (8 * i + 0) * 256);
        e[1] = lds_read128(base + nibble_offset<0>(t, f0) + (8 * i + 1) * 256);
        e[2] = lds_read128(base + nibble_offset<1>(w, f0) + (8 * i + 2) * 256);
        e[3] = lds_read128(base + nibble_offset<1>(t, f0) + (8 * i + 3) * 256);
        e[4] = lds_read128(base + nibble_offset<2>(w, f0) + (8 * i + 4) * 256);
        e[5] = lds_read128(base + nibble_offset<2>(t, f0) + (8 * i + 5) * 256);
        e[6] = lds_read128(base + nibble_offset<3>(w, f0) + (8 * i + 6) * 256);
        e[7] = lds_read128(base + nibble_offset<3>(t, f0) + (8 * i + 7) * 256);
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            z0 = xor3(z0, e[k].x, e[k + 1].x);
            z1 = xor3(z1, e[k].y, e[k + 1].y);
            z2 = xor3(z2, e[k].z, e[k + 1].z);
            z3 = xor3(z3, e[k].w, e[k + 1].w);
        }
    }
    y[0] = z0, y[1] = z1, y[2] = z2, y[3] = z3;
}

// One row's payload in this lane: block `blk` of the chunk.  On `edge` rows (the first and the last
// row of a chunk; a wave-uniform flag) some lanes may lie before the chunk's start and stay idle,
// and the last lane may hold the chunk's ragged last block.
struct RowPayload {
    uint32_t x0, x1, x2, x3;
    uint32_t tail;  // bytes in a ragged block, 0 = whole block or none
    bool whole;

    __device__ __forceinline__ void arrive() {}  // (asked for by load_row, waited for where it is used)
};

// Lanes before the chunk's start get the AAD's blocks, or zero blocks.
__device__ __forceinline__ RowPayload load_row(const uint8_t* src, uint64_t len, int64_t blk,
                                               bool edge, const AadBlocks& aad) {
    RowPayload r{0, 0, 0, 0, 0, true};
    const uint8_t* sp = src + blk * 16;
    if (!edge) {
        const u32x4 v = global_read128(sp);
        r.x0 = v.x, r.x1 = v.y, r.x2 = v.z, r.x3 = v.w;
    } else {
        const bool active = blk >= 0;
        if (active && (uint64_t)blk * 16 + 16 > len) r.tail = (uint32_t)(len & 15);
        r.whole = active && r.tail == 0;
        if (r.whole) {
            const u32x4 v = global_read128(sp);
            r.x0 = v.x, r.x1 = v.y, r.x2 = v.z, r.x3 = v.w;
        }
        if (blk < 0) {
            const Block a = aad.at(blk);
            r.x0 = a.w[0], r.x1 = a.w[1], r.x2 = a.w[2], r.x3 = a.w[3];
        }
        if (__builtin_expect(r.tail != 0, 0)) {
            const Block v = read_bytes(sp, r.tail);
            r.x0 = v.w[0], r.x1 = v.w[1], r.x2 = v.w[2], r.x3 = v.w[3];
        }
    }
    return r;
}

// One row of a unit: the payload loaded by load_row is encrypted or decrypted, stored and hashed.
// On edge rows lanes before the chunk's start store nothing; they hash what load_row gave them.  The counter block of "block -1" is J0, so the idle
// lane there computes E_K(J0), the mask of the chunk's tag (SP 800-38D 7.1 steps 2 and 6), which
// is handed to store_mask.
// kThrough: the payload is written through to memory (see global_write128_through).
// G: the row hash engine, on the matrix cores or from a table.
// `edge` is the same in every lane and held in a scalar register (walk_unit sees to that), so
// the rows that are no edge rows branch past all of the checks.
// through: whole blocks are, too, if that is not known when compiled.
template <bool kDecrypt, int kRounds, bool kThrough, class Keys, class Ctr, class Row, class Hash, class StoreMask>
__device__ __forceinline__ void bulk_row(const Keys& rk, AesAddr& A,
                                         const Ctr& C, Row r, uint8_t* dst,
                                         int64_t blk, bool edge, StoreMask&& store_mask, uint32_t lds_base, Hash& G,
                                         bool through = kThrough) {
    uint8_t* dp = dst + blk * 16;
    // the keystream block ... while the hash state moves one row along
    G.begin();
    uint32_t s0, s1, s2, s3;
    aes_ctr_lds<kRounds>(rk, A, C, G, lds_base, s0, s1, s2, s3);
    r.arrive();
    const uint32_t x0 = r.x0, x1 = r.x1, x2 = r.x2, x3 = r.x3, tail = r.tail;
    uint32_t o0 = x0 ^ s0, o1 = x1 ^ s1, o2 = x2 ^ s2, o3 = x3 ^ s3;

    auto store_block = [&]() __attribute__((always_inline)) {
        u32x4 o = {o0, o1, o2, o3};
        if (through)
            global_write128_through(dp, o);
        else
            global_write128(dp, o);
    };
    if (!edge) {
        store_block();
    } else if (r.whole) {
        store_block();
    }
    if (__builtin_expect(edge && tail, 0)) {
        write_bytes<kThrough>(dp, tail, o0, o1, o2, o3);
        // bytes past the end count as zero in the hash
        const uint32_t keep = tail % 4 ? (1u << (8 * (tail % 4))) - 1u : 0u;  // in the partial word
        const uint32_t q = tail / 4;
        o0 = q > 0 ? o0 : (q == 0 ? o0 & keep : 0u);
        o1 = q > 1 ? o1 : (q == 1 ? o1 & keep : 0u);
        o2 = q > 2 ? o2 : (q == 2 ? o2 & keep : 0u);
        o3 = q == 3 ? o3 & keep : 0u;
    }

    // the ciphertext is what gets hashed: the output when encrypting, the input when decrypting
    uint32_t c0 = kDecrypt ? x0 : o0, c1 = kDecrypt ? x1 : o1, c2 = kDecrypt ? x2 : o2,
             c3 = kDecrypt ? x3 : o3;
    if (edge && blk < 0) {
        if (blk == -1) store_mask(s0, s1, s2, s3);
        c0 = x0, c1 = x1, c2 = x2, c3 = x3;
    }
    G.absorb(c0, c1, c2, c3);
}

// The same for a row that is no edge row, with the payload's places as scalar bases and the lane's
// offset.
template <bool kDecrypt, int kRounds, bool kThrough, class Hash>
__device__ __forceinline__ void inner_row(const uint32_t* __restrict__ rk, AesAddr& A,
                                          const CtrInner& C, const uint8_t* src, uint8_t* dst,
                                          uint32_t lane16, uint32_t lds_base, Hash& G) {
    const u32x4 x = global_read128(src + lane16);
    G.begin();
    uint32_t s0, s1, s2, s3;
    aes_ctr_lds<kRounds>(rk, A, C, G, lds_base, s0, s1, s2, s3);
    const u32x4 o = {x.x ^ s0, x.y ^ s1, x.z ^ s2, x.w ^ s3};
    if constexpr (kThrough)
        global_write128_through(dst, lane16, o);
    else
        global_write128(dst + lane16, o);
    const u32x4 c = kDecrypt ? x : o;
    G.absorb(c.x, c.y, c.z, c.w);
}

}  // namespace

namespace {

// Brings the bulk kernels' tables into LDS; every one of the kThreads threads calls it, and a
// barrier must follow.  kHash: the operands of the row hash, none, the nibble table or the matrix
// images.
enum class FillHash { kNone, kTable, kMatrix };
// The round tables, 1024 / kThreads neighbouring entries of one table a thread, fetched in one load.
// An entry's copies are kLanes / 4 pieces of 16 bytes; neighbouring threads have different tables
// and start with different pieces, so that a wavefront's store covers all banks evenly.
template <class Te, uint32_t kThreads>
struct TeFill {
    static constexpr uint32_t kEntries = 1024 / kThreads, kPieces = Te::kLanes / 4;
    uint32_t v[kEntries];

    __device__ __forceinline__ void fetch(const KeyTables* __restrict__ kt, uint32_t tid) {
        const uint32_t* from = kt->te[tid & 3] + kEntries * (tid >> 2);
#pragma unroll
        for (uint32_t e = 0; e < kEntries; ++e) v[e] = from[e];
    }
    __device__ __forceinline__ void store(uint32_t* te, uint32_t tid) const {
        const uint32_t t = tid & 3, i = tid >> 2;
        u32x4* te4 = reinterpret_cast<u32x4*>(te);
        const uint32_t table = Te::kPairs ? (t >> 1) * (Te::kPairs / 16) + (t & 1) * kPieces : t * kPieces;
#pragma unroll
        for (uint32_t e = 0; e < kEntries; ++e) {
            const u32x4 q = {v[e], v[e], v[e], v[e]};
#pragma unroll
            for (uint32_t k = 0; k < kPieces; ++k)
                te4[table + (kEntries * i + e) * 16 + ((k + i) & (kPieces - 1))] = q;
        }
    }
};
template <FillHash kHash, uint32_t kThreads>
__device__ __forceinline__ void fill_bulk_lds(BulkLds& lds, const KeyTables* __restrict__ kt,
                                              uint32_t tid) {
    TeFill<TeWide, kThreads> te;
    te.fetch(kt, tid);
    te.store(lds.te, tid);
    if constexpr (kHash != FillHash::kNone) {
        constexpr bool kMatrix = kHash == FillHash::kMatrix;
        const Block* from = kMatrix ? reinterpret_cast<const Block*>(kt->hash_image) : kt->ghash[kRowPower];
        constexpr uint32_t kEntries = (kMatrix ? kHashImages : 1) * kNibbleTableEntries;
        for (uint32_t i = tid; i < kEntries; i += kThreads) lds.gh[i] = from[i];
    }
}

// Keeps the wavefronts of a workgroup abreast where each has its fixed share of the rows.  Of four
// wavefronts on a SIMD the oldest is served first: left alone, the four oldest of sixteen finish
// 320 rows in 957 us and the four youngest in 1625, most of a compute unit's lookups going idle
// towards the end.  So a wavefront that is ahead of the workgroup's average steps back in
// priority: all finish within 1445 to 1468 us (4096 chunks of 320 KiB, 2883 -> 2654 us both ways).
struct Pace {
    uint32_t* rows_done;  // LDS: by the workgroup, zero at the start
    uint32_t mine = 0, all = 0;

    __device__ __forceinline__ void start_row(uint32_t lane) {
        // `all` was fetched a row ago: nothing waits for it
        if (mine * kWavesPerGroup > (uint32_t)__builtin_amdgcn_readfirstlane(all))
            __builtin_amdgcn_s_setprio(0);
        else
            __builtin_amdgcn_s_setprio(2);
        if (lane == 0)
            all = __hip_atomic_fetch_add(rows_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        ++mine;
    }
};
struct NoPace {
    __device__ __forceinline__ void start_row(uint32_t) {}
};

// The blocks [b0, b1) of one chunk, walked by one wavefront in rows of 64 that end at b1: keystream,
// XOR, and the lane's GHASH sum over the rows, sum over rows r of C(r, lane) * (H^64)^(rows after
// r), left in y.  Negative block numbers are those of the AAD and "block -1" (see bulk_row).
// last: b1 is the chunk's end.
// kClasses: pieces may be long enough for CtrClass to pay.
template <bool kDecrypt, int kRounds, bool kThrough, bool kMatrixHash, bool kClasses, class Pace,
          class StoreMask>
__device__ __forceinline__ void walk_unit(const uint32_t* __restrict__ rk, AesAddr& A,
                                          uint32_t lane, uint32_t wave, uint32_t lds_base,
                                          const uint8_t* src, uint8_t* dst, uint64_t len,
                                          int64_t b0, int64_t b1, bool last, const AadBlocks& aad,
                                          const Block& j, Pace& pace, StoreMask&& store_mask, uint32_t y[4],
                                          bool through = kThrough) {
    const uint32_t nrows = (uint32_t)((b1 - b0 + kRowBlocks - 1) / kRowBlocks);
    // a row's counter blocks: inc32^(blk + 1)(J0), the first 96 bits of J0, then its counter field
    // plus blk + 1 modulo 2^32 (SP 800-38D 6.2, 7.1 step 3; ctr1 is that field plus 1, 2 for a
    // 96-bit IV)
    const uint32_t ctr1 = __builtin_amdgcn_readfirstlane(bswap32(j.w[3])) + 1u;
    std::conditional_t<kMatrixHash, GhashRowMatrix, GhashRowMul> G;
    G.start(lds_base, lane);
    int64_t row_blk = b1 - (int64_t)nrows * kRowBlocks;
    for (uint32_t r = 0; r < nrows;) {
        // a segment: kSegmentRows rows, or one more when that is all
        const uint32_t first_ctr = (uint32_t)row_blk + ctr1;
        CtrConsts C = ctr_consts(rk, lane, wave, j.w[0], j.w[1], j.w[2], first_ctr, lds_base);
        const uint32_t left = nrows - r;
        const uint32_t end = left <= kSegmentRows + 1 ? nrows : r + kSegmentRows;
        const uint32_t inner_end = last && end == nrows ? end - 1 : end;
        for (; r < end; ++r, row_blk += kRowBlocks, C.rel += kRowBlocks) {
            // (one group of four rows repays the classes' lookups: 300 adapters both ways 178.3 us
            // without; 175.2, 176.0, 180.2 with from four, eight and sixteen rows on)
            if (kClasses && row_blk >= 0 && r + kRowClasses <= inner_end) {
                CtrClass low[kRowClasses];
#pragma unroll
                for (uint32_t i = 0; i < kRowClasses; ++i) low[i] = ctr_class(rk, A, C, i, lds_base);
                u32x4 q = lds_read128(ctr_q_addr(C, C.rel));
                const uint8_t* s = src + row_blk * 16;
                uint8_t* d = dst + row_blk * 16;
#pragma unroll 1
                do {
                    static_for<0, kRowClasses>([&](auto i) __attribute__((always_inline)) {
                        constexpr uint32_t I = decltype(i)::value;
                        pace.start_row(lane);
                        C.rel += kRowBlocks;
                        const CtrInner c{low[I], q, ctr_q_addr(C, C.rel)};
                        inner_row<kDecrypt, kRounds, kThrough>(rk, A, c, s + 1024 * I, d + 1024 * I,
                                                               lane * 16, lds_base, G);
                    });
                    s += 1024 * kRowClasses, d += 1024 * kRowClasses;
                    r += kRowClasses, row_blk += kRowClasses * kRowBlocks;
                } while (r + kRowClasses <= inner_end);
                if (r == end) break;
            }
            const bool edge = row_blk < 0 || (last && r + 1 == nrows);
            pace.start_row(lane);
            const RowPayload p = load_row(src, len, row_blk + lane, edge, aad);
            bulk_row<kDecrypt, kRounds, kThrough>(rk, A, C, p, dst, row_blk + lane, edge,
                                                  store_mask, lds_base, G, through);
        }
    }
    G.home(y);
}

// (the builtin returns a signed int: without the casts to uint32_t a low half with its top
// bit set would be sign-extended over the high half)
__device__ __forceinline__ uint64_t same_in_all_lanes(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

}  // namespace

// The schedule: wavefront w of the launch starts with unit w; when the launch has a wavefront for
// every unit that is all.  Otherwise the remaining units are handed out through `counter` until
// none is left (the counter serves about one request per 11 ns: a launch whose wavefronts all
// began by asking it would spend its first 50 us queueing, and a batch of many small units would
// be bound by it).  Unit i belongs to the
// chunk c with unit_base[c] <= i < unit_base[c + 1] (unit_base has one entry more than there are
// chunks); coarse_map[i >> kCoarseShift] is a chunk at or before the right one.
// sets[i * 64 + lane] receives lane's GHASH sum over the unit's rows.
// ivs: 96-bit IVs (a chunk's at its `index`), read when j0 is null; otherwise j0[c] is chunk c's J0.
// kMatrixHash: which engine the row hash runs on.
template <bool kDecrypt, int kRounds, bool kMatrixHash>
__global__ __launch_bounds__(kGroupThreads) void bulk_kernel(
    const KeyTables* __restrict__ kt, const ChunkDesc* __restrict__ chunks,
    const uint32_t* __restrict__ unit_base, const uint32_t* __restrict__ coarse_map,
    uint32_t nunits_total, uint32_t unit_power, uint32_t* __restrict__ counter,
    const uint8_t* __restrict__ ivs, const Block* __restrict__ j0, Block* __restrict__ ekj0,
    Block* __restrict__ sets) {
    __shared__ BulkLds lds;
    // lookups use raw LDS addresses relative to this object; its own address (0 as long as it
    // is the kernel's only LDS object) rides in the constant part of every lookup address
    const uint32_t lds_base = lds_offset(&lds);

    const uint32_t tid = threadIdx.x;
    fill_bulk_lds<kMatrixHash ? FillHash::kMatrix : FillHash::kTable, kGroupThreads>(lds, kt, tid);
    __syncthreads();

    const uint32_t lane = tid & 63;
    // the round keys stay in scalar registers for the whole kernel (the last one in vector
    // registers, see AesAddr)
    uint32_t rk[4 * (kRounds + 1)];
#pragma unroll
    for (int i = 0; i < 4 * (kRounds + 1); ++i) rk[i] = kt->rk[i];
    AesAddr A;
    aes_addr_init<TeWide>(A, lane, rk + 4 * kRounds);

    const uint32_t nwaves = gridDim.x * kWavesPerGroup;
    const bool one_each = nunits_total <= nwaves;
    uint32_t item = blockIdx.x * kWavesPerGroup + (tid >> 6);
    for (;;) {
        if (item >= nunits_total) break;  // every wavefront gets here: the counter only grows

        uint32_t chunk = coarse_map[item >> kCoarseShift];
        while (unit_base[chunk + 1] <= item) ++chunk;  // ends: unit_base[nchunks] > item
        const ChunkDesc* __restrict__ cd = chunks + chunk;
        const Block j = chunk_j0(kt, ivs, j0, chunk, cd->index);
        // What describes the unit is the same in every lane, and was fetched from memory just now:
        // moved to scalar registers here, (1) the wait for it comes before the row loop (placed at
        // the first use inside the loop, that wait would make every row wait for the previous
        // row's store as well), (2) which rows are edge rows is decided by a scalar branch, and
        // (3) the payload addresses are a scalar base plus the lane's offset.  (The length and the
        // AAD, which only edge rows look at, stay where they are: scalar registers are short, and
        // one that is spilled costs a vector instruction per use.)
        const uint8_t* src = reinterpret_cast<const uint8_t*>(
            same_in_all_lanes(reinterpret_cast<uint64_t>(cd->src)));
        uint8_t* dst = reinterpret_cast<uint8_t*>(
            same_in_all_lanes(reinterpret_cast<uint64_t>(cd->dst)));
        const uint32_t unit = __builtin_amdgcn_readfirstlane(item - cd->unit_base);
        const uint32_t nunits = __builtin_amdgcn_readfirstlane(cd->nunits);
        const uint32_t first_blocks = __builtin_amdgcn_readfirstlane(cd->first_blocks);
        AadBlocks aad = aad_blocks(cd->aad, cd->aad_len, lds.long_aad + (tid >> 6));
        uint64_t len = cd->len;
        asm volatile("" : "+v"(len), "+v"(aad.bytes), "+v"(aad.len), "+v"(aad.blocks));  // (1) for these
        // unit 0 also takes the blocks before block 0
        const int64_t b1 = (int64_t)first_blocks + ((int64_t)unit << unit_power);
        int64_t b0 = b1 - ((int64_t)1 << unit_power);
        if (unit == 0) {
            b0 = -(int64_t)__builtin_amdgcn_readfirstlane(lead_blocks(cd->aad_len));
            aad.prepare(kt, lane);
        }
        Block* mask_out = ekj0 + chunk;
        uint32_t y[4];
        NoPace pace;
        walk_unit<kDecrypt, kRounds, false, kMatrixHash, false>(
            rk, A, lane, tid >> 6, lds_base, src, dst, len, b0, b1, unit + 1 == nunits, aad, j, pace,
            [&](uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3) __attribute__((always_inline)) {
                *mask_out = Block{{s0, s1, s2, s3}};
            },
            y);
        sets[(uint64_t)item * 64 + lane] = Block{{y[0], y[1], y[2], y[3]}};
        if (one_each) break;
        if (lane == 0)
            item = nwaves + __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        item = __builtin_amdgcn_readfirstlane(item);
    }
}

#define PGCM_INSTANTIATE_BULK(D, R, M)                                                       \
    template __global__ void bulk_kernel<D, R, M>(                                              \
        const KeyTables*, const ChunkDesc*, const uint32_t*, const uint32_t*, uint32_t, uint32_t, \
        uint32_t*, const uint8_t*, const Block*, Block*, Block*)
PGCM_INSTANTIATE_BULK(false, 10, false);
PGCM_INSTANTIATE_BULK(false, 12, false);
PGCM_INSTANTIATE_BULK(false, 14, false);
PGCM_INSTANTIATE_BULK(true, 10, false);
PGCM_INSTANTIATE_BULK(true, 12, false);
PGCM_INSTANTIATE_BULK(true, 14, false);
PGCM_INSTANTIATE_BULK(false, 10, true);
PGCM_INSTANTIATE_BULK(false, 12, true);
PGCM_INSTANTIATE_BULK(false, 14, true);
PGCM_INSTANTIATE_BULK(true, 10, true);
PGCM_INSTANTIATE_BULK(true, 12, true);
PGCM_INSTANTIATE_BULK(true, 14, true);
#undef PGCM_INSTANTIATE_BULK

// ------------------------------------------------------------------------------------------
// Folding partial sets.  Consecutive sets of a chunk lie 2^power blocks apart, so, lane by lane,
//   folded = (..(set_0 * G + set_1) * G + ..) + set_last   with G = H^(2^power).
namespace {

__device__ __forceinline__ void copy_power_table(Block* lds_table, const KeyTables* __restrict__ kt,
                                                 uint32_t power, uint32_t tid, uint32_t nthreads) {
    for (uint32_t i = tid; i < kNibbleTableEntries; i += nthreads) lds_table[i] = kt->ghash[power][i];
}

// table_addr: LDS address of G's nibble table, or 0xFFFFFFFF to read it from global memory.
// Sets are fetched eight at a time so that their load latencies overlap.
__device__ __forceinline__ void fold_sets(const KeyTables* __restrict__ kt,
                                          const Block* __restrict__ sets, uint32_t base,
                                          uint32_t count, uint32_t power, uint32_t lane,
                                          uint32_t table_addr, uint32_t y[4]) {
    const Block* __restrict__ p = sets + (uint64_t)base * 64 + lane;
    auto absorb = [&](const Block& next) {
        if (table_addr != 0xFFFFFFFFu) {
            ghash_mul_lds(table_addr, y);
        } else {
            Block m = gf_mul_table(kt->ghash[power], Block{{y[0], y[1], y[2], y[3]}});
            y[0] = m.w[0], y[1] = m.w[1], y[2] = m.w[2], y[3] = m.w[3];
        }
        y[0] ^= next.w[0], y[1] ^= next.w[1], y[2] ^= next.w[2], y[3] ^= next.w[3];
    };
    const Block first = p[0];
    y[0] = first.w[0], y[1] = first.w[1], y[2] = first.w[2], y[3] = first.w[3];
    uint32_t s = 1;
    for (; s + 8 <= count; s += 8) {
        Block n[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) n[k] = p[(uint64_t)(s + k) * 64];
#pragma unroll
        for (int k = 0; k < 8; ++k) absorb(n[k]);
    }
    for (; s < count; ++s) absorb(p[(uint64_t)s * 64]);
}

// value of lane (l + S) for S = 1, 2, 4, 8 inside each row of 16 lanes, by DPP
template <int S>
__device__ __forceinline__ uint32_t row_shift_down(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + S, 0xF, 0xF, true);
}

// The 64 lane sums of a chunk -> its GHASH state, in every lane.  Lane j's sum still lacks
// H^(64 - j).  Tree: with s = 32, 16, .., 1 lane j takes Y_j * H^s + Y_(j+s) (DPP inside rows of
// 16 lanes, LDS permutes across them); lane 0 ends with sum_j Y_j * H^(63 - j); then one more H.
// When only the last 2^levels lanes hold anything (a chunk of at most 2^levels blocks; levels is
// wave-uniform) the steps with s >= 2^levels are skipped and lane 64 - 2^levels has the sum.
// tree_tables: LDS address of the nibble tables of H^(2^k), k = 0 .. 5, 8 KiB apart.
__device__ __forceinline__ void fold_lanes(uint32_t tree_tables, uint32_t y[4],
                                           uint32_t levels = 6) {
    auto tree_step = [&](uint32_t k, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t n3) {
        ghash_mul_lds(tree_tables + k * kLdsGhBytes, y);
        y[0] ^= n0, y[1] ^= n1, y[2] ^= n2, y[3] ^= n3;
    };
    if (levels > 5)
        tree_step(5, __shfl_down(y[0], 32, 64), __shfl_down(y[1], 32, 64),
                  __shfl_down(y[2], 32, 64), __shfl_down(y[3], 32, 64));
    if (levels > 4)
        tree_step(4, __shfl_down(y[0], 16, 64), __shfl_down(y[1], 16, 64),
                  __shfl_down(y[2], 16, 64), __shfl_down(y[3], 16, 64));
    if (levels > 3)
        tree_step(3, row_shift_down<8>(y[0]), row_shift_down<8>(y[1]), row_shift_down<8>(y[2]),
                  row_shift_down<8>(y[3]));
    if (levels > 2)
        tree_step(2, row_shift_down<4>(y[0]), row_shift_down<4>(y[1]), row_shift_down<4>(y[2]),
                  row_shift_down<4>(y[3]));
    if (levels > 1)
        tree_step(1, row_shift_down<2>(y[0]), row_shift_down<2>(y[1]), row_shift_down<2>(y[2]),
                  row_shift_down<2>(y[3]));
    if (levels > 0)
        tree_step(0, row_shift_down<1>(y[0]), row_shift_down<1>(y[1]), row_shift_down<1>(y[2]),
                  row_shift_down<1>(y[3]));
    ghash_mul_lds(tree_tables, y);
    // only one lane holds the chunk's sum: hand it to every lane
    const uint32_t holder = 64u - (1u << levels);
    for (int k = 0; k < 4; ++k) y[k] = __builtin_amdgcn_readlane(y[k], holder);
}

// The same fold for whole rows (every lane may hold a sum), in groups of four: three
// multiplications deep instead of seven.  With l = 16 b + 4 c + j, H^(64 - l) =
// H^(16 (3 - b)) * H^(4 - j) * H^(4 (3 - c)).  In every step the four rows of sixteen lanes take
// one power each (a wavefront's table lookups collide in the LDS banks unless the lanes that are
// served together, sixteen neighbours, read one and the same table), and the four rows' products
// are then added up, every row keeping the sum:
//   1. row b multiplies its own sums by H^(16 (3 - b)); after the addition every row holds, at
//      place q = 4 c + j, the value V_q of the sixteen columns;
//   2. row r takes element j = r of every quad and multiplies by H^(4 - r); after the addition
//      every row holds W_c in all of quad c;
//   3. row r takes W_r and multiplies by H^(4 (3 - r)); the addition leaves the chunk's GHASH
//      state in every lane.
// Tables, 8 KiB apart from lane_tables: H^1, H^2, H^3, H^4, H^8, H^12, H^16, H^32, H^48.
constexpr uint32_t kLaneTables = 9;

__device__ __forceinline__ void copy_lane_tables(Block (*tables)[kNibbleTableEntries],
                                                 const KeyTables* __restrict__ kt, uint32_t tid,
                                                 uint32_t nthreads) {
    for (uint32_t i = tid; i < kNibbleTableEntries; i += nthreads) {
        tables[0][i] = kt->ghash[0][i];
        tables[1][i] = kt->ghash[1][i];
        tables[2][i] = kt->ghash_lane[0][i];
        tables[3][i] = kt->ghash[2][i];
        tables[4][i] = kt->ghash[3][i];
        tables[5][i] = kt->ghash_lane[1][i];
        tables[6][i] = kt->ghash[4][i];
        tables[7][i] = kt->ghash[5][i];
        tables[8][i] = kt->ghash_lane[2][i];
    }
}

// the XOR of the four rows' values, lane by lane, left in every row: rows 1, 3 change places with
// rows 0, 2 of a copy, then lanes 32..63 with lanes 0..31
__device__ __forceinline__ uint32_t rows_summed(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] ^ a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] ^ b[1];
}

// element kElement of every quad in all four lanes of the quad, in the rows of kRowMask only
template <int kElement, int kRowMask>
__device__ __forceinline__ uint32_t quad_element(uint32_t keep, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)v, kElement * 0x55, kRowMask, 0xF,
                                                 false);
}

__device__ __forceinline__ void fold_lanes_by_four(uint32_t lane_tables, uint32_t y[4],
                                                   uint32_t lane) {
    const uint32_t row = lane >> 4;
    const bool last_row = row == 3;
    {
        uint32_t m[4] = {y[0], y[1], y[2], y[3]};
        ghash_mul_lds(lane_tables + (8 - (last_row ? 2 : row)) * kLdsGhBytes, m);  // H^48, 32, 16
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = rows_summed(last_row ? y[k] : m[k]);
    }
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t t = quad_element<0, 1>(y[k], y[k]);
            t = quad_element<1, 2>(t, y[k]);
            t = quad_element<2, 4>(t, y[k]);
            y[k] = quad_element<3, 8>(t, y[k]);
        }
        ghash_mul_lds(lane_tables + (3 - row) * kLdsGhBytes, y);  // H^4, H^3, H^2, H^1
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = rows_summed(y[k]);
    }
    {
        uint32_t m[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t w0 = __builtin_amdgcn_readlane(y[k], 0), w1 = __builtin_amdgcn_readlane(y[k], 4),
                           w2 = __builtin_amdgcn_readlane(y[k], 8), w3 = __builtin_amdgcn_readlane(y[k], 12);
            y[k] = row == 0 ? w0 : row == 1 ? w1 : row == 2 ? w2 : w3;
            m[k] = y[k];
        }
        ghash_mul_lds(lane_tables + (5 - (last_row ? 2 : row)) * kLdsGhBytes, m);  // H^12, 8, 4
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = rows_summed(last_row ? y[k] : m[k]);
    }
}

// Writes the tag, or compares it with the one received and writes the verdict (SP 800-38D 7.2),
// wiping the output of a rejected chunk.  tag, and when decrypting `received`, are the same in
// every lane.
template <bool kDecrypt>
__device__ __forceinline__ void write_or_compare_tag(const Block& tag, uint8_t* __restrict__ tag_out,
                                                     const Block& received,
                                                     uint8_t* __restrict__ ok, uint8_t* dst,
                                                     uint64_t len, uint32_t lane) {
    if (!kDecrypt) {
        if (lane == 0) global_write_block_any(tag_out, tag);
        return;
    }
    // all 16 bytes, no data-dependent exit
    uint32_t diff = 0;
    for (int k = 0; k < 4; ++k) diff |= received.w[k] ^ tag.w[k];
    diff = __builtin_amdgcn_readfirstlane(diff);
    if (lane == 0) *ok = diff == 0 ? 1 : 0;
    if (diff != 0) {
        // rejected: unauthenticated plaintext must not stay behind; the wavefront zero-fills
        // exactly len bytes
        const uint64_t whole = len / 16;
        uint4* d = reinterpret_cast<uint4*>(dst);
        for (uint64_t b = lane; b < whole; b += 64) d[b] = make_uint4(0, 0, 0, 0);
        for (uint64_t b = whole * 16 + lane; b < len; b += 64) dst[b] = 0;
    }
}

// From the GHASH state over A and C (the same in every lane) to the end of the invocation:
// length block, one more H, mask with E_K(J0) (SP 800-38D 7.1 steps 5-6), tag or verdict.
// h_table: LDS address of the nibble table of H.
template <bool kDecrypt>
__device__ __forceinline__ void finish_chunk(uint32_t h_table, uint32_t y[4],
                                             const uint32_t mask[4], const ChunkDesc& cd,
                                             uint8_t* __restrict__ tags, uint8_t* __restrict__ ok,
                                             uint32_t lane) {
    uint8_t* const tag_at = tags + (uint64_t)cd.index * 16;
    Block received{{0, 0, 0, 0}};
    if (kDecrypt) received = global_read_block_any(tag_at);
    // [8 |A|]_64 || [8 |C|]_64, big endian
    const uint64_t abits = (uint64_t)cd.aad_len * 8, cbits = cd.len * 8;
    y[0] ^= bswap32((uint32_t)(abits >> 32));
    y[1] ^= bswap32((uint32_t)abits);
    y[2] ^= bswap32((uint32_t)(cbits >> 32));
    y[3] ^= bswap32((uint32_t)cbits);
    ghash_mul_lds(h_table, y);
    const Block t{{y[0] ^ mask[0], y[1] ^ mask[1], y[2] ^ mask[2], y[3] ^ mask[3]}};
    write_or_compare_tag<kDecrypt>(t, tag_at, received, ok + cd.index, cd.dst, cd.len, lane);
}

}  // namespace

// One wavefront (= one workgroup) per fold item of one level.
__global__ __launch_bounds__(64) void fold_kernel(const KeyTables* __restrict__ kt,
                                                  const FoldItem* __restrict__ items,
                                                  uint32_t power, Block* __restrict__ sets) {
    __shared__ Block table[kNibbleTableEntries];
    const uint32_t lane = threadIdx.x;
    const FoldItem it = items[blockIdx.x];
    copy_power_table(table, kt, power, lane, 64);
    __syncthreads();
    uint32_t y[4];
    fold_sets(kt, sets, it.in_base, it.in_count, power, lane, lds_offset(table), y);
    sets[(uint64_t)it.out_slot * 64 + lane] = Block{{y[0], y[1], y[2], y[3]}};
}

// The same fold as a tree, for batches with few fold items, where the time of one item counts and
// not the number of items the chip gets through: one workgroup of sixteen wavefronts per item.
// The item's sets, counted back from its last, are the leaves; wavefront w first folds leaves
// 2w and 2w + 1 (missing leaves at the front count as zero, which changes nothing), then four
// rounds through LDS halve the number of partial results, round j with H^(2^(power + j)): five
// multiplications deep instead of thirty-one.
__global__ __launch_bounds__(kFoldTreeWaves * 64) void fold_tree_kernel(
    const KeyTables* __restrict__ kt, const FoldItem* __restrict__ items, uint32_t power,
    Block* __restrict__ sets) {
    constexpr uint32_t kLevels = kFanPower;  // 2^5 leaves
    static_assert(kFoldTreeWaves * 2 == kFan, "two leaves per wavefront");
    __shared__ Block tables[kLevels][kNibbleTableEntries];
    __shared__ Block partial[kFoldTreeWaves][64];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const FoldItem it = items[blockIdx.x];
    for (uint32_t j = 0; j < kLevels; ++j) copy_power_table(tables[j], kt, power + j, tid, blockDim.x);

    // leaves 2w and 2w + 1 of 32, the item's sets being leaves 32 - in_count .. 31
    const uint32_t pad = kFan - it.in_count;
    const Block* __restrict__ in = sets + (uint64_t)it.in_base * 64 + lane;
    uint32_t y[4] = {0, 0, 0, 0};
    Block second{{0, 0, 0, 0}};
    if (2 * wave >= pad) {
        const Block first = in[(uint64_t)(2 * wave - pad) * 64];
        y[0] = first.w[0], y[1] = first.w[1], y[2] = first.w[2], y[3] = first.w[3];
    }
    if (2 * wave + 1 >= pad) second = in[(uint64_t)(2 * wave + 1 - pad) * 64];
    __syncthreads();  // tables are in place
    ghash_mul_lds(lds_offset(tables[0]), y);
    y[0] ^= second.w[0], y[1] ^= second.w[1], y[2] ^= second.w[2], y[3] ^= second.w[3];
    // every wavefront passes every barrier; only the shrinking front half has work to do
    for (uint32_t j = 1; j < kLevels; ++j) {
        partial[wave][lane] = Block{{y[0], y[1], y[2], y[3]}};
        __syncthreads();
        if (wave < (kFoldTreeWaves >> j)) {
            const Block a = partial[2 * wave][lane], b = partial[2 * wave + 1][lane];
            y[0] = a.w[0], y[1] = a.w[1], y[2] = a.w[2], y[3] = a.w[3];
            ghash_mul_lds(lds_offset(tables[j]), y);
            y[0] ^= b.w[0], y[1] ^= b.w[1], y[2] ^= b.w[2], y[3] ^= b.w[3];
        }
        __syncthreads();
    }
    if (wave == 0) sets[(uint64_t)it.out_slot * 64 + lane] = Block{{y[0], y[1], y[2], y[3]}};
}

// Per chunk (one wavefront each): fold the remaining sets, fold the 64 lanes, finish the tag.
// A workgroup is sixteen wavefronts; all of them bring the tables in, the first chunks_per_group
// of them then take a chunk each (the host spreads a batch of few chunks over the compute units:
// the wavefronts of one unit share its LDS pipe, and every chunk is a chain of dependent
// multiplications).  Workgroup 0 also clears `counter` for the next batch.
// LDS: the nine nibble tables of the lane tree, and those of the two most common fold distances.
// unit_power: log2 of the blocks per unit the batch was cut into.
constexpr uint32_t kFinalTables = kLaneTables + 2;

template <bool kDecrypt>
__global__ __launch_bounds__(kFinalWaves * 64) void final_kernel(
    const KeyTables* __restrict__ kt, const ChunkDesc* __restrict__ chunks, uint32_t nchunks,
    const uint8_t* __restrict__ ivs, const Block* __restrict__ j0, const Block* __restrict__ ekj0,
    const Block* __restrict__ sets, uint8_t* __restrict__ tags, uint8_t* __restrict__ ok,
    uint32_t unit_power, uint32_t* __restrict__ counter, uint32_t chunks_per_group) {
    __shared__ Block tables[kFinalTables][kNibbleTableEntries];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x == 0 && tid == 0) *counter = 0;
    // tables 0..8: the lane tree's (the first is H's); then the fold distances of chunks with no
    // and with one fold level behind them
    copy_lane_tables(tables, kt, tid, blockDim.x);
    copy_power_table(tables[kLaneTables], kt, unit_power, tid, blockDim.x);
    copy_power_table(tables[kLaneTables + 1], kt, unit_power + kFanPower, tid, blockDim.x);
    __syncthreads();

    if ((tid >> 6) >= chunks_per_group) return;
    const uint32_t i = blockIdx.x * chunks_per_group + (tid >> 6);
    if (i >= nchunks) return;
    const ChunkDesc cd = chunks[i];

    uint32_t y[4] = {0, 0, 0, 0};
    Block mask;
    if (cd.final_count == 0) {
        // no ciphertext, so no unit ran for this chunk: the hash state is what the AAD leaves,
        // and E_K(J0) is still to be computed
        const Block a = aad_hash(kt, cd.aad, cd.aad_len);
        y[0] = a.w[0], y[1] = a.w[1], y[2] = a.w[2], y[3] = a.w[3];
        const Block j = chunk_j0(kt, ivs, j0, i, cd.index);
        uint32_t e[4] = {j.w[0], j.w[1], j.w[2], j.w[3]};
        aes_block_global(kt, e);
        mask = Block{{e[0], e[1], e[2], e[3]}};
    } else {
        uint32_t fold_table = 0xFFFFFFFFu;
        if (cd.final_power == unit_power) fold_table = lds_offset(tables[kLaneTables]);
        if (cd.final_power == unit_power + kFanPower) fold_table = lds_offset(tables[kLaneTables + 1]);
        fold_sets(kt, sets, cd.final_base, cd.final_count, cd.final_power, lane, fold_table, y);
        fold_lanes_by_four(lds_offset(tables[0]), y, lane);
        mask = ekj0[i];
    }
    finish_chunk<kDecrypt>(lds_offset(tables[0]), y, mask.w, cd, tags, ok, lane);
}

template __global__ void final_kernel<false>(const KeyTables*, const ChunkDesc*, uint32_t,
                                             const uint8_t*, const Block*, const Block*,
                                             const Block*, uint8_t*, uint8_t*, uint32_t,
                                             uint32_t*, uint32_t);
template __global__ void final_kernel<true>(const KeyTables*, const ChunkDesc*, uint32_t,
                                            const uint8_t*, const Block*, const Block*,
                                            const Block*, uint8_t*, uint8_t*, uint32_t,
                                            uint32_t*, uint32_t);

// ------------------------------------------------------------------------------------------
// A few chunks in ONE launch (the paper's swaps come a few chunks at a time, section 5.1): here
// the length of the chain of dependent steps counts as much as the work.  Descriptors are kernel
// arguments, or, for more chunks than fit those, one per workgroup in pinned memory.  Every
// wavefront walks one unit, of eight or sixteen rows (batches of up to four go to burst_kernel) or of a
// forced size; unless the unit is of eight, workgroups have as few wavefronts, at least four, as there are
// compute units for (a row takes a lone wavefront 2.6 us, sixteen on one compute unit 4.3 us).  Then
//   1. the workgroup folds its units' sets into one as a tree in LDS (two to four multiplications
//      from nibble tables, which take the round tables' place);
//   2. all its threads form the 64 products of the set's lanes with H^64 .. H^1, bit by bit from
//      the powers themselves (KeyTables::dot), eight to thirty-two bits of a lane each, and add
//      them up: no further tables, and one step where a tree over the lanes takes six;
//   3. one wavefront multiplies the sum by the power of H that takes it to the chunk's end
//      (KeyTables::hop), unless it is there.  The workgroup with "block -1" adds the length block and E_K(J0), so
//      that a chunk's tag is plainly the sum of its workgroups' results;
//   4. a chunk of one workgroup is finished there and then.  Otherwise its workgroups add their
//      results up in memory, by device-scope atomics that count them in at the same time
//      (last_of_chunk), and whoever completes the sum writes the tag or the verdict.  Nobody waits
//      for anybody: every workgroup runs to its end whatever the others do.
// What a step needs from memory is fetched before the row.  Workgroups of fewer than sixteen
// wavefronts have one more, which makes E_K(J0) and prepares the finish meanwhile.
// LDS after the round tables are done with, in tables of 8 KiB: 0..3 H^(2^(p + j)), the tree over the
// workgroup's units (p = unit_power); 4..5 and 6 its sets.
namespace {

// XOR of the sixteen lanes of a row, left in all of them (DPP: pairs, quads, halves, row)
__device__ __forceinline__ uint32_t row_summed(uint32_t v) {
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);   // quad_perm 1 0 3 2
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // row_half_mirror
    v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);  // row_mirror
    return v;
}

// Four words, each XORed over all lanes, left in every one.  Two swaps of lane halves and one of rows
// make one register of the four, a row of lanes for each, so that there is one row to add up.
// kRows: the lanes of a row have the same already.
template <bool kRows = false>
__device__ __forceinline__ void sum_over_lanes(uint32_t (&v)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[1], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v[2], v[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0] ^ a[1], b[0] ^ b[1], false, false);
    uint32_t z = c[0] ^ c[1];  // rows of lanes: words 0, 2, 1, 3
    if constexpr (!kRows) z = row_summed(z);
    v[0] = __builtin_amdgcn_readlane(z, 0);
    v[1] = __builtin_amdgcn_readlane(z, 32);
    v[2] = __builtin_amdgcn_readlane(z, 16);
    v[3] = __builtin_amdgcn_readlane(z, 48);
}

// sum over the slices s of (the eight coefficients of byte[s]) * q[s], by Horner's rule; the byte's
// top bit is its first coefficient
template <int kSlices>
__device__ __forceinline__ GfWords bits_times(uint32_t byte[kSlices], const GfWords q[kSlices]) {
    GfWords acc{{0, 0, 0, 0}};
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        if (bit != 0) gfw_mul_x(acc);
#pragma unroll
        for (int s = 0; s < kSlices; ++s) {
            const uint32_t m = 0u - (byte[s] & 1u);
            byte[s] >>= 1;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc.a[k] = xor_and(acc.a[k], q[s].a[k], m);
        }
    }
    return acc;
}

// times x^32: the word that leaves at the end comes back in at the front
__device__ __forceinline__ void gfw_mul_x32(GfWords& v) {
    const uint32_t over = v.a[3];
    v.a[3] = v.a[2];
    v.a[2] = v.a[1];
    v.a[1] = v.a[0] ^ (over << 31) ^ (over << 30) ^ (over << 25);
    v.a[0] = 0;
    gfw_fold_word(v, over);
}

// steps 2 and 3 of the kernel, per wavefront: this wavefront's share of the 64 products, summed
// over its lanes.  Wavefront w of 16 / kSlices takes bytes kSlices * w .. of every lane's sum.
template <int kSlices>
__device__ __forceinline__ GfWords dot_share(const Block& y, uint32_t wave, const GfWords q[kSlices]) {
    const uint32_t first = kSlices * wave, w = first / 4;
    const uint32_t word = w == 0 ? y.w[0] : w == 1 ? y.w[1] : w == 2 ? y.w[2] : y.w[3];
    uint32_t byte[kSlices];
#pragma unroll
    for (int s = 0; s < kSlices; ++s) byte[s] = word >> (8 * (first % 4 + s));
    GfWords acc = bits_times<kSlices>(byte, q);
    sum_over_lanes(acc.a);
    return acc;
}

// Lane l gets v * x^(8 (l % 16)), to be multiplied by a value that is the same in all lanes, a byte a
// lane.
__device__ __forceinline__ void spread_over_row(GfWords& v, uint32_t lane) {
    GfWords t = v;
    gfw_mul_x8(t);
    if (lane & 1) v = t;
    t = v;
    gfw_mul_x8(t), gfw_mul_x8(t);
    if (lane & 2) v = t;
    t = v;
    gfw_mul_x32(t);
    if (lane & 4) v = t;
    t = v;
    gfw_mul_x32(t), gfw_mul_x32(t);
    if (lane & 8) v = t;
}
__device__ __forceinline__ GfWords times_spread(const GfWords& v, const GfWords& spread, uint32_t lane) {
    const uint32_t w = (lane / 4) % 4;
    const uint32_t word = w == 0 ? v.a[0] : w == 1 ? v.a[1] : w == 2 ? v.a[2] : v.a[3];
    uint32_t byte[1] = {word >> (24 - 8 * (lane % 4))};
    GfWords z = bits_times<1>(byte, &spread);
#pragma unroll
    for (int k = 0; k < 4; ++k) z.a[k] = row_summed(z.a[k]);
    return z;
}

// The GHASH state after `blocks` whole blocks, two at least, from p, by a wavefront, in all lanes.  All but the last
// in rows counted back from the one before it, lane l's block times H^(65 - l); the last one times H, a nibble a lane.
// (6 to 7 us for a row; block after block from the table in memory it takes 0.5 to 0.75 us a block: 20 chunks of 8 KB
// with AAD of 3000 bytes 142 -> 26 us, one of 320 KiB 114 -> 26.  Without AAD they take 6.4 and 7.0, and 300 of
// 400 KB in spans, where others have work meanwhile, 123, with it 140.)
// The powers one at a time: the registers are needed by what is usual.
// A function of its own: in the middle of the span kernels' code it cost every launch of few rows 0.1 to 0.4 us (60
// chunks of up to 8 KB of three keys both ways 32.0 us without, 32.2 so, 31.7 now; three of 0.1 to 2 MB 41.9, 42.6, 42.4).
__device__ __attribute__((noinline)) Block long_hash(const KeyTables* __restrict__ kt, const uint8_t* p,
                                                     uint32_t blocks, uint32_t lane) {
    asm volatile("" : "+v"(lane));  // what is made of it is not to be kept for later
    const uint32_t n = blocks - 1, rows = (n - 1) / kRowBlocks + 1;
    GfWords sum{{0, 0, 0, 0}}, hop{{0, 0, 0, 0}};
#pragma unroll 1
    for (uint32_t r = 0; r < rows; ++r) {
        if (r == 1) {
            hop = kt->row_hop[1];
            spread_over_row(hop, lane);
        }
        if (r != 0) sum = times_spread(sum, hop, lane);
        const uint32_t end = n - (rows - 1 - r) * kRowBlocks;  // of the row
        Block b{{0, 0, 0, 0}};
        if (end + lane >= kRowBlocks) b = global_read_block_any(p + 16 * (uint64_t)(end + lane - kRowBlocks));
        GfWords row{{0, 0, 0, 0}};
#pragma unroll 1
        for (uint32_t t = 0; t < kDotSlices; ++t) {  // in the order they lie in: the words' first bytes, their second, ..
            GfWords q = (&kt->dot[kRowDot][0][0][lane])[t * kRowBlocks];
            uint32_t v = b.w[0], bits = 8;
            // (the power times the bits of the byte, the first coefficient at its top)
            v <<= 24;
#pragma unroll 1
            for (; bits != 0; --bits, v <<= 1) {
                const uint32_t m = (uint32_t)((int32_t)v >> 31);
#pragma unroll
                for (int k = 0; k < 4; ++k) row.a[k] = xor_and(row.a[k], q.a[k], m);
                gfw_mul_x(q);
            }
            const uint32_t rest = b.w[0] >> 8;
            b.w[0] = b.w[1], b.w[1] = b.w[2], b.w[2] = b.w[3], b.w[3] = rest;
        }
        sum_over_lanes(row.a);
#pragma unroll
        for (int k = 0; k < 4; ++k) sum.a[k] ^= row.a[k];
    }
    Block last{{0, 0, 0, 0}};
    if (lane < 32) {
        const uint32_t byte = global_read8(p + 16 * (uint64_t)n + lane / 2);
        last = kt->ghash[0][lane * 16 + ((lane & 1) ? byte & 15 : byte >> 4)];
    }
    sum_over_lanes(last.w);
    const Block y = gfw_to_block(sum);
    block_xor(last, y);
    return last;
}

// The slots' operations, at device scope
struct SlotMemory {
    static __device__ __forceinline__ uint64_t fetch_xor(uint64_t* at, uint64_t v) {
        return __hip_atomic_fetch_xor(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ uint32_t fetch_add(uint32_t* at, uint32_t v) {
        return __hip_atomic_fetch_add(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    template <class T>
    static __device__ __forceinline__ void clear(T* at) {
        __hip_atomic_store(at, (T)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// One trip to memory and back where it was three (the share stored, an arrival counted when it had got
// there, the shares read by the last), or two instead of four: a chunk of 64 KiB in 7.7 us instead of 8.2,
// 320 KiB 8.5 instead of 9.2, 1 MiB 10.5 instead of 11.3, 2 MiB decrypted 14.2 instead of 15.5 (sums in
// sets of 16: 8.5, 8.8, 10.5, 14.2).
//
// The end of workgroup g of the n of a chunk, whose slots begin at `slots`: `tag`, the same in every lane,
// is its share.  The shares are added up a word a lane, and whoever completes a word has it: usually one
// workgroup all four.  True in the workgroup that is to end the chunk, with its tag.  Where different ones
// completed the words, the encrypting ones write theirs each and nothing is left to do, and the
// decrypting ones compare theirs and add up the verdicts.
template <bool kDecrypt>
__device__ __forceinline__ bool last_of_chunk(ArriveSlot* slots, uint32_t g, uint32_t n, Block& tag,
                                              uint8_t* __restrict__ tag_at, const Block& received,
                                              uint32_t lane) {
    uint32_t t0 = tag.w[0], t1 = tag.w[1], t2 = tag.w[2], t3 = tag.w[3];
    asm volatile("" : "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3));  // (chosen from as an array, they go by way of memory)
    uint32_t word = lane == 0 ? t0 : lane == 1 ? t1 : lane == 2 ? t2 : t3;
    bool whole = lane < 4;
    ChunkMember member{g, n};
    if (n > kArriveSet) {
        if (whole) whole = add_in_set<SlotMemory>(slots, g, n, lane, word);
        member = set_of_chunk(g, n);
    }
    if (whole) whole = add_in_chunk<SlotMemory>(slots, member, lane, word);
    const uint32_t mine = (uint32_t)__ballot(whole);
    if (mine == 0) return false;
    if (mine == 0xF) {
#pragma unroll
        for (int k = 0; k < 4; ++k) tag.w[k] = __builtin_amdgcn_readlane(word, k);
        return true;
    }
    if (!kDecrypt) {
        typedef uint32_t any __attribute__((aligned(1)));
        if (whole)
            *reinterpret_cast<__attribute__((address_space(1))) any*>(
                reinterpret_cast<uintptr_t>(tag_at + 4 * lane)) = word;
        return false;
    }
    const uint32_t expected = lane == 0   ? received.w[0]
                              : lane == 1 ? received.w[1]
                              : lane == 2 ? received.w[2]
                                          : received.w[3];
    const bool differs = __ballot(whole && word != expected) != 0;
    uint32_t count = 0;
    if (lane == 0) count = count_verdict<SlotMemory>(slots, (uint32_t)__popc(mine), differs);
    count = __builtin_amdgcn_readfirstlane(count);
    if (!verdict_whole(count)) return false;
    if (lane == 0) clear_verdict<SlotMemory>(slots);
    tag = received;
    if (verdict_differs(count)) tag.w[0] = ~tag.w[0];
    return true;
}

// this lane's share of (the length block) * H, to be summed over the lanes, from H's nibble table in
// memory: lane p < 32 looks up nibble p
__device__ __forceinline__ Block length_block_entry(const Block* __restrict__ h_table,
                                                    uint64_t aad_len, uint64_t len, uint32_t lane) {
    const uint64_t abits = aad_len * 8, cbits = len * 8;
    const uint32_t w = (lane / 8) % 4;
    const uint32_t be = w == 0 ? (uint32_t)(abits >> 32) : w == 1 ? (uint32_t)abits
                        : w == 2 ? (uint32_t)(cbits >> 32) : (uint32_t)cbits;
    const uint32_t nibble = (be >> (28 - 4 * (lane % 8))) & 15;
    return lane < 32 ? h_table[lane * 16 + nibble] : Block{{0, 0, 0, 0}};
}

// the sum over the lanes of y * H^(65 - lane), in all lanes
__device__ __forceinline__ GfWords lanes_summed(const KeyTables* __restrict__ kt, uint32_t lane,
                                                const uint32_t y[4]) {
    GfWords q[kDotSlices];
    // (an instruction's offset reaches four slices: a scalar base for every four, and one offset in a register)
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b) {
        uint64_t base = reinterpret_cast<uint64_t>(kt->dot[kRowDot][b]);
        asm("" : "+s"(base));
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            const u32x4 v = reinterpret_cast<global_u128_cptr>(base)[w * kRowBlocks + lane];
            q[4 * w + b] = GfWords{{v[0], v[1], v[2], v[3]}};
        }
    }
    GfWords acc{{0, 0, 0, 0}};
    uint32_t v[4] = {y[0], y[1], y[2], y[3]};
    // (a loop: unrolled, its masks are made ahead of their use and take the registers of the powers)
#pragma unroll 1
    for (int bit = 0; bit < 8; ++bit) {
        gfw_mul_x(acc);
#pragma unroll
        for (uint32_t t = 0; t < kDotSlices; ++t) {
            const uint32_t m = (uint32_t)((int32_t)(v[t / 4] << (31 - 8 * (t % 4))) >> 31);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc.a[k] = xor_and(acc.a[k], q[t].a[k], m);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] >>= 1;
    }
    sum_over_lanes(acc.a);
    return acc;
}

// J0 (see j0_from_iv) of an IV of more than one block, by a wavefront, in all lanes.  The blocks go into
// rows counted back from the last one, like a chunk's: one round of loads and a sum over the lanes
// for 1 KiB of IV, where hashing it block after block from the table in memory takes 2.1 us a block,
// and that for every piece of a chunk again (300 adapters, 16-byte IVs: 102 us; of 200 bytes
// 174 -> 106, of 1000 499 -> 106; one 320 KiB chunk, 12 us, with 200 bytes 40 -> 16).
__device__ __forceinline__ Block wave_j0_rows(const KeyTables* __restrict__ kt, const uint8_t* iv,
                                              uint32_t iv_len, uint32_t lane) {
    const uint32_t blocks = iv_len / 16 + (iv_len % 16 != 0);
    const uint32_t rows = (blocks - 1) / kRowBlocks + 1;
    GfWords sum{{0, 0, 0, 0}}, hop{{0, 0, 0, 0}};
#pragma unroll 1
    for (uint32_t r = 0; r < rows; ++r) {
        if (r == 1) {
            hop = kt->row_hop[1];
            spread_over_row(hop, lane);
        }
        if (r != 0) sum = times_spread(sum, hop, lane);
        Block b{{0, 0, 0, 0}};
        const uint32_t end = blocks - (rows - 1 - r) * kRowBlocks;  // of the row
        if (end + lane >= kRowBlocks) b = padded_block(iv, iv_len, end + lane - kRowBlocks);
        const GfWords row = lanes_summed(kt, lane, b.w);
#pragma unroll
        for (int k = 0; k < 4; ++k) sum.a[k] ^= row.a[k];
    }
    Block j = gfw_to_block(sum), last = length_block_entry(kt->ghash[0], 0, iv_len, lane);
    sum_over_lanes(last.w);
    block_xor(j, last);
    return j;
}

// J0 (see j0_from_iv) of an IV of at most one block by a wavefront, in all lanes: IV * H^2 + (length
// block) * H, a nibble of the one or the other per lane, in one round of loads instead of two
// products one after the other (16-byte IVs, 240 chunks of three keys: first row after 13.4 us).
// kLong: there may be longer ones.
template <bool kLong>
__device__ __forceinline__ Block wave_j0(const KeyTables* __restrict__ kt, const uint8_t* iv,
                                         uint32_t iv_len, uint32_t lane) {
    if (iv_len == 12) return j0_from_iv(kt, iv, 12);
    if constexpr (kLong)
        if (iv_len > kShortIvBytes) return wave_j0_rows(kt, iv, iv_len, lane);
    const bool of_iv = lane < 32;
    const uint32_t place = lane % 32, at = place / 2;
    uint32_t byte = 0;
    if (of_iv) {
        if (at < iv_len) byte = global_read8(iv + at);
    } else if (at == 15) {
        byte = iv_len * 8;  // bits: at most 128
    }
    const uint32_t nibble = (place & 1) ? byte & 15 : byte >> 4;
    Block z = kt->ghash[of_iv ? 1 : 0][place * 16 + nibble];
    sum_over_lanes(z.w);
    return z;
}

}  // namespace

template <bool kDecrypt, int kRounds>
__global__ __launch_bounds__(kGroupThreads) void swap_kernel(
    const KeyTables* __restrict__ kt, const uint8_t* __restrict__ ivs, uint32_t iv_len,
    SwapMeta meta, ArriveSlot* __restrict__ slots, uint8_t* __restrict__ tags,
    uint8_t* __restrict__ ok, const GroupDesc* __restrict__ staged, const ArgBatch batch) {
    using Te = TeWide;
    __shared__ BulkLds lds;
    __shared__ Block mask_lds;                   // E_K(J0), where a wavefront with units makes it
    __shared__ GfWords shares[kWavesPerGroup];
    const uint32_t lds_base = lds_offset(&lds);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wave_power = meta.wave_power(), nwaves = 1u << wave_power;
    const uint32_t p = meta.unit_power();
    // The wavefront that finishes the workgroup's part: one beyond those with units, or, where a
    // workgroup can have no more, the last of them, which the tree leaves idle.
    const bool beyond = wave_power < 4;
    const bool finisher = wave == (beyond ? nwaves : nwaves - 1);
    const bool worker = wave < nwaves;

    // Everything the workgroup needs from memory is asked for as early as it can be: a launch starts
    // with cold caches, and every further round of dependent loads costs it a microsecond (the
    // arguments that do not come in registers are a load from host memory themselves).
    TeFill<Te, 256> te4;
    TeFill<Te, 512> te2;
    TeFill<Te, 1024> te1;
    if (worker) {
        if (wave_power == 2) te4.fetch(kt, tid);
        else if (wave_power == 3) te2.fetch(kt, tid);
        else te1.fetch(kt, tid);
    }
    const uint32_t key_word = lane < 60 ? kt->rk[lane] : 0u;  // lane i: round key word i

    // this workgroup's chunk: the last one whose first workgroup is not behind it.  Of the chunks of
    // the caller's arrays in order, one or a workgroup each, it is known before any argument is
    // loaded, and so is the place of the IV.
    const bool alone = meta.nchunks() == 1, each = meta.one_group_each();
    const bool iv_known = staged == nullptr && meta.in_order() && (alone || each);
    Block j{{0, 0, 0, 0}};
    if (iv_known)
        j = wave_j0<true>(kt, ivs + (uint64_t)(alone ? 0 : blockIdx.x) * iv_len, iv_len, lane);
    ArgChunk cd;
    uint32_t group_base, ngroups;
    if (staged != nullptr) {
        const GroupDesc d = staged[blockIdx.x];
        cd = d.c, group_base = d.group_base, ngroups = d.ngroups;
    } else {
        uint32_t chunk = 0;
        if (alone) {
            group_base = 0, ngroups = meta.groups();
        } else if (each) {
            chunk = group_base = blockIdx.x, ngroups = 1;
        } else {
            const uint32_t first = lane < meta.nchunks() ? batch.group_base[lane] : ~0u;
            chunk = __builtin_amdgcn_readfirstlane(
                (uint32_t)__popcll(__ballot(first <= blockIdx.x)) - 1u);
            group_base = batch.group_base[chunk];
            ngroups = batch.group_base[chunk + 1] - group_base;
        }
        cd = batch.c[chunk];
    }
    if (!iv_known) j = wave_j0<true>(kt, ivs + (uint64_t)cd.index * iv_len, iv_len, lane);
    const uint32_t g = blockIdx.x - group_base;
    // its units, counted back from the chunk's end; a negative number is a wavefront without one
    const int64_t nblk = (int64_t)((cd.len + 15) / 16);
    const int64_t lead = swap_lead_blocks(cd.aad_len, beyond);
    const int32_t nunits = (int32_t)((nblk + lead + ((int64_t)1 << p) - 1) >> p);
    const int32_t unit =
        worker ? nunits - (int32_t)((ngroups - g) << wave_power) + (int32_t)wave : -1;
    const int64_t b1 = nblk - ((int64_t)(nunits - 1 - unit) << p);
    const int64_t b0 = unit == 0 ? -lead : b1 - ((int64_t)1 << p);
    // is E_K(J0) made in this workgroup?  By the wavefront beyond the others in the chunk's first
    // workgroup, or in "block -1" of the unit that has it
    const int64_t end = nblk - ((int64_t)(ngroups - 1 - g) << (p + wave_power));
    const bool has_mask = beyond ? g == 0
                                 : end >= 0 && end - ((int64_t)1 << (p + wave_power)) < 0;

    u32x4 gh[2];
    if (worker)
#pragma unroll
        for (uint32_t k = 0; k < 2; ++k)
            if (tid + (k << (6 + wave_power)) < kNibbleTableEntries)
                gh[k] = reinterpret_cast<const u32x4*>(kt->ghash[kRowPower])[tid + (k << (6 + wave_power))];
    auto store_tables = [&]() __attribute__((always_inline)) {
        if (!worker) return;
        if (wave_power == 2) te4.store(lds.te, tid);
        else if (wave_power == 3) te2.store(lds.te, tid);
        else te1.store(lds.te, tid);
#pragma unroll
        for (uint32_t k = 0; k < 2; ++k)
            if (tid + (k << (6 + wave_power)) < kNibbleTableEntries)
                reinterpret_cast<u32x4*>(lds.gh)[tid + (k << (6 + wave_power))] = gh[k];
    };

    // tree tables and powers of H: entry k * threads + tid of the 512 * wave_power, slices
    // 16 / nwaves * wave .. of lane's
    u32x4 tree[4];
    GfWords q[4];
    uint8_t* const tag_at = tags + (uint64_t)cd.index * 16;
    Block extra{{0, 0, 0, 0}};     // what the workgroup with E_K(J0) adds to the tag
    GfWords hop{{0, 0, 0, 0}};     // the power of H to the chunk's end, then times x^(8 (lane % 16))
    Block received{{0, 0, 0, 0}};  // the tag to compare with
    auto fetch_ahead = [&]() __attribute__((always_inline)) {
        const u32x4* from = reinterpret_cast<const u32x4*>(kt->ghash[p]);
        const uint32_t per_thread = (8 * wave_power) >> wave_power;  // 4, 3, 2
        const uint32_t slices = kDotSlices >> wave_power;            // 4, 2, 1
        if (worker) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (k < per_thread) tree[k] = from[(k << (6 + wave_power)) + tid];
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s)
                if (s < slices)
                    q[s] = kt->dot[kRowDot][(slices * wave + s) % 4][(slices * wave + s) / 4][lane];
        }
        if (finisher) {
            if (ngroups - 1 != g) hop = kt->hop[p + wave_power - kHopMinPower][ngroups - 1 - g];
            if (has_mask) extra = length_block_entry(kt->ghash[0], cd.aad_len, cd.len, lane);
            if (kDecrypt) received = global_read_block_any(tag_at);
        }
    };

    // by the finisher, from what fetch_ahead brought
    auto prepare_finish = [&]() __attribute__((always_inline)) {
        if (!finisher) return;
        if (has_mask) {
            sum_over_lanes(extra.w);
        }
        if (ngroups - 1 != g) spread_over_row(hop, lane);  // otherwise the part ends with the chunk
    };

    AadBlocks aad = aad_blocks(cd.aad, worker ? cd.aad_len : 0, lds.long_aad + wave);
    auto keep_mask = [&](uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3)
        __attribute__((always_inline)) { mask_lds = Block{{s0, s1, s2, s3}}; };
    uint32_t y[4] = {0, 0, 0, 0};
    const bool at_start = unit == 0 && cd.aad_len != 0;
    if (!worker) {
        // J0 in every lane: its keystream block is the tag's mask
        fetch_ahead();
        prepare_finish();
        __syncthreads();  // the tables are in place
        if (has_mask) {
            uint32_t e[4] = {j.w[0], j.w[1], j.w[2], j.w[3]};
            aes_block_lds<Te>(key_word, meta.rounds(), lane, lds_base, e);
            keep_mask(e[0], e[1], e[2], e[3]);
        }
    } else {
        store_tables();
        __syncthreads();
        if (unit >= 0) {
            if (at_start) aad.prepare(kt, lane);
            uint32_t rk[4 * (kRounds + 1)];
#pragma unroll
            for (int i = 0; i < 4 * (kRounds + 1); ++i) rk[i] = __builtin_amdgcn_readlane(key_word, i);
            AesAddr A;
            aes_addr_init<Te>(A, lane, rk + 4 * kRounds);
            NoPace pace;
            walk_unit<kDecrypt, kRounds, kDecrypt, false, false>(
                rk, A, lane, wave, lds_base, cd.src, cd.dst, cd.len, b0, b1, b1 == nblk, aad, j,
                pace, keep_mask, y, kDecrypt || rows_of_whole_lines(cd.dst, nblk));
        }
        fetch_ahead();
    }
    if (!beyond) prepare_finish();
    __syncthreads();  // the round tables are done with: their LDS now takes the tree's

    Block(*tables)[kNibbleTableEntries] = reinterpret_cast<Block(*)[kNibbleTableEntries]>(&lds);
    Block(*sets[2])[64] = {reinterpret_cast<Block(*)[64]>(tables[4]),
                           reinterpret_cast<Block(*)[64]>(tables[6])};
    const uint32_t here = (uint32_t)nunits >= (ngroups - g) << wave_power
                              ? nwaves : (uint32_t)nunits - ((ngroups - g - 1) << wave_power);
    uint32_t levels = 0;
    while ((1u << levels) < here) ++levels;
    if (worker) {
        u32x4* to = reinterpret_cast<u32x4*>(tables);
        const uint32_t per_thread = (8 * wave_power) >> wave_power;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (k < per_thread) to[(k << (6 + wave_power)) + tid] = tree[k];
        sets[0][wave][lane] = Block{{y[0], y[1], y[2], y[3]}};
    }
    __syncthreads();

    // 1. every wavefront passes every barrier; only the shrinking front half has work to do.  The
    // units at hand are the last of the workgroup's leaves: the tree goes as far up as they reach.
    for (uint32_t level = 0; level < levels; ++level) {
        if (wave < (nwaves >> (level + 1))) {
            const Block a = sets[level & 1][2 * wave][lane], b = sets[level & 1][2 * wave + 1][lane];
            y[0] = a.w[0], y[1] = a.w[1], y[2] = a.w[2], y[3] = a.w[3];
            ghash_mul_lds(lds_offset(tables[level]), y);
            sets[1 - (level & 1)][wave][lane] =
                Block{{y[0] ^ b.w[0], y[1] ^ b.w[1], y[2] ^ b.w[2], y[3] ^ b.w[3]}};
        }
        __syncthreads();
    }
    // 2.
    if (worker) {
        const Block set = sets[levels & 1][(nwaves >> levels) - 1][lane];
        const GfWords share = wave_power == 2   ? dot_share<4>(set, wave, q)
                              : wave_power == 3 ? dot_share<2>(set, wave, q)
                                                : dot_share<1>(set, wave, q);
        if (lane == 0) shares[wave] = share;
    }
    // When decrypting, the wavefront that finishes the chunk may have to wipe plaintext that
    // others (on other XCDs) wrote: their stores go through to memory, and must be there before
    // the arrival is counted.
    if (kDecrypt) wait_for_own_global_accesses();
    __syncthreads();
    if (!finisher) return;
    // 3.
    GfWords sum{{0, 0, 0, 0}};
    if (lane < nwaves) sum = shares[lane];
#pragma unroll
    for (int k = 0; k < 4; ++k) sum.a[k] = __builtin_amdgcn_readfirstlane(row_summed(sum.a[k]));
    if (ngroups - 1 != g) sum = times_spread(sum, hop, lane);
    Block tag = gfw_to_block(sum);
    if (has_mask) {
        block_xor(tag, extra);
        const Block m = mask_lds;
        block_xor(tag, m);
    }
    // 4.
    if (ngroups > 1 &&
        !last_of_chunk<kDecrypt>(slots + group_base, g, ngroups, tag, tag_at, received, lane))
        return;
    write_or_compare_tag<kDecrypt>(tag, tag_at, received, ok + cd.index, cd.dst, cd.len, lane);
}

#define PGCM_SWAP_SIGNATURE                                                                    \
    (const KeyTables*, const uint8_t*, uint32_t, SwapMeta, ArriveSlot*, uint8_t*, uint8_t*,        \
     const GroupDesc*, ArgBatch)
#define PGCM_INSTANTIATE_SWAP(D)                                    \
    template __global__ void swap_kernel<D, 10> PGCM_SWAP_SIGNATURE; \
    template __global__ void swap_kernel<D, 12> PGCM_SWAP_SIGNATURE; \
    template __global__ void swap_kernel<D, 14> PGCM_SWAP_SIGNATURE
PGCM_INSTANTIATE_SWAP(false);
PGCM_INSTANTIATE_SWAP(true);
#undef PGCM_SWAP_SIGNATURE
#undef PGCM_INSTANTIATE_SWAP

// ------------------------------------------------------------------------------------------
// Short bursts in ONE launch: so few rows that the time of a call is that of its chain of dependent steps.
// A workgroup of 4, 8 or 16 wavefronts makes one or more passes over 64, 128 or 256 blocks.
//   * Of a chunk that begins with one pass, that pass is made in quads: a wavefront takes sixteen blocks, a
//     quad of lanes a block and a lane a column of its state.  A round is four lookups in every lane,
//     whose results go to the lanes beside it, where a lane with a block to itself makes sixteen (64
//     blocks, four wavefronts instead of one: 1.8 -> 1.3 us).  Workgroups of sixteen wavefronts whose last
//     block has more than a pass of payload before its end take rows, a wavefront 64 blocks, a lane a
//     block: more steps, but fewer for each block (128 KiB... 2 MiB: eight rows a compute unit, 12.5 us in
//     quads, 11.9 in rows).  Where such a workgroup makes a single pass there is nothing in it (us, rows
//     and quads: 64 KiB 7.1 and 7.0, 320 KiB 7.6 and 7.7, decrypted 7.6 and 7.5, 1 MiB 7.8 and 7.8, 20 of
//     40 KiB decrypted 7.8 and 7.9), so the number of passes is not asked for.
//   * The round tables are te[0] and, of sixteen wavefronts, te[1], 32 times each: the others are these turned
//     by one byte or two.  A workgroup fills 64 bytes of LDS a clock, so that what a table less saves is as
//     long as the wavefronts are few (one byte: tables in place 1.6 us after the start with both, 1.2
//     with te[0] alone, a call 4.6 -> 4.4; one block of 320 KiB 6.33 -> 6.29).  Sixteen wavefronts keep the
//     vector units busy and pay more for the two turns a round (64 chunks of 4 KiB both ways 12.4 with te[1],
//     12.9 without); they store te[1] behind te[0], as they go on (2 MiB decrypted 8.46 -> 8.27, both in one go
//     8.32).  No lookups collide (te[0..3] sixteen times each, as short transfers once had them, took twice the
//     cycles), and two workgroups fit a compute unit.
//   * What the tables are not needed for is asked for after they are in place: sixteen wavefronts' loads
//     of keys and powers ahead of the last one's of the tables made that wait 1.2 us longer.
//   * Sixteen wavefronts: the first three rows of a pass are multiplied by H^192, H^128, H^64 and added to
//     the fourth, a word of a row a wavefront (eight lookups; 0.4 us, where a tree over the rows, a
//     multiplication of 32 lookups a level, took 1.5 for four rows and 2.3 for eight); then the row's
//     64 columns are multiplied with H^64 .. H^1 bit by bit (KeyTables::dot), a word a wavefront.  Fewer
//     wavefronts: every lane multiplies its own word, by the power that takes its block to the end of the
//     pass, and there is nothing to fold.
//     Without a fold and with fewer wavefronts to bring the tables in a pass is over sooner, so that batches
//     of up to a pass of 64 or 128 blocks a compute unit are made so (one_pass_each: 250 KiB 7.5 -> 6.4 us,
//     320 KiB 7.5 -> 6.9).  Passes of 256 blocks in that way are no gain: 700 KiB 7.6 -> 8.3.
//   * What the end of a workgroup needs besides its sum, the power of H that takes it to the chunk's end with x^8,
//     x^16, .. of it, the length block's product, E_K(J0), is made by a wavefront that has no blocks, while the others
//     are at theirs: one more than they are where at most eight have blocks and a compute unit has one workgroup (one
//     block of 320 KiB 6.42 -> 5.94 us), or the last where rows are taken and it has none, at lower
//     priority than theirs (2 MiB decrypted 8.34 -> 8.24, at the same priority 8.38).
//     Where two share a compute unit there is none more (kWordsShared): with nine wavefronts the second begins when the
//     first has ended, 5.2 us on (300 of up to 8 KiB decrypted 8.9 -> 11.9, 512 of 1900 bytes 8.5 -> 11.9, 257 of them 7.2 ->
//     10.7).  They use 62 to 64 registers and are given 88 (with long IVs 91 and 96), as the compiler sees that LDS leaves a
//     SIMD five wavefronts and has no use for less; of nine, three are on one SIMD, and six would need 528 of its 512.  With
//     five wavefronts instead of four they do fit, and 300 to 512 chunks of 976 bytes gain nothing by it (7.0 and 7.1).
//   * Decrypting, what is hashed is there before it is deciphered.  Of two passes in rows half the wavefronts have
//     no row, and hash those of the others while these decipher: nothing is left to fold and to add up behind the
//     cipher (2 MiB 8.35 -> 7.8 us; eight layers of 2 MiB through the pipe and its receiver 136.0 -> 131.3).  They wait for each other by counters in LDS, as a
//     barrier would hold the cipher up.  Neither half goes first: with the cipher ahead the hash ends 1.2 us behind it,
//     with the hash ahead the cipher ends 1.0 us later.  (Each row from the powers alone, with no tables and nobody to
//     wait for, is three times the instructions: 8.12.)  Of one pass there is nothing in it, 1 MiB 7.06 and 7.11, and
//     beside other shapes' code it costs them 0.1 us, so that two passes have a kernel of their own.
//   * Elsewhere E_K(J0) is the keystream of "block -1" where there is a lane for it, otherwise a second block
//     in every quad of one wavefront, its steps between the first one's.
// A pass's sum is taken to the chunk's end with one more product (KeyTables::row_hop; past 4 MiB, one
// with far_hop as well), four passes at once.  Results of several workgroups are added up as in the kernel for units, see there.
// Against that kernel, with units of a row and the round tables 64 or 128 KiB, per call back to back:
// 1 byte encrypted 6.1 -> 5.2 us; 64 chunks of 4 KiB both ways 16.4 -> 13.8; 300 of 1 byte to 8 KiB, 70 %
// of them ragged, decrypted 14.5 -> 12.5; one of 320 KiB encrypted 12.5 -> 11.4; one of 2 MiB decrypted
// 13.7 -> 12.9; 512 of 8 KiB 25.8 -> 19.8.  With what came later (an event less, shares added up by
// atomics, any number of passes): 1 byte 5.2, 320 KiB 8.2, 2 MiB 10.1, 100 chunks of 20 KB 13.3 (were 15.4).
namespace {

struct QuadTables {
    uint32_t te[256 * 64];  // 256 bytes a value: te[0] 32 times, te[1] 32 times or nothing
    u32x4 keys[4][4];       // KeyTables::column_keys
    Block long_aad[kWavesPerGroup];
    GfWords shares[kFoldPasses][kWavesPerGroup];
    Block mask;  // E_K(J0)
};
typedef Block FoldTables[3][kNibbleTableEntries];  // nibble tables of H^64, H^128, H^192
template <BurstKind kKind>
struct QuadLds : QuadTables {};
template <>
struct QuadLds<BurstKind::kFold> : QuadTables {
    FoldTables fold;
    Block rows[kFoldPasses][4 * kRowBlocks];  // what a pass's blocks add to the hash
};
template <>
struct QuadLds<BurstKind::kFoldApart> : QuadLds<BurstKind::kFold> {
    uint32_t stored, added[kFoldPasses / 2];  // wavefronts that have got so far
};
template <>
struct QuadLds<BurstKind::kSweep> : QuadLds<BurstKind::kFold> {
    Block sweep[kNibbleTableEntries];  // H^1024's
};
template <>
struct QuadLds<BurstKind::kFoldShared> : QuadTables {  // (its tables take the place of the round tables)
    Block rows[kFoldPasses - 1][4 * kRowBlocks];
};
static_assert(2 * sizeof(QuadLds<BurstKind::kFoldShared>) <= 160 << 10 &&
                  2 * sizeof(QuadLds<BurstKind::kWordsShared>) <= 160 << 10,
              "two workgroups on a compute unit");
// The first round table, by 64 << kWavePower threads: an entry a thread and eight pieces of sixteen bytes,
// or, of more threads, a half or a quarter of them.  Eight neighbours have all eight pieces between them,
// so that a wavefront's store covers the table's banks evenly.
template <int kWavePower>
struct QuadFill {
    static constexpr uint32_t kShare = kWavePower - 2, kPieces = 8 >> kShare;
    uint32_t v;

    __device__ __forceinline__ void fetch(const KeyTables* __restrict__ kt, uint32_t tid) {
        v = kt->te[0][tid >> kShare];
    }
    // kTable: te[0], or te[1], which is te[0] turned by a byte
    template <int kTable>
    __device__ __forceinline__ void store(uint32_t* te, uint32_t tid) const {
        const uint32_t i = tid >> kShare;
        u32x4* const te4 = reinterpret_cast<u32x4*>(te) + kTable * 8 + i * 16;
        const uint32_t e = kTable == 0 ? v : __builtin_amdgcn_alignbit(v, v, 24);
        const u32x4 q = {e, e, e, e};
#pragma unroll
        for (uint32_t k = 0; k < kPieces; ++k) te4[(tid + (k << kShare)) & 7] = q;
    }
};

// this lane's column of every round key; the last one apart
struct QuadKeys {
    uint32_t k[14], last, rounds;
};

template <int kTurn>
__device__ __forceinline__ uint32_t quad_turned(uint32_t v) {
    constexpr int kPerm = kTurn == 1 ? 0x39 : kTurn == 2 ? 0x4E : 0x93;  // lane c has column c + kTurn
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kPerm, 0xF, 0xF, true);
}
// a lookup address: byte K of v in byte 1, byte 0 that of `lane_bytes`
template <int K>
__device__ __forceinline__ uint32_t quad_addr(uint32_t v, uint32_t lane_bytes) {
    return __builtin_amdgcn_perm(v, lane_bytes, 0x0c0c0000u | (4u + K) << 8);
}
// kTables: te[0] and te[1], or te[0] alone; of a round's lookups that of the lane's own column is the last,
// and all turning is done when it comes.
// x: a column of the counter block in every lane, and of the keystream block on return.  (With every lane
// looking up its own column's bytes, and the results turned instead of the bytes, a round takes eight
// vector instructions and not eleven, but 64 chunks of 4 KiB both ways 14.2 us and not 13.8.)
template <int kTables, int kBlocks>
__device__ __forceinline__ void quad_encrypt(const QuadKeys& keys, uint32_t lane, uint32_t base,
                                             uint32_t (&x)[kBlocks]) {
    const uint32_t lane_bytes = (lane & 31) * 4;
    uint32_t t[kBlocks][4];
    auto lookups = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) {
            const uint32_t a0 = quad_addr<0>(x[i], lane_bytes),
                           a1 = quad_addr<1>(quad_turned<1>(x[i]), lane_bytes),
                           a2 = quad_addr<2>(quad_turned<2>(x[i]), lane_bytes),
                           a3 = quad_addr<3>(quad_turned<3>(x[i]), lane_bytes);
            if constexpr (kTables == 2) {
                t[i][2] = lds_read32(a2 + base);
                t[i][3] = lds_read32(a3 + base + 128);
                t[i][0] = lds_read32(a0 + base);
                t[i][1] = lds_read32(a1 + base + 128);
            } else {
                t[i][3] = lds_read32(a3 + base);
                t[i][1] = lds_read32(a1 + base);
                t[i][2] = lds_read32(a2 + base);
                t[i][0] = lds_read32(a0 + base);
            }
        }
    };
    auto round = [&](uint32_t key) __attribute__((always_inline)) {
        lookups();
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) {
            if constexpr (kTables == 2) {
                const uint32_t turned = t[i][2] ^ t[i][3];
                x[i] = xor3(t[i][0], t[i][1], key) ^ __builtin_amdgcn_alignbit(turned, turned, 16);
                continue;
            }
            const uint32_t odd = t[i][1] ^ __builtin_amdgcn_alignbit(t[i][3], t[i][3], 16);
            x[i] = xor3(__builtin_amdgcn_alignbit(odd, odd, 24) ^ key,
                        __builtin_amdgcn_alignbit(t[i][2], t[i][2], 16), t[i][0]);
        }
    };
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) x[i] ^= keys.k[0];
#pragma unroll
    for (int r = 1; r < 10; ++r) round(keys.k[r]);
    if (keys.rounds > 10) {
        round(keys.k[10]), round(keys.k[11]);
        if (keys.rounds > 12) round(keys.k[12]), round(keys.k[13]);
    }
    lookups();
    // no MixColumns: S(x) is bytes 1 and 2 of te[0]
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
        const uint32_t lo = __builtin_amdgcn_perm(t[i][0], t[i][1], 0x0c0c0205u);
        const uint32_t hi = __builtin_amdgcn_perm(t[i][2], t[i][3], kTables == 2 ? 0x03060c0cu : 0x02060c0cu);
        x[i] = xor3(lo, hi, keys.last);
    }
}

// Where there is a lane for a block: the keys wait in the lanes of a register, fetched with everything
// else a launch starts with, and one kernel serves every round count.  A wavefront being alone or nearly
// alone on its SIMD, every column's lookups go out as soon as their four addresses are formed, and its
// sum is formed while the later columns' are under way.
struct TeHalf {
    static constexpr uint32_t kPairs = 0, kLanes = 32;
    static constexpr uint32_t offset(int t) { return 128u * (t & 1); }
};
// a.byte1 = near.byte[K] ^ far.byte[K + 2], every other byte of a kept
template <int K>
__device__ __forceinline__ void halves_into_addr(uint32_t& a, uint32_t near, uint32_t far) {
    if constexpr (K == 0)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:BYTE_2" : "+v"(a) : "v"(near), "v"(far));
    else if constexpr (K == 1)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:BYTE_3" : "+v"(a) : "v"(near), "v"(far));
    else if constexpr (K == 2)
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:BYTE_0" : "+v"(a) : "v"(near), "v"(far));
    else
        asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_1" : "+v"(a) : "v"(near), "v"(far));
}
struct LaneKeys {
    uint32_t word;    // lane i: round key word i
    uint32_t rounds;
};
struct CtrBlock {
    uint32_t iv0, iv1, iv2, ctr;
};
// in the place of a row hash: the row's blocks
struct GhashNone {
    uint32_t w[4];
    __device__ __forceinline__ void begin() {}
    __device__ __forceinline__ void absorb(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
        w[0] = c0, w[1] = c1, w[2] = c2, w[3] = c3;
    }
};
template <int kRounds>
__device__ __forceinline__ void aes_ctr_lds(const LaneKeys& keys, AesAddr& A, const CtrBlock& C,
                                            GhashNone&, uint32_t base, uint32_t& o0, uint32_t& o1,
                                            uint32_t& o2, uint32_t& o3) {
    static_assert(kRounds == 0, "any round count");
    using Te = TeHalf;
    // a column between rounds is near ^ (far turned by two bytes), its key in `near`: nothing is turned, the
    // bytes meet when the next addresses are formed
    uint32_t near[4], far[4], t[4][4];
    auto look_up = [&](int c) __attribute__((always_inline)) {
        t[c][0] = te_read<Te, 0>(A.a[c][0], base);
        t[c][1] = te_read<Te, 1>(A.a[(c + 1) & 3][1], base);
        t[c][2] = te_read<Te, 2>(A.a[(c + 2) & 3][2], base);
        t[c][3] = te_read<Te, 3>(A.a[(c + 3) & 3][3], base);
        __builtin_amdgcn_sched_barrier(0);
    };
    {
        const uint32_t u[4] = {C.iv0, C.iv1, C.iv2, bswap32(C.ctr)};
        static_for<0, 4>([&](auto col) __attribute__((always_inline)) {
            constexpr int c = decltype(col)::value;
            const uint32_t k = __builtin_amdgcn_readlane(keys.word, c);
            key_xor_into_addr<0, 0>(A.a[c][0], k, u[c]);
            key_xor_into_addr<1, 1>(A.a[c][1], k, u[c]);
            key_xor_into_addr<2, 2>(A.a[c][2], k, u[c]);
            key_xor_into_addr<3, 3>(A.a[c][3], k, u[c]);
        });
#pragma unroll
        for (int c = 0; c < 4; ++c) look_up(c);
    }
    // the sums of round r, and the lookups of the next
    auto round = [&](uint32_t r) __attribute__((always_inline)) {
        uint32_t k[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) k[c] = __builtin_amdgcn_readlane(keys.word, 4 * r + c);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            near[c] = xor3(t[c][0], t[c][1], k[c]);
            far[c] = t[c][2] ^ t[c][3];
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<0, 4>([&](auto col) __attribute__((always_inline)) {
            constexpr int c = decltype(col)::value;
            halves_into_addr<0>(A.a[c][0], near[c], far[c]);
            halves_into_addr<1>(A.a[(c + 1) & 3][1], near[(c + 1) & 3], far[(c + 1) & 3]);
            halves_into_addr<2>(A.a[(c + 2) & 3][2], near[(c + 2) & 3], far[(c + 2) & 3]);
            halves_into_addr<3>(A.a[(c + 3) & 3][3], near[(c + 3) & 3], far[(c + 3) & 3]);
            look_up(c);
        });
    };
#pragma unroll
    for (uint32_t r = 1; r < 10; ++r) round(r);
    if (keys.rounds > 10) {
        round(10), round(11);
        if (keys.rounds > 12) round(12), round(13);
    }
    uint32_t u[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t lo = __builtin_amdgcn_perm(t[c][0], t[c][1], 0x0c0c0205u);
        const uint32_t hi = __builtin_amdgcn_perm(t[c][2], t[c][3], 0x03060c0cu);
        u[c] = xor3(lo, hi, __builtin_amdgcn_readlane(keys.word, 4 * keys.rounds + c));
    }
    o0 = u[0], o1 = u[1], o2 = u[2], o3 = u[3];
}

// the n <= 4 bytes of a word at any alignment, put together only when they are used
struct WordPieces {
    uint32_t v4 = 0, v2 = 0, v1 = 0;
    bool three = false;

    __device__ __forceinline__ void read(const uint8_t* p, uint32_t n) {
        if (n == 4) v4 = global_read_any<uint32_t>(p);
        if (n & 2) v2 = global_read_any<uint16_t>(p);
        if (n & 1) v1 = global_read8(p + (n & 2));
        three = n == 3;
    }
    __device__ __forceinline__ uint32_t word() const { return v4 | v2 | (three ? v1 << 16 : v1); }
};
template <bool kThrough>
__device__ __forceinline__ void write_word(uint8_t* p, uint32_t n, uint32_t v) {
    if (n == 4) {
        global_write_piece<kThrough>(p, v);
    } else {
        if (n & 2) global_write_piece<kThrough>(p, (uint16_t)v);
        if (n & 1) global_write_piece<kThrough>(p + (n & 2), (uint8_t)((n & 2) ? v >> 16 : v));
    }
}
// the sum over the lanes of (the four bytes of v, the first of them the lowest) * powers, in all lanes
__device__ __forceinline__ GfWords bytes_dot(uint32_t v, const GfWords (&powers)[4]) {
    GfWords sum{{0, 0, 0, 0}};
    // (a loop: unrolled, its masks are made ahead of their use and take too many registers)
#pragma unroll 1
    for (int bit = 0; bit < 8; ++bit) {
        gfw_mul_x(sum);
#pragma unroll
        for (uint32_t s = 0; s < 4; ++s) {
            const uint32_t m = (uint32_t)((int32_t)(v << (31 - 8 * s)) >> 31);
#pragma unroll
            for (int k = 0; k < 4; ++k) sum.a[k] = xor_and(sum.a[k], powers[s].a[k], m);
        }
        v >>= 1;
    }
    sum_over_lanes(sum.a);
    return sum;
}
// (a word of a block) * C, from the eight nibble positions of that word at LDS address `table`
__device__ __forceinline__ u32x4 word_times(uint32_t table, uint32_t v) {
    const uint32_t f0 = 0xF0u, t = v << 4;
    u32x4 e[8];
    e[0] = lds_read128(table + nibble_offset<0>(v, f0));
    e[1] = lds_read128(table + nibble_offset<0>(t, f0) + 256);
    e[2] = lds_read128(table + nibble_offset<1>(v, f0) + 512);
    e[3] = lds_read128(table + nibble_offset<1>(t, f0) + 768);
    e[4] = lds_read128(table + nibble_offset<2>(v, f0) + 1024);
    e[5] = lds_read128(table + nibble_offset<2>(t, f0) + 1280);
    e[6] = lds_read128(table + nibble_offset<3>(v, f0) + 1536);
    e[7] = lds_read128(table + nibble_offset<3>(t, f0) + 1792);
    u32x4 z = e[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) z ^= e[k];
    return z;
}
// Until n wavefronts of the workgroup, all resident and on their way there, have counted themselves in.
__device__ __forceinline__ void wait_for_count(uint32_t* at, uint32_t n) {
    while ((uint32_t)__builtin_amdgcn_readfirstlane(
               __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < n)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
}
// A row whose blocks come with one load in every lane (of anything, where a lane has no whole block), which is waited for
// when they are used.
struct LateRow : RowPayload {
    u32x4 block;

    __device__ __forceinline__ void arrive() {
        if (whole) x0 = block.x, x1 = block.y, x2 = block.z, x3 = block.w;
    }
};
// ... or that is taken from LDS, where others have stored it.  (A second read may be one of host memory, 2 MiB out of it
// 52.2 -> 55.1 us; in place, nothing is overwritten before it is hashed.)
struct SharedRow : LateRow {
    const Block* at = nullptr;
    uint32_t* stored = nullptr;  // wavefronts that have

    __device__ __forceinline__ void arrive() {
        if (at == nullptr) return LateRow::arrive();
        wait_for_count(stored, kWavesPerGroup / 2);
        const Block b = *at;
        x0 = b.w[0], x1 = b.w[1], x2 = b.w[2], x3 = b.w[3];
    }
};
// how many of the four bytes from `at` on lie before `end`
__device__ __forceinline__ uint32_t word_bytes(uint64_t at, uint64_t end) {
    return at + 4 <= end ? 4u : at < end ? (uint32_t)(end - at) : 0u;
}

}  // namespace

template <bool kDecrypt, bool kLongIv, BurstKind kKind, class Args>
__global__ __launch_bounds__(kKind == BurstKind::kWords         ? kGroupThreads / 2 + 64
                             : kKind == BurstKind::kWordsShared ? kGroupThreads / 2
                                                                : kGroupThreads,
                             kKind == BurstKind::kFoldShared ? 8 : 4) void burst_kernel(
    const KeyTables* __restrict__ kt, const uint8_t* __restrict__ ivs, uint32_t iv_len,
    SwapMeta meta, ArriveSlot* __restrict__ slots, uint8_t* __restrict__ tags,
    uint8_t* __restrict__ ok, const Args args) {
    constexpr bool kOne = std::is_same_v<Args, ArgOne>, kStaged = std::is_same_v<Args, ArgStaged>;
    constexpr bool kMore = kKind == BurstKind::kWords;  // a wavefront more
    constexpr bool kFold = !kMore && kKind != BurstKind::kWordsShared, kSweep = kKind == BurstKind::kSweep;
    constexpr bool kApart = kKind == BurstKind::kFoldApart;
    static_assert(!kApart || kDecrypt, "what is hashed is there");
    constexpr bool kRows = kKind == BurstKind::kFold || kApart || kSweep;  // a compute unit to itself
    __shared__ QuadLds<kKind> lds;
    __shared__ Block long_j0;  // J0, of a long IV
    const uint32_t lds_base = lds_offset(&lds);
    const uint32_t tid = threadIdx.x, lane = tid & 63, column = lane & 3;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wave_power = kFold ? 4 : meta.wave_power(), nwaves = 1u << wave_power;
    const uint32_t pass_power = 4 + wave_power, pass_blocks = 1u << pass_power;
    // In kWords the finisher has no blocks: it makes E_K(J0) and prepares the end while the others are at theirs.
    const bool finisher = wave == (kMore ? nwaves : nwaves - 1);
    const bool has_blocks = !kMore || wave < nwaves;

    // Everything the workgroup needs from memory is asked for as early as it can be: a launch starts
    // with cold caches, and every further round of dependent loads costs it a microsecond.
    QuadFill<2> te2;
    QuadFill<3> te3;
    QuadFill<4> te4;
    if constexpr (kFold) te4.fetch(kt, tid);
    else if (!has_blocks) ;
    else if (wave_power == 3) te3.fetch(kt, tid);
    else te2.fetch(kt, tid);
    u32x4 column_keys{};
    if (tid < 16) column_keys = reinterpret_cast<const u32x4*>(kt->column_keys)[tid];
    const uint32_t key_word = lane < 60 ? kt->rk[lane] : 0u;  // lane i: round key word i

    // this workgroup's chunk (as in swap_kernel)
    const bool each = !kOne && !kStaged && meta.one_group_each();
    const bool iv_known = !kLongIv && (kOne || (meta.in_order() && each));
    Block j{{0, 0, 0, 0}};
    if (kOne && !kLongIv && meta.iv_in_place()) {
        const uint64_t iv = reinterpret_cast<uint64_t>(ivs);
        j = Block{{(uint32_t)iv, (uint32_t)(iv >> 32), iv_len, 0x01000000u}};  // IV || be32(1)
    } else if (iv_known) {
        j = wave_j0<false>(kt, ivs + (uint64_t)(kOne ? 0 : blockIdx.x) * iv_len, iv_len, lane);
    }
    ArgChunk cd;
    uint32_t group_base = 0, ngroups = meta.groups();
    if constexpr (kOne) {
        cd = args.c;
        cd.index = 0;
    } else if constexpr (kStaged) {
        const GroupDesc d = args.groups[blockIdx.x];
        cd = d.c, group_base = d.group_base, ngroups = d.ngroups;
    } else {
        uint32_t chunk = 0;
        if (each) {
            chunk = group_base = blockIdx.x, ngroups = 1;
        } else {
            const uint32_t first = lane < meta.nchunks() ? args.group_base[lane] : ~0u;
            chunk = __builtin_amdgcn_readfirstlane(
                (uint32_t)__popcll(__ballot(first <= blockIdx.x)) - 1u);
            group_base = args.group_base[chunk];
            ngroups = args.group_base[chunk + 1] - group_base;
        }
        cd = args.c[chunk];
    }
    if constexpr (kFold) te4.template store<0>(lds.te, tid);
    else if (!has_blocks) ;
    else if (wave_power == 3) te3.template store<0>(lds.te, tid);
    else te2.template store<0>(lds.te, tid);
    if (tid < 16) lds.keys[tid / 4][tid % 4] = column_keys;
    // What comes next is asked for only now: sixteen wavefronts' loads of it ahead of the last one's of the
    // tables made that wait 1.2 us longer, and so did a descriptor or ragged payload waited for before.
    asm volatile("" ::: "memory");
    if constexpr (kLongIv) {
        // by one wavefront for all, which mostly has no row: all sixteen at it are in each
        // other's way (320 KiB with IVs of 60 bytes 17.7 us, 11.1 now; 20 of 8 KB 18.2, 11.9; 8 of 2 MiB 39.6, 34.5)
        if (wave == (kMore ? nwaves : nwaves - 2)) {
            j = wave_j0<true>(kt, ivs + (uint64_t)cd.index * iv_len, iv_len, lane);
            if (lane == 0) long_j0 = j;
        }
    } else if (!iv_known) {
        j = wave_j0<false>(kt, ivs + (uint64_t)cd.index * iv_len, iv_len, lane);
    }

    // its passes, counted back from the chunk's end: pass q of the workgroup is number `behind` + have
    // - 1 - q from there; the chunk's first workgroup has what is left (burst_groups)
    const uint32_t g = blockIdx.x - group_base;
    const int64_t nblk = (int64_t)((cd.len + 15) / 16);
    const int64_t lead = swap_lead_blocks(cd.aad_len, true);
    const uint32_t in_chunk = (uint32_t)((nblk + lead + pass_blocks - 1) >> pass_power);
    const uint32_t passes = ngroups == 1 ? in_chunk : meta.unit_power();
    const uint32_t behind = (ngroups - 1 - g) * passes;
    const uint32_t have = g == 0 ? in_chunk - behind : passes;
    // More passes than kFoldPasses are made in sweeps of so many, the last of them at the end, and the
    // sweeps' rows moved along and added up: what follows them knows kFoldPasses passes.  A sweep takes
    // 4.5 us (4 MiB 15 us, 6 MB 18.9, 8 MiB decrypted 22, 12 MB 25.9; in units of swap_kernel 21.7 for
    // the first two, 29.3, 30.8, and 30.9 for 16 MB, where four sweeps take as long).
    // A kind of its own has them: in kFold they were 23 more registers and 29 more scalar ones, and a call
    // of any number of passes was 0.1 to 0.3 us longer (2 MiB with AAD decrypted 11.80 -> 11.52, 1 MiB
    // 9.52 -> 9.30, 320 KiB encrypted 8.18 -> 8.06, 100 of 20 KB 13.2 -> 12.9; 8 MiB 20.4 either way).
    const uint32_t sweeps = kSweep ? (have + kFoldPasses - 1) / kFoldPasses : 1;
    const uint32_t folded = sweeps > 1 ? kFoldPasses : have;
    const bool has_mask = g == 0;
    // Behind a chunk's first pass of payload: a row a wavefront, a lane a block, which takes fewer instructions
    // a block (see above)
    const bool by_rows = kRows && nblk - ((int64_t)behind << pass_power) > pass_blocks;
    if constexpr (kFold) te4.template store<1>(lds.te, tid);
    // E_K(J0) is the keystream of "block -1", if that is in a pass of this workgroup (the AAD before it may
    // have one of its own) with payload; otherwise it is made beside the first pass
    const bool mask_apart =
        !kMore && has_mask && (nblk >= (int64_t)(behind + have) << pass_power ||
                     nblk < (int64_t)behind << pass_power ||
                     (!by_rows && have > 1 && nblk <= (int64_t)(behind + have - 1) << pass_power));

    const AadBlocks aad = aad_blocks(cd.aad, cd.aad_len, lds.long_aad + wave);
    // Decrypting, what is hashed is there before it is deciphered, and of two passes in rows half the wavefronts
    // have none to decipher: those hash the rows meanwhile, a row each.  (A first workgroup has one pass, and no rows, or
    // a third to spare, and hashes behind the cipher; all others have the launch's two.)
    const bool apart = kApart && by_rows && folded == kFoldPasses / 2 && aad.blocks <= kAadLaneBlocks;
    const bool hashes = apart && wave >= kWavesPerGroup / 2;
    const uint32_t row_wave = apart ? wave % (kWavesPerGroup / 2) : wave;  // the wavefront's row
    // this lane's block in the pass number m from the end
    auto block_of = [&](uint32_t m) __attribute__((always_inline)) {
        return nblk - ((int64_t)(m + 1) << pass_power) + (int64_t)(16 * wave + (lane >> 2));
    };
    // ... and what it has of it: payload, a word of the AAD, or nothing
    auto load_word = [&](int64_t blk) __attribute__((always_inline)) {
        WordPieces v;
        if (blk >= 0) {
            const uint64_t at = (uint64_t)blk * 16 + 4 * column;
            v.read(cd.src + at, word_bytes(at, cd.len));
        } else if (blk >= -lead) {
            if (aad.blocks <= kAadLaneBlocks) {
                const uint32_t at = (aad.blocks + (uint32_t)(int32_t)blk) * 16 + 4 * column;
                v.read(cd.aad + at, word_bytes(at, cd.aad_len));
            } else {
                v.v4 = lds_read32(aad.stand_in + 4 * column);  // block -1
            }
        }
        return v;
    };
    if (aad.blocks > kAadLaneBlocks) {  // rare
        // by the wavefront that has block -1 alone: sixteen at it are in each other's way (8 chunks of 2 MiB
        // with 3000 bytes 700 us, 48 now)
        bool mine = by_rows && wave == wave_of_lead((uint32_t)nblk, behind, folded);
        for (uint32_t q = 0; !by_rows && q < have; ++q)
            mine |= has_blocks && __ballot(block_of(behind + q) == -1) != 0;
        if (mine && g == 0) {
            AadBlocks a = aad;
            a.prepare(kt, lane);
        }
    }
    int64_t blk = have != 0 && has_blocks ? block_of(behind + have - 1) : -lead - 1;
    WordPieces loaded;
    // Decrypting, the payload may be in host memory and take longer than all else: it is asked for last, ahead of the
    // barrier, and nothing else waits for it.  (Its load stands in no branch: behind one, the compiler waits for all loads
    // where the fold tables are stored, that is for the payload, before the keystream is begun.)  Out of host memory,
    // asked for first and waited for there, and now: 2 MiB 52.5 -> 48.7 us, 4 of 512 KiB 53.5 -> 50.4, 100 of 20 KiB 50.7 ->
    // 44.6, 3 MiB 70.3 -> 68.0, 1 MiB 28.4 -> 27.6; in device memory 2 MiB 7.83 -> 7.78, 4 of 512 KiB 8.43 -> 8.50, 3 MiB
    // 9.88 -> 9.93.  Of those that hash apart, asked for behind the barrier: 7.75 and 8.49, out of host memory 51.3 and
    // 52.4.  Encrypting, and in sweeps, it is asked for first.
    constexpr bool kRowLast = kDecrypt && kRows && !kSweep;
    std::conditional_t<kApart, SharedRow, std::conditional_t<kRowLast, LateRow, RowPayload>> row{};
    bool row_edge = true;
    // this wavefront's row of a sweep, if it has one: of the first sweep's passes some may be missing
    auto has_row = [&](uint32_t sweep) __attribute__((always_inline)) {
        return row_wave < 4 * folded && (sweep > 0 || row_wave / 4 >= sweeps * folded - have);
    };
    auto place_row = [&](uint32_t sweep) __attribute__((always_inline)) {
        const uint32_t m1 = behind + folded - row_wave / 4 + kFoldPasses * (sweeps - 1 - sweep);
        blk = nblk - ((int64_t)m1 << pass_power) + (row_wave & 3) * kRowBlocks + lane;
        const int64_t first = same_in_all_lanes((uint64_t)(blk - lane));
        row_edge = first < 0 || first + kRowBlocks == nblk;
    };
    auto fetch_row = [&](uint32_t sweep) __attribute__((always_inline)) {
        if constexpr (!kRowLast) {
            if (!has_row(sweep)) return;
            place_row(sweep);
            row = load_row(cd.src, cd.len, blk, row_edge, aad);
        }
    };
    // ... as load_row has it, for kRowLast
    auto fetch_row_last = [&]() __attribute__((always_inline)) {
        if constexpr (kRowLast) {
            const uint8_t* at = reinterpret_cast<const uint8_t*>(kt);
            if (by_rows && has_row(0)) {
                place_row(0);
                row.tail = row_edge && blk >= 0 && (uint64_t)blk * 16 + 16 > cd.len ? (uint32_t)(cd.len & 15) : 0;
                row.whole = blk >= 0 && row.tail == 0;
                bool here = true;
                if constexpr (kApart) {
                    if (apart && !hashes) {
                        here = false;
                        row.at = &lds.rows[row_wave / 4][(row_wave & 3) * kRowBlocks + lane];
                        row.stored = &lds.stored;
                    }
                }
                if (here && row.whole) {
                    at = cd.src + blk * 16;
                } else if (here) {
                    const Block b = blk < 0 ? aad.at(blk) : read_bytes(cd.src + blk * 16, row.tail);
                    row.x0 = b.w[0], row.x1 = b.w[1], row.x2 = b.w[2], row.x3 = b.w[3];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            row.block = global_read128(at);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (by_rows) {
        fetch_row(0);
    } else {
        loaded = load_word(blk);
    }
    Block extra{{0, 0, 0, 0}};     // what the workgroup with E_K(J0) adds to the tag
    // the tag to compare with, a word of it in a lane (whole in every lane, with 64 registers, it was put away to
    // scratch memory, waited for before the tables were in place: 512 of 4 to 8 KB decrypted 17.6 us, 16.2 now)
    uint32_t tag_word = 0;
    GfWords hop{{0, 0, 0, 0}};     // in row r of sixteen lanes: the power of H for pass r
    const bool hops = behind + folded > 1;
    uint8_t* const tag_at = tags + (uint64_t)cd.index * 16;
    // ... times one more, if there is a pass so far from the chunk's end
    static_assert(kSwapChunkGroups * kFoldPasses * 4 <= kRowHopEntries, "none, of kFoldPasses a workgroup");
    const bool far = kSweep && (behind + folded - 1) << pass_power >= kRowHopEntries * kRowBlocks;
    if (finisher) {
        if (hops) {
            const uint32_t m = lane >> 4 < folded ? behind + folded - 1 - (lane >> 4) : 0;
            hop = kt->row_hop[((m << pass_power) / kRowBlocks) % kRowHopEntries];
        }
        if (has_mask) extra = length_block_entry(kt->ghash[0], cd.aad_len, cd.len, lane);
        if (kDecrypt) tag_word = global_read_any<uint32_t>(tag_at + 4 * column);
    }
    // a word's four bytes: of the lane's own, or of a column of the pass when its rows are folded
    GfWords powers[4];
    auto fetch_powers = [&]() __attribute__((always_inline)) {
        // Where a quad has a block: its number, by lanes, though its row is the wavefront's.  (The row made by scalar
        // instructions, one after the other ahead of the loads: 64 chunks of 1 KiB 5.24 us instead of 5.19.)
        const uint32_t block = kDotBlocks - pass_blocks + 16 * wave + (lane >> 2);
        const GfWords* const from =
            kFold ? &kt->dot[kRowDot][0][wave & 3][lane]
                  : &kt->dot[0][0][0][0] + ((block / kRowBlocks * kDotSlices + column) * kRowBlocks + block % kRowBlocks);
        if (kFold ? row_wave < 4 * folded : has_blocks)
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s) powers[s] = from[s * 4 * kRowBlocks];
    };
    if (kKind != BurstKind::kFoldShared && !kRows) fetch_powers();
    u32x4 fold[2];  // the latter only of the first half of the threads, or in the other half for sweeps
    auto fetch_fold = [&]() __attribute__((always_inline)) {
        fold[0] = reinterpret_cast<const u32x4*>(kt->ghash[kRowPower])[tid];  // and the next power's
        if (tid < kNibbleTableEntries) fold[1] = reinterpret_cast<const u32x4*>(kt->ghash_rows3)[tid];
        else if (kSweep && sweeps > 1)
            fold[1] = reinterpret_cast<const u32x4*>(kt->ghash[kRowPower + 4])[tid - kNibbleTableEntries];
    };
    if constexpr (kRows) {
        if (!apart) fetch_powers(), fetch_fold();
    }
    u32x4 fold_apart[3];  // an entry of each table
    if constexpr (kApart) {
        if (hashes) {
            const uint32_t i = tid % kNibbleTableEntries;
            fold_apart[0] = reinterpret_cast<const u32x4*>(kt->ghash[kRowPower])[i];
            fold_apart[1] = reinterpret_cast<const u32x4*>(kt->ghash[kRowPower + 1])[i];
            fold_apart[2] = reinterpret_cast<const u32x4*>(kt->ghash_rows3)[i];
            if (row_wave % 4 == 3) lds.rows[2 + row_wave / 4][lane] = Block{{0, 0, 0, 0}};  // the sum of pass q: rows[2 + q]
            if (tid == kGroupThreads / 2) lds.stored = lds.added[0] = lds.added[1] = 0;
        }
    }
    fetch_row_last();
    __syncthreads();  // the tables are in place
    if constexpr (kLongIv) j = long_j0;
    QuadKeys keys;
    keys.rounds = meta.rounds();
    {
        u32x4 k[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) k[i] = lds.keys[column][i];
#pragma unroll
        for (uint32_t r = 0; r < 14; ++r) keys.k[r] = k[r / 4][r % 4];
        keys.last = k[3].w;
    }
    Block(*fold_tables)[kNibbleTableEntries] = nullptr;
    if constexpr (kRows) fold_tables = lds.fold;
    if constexpr (kKind == BurstKind::kFoldShared)
        fold_tables = reinterpret_cast<Block(*)[kNibbleTableEntries]>(lds.te);
    auto store_fold = [&]() __attribute__((always_inline)) {
        reinterpret_cast<u32x4*>(fold_tables)[tid] = fold[0];
        if (tid < kNibbleTableEntries) reinterpret_cast<u32x4*>(fold_tables[2])[tid] = fold[1];
        if constexpr (kSweep)
            if (tid >= kNibbleTableEntries && sweeps > 1)
                reinterpret_cast<u32x4*>(lds.sweep)[tid - kNibbleTableEntries] = fold[1];
    };
    if constexpr (kRows)
        if (!apart) store_fold();

    const uint32_t first_ctr = __builtin_amdgcn_readfirstlane(bswap32(j.w[3])) + 1u;
    const uint32_t iv_word = column == 0 ? j.w[0] : column == 1 ? j.w[1] : j.w[2];
    // What the end needs besides the passes' sums, ahead of them where the finisher has no blocks (see above).
    GfWords far_hop{{0, 0, 0, 0}};
    auto prepare = [&]() __attribute__((always_inline)) {
        if (far) {
            const uint32_t m = lane >> 4 < folded ? behind + folded - 1 - (lane >> 4) : 0;
            far_hop = kt->far_hop[(m << pass_power) / kRowBlocks / kRowHopEntries];
        }
        if (has_mask) {
            sum_over_lanes(extra.w);
        }
        if (hops) spread_over_row(hop, lane);
        if (far) spread_over_row(far_hop, lane);
    };
    const bool ahead = kMore || (by_rows && folded < kFoldPasses);  // (it has none)
    if (finisher && ahead && !apart) {
        if (kMore && has_mask) {
            uint32_t y[1] = {column == 3 ? j.w[3] : iv_word};
            quad_encrypt<1, 1>(keys, lane, lds_base, y);
            if (lane < 4) lds.mask.w[lane] = y[0];
        }
        prepare();
    }
    if constexpr (kRows) {
        if (by_rows) {
            auto keep_mask = [&](uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3)
                __attribute__((always_inline)) {
                    if (!mask_apart) lds.mask = Block{{s0, s1, s2, s3}};
                };
            AesAddr A;
            aes_addr_init<TeHalf>(A, lane);
            if (wave < 4 * folded && !apart) __builtin_amdgcn_s_setprio(2);  // ahead of a finisher without a row
            uint32_t y[4] = {0, 0, 0, 0};
            const bool through = kDecrypt || rows_of_whole_lines(cd.dst, nblk);
            auto make_row = [&](uint32_t sweep) __attribute__((always_inline)) {
                if (!has_row(sweep) || hashes) return;
                GhashNone G;
                const CtrBlock C{j.w[0], j.w[1], j.w[2], (uint32_t)blk + first_ctr};
                bulk_row<kDecrypt, 0, kDecrypt>(LaneKeys{key_word, meta.rounds()}, A, C, row, cd.dst, blk,
                                                row_edge, keep_mask, lds_base, G,
                                                through && (!kSweep || kDecrypt ||
                                                            sweep_through(meta.unit_power(), sweep, sweeps)));
#pragma unroll
                for (int k = 0; k < 4; ++k) y[k] ^= G.w[k];
            };
            if constexpr (kSweep) {
                if (sweeps > 1) __syncthreads();  // lds.sweep is in place
                // (the last sweep apart: in the loop it would wait for its row first)
#pragma unroll 1
                for (uint32_t sweep = 0; sweep + 1 < sweeps; ++sweep) {
                    make_row(sweep);
                    fetch_row(sweep + 1);  // wanted when the keystream is there
                    ghash_mul_lds(lds_offset(lds.sweep), y);
                }
            }
            make_row(sweeps - 1);
            __builtin_amdgcn_s_setprio(0);
            if (wave < 4 * folded && !apart)
                lds.rows[wave / 4][(wave & 3) * kRowBlocks + lane] = Block{{y[0], y[1], y[2], y[3]}};
            if (mask_apart && !apart && wave == (folded < kFoldPasses ? kWavesPerGroup - 1 : 0)) {
                uint32_t y[1] = {j.w[0]};
                y[0] = column == 3 ? j.w[3] : iv_word;
                quad_encrypt<kFold ? 2 : 1, 1>(keys, lane, lds_base, y);
                if (lane < 4) lds.mask.w[lane] = y[0];
            }
        }
    }
    if constexpr (kApart) {
        if (hashes) {
            // (the eight are resident together, each has a row of the two passes' eight, and each counts itself in before
            // it waits: no wait is for long)
            auto counted = [&](uint32_t* at) __attribute__((always_inline)) {
                asm volatile("" ::: "memory");  // (LDS serves a wavefront's accesses in order)
                if (lane == 0) __hip_atomic_fetch_add(at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            const uint32_t i = tid % kNibbleTableEntries, q = row_wave / 4, r = row_wave % 4;
#pragma unroll
            for (int t = 0; t < 3; ++t) reinterpret_cast<u32x4*>(lds.fold[t])[i] = fold_apart[t];
            row.arrive();
            lds.rows[q][r * kRowBlocks + lane] = Block{{row.x0, row.x1, row.x2, row.x3}};
            counted(&lds.stored);  // the wavefronts that decipher wait for it as well
            fetch_powers();
            uint32_t c[4] = {row.x0, row.x1, row.x2, row.x3};
            if (r != 3) {
                wait_for_count(&lds.stored, kWavesPerGroup / 2);
                ghash_mul_lds(lds_offset(lds.fold[2 - r]), c);
            }
            uint64_t* const to = reinterpret_cast<uint64_t*>(&lds.rows[2 + q][lane]);
            __hip_atomic_fetch_xor(to, (uint64_t)c[0] | (uint64_t)c[1] << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_xor(to + 1, (uint64_t)c[2] | (uint64_t)c[3] << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            counted(&lds.added[q]);
            // (the last rows' wavefronts, which have nothing to multiply, have this as well)
            if (finisher) prepare();
            if (mask_apart && wave == kWavesPerGroup / 2 + 3) {
                uint32_t y[1] = {column == 3 ? j.w[3] : iv_word};
                quad_encrypt<2, 1>(keys, lane, lds_base, y);
                if (lane < 4) lds.mask.w[lane] = y[0];
            }
            wait_for_count(&lds.added[q], 4);
            lds.shares[q][r] = bytes_dot(lds.rows[2 + q][lane].w[r], powers);
        }
    }
    for (uint32_t q = 0; !by_rows && has_blocks && (q < have || (q == 0 && mask_apart)); ++q) {
        uint32_t x[2] = {column == 3 ? bswap32((uint32_t)blk + first_ctr) : iv_word,
                         column == 3 ? j.w[3] : iv_word};
        const bool mask_here = q == 0 && mask_apart && wave == 0;
        const bool mine = __ballot(blk >= (!kMore && has_mask && !mask_apart ? -1 : 0)) != 0;
        if (mask_here && mine) {
            quad_encrypt<kFold ? 2 : 1, 2>(keys, lane, lds_base, x);
        } else if (mask_here || mine) {
            uint32_t y[1] = {mine ? x[0] : x[1]};
            quad_encrypt<kFold ? 2 : 1, 1>(keys, lane, lds_base, y);
            x[0] = x[1] = y[0];
        }
        if (mask_here && lane < 4) lds.mask.w[lane] = x[1];
        if (!kMore && has_mask && !mask_apart && blk == -1) lds.mask.w[column] = x[0];
        const uint32_t word = loaded.word();
        uint32_t hashed = word;  // the ciphertext, or the AAD
        if (blk >= 0) {
            const uint64_t at = (uint64_t)blk * 16 + 4 * column;
            const uint32_t n = word_bytes(at, cd.len);
            uint32_t out = word ^ x[0];
            write_word<kDecrypt>(cd.dst + at, n, out);
            // bytes past the end count as zero in the hash
            if (!kDecrypt) hashed = n == 4 ? out : out & ((1u << (8 * n)) - 1u);
        }
        if (q + 1 < have) {
            blk = block_of(behind + have - 2 - q);
            loaded = load_word(blk);
        }
        if (q < have) {
            if constexpr (kFold)
                lds.rows[q][16 * wave + (lane >> 2)].w[column] = hashed;
            else
                lds.shares[q][wave] = bytes_dot(hashed, powers);
        }
    }
    if constexpr (kFold) if (!apart) {
        // the first three rows of every pass, a word a wavefront, times H^192, H^128, H^64, and added to
        // the fourth
        if constexpr (kKind == BurstKind::kFoldShared) {
            fetch_fold();
            asm volatile("" ::: "memory");
            fetch_powers();  // no registers for them before
        }
        __syncthreads();
        if constexpr (kKind == BurstKind::kFoldShared) {
            store_fold();
            __syncthreads();
        }
        for (uint32_t i = wave; i < 12 * folded; i += kWavesPerGroup) {
            const uint32_t q = i / 12, row = i % 12 / 4, w = i % 4;
            const uint32_t v = lds.rows[q][row * kRowBlocks + lane].w[w];
            u32x4 z = word_times(lds_offset(fold_tables[2 - row]) + w * 2048, v);
            uint64_t* const to = reinterpret_cast<uint64_t*>(&lds.rows[q][3 * kRowBlocks + lane]);
            __hip_atomic_fetch_xor(to, (uint64_t)z.x | (uint64_t)z.y << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_xor(to + 1, (uint64_t)z.z | (uint64_t)z.w << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        if (wave < 4 * folded)
            lds.shares[wave / 4][wave % 4] =
                bytes_dot(lds.rows[wave / 4][3 * kRowBlocks + lane].w[wave % 4], powers);
    }
    if (finisher && !ahead) prepare();
    // When decrypting, the wavefront that finishes the chunk may have to wipe plaintext that
    // others (on other XCDs) wrote: their stores go through to memory, and must be there before
    // the arrival is counted.
    if (kDecrypt) wait_for_own_global_accesses();
    __syncthreads();
    if (!finisher) return;

    // a pass in every row of sixteen lanes
    static_assert(kFoldPasses * 16 == 64, "all passes at once");
    GfWords sum{{0, 0, 0, 0}};
    {
        const uint32_t q = lane >> 4, w = lane & 15;
        if (q < folded && w < (kFold ? 4 : nwaves)) sum = lds.shares[q][w];
#pragma unroll
        for (int k = 0; k < 4; ++k) sum.a[k] = row_summed(sum.a[k]);
        if (hops) {
            uint32_t l = lane;
            asm volatile("" : "+v"(l));  // what is made of it is not to be kept from before
            sum = times_spread(sum, hop, l);
            if (far) sum = times_spread(sum, far_hop, l);
        }
        sum_over_lanes<true>(sum.a);
    }
    Block tag = gfw_to_block(sum);
    if (has_mask) {
        block_xor(tag, extra);
        const Block m = lds.mask;
        block_xor(tag, m);
    }
    Block received;
#pragma unroll
    for (int k = 0; k < 4; ++k) received.w[k] = __builtin_amdgcn_readlane(tag_word, k);
    if (ngroups > 1 &&
        !last_of_chunk<kDecrypt>(slots + group_base, g, ngroups, tag, tag_at, received, lane))
        return;
    write_or_compare_tag<kDecrypt>(tag, tag_at, received, ok + cd.index, cd.dst, cd.len, lane);
}

#define PGCM_INSTANTIATE_BURST(K, A)                                                              \
    template __global__ void burst_kernel<false, false, BurstKind::K, A> PGCM_BURST_SIGNATURE(A); \
    template __global__ void burst_kernel<true, false, BurstKind::K, A> PGCM_BURST_SIGNATURE(A);  \
    template __global__ void burst_kernel<false, true, BurstKind::K, A> PGCM_BURST_SIGNATURE(A);  \
    template __global__ void burst_kernel<true, true, BurstKind::K, A> PGCM_BURST_SIGNATURE(A)
#define PGCM_INSTANTIATE_APART(A)                                                                       \
    template __global__ void burst_kernel<true, false, BurstKind::kFoldApart, A> PGCM_BURST_SIGNATURE(A); \
    template __global__ void burst_kernel<true, true, BurstKind::kFoldApart, A> PGCM_BURST_SIGNATURE(A)
#define PGCM_BURST_SIGNATURE(A) \
    (const KeyTables*, const uint8_t*, uint32_t, SwapMeta, ArriveSlot*, uint8_t*, uint8_t*, A)
PGCM_INSTANTIATE_BURST(kWords, ArgOne);
PGCM_INSTANTIATE_BURST(kWords, ArgBatch);
PGCM_INSTANTIATE_BURST(kWords, ArgStaged);
PGCM_INSTANTIATE_BURST(kFold, ArgOne);
PGCM_INSTANTIATE_BURST(kFold, ArgBatch);
PGCM_INSTANTIATE_BURST(kFold, ArgStaged);
PGCM_INSTANTIATE_BURST(kSweep, ArgOne);
PGCM_INSTANTIATE_BURST(kSweep, ArgBatch);
PGCM_INSTANTIATE_BURST(kSweep, ArgStaged);
PGCM_INSTANTIATE_BURST(kFoldShared, ArgBatch);
PGCM_INSTANTIATE_BURST(kFoldShared, ArgStaged);
PGCM_INSTANTIATE_BURST(kWordsShared, ArgBatch);
PGCM_INSTANTIATE_BURST(kWordsShared, ArgStaged);
PGCM_INSTANTIATE_APART(ArgOne);
PGCM_INSTANTIATE_APART(ArgBatch);
PGCM_INSTANTIATE_APART(ArgStaged);
#undef PGCM_BURST_SIGNATURE
#undef PGCM_INSTANTIATE_APART
#undef PGCM_INSTANTIATE_BURST

// ------------------------------------------------------------------------------------------
// Batches of any number of chunks, and of any number of keys, in one launch: every wavefront walks a
// span of rows, and the spans are equally long but for what their pieces cost (pgcm_spans.h).  The
// workgroups read their descriptors from host memory themselves if those are few (kSpanHostBytes);
// otherwise they are uploaded before.  A row takes every wavefront the same time, so a compute unit is
// busy to the end, where units of a fixed size leave most of the chip idle in their last round, and
// keys one after the other all of it between them.  A piece (the part of a chunk in a span) is summed over its lanes at once, as in
// the one-launch kernel but by one wavefront: the 64 products with H^64 .. H^1 bit by bit from
// KeyTables::dot, then one or two more with the power that takes the sum to the chunk's end.  The
// results of a chunk's pieces then only have to be added; the wavefront that finishes the last
// piece does that and writes the tag or the verdict (see the one-launch kernel).
// IVs of more than a block have kernels of their own: with the code that hashes them in the same
// ones, the registers of the row loop come out otherwise, and layers take 0.5 % longer (1728 chunks of
// 2 MiB decrypted, 3717 and 3739 us, four runs of each).
namespace {

struct SpanArgs {
    const SpanPart* parts;  // in memory, of the workgroup
    const uint8_t* ivs;
    uint32_t iv_len;
    ArriveSlot* slots;
    uint8_t *tags, *ok;
};
struct SpanLds {
    BulkLds tables;
    Block mask[kWavesPerGroup];     // E_K(J0), by the wavefront with "block -1"
    // results of parts that several wavefronts have rows of, at the place of the first of them, and
    // how many of those are done
    Block sums[kWavesPerGroup];
    uint32_t arrived[kWavesPerGroup];
    u32x4 packet[(sizeof(SpanGroup) + kSpanLdsParts * sizeof(SpanPart)) / 16];

    __device__ __forceinline__ const SpanGroup* group() const {
        return reinterpret_cast<const SpanGroup*>(packet);
    }
    __device__ __forceinline__ const SpanPart* parts() const {
        return reinterpret_cast<const SpanPart*>(packet + sizeof(SpanGroup) / 16);
    }
};

// A part's descriptor in one register: lane i has its word i.
struct PartWords {
    uint32_t v;
    static constexpr uint32_t kWords = sizeof(SpanPart) / 4;

    __device__ __forceinline__ PartWords(const SpanLds& lds, const SpanPart* parts, uint32_t part,
                                         uint32_t lane) {
        v = 0;
        if (lane >= kWords) return;
        if (part < kSpanLdsParts)
            v = reinterpret_cast<const uint32_t*>(lds.parts() + part)[lane];
        else
            v = reinterpret_cast<const uint32_t*>(parts + part)[lane];
    }
    template <size_t kOffset>
    __device__ __forceinline__ uint32_t word() const {
        return __builtin_amdgcn_readlane(v, kOffset / 4);
    }
    template <size_t kOffset>
    __device__ __forceinline__ uint64_t pair() const {
        return word<kOffset>() | (uint64_t)word<kOffset + 4>() << 32;
    }
};

// rows [row, end) of the batch, of which the workgroup's part number `part` has the first;
// key_word: lane i has round key word i
template <bool kDecrypt, bool kLongIv, int kRounds>
__device__ __forceinline__ void walk_span(const KeyTables* __restrict__ kt, uint32_t key_word,
                                          const SpanArgs& args, uint32_t row, uint32_t end,
                                          uint32_t part, uint32_t lane_id, uint32_t wave,
                                          SpanLds& lds) {
    Pace pace{lds.tables.rows_done};
    const uint32_t lds_base = lds_offset(&lds.tables);
    uint32_t rk[4 * (kRounds + 1)];
#pragma unroll
    for (int i = 0; i < 4 * (kRounds + 1); ++i) rk[i] = __builtin_amdgcn_readlane(key_word, i);
    for (; row < end; ++part) {
        uint32_t lane = lane_id;
        asm volatile("" : "+v"(lane));  // what depends on it is not to take registers between pieces
        AesAddr A;
        aes_addr_init<TeWide>(A, lane, rk + 4 * kRounds);
        const PartWords cd(lds, args.parts, part, lane);
#define PGCM_WORD(f) cd.word<offsetof(SpanPart, f)>()
#define PGCM_PAIR(f) cd.pair<offsetof(SpanPart, f)>()
        Block j = wave_j0<kLongIv>(kt, args.ivs + (uint64_t)PGCM_WORD(index) * args.iv_len,
                                   args.iv_len, lane);
        const uint32_t aad_len = PGCM_WORD(aad_len), first_row = PGCM_WORD(first_row),
                       last_row = first_row + PGCM_WORD(rows);
        const uint32_t stop = last_row < end ? last_row : end;
        const uint32_t behind = last_row - stop;  // rows of the chunk after this piece
        // the power of H that takes the piece to the chunk's end: asked for here, used after the rows
        GfWords hop = kt->row_hop[behind % kRowHopEntries];
        const int64_t nblk = (int64_t)((PGCM_PAIR(len) + 15) / 16);
        const int64_t b1 = nblk - (int64_t)behind * kRowBlocks;
        int64_t b0 = b1 - (int64_t)(stop - row) * kRowBlocks;
        if (row == first_row) b0 = -(int64_t)lead_blocks(aad_len);
        // scalar registers are short: what only edge rows look at is kept in vector registers
        AadBlocks aad = aad_blocks(reinterpret_cast<const uint8_t*>(PGCM_PAIR(aad)), aad_len,
                                   lds.tables.long_aad + wave);
        uint64_t len = PGCM_PAIR(len);
        asm volatile("" : "+v"(len), "+v"(aad.bytes), "+v"(aad.len), "+v"(aad.blocks));
        if (b0 < 0) aad.prepare(kt, lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) j.w[k] = __builtin_amdgcn_readfirstlane(j.w[k]);
        uint32_t y[4];
        walk_unit<kDecrypt, kRounds, kDecrypt, false, true>(
            rk, A, lane, wave, lds_base, reinterpret_cast<const uint8_t*>(PGCM_PAIR(src)),
            reinterpret_cast<uint8_t*>(PGCM_PAIR(dst)), len, b0, b1, behind == 0, aad, j, pace,
            [&](uint32_t s0, uint32_t s1, uint32_t s2, uint32_t s3) __attribute__((always_inline)) {
                lds.mask[wave] = Block{{s0, s1, s2, s3}};
            },
            y);
        row = stop;
        GfWords sum = lanes_summed(kt, lane, y);
        if (behind % kRowHopEntries != 0) {
            spread_over_row(hop, lane);
            sum = times_spread(sum, hop, lane);
        }
        if (behind >= kRowHopEntries) {
            hop = kt->far_hop[behind / kRowHopEntries];
            spread_over_row(hop, lane);
            sum = times_spread(sum, hop, lane);
        }
        Block tag = gfw_to_block(sum);
        if (b0 < 0 && b1 >= 0) {
            // the piece with "block -1": the length block's product and E_K(J0)
            Block extra = length_block_entry(kt->ghash[0], PGCM_WORD(aad_len), PGCM_PAIR(len), lane);
            sum_over_lanes(extra.w);
            block_xor(tag, extra);
            const Block m = lds.mask[wave];
            block_xor(tag, m);
        }
        const uint32_t waves = PGCM_WORD(waves) >> 8, slots = PGCM_WORD(slots);
        uint8_t* const tag_at = args.tags + (uint64_t)PGCM_WORD(index) * 16;
        Block received{{0, 0, 0, 0}};  // asked for here: on its way while the arrival is counted
        if (kDecrypt) {
            received = global_read_block_any(tag_at);
            // the plaintext is in memory before the piece counts as done: whoever finishes the chunk may
            // have to wipe it
            if (waves > 1 || slots > 1) wait_for_own_global_accesses();
        }
        if (waves > 1) {
            // LDS serves a wavefront's accesses in order: the sum is there before the count
            const uint32_t at = PGCM_WORD(waves) & 0xFF;
            const uint32_t word = lane == 0 ? tag.w[0] : lane == 1 ? tag.w[1] : lane == 2 ? tag.w[2] : tag.w[3];
            uint32_t before = 0;
            if (lane < 4)
                __hip_atomic_fetch_xor(&lds.sums[at].w[lane], word, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("" ::: "memory");
            if (lane == 0)
                before = __hip_atomic_fetch_add(&lds.arrived[at], 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
            if (__builtin_amdgcn_readfirstlane(before) + 1 != waves) continue;
            asm volatile("" ::: "memory");
            tag = lds.sums[at];
        }
        if (slots > 1) {
            const uint32_t slot = PGCM_WORD(slot);
            if (!last_of_chunk<kDecrypt>(args.slots + slot, PGCM_WORD(own_slot) - slot, slots, tag, tag_at,
                                         received, lane))
                continue;
        }
        write_or_compare_tag<kDecrypt>(tag, tag_at, received, args.ok + PGCM_WORD(index),
                                       reinterpret_cast<uint8_t*>(PGCM_PAIR(dst)), PGCM_PAIR(len), lane);
#undef PGCM_WORD
#undef PGCM_PAIR
    }
}

}  // namespace

template <bool kDecrypt, bool kLongIv>
__global__ __launch_bounds__(kGroupThreads) void span_kernel(
    const KeyTables* __restrict__ key, const uint8_t* __restrict__ packets,
    const SpanPart* __restrict__ all_parts, uint32_t iv_len, uint32_t mapped,
    const uint8_t* __restrict__ ivs, ArriveSlot* __restrict__ slots, uint8_t* __restrict__ tags,
    uint8_t* __restrict__ ok, const SpanMap map) {
    __shared__ SpanLds lds;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Everything is asked for at once: the tables, if the key is known already, and the descriptors, by
    // the first wavefronts only, as they may come from host memory.
    const uint32_t place = mapped != 0 ? map.place[blockIdx.x] : 0;
    const KeyTables* __restrict__ kt = mapped & kSpanKeysMapped ? map.key[place >> SpanMap::kKeyShift] : key;
    TeFill<TeWide, kGroupThreads> te;
    u32x4 gh{};
    uint32_t key_word = 0;
    auto fetch_tables = [&]() __attribute__((always_inline)) {
        te.fetch(kt, tid);
        // the threads without an entry of the row hash bring what the end needs into the caches: a
        // line each of the powers and of H's table
        const uint32_t t = tid - kNibbleTableEntries;
        const uint8_t* const from =
            tid < kNibbleTableEntries ? reinterpret_cast<const uint8_t*>(&kt->ghash[kRowPower][tid])
            : t < sizeof(kt->dot[kRowDot]) / 128
                ? reinterpret_cast<const uint8_t*>(kt->dot[kRowDot]) + t * 128
                                        : reinterpret_cast<const uint8_t*>(kt->ghash[0]) + t % 64 * 128;
        gh = global_read128(from);
        key_word = lane < 60 ? kt->rk[lane] : lane == 60 ? kt->rounds : 0u;
    };
    if (kt != nullptr) fetch_tables();
    const SpanPart* parts = nullptr;
    if (mapped & kSpanPlaced) {
        const uint32_t from = place % (1u << SpanMap::kLengthShift), n = (place >> SpanMap::kLengthShift) % 64;
        if (tid < (sizeof(SpanGroup) + n * sizeof(SpanPart)) / 16)
            lds.packet[tid] = reinterpret_cast<const u32x4*>(packets + (uint64_t)from * kPacketAlign)[tid];
    } else {
        constexpr uint32_t kGroup16 = sizeof(SpanGroup) / 16, kPart16 = sizeof(SpanPart) / 16;
        const SpanGroup* const gd = reinterpret_cast<const SpanGroup*>(packets) + blockIdx.x;
        parts = all_parts + gd->part;
        const uint32_t n = gd->nparts < kSpanLdsParts ? gd->nparts : kSpanLdsParts;
        if (tid < kGroup16)
            lds.packet[tid] = reinterpret_cast<const u32x4*>(gd)[tid];
        else if (tid < kGroup16 + n * kPart16)
            lds.packet[tid] = reinterpret_cast<const u32x4*>(parts)[tid - kGroup16];
    }
    if (tid == 0) lds.tables.rows_done[0] = 0;
    if (tid < kWavesPerGroup) {
        lds.sums[tid] = Block{{0, 0, 0, 0}};
        lds.arrived[tid] = 0;
    }
    const SpanGroup* const group = lds.group();
    if (kt == nullptr) {
        __syncthreads();
        kt = reinterpret_cast<const KeyTables*>(same_in_all_lanes(reinterpret_cast<uint64_t>(group->kt)));
        fetch_tables();
    }
    te.store(lds.tables.te, tid);
    if (tid < kNibbleTableEntries)
        reinterpret_cast<u32x4*>(lds.tables.gh)[tid] = gh;
    else
        asm volatile("" : : "v"(gh));
    __syncthreads();

    if (wave >= __builtin_amdgcn_readfirstlane(group->waves)) return;
    const uint32_t first_row = __builtin_amdgcn_readfirstlane(group->first_row);
    const uint32_t row = first_row + __builtin_amdgcn_readfirstlane(group->cut[wave]);
    const uint32_t end = first_row + __builtin_amdgcn_readfirstlane(group->cut[wave + 1]);
    // its first part: the last one that does not begin behind `row`
    const uint32_t nparts = __builtin_amdgcn_readfirstlane(group->nparts);
    uint32_t part = 0;
    for (uint32_t i = 1; i < nparts; i += 64) {
        bool begins = false;
        if (i + lane < nparts) {
            const uint32_t first = i + lane < kSpanLdsParts ? lds.parts()[i + lane].first_row
                                                            : parts[i + lane].first_row;
            begins = first <= row;
        }
        const uint32_t more = __builtin_amdgcn_readfirstlane((uint32_t)__popcll(__ballot(begins)));
        part += more;
        if (more < 64) break;
    }
    const SpanArgs args{parts, ivs, iv_len, slots, tags, ok};
    const uint32_t rounds = __builtin_amdgcn_readlane(key_word, 60);
    if (rounds == 14)
        walk_span<kDecrypt, kLongIv, 14>(kt, key_word, args, row, end, part, lane, wave, lds);
    else if (rounds == 12)
        walk_span<kDecrypt, kLongIv, 12>(kt, key_word, args, row, end, part, lane, wave, lds);
    else
        walk_span<kDecrypt, kLongIv, 10>(kt, key_word, args, row, end, part, lane, wave, lds);
}

#define PGCM_INSTANTIATE_SPAN(D, L)                                                               \
    template __global__ void span_kernel<D, L>(const KeyTables*, const uint8_t*, const SpanPart*, \
                                               uint32_t, uint32_t, const uint8_t*, ArriveSlot*,   \
                                               uint8_t*, uint8_t*, SpanMap)
PGCM_INSTANTIATE_SPAN(false, false);
PGCM_INSTANTIATE_SPAN(true, false);
PGCM_INSTANTIATE_SPAN(false, true);
PGCM_INSTANTIATE_SPAN(true, true);
#undef PGCM_INSTANTIATE_SPAN

// ------------------------------------------------------------------------------------------
// Many chunks of one row (of the paper's "other I/O", usually < 8 KB, and the 1-byte NOPs of its
// error handler, sections 4.2 and 5.3; up to kSmallMaxChunks of them go to burst_kernel): ONE kernel
// from the first block to the tag, a wavefront per chunk, descriptors read straight from pinned
// host memory.  LDS: the four round tables once (lookups may collide; there are few) and the nibble
// tables the chunks at hand need.
namespace {

template <int kRounds>
__device__ __forceinline__ void aes_block_lds_plain(const uint32_t* __restrict__ rk,
                                                    const uint32_t (*te)[256], uint32_t s[4]) {
    uint32_t a0 = s[0] ^ rk[0], a1 = s[1] ^ rk[1], a2 = s[2] ^ rk[2], a3 = s[3] ^ rk[3];
#pragma unroll
    for (int r = 1; r < kRounds; ++r) {
        uint32_t t0 = xor3(te[0][byte_of(a0, 0)], te[1][byte_of(a1, 1)], te[2][byte_of(a2, 2)]) ^
                      te[3][byte_of(a3, 3)] ^ rk[4 * r + 0];
        uint32_t t1 = xor3(te[0][byte_of(a1, 0)], te[1][byte_of(a2, 1)], te[2][byte_of(a3, 2)]) ^
                      te[3][byte_of(a0, 3)] ^ rk[4 * r + 1];
        uint32_t t2 = xor3(te[0][byte_of(a2, 0)], te[1][byte_of(a3, 1)], te[2][byte_of(a0, 2)]) ^
                      te[3][byte_of(a1, 3)] ^ rk[4 * r + 2];
        uint32_t t3 = xor3(te[0][byte_of(a3, 0)], te[1][byte_of(a0, 1)], te[2][byte_of(a1, 2)]) ^
                      te[3][byte_of(a2, 3)] ^ rk[4 * r + 3];
        a0 = t0, a1 = t1, a2 = t2, a3 = t3;
    }
    // last round: S(x) is byte 1 of te[0], byte 2 of te[1], byte 0 of te[2] and te[3]
    auto last = [&](uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
        uint32_t lo = __builtin_amdgcn_perm(te[0][byte_of(c0, 0)], te[1][byte_of(c1, 1)], 0x0c0c0205u);
        uint32_t hi = __builtin_amdgcn_perm(te[2][byte_of(c2, 2)], te[3][byte_of(c3, 3)], 0x00040c0cu);
        return lo | hi;
    };
    s[0] = last(a0, a1, a2, a3) ^ rk[4 * kRounds + 0];
    s[1] = last(a1, a2, a3, a0) ^ rk[4 * kRounds + 1];
    s[2] = last(a2, a3, a0, a1) ^ rk[4 * kRounds + 2];
    s[3] = last(a3, a0, a1, a2) ^ rk[4 * kRounds + 3];
}

// One row of a short chunk: block `blk` (may be -1 or lower: idle) in this lane.  Reads and writes
// the payload, returns the lane's keystream block in s and what it contributes to the hash in c
// (the ciphertext block, zero-padded; for block 0 with the AAD state folded in; zero when idle).
template <bool kDecrypt, int kRounds>
__device__ __forceinline__ void small_row(const uint32_t* __restrict__ rk,
                                          const uint32_t (*te)[256], const ChunkDesc& cd,
                                          const Block& j, uint32_t ctr1, int64_t blk,
                                          const Block& aad_y, uint32_t s[4], uint32_t c[4]) {
    const bool active = blk >= 0;
    uint32_t tail = 0;
    if (active && (uint64_t)blk * 16 + 16 > cd.len) tail = (uint32_t)(cd.len & 15);
    const bool whole = active && tail == 0;
    uint32_t x[4] = {0, 0, 0, 0};
    const uint8_t* sp = cd.src + blk * 16;
    uint8_t* dp = cd.dst + blk * 16;
    if (whole) {
        u32x4 v = global_read128(sp);
        x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    }
    if (tail) {
        const Block v = read_bytes(sp, tail);
        for (int w = 0; w < 4; ++w) x[w] = v.w[w];
    }
    s[0] = j.w[0], s[1] = j.w[1], s[2] = j.w[2], s[3] = bswap32((uint32_t)blk + ctr1);
    aes_block_lds_plain<kRounds>(rk, te, s);
    uint32_t o[4] = {x[0] ^ s[0], x[1] ^ s[1], x[2] ^ s[2], x[3] ^ s[3]};
    if (whole) {
        u32x4 v = {o[0], o[1], o[2], o[3]};
        global_write128(dp, v);
    }
    if (tail) {
        write_bytes<false>(dp, tail, o[0], o[1], o[2], o[3]);
        // bytes past the end count as zero in the hash
#pragma unroll
        for (uint32_t b = 1; b < 16; ++b)
            if (b >= tail) o[b / 4] &= ~(0xFFu << (8 * (b % 4)));
    }
    for (int w = 0; w < 4; ++w) c[w] = kDecrypt ? x[w] : o[w];
    if (blk == 0)
        for (int w = 0; w < 4; ++w) c[w] ^= aad_y.w[w];
    if (!active)
        for (int w = 0; w < 4; ++w) c[w] = 0;
}

// levels of the lane tree a chunk of nblk <= 64 blocks in one row needs
__device__ __forceinline__ uint32_t lane_tree_levels(uint32_t nblk) {
    uint32_t levels = 0;
    while ((1u << levels) < nblk) ++levels;
    return levels;
}

// brings the round tables and the nibble tables named in `needed` (bit k: H^(2^k)) into LDS;
// every thread of the workgroup calls it
template <int kTables>
__device__ __forceinline__ void load_small_tables(uint32_t (*te)[256],
                                                  Block (*tables)[kNibbleTableEntries],
                                                  const KeyTables* __restrict__ kt,
                                                  uint32_t needed, uint32_t tid) {
    for (uint32_t t = tid; t < 4 * 256; t += blockDim.x) te[t >> 8][t & 255] = kt->te[t >> 8][t & 255];
    for (uint32_t k = 0; k < (uint32_t)kTables; ++k)
        if (needed & (1u << k)) copy_power_table(tables[k], kt, k, tid, blockDim.x);
}

}  // namespace

// Chunks of at most one row including "block -1" (63 blocks, 1008 bytes: the NOPs and most of the
// small traffic): one wavefront per chunk, several chunks a workgroup.
// ivs: IVs of iv_len bytes each, a chunk's at its `index`; J0 of an IV that is not 96 bits long is
// hashed here.
template <bool kDecrypt, int kRounds>
__global__ __launch_bounds__(kSmallChunksPerGroup * 64) void small_kernel(
    const KeyTables* __restrict__ kt, const ChunkDesc* __restrict__ chunks_host, uint32_t nchunks,
    const uint8_t* __restrict__ ivs, uint32_t iv_len, uint8_t* __restrict__ tags,
    uint8_t* __restrict__ ok) {
    __shared__ uint32_t te[4][256];
    __shared__ Block tables[6][kNibbleTableEntries];  // H^(2^k), k = 0 .. 5
    __shared__ uint32_t tables_needed;                // bit k: some chunk here uses tables[k]
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t i = blockIdx.x * kSmallChunksPerGroup + (tid >> 6);
    const bool have_chunk = i < nchunks;
    ChunkDesc cd{};
    if (have_chunk) cd = chunks_host[i];
    const uint32_t nblk = (uint32_t)((cd.len + 15) / 16);  // <= 63, the host saw to that
    // the chunk fills only the last nblk lanes of its row: the lane tree starts lower down
    const uint32_t levels = lane_tree_levels(nblk);

    // only the tables this workgroup's chunks use are brought into LDS: H always, H^(2^k) for
    // the lane tree's levels (a 1-byte transfer needs H only)
    if (tid == 0) tables_needed = 0;
    __syncthreads();
    if (lane == 0 && have_chunk) atomicOr(&tables_needed, 1u | ((1u << levels) - 1u));
    __syncthreads();
    load_small_tables<6>(te, tables, kt, tables_needed, tid);
    __syncthreads();
    if (!have_chunk) return;
    const uint32_t* __restrict__ rk = kt->rk;

    Block aad_y{{0, 0, 0, 0}};
    if (cd.aad_len != 0) aad_y = aad_hash(kt, cd.aad, cd.aad_len);
    const Block j = j0_from_iv(kt, ivs + (uint64_t)cd.index * iv_len, iv_len);
    const uint32_t ctr1 = bswap32(j.w[3]) + 1u;

    // the row is aligned to the chunk's end; "block -1" (counter block J0) rides along in the
    // lane before block 0, and its keystream is E_K(J0)
    const int64_t blk = (int64_t)nblk - kRowBlocks + lane;
    uint32_t s[4], y[4], mask[4];
    small_row<kDecrypt, kRounds>(rk, te, cd, j, ctr1, blk, aad_y, s, y);
    for (int w = 0; w < 4; ++w) mask[w] = __shfl(s[w], (int)(kRowBlocks - nblk - 1), 64);

    if (nblk == 0) {
        // nothing was hashed yet: the state is what the AAD left
        for (int w = 0; w < 4; ++w) y[w] = aad_y.w[w];
    } else {
        fold_lanes(lds_offset(tables[0]), y, levels);
    }
    finish_chunk<kDecrypt>(lds_offset(tables[0]), y, mask, cd, tags, ok, lane);
}

#define PGCM_INSTANTIATE_SMALL(D, R)                                                      \
    template __global__ void small_kernel<D, R>(const KeyTables*, const ChunkDesc*, uint32_t, \
                                                const uint8_t*, uint32_t, uint8_t*, uint8_t*)
PGCM_INSTANTIATE_SMALL(false, 10);
PGCM_INSTANTIATE_SMALL(false, 12);
PGCM_INSTANTIATE_SMALL(false, 14);
PGCM_INSTANTIATE_SMALL(true, 10);
PGCM_INSTANTIATE_SMALL(true, 12);
PGCM_INSTANTIATE_SMALL(true, 14);
#undef PGCM_INSTANTIATE_SMALL

// Brings a batch's descriptors from pinned host memory into the device workspace.  Done by a
// kernel so that the batch stays on one hardware queue: a DMA copy between kernels costs two
// cross-queue hand-overs.  The n_clear pieces of sixteen bytes from `clear` on are set to zero as well
// (counters of a new workspace: a fill by a kernel, not a memset node, so that the stream's work
// stays of one kind).
__global__ __launch_bounds__(256) void upload_kernel(uint4* __restrict__ dst,
                                                     const uint4* __restrict__ src_host,
                                                     uint32_t n16, uint4* __restrict__ clear,
                                                     uint32_t n_clear) {
    const uint32_t first = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (uint32_t i = first; i < n_clear; i += step) clear[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = first; i < n16; i += step) dst[i] = src_host[i];
}

}  // namespace pgcm
