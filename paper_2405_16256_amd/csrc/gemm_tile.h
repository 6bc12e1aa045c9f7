// Pieces shared by the bf16 matrix-core GEMM kernels: the workgroup -> tile map and operand tiles that are filled
// straight from global memory into LDS (buffer_load ... lds) and read back as MFMA fragments.
#pragma once
#include "common.h"

namespace hh {

// Workgroup -> tile mapping.  Consecutive workgroup ids land on different XCDs
// (8 of them, each with its own L2), so ids are first regrouped per XCD and each
// XCD then walks a compact block of tiles, GROUP_M tile rows at a time.
constexpr int GROUP_M = 8;
struct TileMap {
    int tiles_m, tiles_n;
    Divisor width, last;   // tiles of a whole group of rows; rows of the last, smaller one
    int tiles() const { return tiles_m * tiles_n; }
    // Without a branch, so that the fields are loaded together and not each group of them behind the branch before it.
    __device__ __forceinline__ void tile(int id, int& tm, int& tn) const {
        const int per = (tiles_m * tiles_n) >> 3, there = (id & 7) * per + (id >> 3);
        id = id < per * 8 ? there : id;
        const int within = split_off(id, width);   // id: the group
        const int first_m = id * GROUP_M;
        const bool whole = tiles_m - first_m >= GROUP_M;
        const Divisor rows = {whole ? GROUP_M : last.d, whole ? 1u << 31 : last.mul, whole ? 3 : last.shift};
        tn = within;
        tm = first_m + split_off(tn, rows);
    }
};
inline TileMap tile_map(int M, int N, int bm, int bn) {
    const int tiles_m = (M + bm - 1) / bm, tiles_n = (N + bn - 1) / bn;
    return TileMap{tiles_m, tiles_n, divisor(GROUP_M * tiles_n), divisor(tiles_m % GROUP_M ? tiles_m % GROUP_M : GROUP_M)};
}

// Which of up to four problems a workgroup belongs to, from the first workgroup of the second, third and fourth (INT_MAX: no
// such problem).  The index is hidden from the compiler, which otherwise chooses between the addresses of every single field
// instead of loading the problem's fields from one base, up to 16 words at a time.
struct Firsts { int second, third, fourth; };
__device__ __forceinline__ int own_problem(const Firsts& f) {
    const int b = (int)blockIdx.x;
    auto from = [&](int first) { return (int)((uint32_t)(first - 1 - b) >> 31); };   // b >= first
    int i = from(f.second) + from(f.third) + from(f.fourth);
    asm("" : "+s"(i));
    return i;
}

// The rotary embedding and SwiGLU combine columns far apart: (c, c + period/2) of a head or of a gate|up row.  A GEMM that
// does them on its way out takes its columns from B's rows in another order (any order is free: each lane asks for its own
// row): a 32-column block holds 16 columns of the first half and their 16 partners.  This is the column of C that column c (of
// N) of that order stands for; period 2^shift, or N (shift 31).
__device__ __forceinline__ int pair_column(int c, int period, int shift, int N) {
    if (c >= N) return c;
    const int first = (c >> shift) * period, r = c - first;
    return first + (r >> 5) * 16 + (r & 15) + ((r & 16) ? period / 2 : 0);
}

constexpr int DK = 64;           // k values per LDS stage

__device__ __forceinline__ void dma16(uint32_t lds_addr, uint32_t voff, i32x4 rs) {
    // each lane moves 16 bytes from (rs.base + voff) to LDS byte (lds_addr + 16*lane); lanes past the
    // buffer's extent deposit zeros
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rs) : "memory");
}

// One operand's tile of ROWS rows of C's dimension x DK values of k, shared by NW waves.
//   KC (k contiguous in memory): LDS [row][k], 128 bytes a row, 16-byte chunks XOR-swizzled by the row index;
//      fragments come out with ds_read_b128.
//   otherwise (k strided):       LDS [k][row], 64-byte slots XOR-swizzled by the k index; fragments come out with the
//      transposing ds_read_b64_tr_b16.
// Either way lane l of a fragment holds row (l % 32), k = 16*step + 8*(l/32) .. +7.
template <bool KC, int ROWS, int NW>
struct DmaTile {
    static constexpr int BYTES = ROWS * DK * 2;
    static constexpr int PER_WAVE = BYTES / 1024 / NW;   // DMA instructions of 1 KB a wave issues per stage
    static_assert(PER_WAVE * NW * 1024 == BYTES, "the tile must split evenly over the waves");
    static constexpr int PITCH = ROWS * 2;               // bytes of a k row (k strided)
    // slot swizzle of k row k: four consecutive k rows must fall into four different 64-byte slots of 256 bytes
    __device__ static __forceinline__ int slot(int k) { return ROWS == 64 ? ((k >> 1) & 1) << 6 : (k & 3) << 6; }
    // k contiguous: the tile row that this lane fetches with instruction i of wave w
    __device__ static __forceinline__ int row(int wave, int i) { return 8 * (wave * PER_WAVE + i) + ((threadIdx.x & 63) >> 3); }
    // source byte offset of instruction i of wave w: the global address picks the logical chunk that the swizzle
    // places at the physical slot the lane writes
    __device__ static __forceinline__ uint32_t voff(int wave, int i, int row0, int ld) {
        const int idx = wave * PER_WAVE + i, L = threadIdx.x & 63;
        if (KC) {
            const int r = 8 * idx + (L >> 3);
            const int logical = (L & 7) ^ ((r >> 1) & 7);
            return ((uint32_t)(row0 + r) * (uint32_t)ld + (uint32_t)(logical * 8)) * 2u;
        } else {
            constexpr int LPR = PITCH / 16;              // lanes per k row
            const int k = idx * (64 / LPR) + L / LPR;
            const int lbyte = ((L % LPR) * 16) ^ slot(k);
            return ((uint32_t)k * (uint32_t)ld + (uint32_t)row0) * 2u + (uint32_t)lbyte;
        }
    }
    __device__ static __forceinline__ uint32_t kstep_bytes(int ld) { return KC ? DK * 2u : (uint32_t)DK * (uint32_t)ld * 2u; }
    // fragment of 32 rows starting at rb, k step kk (0..3)
    __device__ static __forceinline__ bf16x8 frag(const char* lds, int rb, int kk) {
        const int l = threadIdx.x & 63;
        if (KC) {
            const int r = rb + (l & 31), c = 2 * kk + (l >> 5);
            return *reinterpret_cast<const bf16x8*>(lds + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
        } else {
            typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
            const int col = rb + 16 * ((l >> 4) & 1) + 4 * (l & 3);
            const int kr0 = 16 * kk + 8 * (l >> 5) + ((l & 15) >> 2);
            const int kr1 = kr0 + 4;
            const char* p0 = lds + kr0 * PITCH + ((col * 2) ^ slot(kr0));
            const char* p1 = lds + kr1 * PITCH + ((col * 2) ^ slot(kr1));
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p0);
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p1);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
};

}  // namespace hh
