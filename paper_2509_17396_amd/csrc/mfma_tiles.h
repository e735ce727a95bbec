// Device helpers shared by the MFMA kernels (scoring passes, patch attention): vector types, the
// direct global->LDS staging of 64-row tiles with an XOR-swizzled LDS image, MFMA operand fragments.
#pragma once

#include "epicache_internal.h"

namespace epicache {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef uint16_t bf16_t;  // raw storage

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

__device__ __forceinline__ bf16x8 as_frag(uint4 u) { return __builtin_bit_cast(bf16x8, u); }
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
// The bare instructions: fmaxf() on values that went through pin() gets a canonicalising v_max x, x
// in front of every operand, which doubled the ALU work of the max reduction.  The compiler's hazard pass does
// not see inline assembly as a vector ALU instruction and inserts no wait states for it: these must never be
// the first reader of an MFMA result (12 wait states after an 8-pass MFMA on gfx950) or of a transcendental's
// result.  The callers read values that a compiler-visible instruction has already read or produced;
// tests/test_isa_hazards.py checks the generated ISA for it.
__device__ __forceinline__ float vmax(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float vmax3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ void fence_sched() { __builtin_amdgcn_sched_barrier(0); }
// Keeps the computation of x above this point: without it the optimiser sinks a slice of
// arithmetic down to its first use, past the MFMAs it is meant to fill the shadow of.
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)


// HD is the row layout in LDS (64, 128 or 256 elements); a head_dim in between uses the next one, and the operand that
// is kept in registers is zero behind its last chunk.
template <int HD>
struct Tile {
  static constexpr int kSteps = HD / 16;          // MFMAs per 32x32 output tile when all of HD is used
  static constexpr int kChunks = HD / 8;          // 16-byte chunks per row
  static constexpr int kRowBytes = HD * 2;
  static constexpr int kTileBytes = 64 * kRowBytes;
  static constexpr int kSlabs = kTileBytes / 1024;   // 1 KiB wave-wide direct loads per tile
  static constexpr int kRowsPerSlab = 1024 / kRowBytes;
  // XOR swizzle: chunk c of row r sits at position c ^ swz(r)
  __device__ static __forceinline__ int swz(int r) { return kChunks < 16 ? (r / (16 / (kChunks < 16 ? kChunks : 16))) % kChunks : r % kChunks; }
};

// 16 bytes per lane, global memory -> LDS without passing through registers: lane l of the wave
// writes LDS bytes [lds_addr + 16*l, +16).  Issued as inline assembly so that the compiler's
// wait-count pass does not serialise later ds_reads of the *other* LDS buffer behind these loads;
// completion is awaited explicitly (wait_vmem) before the barrier that publishes the tile.
// M0 is on the clobber lists: the statements overwrite it, and the compiler (which sets M0 itself right before
// its own users of it) must not assume a value survives them.  Clang flags any reserved register on a clobber
// list; for M0 the entry is exactly the definition that has to be declared.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16_uniform_base(uint32_t lds_addr, const void* base, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(voff), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void dma16_lane_ptr(uint32_t lds_addr, const void* ptr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds_addr), "v"(ptr)
               : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)LDS_PTR(p);
}

// What the chunks behind a row's last one are filled with: whatever else there were, times the zeros of the other
// operand, is no zero where it is an infinity or a NaN.
static __device__ const uint4 kZeroChunk = {0, 0, 0, 0};

// Staging of one 64-row tile, global -> LDS, by NW waves.  Rows are `stride` bytes apart and have last_chunk + 1 chunks
// of 16 bytes.  Wave w issues the 1 KiB slabs w, w + NW, w + 2*NW, ...; `wave` must be wave-uniform.
// EXACT_ROWS: the rows fill the layout.  Otherwise the products read 2 * KS chunks: those of them that a row does not
// have come from kZeroChunk, and the ones behind them re-fetch the row's last chunk.
template <int HD, int KS, int NW, bool EXACT_ROWS>
struct Stager {
  using TL = Tile<HD>;
  static constexpr int kSlabs = TL::kSlabs;
  static constexpr int kPer = (kSlabs + NW - 1) / NW;  // direct loads per wave and tile (at most)
  static constexpr uint32_t kPadding = ~0u;
  // The swizzle repeats after kPeriod rows: where registers are short a wave keeps the offsets of that many rows.
  static constexpr int kPeriod = TL::kChunks > 16 ? TL::kChunks : 16, kStep = NW * TL::kRowsPerSlab;
  static constexpr int kOffsets = EXACT_ROWS ? kPer : kStep >= kPeriod ? 1 : kPeriod / kStep < kPer ? kPeriod / kStep : kPer;
  struct Offsets {
    uint32_t off[kOffsets];  // from the first row of a tile to the chunk that the lane fetches in load i < kOffsets
    uint32_t stride;
    bool padded;             // wave-uniform: some off[] are kPadding
  };
  __device__ static __forceinline__ Offsets offsets(int wave, int lane, uint32_t stride, int last_chunk) {
    Offsets o;
    o.stride = stride;
    o.padded = !EXACT_ROWS && last_chunk + 1 < 2 * KS;
#pragma unroll
    for (int i = 0; i < kOffsets; i++) {
      const int row = (wave + i * NW) * TL::kRowsPerSlab + lane / TL::kChunks;
      const int chunk = (lane % TL::kChunks) ^ TL::swz(row);
      o.off[i] = row * stride + min(chunk, last_chunk) * 16;
      if (!EXACT_ROWS && chunk > last_chunk && chunk < 2 * KS) o.off[i] = kPadding;
    }
    return o;
  }
  // Address of slab i of the wave.  Where there are other things to keep in scalar registers the addresses are made one
  // from the other: made in advance for all loads, like the masks of the padding, they would be spilled to vector
  // registers, and a load must not follow the lane read that fetches its address too closely.
  __device__ static __forceinline__ uint32_t slab(uint32_t lds_tile, int wave, int i, uint32_t& at) {
    at = i == 0 ? lds_tile + wave * 1024 : at + NW * 1024;
    asm volatile("" : "+s"(at));
    return at;
  }
  // all 64 rows exist: tile base (wave-uniform) + per-lane offsets
  __device__ static __forceinline__ void run(uint32_t lds_tile, const unsigned char* base, const Offsets& o, int wave) {
    uint32_t at = 0;
    if (!EXACT_ROWS && __builtin_expect(o.padded, 0)) {  // out of the way of the rows that fill their products
#pragma unroll
      for (int i = 0; i < kPer; i++)
        if (kSlabs % NW == 0 || wave + i * NW < kSlabs) {
          uint32_t off = o.off[i % kOffsets];
          asm volatile("" : "+v"(off));
          const unsigned char* from = base + (size_t)(i / kOffsets * kOffsets * kStep) * o.stride + off;
          dma16_lane_ptr(slab(lds_tile, wave, i, at), off == kPadding ? reinterpret_cast<const unsigned char*>(&kZeroChunk) : from);
        }
      return;
    }
#pragma unroll
    for (int i = 0; i < kPer; i++)
      if (kSlabs % NW == 0 || wave + i * NW < kSlabs)
        dma16_uniform_base(EXACT_ROWS ? lds_tile + (wave + i * NW) * 1024 : slab(lds_tile, wave, i, at),
                           base + (size_t)(i / kOffsets * kOffsets * kStep) * o.stride, o.off[i % kOffsets]);
  }
  // general form: `row_ptr(r)` gives the address of row r of the tile (clamping, ragged strides)
  template <typename RowPtr>
  __device__ static __forceinline__ void run_rows(uint32_t lds_tile, int wave, int lane, RowPtr row_ptr, int last_chunk) {
    uint32_t at = 0;
#pragma unroll
    for (int i = 0; i < kPer; i++) {
      if (kSlabs % NW == 0 || wave + i * NW < kSlabs) {
        const int row = (wave + i * NW) * TL::kRowsPerSlab + lane / TL::kChunks;
        int chunk = (lane % TL::kChunks) ^ TL::swz(row);
        if (!EXACT_ROWS) asm volatile("" : "+v"(chunk));
        const unsigned char* from = row_ptr(row) + min(chunk, last_chunk) * 16;
        if (!EXACT_ROWS && chunk > last_chunk) from = reinterpret_cast<const unsigned char*>(&kZeroChunk);
        dma16_lane_ptr(EXACT_ROWS ? lds_tile + (wave + i * NW) * 1024 : slab(lds_tile, wave, i, at), from);
      }
    }
  }
};

// MFMA operand fragments J0 .. J1 - 1 of one 32-row sub-tile of a staged tile.
template <int HD, int KS, int J0 = 0, int J1 = KS>
__device__ __forceinline__ void read_frags(bf16x8 (&f)[KS], const unsigned char* lds_tile, int sub,
                                           int l32, int hi) {
  using TL = Tile<HD>;
  const int row = sub * 32 + l32;
  const unsigned char* base = lds_tile + row * TL::kRowBytes;
  const int s = TL::swz(row);
#pragma unroll
  for (int j = J0; j < J1; j++)
    f[j] = as_frag(*reinterpret_cast<const uint4*>(base + (((2 * j + hi) ^ s) * 16)));
}

// The operand that stays in registers: 16-byte chunks hi, 2 + hi, .. of a row of head_dim elements; beyond head_dim
// it is zero.  The loads are unconditional.
template <int KS>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[KS], const bf16_t* row, int hi, int d) {
  if (d == KS * 16) {  // all of it: one lane address and immediate offsets
    row += hi * 8;
#pragma unroll
    for (int j = 0; j < KS; j++) f[j] = as_frag(*reinterpret_cast<const uint4*>(row + j * 16));
    return;
  }
  const int last = d / 8 - 1;
#pragma unroll
  for (int j = 0; j < KS; j++)
    f[j] = as_frag(*reinterpret_cast<const uint4*>(row + min(2 * j + hi, last) * 8));
#pragma unroll
  for (int j = 0; j < KS; j++)
    if (2 * j + hi > last) f[j] = as_frag(make_uint4(0, 0, 0, 0));
}

// Finite sentinels instead of infinities keep the running-max updates branch-free and NaN-free:
// kNoMax is the "no key seen yet" maximum, kMasked (< kNoMax) the logit of a key that must not count.
// Their products with c2 = scale * log2(e) must stay finite (no inf - inf in the exponent arithmetic), which
// holds for every scale the host accepts (<= 1e6); raw dot products are assumed to lie above kNoMax.
constexpr float kNoMax = -1.0e30f;
constexpr float kMasked = -2.0e30f;

// acc += A B over 32 bytes of every operand row: one MFMA of 16 bf16 values, or (F32) four of 2 fp32 values, each lane
// half feeding the four values of its own 16-byte chunk.
template <bool F32 = false>
__device__ __forceinline__ void mfma_step(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  if constexpr (F32) {
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; i++) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], y[i], acc, 0, 0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  }
}

template <int KS, bool F32 = false>
__device__ __forceinline__ void mfma_chain(f32x16& acc, const bf16x8 (&a)[KS], const bf16x8 (&b)[KS]) {
  acc = f32x16{0};
#pragma unroll
  for (int j = 0; j < KS; j++) mfma_step<F32>(acc, a[j], b[j]);
}

}  // namespace epicache
