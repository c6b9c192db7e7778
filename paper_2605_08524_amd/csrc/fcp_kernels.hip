// HIP kernels for gfx950 (MI355X) and their launchers.
//
// Contractions run on v_mfma_f32_32x32x16_bf16.  Operand layouts (64 lanes, l = lane):
//   A (32 x 16): lane holds row l%32, k = 8*(l/32) .. +7          (8 bf16 = 4 VGPRs)
//   B (16 x 32): lane holds col l%32, k = 8*(l/32) .. +7
//   C/D (32 x 32 fp32, 16 VGPRs): reg r of lane l = row 8*(r/4) + 4*(l/32) + r%4, col l%32
// Because a sum over k does not care about the order of k, any k-slot assignment is valid as
// long as A and B use the same one; the kernels exploit this to feed an accumulator straight
// back as the B operand of the next contraction.
//
// ds_read_b64_tr_b16 (LDS transpose read): inside each group of 16 lanes, lane i receives, for
// e = 0..3, element (i%4) of the 8-byte row addressed by lane 4*e + i/4.  With lane s of a
// group pointing at M[r0 + s/4][c0 + 4*(s%4)], lane i ends up with M[r0 + 0..3][c0 + i]: four
// consecutive rows of one column, which is what an MFMA operand needs when the contracted index
// runs down the rows of a row-major LDS tile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "fcp_internal.h"

namespace fcp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 h = __builtin_convertvector(f, bf16x2);   // round-to-nearest-even
  return __builtin_bit_cast(uint32_t, h);
}

// Two transpose reads -> one 8-slot MFMA operand.
__device__ __forceinline__ bf16x8 lds_tr_pair(const unsigned char* lo, const unsigned char* hi) {
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, lo));
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, hi));
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  s16x8 c = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, c);
}

__device__ __forceinline__ float xor32(float x) { return __shfl_xor(x, 32, 64); }
// Maximum over a lane and its partner (lane ^ 32), without a trip through LDS: the swap leaves the lower half of x in both
// halves of one result, the upper half in the other.  (__builtin_bit_cast of a vector element takes element 0: copies first.)
__device__ __forceinline__ float max32(float x) {
  const uint32_t a = __builtin_bit_cast(uint32_t, x);
  const u32x2 r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
  const uint32_t lo = r[0], hi = r[1];
  return fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
}

// LDS accesses through 32-bit LDS addresses kept in registers: a tile buffer switch is then one
// add per address (in place) and row / tile offsets fold into the instruction's immediate field.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}
__device__ __forceinline__ u32x4 lds_read16(uint32_t addr) {
  return *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)addr;
}
__device__ __forceinline__ bf16x8 lds_tr_pair_at(uint32_t lo, uint32_t hi) {
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)lo);
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)hi);
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  s16x8 c = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, c);
}

// Byte offset of 16-byte chunk c of row r in an LDS tile.  Rows are unpadded (D*2 bytes) because
// tiles are filled by LDS-DMA loads that write 1 KB of consecutive LDS per wave instruction; the
// chunk index is XOR-swizzled with the row so that both access patterns are conflict free for
// D = 128 (rows of exactly 64 banks): row-wise ds_read_b128 (16 lanes = 16 consecutive rows, one
// chunk column) and transpose reads (32 lanes = 4 consecutive rows x 4 consecutive chunks).
template <int D>
__device__ __forceinline__ int swz(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else return (r >> 1) & 7;
}
template <int D>
__device__ __forceinline__ int tile_off(int r, int c) { return r * (D * 2) + ((c ^ swz<D>(r)) << 4); }

// Asynchronous copy of a [ROWS x D] bf16 tile from global memory straight into LDS (no
// registers): each global_load_lds_dwordx4 moves 64 x 16 B into 1 KB of consecutive LDS, so lane
// i of instruction n fills physical chunk i % (D/8) of row n*(1024/(2D)) + i/(D/8) and fetches
// the logical chunk that the swizzle places there.  Rows >= valid_rows are filled from a zero
// page.  Completion: s_waitcnt vmcnt(0) by the issuing wave, then a workgroup barrier.
// The load is issued through inline assembly on purpose: the compiler then does not model it as
// a write to LDS, so it does not make every later LDS read of the *other* buffer wait for it
// (it cannot tell run-time-indexed buffers apart).  Ordering is explicit instead: dma_wait()
// and a barrier before anyone reads what was loaded.  m0 carries the wave-uniform LDS address.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is clobbered on purpose; nothing else here lives in it
__device__ __forceinline__ void lds_dma16(const unsigned char* gptr, uint32_t lds_addr) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(gptr), "s"(m0) : "memory", "m0");
}
#pragma clang diagnostic pop
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16_s(const unsigned char* sbase, uint32_t voff, uint32_t lds_addr) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
  const uint64_t b = reinterpret_cast<uint64_t>(sbase);       // wave-uniform by construction
  // readfirstlane returns a signed int: widen through uint32_t, or the low half sign-extends
  // into the high half of the address.
  const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  const uint64_t sb = ((uint64_t)b_hi << 32) | (uint64_t)b_lo;
  // s_nop 4: a vector-memory instruction may read an SGPR only 5 wait states after a scalar or
  // v_readfirstlane write to it; the compiler's hazard pass does not look inside inline assembly,
  // and the base in %1 is typically produced right before this statement.  (Also covers m0.)
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(sb), "s"(m0) : "memory", "m0");
}
#pragma clang diagnostic pop
// Same for 64 x 4 bytes: lane i's dword lands at lds_addr + 4*i.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma4(const float* gptr, uint32_t lds_addr) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :: "v"(gptr), "s"(m0) : "memory", "m0");
}
#pragma clang diagnostic pop
// Byte offset, from the first row of a 1 KB load instruction, of the chunk that lane `lane` of
// wave `wave` fetches.  Instruction n*NWAVES + wave covers rows that differ from wave's first
// instruction by a multiple of 16, the period of the swizzle, so the offset is one per-lane
// constant for the whole kernel.
template <int D>
__device__ __forceinline__ uint32_t dma_lane_offset(int wave, int lane, int64_t row_stride) {
  constexpr int CPR = D / 8, RPI = 64 / CPR;
  const int r = wave * RPI + lane / CPR, pc = lane % CPR;
  return (uint32_t)((lane / CPR) * row_stride * 2 + ((pc ^ swz<D>(r)) << 4));
}
template <int D, int ROWS, int NWAVES>
__device__ __forceinline__ void tile_dma(unsigned char* lds_tile, const uint16_t* src, int64_t row_stride,
                                         int valid_rows, const unsigned char* zeros, int wave, int lane,
                                         uint32_t lane_off) {
  constexpr int CPR = D / 8, RPI = 64 / CPR, NI = ROWS / RPI;
  static_assert(NI % NWAVES == 0, "tile does not split evenly over the waves");
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_tile;
  if (valid_rows >= ROWS) {
    // whole tile in range (wave-uniform): scalar base per instruction + the per-lane constant
#pragma unroll
    for (int n = 0; n < NI / NWAVES; n++) {
      const int inst = n * NWAVES + wave;
      lds_dma16_s(reinterpret_cast<const unsigned char*>(src + (int64_t)inst * RPI * row_stride), lane_off,
                  lds_base + inst * 1024);
    }
    return;
  }
#pragma unroll
  for (int n = 0; n < NI / NWAVES; n++) {
    const int inst = n * NWAVES + wave;
    const int r = inst * RPI + lane / CPR;
    const int pc = lane % CPR;
    const unsigned char* gp = zeros + pc * 16;
    if (r < valid_rows) gp = reinterpret_cast<const unsigned char*>(src + (int64_t)r * row_stride + ((pc ^ swz<D>(r)) << 3));
    lds_dma16(gp, lds_base + inst * 1024);
  }
}
__device__ __forceinline__ void dma_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Workgroup barrier that waits for this wave's LDS accesses only (__syncthreads() may also wait for its stores).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
  asm volatile("s_barrier" ::: "memory");
}

// Rows between global memory and the MFMA layouts, through 2 KB of LDS that belongs to one wave.  In an accumulator tile
// and in a B operand a lane owns a row, so direct accesses are 64 separate 16-byte pieces per instruction, which the
// vector memory pipe takes one at a time (measured: 1 lane per clock; the 128 KB of fp32 results of a forward item kept it
// busy for 8000 cycles).  Here four lanes handle 64 consecutive bytes of a row and an instruction covers 16 rows: 16
// cycles.  Stage layout: 32 rows of 64 bytes, 16-byte chunk c of row r at position c ^ ((r >> 2) & 3): conflict free by
// row (lane = row) and by chunk (4 lanes = 1 row).  The LDS accesses of a wave are executed in order: no barrier.
// Forward of 16-256 token sequences (65536 tokens, GQA 32/8, d = 128, fp32 O): 691 -> 587 us, dK/dV 626 -> 581, dQ from dS 433 -> 370.
constexpr int kStageBytes = 2048;
__device__ __forceinline__ int stage_off(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }

// dst = first of the tile's 32 columns in row 0 of the 32 rows; rows at or past `rows` are not written.
template <bool BF16>
__device__ __forceinline__ void store_tile(void* dst, int64_t row_stride, int rows, const f32x16& x, float mul, unsigned char* stage, int lane) {
  asm volatile("" : "+v"(lane));       // the addresses are formed here, not kept in registers through the caller's tile loop
  const int l32 = lane & 31, g = lane >> 5, sr = lane >> 2, sc = lane & 3;
#pragma unroll
  for (int h = 0; h < (BF16 ? 1 : 2); h++) {       // 64 bytes of every row: 32 bf16 or 16 fp32 columns
#pragma unroll
    for (int m = 0; m < 2; m++) {
      u32x4 w;
      if constexpr (BF16) {
        // the lane holds columns 8 q4 + 4 g .. +3, its partner (lane ^ 32, same row) the other four of every eight: they trade halves
        const uint32_t e0 = pack_bf16(x[8 * m] * mul, x[8 * m + 1] * mul), e1 = pack_bf16(x[8 * m + 2] * mul, x[8 * m + 3] * mul);
        const uint32_t f0 = pack_bf16(x[8 * m + 4] * mul, x[8 * m + 5] * mul), f1 = pack_bf16(x[8 * m + 6] * mul, x[8 * m + 7] * mul);
        // swap(x, y): lanes 32-63 of x trade places with lanes 0-31 of y
        const u32x2 r = __builtin_amdgcn_permlane32_swap(e0, f0, false, false);
        const u32x2 t = __builtin_amdgcn_permlane32_swap(e1, f1, false, false);
        w = u32x4{r[0], t[0], r[1], t[1]};
      } else {
        const int q = 4 * (2 * h + m);
        w = __builtin_bit_cast(u32x4, f32x4{x[q] * mul, x[q + 1] * mul, x[q + 2] * mul, x[q + 3] * mul});
      }
      *reinterpret_cast<u32x4*>(stage + stage_off(l32, 2 * m + g)) = w;
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int r = 16 * i + sr;
      const u32x4 w = *reinterpret_cast<const u32x4*>(stage + stage_off(r, sc));
      if (r < rows) {
        if constexpr (BF16) *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(dst) + r * row_stride + 8 * sc) = w;
        else *reinterpret_cast<u32x4*>(reinterpret_cast<float*>(dst) + r * row_stride + 16 * h + 4 * sc) = w;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Rows row0 .. row0 + 31 of a [rows x D] bf16 slab as B operands (lane = row, 8 consecutive d per k-chunk); rows at or past
// `rows` read as zero (their loads repeat the last valid row, or row 0 of an empty slab, so they need no branch).
template <int D>
__device__ __forceinline__ void load_rows(bf16x8 (&f)[D / 16], const uint16_t* slab, int64_t row_stride, int row0, int rows, unsigned char* stage, int lane) {
  asm volatile("" : "+v"(lane));
  const int l32 = lane & 31, g = lane >> 5, sr = lane >> 2, sc = lane & 3;
  const int last = max(rows, 1) - 1;
  const uint16_t* p0 = slab + min(row0 + sr, last) * row_stride + 8 * sc;
  const uint16_t* p1 = slab + min(row0 + 16 + sr, last) * row_stride + 8 * sc;
  u32x4 t[D / 16];
#pragma unroll
  for (int p = 0; p < D / 32; p++) {
    t[2 * p] = *reinterpret_cast<const u32x4*>(p0 + 32 * p);
    t[2 * p + 1] = *reinterpret_cast<const u32x4*>(p1 + 32 * p);
  }
  const bool ok = row0 + l32 < rows;
#pragma unroll
  for (int p = 0; p < D / 32; p++) {
    *reinterpret_cast<u32x4*>(stage + stage_off(sr, sc)) = t[2 * p];
    *reinterpret_cast<u32x4*>(stage + stage_off(16 + sr, sc)) = t[2 * p + 1];
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(stage + stage_off(l32, 2 * j + g));
      f[2 * p + j] = as_bf16x8(ok ? w : u32x4{0, 0, 0, 0});
    }
  }
  __builtin_amdgcn_sched_barrier(0);
}

template <int D> constexpr int tile_bytes(int rows) { return rows * D * 2; }

// The last workgroup to run dry clears the counters for the next launch.
__device__ __forceinline__ void retire(int32_t* counter, int32_t* done) {
  const int prev = atomicAdd(done, 1);
  if (prev == (int)gridDim.x - 1) {
    for (int q = 0; q < kNumXcd; q++) atomicExch(&counter[q * kCounterStride], 0);
    atomicExch(done, 0);
  }
}

// The item sequence of one persistent workgroup.  Item indices are tickets of the eight XCD queues, drawn from the queue of
// the XCD the workgroup runs on (hardware register XCC_ID) and, once that is dry, from the other queues.  No item belongs to
// a workgroup that has not started: one that has to wait for a compute unit (another stream's kernel may hold it for long)
// finds the queues dry.  First tickets by block index save 0.2-0.8 us of a launch on an idle chip, but where another stream
// held 32 compute units the heaviest items then ran last: training step of an 8-worker share (103746 tokens, heads 9/3,
// d = 128) 5220 us, drawn 4576; 16384 tokens, 16 heads, d = 64: 830 and 763.  request() asks for a ticket without waiting, take() turns it into an item index some tiles later;
// both near the end of the current item (early draws unbalance the end of a launch).  Both are for one wave.  Every
// workgroup leaves its loop when all queues are dry.
struct ItemStream {
  int32_t* counter; const int32_t* begin;
  int ticket, bounds;      // bounds: lane 0 the home queue's begin, lane 1 its end
  bool dry;
  // An increment that wraps at 2^32: of an add the compiler makes one add per wave and waits for its result on the spot (4000
  // tokens, 4 heads, d = 64, forward: 19.6 us with adds, 19.1 so; training step of 2000 tokens: 53.2 and 52.5).
  __device__ __forceinline__ static int draw(int32_t* c) { return (int)atomicInc(reinterpret_cast<unsigned*>(c), 0xffffffffu); }
  __device__ __forceinline__ static int home_queue() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & (kNumXcd - 1); }   // XCC_ID (id 20), bits [3:0]
  // The first item, or -1.  The queue's bounds (lane 0: its begin, lane 1: its end) are in flight beside the ticket: one
  // round trip to memory in front of the first record instead of two.
  __device__ __forceinline__ int start(int32_t* c, const int32_t* b, int lane) {
    counter = c; begin = b; ticket = 0; dry = false;
    bounds = begin[home_queue() + (lane & 1)];
    request(lane);
    const int t = __builtin_amdgcn_readfirstlane(ticket), b0 = __builtin_amdgcn_readlane(bounds, 0);
    if (t < __builtin_amdgcn_readlane(bounds, 1) - b0) return b0 + t;
    dry = true;
    return steal(lane);
  }
  __device__ __forceinline__ void request(int lane) { if (!dry && lane == 0) ticket = draw(&counter[home_queue() * kCounterStride]); }
  __device__ __forceinline__ int take(int lane) {
    if (!dry) {
      const int t = __builtin_amdgcn_readfirstlane(ticket), b0 = __builtin_amdgcn_readlane(bounds, 0);
      if (t < __builtin_amdgcn_readlane(bounds, 1) - b0) return b0 + t;
      dry = true;
    }
    return steal(lane);
  }
  // Lane t looks at queue home + t: one round trip for all eight counters, a second one for a ticket if any is left.
  // Asking one queue after the other put 5 us at the end of every launch.
  __device__ __forceinline__ int steal(int lane) {
    const int home = home_queue(), q = (home + lane) % kNumXcd, b0 = begin[q];
    const int n = begin[q + 1] - b0;
    uint64_t left = __builtin_amdgcn_ballot_w64(lane < kNumXcd && n > 0 && __hip_atomic_load(&counter[q * kCounterStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n);
    while (left) {
      const int l = __builtin_ctzll(left);
      left &= left - 1;
      const int ql = (home + l) % kNumXcd;
      int i = 0;
      if (lane == 0) i = draw(&counter[ql * kCounterStride]);
      i = __builtin_amdgcn_readfirstlane(i);
      if (i < __builtin_amdgcn_readlane(n, l)) return __builtin_amdgcn_readlane(b0, l) + i;
    }
    return -1;
  }
};

// The record of the next item travels through LDS: wave 0 requests it by LDS-DMA before the current item ends, so the
// cold table reads (record, then its first pair: 4 us of a 14 us item of short sequences) are not in front of the next.
template <class Item>
__device__ __forceinline__ void fetch_item(const Item* items, int idx, int32_t* rec, int lane) {
  static_assert(sizeof(Item) % 16 == 0 && sizeof(Item) <= 256, "read in 16-byte pieces, fetched by one instruction");
  lds_dma4(reinterpret_cast<const float*>(items + idx) + min(lane, (int)sizeof(Item) / 4 - 1), lds_addr(rec));
}
template <class Item>
__device__ __forceinline__ Item read_item(const int32_t* rec) {
  union { Item it; u32x4 w[sizeof(Item) / 16]; } u;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(Item) / 16); i++) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(rec + 4 * i);
#pragma unroll
    for (int j = 0; j < 4; j++) u.w[i][j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)v[j]);   // wave-uniform: scalar registers
  }
  return u.it;
}

// =====================================================================================
// Forward: partial attention.  Item = (slot, two 128-row query sub-tiles that share the slot's
// K/V stream: two query heads of one KV head, or two neighbouring row tiles of one head);
// workgroup of 8 waves, two per SIMD, 32 query rows per wave.
// The wave computes S^T = K Q^T so that a lane owns one query row (column of S^T): row
// statistics need one cross-half exchange, and the exponentiated accumulator is, as is,
// the B operand of O^T += V^T P^T.  The loop over 64-row K/V tiles is software-pipelined by
// hand: in iteration i the wave issues the MFMAs of S(i+1) and then of O += V(i)^T P(i), and
// places the exponentials of tile i, and later the maximum of tile i+1, between them, so the
// matrix pipe does not wait for the vector ALU inside a wave.  [K | V] tiles sit in a ring of
// four LDS buffers filled by LDS-DMA three tiles ahead (all 8 waves share one stream); one
// workgroup barrier per tile.  The first iteration of an item computes S of its first tile only
// and the last one only adds the last tile to O, so the pipeline fill costs no MFMAs; all
// iterations issue the same tile loads.  Every item starts at buffer 0, without a barrier of its own: no wave reads the ring
// behind the last tile barrier, and a wave fills the same rows of every buffer, so the look-ahead loads that could still land in
// the next item's first tiles are its own, and it waits for them at the item's end.
// Between the last MFMA of an iteration and the first of the next lie the barrier, the row maximum and the walk to the next tile,
// without an MFMA beside them in either wave of the SIMD (both have just passed the barrier): 1150 of 3650 cycles at d = 128,
// 1050 of 2350 at d = 64 (timestamps).  What runs there is kept short: spans instead of pairs (DevPair) and a step of a few scalar
// additions inside one, one word per tile that says from where on it is masked, buffer offsets as immediates, the maximum
// over both halves without LDS, the row sums pinned into the exponential phase.  Forward, before and after: 4000 tokens, 4 heads,
// d = 64 19.1 -> 16.4 us; 65536 lognormal tokens, GQA 32/8, d = 128 2357 -> 2211 (977 -> 1042 algorithmic TFLOP/s); 32768 rows of a
// 262144-token sequence 64.2 -> 60.4 ms; short sequences in shared blocks 335 -> 309 us.
// A wave computes only the tiles its own rows can see: past them (a diagonal, a ragged end, an item of one sub-tile) it
// loads and waits.  65536 packed tokens (lognormal, GQA 32/8, d = 128): 2.66 -> 2.60 ms; sequences of 16-256 tokens:
// 0.72 -> 0.66 ms.
// =====================================================================================
constexpr int kFwdTileN = kQTileN;   // KV rows per LDS tile (the host counts an item's tiles with the same constant)
constexpr int kFwdBufs = 4;     // ring of [K | V] tile buffers
constexpr float kRescaleSlack = 8.0f;   // log2 units

struct FwdArgs {
  const uint16_t* q; const uint16_t* k; const uint16_t* v;
  void* o_part; float* lse_part; int32_t part_is_bf16;
  void* o; float* lse; int32_t o_is_f32;     // final outputs for query blocks with a single slot (or NULL)
  int32_t running;                            // fold every slot into the running (o, lse) in place (fp32 o)
  WsHeader* hdr; const DevPair* spans; const QItem* items; const uint16_t* q_seg;
  int32_t n_q_heads, n_kv_heads;
  float scale_log2;   // softmax scale * log2(e)
};

// Iterator over the KV tiles of an item's pairs, in pair order.  For a DIAG pair only the
// columns up to the tile's last query row are visited.
struct TileIter {
  const DevPair* pairs;
  int pair, pair_end, c0, ncols, row_hi;   // row_hi = tile_off + q_rows (first row past the tile)
  DevPair cur;
  bool more;
  __device__ __forceinline__ void set(int kv_start, int kv_len, int kind, int ext) {
    // the pair index is wave-uniform; readfirstlane says so to the compiler, which then keeps the record (and
    // everything derived from it) in scalar registers and branches on it with scalar branches
    cur.kv_start = __builtin_amdgcn_readfirstlane(kv_start); cur.kv_len = __builtin_amdgcn_readfirstlane(kv_len);
    cur.kind = __builtin_amdgcn_readfirstlane(kind); cur.ext = __builtin_amdgcn_readfirstlane(ext);
    ncols = (cur.kind & 1) ? min(cur.kv_len, row_hi) : cur.kv_len;
  }
  __device__ __forceinline__ void load_pair() {
    const DevPair p = pairs[pair];
    set(p.kv_start, p.kv_len, p.kind, p.ext);
  }
  __device__ __forceinline__ void init(const DevPair* p, const QItem& it) {
    pairs = p; pair = it.pair_begin; pair_end = it.pair_begin + it.n_pairs; c0 = 0; ncols = 0;
    row_hi = max(it.tile_off[0] + it.q_rows[0], it.tile_off[1] + it.q_rows[1]);
    cur = DevPair{0, 0, 0, 0};
    more = it.n_pairs > 0;
    if (more) set(it.first.kv_start, it.first.kv_len, it.first.kind, it.first.ext);
  }
  __device__ __forceinline__ void advance() {
    c0 += kFwdTileN;
    if (c0 >= ncols) {
      pair++;
      c0 = 0;
      if (pair < pair_end) load_pair(); else more = false;
    }
  }
};

// The scores of a 64-column tile that a lane keeps if only columns < c count, one bit per score: score e = 16 rt + r of a lane
// is column 8 (e / 4) + 4 g + e % 4.  A mask of bits costs a score two operations, as a compare with a bound does, but only
// one register in all beside the scores, also where a row has two bounds (a joined run).
__device__ __forceinline__ uint32_t keep_below(int c, int g) {
  c = min(max(c, 0), kFwdTileN);
  const int n = 4 * (c >> 3) + min(max((c & 7) - 4 * g, 0), 4);
  return n < 32 ? (1u << n) - 1 : 0xffffffffu;
}

template <int D>
__global__ void __launch_bounds__(512, 2) fwd_kernel(FwdArgs a) {
  constexpr int KC = D / 16;      // k-chunks of the QK^T contraction
  constexpr int DT = D / 32;      // row tiles of O^T
  constexpr int NS1 = 2 * KC;     // MFMAs of S^T (two 32-row halves of the KV tile)
  constexpr int NS2 = 4 * DT;     // MFMAs of O^T += V^T P^T
  constexpr int PF = 2;           // an LDS operand is requested this many MFMAs before its use (4: more spills, 1-3 % slower)
  constexpr int TB = tile_bytes<D>(kFwdTileN);
  constexpr int BUF = 2 * TB;     // [K tile | V tile]
  constexpr int NB = kFwdBufs;
  constexpr int CPR = D / 8, RPI = 64 / CPR, NDMA = kFwdTileN / RPI / 8;   // LDS-DMA geometry, see issue()
  constexpr int DMA_PER_TILE = 2 * NDMA;
  __shared__ __attribute__((aligned(1024))) unsigned char lds_kv[NB][BUF];
  __shared__ __attribute__((aligned(16))) int32_t s_rec[2][64];   // records of this item and the next
  __shared__ int s_next;
  __shared__ __attribute__((aligned(16))) unsigned char s_stage[8][kStageBytes];
  __shared__ uint32_t s_mask[2 * kFwdTileM / kFwdTileN][512];   // joined run: scores that each lane keeps of each KV tile (written and read by that lane)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
  const int l32 = lane & 31, g = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D;     // elements
  const int64_t kv_row_stride = (int64_t)a.n_kv_heads * D;
  const unsigned char* zeros = reinterpret_cast<const unsigned char*>(a.hdr->zeros);
  // LDS-DMA of a 64-row tile: instruction n of this wave fills LDS rows r_n = (8n + wave) * RPI + lane / CPR.
  // A lane fetches chunk (pc ^ swz(r_n)) of global row min(r_n, valid - 1): rows past a ragged end
  // repeat the last valid row (finite values; those columns are masked).
  // (r_n and r_0 differ by a multiple of 16, the period of the swizzle: one chunk offset serves all n.)
  static_assert(8 * RPI % 16 == 0, "swizzle period");
  const uint32_t dma_row0 = (uint32_t)((wave * RPI + lane / CPR) * kv_row_stride * 2);
  const uint32_t dma_chunk = (uint32_t)(((lane % CPR) ^ swz<D>(wave * RPI + lane / CPR)) << 4);
  const uint32_t dma_step = (uint32_t)(8 * RPI * kv_row_stride * 2);
  // transpose-read pattern inside a 16-lane group: row tr_row, 4 columns from tr_col
  const int tr_row = (lane & 15) >> 2, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  // Tile t of an item is in buffer t % 4: in iteration i the wave reads the K rows of tile i+1, transposes V of tile i, and
  // tile i+3 is requested.  Per-lane LDS addresses (the swizzle has period 16 in the row, so rows +16 / +32 are plain
  // immediate offsets) of a pair of buffers: the second one is an immediate offset too, and the addresses change pairs
  // every other tile.
  static_assert(NB == 4 && BUF + 3 * 16 * D * 2 < 65536 && BUF + 32 * D * 2 < 65536, "two pairs of buffers, offsets of 16 bits");
  uint32_t tr_lo[DT], tr_hi[DT], kk_off[KC];
#pragma unroll
  for (int dt = 0; dt < DT; dt++) {
    tr_lo[dt] = lds_addr(lds_kv[0]) + TB + tile_off<D>(4 * g + tr_row, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
    tr_hi[dt] = lds_addr(lds_kv[0]) + TB + tile_off<D>(4 * g + tr_row + 8, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
  }
#pragma unroll
  for (int kc = 0; kc < KC; kc++) kk_off[kc] = lds_addr(lds_kv[0]) + tile_off<D>(l32, 2 * kc + g);
  auto move_k = [&](int by) {
#pragma unroll
    for (int kc = 0; kc < KC; kc++) kk_off[kc] += by;
  };
  auto move_v = [&](int by) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) { tr_lo[dt] += by; tr_hi[dt] += by; }
  };

  ItemStream items;
  if (wave == 0) {
    const int first = items.start(a.hdr->fwd_counter, a.hdr->fwd_begin, lane);
    if (first >= 0) fetch_item(a.items, first, s_rec[0], lane);
    if (lane == 0) s_next = first;
    dma_wait();
  }
  __syncthreads();
  int item_idx = __builtin_amdgcn_readfirstlane(s_next);   // wave-uniform
  for (int par = 0; item_idx >= 0; par ^= 1) {
    const QItem it = read_item<QItem>(s_rec[par]);
    // Sub-item, 32-row group inside it.  The groups of sub-item 1 run backwards over the waves: waves w and w + 4 share a
    // SIMD, so the group that sees least of a diagonal (or nothing, past a ragged end) sits next to one that sees most.
    // Four heads on 64 rows: two waves a head, both groups on every pair of SIMDs.
    const bool four = it.head[1] - it.head[0] == 3;
    const int sub = wave >> 2, wq = four ? (wave & 1) ^ sub : sub ? 3 - (wave & 3) : wave & 3;
    // selects, not it.q_rows[sub]: a run-time index would put the whole item into private memory
    const int q_rows = (sub ? it.q_rows[1] : it.q_rows[0]), tile_off_q = (sub ? it.tile_off[1] : it.tile_off[0]), head = four ? it.head[0] + (wave >> 1) : (sub ? it.head[1] : it.head[0]);
    const int kvh = __builtin_amdgcn_readfirstlane(it.head[0] / group);     // the division runs on the vector unit
    const int my_row = wq * 32 + l32;                        // row inside the sub-tile
    const int wave_row_lo = tile_off_q + wq * 32;            // rows of this wave inside the block
    const int my_limit = tile_off_q + my_row;                // last visible column of a DIAG pair for this lane
    const uint16_t* kbase = a.k + (int64_t)kvh * D;
    const uint16_t* vbase = a.v + (int64_t)kvh * D;

    if (it.first.kind & 2) {
      // joined run: the columns of the row's member, up to the row itself under a causal mask; rows past the end: none
      int lo = 0, hi = 0;
      if (my_row < q_rows) {
        const int sg = a.q_seg[(sub ? it.q_start[1] : it.q_start[0]) + my_row];
        lo = sg & 0xff; hi = ((it.first.kind & 1) ? min(sg >> 8, my_limit) : sg >> 8) + 1;
      }
#pragma unroll
      for (int t = 0; t < 2 * kFwdTileM / kFwdTileN; t++)
        s_mask[t][tid] = keep_below(hi - t * kFwdTileN, g) & ~keep_below(lo - t * kFwdTileN, g);
    }

    // Q^T fragments (B operand of S^T = K Q^T): lane = query row, 8 consecutive d per k-chunk.
    bf16x8 qf[KC];
    load_rows<D>(qf, a.q + (int64_t)(sub ? it.q_start[1] : it.q_start[0]) * q_row_stride + (int64_t)head * D, q_row_stride,
                 wq * 32, q_rows, s_stage[wave], lane);
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) o[dt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // Tiles this wave computes: all of the item's, less the trailing ones of a last DIAG span that start past its own
    // last row; none if its rows lie past the ragged end.  What remains it only loads and waits for.
    const int row_hi = max(it.tile_off[0] + it.q_rows[0], it.tile_off[1] + it.q_rows[1]);
    const int wave_row_hi = min(wave_row_lo + 32, tile_off_q + q_rows);
    const int n_tiles = it.n_tiles;
    const int n_vis = wq * 32 >= q_rows ? 0
                    : it.diag_last >= 0 ? n_tiles - ((it.diag_last + row_hi + kFwdTileN - 1) / kFwdTileN - (it.diag_last + wave_row_hi + kFwdTileN - 1) / kFwdTileN)
                                        : n_tiles;

    // The load of one tile in two parts.  describe(): scalar bookkeeping, run at an iteration boundary, where no MFMA
    // covers it: inside a span a handful of additions.  issue(): branch-free, sits between the MFMAs.
    // A tile is masked for this wave from the column on where its first row sees nothing more (a DIAG span), the span ends, or at
    // once (a joined run): d_word, and word[] of the tiles described ahead.
    const uint32_t lim_whole = (uint32_t)((kFwdTileN - 1) * kv_row_stride * 2);
    const uint64_t tile_step = (uint64_t)(kFwdTileN * kv_row_stride * 2);        // from 2^18 KV heads on more than 32 bits
    uint64_t d_k = 0, d_v = 0;
    uint32_t d_lim = 0, lim_last = 0;
    int left = 0, span = 0;           // tiles of the span in hand not yet described, less one; its number
    int d_word = 0;                   // 4 * (columns that need no mask - first column - 64) + kind: below zero needs a mask
    auto open_span = [&](const DevPair& sp) {
      // wave-uniform: readfirstlane says so to the compiler, which then keeps what follows in scalar registers
      const int kv_start = __builtin_amdgcn_readfirstlane(sp.kv_start), kv_len = __builtin_amdgcn_readfirstlane(sp.kv_len);
      const int kind = __builtin_amdgcn_readfirstlane(sp.kind), diag = __builtin_amdgcn_readfirstlane(sp.ext);
      const int ncols = (kind & 1) ? min(kv_len, diag + row_hi) : kv_len;
      left = (ncols - 1) / kFwdTileN;
      lim_last = (uint32_t)((min(kFwdTileN, kv_len - left * kFwdTileN) - 1) * kv_row_stride * 2);
      d_lim = left > 0 ? lim_whole : lim_last;
      const int64_t row0 = (int64_t)kv_start * kv_row_stride;
      d_k = reinterpret_cast<uint64_t>(kbase + row0);
      d_v = reinterpret_cast<uint64_t>(vbase + row0);
      const int open = (kind & 2) ? 0 : (kind & 1) ? diag + wave_row_lo + 1 : kv_len;
      d_word = 4 * (open - kFwdTileN) + kind;
      span++;
    };
    auto describe = [&]() {
      if (__builtin_expect(left > 0, 1)) {
        left--;
        d_k += tile_step; d_v += tile_step;
        d_word -= 4 * kFwdTileN;
        d_lim = left > 0 ? lim_whole : lim_last;
      } else if (span < it.n_pairs) {
        open_span(a.spans[it.pair_begin + span]);
      } else {
        d_k = reinterpret_cast<uint64_t>(zeros); d_v = d_k; d_lim = 0;      // past the end
      }
    };
    int dma_tile = 0;
    auto issue = [&]() {
      const uint32_t lbase = lds_addr(lds_kv[0]) + (dma_tile & (NB - 1)) * BUF;
#pragma unroll
      for (int n = 0; n < NDMA; n++) {
        const uint32_t voff = min(dma_row0 + n * dma_step, d_lim) + dma_chunk;
        lds_dma16_s(reinterpret_cast<const unsigned char*>(d_k), voff, lbase + (8 * n + wave) * 1024);
        lds_dma16_s(reinterpret_cast<const unsigned char*>(d_v), voff, lbase + TB + (8 * n + wave) * 1024);
      }
      dma_tile++;
    };
    const bool short_item = n_vis < 7;         // too short to ask for the next ticket later than here
    if (wave == 0 && short_item) items.request(lane);
    // prologue: tiles 0 and 1
    int word[3];                      // d_word of tiles i+1, i+2, i+3 (shift register)
    if (it.n_pairs > 0) open_span(it.first); else describe();
    issue(); word[0] = d_word;
    describe(); issue(); word[1] = d_word;
    describe(); word[2] = d_word;     // tile 2, requested inside the first iteration
    dma_wait();
    __syncthreads();

    f32x16 s_a[2], s_b[2];            // S^T of the tile being exponentiated / being computed
#pragma unroll
    for (int rt = 0; rt < 2; rt++)
#pragma unroll
      for (int r = 0; r < 16; r++) { s_a[rt][r] = -INFINITY; s_b[rt][r] = 0.f; }

    auto next_tile = [&]() { word[0] = word[1]; word[1] = word[2]; describe(); word[2] = d_word; };
    int k_step = 2 * BUF, v_step = 2 * BUF;      // to the other pair of buffers
    // the tile two ahead has landed once at most one tile's loads are in flight
    auto tile_barrier = [&]() {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (DMA_PER_TILE & 15) | ((DMA_PER_TILE >> 4) << 14));
      __syncthreads();
    };
    // One iteration.  sc = scores of tile i (masked, maximum already folded into m_run);
    // sn receives S^T of tile i+1.  ODD: i is odd (the buffer of its pair that V of tile i is in; K of tile i+1: the other one).
    // FIRST: nothing to exponentiate or to add to O yet (S^T of tile 0 only); LAST: no next tile (O += V P of the
    // last tile only).  An item thus costs one iteration's worth of MFMAs per tile and nothing for the pipeline fill.
    auto iteration = [&](auto first_t, auto last_t, auto odd_t, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
      constexpr bool FIRST = decltype(first_t)::value, LAST = decltype(last_t)::value, ODD = decltype(odd_t)::value;
      constexpr uint32_t K_OFF = ODD ? 0 : BUF, V_OFF = ODD ? BUF : 0;
      const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
      u32x4 pb[4];                    // P^T of tile i as four B operands (rt, j)
      float rs = 0.f;
      float p_prev = 0.f;
      // the exponential of the NEXT element is issued before this one is consumed, so its latency
      // does not sit in a dependent chain (the wave issues in order)
      float p_ahead = 0.f;
      if constexpr (!FIRST) p_ahead = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0][0], a.scale_log2, -m_use));
      auto expo = [&](int e) {        // element e = (rt, r) of tile i
        const int r = e & 15;
        const float p = p_ahead;
        if (e + 1 < 32) p_ahead = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[(e + 1) >> 4][(e + 1) & 15], a.scale_log2, -m_use));
        rs += p;
        if (r & 1) {
          pb[e >> 3][(e >> 1) & 3] = pack_bf16(p_prev, p);
          // keeps the vector work between the MFMAs it was written between; without rs the 32 additions all sank behind the
          // barrier, where no MFMA covers them, and held 32 registers until then
          asm volatile("" : "+v"(rs) : "v"(pb[e >> 3][(e >> 1) & 3]));
        } else p_prev = p;
      };
      // ---- phase 1: S^T(i+1) = K Q^T (two 32-row halves); exponentials of tile i between the MFMAs
      if constexpr (LAST) {
        issue();
#pragma unroll
        for (int e = 0; e < 24; e++) expo(e);
      } else {
        u32x4 op[PF];
#pragma unroll
        for (int u = 0; u < PF; u++) op[u] = lds_read16(kk_off[u / 2] + K_OFF + (u & 1) * 32 * (D * 2));
#pragma unroll
        for (int u = 0; u < NS1; u++) {
          const int kc = u / 2, rt = u & 1;
          if (kc == 0) {
#pragma unroll
            for (int r = 0; r < 16; r++) sn[rt][r] = 0.f;
          }
          sn[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[u % PF]), qf[kc], sn[rt], 0, 0, 0);
          if (u + PF < NS1) op[u % PF] = lds_read16(kk_off[(u + PF) / 2] + K_OFF + ((u + PF) & 1) * 32 * (D * 2));
          // 24 of the 32 elements in this phase
          if constexpr (!FIRST) {
#pragma unroll
            for (int e = u * 24 / NS1; e < (u + 1) * 24 / NS1; e++) expo(e);
          }
          if (u == NS1 / 2) issue();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // ---- phase 2: O^T += V^T P^T; the rest of the exponentials
      if constexpr (!FIRST) {
        u32x4 op[PF];
        auto fetch = [&](int u) {
          const uint32_t rows = V_OFF + 16 * (u / DT) * (D * 2);
          return __builtin_bit_cast(u32x4, lds_tr_pair_at(tr_lo[u % DT] + rows, tr_hi[u % DT] + rows));
        };
#pragma unroll
        for (int u = 0; u < PF; u++) op[u] = fetch(u);
#pragma unroll
        for (int u = 0; u < NS2; u++) {
          o[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[u % PF]), as_bf16x8(pb[u / DT]), o[u % DT], 0, 0, 0);
          if (u + PF < NS2) op[u % PF] = fetch(u + PF);
#pragma unroll
          for (int e = 24 + u * 8 / (NS2 / 2); e < 24 + (u + 1) * 8 / (NS2 / 2) && u < NS2 / 2; e++) expo(e);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      l_run += rs;
      tile_barrier();
      // ---- mask of tile i+1 (only tiles that touch the diagonal or a ragged end, or lie past the
      // end of the item), then its maximum
      if constexpr (!LAST) {
        const int w = __builtin_amdgcn_readfirstlane(word[0]);
        if (__builtin_expect(w < 0, 0)) {
          // one bit per score of this lane (see keep_below): columns up to the last visible one, or of the row's member
          const int open = (w >> 2) + kFwdTileN;       // columns of the tile that the wave's first row sees
          uint32_t keep = keep_below(open + ((w & 1) ? l32 : 0), g);
          if (w & 2) keep = s_mask[-(w >> 2) / kFwdTileN - 1][tid];
#pragma unroll
          for (int rt = 0; rt < 2; rt++)
#pragma unroll
            for (int r = 0; r < 16; r++)
              if (!(keep & (1u << (16 * rt + r)))) sn[rt][r] = -INFINITY;
        }
      }
      if constexpr (!LAST) {
        float mx = fmaxf(sn[0][0], sn[1][0]);
#pragma unroll
        for (int r = 1; r < 16; r++) mx = fmaxf(fmaxf(mx, sn[0][r]), sn[1][r]);
        // ---- online softmax bookkeeping for tile i+1, in the log2 domain.  The reference maximum
        // m_run only moves when some row's maximum exceeds it by more than kRescaleSlack (a
        // wave-uniform decision): any reference gives the same O and LSE as long as exp2 stays in
        // range, and P <= 2^slack is harmless in bf16/fp32.  Most tiles skip the rescaling of O.
        mx = max32(mx) * a.scale_log2;
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleSlack) != 0) {
          const float m_new = fmaxf(m_run, mx);
          const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
          const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);   // m_run = -inf -> 0
          m_run = m_new;
          l_run *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; dt++)
#pragma unroll
            for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
        }
      }
      if constexpr (ODD && !FIRST) {
        move_v(v_step); v_step = -v_step;
      } else if constexpr (!LAST && !FIRST) {
        move_k(k_step); k_step = -k_step;
      }
      next_tile();
    };
    const std::true_type yes;
    const std::false_type no;
    // The item takes n_tiles + 1 iterations (barriers); a wave computes in the first n_vis + 1 of them.
    // The next item (wave 0): its ticket is requested some tiles before it is turned into an index, and the record behind
    // that index is requested before the item's last tile barrier, which publishes both.
    auto next_item = [&]() {
      const int nx = items.take(lane);
      if (lane == 0) s_next = nx;
      if (nx >= 0) fetch_item(a.items, nx, s_rec[par ^ 1], lane);
    };
    int idle = n_tiles - n_vis;
    if (n_vis > 0) {
      iteration(yes, no, yes, s_a, s_b);   // S^T of tile 0 (i = -1)
      // iterations that do both phases; they alternate (s_b, s_a), (s_a, s_b)
      int rem = n_vis - 1;
      for (int stop = 4; stop >= 0; stop -= 2) {      // down to 4 (5) of them, to 2 (3), to 0 (1)
        for (; rem >= stop + 2; rem -= 2) {
          iteration(no, no, no, s_b, s_a);
          iteration(no, no, yes, s_a, s_b);
        }
        if (wave == 0) {
          if (stop == 4 && !short_item) items.request(lane);
          if (stop == 2) next_item();
        }
      }
      if (rem) {
        iteration(no, no, no, s_b, s_a);   // a tail, not a branch inside the loop (which costs dozens of spills)
        move_v(BUF);                       // V of the last tile is in the second buffer of its pair
      } else {
#pragma unroll
        for (int rt = 0; rt < 2; rt++) s_a[rt] = s_b[rt];
      }
      iteration(no, yes, no, s_a, s_b);    // O += V P of the last tile
      move_v((rem ? -BUF : 0) + (v_step < 0 ? -2 * BUF : 0));       // back to buffer 0 for the next item
      move_k(k_step < 0 ? -2 * BUF : 0);
    } else {
      issue(); tile_barrier(); next_tile();
      if (wave == 0) next_item();
    }
    for (; idle > 0; idle--) { issue(); tile_barrier(); next_tile(); }
    if (n_tiles == 0) { dma_wait(); __syncthreads(); }      // an item without tiles has no barrier behind next_item()
    dma_wait();         // the look-ahead loads past the end of the item (zero tiles)

    // ---- epilogue (the record is read again, not kept in registers through the tile loop): normalise, write the partial (fp32) and its LSE
    const QItem e = read_item<QItem>(s_rec[par]);
    const int e_row = wq * 32 + l32, e_head = e.head[1] - e.head[0] == 3 ? e.head[0] + (wave >> 1) : sub ? e.head[1] : e.head[0];
    const bool e_ok = e_row < (sub ? e.q_rows[1] : e.q_rows[0]);
    const int64_t e_q_row = (int64_t)((sub ? e.q_start[1] : e.q_start[0]) + e_row);
    const float l_tot = l_run + xor32(l_run);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (e_ok && a.running) {
      // Two-way reduction in place: the running (O, LSE) of this row and head, as the earlier stages left it, and
      // this slot's (o / l_tot, lse_s) combine with weights exp(LSE - m); a running LSE of -inf means "nothing
      // yet" (whatever O holds then is ignored).  One writer per row and launch; stages are ordered by the stream.
      const int64_t row = e_q_row;
      float* op = reinterpret_cast<float*>(a.o) + row * q_row_stride + (int64_t)e_head * D;
      float* lp = a.lse + row * a.n_q_heads + e_head;
      const float lse_s = l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
      const float lse_o = *lp;
      const float m = fmaxf(lse_o, lse_s);
      const float w_o = lse_o == -INFINITY ? 0.f : __expf(lse_o - m);
      const float w_s = lse_s == -INFINITY ? 0.f : __expf(lse_s - m);
      const float tot = w_o + w_s;
      const float c_o = tot > 0.f ? w_o / tot : 0.f, c_s = tot > 0.f ? w_s / tot * inv : 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
          f32x4* ptr = reinterpret_cast<f32x4*>(op + dt * 32 + 8 * q4 + 4 * g);
          f32x4 old = *ptr;
          if (lse_o == -INFINITY) old = f32x4{0.f, 0.f, 0.f, 0.f};
          const f32x4 cur = {o[dt][4 * q4], o[dt][4 * q4 + 1], o[dt][4 * q4 + 2], o[dt][4 * q4 + 3]};
          *ptr = old * c_o + cur * c_s;
        }
      if (g == 0) *lp = tot > 0.f ? m + __logf(tot) : -INFINITY;
    } else if (!a.running) {
      // the only slot of its query block: this is the final result, not a partial
      const bool to_final = e.to_final != 0;
      const int64_t row0 = (to_final ? (sub ? e.q_start[1] : e.q_start[0]) : (sub ? e.out_row[1] : e.out_row[0])) + wq * 32;
      const int64_t off = row0 * q_row_stride + (int64_t)e_head * D;
      const int rows = (sub ? e.q_rows[1] : e.q_rows[0]) - wq * 32;
      if (to_final ? !a.o_is_f32 : a.part_is_bf16) {
        uint16_t* op = reinterpret_cast<uint16_t*>(to_final ? a.o : a.o_part) + off;
#pragma unroll
        for (int dt = 0; dt < DT; dt++) store_tile<true>(op + dt * 32, q_row_stride, rows, o[dt], inv, s_stage[wave], lane);
      } else {
        float* op = reinterpret_cast<float*>(to_final ? a.o : a.o_part) + off;
#pragma unroll
        for (int dt = 0; dt < DT; dt++) store_tile<false>(op + dt * 32, q_row_stride, rows, o[dt], inv, s_stage[wave], lane);
      }
      if (g == 0 && e_ok) {
        const float lse = l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
        (to_final ? a.lse : a.lse_part)[(row0 + l32) * a.n_q_heads + e_head] = lse;
      }
    }
    // No barrier here: behind the last tile barrier no wave reads the ring, and the next item's loads start at once.
    item_idx = __builtin_amdgcn_readfirstlane(s_next);
  }
  if (tid == 0) retire(a.hdr->fwd_counter, &a.hdr->fwd_done);
}

// =====================================================================================
// Launches that leave most of the chip idle.  An item of the kernels above is 256 query rows (128 KV rows) and a serial chain of
// tiles; with few items the chain of the longest one is the launch (4000 tokens, 4 heads, d = 64: 140 items, 16 tiles of 1 us).
// Here a workgroup owns 32 rows, a quarter of a sub-tile (KV tile), and its eight waves share what those rows stream: wave w
// takes the 32-row tiles w, w + 8, .. of it through LDS of its own (LDS-DMA, waited for by count, no barrier in the loop), and
// the eight results meet in LDS at the end.  A wave walks an eighth of the columns (steps) that an item walks in one chain, and
// there are eight (four) times the workgroups.  Same items, same tables, no queues: a workgroup's place in the grid names its rows.
// Where there is room two workgroups share a compute unit (d = 64); nothing is scheduled by hand, the other waves cover the waits.
// The price: 32 rows read every K / V (Q / dO) row of theirs by themselves, where an item reads them once for 256, and each
// workgroup pays for its start and its reduction; choose_split weighs both.  Before / after, us: forward of 4000 tokens, 4 heads,
// d = 64 16.6 / 9.2, of one 8192-token sequence 129 / 34 (4 heads: 131 / 62; d = 128: 167 / 49 and 169 / 118); backward of 2000
// tokens, 4/2 heads, d = 64 35 / 14, of 8192 tokens 315 / 75 (4/1 heads: 730 / 268; d = 128: 424 / 111 and 952 / 378).
// Four waves instead of eight: up to 25 % faster where the chip is full, 30-40 % slower where it is not; at d = 128, two such
// workgroups to a compute unit where there are more than units, 0.6 to 1.2 times as fast.
// =====================================================================================
constexpr int kSplitRows = 32, kSplitWaves = 8;

// A workgroup's item and which 32 rows of it: the units of an item follow each other on one XCD (apart, they read what they
// share from further away: 2048-token sequences, 8 heads, d = 64, forward 68 -> 143 us).
struct SplitPlace {
  int item, unit;
  __device__ __forceinline__ SplitPlace(int b, int units) { const int j = b / kNumXcd; unit = j % units; item = j / units * kNumXcd + b % kNumXcd; }
};

// A table record by scalar loads (wave-uniform address; no kernel writes the tables).
template <class Item>
__device__ __forceinline__ Item load_record(const Item* p) {
  union { Item it; u32x4 w[sizeof(Item) / 16]; } u;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(Item) / 16); i++) {
    const u32x4 v = ((const __attribute__((address_space(4))) u32x4*)(uintptr_t)p)[i];
#pragma unroll
    for (int j = 0; j < 4; j++) u.w[i][j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)v[j]);
  }
  return u.it;
}

// Records of 16 bytes (pairs, spans, dependencies), 64 at a time in a wave's registers: the walk to a wave's next tile passes
// several of them and would wait for each.  The first one comes with the item.
template <class Rec>
struct RecordWindow {
  const Rec* table;
  int n, from;                  // records; number of the first one in the window, -1: nothing loaded yet
  Rec head;
  u32x4 w;
  __device__ __forceinline__ void init(const Rec* t, int n_, const Rec& first) { table = t; n = n_; from = -1; head = first; w = u32x4{0, 0, 0, 0}; }
  __device__ __forceinline__ Rec get(int i, int lane) {       // i: wave-uniform, below n
    if (i == 0) return head;
    if (from < 0 || i >= from + 64) { from = i; w = *reinterpret_cast<const u32x4*>(table + min(from + lane, n - 1)); }
    const int l = i - from;
    return Rec{__builtin_amdgcn_readlane((int)w[0], l), __builtin_amdgcn_readlane((int)w[1], l), __builtin_amdgcn_readlane((int)w[2], l), __builtin_amdgcn_readlane((int)w[3], l)};
  }
};

// 32 rows of a [rows x D] slab into the wave's own LDS, rows past `valid` as repeats of the last valid one.
template <int D>
__device__ __forceinline__ void wave_tile_dma(uint32_t lds, const uint16_t* src, uint32_t row_bytes, int valid, int lane) {
  constexpr int CPR = D / 8, RPI = 64 / CPR;
  asm volatile("" : "+v"(lane));       // the offsets are formed here, not kept in registers through the caller's loop
  const uint32_t lim = (uint32_t)(valid - 1) * row_bytes, own = (uint32_t)(lane / CPR) * row_bytes;
#pragma unroll
  for (int n = 0; n < kSplitRows / RPI; n++)
    lds_dma16_s(reinterpret_cast<const unsigned char*>(src), min(own + n * RPI * row_bytes, lim) + (((lane % CPR) ^ swz<D>(n * RPI + lane / CPR)) << 4), lds + n * 1024);
}
// The same by the waves of a workgroup, one instruction each: the rows that stay.
template <int D>
__device__ __forceinline__ void group_tile_dma(uint32_t lds, const uint16_t* src, uint32_t row_bytes, int valid, int piece, int lane) {
  constexpr int CPR = D / 8, RPI = 64 / CPR;
  static_assert(kSplitRows / RPI <= kSplitWaves, "one instruction a wave");
  if (piece >= kSplitRows / RPI) return;
  const int r = piece * RPI + lane / CPR;
  lds_dma16_s(reinterpret_cast<const unsigned char*>(src), (uint32_t)min(r, valid - 1) * row_bytes + (((lane % CPR) ^ swz<D>(r)) << 4), lds + piece * 1024);
}
// Waits in the loops of the split kernels; the memory clobber keeps LDS accesses on their side.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N>
__device__ __forceinline__ void loads_left() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// A wave's [D x 32] accumulators as 32 rows of D floats in its LDS region (32 * D * 4 bytes, what its two tiles take); 16-byte
// chunk c of row r at c ^ (r & 15): conflict free by row and by chunk.
template <int D>
__device__ __forceinline__ void put_result(unsigned char* region, const f32x16 (&acc)[D / 32], int lane) {
  asm volatile("" : "+v"(lane));
  const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++)
      *reinterpret_cast<f32x4*>(region + l32 * (D * 4) + (((8 * dt + 2 * q4 + g) ^ (l32 & 15)) << 4)) =
          f32x4{acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]};
}
template <int D>
__device__ __forceinline__ f32x4 get_result(const unsigned char* region, int row, int chunk) {
  return *reinterpret_cast<const f32x4*>(region + row * (D * 4) + ((chunk ^ (row & 15)) << 4));
}
// Four neighbouring columns of a row, in fp32 or rounded to bf16.
__device__ __forceinline__ void store4(void* base, int64_t at, const f32x4& x, bool bf16) {
  if (bf16) *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(base) + at) = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
  else *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(base) + at) = x;
}

// What a query-stationary workgroup (forward, dQ) is about: the 32 rows of unit u of an item, per_tile units to a sub-tile.
struct SplitQ {
  int q_start, rows, tile_off, head, out_row;    // the unit's first row in the Q buffer, its rows (32, fewer at the end), its first row in the segment
  __device__ __forceinline__ SplitQ(const QItem& it, int u, int per_tile) {
    const bool four = it.head[1] - it.head[0] == 3;      // four heads, two units each at most
    if (four) per_tile = min(per_tile, 2);
    const int off = u % per_tile * kSplitRows, part = u / per_tile, second = four ? 0 : -part;
    // by mask: a select becomes an index into the record, which then lives in memory
    auto of = [&](const int32_t (&v)[2]) { return v[0] ^ ((v[0] ^ v[1]) & second); };
    q_start = of(it.q_start) + off;
    rows = min(of(it.q_rows) - off, kSplitRows);
    tile_off = of(it.tile_off) + off;
    head = four ? it.head[0] + part : of(it.head);
    out_row = of(it.out_row) + off;
  }
};
// The 32-column tiles of an item's pairs (spans) that one wave takes: every eighth.
struct SplitTiles {
  RecordWindow<DevPair> rec;
  int pair, t, row_hi;          // the wave's tile t of pair `pair`; first row past the unit's
  bool spans, have;
  DevPair cur;
  __device__ __forceinline__ void init(const DevPair* table, const QItem& it, bool spans_, int row_hi_, int wave, int lane) {
    rec.init(table + it.pair_begin, it.n_pairs, it.first);
    spans = spans_; row_hi = row_hi_; pair = -1; t = wave;
    cur = it.first; have = it.n_pairs > 0;
    if (have) { pair = 0; seek(lane); }
  }
  __device__ __forceinline__ int tiles() const {
    return ((cur.kind & 1 ? min(cur.kv_len, (spans ? cur.ext : 0) + row_hi) : cur.kv_len) + kSplitRows - 1) / kSplitRows;
  }
  __device__ __forceinline__ void seek(int lane) {
    for (int n = tiles(); t >= n; n = tiles()) {
      t -= n;
      if (++pair >= rec.n) { have = false; return; }
      cur = rec.get(pair, lane);
    }
  }
  __device__ __forceinline__ void next(int lane) { t += kSplitWaves; seek(lane); }
};

// Forward, 32 query rows of one head.
template <int D>
__global__ void __launch_bounds__(64 * kSplitWaves, D == 64 ? 4 : 2) fwd_split_kernel(FwdArgs a, int n_items, int units, int per_tile) {
  constexpr int KC = D / 16, DT = D / 32, T = tile_bytes<D>(kSplitRows), NI = T / 1024;
  __shared__ __attribute__((aligned(1024))) unsigned char lds_kv[kSplitWaves][2 * T];    // [K tile | V tile], at the end the wave's O
  __shared__ __attribute__((aligned(1024))) unsigned char lds_q[T];
  __shared__ float s_m[kSplitWaves][kSplitRows], s_l[kSplitWaves][kSplitRows];
  __shared__ int s_act[kSplitWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
  const SplitPlace place(blockIdx.x, units);
  if (place.item >= n_items) return;
  const QItem it = load_record(a.items + place.item);
  const SplitQ u(it, place.unit, per_tile);
  if (u.rows <= 0) return;
  const int group = a.n_q_heads / a.n_kv_heads, kvh = __builtin_amdgcn_readfirstlane(u.head / group);
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D, kv_row_stride = (int64_t)a.n_kv_heads * D;
  const uint32_t kv_row_bytes = (uint32_t)(kv_row_stride * 2);
  const uint16_t* kbase = a.k + (int64_t)kvh * D;
  const uint16_t* vbase = a.v + (int64_t)kvh * D;
  const uint32_t lk = lds_addr(lds_kv[wave]), lv = lk + T;

  SplitTiles tiles;
  tiles.init(a.spans, it, true, u.tile_off + u.rows, wave, lane);
  auto issue = [&](const uint16_t* base, uint32_t lds) {
    const int c0 = tiles.t * kSplitRows;
    wave_tile_dma<D>(lds, base + (int64_t)(tiles.cur.kv_start + c0) * kv_row_stride, kv_row_bytes, min(kSplitRows, tiles.cur.kv_len - c0), lane);
  };
  group_tile_dma<D>(lds_addr(lds_q), a.q + (int64_t)u.q_start * q_row_stride + (int64_t)u.head * D, (uint32_t)(q_row_stride * 2), u.rows, wave, lane);
  const bool active = tiles.have;
  if (active) { issue(kbase, lk); issue(vbase, lv); }
  int seg_lo = 0, seg_hi = 0;          // joined run: the columns of this lane's member
  const int my_limit = u.tile_off + l32;
  if (it.first.kind & 2) {
    const int sg = l32 < u.rows ? a.q_seg[u.q_start + l32] : 0;
    seg_lo = sg & 0xff; seg_hi = (sg >> 8) + 1;
    if (l32 >= u.rows) seg_hi = 0;
  }
  loads_left<0>();
  __syncthreads();

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[dt][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  bf16x8 qf[KC];
#pragma unroll
  for (int kc = 0; kc < KC; kc++) qf[kc] = as_bf16x8(lds_read16(lds_addr(lds_q) + tile_off<D>(l32, 2 * kc + g)));
  const int tr_row = (lane & 15) >> 2, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  while (tiles.have) {
    const DevPair cur = tiles.cur;
    const int c0 = tiles.t * kSplitRows;
    tiles.next(lane);
    const bool more = tiles.have;
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(lds_read16(lk + tile_off<D>(l32, 2 * kc + g))), qf[kc], s, 0, 0, 0);
    lds_reads_done();
    if (more) issue(kbase, lk);
    // first column that this lane does not see / that some lane of the wave does not see
    int lo = 0, hi = (cur.kind & 1) ? min(cur.kv_len, cur.ext + my_limit + 1) : cur.kv_len;
    const int open = (cur.kind & 2) ? 0 : (cur.kind & 1) ? min(cur.kv_len, cur.ext + u.tile_off + 1) : cur.kv_len;
    if (c0 + kSplitRows > open) {
      if (cur.kind & 2) { lo = seg_lo; hi = min(seg_hi, hi); }
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int c = c0 + 8 * (r >> 2) + 4 * g + (r & 3);
        if (c < lo || c >= hi) s[r] = -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; r++) mx = fmaxf(mx, s[r]);
    mx = max32(mx) * a.scale_log2;
    if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleSlack) != 0) {       // as in fwd_kernel
      const float m_new = fmaxf(m_run, mx), m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    u32x4 pb[2];
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.scale_log2, -m_use)), p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r + 1], a.scale_log2, -m_use));
      l_run += p0 + p1;
      pb[r >> 3][(r >> 1) & 3] = pack_bf16(p0, p1);
    }
    if (more) loads_left<NI>(); else loads_left<0>();        // V has landed once only the next K is in flight
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        const int c = 4 * dt + (tr_col >> 3);
        const bf16x8 vt = lds_tr_pair_at(lv + tile_off<D>(16 * j + 4 * g + tr_row, c) + (tr_col & 4) * 2, lv + tile_off<D>(16 * j + 4 * g + tr_row + 8, c) + (tr_col & 4) * 2);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt, as_bf16x8(pb[j]), o[dt], 0, 0, 0);
      }
    lds_reads_done();
    if (more) { issue(vbase, lv); loads_left<NI>(); }        // the next K has landed once only the next V is in flight
  }
  if (active) put_result<D>(lds_kv[wave], o, lane);
  const float l_tot = l_run + xor32(l_run);
  if (g == 0) { s_m[wave][l32] = m_run; s_l[wave][l32] = l_tot; }
  if (lane == 0) s_act[wave] = active;
  __syncthreads();

  // the waves' results, D / 4 lanes to a row
  const bool to_final = it.to_final != 0;
#pragma unroll
  for (int pass = 0; pass < D * 8 / (64 * kSplitWaves); pass++) {
    const int row = (tid + 64 * kSplitWaves * pass) / (D / 4), chunk = tid % (D / 4);
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int w = 0; w < kSplitWaves; w++) m = fmaxf(m, s_m[w][row]);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kSplitWaves; w++) {
      if (!s_act[w]) break;              // waves without a tile are the last ones
      const float mw = s_m[w][row], f = mw == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mw - m);      // nothing seen: O and l are zero
      l += f * s_l[w][row];
      x += f * get_result<D>(lds_kv[w], row, chunk);
    }
    if (row >= u.rows) continue;
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const float lse = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
    if (a.running) {
      // as in fwd_kernel
      const int64_t r = u.q_start + row;
      float* op = reinterpret_cast<float*>(a.o) + r * q_row_stride + (int64_t)u.head * D + 4 * chunk;
      float* lp = a.lse + r * a.n_q_heads + u.head;
      const float lse_o = *lp, top = fmaxf(lse_o, lse);
      const float w_o = lse_o == -INFINITY ? 0.f : __expf(lse_o - top), w_s = lse == -INFINITY ? 0.f : __expf(lse - top), tot = w_o + w_s;
      const float c_o = tot > 0.f ? w_o / tot : 0.f, c_s = tot > 0.f ? w_s / tot * inv : 0.f;
      f32x4 old = *reinterpret_cast<f32x4*>(op);
      if (lse_o == -INFINITY) old = f32x4{0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4*>(op) = old * c_o + x * c_s;
      if (chunk == 0) *lp = tot > 0.f ? top + __logf(tot) : -INFINITY;
    } else {
      const int64_t r = (to_final ? u.q_start : u.out_row) + row;
      store4(to_final ? a.o : a.o_part, r * q_row_stride + (int64_t)u.head * D + 4 * chunk, x * inv, to_final ? !a.o_is_f32 : a.part_is_bf16);
      if (chunk == 0) (to_final ? a.lse : a.lse_part)[r * a.n_q_heads + u.head] = lse;
    }
  }
}

// =====================================================================================
// Merge: LSE-weighted reduction of the partials of each query block.  HBM-bound.
// One group of D/4 lanes owns one (row, head) entry: a float4 of the head vector per lane.
// =====================================================================================
struct MergeArgs {
  const void* o_part; const float* lse_part; void* o; float* lse;
  const MergeItem* items; const int32_t* slot_rh;
  int32_t o_is_f32, part_is_bf16;
};

template <int D>
__global__ void __launch_bounds__(256) merge_kernel(MergeArgs a) {
  constexpr int LPE = D / 4;            // lanes per entry
  constexpr int EPP = 256 / LPE;        // entries per pass
  constexpr int U = 4;                  // entries per thread and step (independent loads; 2, 6 and 8 measured slower)
  constexpr int STEP = EPP * U;         // entries the workgroup handles per step
  const MergeItem it = a.items[blockIdx.x];
  const int sub = threadIdx.x / LPE, ln = threadIdx.x % LPE;
  // The item is one stream of steps (chunk of STEP entries, slot), slots innermost; the loads of a step are issued two
  // steps before they are used, across chunk boundaries too, so that a query block with few partials keeps as many
  // bytes in flight as one with many.  acc and tot are kept relative to a running maximum (the online-softmax
  // recurrence) and rescaled when a larger LSE arrives.
  const int n_chunks = (it.n_rh + STEP - 1) / STEP;
  const int ns = max(it.n_slots, 1);    // a query block without any partial still gets O = 0, LSE = -inf: one empty step per chunk
  const int n_steps = n_chunks * ns;
  struct Buf { float l[U]; f32x4 x[U]; };
  auto load = [&](int t, Buf& bf) {
#pragma unroll
    for (int u = 0; u < U; u++) { bf.l[u] = -INFINITY; bf.x[u] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    if (t >= n_steps || it.n_slots == 0) return;
    const int c = t / ns, s = t - c * ns;
    const int e0 = c * STEP + sub;
    const int64_t base = (int64_t)a.slot_rh[it.slot_begin + s] + it.rh_off + e0;
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (e0 + u * EPP < it.n_rh) {
        bf.l[u] = a.lse_part[base + u * EPP];
        if (a.part_is_bf16) {
          const u32x2 h = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(a.o_part) + (base + u * EPP) * D + ln * 4));
          bf.x[u] = f32x4{__builtin_bit_cast(float, h[0] << 16), __builtin_bit_cast(float, h[0] & 0xffff0000u),
                          __builtin_bit_cast(float, h[1] << 16), __builtin_bit_cast(float, h[1] & 0xffff0000u)};
        } else {
          bf.x[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(a.o_part) + (base + u * EPP) * D + ln * 4));
        }
      }
    }
  };
  float mx[U], tot[U];
  f32x4 acc[U];
  int s_in_chunk = 0, chunk = 0;
  auto fold = [&](const Buf& bf) {
    if (s_in_chunk == 0) {
#pragma unroll
      for (int u = 0; u < U; u++) { mx[u] = -INFINITY; tot[u] = 0.f; acc[u] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      // an empty partial (LSE = -inf) carries weight 0; its payload must not leak through (0 * NaN)
      if (bf.l[u] != -INFINITY) {
        const float m_new = fmaxf(mx[u], bf.l[u]);
        const float keep = __expf(mx[u] - m_new);        // mx = -inf -> 0
        const float w = __expf(bf.l[u] - m_new);
        tot[u] = tot[u] * keep + w;
        acc[u] = acc[u] * keep + w * bf.x[u];
        mx[u] = m_new;
      }
    }
    if (++s_in_chunk == ns) {
      const int e0 = chunk * STEP + sub;
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (e0 + u * EPP >= it.n_rh) continue;
        const float inv = tot[u] > 0.f ? 1.0f / tot[u] : 0.f;
        const f32x4 r = acc[u] * inv;
        const int64_t out = (int64_t)it.out_rh + e0 + u * EPP;
        if (a.o_is_f32) {
          __builtin_nontemporal_store(r, reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.o) + out * D + ln * 4));
        } else {
          u32x2 h = {pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3])};
          __builtin_nontemporal_store(h, reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(a.o) + out * D + ln * 4));
        }
        if (ln == 0) a.lse[out] = tot[u] > 0.f ? mx[u] + __logf(tot[u]) : -INFINITY;
      }
      s_in_chunk = 0; chunk++;
    }
  };
  constexpr int NBUF = 3;               // two steps in flight + the one being folded (three in flight: no faster)
  Buf b[NBUF];
#pragma unroll
  for (int k = 0; k < NBUF - 1; k++) load(k, b[k]);
  for (int t = 0; t < n_steps; t += NBUF) {
#pragma unroll
    for (int k = 0; k < NBUF; k++) {
      if (t + k < n_steps) {
        load(t + k + NBUF - 1, b[(k + NBUF - 1) % NBUF]);
        fold(b[k]);
      }
    }
  }
}

// =====================================================================================
// Backward preprocess: D[t,h] = sum_c dO[t,h,c] * O[t,h,c].  HBM-bound.
// Emits what the two backward kernels consume, head-major [Hq][T_q] so that 32 consecutive
// query rows of one head are one 128-byte line:  dls = scale * D  and  lse2 = log2(e) * LSE,
// with +inf in place of an LSE of -inf (a row that saw no key has P = 0 and no gradient).
// One workgroup handles 16 tokens x all heads; results pass through LDS for the transposition.
// =====================================================================================
constexpr int kDeltaTok = 16;       // tokens per workgroup
constexpr int kDeltaHeads = 128;    // heads per pass through LDS

template <int D>
__global__ void __launch_bounds__(256) delta_kernel(const void* o, int o_is_f32, const uint16_t* d_o, const float* lse,
                                                    float* dls, float* lse2, int64_t t_q, int n_heads, float scale) {
  constexpr int LPE = D / 8;      // lanes per (token, head) entry, 8 elements each
  constexpr int EPP = 256 / LPE;  // entries per pass
  __shared__ float sm_d[kDeltaHeads][kDeltaTok + 1];
  __shared__ float sm_l[kDeltaHeads][kDeltaTok + 1];
  const int64_t t0 = (int64_t)blockIdx.x * kDeltaTok;
  const int n_tok = (int)min((int64_t)kDeltaTok, t_q - t0);
  const int sub = threadIdx.x / LPE, ln = threadIdx.x % LPE;
  for (int h0 = 0; h0 < n_heads; h0 += kDeltaHeads) {
    const int nh = min(kDeltaHeads, n_heads - h0);
    for (int e0 = 0; e0 < n_tok * nh; e0 += EPP) {
      const int el = e0 + sub;                 // entry inside the (token, head chunk) tile
      float acc = 0.f;
      const bool ok = el < n_tok * nh;
      const int tt = ok ? el / nh : 0, hh = ok ? el % nh : 0;
      const int64_t e = (t0 + tt) * n_heads + h0 + hh;
      if (ok) {
        const u32x4 dv = *reinterpret_cast<const u32x4*>(d_o + e * D + ln * 8);
        float ov[8];
        if (o_is_f32) {
          const f32x4 x0 = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(o) + e * D + ln * 8);
          const f32x4 x1 = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(o) + e * D + ln * 8 + 4);
          for (int i = 0; i < 4; i++) { ov[i] = x0[i]; ov[4 + i] = x1[i]; }
        } else {
          const u32x4 x = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(o) + e * D + ln * 8);
          for (int i = 0; i < 4; i++) {
            ov[2 * i] = __uint_as_float(x[i] << 16);
            ov[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u);
          }
        }
        for (int i = 0; i < 4; i++) {
          acc += __uint_as_float(dv[i] << 16) * ov[2 * i];
          acc += __uint_as_float(dv[i] & 0xffff0000u) * ov[2 * i + 1];
        }
      }
      for (int off = LPE / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
      if (ok && ln == 0) {
        const float l = lse[e];
        sm_d[hh][tt] = acc * scale;
        sm_l[hh][tt] = (l == -INFINITY) ? INFINITY : l * kLog2e;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nh * kDeltaTok; i += 256) {
      const int hh = i / kDeltaTok, tt = i % kDeltaTok;
      if (tt < n_tok) {
        const int64_t dst = (int64_t)(h0 + hh) * t_q + t0 + tt;
        dls[dst] = sm_d[hh][tt];
        lse2[dst] = sm_l[hh][tt];
      }
    }
    __syncthreads();
  }
}

// =====================================================================================
// Backward, part 1 -- dK and dV.  Item = (KV tile of 128 rows, KV head); workgroup of 8 waves, two
// per SIMD: four producers and four consumers.  A step is 32 query rows of one head:
//   producer s, KV rows 32*s .. +32 of the tile:
//             A(t): S = Q K^T, dP = dO V^T      (A operands: row-wise reads of the Q / dO tiles in
//                                                LDS; B operands: the wave's K / V rows in registers)
//             B(t): P = exp2(S*c - LSE*log2e), masked on the diagonal; dS = P o (dP*scale - D*scale);
//                   P and dS go to the consumers as bf16 MFMA B operands through LDS
//   consumer c, d rows 32*c .. +32 of dK^T / dV^T for all 128 KV rows (d = 64: 32 d rows x 64 KV rows):
//             C(t): dV^T += dO^T P, dK^T += Q^T dS   (A operands: transpose reads of its d rows of the
//                   same tiles, each used for every 32-row KV group; B operands: every producer's P / dS)
// dK^T / dV^T (rows = d, cols = KV rows) stay in the consumers' accumulators across every dependent
// query block and the G query heads of the group, so each dK / dV element has exactly one writer.
// The roles are decoupled by whole steps: in one barrier interval the consumer runs C(t) while
// the producer issues the MFMAs of A(t+2) with the vector work B(t+1) interleaved between them by
// hand.  The vector ALU work of the SIMD thus sits in one wave and half of its MFMAs in the
// other, and neither wave waits for the other inside an interval.  Q / dO tiles and the per-row
// scalars sit in a ring of seven LDS buffers filled by LDS-DMA (issued by the consumers) six
// steps ahead of their C phase; a tile is in place two intervals before the producer reads it,
// so the producer requests its first LDS operands of an interval, and the consumer all its A
// operands, before the barrier that opens it.
// One workgroup barrier per step.  Steps before the first and past the last of an item run on
// +inf LSE (P = dS = 0), which keeps the instruction stream and the count of loads in flight
// identical for every step; the ring runs on from item to item.
// LDS time per step and SIMD pair: 16 row reads + 8 scalar reads + 16 hand-over reads (b128,
// 256 B/clk), 8 transpose reads (b64, 160 B/clk), the 8 KB hand-over and the 4 KB of DMA writes
// (writes: 76 B/clk), about 1.15x the 1024 cycles of the 32 MFMAs (rates measured on this chip).
// dQ is not produced here: accumulating it across KV tiles needs fp32 atomics, and the chip
// sustains only about 1.35 TB/s of them (measured), several times below what this kernel would
// emit.  dq_kernel below recomputes S and dP query-stationary instead.
// =====================================================================================
struct BwdArgs {
  const uint16_t* q; const uint16_t* k; const uint16_t* v; const uint16_t* d_o;
  const float* lse2; const float* dls;     // head-major [Hq][T_q]: LSE*log2(e) (+inf for empty rows), D*scale
  // dq_kernel<D, true, *> computes those two itself from O, LSE and dO and writes them for dkdv_kernel
  const void* o; const float* lse; int32_t o_is_f32; float* lse2_out; float* dls_out;
  void* dq; void* dk; void* dv;    // fp32, or bf16 in the GRAD_BF16 instances of the kernels
  unsigned char* ds;               // dS spill buffer (2 KB fragments), or NULL
  WsHeader* hdr; const DevPair* pairs; const BwdDep* deps; const BwdItem* items; const QItem* dq_items; const uint16_t* q_seg;
  int64_t t_q;
  int32_t n_q_heads, n_kv_heads;
  float scale, scale_log2;
};

// Iterator over the runs of a backward item: the 32-row query steps of one dependent query block and head, in order; the G
// query heads of the group inside a dependency.  A DIAG dependency starts at the tile's own rows.  Inside a run a step is a
// few additions; what a new run needs is worked out at its start (consumers spent 350-600 of an interval's 2000 cycles on a walk
// with branches per step, no MFMA beside it; dK/dV of a training step, d = 128: 65536 lognormal tokens, 32/8 heads, dS kept 5183 ->
// 5005 us; 32768 tokens, 64/8 heads 4368 -> 4035).
// A dependency's record comes by a scalar load, requested when the one before it is done with, one step or more before its use: a
// vector load requested on use waited for the tile loads in flight too, and runs of one step were slower than in that walk
// (8192 tokens in 32-token blocks, 16 heads, d = 64, dS kept: that walk 326 us, a vector load on use 365, so 313; recomputing 283,
// 304, 276; packed blocks of 16-256 tokens, d = 64: 309, 317, 304).
struct RunIter {
  const BwdDep* deps;
  int dep, n_deps, hh, group, first_diag;
  int q0, left, last_rows;      // of the run: first row of its first step, steps not yet passed, rows of its last step
  BwdDep cur;
  __device__ __forceinline__ void init(const BwdDep* d, const BwdItem& it, int group_) {
    deps = d + it.dep_begin; dep = 0; n_deps = it.n_deps; hh = 0; group = group_; first_diag = it.tile_off & ~31;
    cur = it.first;
    q0 = 0; left = 0; last_rows = 0;
  }
  // The next run (cur, head hh of the group), or false behind the last one.  ahead() follows once cur and hh have been used.
  __device__ __forceinline__ bool next() {
    left = 0;
    if (dep >= n_deps) return false;
    q0 = (cur.kind & 1) ? first_diag : 0;
    left = (cur.q_len - q0 + 31) / 32;
    last_rows = cur.q_len - q0 - 32 * (left - 1);
    return true;
  }
  __device__ __forceinline__ void ahead() {
    if (++hh < group) return;
    hh = 0;
    if (++dep < n_deps) {
      // the constant address space makes the load a scalar one: no kernel writes the table
      const u32x4 r = *(const __attribute__((address_space(4))) u32x4*)(uintptr_t)(deps + dep);
      cur = BwdDep{(int)r[0], (int)r[1], (int)r[2], (int)r[3]};
    }
  }
};

constexpr int kDkdvBufs = 7;        // ring of LDS step buffers
constexpr int kNoMask = 1 << 30;    // diagonal threshold of a step that needs no mask

// JOINED: the problem has packed blocks, so items may be joined runs.  Only that instance masks by member: compiled into the
// other one, the third form of the interval took registers from the other two (8-worker share, d = 128, without SPILL: 5441 ->
// 5607 us).
template <int D, bool GRAD_BF16, bool SPILL, bool JOINED>
__global__ void __launch_bounds__(512, 2) dkdv_kernel(BwdArgs a) {
  constexpr int KC = D / 16;
  constexpr int DT = D / 32;
  constexpr int NS = 2 * KC;                 // MFMAs per wave and step (= 4 * DT)
  constexpr int PFC = 4;                     // consumer: an LDS operand is requested this many MFMAs before its use
  constexpr int PFP = 4;                     // producer
  constexpr int TB = tile_bytes<D>(32);
  constexpr int BUF = 2 * TB;                // [Q tile | dO tile]
  constexpr int NB = kDkdvBufs;
  constexpr int CPR = D / 8, RPI = 64 / CPR, NDMA = 32 / RPI / 4;   // LDS-DMA geometry, see issue()
  constexpr int DMA_PER_STEP = 2 * NDMA + 1;                        // instructions per consumer wave and step
  __shared__ __attribute__((aligned(1024))) unsigned char lds_t[NB][BUF];
  __shared__ __attribute__((aligned(1024))) unsigned char lds_h[2][4][4096];   // [parity][KV sub-tile][operand][lane] 16 B
  __shared__ __attribute__((aligned(256))) float lds_sc[NB][64];   // [LSE*log2e x 32 | D*scale x 32]
  __shared__ int s_next;
  __shared__ __attribute__((aligned(16))) int32_t s_rec[64];       // next item's record, as in fwd_kernel
  __shared__ int s_klo[JOINED ? 256 : 1], s_khi[JOINED ? 256 : 1];   // joined run: the query rows of the member of each producer lane's KV row, minus 4g
  __shared__ __attribute__((aligned(16))) unsigned char s_stage[4][kStageBytes];   // producers at an item's start, consumers at its end

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
  const int sub = wave & 3;
  const bool consumer = wave >= 4;
  const int l32 = lane & 31, g = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D;
  const int64_t kv_row_stride = (int64_t)a.n_kv_heads * D;
  const unsigned char* zeros = reinterpret_cast<const unsigned char*>(a.hdr->zeros);
  const float* infs = a.hdr->infs;
  const uint32_t lds_sc0 = lds_addr(lds_sc[0]);
  const uint32_t lds_h0 = lds_addr(lds_h[0][sub]) + lane * 16;

  // The two steps before the first one of the first item must contribute nothing: zero into the two tile buffers and the
  // hand-over buffer they read, +inf / 0 into the scalars.
  for (int i = tid * 16; i < 2 * BUF; i += 512 * 16)
    *reinterpret_cast<u32x4*>(&lds_t[NB - 2][0] + i) = u32x4{0, 0, 0, 0};
  for (int i = tid * 16; i < 4 * 4096; i += 512 * 16)
    *reinterpret_cast<u32x4*>(&lds_h[0][0][0] + i) = u32x4{0, 0, 0, 0};
  for (int i = tid; i < NB * 64; i += 512) lds_sc[0][i] = (i & 32) ? 0.f : INFINITY;
  // Ring positions, advanced by one buffer per step and kept across items.  In interval i the
  // consumer transposes tile i (b_c), the producer reads the rows of tile i+2 and the scalars of
  // step i+1 (b_p, b_s), and the consumers request tile i+6 (b_dma).  A tile is in place (landed
  // and published by a barrier) two intervals before the producer's interval, so both roles can
  // request their first LDS operands of an interval before the barrier that opens it.
  int b_c = NB - 2, b_p = 0, b_s = NB - 1, b_dma = 4, hb = 0;
  ItemStream items;             // of wave 4, a consumer: the producers have no register to spare
  if (wave == 4) {
    const int first = items.start(a.hdr->bwd_counter, a.hdr->bwd_begin, lane);
    if (first >= 0) fetch_item(a.items, first, s_rec, lane);
    if (lane == 0) s_next = first;
    dma_wait();
  }
  __syncthreads();
  while (__builtin_amdgcn_readfirstlane(s_next) >= 0) {
    const BwdItem it = read_item<BwdItem>(s_rec);
    const int my_kv = sub * 32 + l32;                  // KV row inside the tile
    const bool kv_ok = my_kv < it.kv_rows;
    const int n_iv = it.n_iv;                          // barrier intervals of the item
    RunIter run;                                       // consumer: the step to load; producer: the step of the next B
    run.init(a.deps, it, group);

    if (consumer) {
      // =============================== consumer ===============================
      const int cw = sub;     // index among the four loading waves
      // LDS-DMA of a 32-row tile: instruction n of this wave fills LDS rows r_n = (4n + cw) * RPI + lane / CPR.
      // A lane fetches chunk (pc ^ swz(r_n)) of global row min(r_n, valid - 1): rows past a ragged end
      // repeat the last valid row (finite values; their P is 0 because their LSE is +inf).
      uint32_t dma_row[NDMA], dma_chunk[NDMA];
#pragma unroll
      for (int n = 0; n < NDMA; n++) {
        const int r = (4 * n + cw) * RPI + lane / CPR, pc = lane % CPR;
        dma_row[n] = (uint32_t)(r * q_row_stride * 2);
        dma_chunk[n] = (uint32_t)((pc ^ swz<D>(r)) << 4);
      }
      // scalars: lanes 0-31 fetch LSE*log2e of row lane, lanes 32-63 D*scale of row lane-32
      const float* sc_arr = (g ? a.dls : a.lse2) + l32;
      const float* sc_page = (g ? reinterpret_cast<const float*>(zeros) : infs) + l32;
      const int tr_row = (lane & 15) >> 2, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      // This wave owns d rows 32*cdt .. +31 of dK^T / dV^T for NN of the tile's 32-row KV groups.
      constexpr int NN = DT;
      const int cdt = sub % DT, n0 = (sub / DT) * NN;
      uint32_t tr_lo1 = lds_addr(lds_t[0]) + b_c * BUF + tile_off<D>(4 * g + tr_row, 4 * cdt + (tr_col >> 3)) + (tr_col & 4) * 2;
      uint32_t tr_hi1 = lds_addr(lds_t[0]) + b_c * BUF + tile_off<D>(4 * g + tr_row + 8, 4 * cdt + (tr_col >> 3)) + (tr_col & 4) * 2;
      const uint32_t hsrc = lds_addr(lds_h[0][0]) + n0 * 4096 + lane * 16;
      f32x16 acc_k[DT], acc_v[DT];     // dK^T, dV^T: rows = d, cols = KV rows
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) { acc_k[dt][r] = 0.f; acc_v[dt][r] = 0.f; }

      // The load of one step in two parts.  describe(): scalar bookkeeping with branches, run at a
      // step boundary.  issue(): branch-free, sits between the MFMAs of the step.
      uint64_t d_q = 0, d_do = 0;          // tile sources (first row of the step)
      uint32_t d_lim = 0;                  // byte offset of the last valid row
      int d_valid = 0;
      int64_t d_sc = 0;                    // element offset of the step's first row in the head-major scalars
      const uint32_t row_bytes = (uint32_t)(q_row_stride * 2), lim_whole = 31 * row_bytes;
      uint32_t lim_last = 0;
      auto describe = [&]() {
        if (__builtin_expect(run.left > 1, 1)) {
          // the next 32 rows of the same run: only its last step may be ragged
          run.left--;
          d_q += 32 * (uint64_t)row_bytes; d_do += 32 * (uint64_t)row_bytes; d_sc += 32;
          d_valid = run.left > 1 ? 32 : run.last_rows;
          d_lim = run.left > 1 ? lim_whole : lim_last;
        } else if (run.next()) {
          const int head = it.kv_head * group + run.hh;
          const int64_t row = (int64_t)(run.cur.q_start + run.q0);
          d_q = reinterpret_cast<uint64_t>(a.q + row * q_row_stride + (int64_t)head * D);
          d_do = reinterpret_cast<uint64_t>(a.d_o + row * q_row_stride + (int64_t)head * D);
          d_sc = (int64_t)head * a.t_q + row;
          lim_last = (uint32_t)(run.last_rows - 1) * row_bytes;
          d_valid = run.left > 1 ? 32 : run.last_rows;
          d_lim = run.left > 1 ? lim_whole : lim_last;
          run.ahead();
        } else {
          d_q = reinterpret_cast<uint64_t>(zeros); d_do = d_q; d_lim = 0; d_valid = 0; d_sc = 0;
        }
      };
      auto issue = [&]() {
        const uint32_t lbase = lds_addr(lds_t[0]) + b_dma * BUF;
#pragma unroll
        for (int n = 0; n < NDMA; n++) {
          const uint32_t voff = min(dma_row[n], d_lim) + dma_chunk[n];
          lds_dma16_s(reinterpret_cast<const unsigned char*>(d_q), voff, lbase + (4 * n + cw) * 1024);
          lds_dma16_s(reinterpret_cast<const unsigned char*>(d_do), voff, lbase + TB + (4 * n + cw) * 1024);
        }
        // all four loading waves fetch the 64 scalars (same values, same place): they then have
        // the same number of loads in flight
        const float* sp = (l32 < d_valid) ? sc_arr + d_sc : sc_page;
        lds_dma4(sp, lds_sc0 + b_dma * 256);
        b_dma = (b_dma == NB - 1) ? 0 : b_dma + 1;
      };
      // prologue: tiles 0 .. 3 into the four buffers before the next one to load
      b_dma = (b_dma + NB - 4) % NB;
#pragma unroll
      for (int i = 0; i < 4; i++) { describe(); issue(); }
      describe();          // tile 4, requested inside the first interval
      dma_wait();
      __syncthreads();
      // A operands of a step: (k-chunk j of 16 query rows, w = 0: dO^T for dV, 1: Q^T for dK), index 2j + w.
      // Each serves the NN MFMAs of its KV groups; the B operands (P / dS of every group) stream from the
      // hand-over buffers, PFC MFMAs ahead.  While interval i runs, the A operands of step i+1 are fetched
      // from the next tile as soon as their registers are free.
      auto fetch_a = [&](int jw) {
        const uint32_t o = 16 * (jw >> 1) * (D * 2) + ((jw & 1) == 0 ? TB : 0);
        return __builtin_bit_cast(u32x4, lds_tr_pair_at(tr_lo1 + o, tr_hi1 + o));
      };
      auto next_tile = [&]() {
        const int st = (b_c == NB - 1) ? -(NB - 1) * BUF : BUF;
        tr_lo1 += st; tr_hi1 += st;
        b_c = (b_c == NB - 1) ? 0 : b_c + 1;
      };
      u32x4 aop[4];
#pragma unroll
      for (int jw = 0; jw < 4; jw++) aop[jw] = fetch_a(jw);
      next_tile();
      // Down to 6 intervals before the end, to 2, to 0: a test for the next item in every interval costs long items 3-8 %
      // (14 query blocks of a 19429-token sequence, heads 3/1, d = 128: 1412 -> 1305 us).
      for (int iv = 0, left = 6; left >= 0; left = left == 6 ? 2 : left - 2) {
        for (; iv < n_iv - left; iv++) {
          const uint32_t hb_src = hsrc + hb * (4 * 4096);
          // MFMA u = (2j + w) * NN + n reads operand (w ? 2 : 0) + j of KV group n0 + n
          auto fetch_b = [&](int u) {
            const int jw = u / NN, n = u % NN;
            return lds_read16(hb_src + n * 4096 + (((jw & 1) ? 2 : 0) + (jw >> 1)) * 1024);
          };
          u32x4 bop[PFC];
#pragma unroll
          for (int u = 0; u < PFC; u++) bop[u] = fetch_b(u);
#pragma unroll
          for (int u = 0; u < NS; u++) {
            const int jw = u / NN, n = u % NN;
            if ((jw & 1) == 0) acc_v[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(aop[jw]), as_bf16x8(bop[u % PFC]), acc_v[n], 0, 0, 0);
            else acc_k[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(aop[jw]), as_bf16x8(bop[u % PFC]), acc_k[n], 0, 0, 0);
            if (u + PFC < NS) bop[u % PFC] = fetch_b(u + PFC);
            if (n == NN - 1) aop[jw] = fetch_a(jw);
            // Early in the interval: dK/dV of an 8-worker share (32/8 heads, d = 128) takes 5700 us with the loads behind the 9th of
            // the 16 MFMAs, 5640 behind the 7th, 5564 the 5th, 5578 the 3rd, 5510 the 2nd.
            if (u == 1) issue();
            __builtin_amdgcn_sched_barrier(0);
          }
          next_tile();
          __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * DMA_PER_STEP) & 15) | (((2 * DMA_PER_STEP) >> 4) << 14));
          asm volatile("s_barrier" ::: "memory");
          describe();
          hb ^= 1;
        }
        if (wave == 4) {                 // the next item (every wave has read this one's record)
          if (left == 6) items.request(lane);
          if (left == 2) {
            const int nx = items.take(lane);
            if (lane == 0) s_next = nx;
            if (nx >= 0) fetch_item(a.items, nx, s_rec, lane);
          }
        }
      }
      b_c = (b_c == 0) ? NB - 1 : b_c - 1;     // the tile looked ahead to belongs to the next item's first interval
      dma_wait();
      // ---- epilogue: the only writer of these dK / dV elements
#pragma unroll
      for (int n = 0; n < NN; n++) {
        const int64_t off = (int64_t)(it.kv_start + (n0 + n) * 32) * kv_row_stride + (int64_t)it.kv_head * D + cdt * 32;
        constexpr int ES = GRAD_BF16 ? 2 : 4;
        store_tile<GRAD_BF16>(static_cast<unsigned char*>(a.dk) + off * ES, kv_row_stride, it.kv_rows - (n0 + n) * 32, acc_k[n], 1.0f, s_stage[sub], lane);
        store_tile<GRAD_BF16>(static_cast<unsigned char*>(a.dv) + off * ES, kv_row_stride, it.kv_rows - (n0 + n) * 32, acc_v[n], 1.0f, s_stage[sub], lane);
      }
    } else {
      // =============================== producer ===============================
      int kvg = it.tile_off + my_kv - 4 * g;       // masked iff kvg > q0 + 8*(r/4) + r%4 on a DIAG step
      const bool joined = JOINED && (it.first.kind & 2);
      if (joined) {
        // Joined run: a KV row is seen by the query rows of its own member only, from the first of them on under a full mask,
        // from the row itself under a causal one (as above).
        const int sg = kv_ok ? a.q_seg[it.first.q_start + it.tile_off + my_kv] : 0;
        s_klo[tid] = kv_ok ? (sg & 0xff) - 4 * g : 0x7fff0000;
        s_khi[tid] = (sg >> 8) + 1 - 4 * g;
      }
      // SPILL: the dS this wave forms also goes to memory, one 2 KB fragment per step, for the dQ pass.  There a
      // KV row past the ragged end of the tile must carry dS = 0 (here its column of dK^T / dV^T is simply never
      // stored): such lanes get a KV row that no threshold lets pass, and a ragged tile runs every step through the masked
      // variant.  Fragment layout, shared with dq_ds_kernel: the 16 bytes that lane (KV row r = lane % 32,
      // g = lane / 32) holds for j = 0, 1 (query rows 16j + 4g + {0..3} and 16j + 8 + 4g + {0..3} of the step)
      // sit at byte 1024 j + 512 g + 16 ((r + 8 j + 4 g) % 32): every store instruction writes 1 KB of consecutive
      // memory, and the rotation makes the transposing LDS reads of the dQ pass bank-conflict free.
      if constexpr (SPILL) { if (!kv_ok) kvg = 0x7fff0000; }
      // a step whose first query row is below this one is masked: the diagonal rows that this wave's last KV row does not reach
      // need none
      const int mask_below = (SPILL && it.kv_rows < kBwdTileN) ? kNoMask + 1 : it.tile_off + sub * 32 + 31;
      const int kv0 = it.tile_off + sub * 32;              // the wave's first KV row inside the segment
      const int frag_from = sub * 32 < it.kv_rows ? kv0 : 0x7fffffff;   // first query row whose step has a fragment under a causal mask
      const int sink = (int)(blockIdx.x & (kDsSinkFrags - 1));
      int frag_t = sink, d_frag = 0;   // fragment of the step that B handles in this interval; its increment inside a run
      uint32_t sp_off[2];
#pragma unroll
      for (int j = 0; j < 2; j++) sp_off[j] = 1024 * j + 512 * g + 16 * ((l32 + 8 * j + 4 * g) & 31);
      // B operands of S and dP: this pair's K and V rows; lane = KV row, 8 consecutive d per k-chunk.
      bf16x8 kf[KC], vf[KC];
      {
        const int64_t off = (int64_t)it.kv_start * kv_row_stride + (int64_t)it.kv_head * D;
        load_rows<D>(kf, a.k + off, kv_row_stride, sub * 32, it.kv_rows, s_stage[sub], lane);
        load_rows<D>(vf, a.v + off, kv_row_stride, sub * 32, it.kv_rows, s_stage[sub], lane);
      }
      uint32_t row_a[KC];        // row-read addresses inside the step buffer of tile i+2 (Q tile; dO is +TB)
#pragma unroll
      for (int kc = 0; kc < KC; kc++) row_a[kc] = lds_addr(lds_t[0]) + b_p * BUF + tile_off<D>(l32, 2 * kc + g);
      uint32_t sc_a = lds_sc0 + b_s * 256 + 16 * g;      // scalars of step i+1: rows 8*q4 + 4g .. +3 at +32*q4, D*scale at +128
      int thr_t = kNoMask, d_thr = 0;     // diagonal threshold of the step that B handles in this interval
      int causal_t = 0;          // 1: the run of that step is causal (a row group then keeps one fragment more than the one before it)
      f32x16 s_a, dp_a, s_b, dp_b;
#pragma unroll
      for (int r = 0; r < 16; r++) { s_a[r] = 0.f; dp_a[r] = 0.f; s_b[r] = 0.f; dp_b[r] = 0.f; }
      dma_wait();          // K / V fragments
      __syncthreads();     // the prologue's tiles are in place
      // requested before an interval starts: its first PFP row operands and its first four scalars
      u32x4 op[PFP];
#pragma unroll
      for (int k = 0; k < PFP; k++) op[k] = lds_read16(row_a[k / 2] + ((k & 1) ? TB : 0));
      f32x4 lse_n = __builtin_bit_cast(f32x4, lds_read16(sc_a)), dl_n = __builtin_bit_cast(f32x4, lds_read16(sc_a + 128));

      // One interval: MFMAs of A(i+2) into (sn, dpn); B(i+1) on (sc, dpc) between them.
      auto interval = [&](auto masked, f32x16& sc, f32x16& dpc, f32x16& sn, f32x16& dpn) {
        constexpr int MASK = decltype(masked)::value;     // 0: no mask, 1: diagonal / ragged end, 2: joined run
        const int thr_s = __builtin_amdgcn_readfirstlane(thr_t);
        int klo = kvg, hlim = 0;                          // joined run: rows 8*(r/4) + r%4 >= hlim of the step are past the member
        if constexpr (MASK == 2) {
          hlim = s_khi[tid] - thr_s;
          if (!causal_t) klo = s_klo[tid];
        }
        f32x4 lse_c = lse_n, dl_c = dl_n;      // scalars of rows 8*q4 + 4g .. +3, one group of four ahead
        uint32_t pk[16];           // [0..7] P pairs, [8..15] dS pairs: four B operands for the consumer
        float p_prev = 0.f, ds_prev = 0.f;
        const uint32_t hdst = lds_h0 + (hb ^ 1) * (4 * 4096);
        unsigned char* fptr = nullptr;
        // no fragment: KV rows past the tile's end, above the diagonal
        if constexpr (SPILL) fptr = a.ds + (int64_t)__builtin_amdgcn_readfirstlane((JOINED && !causal_t ? kNoMask : thr_t) >= frag_from ? frag_t : sink) * kDsFragBytes;
        float p_ahead = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0], a.scale_log2, -lse_c[0]));
#pragma unroll
        for (int k = 0; k < NS; k++) {
          const int kc = k / 2;
          if (k == 0) {
#pragma unroll
            for (int r = 0; r < 16; r++) { sn[r] = 0.f; dpn[r] = 0.f; }
          }
          if ((k & 1) == 0) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[k % PFP]), kf[kc], sn, 0, 0, 0);
          else dpn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[k % PFP]), vf[kc], dpn, 0, 0, 0);
          if (k == NS - PFP) {
            // the last row operand of this tile has been requested: move on to the next tile
            const int st = (b_p == NB - 1) ? -(NB - 1) * BUF : BUF;
#pragma unroll
            for (int kc2 = 0; kc2 < KC; kc2++) row_a[kc2] += st;
            b_p = (b_p == NB - 1) ? 0 : b_p + 1;
          }
          {
            const int kk = (k + PFP) % NS;
            op[k % PFP] = lds_read16(row_a[kk / 2] + ((kk & 1) ? TB : 0));
          }
          // vector work: 16 / NS score registers per slot
#pragma unroll
          for (int r = k * 16 / NS; r < (k + 1) * 16 / NS; r++) {
            if ((r & 3) == 0) {
              if (r > 0) { lse_c = lse_n; dl_c = dl_n; }
              if (r == 12) {
                // the scalars of the next interval's first four rows
                sc_a += (b_s == NB - 1) ? -(NB - 1) * 256 : 256;
                b_s = (b_s == NB - 1) ? 0 : b_s + 1;
                lse_n = __builtin_bit_cast(f32x4, lds_read16(sc_a));
                dl_n = __builtin_bit_cast(f32x4, lds_read16(sc_a + 128));
              } else {
                lse_n = __builtin_bit_cast(f32x4, lds_read16(sc_a + 32 * ((r >> 2) + 1)));
                dl_n = __builtin_bit_cast(f32x4, lds_read16(sc_a + 32 * ((r >> 2) + 1) + 128));
              }
            }
            // the exponential of the NEXT register is issued before this register is finished, so
            // its latency does not sit in a dependent chain (the wave issues in order)
            float p = p_ahead;
            if (r + 1 < 16) {
              const float lse_q = ((r + 1) & 3) ? lse_c[(r + 1) & 3] : lse_n[0];
              p_ahead = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r + 1], a.scale_log2, -lse_q));
            }
            const float dl_r = dl_c[r & 3];
            if constexpr (MASK == 1) p = (kvg > thr_s + 8 * (r >> 2) + (r & 3)) ? 0.f : p;
            if constexpr (MASK == 2) p = (klo > thr_s + 8 * (r >> 2) + (r & 3) || 8 * (r >> 2) + (r & 3) >= hlim) ? 0.f : p;
            const float ds = p * __builtin_fmaf(dpc[r], a.scale, -dl_r);
            if (r & 1) {
              pk[r >> 1] = pack_bf16(p_prev, p); pk[8 + (r >> 1)] = pack_bf16(ds_prev, ds);
              // keeps the vector work between the MFMAs it was written between
              asm volatile("" :: "v"(pk[r >> 1]), "v"(pk[8 + (r >> 1)]));
            } else { p_prev = p; ds_prev = ds; }
            if ((r & 7) == 7) {
              // rows 8*(r/8) .. r done: one P operand and one dS operand (k-chunk r/8)
              const int j = r >> 3;
              const u32x4 wp = {pk[4 * j], pk[4 * j + 1], pk[4 * j + 2], pk[4 * j + 3]};
              const u32x4 wd = {pk[8 + 4 * j], pk[8 + 4 * j + 1], pk[8 + 4 * j + 2], pk[8 + 4 * j + 3]};
              *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(hdst + j * 1024) = wp;
              *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(hdst + (2 + j) * 1024) = wd;
              if constexpr (SPILL) *reinterpret_cast<u32x4*>(fptr + sp_off[j]) = wd;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (SPILL) {
          // the hand-over writes must have landed; the fragment stores need not (a full fence would wait for them)
          __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
          asm volatile("s_barrier" ::: "memory");
        } else {
          __syncthreads();
        }
        // the step that B handles next
        if (__builtin_expect(run.left > 1, 1)) {
          run.left--;
          thr_t += d_thr;
          if constexpr (SPILL) { frag_t += d_frag; d_frag += causal_t; }
        } else if (run.next()) {
          thr_t = run.cur.kind != FCP_KIND_FULL ? run.q0 : kNoMask;
          d_thr = run.cur.kind != FCP_KIND_FULL ? 32 : 0;
          if constexpr (SPILL || JOINED) causal_t = run.cur.kind & 1;
          if constexpr (SPILL) {
            const int q32 = run.q0 >> 5, nq32 = (run.cur.q_len + 31) >> 5, nkv32 = (it.kv_blk_len + 31) >> 5, head = it.kv_head * group + run.hh;
            frag_t = run.cur.ds_frag + (kv0 >> 5) + (causal_t ? head * (nq32 * (nq32 + 1) / 2) + q32 * (q32 + 1) / 2 : (head * nq32 + q32) * nkv32);
            d_frag = causal_t ? q32 + 1 : nkv32;
          }
          run.ahead();
        } else {
          thr_t = kNoMask; d_thr = 0;
          frag_t = sink; d_frag = 0; causal_t = 0;
        }
        hb ^= 1;
      };
      // the first interval handles B(-1) (nothing) and A(0), the second B(0) and A(1), ...
      const std::integral_constant<int, 0> no_mask;
      const std::integral_constant<int, 1> with_mask;
      const std::integral_constant<int, 2> member_mask;
      if (joined) {
        // every step masked by member; outside the item's steps thr_t names no row at all, which masks everything
        for (int iv = 0; iv < n_iv; iv += 2) {
          interval(member_mask, s_a, dp_a, s_b, dp_b);
          interval(member_mask, s_b, dp_b, s_a, dp_a);
        }
      } else {
        for (int iv = 0; iv < n_iv; iv += 2) {
          if (thr_t < mask_below) interval(with_mask, s_a, dp_a, s_b, dp_b); else interval(no_mask, s_a, dp_a, s_b, dp_b);
          if (thr_t < mask_below) interval(with_mask, s_b, dp_b, s_a, dp_a); else interval(no_mask, s_b, dp_b, s_a, dp_a);
        }
      }
    }
    __syncthreads();
  }
  if (wave == 4 && lane == 0) retire(a.hdr->bwd_counter, &a.hdr->bwd_done);
}

// =====================================================================================
// Backward, part 2 -- dQ.  Query-stationary like the forward and with the same item shape (two
// 128-row query sub-tiles that share a KV head, here over all pairs of the query block); 8 waves
// share one double-buffered stream of [K | V] tiles; lane = query row.
//   S^T = K Q^T, dP^T = V dO^T       (A = K / V rows from LDS, B = Q / dO fragments in registers)
//   P^T = exp2(S^T*c - LSE*log2e), dS^T = P^T o (dP^T - D) * scale     (LSE, D per lane)
//   dQ^T += K^T dS^T                 (A = K by transpose reads, B = accumulator registers)
// Columns past the diagonal or past a ragged end get P = 0.  Every dQ row has one writer: plain
// stores, deterministic.
// =====================================================================================
// JOINED as in dkdv_kernel (8-worker share, d = 128: 3687 -> 3734 us with both masks in one instance).
template <int D, bool WITH_D, bool GRAD_BF16, bool JOINED>
__global__ void __launch_bounds__(512, 2) dq_kernel(BwdArgs a) {
  constexpr int KC = D / 16;
  constexpr int DT = D / 32;
  constexpr int TB = tile_bytes<D>(kFwdTileN);
  __shared__ __attribute__((aligned(1024))) unsigned char lds_kv[2][2 * TB];   // [buffer][K tile | V tile]
  __shared__ __attribute__((aligned(16))) int32_t s_rec[64];   // next item's record, as in fwd_kernel
  __shared__ int s_next;
  __shared__ __attribute__((aligned(16))) unsigned char s_stage[8][kStageBytes];
  __shared__ uint16_t s_seg[JOINED ? 512 : 1];   // joined run: member bounds of each lane's query row, as in fwd_kernel

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
  const int sub = wave >> 2;
  const int l32 = lane & 31, g = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D;
  const int64_t kv_row_stride = (int64_t)a.n_kv_heads * D;
  const unsigned char* zeros = reinterpret_cast<const unsigned char*>(a.hdr->zeros);
  const uint32_t dma_off = dma_lane_offset<D>(wave, lane, kv_row_stride);
  const int tr_row = (lane & 15) >> 2, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  // absolute LDS addresses into the K tile of the CURRENT buffer (V = +TB), switched in place
  uint32_t tr_lo[DT], tr_hi[DT], row_off[KC];
#pragma unroll
  for (int dt = 0; dt < DT; dt++) {
    tr_lo[dt] = lds_addr(lds_kv[0]) + tile_off<D>(4 * g + tr_row, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
    tr_hi[dt] = lds_addr(lds_kv[0]) + tile_off<D>(4 * g + tr_row + 8, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
  }
#pragma unroll
  for (int kc = 0; kc < KC; kc++) row_off[kc] = lds_addr(lds_kv[0]) + tile_off<D>(l32, 2 * kc + g);
  int buf = 0;                              // buffer the addresses above point into
  auto switch_buffer = [&]() {
    const int step = buf ? -2 * TB : 2 * TB;
#pragma unroll
    for (int dt = 0; dt < DT; dt++) { tr_lo[dt] += step; tr_hi[dt] += step; }
#pragma unroll
    for (int kc = 0; kc < KC; kc++) row_off[kc] += step;
    buf ^= 1;
  };

  ItemStream items;
  if (wave == 0) {
    const int first = items.start(a.hdr->dq_counter, a.hdr->dq_begin, lane);
    if (first >= 0) fetch_item(a.dq_items, first, s_rec, lane);
    if (lane == 0) s_next = first;
    dma_wait();
  }
  __syncthreads();
  int item_idx = __builtin_amdgcn_readfirstlane(s_next);   // wave-uniform
  while (item_idx >= 0) {
    const QItem it = read_item<QItem>(s_rec);
    const bool four = it.head[1] - it.head[0] == 3;
    const int wq = four ? (wave & 1) ^ sub : sub ? 3 - (wave & 3) : wave & 3;      // 32-row group inside the sub-item (order: see fwd_kernel)
    const int q_start = (sub ? it.q_start[1] : it.q_start[0]), q_rows = (sub ? it.q_rows[1] : it.q_rows[0]), tile_off_q = (sub ? it.tile_off[1] : it.tile_off[0]), head = four ? it.head[0] + (wave >> 1) : (sub ? it.head[1] : it.head[0]);
    const int kvh = it.head[0] / group;
    const int my_row = wq * 32 + l32;
    const bool row_ok = my_row < q_rows;
    const bool wave_ok = wq * 32 < q_rows;                   // the wave has at least one valid row
    const int wave_row_lo = tile_off_q + wq * 32;
    const uint16_t* kbase = a.k + (int64_t)kvh * D;
    const uint16_t* vbase = a.v + (int64_t)kvh * D;

    if (JOINED) s_seg[tid] = row_ok ? a.q_seg[q_start + my_row] : (uint16_t)0;
    bf16x8 qf[KC], dof[KC];
    float lse_l = INFINITY, dl_l = 0.f;     // rows past the end: P = exp2(-inf) = 0
    {
      const int64_t row0 = (int64_t)q_start * q_row_stride + (int64_t)head * D;
      load_rows<D>(qf, a.q + row0, q_row_stride, wq * 32, q_rows, s_stage[wave], lane);
      load_rows<D>(dof, a.d_o + row0, q_row_stride, wq * 32, q_rows, s_stage[wave], lane);
      const int64_t off = (int64_t)(q_start + my_row) * q_row_stride + (int64_t)head * D + 8 * g;
      if constexpr (WITH_D) {
        // D = rowsum(dO o O) of this lane's row: its 8 columns of every k-chunk, plus the partner lane's
        // (lane ^ 32, same row, the other 8).  The backward preprocess pass is then not needed: the two
        // per-row scalars are written here, head-major, for the dK/dV kernel that runs afterwards.
        float part = 0.f;
        if (row_ok) {
          // all loads of the row first, then the arithmetic: one round trip to memory, not one per k-chunk
          auto dot8 = [&](const u32x4 dv, const float (&ov)[8]) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
              part += __uint_as_float(dv[i] << 16) * ov[2 * i];
              part += __uint_as_float(dv[i] & 0xffff0000u) * ov[2 * i + 1];
            }
          };
          if (a.o_is_f32) {
            const float* op = reinterpret_cast<const float*>(a.o) + off;
            f32x4 x[2 * KC];
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
              x[2 * kc] = *reinterpret_cast<const f32x4*>(op + kc * 16);
              x[2 * kc + 1] = *reinterpret_cast<const f32x4*>(op + kc * 16 + 4);
            }
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
              const float ov[8] = {x[2 * kc][0], x[2 * kc][1], x[2 * kc][2], x[2 * kc][3], x[2 * kc + 1][0], x[2 * kc + 1][1], x[2 * kc + 1][2], x[2 * kc + 1][3]};
              dot8(__builtin_bit_cast(u32x4, dof[kc]), ov);
            }
          } else {
            const uint16_t* op = reinterpret_cast<const uint16_t*>(a.o) + off;
            u32x4 x[KC];
#pragma unroll
            for (int kc = 0; kc < KC; kc++) x[kc] = *reinterpret_cast<const u32x4*>(op + kc * 16);
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
              float ov[8];
#pragma unroll
              for (int i = 0; i < 4; i++) { ov[2 * i] = __uint_as_float(x[kc][i] << 16); ov[2 * i + 1] = __uint_as_float(x[kc][i] & 0xffff0000u); }
              dot8(__builtin_bit_cast(u32x4, dof[kc]), ov);
            }
          }
        }
        const float d_row = part + xor32(part);
        if (row_ok) {
          const float l = a.lse[(int64_t)(q_start + my_row) * a.n_q_heads + head];
          lse_l = (l == -INFINITY) ? INFINITY : l * kLog2e;
          dl_l = d_row * a.scale;
          if (g == 0) {
            const int64_t hr = (int64_t)head * a.t_q + q_start + my_row;
            a.lse2_out[hr] = lse_l;
            a.dls_out[hr] = dl_l;
          }
        }
      } else if (row_ok) {
        const int64_t hr = (int64_t)head * a.t_q + q_start + my_row;
        lse_l = a.lse2[hr];
        dl_l = a.dls[hr];
      }
    }
    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[dt][r] = 0.f;

    TileIter ti;
    ti.init(a.pairs, it);
    auto dma = [&](int b) {
      const int64_t row0 = (int64_t)(ti.cur.kv_start + ti.c0) * kv_row_stride;
      // Only the waves of sub-item 0 load: they reach every tile barrier well before the others (the SIMD
      // favours the wave that was started first), so the loads cost them nothing and relieve the slower four.
      if (sub == 0) {
        tile_dma<D, kFwdTileN, 4>(lds_kv[b], kbase + row0, kv_row_stride, ti.cur.kv_len - ti.c0, zeros, wave, lane, dma_off);
        tile_dma<D, kFwdTileN, 4>(lds_kv[b] + TB, vbase + row0, kv_row_stride, ti.cur.kv_len - ti.c0, zeros, wave, lane, dma_off);
      }
    };
    DevPair tp = ti.cur;
    int tc0 = 0;
    if (ti.more) { dma(buf); ti.advance(); }
    int left = it.n_tiles;
    dma_wait();
    __syncthreads();
    auto next_item = [&]() {             // wave 0, see fwd_kernel
      const int nx = items.take(lane);
      if (lane == 0) s_next = nx;
      if (nx >= 0) fetch_item(a.dq_items, nx, s_rec, lane);
    };
    if (left == 0) {                     // no tile barrier to publish the next item
      if (wave == 0) { items.request(lane); next_item(); }
      dma_wait();
      __syncthreads();
    }
    // Down to 3 tiles, to 1, to 0: a test for the next item at every tile costs long items 3-5 % (end of a 103755-token
    // sequence, 2 heads, d = 128: 2267 -> 2161 us).
    for (int stop = 3; stop >= 0; stop = stop == 3 ? 1 : stop - 1) {
      for (; left > stop; left--) {
        const DevPair np = ti.cur;
        const int nc0 = ti.c0;
        const bool nhave = ti.more;
        if (nhave) { dma(buf ^ 1); ti.advance(); }

        const bool diag = (tp.kind & 1) != 0;
        if (wave_ok && !(diag && tc0 > wave_row_lo + 31)) {      // else nothing visible for this wave
          // wave-uniform: tiles that straddle the diagonal, and tiles that hold a ragged end (their K rows past
          // the end are zero in LDS, but S = 0 there still gives P = exp2(-LSE), which overflows for a row whose
          // logits are all strongly negative; inf * 0 would then poison the whole dQ row)
          const bool joined = JOINED && (tp.kind & 2);
          const bool need_mask = joined || (diag && tc0 + kFwdTileN - 1 > wave_row_lo) || tc0 + kFwdTileN > tp.kv_len;
          int limit = diag ? tile_off_q + my_row : tp.kv_len - 1;            // last visible column for this lane
          int first = 0;                                                     // first one (a joined run: of the row's member)
          if (joined) {
            const int sg = s_seg[tid];
            first = sg & 0xff;
            limit = min(limit, sg >> 8);
          }
          // the two 32-row halves of the KV tile one after the other: half the live accumulators
#pragma unroll
          for (int rt = 0; rt < 2; rt++) {
            f32x16 s, dp;
#pragma unroll
            for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
            // All MFMAs of S, then those of dP with the exponentials of S between them, then those of dQ: the second half of dS
            // is formed between the MFMAs of the first.  S and dP in turn, as the operands come, left all 88 issue slots of
            // vector work without an MFMA of the same wave beside them; the other wave of the SIMD covered most of that, and power
            // bounds the rest: training step of 32768 tokens, 64/8 heads, d = 128 8899 -> 8827 us, 8-worker share 11941 -> 11877.
            // Operands: row chunks of K, then of V, four in flight; two of them are requested in front of the first MFMA, which
            // waits for one (with all four in front of it d = 64 is 4 % slower).
            constexpr int PFQ = 4;
            u32x4 op[PFQ];
            auto request = [&](int u) { op[u % PFQ] = lds_read16(row_off[u % KC] + rt * 32 * (D * 2) + (u < KC ? 0 : TB)); };
            request(0);
            request(1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 2 * KC; u++) {
              if (u < KC) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[u % PFQ]), qf[u], s, 0, 0, 0);
              else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(op[u % PFQ]), dof[u % KC], dp, 0, 0, 0);
              if (u == 0) { request(2); request(3); }
              if (u + PFQ < 2 * KC) request(u + PFQ);
              // from the second MFMA of dP on: the first one covers the wait for S
              if (u > KC) {
#pragma unroll
                for (int r = (u - KC - 1) * 16 / (KC - 1); r < (u - KC) * 16 / (KC - 1); r++) {
                  float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.scale_log2, -lse_l));
                  asm volatile("" : "+v"(p));        // keeps it between the MFMAs it was written between
                  s[r] = p;
                }
              }
              __builtin_amdgcn_sched_barrier(0);
            }
            if (need_mask) {                    // wave-uniform: only tiles that straddle the diagonal
#pragma unroll
              for (int r = 0; r < 16; r++) {
                const int c = tc0 + rt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (c > limit || (JOINED && c < first)) s[r] = 0.f;
              }
            }
            constexpr int PFT = 2;
            bf16x8 kt[PFT];
            u32x4 db[2];                        // dS^T as two B operands
            auto fetch = [&](int u) {
              const uint32_t rows = (rt * 32 + 16 * (u / DT)) * (D * 2);
              kt[u % PFT] = lds_tr_pair_at(tr_lo[u % DT] + rows, tr_hi[u % DT] + rows);
            };
            auto ds_pair = [&](int i) {
              const float x = s[2 * i] * __builtin_fmaf(dp[2 * i], a.scale, -dl_l), y = s[2 * i + 1] * __builtin_fmaf(dp[2 * i + 1], a.scale, -dl_l);
              db[i >> 2][i & 3] = pack_bf16(x, y);
              asm volatile("" :: "v"(db[i >> 2][i & 3]));
            };
#pragma unroll
            for (int u = 0; u < PFT; u++) fetch(u);
#pragma unroll
            for (int i = 0; i < 4; i++) ds_pair(i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 2 * DT; u++) {
              acc[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[u % PFT], as_bf16x8(db[u / DT]), acc[u % DT], 0, 0, 0);
              if (u + PFT < 2 * DT) fetch(u + PFT);
              if (u < DT) {
#pragma unroll
                for (int i = 4 + u * 4 / DT; i < 4 + (u + 1) * 4 / DT; i++) ds_pair(i);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        tp = np; tc0 = nc0;
        dma_wait();
        __syncthreads();
        switch_buffer();
      }
      if (wave == 0 && it.n_tiles > 0) {
        if (stop == 3) items.request(lane);
        if (stop == 1) next_item();
      }
    }
    {
      const int64_t off = (int64_t)(q_start + wq * 32) * q_row_stride + (int64_t)head * D;
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
        store_tile<GRAD_BF16>(static_cast<unsigned char*>(a.dq) + (off + dt * 32) * (GRAD_BF16 ? 2 : 4), q_row_stride, q_rows - wq * 32, acc[dt], 1.0f, s_stage[wave], lane);
    }
    item_idx = __builtin_amdgcn_readfirstlane(s_next);
  }
  if (tid == 0) retire(a.hdr->dq_counter, &a.hdr->dq_done);
}

// =====================================================================================
// Backward, part 2 without recomputation -- dQ from the dS fragments that dkdv_kernel<.., SPILL> left in memory.
// Same items as dq_kernel (two 128-row query sub-tiles that share a KV head, over all pairs of the query block);
// 8 waves, wave = (sub-item, 32-row query group).  Per 64-row KV tile:
//   dQ^T (d x 32 query rows) += K^T (d x 64) dS^T (64 x 32)
// A = K^T by transpose reads of the shared K tile; B = dS^T by transpose reads of the wave's own two fragments,
// which hold dS^T[kv][q] in the 8-byte pieces the producer wrote (4 consecutive query rows of one KV row) at
// rotated positions (see dkdv_kernel), so that a half-wave's 32 pieces cover the 64 banks once.  Both operands
// assign the 8 k-slots of lane half g to KV rows {4g..4g+3} and {8+4g..8+4g+3} of the 16-row chunk.
// The kernel is bound by the HBM stream of fragments (2 bytes per score entry and head against 2 d FLOPs), so the
// ring of three stages (K tile + 8 x 2 fragments each) is there to keep two stages of loads in flight, filled by
// LDS-DMA; one workgroup barrier per tile.  Nothing is masked here: dS is already zero wherever a score is masked,
// and fragments above a wave's diagonal or past a ragged end are skipped, not read.
// =====================================================================================
constexpr int kDqDsBufs = 3;

template <int D, bool GRAD_BF16>
__global__ void __launch_bounds__(512, 2) dq_ds_kernel(BwdArgs a) {
  constexpr int DT = D / 32;
  constexpr int TBK = tile_bytes<D>(kFwdTileN);
  constexpr int WDS = 2 * kDsFragBytes;               // a wave's two fragments of a tile
  constexpr int STAGE = TBK + 8 * WDS;
  constexpr int NB = kDqDsBufs;
  constexpr int CPR = D / 8, RPI = 64 / CPR, NDMA = kFwdTileN / RPI / 8;
  constexpr int DMA_PER_FRAG = kDsFragBytes / 1024;
  __shared__ __attribute__((aligned(1024))) unsigned char lds_st[NB][STAGE];
  __shared__ __attribute__((aligned(16))) int32_t s_rec[64];   // next item's record, as in fwd_kernel
  __shared__ int s_next;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = wave >> 2;
  const int l32 = lane & 31, g = lane >> 5;
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D;
  const int64_t kv_row_stride = (int64_t)a.n_kv_heads * D;
  // K tile loads: as in the forward (rows past a ragged end repeat the last valid row: their dS is zero)
  uint32_t dma_row[NDMA], dma_chunk[NDMA];
#pragma unroll
  for (int n = 0; n < NDMA; n++) {
    const int r = (8 * n + wave) * RPI + lane / CPR, pc = lane % CPR;
    dma_row[n] = (uint32_t)(r * kv_row_stride * 2);
    dma_chunk[n] = (uint32_t)((pc ^ swz<D>(r)) << 4);
  }
  // K^T operands: transpose reads of the K tile, d rows 32 dt .. of k-chunk rows {4g..} / {8+4g..}
  const int tr_row = (lane & 15) >> 2, tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  uint32_t tr_lo[DT], tr_hi[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++) {
    tr_lo[dt] = lds_addr(lds_st[0]) + tile_off<D>(4 * g + tr_row, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
    tr_hi[dt] = lds_addr(lds_st[0]) + tile_off<D>(4 * g + tr_row + 8, 4 * dt + (tr_col >> 3)) + (tr_col & 4) * 2;
  }
  // dS^T operands: lane s of a 16-lane group names the piece of KV row r0 + s / 4, query columns 16 (G & 1) + 4 (s & 3) ..
  uint32_t ds_a[2][2];      // [k-chunk of the fragment][rows +0..3 / +8..11]
  {
    const int s16 = lane & 15, G = lane >> 4;
    const int j = G & 1, gg = s16 & 1, mm = (s16 >> 1) & 1;
#pragma unroll
    for (int kc = 0; kc < 2; kc++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const int r = 16 * kc + 8 * h + 4 * g + (s16 >> 2);
        ds_a[kc][h] = lds_addr(lds_st[0]) + TBK + wave * WDS + 1024 * j + 512 * gg + 16 * ((r + 8 * j + 4 * gg) & 31) + 8 * mm;
      }
  }
  int b_c = 0, b_dma = 0;       // ring positions: stage being read, stage being filled
  auto advance_read_stage = [&]() {
    const int st = (b_c == NB - 1) ? -(NB - 1) * STAGE : STAGE;
#pragma unroll
    for (int dt = 0; dt < DT; dt++) { tr_lo[dt] += st; tr_hi[dt] += st; }
#pragma unroll
    for (int kc = 0; kc < 2; kc++) { ds_a[kc][0] += st; ds_a[kc][1] += st; }
    b_c = (b_c == NB - 1) ? 0 : b_c + 1;
  };

  ItemStream items;
  if (wave == 0) {
    const int first = items.start(a.hdr->dq_counter, a.hdr->dq_begin, lane);
    if (first >= 0) fetch_item(a.dq_items, first, s_rec, lane);
    if (lane == 0) s_next = first;
    dma_wait();
  }
  __syncthreads();
  int item_idx = __builtin_amdgcn_readfirstlane(s_next);   // wave-uniform
  while (item_idx >= 0) {
    const QItem it = read_item<QItem>(s_rec);
    const bool four = it.head[1] - it.head[0] == 3;
    const int wq = four ? wave & 1 : wave & 3;
    const int q_start = (sub ? it.q_start[1] : it.q_start[0]), q_rows = (sub ? it.q_rows[1] : it.q_rows[0]), tile_off_q = (sub ? it.tile_off[1] : it.tile_off[0]), head = four ? it.head[0] + (wave >> 1) : (sub ? it.head[1] : it.head[0]);
    const int kvh = it.head[0] / group;
    const int my_row = wq * 32 + l32;
    const bool row_ok = my_row < q_rows;
    const int wave_row_lo = tile_off_q + wq * 32;
    const bool wave_ok = wq * 32 < q_rows;                       // the wave has at least one valid row
    const int nq32 = (it.q_blk_len + 31) >> 5;
    const int q32 = min((tile_off_q >> 5) + wq, nq32 - 1);       // clamped: a wave past the ragged end reads valid memory and uses nothing
    const uint16_t* kbase = a.k + (int64_t)kvh * D;

    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[dt][r] = 0.f;

    TileIter ti;
    ti.init(a.pairs, it);
    const int n_tiles = it.n_tiles;
    // The load of one tile: describe() = scalar bookkeeping, issue() = the requests.  Up to the last four tiles of an item a
    // tile is requested whole, without a branch: branches on what a wave's rows can see and on the count to wait for made
    // long items 20 % slower (end of a 37133-token sequence, heads 2/1, d = 64: 741 us, without them 627).  The last four
    // are requested as needed: nothing past the item's end, and of the wave's two fragments only those its rows can see (a
    // third of the loads of 16-256 token sequences were neither; 65536 tokens, GQA 32/8, d = 128: 375 -> 352 us).
    uint64_t d_k = 0, d_ds = 0;
    uint32_t d_lim = 0;
    int d_vis = 0;                  // columns of the tile that this wave's rows can see (0 .. 64); -1: there is no such tile
    int req = 0;                    // d_vis of the tile requested last (64: it was requested whole)
    auto describe = [&](auto exists) {
      d_vis = -1;
      if (exists || ti.more) {
        const int64_t row0 = (int64_t)(ti.cur.kv_start + ti.c0) * kv_row_stride;
        d_k = reinterpret_cast<uint64_t>(kbase + row0);
        const int valid = min(kFwdTileN, ti.cur.kv_len - ti.c0);
        d_lim = (uint32_t)((valid - 1) * kv_row_stride * 2);
        const int f0 = ti.c0 >> 5;
        int frag;
        if (ti.cur.kind & 1) {
          frag = ti.cur.ext + head * (nq32 * (nq32 + 1) / 2) + q32 * (q32 + 1) / 2 + min(f0, q32);
        } else {
          const int nkv32 = (ti.cur.kv_len + 31) >> 5;
          frag = ti.cur.ext + (head * nq32 + q32) * nkv32 + min(f0, nkv32 - 1);
        }
        d_ds = reinterpret_cast<uint64_t>(a.ds + (int64_t)frag * kDsFragBytes);
        const int vis = (ti.cur.kind & 1) ? min(ti.cur.kv_len, wave_row_lo + 32) : ti.cur.kv_len;
        d_vis = wave_ok ? max(0, min(kFwdTileN, vis - ti.c0)) : 0;
        ti.advance();
      }
    };
    auto issue = [&](auto whole) {
      const uint32_t lbase = lds_addr(lds_st[0]) + b_dma * STAGE;
      auto k_rows = [&]() {
#pragma unroll
        for (int n = 0; n < NDMA; n++) {
          const uint32_t voff = min(dma_row[n], d_lim) + dma_chunk[n];
          lds_dma16_s(reinterpret_cast<const unsigned char*>(d_k), voff, lbase + (8 * n + wave) * 1024);
        }
      };
      auto fragment = [&](int f) {
#pragma unroll
        for (int n = DMA_PER_FRAG * f; n < DMA_PER_FRAG * (f + 1); n++)
          lds_dma16_s(reinterpret_cast<const unsigned char*>(d_ds), (uint32_t)(1024 * n + 16 * lane), lbase + TBK + wave * WDS + 1024 * n);
      };
      req = whole ? kFwdTileN : d_vis;
      if (whole || d_vis > 32) { k_rows(); fragment(0); fragment(1); }
      else if (d_vis >= 0) { k_rows(); if (d_vis > 0) fragment(0); }
      b_dma = (b_dma == NB - 1) ? 0 : b_dma + 1;
    };
    const std::true_type yes;
    const std::false_type no;
    // prologue: tiles 0 and 1 of the item into the stage to be read first and the one after it
    int vis[3];
    b_dma = b_c;
    if (n_tiles > 4) {
      describe(yes); issue(yes); vis[0] = d_vis;
      describe(yes); issue(yes); vis[1] = d_vis;
    } else {
      describe(no); issue(no); vis[0] = d_vis;
      describe(no); issue(no); vis[1] = d_vis;
    }
    auto next_item = [&]() {             // wave 0, see fwd_kernel
      const int nx = items.take(lane);
      if (lane == 0) s_next = nx;
      if (nx >= 0) fetch_item(a.dq_items, nx, s_rec, lane);
    };
    auto arrive = [&](auto whole) {
      // the tile to be computed has landed once only the loads of the next one are in flight (those of a whole tile; if it has
      // fewer, both are waited for); the barrier also says that every wave is done with the stage that the tile after next goes into
      if (whole || req > 32) __builtin_amdgcn_s_waitcnt(0x0F70 | (NDMA + 2 * DMA_PER_FRAG));
      else dma_wait();
      lds_barrier();
      describe(whole); issue(whole); vis[2] = d_vis;
    };
    auto compute = [&]() {
      const int nv = __builtin_amdgcn_readfirstlane(vis[0]);
#pragma unroll
      for (int f = 0; f < 2; f++) {
        if (nv > 32 * f) {
#pragma unroll
          for (int kc = 0; kc < 2; kc++) {
            const bf16x8 b = lds_tr_pair_at(ds_a[kc][0] + kDsFragBytes * f, ds_a[kc][1] + kDsFragBytes * f);
            const uint32_t rows = (32 * f + 16 * kc) * (D * 2);
#pragma unroll
            for (int dt = 0; dt < DT; dt++) {
              const bf16x8 kt = lds_tr_pair_at(tr_lo[dt] + rows, tr_hi[dt] + rows);
              acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt, b, acc[dt], 0, 0, 0);
            }
          }
        }
      }
      vis[0] = vis[1]; vis[1] = vis[2];
      advance_read_stage();
    };
    // The next item's ticket is drawn 4 tiles before the end (no test for it per tile: the queue's bookkeeping inside the
    // loop slows every tile of a long item), its record behind the barrier of the last tile: until then a wave may not have
    // read this item's index and record, which next_item() overwrites.  An item without tiles has a barrier for that alone.
    int t = 0;
    for (; t < n_tiles - 4; t++) { arrive(yes); compute(); }
    if (wave == 0) items.request(lane);
    for (; t < n_tiles - 1; t++) { arrive(no); compute(); }
    if (n_tiles > 0) arrive(no); else lds_barrier();
    if (wave == 0) next_item();
    compute();
    dma_wait();          // the next item's record
    lds_barrier();       // publishes the next item's record
    // the stage read last serves as the waves' staging areas: the next item's first two tiles go into the other two
    unsigned char* stage = lds_st[(b_c + NB - 1) % NB] + wave * kStageBytes;
    {
      const int64_t off = (int64_t)(q_start + wq * 32) * q_row_stride + (int64_t)head * D;
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
        store_tile<GRAD_BF16>(static_cast<unsigned char*>(a.dq) + (off + dt * 32) * (GRAD_BF16 ? 2 : 4), q_row_stride, q_rows - wq * 32, acc[dt], 1.0f, stage, lane);
    }
    item_idx = __builtin_amdgcn_readfirstlane(s_next);
  }
  if (tid == 0) retire(a.hdr->dq_counter, &a.hdr->dq_done);
}

// =====================================================================================
// Backward for launches that leave most of the chip idle (see fwd_split_kernel).  dQ and dK / dV in one launch: they only share
// D and LSE, which a launch of delta_kernel leaves for both (2000 tokens, 4/2 heads, d = 64, us: one after the other, D inside dQ,
// 8.8 + 8.9; so 3.4 + 10.3).
// dQ: 32 query rows of one head, the waves share their KV tiles.
// =====================================================================================
// LDS of both: the waves' streams, the rows that stay, 64 scalars a wave, the waves that had a tile.
template <int D> constexpr int split_lds() { return (kSplitWaves + 1) * 2 * tile_bytes<D>(kSplitRows) + kSplitWaves * 256 + kSplitWaves * 4; }

template <int D, bool WITH_D, bool GRAD_BF16>
__device__ __forceinline__ void dq_split(const BwdArgs& a, int block, int n_items, int units, int per_tile, bool members, unsigned char* lds) {
  constexpr int KC = D / 16, DT = D / 32, T = tile_bytes<D>(kSplitRows);
  unsigned char* const lds_kv = lds;                                  // a wave's [K tile | V tile], at the end its dQ
  unsigned char* const lds_q = lds + kSplitWaves * 2 * T;             // Q, dO
  float* const s_lse = reinterpret_cast<float*>(lds_q + 2 * T);
  float* const s_dl = s_lse + kSplitRows;
  int* const s_act = reinterpret_cast<int*>(lds_q + 2 * T + kSplitWaves * 256);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
  const SplitPlace place(block, units);
  if (place.item >= n_items) return;
  const QItem it = load_record(a.dq_items + place.item);
  const SplitQ u(it, place.unit, per_tile);
  if (u.rows <= 0) return;
  const int group = a.n_q_heads / a.n_kv_heads, kvh = __builtin_amdgcn_readfirstlane(u.head / group);
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D, kv_row_stride = (int64_t)a.n_kv_heads * D;
  const uint32_t kv_row_bytes = (uint32_t)(kv_row_stride * 2);
  const int64_t row0 = (int64_t)u.q_start * q_row_stride + (int64_t)u.head * D;
  const uint16_t* kbase = a.k + (int64_t)kvh * D;
  const uint16_t* vbase = a.v + (int64_t)kvh * D;
  const uint32_t lk = lds_addr(lds_kv) + wave * 2 * T, lv = lk + T;

  SplitTiles tiles;
  tiles.init(a.pairs, it, false, u.tile_off + u.rows, wave, lane);
  auto issue = [&](const uint16_t* base, uint32_t lds) {
    const int c0 = tiles.t * kSplitRows;
    wave_tile_dma<D>(lds, base + (int64_t)(tiles.cur.kv_start + c0) * kv_row_stride, kv_row_bytes, min(kSplitRows, tiles.cur.kv_len - c0), lane);
  };
  group_tile_dma<D>(lds_addr(lds_q), a.q + row0, (uint32_t)(q_row_stride * 2), u.rows, wave, lane);
  group_tile_dma<D>(lds_addr(lds_q) + T, a.d_o + row0, (uint32_t)(q_row_stride * 2), u.rows, kSplitWaves - 1 - wave, lane);
  const bool active = tiles.have;
  if (active) { issue(kbase, lk); issue(vbase, lv); }
  int seg_lo = 0, seg_hi = 0;          // joined run: first and last column of this lane's member
  if (members) {                       // some of its pairs may be joined, not only the first
    const int sg = l32 < u.rows ? a.q_seg[u.q_start + l32] : 0;
    seg_lo = sg & 0xff; seg_hi = sg >> 8;
  }
  if constexpr (WITH_D) {
    // D = rowsum(dO o O), D / 8 lanes to a row
    constexpr int LPR = D / 8;
    static_assert(kSplitRows * LPR <= 64 * kSplitWaves, "one row a thread");
    const int r = tid / LPR, c = 8 * (tid % LPR);
    float d = 0.f;
    if (r < u.rows) {
      const int64_t at = row0 + r * q_row_stride + c;
      const u32x4 dv = *reinterpret_cast<const u32x4*>(a.d_o + at);
      float ov[8];
      if (a.o_is_f32) {
        const f32x4 x0 = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(a.o) + at), x1 = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(a.o) + at + 4);
#pragma unroll
        for (int i = 0; i < 4; i++) { ov[i] = x0[i]; ov[4 + i] = x1[i]; }
      } else {
        const u32x4 x = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(a.o) + at);
#pragma unroll
        for (int i = 0; i < 4; i++) { ov[2 * i] = __uint_as_float(x[i] << 16); ov[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u); }
      }
#pragma unroll
      for (int i = 0; i < 4; i++) {
        d += __uint_as_float(dv[i] << 16) * ov[2 * i];
        d += __uint_as_float(dv[i] & 0xffff0000u) * ov[2 * i + 1];
      }
    }
    for (int off = LPR / 2; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
    if (r < kSplitRows && c == 0) {
      float lse2 = INFINITY, dl = 0.f;
      if (r < u.rows) {
        const float l = a.lse[(int64_t)(u.q_start + r) * a.n_q_heads + u.head];
        lse2 = (l == -INFINITY) ? INFINITY : l * kLog2e;
        dl = d * a.scale;
        const int64_t hr = (int64_t)u.head * a.t_q + u.q_start + r;
        a.lse2_out[hr] = lse2;
        a.dls_out[hr] = dl;
      }
      s_lse[r] = lse2; s_dl[r] = dl;
    }
  } else if (tid < kSplitRows) {
    const int64_t hr = (int64_t)u.head * a.t_q + u.q_start + min(tid, u.rows - 1);
    s_lse[tid] = tid < u.rows ? a.lse2[hr] : INFINITY;
    s_dl[tid] = a.dls[hr];
  }
  loads_left<0>();
  __syncthreads();

  f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[dt][r] = 0.f;
  bf16x8 qf[KC], dof[KC];
#pragma unroll
  for (int kc = 0; kc < KC; kc++) {
    qf[kc] = as_bf16x8(lds_read16(lds_addr(lds_q) + tile_off<D>(l32, 2 * kc + g)));
    dof[kc] = as_bf16x8(lds_read16(lds_addr(lds_q) + T + tile_off<D>(l32, 2 * kc + g)));
  }
  const float lse_l = s_lse[l32], dl_l = s_dl[l32];

  while (tiles.have) {
    int ln = lane;
    asm volatile("" : "+v"(ln));       // as in dkdv_split
    const int l32 = ln & 31, g = ln >> 5, tr_row = (ln & 15) >> 2, tr_col = 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
    const DevPair cur = tiles.cur;
    const int c0 = tiles.t * kSplitRows;
    tiles.next(lane);
    const bool more = tiles.have;
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(lds_read16(lk + tile_off<D>(l32, 2 * kc + g))), qf[kc], s, 0, 0, 0);
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(lds_read16(lv + tile_off<D>(l32, 2 * kc + g))), dof[kc], dp, 0, 0, 0);
    lds_reads_done();
    if (more) issue(vbase, lv);
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.scale_log2, -lse_l));
    const int open = (cur.kind & 2) ? 0 : (cur.kind & 1) ? min(cur.kv_len, u.tile_off + 1) : cur.kv_len;
    if (c0 + kSplitRows > open) {
      int first = 0, last = (cur.kind & 1) ? min(cur.kv_len - 1, u.tile_off + l32) : cur.kv_len - 1;
      if (cur.kind & 2) { first = seg_lo; last = min(last, seg_hi); }
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int c = c0 + 8 * (r >> 2) + 4 * g + (r & 3);
        if (c < first || c > last) s[r] = 0.f;
      }
    }
    u32x4 db[2];
#pragma unroll
    for (int r = 0; r < 16; r += 2)
      db[r >> 3][(r >> 1) & 3] = pack_bf16(s[r] * __builtin_fmaf(dp[r], a.scale, -dl_l), s[r + 1] * __builtin_fmaf(dp[r + 1], a.scale, -dl_l));
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        const int c = 4 * dt + (tr_col >> 3);
        const bf16x8 kt = lds_tr_pair_at(lk + tile_off<D>(16 * j + 4 * g + tr_row, c) + (tr_col & 4) * 2, lk + tile_off<D>(16 * j + 4 * g + tr_row + 8, c) + (tr_col & 4) * 2);
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt, as_bf16x8(db[j]), acc[dt], 0, 0, 0);
      }
    lds_reads_done();
    if (more) { issue(kbase, lk); loads_left<0>(); }
  }
  if (active) put_result<D>(lds_kv + wave * 2 * T, acc, lane);
  if (lane == 0) s_act[wave] = active;
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < D * 8 / (64 * kSplitWaves); pass++) {
    const int row = (tid + 64 * kSplitWaves * pass) / (D / 4), chunk = tid % (D / 4);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kSplitWaves; w++) {
      if (!s_act[w]) break;
      x += get_result<D>(lds_kv + w * 2 * T, row, chunk);
    }
    if (row < u.rows) store4(a.dq, row0 + row * q_row_stride + 4 * chunk, x, GRAD_BF16);
  }
}

// dK, dV: 32 KV rows of one KV head, the waves share the 32-row query steps of their dependencies and query heads.
// SPILL: dS goes to memory too, as dkdv_kernel leaves it.
template <int D, bool GRAD_BF16, bool SPILL>
__device__ __forceinline__ void dkdv_split(const BwdArgs& a, int block, int n_items, int units, unsigned char* lds) {
  constexpr int KC = D / 16, DT = D / 32, T = tile_bytes<D>(kSplitRows);
  unsigned char* const lds_t = lds;                                   // a wave's [Q tile | dO tile], at the end its dK, then its dV
  unsigned char* const lds_kv = lds + kSplitWaves * 2 * T;            // K, V
  unsigned char* const lds_sc = lds_kv + 2 * T;                       // a wave's [LSE*log2e x 32 | D*scale x 32]
  int* const s_act = reinterpret_cast<int*>(lds_sc + kSplitWaves * 256);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
  const SplitPlace place(block, units);
  const int off = place.unit * kSplitRows;
  if (place.item >= n_items) return;
  const BwdItem it = load_record(a.items + place.item);
  const int rows = min(it.kv_rows - off, kSplitRows);
  if (rows <= 0) return;
  const int kv0 = it.tile_off + off;                     // first of the rows inside the segment
  const int group = a.n_q_heads / a.n_kv_heads;
  const int64_t q_row_stride = (int64_t)a.n_q_heads * D, kv_row_stride = (int64_t)a.n_kv_heads * D;
  const int64_t kv_at = (int64_t)(it.kv_start + off) * kv_row_stride + (int64_t)it.kv_head * D;
  const uint32_t lq = lds_addr(lds_t) + wave * 2 * T, lo = lq + T, lsc = lds_addr(lds_sc) + wave * 256;

  // The wave's steps: every eighth of (dependency, head of the group, 32 query rows); a DIAG dependency from the rows' own on.
  RecordWindow<BwdDep> rec;
  rec.init(a.deps + it.dep_begin, it.n_deps, it.first);
  BwdDep cur = it.first;
  int dep = 0, t = wave, per_head = 0;
  bool have = it.n_deps > 0;
  auto first_row = [&]() { return (cur.kind & 1) ? kv0 : 0; };
  auto seek = [&]() {
    for (;;) {
      per_head = (cur.q_len - first_row() + kSplitRows - 1) / kSplitRows;
      if (t < per_head * group) return;
      t -= per_head * group;
      if (++dep >= it.n_deps) { have = false; return; }
      cur = rec.get(dep, lane);
    }
  };
  int q0 = 0;                                            // first query row of the step inside its segment
  int frag = 0;                                          // its dS fragment
  auto issue = [&]() {
    const int hh = __builtin_amdgcn_readfirstlane(t / per_head), head = it.kv_head * group + hh;
    q0 = first_row() + (t - hh * per_head) * kSplitRows;
    if constexpr (SPILL) {
      const int q32 = q0 >> 5, nq32 = (cur.q_len + 31) >> 5;
      frag = cur.ds_frag + (kv0 >> 5) + ((cur.kind & 1) ? head * (nq32 * (nq32 + 1) / 2) + q32 * (q32 + 1) / 2 : (head * nq32 + q32) * ((it.kv_blk_len + 31) >> 5));
    }
    const int valid = min(kSplitRows, cur.q_len - q0);
    const int64_t row = cur.q_start + q0, at = row * q_row_stride + (int64_t)head * D;
    wave_tile_dma<D>(lq, a.q + at, (uint32_t)(q_row_stride * 2), valid, lane);
    wave_tile_dma<D>(lo, a.d_o + at, (uint32_t)(q_row_stride * 2), valid, lane);
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const float* in_range = (ln >> 5 ? a.dls : a.lse2) + (int64_t)head * a.t_q + row;
    const float* past_end = ln >> 5 ? reinterpret_cast<const float*>(a.hdr->zeros) : a.hdr->infs;
    lds_dma4(((ln & 31) < valid ? in_range : past_end) + (ln & 31), lsc);
  };
  if (have) seek();
  group_tile_dma<D>(lds_addr(lds_kv), a.k + kv_at, (uint32_t)(kv_row_stride * 2), rows, wave, lane);
  group_tile_dma<D>(lds_addr(lds_kv) + T, a.v + kv_at, (uint32_t)(kv_row_stride * 2), rows, kSplitWaves - 1 - wave, lane);
  const bool active = have;
  if (active) issue();
  // query rows (of the segment) that see this lane's KV row: a joined run's of its own member, a diagonal's from the row itself on
  int seg_lo = 0, seg_hi = 0x7fffffff;
  if (it.first.kind & 2) {
    const int sg = l32 < rows ? a.q_seg[it.first.q_start + kv0 + l32] : 0;
    seg_lo = sg & 0xff; seg_hi = sg >> 8;
  }
  loads_left<0>();
  __syncthreads();

  f32x16 acc_k[DT], acc_v[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) { acc_k[dt][r] = 0.f; acc_v[dt][r] = 0.f; }

  while (have) {
    const int kind = cur.kind, first_q = q0, frag_now = frag;
    int ln = lane;
    asm volatile("" : "+v"(ln));       // the LDS addresses are formed in every step: held through the loop they cost d = 64 two dozen spills
    const int l32 = ln & 31, g = ln >> 5, tr_row = (ln & 15) >> 2, tr_col = 16 * ((ln >> 4) & 1) + 4 * (ln & 3);
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
      const uint32_t at = tile_off<D>(l32, 2 * kc + g);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(lds_read16(lq + at)), as_bf16x8(lds_read16(lds_addr(lds_kv) + at)), s, 0, 0, 0);
      if (kc & 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
      const uint32_t at = tile_off<D>(l32, 2 * kc + g);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(lds_read16(lo + at)), as_bf16x8(lds_read16(lds_addr(lds_kv) + T + at)), dp, 0, 0, 0);
      if (kc & 1) __builtin_amdgcn_sched_barrier(0);
    }
    // scalars of rows 8 q4 + 4 g .. +3 of the step; the barriers keep the operands of one phase out of the next (d = 64: 128 registers)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const f32x4 lse4 = __builtin_bit_cast(f32x4, lds_read16(lsc + 32 * q4 + 16 * g));
#pragma unroll
      for (int i = 0; i < 4; i++) s[4 * q4 + i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[4 * q4 + i], a.scale_log2, -lse4[i]));
    }
    __builtin_amdgcn_sched_barrier(0);
    if ((kind & 2) || ((kind & 1) && first_q < kv0 + kSplitRows - 1) || (SPILL && rows < kSplitRows)) {
      int lo_q = (kind & 1) ? kv0 + l32 : 0, hi_q = 0x7fffffff;
      if (kind & 2) { lo_q = max(lo_q, seg_lo); hi_q = seg_hi; }
      if (SPILL && l32 >= rows) lo_q = 0x7fffffff;       // the dQ pass multiplies a row past the end with whatever K sits there
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int q = first_q + 8 * (r >> 2) + 4 * g + (r & 3);
        if (q < lo_q || q > hi_q) s[r] = 0.f;
      }
    }
    u32x4 pb[2], db[2];
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const f32x4 dl4 = __builtin_bit_cast(f32x4, lds_read16(lsc + 32 * q4 + 16 * g + 128));
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const int r = 4 * q4 + i;
        pb[q4 >> 1][(r >> 1) & 3] = pack_bf16(s[r], s[r + 1]);
        db[q4 >> 1][(r >> 1) & 3] = pack_bf16(s[r] * __builtin_fmaf(dp[r], a.scale, -dl4[i]), s[r + 1] * __builtin_fmaf(dp[r + 1], a.scale, -dl4[i + 1]));
      }
    }
    if constexpr (SPILL) {
#pragma unroll
      for (int j = 0; j < 2; j++)
        *reinterpret_cast<u32x4*>(a.ds + (int64_t)__builtin_amdgcn_readfirstlane(frag_now) * kDsFragBytes + 1024 * j + 512 * g + 16 * ((l32 + 8 * j + 4 * g) & 31)) = db[j];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        const int c = 4 * dt + (tr_col >> 3);
        const uint32_t lo16 = tile_off<D>(16 * j + 4 * g + tr_row, c) + (tr_col & 4) * 2, hi16 = tile_off<D>(16 * j + 4 * g + tr_row + 8, c) + (tr_col & 4) * 2;
        acc_v[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_tr_pair_at(lo + lo16, lo + hi16), as_bf16x8(pb[j]), acc_v[dt], 0, 0, 0);
        acc_k[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_tr_pair_at(lq + lo16, lq + hi16), as_bf16x8(db[j]), acc_k[dt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    t += kSplitWaves;
    seek();
    lds_reads_done();
    if (have) { issue(); loads_left<0>(); }
  }
  if (lane == 0) s_act[wave] = active;
#pragma unroll
  for (int o = 0; o < 2; o++) {
    if (o) __syncthreads();          // dK has been read
    if (active) put_result<D>(lds_t + wave * 2 * T, o ? acc_v : acc_k, lane);
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < D * 8 / (64 * kSplitWaves); pass++) {
      const int row = (tid + 64 * kSplitWaves * pass) / (D / 4), chunk = tid % (D / 4);
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kSplitWaves; w++) {
        if (!s_act[w]) break;
        x += get_result<D>(lds_t + w * 2 * T, row, chunk);
      }
      if (row < rows) store4(o ? a.dv : a.dk, kv_at + row * kv_row_stride + 4 * chunk, x, GRAD_BF16);
    }
  }
}

// Items of each kind and the workgroups of an item (of them in a sub-tile).  Items in eights: one to an XCD.
struct SplitGrid {
  int n_kv, kv_units, n_q, q_units, q_per_tile;
  bool members;                 // the problem has packed blocks
  __host__ __device__ int kv_blocks() const { return (n_kv + kNumXcd - 1) / kNumXcd * kNumXcd * kv_units; }
  __host__ __device__ int q_blocks() const { return (n_q + kNumXcd - 1) / kNumXcd * kNumXcd * q_units; }
};

// Both in one launch, or either: dK / dV take the first workgroups of the grid, dQ the rest.  Launches that write dS are of dK / dV
// alone, launches that form D of dQ alone.
template <int D, bool WITH_D, bool GRAD_BF16, bool SPILL>
__global__ void __launch_bounds__(64 * kSplitWaves, D == 64 ? 4 : 2) bwd_split_kernel(BwdArgs a, SplitGrid grid) {
  static_assert(!(WITH_D && SPILL), "no such launch");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[split_lds<D>()];
  const int kv = WITH_D ? 0 : grid.kv_blocks();
  if constexpr (!WITH_D) {
    if (SPILL || (int)blockIdx.x < kv) { dkdv_split<D, GRAD_BF16, SPILL>(a, blockIdx.x, grid.n_kv, grid.kv_units, lds); return; }
  }
  if constexpr (!SPILL) dq_split<D, WITH_D, GRAD_BF16>(a, blockIdx.x - kv, grid.n_q, grid.q_units, grid.q_per_tile, grid.members, lds);
}

// =====================================================================================
// Launchers
// =====================================================================================
static int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

static int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("%s: %s", what, hipGetErrorString(e)); return FCP_ERR_HIP; }
  return FCP_OK;
}

static float resolve_scale(const fcp_problem* p) {
  return p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->head_dim);
}

constexpr int kFwdWgPerCu = 1;   // 8 waves, two per SIMD
constexpr int kDkdvWgPerCu = 1;   // 8 waves, two per SIMD
constexpr int kDqWgPerCu = 1;   // 8 waves, two per SIMD

}  // namespace fcp

using namespace fcp;

extern "C" int fcp_device_info(int32_t* n_compute_units, int32_t* fwd_grid, int32_t* bwd_grid) {
  const int n = cu_count();
  if (n_compute_units) *n_compute_units = n;
  if (fwd_grid) *fwd_grid = n * kFwdWgPerCu;
  if (bwd_grid) *bwd_grid = n * kDkdvWgPerCu;
  return FCP_OK;
}

static int launch_fwd(const char* who, const fcp_problem* p, const WsLayout* layout, const void* q, const void* k, const void* v,
                      void* o_part, float* lse_part, void* o, float* lse, void* workspace, void* stream) {
  WsLayout L;
  if (layout) L = *layout;
  else if (int rc = layout_for(p, workspace, &L)) return rc;
  if (L.n_fwd_items == 0) return FCP_OK;
  if (!q || !k || !v || !workspace || (p->n_slot_rows && !(p->flags & FCP_FLAG_RUNNING_MERGE) && (!o_part || !lse_part))) {
    set_error("%s: NULL pointer", who); return FCP_ERR_INVALID_ARG;
  }
  const bool direct = (p->flags & FCP_FLAG_DIRECT_SINGLE) != 0;
  const bool running = (p->flags & FCP_FLAG_RUNNING_MERGE) != 0;
  if (running) {
    if (!o || !lse || !(p->flags & FCP_FLAG_O_F32)) {
      set_error("%s: FCP_FLAG_RUNNING_MERGE needs the running o (fp32: FCP_FLAG_O_F32) and lse (call fcp_block_attn_fwd_out)", who);
      return FCP_ERR_INVALID_ARG;
    }
    for (int s = 1; s < p->n_slots; s++)
      if (p->slots[s].q_blk == p->slots[s - 1].q_blk) {
        set_error("%s: FCP_FLAG_RUNNING_MERGE takes one stage per launch, but query block %d has several slots (see fcp_stage_tables)",
                  who, p->slots[s].q_blk);
        return FCP_ERR_INVALID_ARG;
      }
  }
  if (direct && (!o || !lse)) {
    set_error("%s: FCP_FLAG_DIRECT_SINGLE needs the final o and lse (call fcp_block_attn_fwd_out)", who);
    return FCP_ERR_INVALID_ARG;
  }
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  FwdArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
  a.o_part = o_part; a.lse_part = lse_part; a.part_is_bf16 = (p->flags & FCP_FLAG_PART_BF16) ? 1 : 0;
  a.o = (direct || running) ? o : nullptr; a.lse = (direct || running) ? lse : nullptr;
  a.running = running ? 1 : 0;
  a.o_is_f32 = (p->flags & FCP_FLAG_O_F32) ? 1 : 0;
  a.hdr = reinterpret_cast<WsHeader*>(ws);
  a.spans = reinterpret_cast<const DevPair*>(ws + L.off_spans);
  a.items = reinterpret_cast<const QItem*>(ws + L.off_fwd_items);
  a.q_seg = reinterpret_cast<const uint16_t*>(ws + L.off_q_seg);
  a.n_q_heads = p->n_q_heads; a.n_kv_heads = p->n_kv_heads;
  a.scale_log2 = resolve_scale(p) * kLog2e;
  if (L.split_fwd) {
    const SplitGrid g = {0, 0, (int)L.n_fwd_items, L.fwd_units.units, L.fwd_units.per_tile, false};
    void (*kern)(FwdArgs, int, int, int) = p->head_dim == 128 ? fwd_split_kernel<128> : fwd_split_kernel<64>;
    hipLaunchKernelGGL(kern, dim3(g.q_blocks()), dim3(64 * kSplitWaves), 0, (hipStream_t)stream, a, g.n_q, g.q_units, g.q_per_tile);
    return check_launch(who);
  }
  const int grid = (int)std::min<int64_t>(L.n_fwd_items, (int64_t)cu_count() * kFwdWgPerCu);
  if (p->head_dim == 128) hipLaunchKernelGGL(fwd_kernel<128>, dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
  else hipLaunchKernelGGL(fwd_kernel<64>, dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
  return check_launch(who);
}

extern "C" int fcp_block_attn_fwd(const fcp_problem* p, const void* q, const void* k, const void* v,
                                  void* o_part, float* lse_part, void* workspace, void* stream) {
  return launch_fwd("fcp_block_attn_fwd", p, nullptr, q, k, v, o_part, lse_part, nullptr, nullptr, workspace, stream);
}

// ---- forward without any allocation: the queue tables live in a fixed device array ----
namespace fcp {
// A call is limited by the tables of its plan as given (static_plan_bytes, 2 MiB).  The array holds whatever such a plan
// becomes: two neighbouring runs of a packed block have more rows than one item, so a block of n items' rows has at
// most 3 n items (members one row longer than an item between members of one row) and as many pairs, and 16 + 80 bytes for
// each of 3 n are 4 times the 72 counted for each of n.  Only the member bounds (2 bytes per query row) can be more.
constexpr size_t kStaticPlanBytes = 2u << 20, kStaticScratchBytes = (8u << 20) + (16u << 10);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
// Device address of `scratch` on each device (the array's name is a host-side stand-in, not an
// address a kernel can use; every device holds its own copy at its own address).
static void* g_scratch_ptr[64] = {nullptr};

static int static_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { set_error("fcp_block_attn_fwd_static: hipGetDevice: %s", hipGetErrorString(e)); return FCP_ERR_HIP; }
  if (dev < 0 || dev >= 64) { set_error("fcp_block_attn_fwd_static: device index %d out of range", dev); return FCP_ERR_UNSUPPORTED; }
  if (!g_scratch_ptr[dev]) {
    void* sym = nullptr;
    e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !sym) {
      set_error("fcp_block_attn_fwd_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
      return FCP_ERR_HIP;
    }
    g_scratch_ptr[dev] = sym;
  }
  *ptr = g_scratch_ptr[dev];
  return FCP_OK;
}
}  // namespace fcp

extern "C" int fcp_block_attn_fwd_static(const fcp_problem* p, const void* q, const void* k, const void* v,
                                         void* o_part, float* lse_part, void* stream) {
  int rc = validate_problem(p);
  if (rc) return rc;
  if (p->flags & FCP_FLAG_DIRECT_SINGLE) {
    set_error("fcp_block_attn_fwd_static: FCP_FLAG_DIRECT_SINGLE is not supported here (all slots go to the partial buffers)");
    return FCP_ERR_INVALID_ARG;
  }
  WsLayout L;
  rc = compute_layout(p, true, &L);
  if (rc) return rc;
  choose_split(p, true, &L);
  const size_t plan_bytes = static_plan_bytes(p);
  if (plan_bytes > kStaticPlanBytes || L.off_dls > kStaticScratchBytes) {
    set_error("fcp_block_attn_fwd_static: the forward's queue tables need %zu bytes, the limit is %zu "
              "(use fcp_queue_build + fcp_block_attn_fwd with a workspace of your own)", plan_bytes, kStaticPlanBytes);
    return FCP_ERR_BUFFER_TOO_SMALL;
  }
  if (L.n_fwd_items == 0) return FCP_OK;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc) return rc;
  // The tables are rebuilt on every call (the array keeps the previous call's contents): header with
  // zeroed counters, spans, forward items.  Host memory only; one copy; the copy is waited for
  // because its source dies with this frame.
  Expanded x;
  expand_problem(p, true, &x);
  std::vector<unsigned char> image;
  rc = build_queue_image(p, x, L, true, &image);
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(ws, image.data(), image.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) { set_error("fcp_block_attn_fwd_static: %s", hipGetErrorString(e)); return FCP_ERR_HIP; }
  return launch_fwd("fcp_block_attn_fwd_static", p, &L, q, k, v, o_part, lse_part, nullptr, nullptr, ws, stream);
}

extern "C" int fcp_block_attn_fwd_out(const fcp_problem* p, const void* q, const void* k, const void* v,
                                      void* o_part, float* lse_part, void* o, float* lse,
                                      void* workspace, void* stream) {
  return launch_fwd("fcp_block_attn_fwd_out", p, nullptr, q, k, v, o_part, lse_part, o, lse, workspace, stream);
}

extern "C" int fcp_merge_partials(const fcp_problem* p, const void* o_part, const float* lse_part,
                                  void* o, float* lse, void* workspace, void* stream) {
  WsLayout L;
  int rc = layout_for(p, workspace, &L);
  if (rc) return rc;
  if (L.n_merge_items == 0) return FCP_OK;
  if (!o || !lse || !workspace || (p->n_slots && (!o_part || !lse_part))) { set_error("fcp_merge_partials: NULL pointer"); return FCP_ERR_INVALID_ARG; }
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  MergeArgs a;
  a.o_part = o_part; a.lse_part = lse_part; a.o = o; a.lse = lse;
  a.items = reinterpret_cast<const MergeItem*>(ws + L.off_merge_items);
  a.slot_rh = reinterpret_cast<const int32_t*>(ws + L.off_slot_rh);
  a.o_is_f32 = (p->flags & FCP_FLAG_O_F32) ? 1 : 0;
  a.part_is_bf16 = (p->flags & FCP_FLAG_PART_BF16) ? 1 : 0;
  if (p->head_dim == 128) hipLaunchKernelGGL(merge_kernel<128>, dim3((unsigned)L.n_merge_items), dim3(256), 0, (hipStream_t)stream, a);
  else hipLaunchKernelGGL(merge_kernel<64>, dim3((unsigned)L.n_merge_items), dim3(256), 0, (hipStream_t)stream, a);
  return check_launch("fcp_merge_partials");
}

extern "C" int fcp_bwd_preprocess(const fcp_problem* p, const void* o, const float* lse, const void* d_o,
                                  void* workspace, void* stream) {
  WsLayout L;
  int rc = layout_for(p, workspace, &L);
  if (rc) return rc;
  if (L.t_q == 0) return FCP_OK;
  if (!o || !lse || !d_o || !workspace) { set_error("fcp_bwd_preprocess: NULL pointer"); return FCP_ERR_INVALID_ARG; }
  hipStream_t st = (hipStream_t)stream;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  float* dls = reinterpret_cast<float*>(ws + L.off_dls);
  float* lse2 = reinterpret_cast<float*>(ws + L.off_lse2);
  const int o_f32 = (p->flags & FCP_FLAG_O_F32) ? 1 : 0;
  const float scale = resolve_scale(p);
  const unsigned blocks = (unsigned)((L.t_q + kDeltaTok - 1) / kDeltaTok);
  if (p->head_dim == 128) hipLaunchKernelGGL(delta_kernel<128>, dim3(blocks), dim3(256), 0, st, o, o_f32, (const uint16_t*)d_o, lse, dls, lse2, L.t_q, p->n_q_heads, scale);
  else hipLaunchKernelGGL(delta_kernel<64>, dim3(blocks), dim3(256), 0, st, o, o_f32, (const uint16_t*)d_o, lse, dls, lse2, L.t_q, p->n_q_heads, scale);
  return check_launch("fcp_bwd_preprocess");
}

static int fill_bwd_args(const fcp_problem* p, WsLayout* L, BwdArgs* a, void* workspace) {
  int rc = layout_for(p, workspace, L);
  if (rc) return rc;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  a->hdr = reinterpret_cast<WsHeader*>(ws);
  a->dls = reinterpret_cast<const float*>(ws + L->off_dls);
  a->lse2 = reinterpret_cast<const float*>(ws + L->off_lse2);
  a->t_q = L->t_q;
  a->pairs = reinterpret_cast<const DevPair*>(ws + L->off_pairs);
  a->deps = reinterpret_cast<const BwdDep*>(ws + L->off_bwd_deps);
  a->items = reinterpret_cast<const BwdItem*>(ws + L->off_bwd_items);
  a->dq_items = reinterpret_cast<const QItem*>(ws + L->off_dq_items);
  a->q_seg = reinterpret_cast<const uint16_t*>(ws + L->off_q_seg);
  a->n_q_heads = p->n_q_heads; a->n_kv_heads = p->n_kv_heads;
  a->scale = resolve_scale(p); a->scale_log2 = a->scale * kLog2e;
  a->dq = nullptr; a->dk = nullptr; a->dv = nullptr;
  a->o = nullptr; a->lse = nullptr; a->o_is_f32 = 0; a->lse2_out = nullptr; a->dls_out = nullptr; a->ds = nullptr;
  return FCP_OK;
}

template <int D>
static auto bwd_split_instance(bool with_d, bool gb, bool spill) -> void (*)(BwdArgs, SplitGrid) {
  if (spill) return gb ? bwd_split_kernel<D, false, true, true> : bwd_split_kernel<D, false, false, true>;
  return with_d ? (gb ? bwd_split_kernel<D, true, true, false> : bwd_split_kernel<D, true, false, false>)
                : (gb ? bwd_split_kernel<D, false, true, false> : bwd_split_kernel<D, false, false, false>);
}

// dK / dV, dQ, or both
static int launch_bwd_split(const char* who, const fcp_problem* p, const WsLayout& L, const BwdArgs& a, bool kv, bool q, bool with_d, void* stream) {
  const bool gb = (p->flags & FCP_FLAG_GRAD_BF16) != 0, spill = a.ds != nullptr;
  void (*kern)(BwdArgs, SplitGrid) = p->head_dim == 128 ? bwd_split_instance<128>(with_d, gb, spill) : bwd_split_instance<64>(with_d, gb, spill);
  const SplitGrid g = {kv ? (int)L.n_bwd_items : 0, L.split_kv_units, q ? (int)L.n_dq_items : 0, L.dq_units.units, L.dq_units.per_tile, p->n_segments > 0};
  hipLaunchKernelGGL(kern, dim3(g.kv_blocks() + g.q_blocks()), dim3(64 * kSplitWaves), 0, (hipStream_t)stream, a, g);
  return check_launch(who);
}

template <bool J>
static auto dkdv_instance(bool d128, bool gb, bool spill) -> void (*)(BwdArgs) {
  if (d128) return spill ? (gb ? dkdv_kernel<128, true, true, J> : dkdv_kernel<128, false, true, J>)
                         : (gb ? dkdv_kernel<128, true, false, J> : dkdv_kernel<128, false, false, J>);
  return spill ? (gb ? dkdv_kernel<64, true, true, J> : dkdv_kernel<64, false, true, J>)
               : (gb ? dkdv_kernel<64, true, false, J> : dkdv_kernel<64, false, false, J>);
}

extern "C" int fcp_block_attn_bwd_dkdv(const fcp_problem* p, const void* q, const void* k, const void* v,
                                       const void* d_o, void* dk, void* dv, void* workspace, void* stream) {
  WsLayout L;
  BwdArgs a;
  int rc = fill_bwd_args(p, &L, &a, workspace);
  if (rc) return rc;
  if (L.n_bwd_items == 0) return FCP_OK;
  if (!q || !k || !v || !d_o || !dk || !dv || !workspace) { set_error("fcp_block_attn_bwd_dkdv: NULL pointer"); return FCP_ERR_INVALID_ARG; }
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_o;
  a.dk = dk; a.dv = dv;
  int grid = (int)std::min<int64_t>(L.n_bwd_items, (int64_t)cu_count() * kDkdvWgPerCu);
  const bool gb = (p->flags & FCP_FLAG_GRAD_BF16) != 0, d128 = p->head_dim == 128;
  const bool spill = (p->flags & FCP_FLAG_BWD_SPILL_DS) != 0;
  if (spill) a.ds = static_cast<unsigned char*>(workspace) + L.off_ds;
  if (L.split_dkdv) return launch_bwd_split("fcp_block_attn_bwd_dkdv", p, L, a, true, false, false, stream);
  void (*kern)(BwdArgs) = p->n_segments > 0 ? dkdv_instance<true>(d128, gb, spill) : dkdv_instance<false>(d128, gb, spill);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
  return check_launch("fcp_block_attn_bwd_dkdv");
}

// o / lse == NULL: the per-row scalars come from fcp_bwd_preprocess; else the kernel computes and publishes them.
template <bool J>
static auto dq_instance(bool d128, bool with_d, bool gb) -> void (*)(BwdArgs) {
  if (d128) return with_d ? (gb ? dq_kernel<128, true, true, J> : dq_kernel<128, true, false, J>)
                          : (gb ? dq_kernel<128, false, true, J> : dq_kernel<128, false, false, J>);
  return with_d ? (gb ? dq_kernel<64, true, true, J> : dq_kernel<64, true, false, J>)
                : (gb ? dq_kernel<64, false, true, J> : dq_kernel<64, false, false, J>);
}

static int launch_dq(const char* who, const fcp_problem* p, const void* q, const void* k, const void* v,
                     const void* o, const float* lse, const void* d_o, void* dq, void* workspace, void* stream) {
  WsLayout L;
  BwdArgs a;
  int rc = fill_bwd_args(p, &L, &a, workspace);
  if (rc) return rc;
  if (L.n_dq_items == 0) return FCP_OK;
  if (!q || !k || !v || !d_o || !dq || !workspace) { set_error("%s: NULL pointer", who); return FCP_ERR_INVALID_ARG; }
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_o;
  a.dq = dq;
  const int grid = (int)std::min<int64_t>(L.n_dq_items, (int64_t)cu_count() * kDqWgPerCu);
  const bool gb = (p->flags & FCP_FLAG_GRAD_BF16) != 0, d128 = p->head_dim == 128;
  const bool with_d = o != nullptr;
  if (with_d) {
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    a.o = o; a.lse = lse; a.o_is_f32 = (p->flags & FCP_FLAG_O_F32) ? 1 : 0;
    a.dls_out = reinterpret_cast<float*>(ws + L.off_dls);
    a.lse2_out = reinterpret_cast<float*>(ws + L.off_lse2);
  }
  if (L.split_dq) return launch_bwd_split(who, p, L, a, false, true, with_d, stream);
  void (*kern)(BwdArgs) = p->n_segments > 0 ? dq_instance<true>(d128, with_d, gb) : dq_instance<false>(d128, with_d, gb);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
  return check_launch(who);
}

extern "C" int fcp_block_attn_bwd_dq(const fcp_problem* p, const void* q, const void* k, const void* v,
                                     const void* d_o, void* dq, void* workspace, void* stream) {
  return launch_dq("fcp_block_attn_bwd_dq", p, q, k, v, nullptr, nullptr, d_o, dq, workspace, stream);
}

extern "C" int fcp_block_attn_bwd_dq_d(const fcp_problem* p, const void* q, const void* k, const void* v,
                                       const void* o, const float* lse, const void* d_o, void* dq,
                                       void* workspace, void* stream) {
  if (!o || !lse) {
    int rc = validate_problem(p);
    if (rc) return rc;
    set_error("fcp_block_attn_bwd_dq_d: NULL pointer");
    return FCP_ERR_INVALID_ARG;
  }
  return launch_dq("fcp_block_attn_bwd_dq_d", p, q, k, v, o, lse, d_o, dq, workspace, stream);
}

extern "C" int fcp_block_attn_bwd_dq_ds(const fcp_problem* p, const void* k, void* dq, void* workspace, void* stream) {
  WsLayout L;
  BwdArgs a;
  int rc = fill_bwd_args(p, &L, &a, workspace);
  if (rc) return rc;
  if (!(p->flags & FCP_FLAG_BWD_SPILL_DS)) {
    set_error("fcp_block_attn_bwd_dq_ds: FCP_FLAG_BWD_SPILL_DS is not set on this problem");
    return FCP_ERR_INVALID_ARG;
  }
  if (L.n_dq_items == 0) return FCP_OK;
  if (!k || !dq || !workspace) { set_error("fcp_block_attn_bwd_dq_ds: NULL pointer"); return FCP_ERR_INVALID_ARG; }
  a.k = (const uint16_t*)k;
  a.dq = dq;
  a.ds = static_cast<unsigned char*>(workspace) + L.off_ds;
  const int grid = (int)std::min<int64_t>(L.n_dq_items, (int64_t)cu_count() * kDqWgPerCu);
  const bool gb = (p->flags & FCP_FLAG_GRAD_BF16) != 0;
  void (*kern)(BwdArgs) = p->head_dim == 128 ? (gb ? dq_ds_kernel<128, true> : dq_ds_kernel<128, false>)
                                             : (gb ? dq_ds_kernel<64, true> : dq_ds_kernel<64, false>);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
  return check_launch("fcp_block_attn_bwd_dq_ds");
}

extern "C" int fcp_block_attn_bwd(const fcp_problem* p, const void* q, const void* k, const void* v,
                                  const void* o, const float* lse, const void* d_o,
                                  void* dq, void* dk, void* dv, void* workspace, void* stream) {
  if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv || !workspace) {
    int rc = validate_problem(p);
    if (rc) return rc;
    set_error("fcp_block_attn_bwd: NULL pointer");
    return FCP_ERR_INVALID_ARG;
  }
  WsLayout L;
  BwdArgs a;
  if (int rc = fill_bwd_args(p, &L, &a, workspace)) return rc;
  if (p->flags & FCP_FLAG_BWD_SPILL_DS) {
    // D first (a pass of its own), then dK/dV, which also writes dS, then dQ from that dS
    int rc = fcp_bwd_preprocess(p, o, lse, d_o, workspace, stream);
    if (rc) return rc;
    rc = fcp_block_attn_bwd_dkdv(p, q, k, v, d_o, dk, dv, workspace, stream);
    if (rc) return rc;
    return fcp_block_attn_bwd_dq_ds(p, k, dq, workspace, stream);
  }
  if (L.joint_bwd) {
    // D by a launch of its own, then dK / dV and dQ side by side
    if (int rc = fcp_bwd_preprocess(p, o, lse, d_o, workspace, stream)) return rc;
    a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_o;
    a.dq = dq; a.dk = dk; a.dv = dv;
    return launch_bwd_split("fcp_block_attn_bwd", p, L, a, true, true, false, stream);
  }
  // dQ first: its kernel also leaves the per-row scalars (D * scale, LSE * log2 e) that dK/dV needs
  int rc = fcp_block_attn_bwd_dq_d(p, q, k, v, o, lse, d_o, dq, workspace, stream);
  if (rc) return rc;
  return fcp_block_attn_bwd_dkdv(p, q, k, v, d_o, dk, dv, workspace, stream);
}

