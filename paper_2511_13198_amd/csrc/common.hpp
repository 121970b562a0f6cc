// Shared device-side building blocks for the gfx950 attention kernels.
//
// Matrix-core conventions (verified lane layouts of the CDNA4 instruction
// v_mfma_f32_32x32x16_bf16, wave64):
//   A (32 x 16): lane l holds A[l % 32][(l / 32) * 8 + j],   j = 0..7
//   B (16 x 32): lane l holds B[(l / 32) * 8 + j][l % 32],   j = 0..7
//   C (32 x 32): lane l holds C[(r / 4) * 8 + (l / 32) * 4 + r % 4][l % 32], r = 0..15
// Every kernel keeps one "owned" index per lane on the C column (l % 32), so
// per-row softmax statistics stay lane-local.  The contraction index of the
// second product in each chain is taken in the permuted order
//   sigma(hh, j) = (j / 4) * 8 + hh * 4 + j % 4      (hh = l / 32)
// which is exactly the order in which a C tile's registers r = 8t..8t+7 list
// their rows; the matching A operand is then fetched from a row-major LDS tile
// with the transposing read ds_read_b64_tr_b16 (see lds_tr_a_operand).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace pdy {

// Fourth word of a raw buffer resource on gfx950 (32-bit data format, no
// swizzle): the value the buffer range check and LDS copies were verified with.
constexpr int kBufferFlags = 0x00020000;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0..N-1.
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// LDS byte address of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)(p);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Value of x held by lane (l ^ 32), via v_permlane32_swap.
__device__ __forceinline__ float partner32(float x) {
  const int l = __lane_id();
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(l < 32 ? r[1] : r[0]);
}

// Pack 8 fp32 values (v[0..7]) into a bf16x8 operand (round to nearest even).
__device__ __forceinline__ bf16x8 pack8(const f32x16& s, int base) {
  bf16x8 out;
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    f32x2 two = {s[base + j], s[base + j + 1]};
    bf16x2 b = __builtin_convertvector(two, bf16x2);
    out[j] = b[0];
    out[j + 1] = b[1];
  }
  return out;
}

// 16-byte global load of 8 bf16 as an MFMA operand; zero when !valid.
__device__ __forceinline__ bf16x8 load_bf16x8(const uint16_t* p, bool valid) {
  u32x4 raw = {0u, 0u, 0u, 0u};
  if (valid) raw = *reinterpret_cast<const u32x4*>(p);
  return __builtin_bit_cast(bf16x8, raw);
}

// ---------------------------------------------------------------------------
// LDS tile layouts.  A tile holds rows of D bf16 values as 16-byte chunks; all
// offsets below are in bf16 elements.  Two access patterns occur:
//   * row reads (row_issue): a quarter-wave reads the same chunk of 16
//     consecutive rows;
//   * transposing reads (tr_issue): a half-wave reads 4 consecutive rows
//     x 64 consecutive bytes.
// RowsLayout pads rows to D + 8 elements (272 B for D = 128), which makes row
// reads conflict-free.  DualLayout (D = 128) stores row r at 320 r bytes
// shifted by 16 ((r / 4) mod 4) bytes; its bank pattern 4 (r mod 4) +
// (r / 4) mod 4 (in 16-byte units) makes both patterns conflict-free, and in
// both layouts an operand's address is one per-lane base plus an immediate.
// For D = 64 DualLayout falls back to RowsLayout.
// ---------------------------------------------------------------------------
template <int D>
struct RowsLayout {
  static constexpr int ROW = D + 8;                 // elements per stored row
  static constexpr int SLOTS_PER_ROW = ROW * 2 / 16;  // 16-byte slots incl. padding
  __device__ __forceinline__ static int off(int r, int chunk) { return r * ROW + chunk * 8; }
  // offset of a block shift by (r0 rows, c0 elements); r0 % 16 == 0, c0 % 8 == 0
  static constexpr int delta(int r0, int c0) { return r0 * ROW + c0; }
  // transposing read: offset between the two 8-row halves of a 16-row step
  static constexpr int TR_P1 = 8 * ROW;
  static constexpr int elems(int rows) { return rows * ROW; }
  // chunk stored in slot `w` of row r, or -1 for padding
  __device__ __forceinline__ static int chunk_at(int /*r*/, int w) { return w < D / 8 ? w : -1; }
};

template <int D>
struct DualLayout : RowsLayout<D> {};

template <>
struct DualLayout<128> {
  static constexpr int ROW = 160;  // 320-byte pitch
  static constexpr int SLOTS_PER_ROW = 20;
  __device__ __forceinline__ static int off(int r, int chunk) {
    return r * ROW + (((r >> 2) & 3) + chunk) * 8;
  }
  static constexpr int delta(int r0, int c0) { return r0 * ROW + c0; }
  static constexpr int TR_P1 = 8 * ROW + 16;  // +8 rows moves the shift by 2 chunks
  static constexpr int elems(int rows) { return rows * ROW; }
  __device__ __forceinline__ static int chunk_at(int r, int w) {
    const int c = w - ((r >> 2) & 3);
    return (c >= 0 && c < 16) ? c : -1;
  }
};

// Per-lane base (elements) of a row read: row l % 32, chunk l / 32.
template <class L>
__device__ __forceinline__ int row_lane_base() {
  const int l = __lane_id();
  return L::off(l & 31, l >> 5);
}

// Per-lane base (elements) of a transposing read: in each group of 16 lanes,
// lane i addresses row (hh*4 + i/4) and 4 elements starting at column
// (group % 2) * 16 + 4 * (i % 4).
template <class L>
__device__ __forceinline__ int tr_lane_base() {
  const int l = __lane_id();
  const int hh = l >> 5;
  const int g2 = (l >> 4) & 1;
  const int i = l & 15;
  return L::off(hh * 4 + (i >> 2), g2 * 2 + ((i & 3) >> 1)) + (i & 1) * 4;
}

// A operand "X^T" for an LDS tile X[row][col]: lane l gets
//   element j = X[ROW0 + sigma(l/32, j)][COL0 + l % 32],  j = 0..7,
// i.e. 8 rows (in sigma order) of one column, with two ds_read_b64_tr_b16
// (the instruction hands lane i of a 16-lane group element i % 4 of the rows
// addressed by lanes 4e + i/4, e = 0..3), issued with inline assembly so the
// constant part of the address goes into the instruction's offset field.  (The compiler's
// intrinsic for this instruction neither folds offsets nor knows it cannot
// alias in-flight direct-to-LDS copies, and so waits for them.)  The caller
// must wait with tr_wait before using (or copying) the registers.  `lane_addr` = LDS byte
// address of tile + tr_lane_base<L>(); ROW0 % 16 == 0, COL0 % 32 == 0.
struct TrRegs {
  u32x2 lo, hi;
  __device__ __forceinline__ bf16x8 operand() const {
    const bf16x4 blo = __builtin_bit_cast(bf16x4, lo);
    const bf16x4 bhi = __builtin_bit_cast(bf16x4, hi);
    bf16x8 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      out[j] = blo[j];
      out[4 + j] = bhi[j];
    }
    return out;
  }
};

template <class L, int ROW0, int COL0>
__device__ __forceinline__ void tr_issue(uint32_t lane_addr, TrRegs& r) {
  constexpr int off0 = L::delta(ROW0, COL0) * 2;
  constexpr int off1 = off0 + L::TR_P1 * 2;
  static_assert(off1 < 65536, "LDS offset out of range");
  // early-clobber outputs: the second read still needs the address register
  // after the first one has been issued (its data arrives asynchronously)
  asm volatile(
      "ds_read_b64_tr_b16 %0, %2 offset:%3\n\t"
      "ds_read_b64_tr_b16 %1, %2 offset:%4"
      : "=&v"(r.lo), "=&v"(r.hi)
      : "v"(lane_addr), "i"(off0), "i"(off1));
}

// Wait until at most N LDS operations of this wave are outstanding; the
// registers passed in are tied to the wait so that no use is scheduled above it.
template <int N>
__device__ __forceinline__ void tr_wait(TrRegs& a, TrRegs& b, TrRegs& c, TrRegs& d) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(a.lo), "+v"(a.hi), "+v"(b.lo), "+v"(b.hi), "+v"(c.lo), "+v"(c.hi),
                 "+v"(d.lo), "+v"(d.hi)
               : "i"(N));
}
template <int N>
__device__ __forceinline__ void tr_wait(TrRegs& a, TrRegs& b) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a.lo), "+v"(a.hi), "+v"(b.lo), "+v"(b.hi) : "i"(N));
}
template <int N, int K>
__device__ __forceinline__ void tr_wait(TrRegs (&r)[K]) {
  static_assert(K == 2 || K == 4, "tr_wait handles 2 or 4 operands");
  if constexpr (K == 4) tr_wait<N>(r[0], r[1], r[2], r[3]);
  else tr_wait<N>(r[0], r[1]);
}

// A/B operand whose 8 contraction elements are contiguous in an LDS row:
// element j of lane l comes from row (ROW0 + l % 32), column
// (COL0 + (l/32)*8 + j); ROW0 % 16 == 0, COL0 % 8 == 0.  Issued with inline
// assembly for explicitly pipelined reads; wait with row_wait before use.  `lane_addr` =
// LDS byte address of tile + row_lane_base<L>().
template <class L, int ROW0, int COL0>
__device__ __forceinline__ void row_issue(uint32_t lane_addr, u32x4& r) {
  constexpr int off = L::delta(ROW0, COL0) * 2;
  static_assert(off < 65536, "LDS offset out of range");
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(lane_addr), "i"(off));
}
template <int N>
__device__ __forceinline__ void row_wait(u32x4& a) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "i"(N));
}
template <int N>
__device__ __forceinline__ void row_wait(u32x4& a, u32x4& b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "i"(N));
}
template <int N>
__device__ __forceinline__ void row_wait(u32x4& a, u32x4& b, u32x4& c) {
  asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(a), "+v"(b), "+v"(c) : "i"(N));
}
__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& r) { return __builtin_bit_cast(bf16x8, r); }

// Direct global -> LDS copy (buffer_load_dwordx4 ... lds: no registers, no LDS
// store instructions) of a [ROWS x D] bf16 tile (D = 64 or 128) into layout
// L.  One instruction moves 64 lanes x 16 B into 1 KB of consecutive LDS (lane l at
// base + 16 l, the base in M0); lane l of instruction k therefore fills 16-byte
// slot 64 k + l of the tile and fetches whichever global chunk the layout
// stores there.  The copies read through a buffer resource over the tile's
// valid rows: the hardware's range check turns rows >= valid_rows into zeros
// (callers mask them), and padding slots get an offset past any range, so
// they fetch nothing.  Per copy this leaves one M0 write and the load, with
// the lane offsets computed once.  Completion is tracked by vmcnt (wait_dma).
template <class L, int ROWS, int NW>
struct TileDma {
  static constexpr int SLOTS = ROWS * L::SLOTS_PER_ROW;
  static constexpr int INSTS = SLOTS / 64;
  static constexpr int PER_WAVE = (INSTS + NW - 1) / NW;
  static_assert(SLOTS % 64 == 0, "tile must fill whole 1 KB copies");
  static constexpr uint32_t kPadOffset = 0x80000000u;  // out of range for every tile
  uint32_t voff[PER_WAVE];  // byte offset of this lane's chunk in each copy
  int wave;                 // this wave's index (wave-uniform)

  __device__ __forceinline__ void init(size_t gstride) {
    const int l = __lane_id();
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int slot = (wave + NW * i) * 64 + l;
      const int r = slot / L::SLOTS_PER_ROW;
      const int c = L::chunk_at(r, slot % L::SLOTS_PER_ROW);
      voff[i] = c < 0 ? kPadOffset : (uint32_t)(((size_t)r * gstride + (size_t)c * 8) * 2);
    }
  }
  // Source of one tile: rows [0, min(valid_rows, ROWS)) at gbase.  The
  // values are wave-uniform; passing them through readfirstlane tells the
  // compiler so (it would otherwise wrap each copy in a loop over the
  // distinct values of the lanes).  Built once per tile, used by its copies.
  struct Src {
    uint32_t lo, hi;  // address
    int bytes;        // range of the buffer resource
  };
  __device__ __forceinline__ static Src src(const uint16_t* gbase, size_t gstride, int valid_rows) {
    const int rows = valid_rows < ROWS ? valid_rows : ROWS;
    const uint64_t addr = reinterpret_cast<uint64_t>(gbase);
    return {(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)addr),
            (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32)),
            (int)__builtin_amdgcn_readfirstlane((int)((size_t)rows * gstride * 2))};
  }
  __device__ __forceinline__ static void copy(const Src& s, uint32_t voffset, uint16_t* lds) {
    // device pass only: in the host pass the buffer-resource type makes a
    // second kernel's use of the same copy routine fail to instantiate
#if defined(__HIP_DEVICE_COMPILE__)
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(((uint64_t)s.hi << 32) | s.lo), 0, s.bytes, kBufferFlags);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16,
                                             voffset, 0, 0, 0);
#endif
  }
  // Copy i of this wave alone (0 <= i < PER_WAVE, a constant at the call
  // site); a no-op where the wave has no copy i.  Lets a kernel spread its
  // copies over the products of a step instead of queueing them all at once.
  __device__ __forceinline__ void issue_one(int i, const Src& s, uint16_t* lds) const {
    const int k = wave + NW * i;
    // only a wave's last copy can lie past the tile (NW * (PER_WAVE - 1) <
    // INSTS), so the check folds away for the others once i is a constant
    if (INSTS % NW != 0 && i == PER_WAVE - 1 && k >= INSTS) return;  // wave-uniform
    copy(s, voff[i], lds + k * 512);
  }
  // All of this wave's copies of the tile (valid_rows >= 1).
  __device__ __forceinline__ void issue(const uint16_t* gbase, size_t gstride, int valid_rows,
                                        uint16_t* lds) const {
    const Src s = src(gbase, gstride, valid_rows);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int k = wave + NW * i;
      if (INSTS % NW != 0 && i == PER_WAVE - 1 && k >= INSTS) break;  // wave-uniform
      copy(s, voff[i], lds + k * 512);
    }
  }
};

// Wait until this wave's outstanding direct-to-LDS copies (and any other
// vector-memory loads) have landed.  A workgroup barrier after it publishes
// the tile to every wave.
__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Wait until at most N of this wave's vector-memory loads are outstanding
// (loads complete in issue order, so everything older than the last N is done).
template <int N>
__device__ __forceinline__ void wait_dma_n() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}

// ---------------------------------------------------------------------------
// Output tiles.  An accumulator tile has one row (query or key) per lane, so a
// store straight from it writes 16 or 32 bytes to each of 32 rows per
// instruction, and the L2 channels, which take about one request per clock
// each, bound a workgroup's end (256 workgroups of 64 KB of bf16 rows: about
// 4 us).  The wave instead turns its 32 rows through LDS, so that every store
// instruction writes whole 128-byte lines (forward + backward, one sequence:
// 2,500 tokens x 6/2 heads 117.5 -> 112.6 us, 4,096 x 4 146.9 -> 142.5;
// 32 x 512 tokens x 16 heads of 64 274 -> 262; packed 65,536 x 32 heads 10.13 ->
// 10.00 ms; 131,072 x 4 unchanged).
// The caller has passed a workgroup barrier since the tile buffers in `lds`
// were last read.  A wave's LDS operations complete in order, so its own reads
// need no barrier after its writes; the fences keep the compiler's order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}
// The lane index, computed anew: what an epilogue derives from it then holds no
// registers over the tile loop.
__device__ __forceinline__ int fresh_lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
// Four 16-byte LDS reads at byte offsets O0..O3 from addr, waited for.
template <int O0, int O1, int O2, int O3>
__device__ __forceinline__ void lds_read4(uint32_t addr, u32x4 (&v)[4]) {
  static_assert(O0 < 65536 && O1 < 65536 && O2 < 65536 && O3 < 65536, "LDS offset out of range");
  asm volatile(
      "ds_read_b128 %0, %4 offset:%5\n\t"
      "ds_read_b128 %1, %4 offset:%6\n\t"
      "ds_read_b128 %2, %4 offset:%7\n\t"
      "ds_read_b128 %3, %4 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
      : "v"(addr), "i"(O0), "i"(O1), "i"(O2), "i"(O3)
      : "memory");
}

// A wave's accumulator tile into its LDS slot: 32 rows of D floats in 32-column
// blocks of kF32Pitch floats a row (rows 16 bytes apart in the banks:
// conflict-free written by rows of accumulators and read by rows of columns).
constexpr int kF32Pitch = 36;
constexpr int kF32Block = 32 * kF32Pitch;
__device__ __forceinline__ int acc_slot_lane(int l = __lane_id()) {
  return (l & 31) * kF32Pitch + (l >> 5) * 4;
}
__device__ __forceinline__ void acc_to_lds(const f32x16& x, float mul, float* block, int lane_off) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<f32x4*>(block + lane_off + g * 8) =
        f32x4{x[g * 4] * mul, x[g * 4 + 1] * mul, x[g * 4 + 2] * mul, x[g * 4 + 3] * mul};
}

// One wave's 32 rows of D floats, acc * mul (mul: this lane's row's factor), to
// dst (row 0, column 0; `stride` floats from row to row), rows < nrows only;
// accumulate: added to what dst holds.  PASS blocks are turned at a time:
// PASS * kF32Block floats of LDS per wave.  l: the lane index.
template <int D, int PASS>
__device__ __forceinline__ void store_rows_f32(const f32x16 (&acc)[D / 32], float mul, float* dst,
                                               size_t stride, int nrows, bool accumulate,
                                               float* lds, int l = __lane_id()) {
  static_assert((D / 32) % PASS == 0, "whole passes");
  if (nrows <= 0) return;  // wave-uniform
  const int wr = acc_slot_lane(l);
  const int rr = l >> 3, c = (l & 7) * 4;  // read: 8 lanes a row
  const uint32_t rd = lds_addr(lds) + (rr * kF32Pitch + c) * 4;
  // (one address per lane, then uniform steps of 8 rows)
  float* const mine = dst + (size_t)rr * stride + c;
  static_for<D / 32 / PASS>([&](auto Pass) {
    constexpr int p = decltype(Pass)::value * PASS;
#pragma unroll
    for (int b = 0; b < PASS; ++b) acc_to_lds(acc[p + b], mul, lds + b * kF32Block, wr);
    wave_lds_fence();
    static_for<PASS>([&](auto B) {
      constexpr int b = decltype(B)::value;
      u32x4 raw[4];
      constexpr int o = b * kF32Block * 4, st = 8 * kF32Pitch * 4;
      lds_read4<o, o + st, o + 2 * st, o + 3 * st>(rd, raw);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 v = __builtin_bit_cast(f32x4, raw[i]);
        float* to = mine + (size_t)i * 8 * stride + (p + b) * 32;
        if (i * 8 + rr < nrows) {
          if (accumulate) v += *reinterpret_cast<const f32x4*>(to);
          *reinterpret_cast<f32x4*>(to) = v;
        }
      }
    });
  });
}

// The same in bf16 (rounded to nearest even): kBf16Pitch<D> elements a row in
// LDS, 32 rows per wave.
template <int D>
constexpr int kBf16Pitch = D + 8;
template <int D>
__device__ __forceinline__ void store_rows_bf16(const f32x16 (&acc)[D / 32], float mul,
                                                uint16_t* dst, size_t stride, int nrows,
                                                uint16_t* lds) {
  constexpr int P = kBf16Pitch<D>, LANES = D / 8, ROWS = 64 / LANES;
  if (nrows <= 0) return;  // wave-uniform
  const int l = __lane_id();
  const int wr = (l & 31) * P + (l >> 5) * 4;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x16& x = acc[db];
      const f32x2 v01 = {x[g * 4] * mul, x[g * 4 + 1] * mul};
      const f32x2 v23 = {x[g * 4 + 2] * mul, x[g * 4 + 3] * mul};
      *reinterpret_cast<u32x2*>(lds + wr + db * 32 + g * 8) =
          u32x2{__builtin_bit_cast(uint32_t, __builtin_convertvector(v01, bf16x2)),
                __builtin_bit_cast(uint32_t, __builtin_convertvector(v23, bf16x2))};
    }
  wave_lds_fence();
  const int rr = l / LANES, c = (l % LANES) * 8;
  const uint32_t rd = lds_addr(lds) + (rr * P + c) * 2;
  uint16_t* const mine = dst + (size_t)rr * stride + c;
  static_for<32 / ROWS / 4>([&](auto I) {
    constexpr int i0 = decltype(I)::value * 4;
    u32x4 v[4];
    constexpr int o = i0 * ROWS * P * 2, st = ROWS * P * 2;
    lds_read4<o, o + st, o + 2 * st, o + 3 * st>(rd, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if ((i0 + i) * ROWS + rr < nrows)
        *reinterpret_cast<u32x4*>(mine + (size_t)(i0 + i) * ROWS * stride) = v[i];
    }
  });
}

// Key groups: the KG waves of a row group hold partial sums of the same 32 rows
// over different keys, all in LDS slots of D / 32 blocks (slot rg * KG + kg of
// row group rg, at `slot`).  Wave kg combines the rows [kg, kg + 1) * 32 / KG, 8
// consecutive columns of a row per lane: weights(row, w) sets the groups'
// weights, then out(row, column, x) gets x = sum_j w[j] * partial j.
template <int D, int KG, class W, class F>
__device__ __forceinline__ void combine_groups(const float* slot, int kg, W&& weights, F&& out) {
  constexpr int LANES = D / 8, ROWS = 64 / LANES, SLOT = D / 32 * kF32Block * 4;
  const int l = __lane_id();
  const int c = (l % LANES) * 8;
  static_for<32 / KG / ROWS>([&](auto I) {
    const int r = kg * (32 / KG) + decltype(I)::value * ROWS + l / LANES;
    const uint32_t addr =
        lds_addr(slot) + ((c >> 5) * kF32Block + r * kF32Pitch + (c & 31)) * 4;
    float w[KG];
    weights(r, w);
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    static_for<KG / 2>([&](auto J) {
      constexpr int j = decltype(J)::value * 2, o = j * SLOT;
      u32x4 raw[4];
      lds_read4<o, o + 16, o + SLOT, o + SLOT + 16>(addr, raw);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[e] += w[j] * __uint_as_float(raw[e >> 2][e & 3]) +
                w[j + 1] * __uint_as_float(raw[2 + (e >> 2)][e & 3]);
    });
    out(r, c, x);
  });
}

// Work schedule built by plan_kernel: items are (segment, level) pairs with
// level j meaning "tile j of the segment" (forward / dQ) or "tile nt-1-j"
// (dK/dV); a higher level is a heavier causal tile.  Two orders of the same
// items:
//   * level-major: by descending level over all segments, so the heaviest
//     tiles of every segment start first;
//   * segment-major: the longest segment's tiles (heaviest first), then the
//     next longest segment's, and so on.  Workgroups that run at the same
//     time then hold neighbouring tiles of one segment, which stream the same
//     rows or keys, so those reads are shared in L2; the heaviest tiles of
//     the longest segments still start first.  Taken when the longest
//     segment has at least 8 tiles (measured on the packed 65,536-token
//     batch of 25 segments, 32 heads: fwd+bwd 682 -> 754 TFLOP/s; packed
//     GQA batches of 9-53 segments +1 to +7 %); with only a few tiles per
//     segment (6,000 segments of at most 300 tokens) level-major keeps the
//     tail shorter (4 % faster there).
// Returns false when `item` is past the end.
//
// A batch of few segments needs no plan_kernel: every workgroup places its item
// itself from cu (plan_direct), in the same orders.
struct Plan {
  const int32_t* cu;      // packed segments' offsets [n + 1]
  int32_t n;              // segments; direct: placed from cu, no schedule
  int32_t direct;
  int32_t tile_log2;      // rows or keys per tile
  const int32_t* order;   // segments sorted by tile count, descending [N]
  const int32_t* start;   // first item of each level [max_nt] (level-major)
  const int32_t* total;   // number of items [1]
  const int32_t* cnt;     // segments with more than j tiles [max_nt]
  const int32_t* before;  // first item of the segments with j + 1 tiles [max_nt]
                          // (segment-major)
  int32_t max_nt;
  int32_t seg_major;      // 1: segment-major order
};

// Head and position in that head's work list of workgroup b of a launch of
// n = nheads x (entries per head).  The hardware deals workgroups to the 8
// XCDs round-robin (workgroup b runs on XCD b % 8; each XCD has 32 CUs and
// its own L2), so with head = b % nheads and entry = b / nheads a head is
// spread over 8 / nheads XCDs, each taking every (8 / nheads)-th entry, and
// what the entries running at a time on one XCD stream spreads over a wide
// window.  When nheads divides 8, each of a head's XCDs instead takes 32
// consecutive entries of the head's heaviest-first list at a time (the
// blocks of a head's XCDs run in reverse order every other round, so no XCD
// always gets the lightest block; with 8 heads this is the plain order).
// Measured at 131,072 tokens: dK/dV with 1 kv head -4.7 %, 2 kv heads
// -3.9 %, 4 kv heads -0.3 to -0.8 %; forward and dQ with 4 query heads
// -1.4 % and -0.6 %.  The last, partial round is dealt in the same blocks: in the
// plain order its heavy and light entries met the first round's unevenly (16,200
// tokens x 4 heads over 508 workgroups: forward 308 -> 267 us, dQ 406 -> 360,
// dK/dV 553 -> 487).  Other head counts and launches of less than a round
// keep the plain order.  A bijection on [0, n).
__device__ __forceinline__ void xcd_order(int b, int n, int nheads, int& head, int& entry) {
  constexpr int kXcd = 8, kPer = 32, kRound = kXcd * kPer;
  head = b % nheads;
  entry = b / nheads;
  if (kXcd % nheads != 0 || n < kRound) return;
  const int g = kXcd / nheads;          // XCDs per head
  const int sub = (b % kXcd) / nheads;  // which of them
  const int s = b / kXcd;               // workgroup index on this XCD
  const int r = s / kPer, q = s % kPer;
  // the head's entries of this round, dealt to its XCDs one by one: XCD i has
  // per + (i < more) of them
  const int mine = min(n / nheads - r * g * kPer, g * kPer);
  const int per = mine / g, more = mine % g;
  const int first = (r & 1) ? mine - (sub + 1) * per - min(sub + 1, more)
                            : sub * per + min(sub, more);
  entry = r * g * kPer + first + q;
}

// Split-K of a launch whose work items cannot fill the chip: each item's
// inner loop (its units: the key tiles of a query tile, or the query steps of
// a key tile over the query heads of its group) is cut into contiguous parts,
// one workgroup each, whose partial results a second kernel combines.
//   * uniform (cap == 0): every item in `parts` parts;
//   * balanced (cap > 0, single-segment launches only): item i (the i-th
//     heaviest) in ceil(units(i) / cap) parts, so that light items are not
//     cut into slivers while the heaviest sets the launch's time; `parts` is
//     then the most parts of any item (the number of partial slices).
// A part p of an item with n parts and u units takes units
// [p u / n, (p + 1) u / n).
struct Split {
  int parts;
  int cap;
  int kind;    // 0: items are query tiles of `rows` rows, units key tiles of `keys`
               // 1: items are key tiles of `keys` keys, units steps of `rows` rows
  int nitems;  // items per head (balanced)
  int total;   // tokens of the segment (balanced)
  int causal;
  int rows, keys;
  int group;   // query heads per kv head (kind 1)

  // units of inner work of item i (balanced), i = 0 the heaviest
  __host__ __device__ int units(int i) const {
    if (kind == 0) {
      const int q0 = (nitems - 1 - i) * rows;
      const int kv_end = causal ? (q0 + rows < total ? q0 + rows : total) : total;
      return (kv_end + keys - 1) / keys;
    }
    const int qstart = causal ? i * keys : 0;
    return (total - qstart + rows - 1) / rows * group;
  }
  __host__ __device__ int nparts(int i) const { return cap ? (units(i) + cap - 1) / cap : parts; }
  // item of the query row (kind 0) or key (kind 1) at `pos`
  __host__ __device__ int item_of(int pos) const {
    return kind == 0 ? nitems - 1 - pos / rows : pos / keys;
  }
};

// Item, part and part count of workgroup `entry` (of one head) under split
// sp.  Balanced: the parts of an item are consecutive entries, heavier items
// first; one pass of the wave over the items (a split launch has fewer than
// 512 items) finds the entry's item.  Returns false past the last part.  All
// results are wave-uniform.
__device__ __forceinline__ bool split_entry_scan(const Split& sp, int entry, int& item, int& part,
                                                 int& nparts);
__device__ __forceinline__ bool split_entry(const Split& sp, int entry, int& item, int& part,
                                            int& nparts) {
  bool ok = true;
  if (sp.cap == 0) {
    item = entry / sp.parts;
    part = entry % sp.parts;
    nparts = sp.parts;
  } else {
    ok = split_entry_scan(sp, entry, item, part, nparts);
  }
  // wave-uniform: kept in scalar registers
  item = __builtin_amdgcn_readfirstlane(item);
  part = __builtin_amdgcn_readfirstlane(part);
  nparts = __builtin_amdgcn_readfirstlane(nparts);
  return ok;
}
__device__ __forceinline__ bool split_entry_scan(const Split& sp, int entry, int& item, int& part,
                                                 int& nparts) {
  const int l = __lane_id();
  const int per = (sp.nitems + 63) >> 6;  // items per lane
  int mine = 0;
  for (int k = 0; k < per; ++k) {
    const int i = l * per + k;
    if (i < sp.nitems) mine += sp.nparts(i);
  }
  int incl = mine;  // inclusive prefix sum over the lanes
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(incl, off);
    if (l >= off) incl += t;
  }
  const unsigned long long hit = __ballot(entry >= incl - mine && entry < incl);
  if (hit == 0) return false;
  const int src = __ffsll((long long)hit) - 1;  // the lane whose items hold the entry
  int base = __shfl(incl - mine, src);
  for (int k = 0; k < per; ++k) {
    const int i = src * per + k;
    const int n = sp.nparts(i);
    if (entry < base + n) {
      item = i;
      part = entry - base;
      nparts = n;
      return true;
    }
    base += n;
  }
  return false;
}

// Most segments that a workgroup places itself: one per lane in the
// segment-major order (a pass over the segments gives every lane its segment's
// first item, about 5 instructions a segment), two per lane in the level-major
// order (a ballot per level and 64 segments).  Against plan_kernel (5-6 us and a
// launch per call): forward + backward of 33 segments of 184 tokens x 8 heads of
// 64 49.2 -> 40.0 us, 70 of 16-107 x 16 59.3 -> 51.7, 32 of 512 x 16 272 -> 257;
// 122 of 16-512 tokens x 32/8 heads unchanged (the kernels take 2 % longer).  (The
// segment-major order's pass also bounds segments x workgroups.)
constexpr int kDirectSegMajor = 64;
constexpr int kDirectChunks = 2;

__device__ __forceinline__ bool plan_direct(const Plan& p, int item, int& lo, int& hi, int& level) {
  const int l = __lane_id();
  const int up = (1 << p.tile_log2) - 1;
  if (p.seg_major) {
    const int a = l < p.n ? p.cu[l] : 0, b = l < p.n ? p.cu[l + 1] : 0;
    const int v = min((b - a + up) >> p.tile_log2, p.max_nt);
    int start = 0;  // tiles of the segments before this lane's
    for (int j = 0; j < p.n; ++j) {
      const int vj = __builtin_amdgcn_readlane(v, j);
      start += (vj > v || (vj == v && j < l)) ? vj : 0;
    }
    const uint64_t hit = __builtin_amdgcn_ballot_w64(item >= start && item < start + v);
    if (hit == 0) return false;
    const int src = __builtin_ctzll(hit);
    lo = __builtin_amdgcn_readlane(a, src);
    hi = __builtin_amdgcn_readlane(b, src);
    level = __builtin_amdgcn_readlane(v, src) - 1 - (item - __builtin_amdgcn_readlane(start, src));
    return true;
  }
  int a[kDirectChunks], b[kDirectChunks], v[kDirectChunks];
#pragma unroll
  for (int c = 0; c < kDirectChunks; ++c) {
    const int s = c * 64 + l;
    a[c] = s < p.n ? p.cu[s] : 0;
    b[c] = s < p.n ? p.cu[s + 1] : 0;
  }
#pragma unroll
  for (int c = 0; c < kDirectChunks; ++c) v[c] = min((b[c] - a[c] + up) >> p.tile_log2, p.max_nt);
  int rel = item;  // position among the items of the levels not yet passed
  for (level = p.max_nt - 1; level >= 0; --level) {
#pragma unroll
    for (int c = 0; c < kDirectChunks; ++c) {
      const uint64_t m = __builtin_amdgcn_ballot_w64(v[c] > level);
      const int k = __builtin_popcountll(m);
      if (rel < k) {
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64(v[c] > level && rank == rel));
        lo = __builtin_amdgcn_readlane(a[c], src);
        hi = __builtin_amdgcn_readlane(b[c], src);
        return true;
      }
      rel -= k;
    }
  }
  return false;
}

// Segment [lo, hi) and level of an item; false when it is past the end.
__device__ __forceinline__ bool plan_lookup(const Plan& p, int item, int& lo, int& hi, int& level) {
  if (p.n == 1) {  // one segment (or chunk) [0, hi): item i is its level max_nt - 1 - i
    if (item >= p.max_nt) return false;
    lo = 0;
    level = p.max_nt - 1 - item;
    return true;
  }
  if (p.direct) return plan_direct(p, item, lo, hi, level);
  if (item >= *p.total) return false;
  const int32_t* first = p.seg_major ? p.before : p.start;
  // smallest j with first[j] <= item (first is non-increasing in j)
  int low = 0, high = p.max_nt - 1;
  while (low < high) {
    const int mid = (low + high) >> 1;
    if (first[mid] <= item) high = mid;
    else low = mid + 1;
  }
  int seg;
  if (!p.seg_major) {
    level = low;
    seg = p.order[item - p.start[low]];
  } else {
    // the segments with v = low + 1 tiles hold v consecutive items each, from
    // the heaviest tile (level v - 1) down; they are order[cnt[v] ...]
    const int v = low + 1;
    const int rel = item - first[low];
    const int g = rel / v;
    level = low - (rel - g * v);
    seg = p.order[(v < p.max_nt ? p.cnt[v] : 0) + g];
  }
  lo = p.cu[seg];
  hi = p.cu[seg + 1];
  return true;
}

}  // namespace pdy
