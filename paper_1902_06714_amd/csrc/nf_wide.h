// The fp32 contractions of every layer that has no kernel of its own (forward,
// output and hidden deltas, tendencies; sections 3.2 - 3.5), on the bf16
// matrix cores.
//
// Every operand is split into three bf16 parts and a product formed as six
// (nf_parts.h).
//
// Why: the fp32 matrix instruction gives 64 flops a clock and SIMD, the bf16
// one 1024, so six of them are worth 171, 2.7 times as many.  The sums are no
// less exact: in the 64 x 64 and 128 x 128 tiles the leading products have
// accumulators of their own, rounded once for 16 k, in the 256 x 256 tile all
// six share one, 6 roundings for 16 k, not 8.  Relative errors (2-norm)
// against fp64, operands of both signs / positive, x 1e-7, and those of the
// fp32 instruction in the contraction that this replaced:
//   tile        contraction                            parts        fp32
//   64 x 64     600 x 300, k = 1024 in 8 pieces        0.8 / 0.4    2.1 / 0.7
//   128 x 128   4096 x 1024, k = 784                   1.6 / 1.4    5.0 / 3.9
//               tendencies 1024 x 1024, k = 4096       1.9 / 0.9    5.8 / 2.4
//   256 x 256   8192 x 4096, k = 256                   2.4 / 1.8    2.9 / 2.2
//               k = 1024                               4.9 / 2.9    5.7 / 4.3
//               k = 4096                               10.0 / 5.3   11.5 / 8.4
//               tendencies 4096 x 4096, k = 8192       14.4 / 8.5   16.2 / 13.4
//
// What bounds it: on large problems the power limit and the matrix cores (the
// clock and how busy they are: profiles/gemm_kernels__4096x4-10_batch8192.md),
// else the vector instructions of the split, 13 for two values, which a wave
// does not overlap with its own matrix instructions (a second wave on the SIMD
// does: per matrix instruction 39 clocks alone, 64 with four vector
// instructions in the same wave, 43 with them in another).  Hence tiles as
// large as the grid allows, each operand split once per tile on its way to
// LDS, and for the 64 x 64 tile loading waves of their own.
// Measured (us, random operands, sustained, against the fp32 contraction that
// this replaced, on one card): forward 8192 x 4096 x 4096 1166, 236 TFLOP/s,
// against 1931; 4096 x 1024 x 1024 58 against 85; 10000 x 1024 x 1024 157 against 224;
// tendencies 1024 x 1024 over 4096 in four pieces 58 against 86, 4096 x 4096 over
// 8192 1117 against 2045; 3003 x 517 x 1001 34 against 47 and a fold; 16 x 255 x 300 7.4
// against 9.3.
#pragma once

#include <type_traits>

#include "nf_act.h"
#include "nf_internal.h"
#include "nf_parts.h"
#include "nf_split.h"

namespace nf {

constexpr int WIDE_KI = 16;      // k of one 32x32x16 matrix instruction
constexpr int WIDE_ROLES_BK = 32;   // k of a stage of the tiles with loading waves

// bytes of LDS of 8 k of R rows, and of nb stages of BK
constexpr int wide_half(int R, int BK) { return R * 16 + (BK > 16 ? 64 : 128); }
constexpr int wide_lds(int BM, int BN, int BK, int nb) {
  return nb * 3 * (BK / 8) * (wide_half(BM, BK) + wide_half(BN, BK));
}

// Global -> registers -> LDS of one R x BK operand tile X(r, k) by NT threads,
// Q quads of 4 values each.  In LDS each of the three parts is [BK / 8][R][8]
// bf16 (the groups of 8 k 64 or 128 bytes further apart, in other banks): the 8
// consecutive k of a row that a lane's operand takes are one 16-byte chunk,
// and the 32 rows of a half-wave's read are contiguous.
// KC: quad i holds 4 consecutive k of one row, loaded at once (the hardware
// takes 16-byte loads at any 4-byte address).  VEC: rows are 16-byte aligned
// and their pitch padding is zero, so a quad may reach past the last k;
// otherwise the last, partial stage is read one value at a time, since the
// row's end may be the end of the allocation.  Not KC: a quad holds 4
// consecutive k of one row from 4 rows of memory, and two quads of a thread
// that follow one another make a whole chunk.
template <int R, int BK, int NT, bool KC, bool VEC>
struct SplitLoader {
  static constexpr int Q = R * BK / (4 * NT);
  static constexpr int HALF = wide_half(R, BK);  // bytes of 8 k of every row
  static constexpr int PART = BK / 8 * HALF;     // bytes of one part
  static_assert(Q >= 1 && Q * 4 * NT == R * BK, "whole quads");
  static constexpr int C = KC || Q == 1 ? 1 : 2; // quads of a run of k
  float v[4 * Q];

  // row and k of quad i
  __device__ __forceinline__ static int row(int tid, int i) {
    return KC ? (tid + i * NT) / (BK / 4) : (tid + i / C * NT) % R;
  }
  __device__ __forceinline__ static int kof(int tid, int i) {
    return KC ? tid % (BK / 4) * 4 : ((tid + i / C * NT) / R) * 4 * C + i % C * 4;
  }

  // k0: first k of the stage
  __device__ __forceinline__ void load(const float* __restrict__ X, int64_t ld, int rmax, int kend,
                                       int r0, int k0, int tid) {
    const int left = kend - k0;                  // k of the stage inside the piece
    const int ldi = (int)ld;
    if constexpr (KC) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(X + (int64_t)r0 * ld + k0), (short)0, (int)TILE_OOB, 0x00020000);
      const int k = kof(tid, 0);
      unsigned at[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const int r = row(tid, i);
        at[i] = r0 + r < rmax ? (unsigned)(r * ldi + k) * 4u : TILE_OOB;
      }
      if (VEC || left >= BK || left <= 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const floatx4 u = __builtin_bit_cast(
              floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, k < left ? at[i] : TILE_OOB, 0, 0));
#pragma unroll
          for (int c = 0; c < 4; ++c) v[4 * i + c] = u[c];
        }
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            v[4 * i + c] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, k + c < left ? at[i] + 4u * c : TILE_OOB, 0, 0));
      }
    } else {
      // the buffer ends at the stage's or the piece's last k
      const int rows = __builtin_amdgcn_readfirstlane(min(max(left, 0), BK));
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(X + (int64_t)k0 * ld), (short)0, rows * ldi * 4, 0x00020000);
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const int r = row(tid, i);
        const unsigned at = r0 + r < rmax ? (unsigned)(r0 + r + kof(tid, i) * ldi) * 4u : TILE_OOB;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          v[4 * i + c] = __builtin_bit_cast(
              float, __builtin_amdgcn_raw_buffer_load_b32(rs, at + (unsigned)(c * ldi) * 4u, 0, 0));
      }
    }
  }

  // each quad's values added to its sum (in the tendencies the sums over the
  // rows of A are the bias tendencies)
  __device__ __forceinline__ void add_up(float (&sum)[Q]) const {
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) sum[i] += v[4 * i + c];
  }

  // the three parts of every value
  __device__ __forceinline__ void store(char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < Q; i += C) {
      unsigned h[2 * C], m[2 * C], l[2 * C];
#pragma unroll
      for (int c = 0; c < 2 * C; ++c)
        split3(v[4 * i + 2 * c], v[4 * i + 2 * c + 1], h[c], m[c], l[c]);
      const int k = kof(tid, i);
      char* at = lds + (k >> 3) * HALF + row(tid, i) * 16 + (k & 7) * 2;
      if constexpr (C == 2) {
        *reinterpret_cast<uintx4*>(at) = uintx4{h[0], h[1], h[2], h[3]};
        *reinterpret_cast<uintx4*>(at + PART) = uintx4{m[0], m[1], m[2], m[3]};
        *reinterpret_cast<uintx4*>(at + 2 * PART) = uintx4{l[0], l[1], l[2], l[3]};
      } else {
        *reinterpret_cast<uintx2*>(at) = uintx2{h[0], h[1]};
        *reinterpret_cast<uintx2*>(at + PART) = uintx2{m[0], m[1]};
        *reinterpret_cast<uintx2*>(at + 2 * PART) = uintx2{l[0], l[1]};
      }
    }
  }
};

__device__ __forceinline__ bf16x8 fragment(const char* lds) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(lds));
}

// Buffers over the rows of a tile (BM rows of pitch ld at row m0 of a matrix
// of M rows): rows past the matrix read as zeros and drop their stores, as do
// columns whose offset is set past the buffer.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rows(const float* p, int64_t ld, int m0, int M,
                                                            int BM) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)(p + (int64_t)m0 * ld), (short)0,
                                           min(M - m0, BM) * (int)ld * 4, 0x00020000);
}

__device__ __forceinline__ void put(const __amdgpu_buffer_rsrc_t& rs, unsigned off, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), rs, off, 0, 0);
}
__device__ __forceinline__ float get(const __amdgpu_buffer_rsrc_t& rs, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}

// Calls f(i, j, off) for the blocks of the wave's accumulators; entry v of a
// block lies at off(v) bytes in a tile of pitch ld (past every buffer where
// the column is past the matrix): accumulator register v of a lane holds row
// 8 (v / 4) + 4 (lane / 32) + v % 4 and column lane % 32 of its block.
__device__ __forceinline__ auto block_offsets(int i, int j, int64_t ld, int n0, int N, int wm, int wn,
                                              int lane) {
  const int n = n0 + wn + j * 32 + (lane & 31), ldi = (int)ld;
  const unsigned col = n < N ? (unsigned)((wm + 4 * (lane >> 5)) * ldi + n) * 4u : TILE_OOB;
  return [=](int v) { return col + (unsigned)((i * 32 + 8 * (v >> 2) + (v & 3)) * ldi) * 4u; };
}
template <int TM, int TN, class F>
__device__ __forceinline__ void each_block(int64_t ld, int n0, int N, int wm, int wn, int lane, F f) {
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      f(i, j, block_offsets(i, j, ld, n0, N, wm, wn, lane));
      __builtin_amdgcn_sched_barrier(0);   // one block's offsets in registers at a time
    }
}
// The same with the values of a second matrix at those places, read from
// buffer r: all loads of some blocks before f's stores for them (a load may
// not move up across the stores, so one at a time each would be waited for).
template <int TM, int TN, class F>
__device__ __forceinline__ void with_input(const __amdgpu_buffer_rsrc_t& r, int64_t ld, int n0, int N,
                                           int wm, int wn, int lane, F f) {
  constexpr int NB = TM * TN, G = NB > 4 ? 2 : NB;
#pragma unroll
  for (int g = 0; g < NB; g += G) {
    float x[G][16];
#pragma unroll
    for (int b = 0; b < G; ++b) {
      const auto off = block_offsets((g + b) % TM, (g + b) / TM, ld, n0, N, wm, wn, lane);
#pragma unroll
      for (int v = 0; v < 16; ++v) x[b][v] = get(r, off(v));
    }
#pragma unroll
    for (int b = 0; b < G; ++b) {
      f((g + b) % TM, (g + b) / TM, block_offsets((g + b) % TM, (g + b) / TM, ld, n0, N, wm, wn, lane),
        x[b]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}


// The biases of a wave's columns, requested before the products so that a small
// launch does not wait for them after.
template <int TN, int EPI>
struct Biases {
  float b[TN];
  __device__ __forceinline__ Biases(const GemmParamsT<float>& p, int n0, int wn, int lane) {
    if constexpr (EPI == EPI_FWD_STASH || EPI == EPI_FWD_OUT || EPI == EPI_FWD_DELTA) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn + j * 32 + (lane & 31);
        b[j] = n < p.N ? p.bias[n] : 0.f;
      }
    }
  }
};

template <int BM, int TM, int TN, int EPI, int ACT>
__device__ __forceinline__ void forward_epilogue(const GemmParamsT<float>& p, floatx16 (&acc)[TM][TN],
                                                 const float (&bias)[TN], int m0, int n0, int wm, int wn,
                                                 int lane) {
  const __amdgpu_buffer_rsrc_t r0 = tile_rows(p.out0, p.ld0, m0, p.M, BM);
  // out1 has out0's pitch (the host checks)
  const __amdgpu_buffer_rsrc_t r1 = tile_rows(EPI == EPI_FWD_STASH ? p.out1 : p.out0, p.ld0, m0, p.M, BM);
  each_block<TM, TN>(p.ld0, n0, p.N, wm, wn, lane, [&](int i, int j, auto off) {
    // 8 rows at a time, those past the matrix left out: a small batch waits for
    // every activation (one sample, 8 inputs, 300 units: 5.9 us with all, 4.3)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (i * 32 + 8 * q >= p.M - m0 - wm) break;
#pragma unroll
      for (int v = 4 * q; v < 4 * q + 4; ++v) {
        float f, fp;
        act_eval<float>(ACT, acc[i][j][v] + bias[j], f, fp);
        put(r0, off(v), f);
        if constexpr (EPI == EPI_FWD_STASH) put(r1, off(v), fp);
      }
    }
  });
}

// The output delta: the targets' rows have a pitch of their own.
template <int BM, int TM, int TN, int ACT>
__device__ __forceinline__ void delta_epilogue(const GemmParamsT<float>& p, floatx16 (&acc)[TM][TN],
                                               const float (&bias)[TN], int m0, int n0, int wm, int wn,
                                               int lane) {
  const __amdgpu_buffer_rsrc_t r0 = tile_rows(p.out0, p.ld0, m0, p.M, BM);
  const __amdgpu_buffer_rsrc_t ry = tile_rows(p.aux, p.ldaux, m0, p.M, BM);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn + j * 32 + (lane & 31), row = wm + 4 * (lane >> 5);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float y[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = row + i * 32 + 8 * (v >> 2) + (v & 3);
        y[v] = get(ry, n < p.N ? (unsigned)(m * (int)p.ldaux + n) * 4u : TILE_OOB);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (i * 32 + 8 * q >= p.M - m0 - wm) break;
#pragma unroll
        for (int v = 4 * q; v < 4 * q + 4; ++v) {
          const int m = row + i * 32 + 8 * q + (v & 3);
          float f, fp;
          act_eval<float>(ACT, acc[i][j][v] + bias[j], f, fp);
          put(r0, n < p.N ? (unsigned)(m * (int)p.ld0 + n) * 4u : TILE_OOB, (f - y[v]) * fp);
        }
      }
    }
  }
}

template <int BM, int TM, int TN, int EPI>
__device__ __forceinline__ void wide_epilogue(const GemmParamsT<float>& p, floatx16 (&acc)[TM][TN],
                                              const Biases<TN, EPI>& bias, int m0, int n0, int wm, int wn,
                                              int lane, int bz) {
  if constexpr (EPI == EPI_FWD_STASH || EPI == EPI_FWD_OUT || EPI == EPI_FWD_DELTA) {
    // one switch per tile, not one per entry
    auto emit = [&](auto act) {
      if constexpr (EPI == EPI_FWD_DELTA)
        delta_epilogue<BM, TM, TN, act.value>(p, acc, bias.b, m0, n0, wm, wn, lane);
      else
        forward_epilogue<BM, TM, TN, EPI, act.value>(p, acc, bias.b, m0, n0, wm, wn, lane);
    };
    switch (p.act) {
      case ACT_GAUSSIAN: emit(std::integral_constant<int, ACT_GAUSSIAN>()); break;
      case ACT_RELU: emit(std::integral_constant<int, ACT_RELU>()); break;
      case ACT_SIGMOID: emit(std::integral_constant<int, ACT_SIGMOID>()); break;
      case ACT_TANH: emit(std::integral_constant<int, ACT_TANH>()); break;
      default: emit(std::integral_constant<int, ACT_STEP>()); break;
    }
  } else if constexpr (EPI == EPI_BWD) {
    // aux has out0's pitch; a block's loads before its stores, which the
    // compiler may not move them across
    const __amdgpu_buffer_rsrc_t r0 = tile_rows(p.out0, p.ld0, m0, p.M, BM);
    const __amdgpu_buffer_rsrc_t ra = tile_rows(p.aux, p.ld0, m0, p.M, BM);
    with_input<TM, TN>(ra, p.ld0, n0, p.N, wm, wn, lane, [&](int i, int j, auto off, const float* x) {
#pragma unroll
      for (int v = 0; v < 16; ++v) put(r0, off(v), acc[i][j][v] * x[v]);
    });
  } else if constexpr (EPI == EPI_DW_SGD) {
    // the tendencies and both parameter buffers share one pitch
    const __amdgpu_buffer_rsrc_t rg = tile_rows(p.out0, p.ld0, m0, p.M, BM);
    const __amdgpu_buffer_rsrc_t ri = tile_rows(p.Win, p.ld0, m0, p.M, BM);
    const __amdgpu_buffer_rsrc_t rw = tile_rows(p.W, p.ld0, m0, p.M, BM);
    with_input<TM, TN>(ri, p.ld0, n0, p.N, wm, wn, lane, [&](int i, int j, auto off, const float* x) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float c = acc[i][j][v];
        put(rg, off(v), c);
        put(rw, off(v), fma_t(-p.scale, c, x[v]));
      }
    });
  } else {
    const __amdgpu_buffer_rsrc_t r0 = tile_rows(p.partial + (int64_t)bz * p.pstride, p.ld0, m0, p.M, BM);
    each_block<TM, TN>(p.ld0, n0, p.N, wm, wn, lane, [&](int i, int j, auto off) {
#pragma unroll
      for (int v = 0; v < 16; ++v) put(r0, off(v), acc[i][j][v]);
    });
  }
}

// The k range of piece bz (the whole range outside the piece epilogues), in
// scalar registers: it comes from divisions, which run on the vector unit, and
// a buffer access with anything but scalar registers in its resource loops.
template <int EPI>
__device__ __forceinline__ void piece_range(const GemmParamsT<float>& p, int bz, int& kbeg, int& kend) {
  kbeg = 0;
  kend = p.K;
  if constexpr (EPI == EPI_DW_SGD || EPI == EPI_DW_PARTIAL || EPI == EPI_FWD_PIECE ||
                EPI == EPI_BWD_PIECE) {
    const int shard = bz / p.nsub, sub = bz % p.nsub;
    const int sb = shard * p.shard_len;
    kbeg = sb + sub * p.sub_len;
    kend = __builtin_amdgcn_readfirstlane(min(kbeg + p.sub_len, sb + p.shard_len));
    kbeg = __builtin_amdgcn_readfirstlane(kbeg);
  }
}

template <int TM, int TN>
__device__ __forceinline__ void clear(floatx16 (&acc)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// A lane's values of 16 k of an operand X(r, k) for eight 32x32x2 fp32
// instructions: row r0 + lane % 32, k0 + 8 q + 4 (lane / 32) + c for instruction 4 q
// + c, zeros past the last row and the last k (`left` of them from k0).
template <bool KC>
__device__ __forceinline__ void row_values(const float* X, int64_t ld, int r0, int rmax, int k0,
                                           int left, int lane, float (&x)[8]) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(X + (KC ? (int64_t)r0 * ld + k0 : (int64_t)k0 * ld + r0)), (short)0, (int)TILE_OOB,
      0x00020000);
  const int r = lane & 31, h = 4 * (lane >> 5);
  const bool ok = r0 + r < rmax;
  if (KC && left >= 16) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const floatx4 u = __builtin_bit_cast(
          floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                       rs, ok ? (unsigned)(r * (int)ld + 8 * q + h) * 4u : TILE_OOB, 0, 0));
#pragma unroll
      for (int c = 0; c < 4; ++c) x[4 * q + c] = u[c];
    }
  } else {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 8 * (s >> 2) + h + (s & 3);
      x[s] = get(rs, ok && k < left ? (unsigned)(KC ? r * (int)ld + k : k * (int)ld + r) * 4u : TILE_OOB);
    }
  }
}

// The scale of the parts taken out of a wave's sums.  A block with sums that
// cannot be trusted is formed again on the fp32 matrix cores, straight from
// memory (the 32x32x2 instruction shares the accumulators' layout), and those
// sums, and no others, are replaced: each depends on its own row and column
// alone.
template <bool AKC, bool BKC, int TM, int TN>
__device__ __forceinline__ void finish_sums(const GemmParamsT<float>& p, floatx16 (&acc)[TM][TN], int m0,
                                            int n0, int wm, int wn, int kbeg, int kend, int lane) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      bool bad = false;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        bad |= parts_doubtful(acc[i][j][v]);
        acc[i][j][v] *= PARTS_UNSCALE;
      }
      if (__any(bad)) {
        const int m = m0 + wm + i * 32, n = n0 + wn + j * 32;
        floatx16 f32 = {};
#pragma unroll 1
        for (int k0 = kbeg; k0 < kend; k0 += 16) {
          float x[8], y[8];
          row_values<AKC>(p.A, p.lda, m, p.M, k0, kend - k0, lane, x);
          row_values<BKC>(p.B, p.ldb, n, p.N, k0, kend - k0, lane, y);
#pragma unroll
          for (int s = 0; s < 8; ++s) f32 = __builtin_amdgcn_mfma_f32_32x32x2f32(x[s], y[s], f32, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v)
          acc[i][j][v] = parts_doubtful(acc[i][j][v]) ? f32[v] : acc[i][j][v];
      }
    }
}

// The bias tendencies of a tile's rows from the sums of the quads of k that
// each loading thread kept, added in k order.  Starts with a barrier inside.
template <class LA, int BM, int BK, int EPI>
__device__ __forceinline__ void put_bias_sums(const GemmParamsT<float>& p, const float (&bsum)[LA::Q],
                                              int m0, int bz, int tid, float* sums) {
#pragma unroll
  for (int i = 0; i < LA::Q; ++i) sums[(LA::kof(tid, i) >> 2) * BM + LA::row(tid, i)] = bsum[i];
  __syncthreads();
  const int m = m0 + tid;
  if (tid < BM && m < p.M) {
    float g = sums[tid];
#pragma unroll
    for (int k = 1; k < BK / 4; ++k) g += sums[tid + k * BM];
    if constexpr (EPI == EPI_DW_SGD) {
      p.gbias[m] = g;
      p.bvec[m] = fma_t(-p.scale, g, p.bin[m]);
    } else {
      p.pbias[(int64_t)bz * p.M + m] = g;
    }
  }
}

#define NF_MMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)

// One BM x BN tile by (BM / WM) x (BN / WN) waves of WM x WN that all load and
// multiply.  FD: the next stage's operands are read from LDS into a second set
// of registers while this stage's are multiplied (one wave per SIMD has
// nothing else to hide those reads); otherwise a block row's are read just
// before its products.
template <int BM, int BN, int WM, int WN, bool FD, bool AKC, bool BKC, bool AV, bool BV, int EPI>
__device__ __forceinline__ void wide_tile(const GemmParamsT<float>& p, int bx, int by, int bz,
                                          char* lds) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  constexpr int TM = WM / 32, TN = WN / 32, BK = WIDE_KI;
  typedef SplitLoader<BM, BK, NT, AKC, AV> LA;
  typedef SplitLoader<BN, BK, NT, BKC, BV> LB;
  constexpr int STAGE = 3 * (LA::PART + LB::PART);
  static_assert(2 * STAGE == wide_lds(BM, BN, BK, 2), "LDS size");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave % (BM / WM)) * WM;
  const int wn = (wave / (BM / WM)) * WN;
  const int m0 = __builtin_amdgcn_readfirstlane(bx * BM), n0 = __builtin_amdgcn_readfirstlane(by * BN);
  int kbeg, kend;
  piece_range<EPI>(p, bz, kbeg, kend);
  const int ntiles = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  constexpr bool DW = EPI == EPI_DW_SGD || EPI == EPI_DW_PARTIAL;

  // the hh products and the five small ones in accumulators of their own, where
  // the registers hold both (not in the 256 x 256 tile): the sum of hh is
  // rounded once for 16 k, not six times
  constexpr bool APART = TM * TN <= 4;
  const Biases<TN, EPI> bias(p, n0, wn, lane);
  floatx16 acc[TM][TN], small[APART ? TM : 1][APART ? TN : 1];
  clear(acc);
  clear(small);
  float bsum[LA::Q] = {};
  LA la[2];
  LB lb[2];
  auto request = [&](int set, int t) {
    la[set].load(p.A, p.lda, p.M, kend, m0, kbeg + t * BK, tid);
    lb[set].load(p.B, p.ldb, p.N, kend, n0, kbeg + t * BK, tid);
  };
  auto deliver = [&](int set, char* buf) {
    la[set].store(buf, tid);
    lb[set].store(buf + 3 * LA::PART, tid);
    if constexpr (DW) la[set].add_up(bsum);
  };
  const int fa = (lane >> 5) * LA::HALF + (wm + (lane & 31)) * 16;
  const int fb = (lane >> 5) * LB::HALF + (wn + (lane & 31)) * 16 + 3 * LA::PART;
  constexpr int NF = FD ? 2 : 1;
  bf16x8 a[NF][TM][3], b[NF][TN][3];
  auto fetch_b = [&](int set, const char* buf) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 3; ++q) b[set][j][q] = fragment(buf + fb + j * 512 + q * LB::PART);
  };
  auto fetch_a = [&](int set, int i, const char* buf) {
#pragma unroll
    for (int q = 0; q < 3; ++q) a[set][i][q] = fragment(buf + fa + i * 512 + q * LA::PART);
  };
  // the order of a stage's instructions: matrix instructions with the LDS
  // accesses and a share of the vector instructions between them.  In the 128 x 128
  // tile (FD) the shares are the ones that measured best: forward 10000 x 784-1024^3
  // 409 us at 6, 397 at 5 and 4, 408 at 9; the tendencies of 4096 samples 203 at 6, 196 at
  // 8, 188 at 11, 193 at 16.
  constexpr int NM = 6 * TM * TN, NR = 3 * (TM + TN);
  constexpr int NV = 26 * (LA::Q + LB::Q) + (DW ? 4 * LA::Q : 0) + 16;
  constexpr int VPM = FD ? (DW ? 11 : 5) : (NV + NM - 1) / NM;
  // FD: stage t's operands are in fragment set t & 1, stage t + 1 in LDS
  // buffer (t + 1) & 1, stages t + 2 and t + 3 in the register sets (stage s
  // in set s & 1).  Otherwise stage t is in LDS buffer t & 1, stages t + 1
  // and t + 2 in the register sets.
  auto stage = [&](int cur, int t) {
    if constexpr (FD) {
      char* const next = lds + (cur ^ 1) * STAGE;
      fetch_b(cur ^ 1, next);
#pragma unroll
      for (int i = 0; i < TM; ++i) fetch_a(cur ^ 1, i, next);
#pragma unroll
      for (int x = 0; x < 6; ++x)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            floatx16& c = x == 5 || !APART ? acc[i][j] : small[APART ? i : 0][APART ? j : 0];
            c = NF_MMA(a[cur][i][PART_A[x]], b[cur][j][PART_B[x]], c);
          }
      deliver(cur, lds + cur * STAGE);
      request(cur, t + 4);
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
        if (i >= NR) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      }
    } else {
      char* const now = lds + cur * STAGE;
      fetch_b(0, now);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        fetch_a(0, i, now);
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            floatx16& c = x == 5 || !APART ? acc[i][j] : small[APART ? i : 0][APART ? j : 0];
            c = NF_MMA(a[0][i][PART_A[x]], b[0][j][PART_B[x]], c);
          }
      }
      deliver(cur ^ 1, lds + (cur ^ 1) * STAGE);
      request(cur ^ 1, t + 3);
      __builtin_amdgcn_sched_group_barrier(0x100, 3 * TN + 3, 0);
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i % (6 * TN) < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
        if (i % (6 * TN) >= 6) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      }
    }
    __syncthreads();
  };

  request(0, 0);
  request(1, 1);
  deliver(0, lds);
  request(0, 2);
  if constexpr (FD) {
    deliver(1, lds + STAGE);
    request(1, 3);
    __syncthreads();
    fetch_b(0, lds);
#pragma unroll
    for (int i = 0; i < TM; ++i) fetch_a(0, i, lds);
  }
  __syncthreads();
  // (an odd last stage is followed by one of zeros, but in the smallest tile)
  for (int t = 0; t < ntiles; t += 2) {
    stage(0, t);
    if (BM == 64 && t + 1 == ntiles) break;
    stage(1, t + 1);
  }

  if constexpr (APART) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += small[i][j];
  }
  if constexpr (DW) {
    if (by == 0)
      put_bias_sums<LA, BM, BK, EPI>(p, bsum, m0, bz, tid, reinterpret_cast<float*>(lds));
  }
  finish_sums<AKC, BKC>(p, acc, m0, n0, wm, wn, kbeg, kend, lane);
  wide_epilogue<BM, TM, TN, EPI>(p, acc, bias, m0, n0, wm, wn, lane, bz);
}

// The same by (BM / WM) x (BN / WN) waves that multiply and NP more that load,
// for the tiles too small to hide the one behind the other within a wave.  A
// stage is 32 k: a small grid runs at the pace of the chain load - split - LDS -
// barrier, which two loading waves for each multiplying one and half as many
// barriers make half as long (64 x 64 tile, a stage of 16 k and one loading
// wave each before: a k of 16 took 0.38 us alone, 0.19 now; 16 x 255 x 300 10.0
// us, 7.4; 1024 x 1024 x 1000 28.7, 22.6).  Two workgroups fit on a CU (78 KB of
// LDS and at most 80 registers each), which large grids need.
template <int BM, int BN, int WM, int WN, int NP, bool AKC, bool BKC, bool AV, bool BV, int EPI>
__device__ __forceinline__ void wide_tile_roles(const GemmParamsT<float>& p, int bx, int by, int bz,
                                                char* lds) {
  constexpr int NC = (BM / WM) * (BN / WN);    // waves that multiply
  constexpr int NT = NP * 64;                  // threads that load
  constexpr int TM = WM / 32, TN = WN / 32, BK = WIDE_ROLES_BK, NB = 3, NR = 3, KS = BK / WIDE_KI;
  static_assert(NR % NB == 0 && KS % 2 == 0, "the loops are unrolled by the sets of registers");
  typedef SplitLoader<BM, BK, NT, AKC, AV> LA;
  typedef SplitLoader<BN, BK, NT, BKC, BV> LB;
  constexpr int STAGE = 3 * (LA::PART + LB::PART);
  static_assert(NB * STAGE == wide_lds(BM, BN, BK, NB), "LDS size");

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int m0 = __builtin_amdgcn_readfirstlane(bx * BM), n0 = __builtin_amdgcn_readfirstlane(by * BN);
  int kbeg, kend;
  piece_range<EPI>(p, bz, kbeg, kend);
  const int ntiles = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  constexpr bool DW = EPI == EPI_DW_SGD || EPI == EPI_DW_PARTIAL;

  // Both roles meet at the same barriers: one before the first stage, one
  // after each stage, one for the bias sums.
  if (wave >= NC) {
    const int tid = threadIdx.x - NC * 64;
    LA la[NR];
    LB lb[NR];
    float bsum[LA::Q] = {};
    auto request = [&](int set, int t) {
      la[set].load(p.A, p.lda, p.M, kend, m0, kbeg + t * BK, tid);
      lb[set].load(p.B, p.ldb, p.N, kend, n0, kbeg + t * BK, tid);
    };
    auto deliver = [&](int set, int buf) {
      la[set].store(lds + buf * STAGE, tid);
      lb[set].store(lds + buf * STAGE + 3 * LA::PART, tid);
      if constexpr (DW) la[set].add_up(bsum);
    };
    // stage s passes through register set s % NR and LDS buffer s % NB; while
    // stage t is multiplied stage t + 2 is delivered
#pragma unroll
    for (int d = 0; d < NR; ++d) request(d, d);
    deliver(0, 0);
    request(0, NR);
    deliver(1, 1);
    request(1, NR + 1);
    __syncthreads();
    for (int t = 0; t < ntiles; t += NR) {
#pragma unroll
      for (int d = 0; d < NR; ++d) {
        if (t + d >= ntiles) break;
        const int set = (d + 2) % NR;
        deliver(set, (d + 2) % NB);
        request(set, t + d + 2 + NR);
        __syncthreads();
      }
    }
    if constexpr (DW) {
      if (by == 0)
        put_bias_sums<LA, BM, BK, EPI>(p, bsum, m0, bz, tid, reinterpret_cast<float*>(lds));
    }
    return;
  }

  const int wm = (wave % (BM / WM)) * WM;
  const int wn = (wave / (BM / WM)) * WN;
  // the hh products and the five small ones in accumulators of their own: the
  // chain of dependent matrix instructions is shorter, and the sum of hh is
  // rounded once for 16 k
  const Biases<TN, EPI> bias(p, n0, wn, lane);
  floatx16 acc[TM][TN], small[TM][TN];
  clear(acc);
  clear(small);
  const int fa = (lane >> 5) * LA::HALF + (wm + (lane & 31)) * 16;
  const int fb = (lane >> 5) * LB::HALF + (wn + (lane & 31)) * 16 + 3 * LA::PART;
  bf16x8 a[2][TM][3], b[2][TN][3];
  auto fetch = [&](int set, int buf, int s) {
    const char* const la0 = lds + buf * STAGE + fa + 2 * s * LA::HALF;
    const char* const lb0 = lds + buf * STAGE + fb + 2 * s * LB::HALF;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a[set][i][q] = fragment(la0 + i * 512 + q * LA::PART);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[set][j][q] = fragment(lb0 + j * 512 + q * LB::PART);
    }
  };
  __syncthreads();
  fetch(0, 0, 0);
  for (int t = 0; t < ntiles; t += NB) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      if (t + u >= ntiles) break;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        // the next 16 k's operands are read while these are multiplied
        fetch((s + 1) & 1, s + 1 < KS ? u : (u + 1) % NB, (s + 1) % KS);
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              floatx16& c = x == 5 ? acc[i][j] : small[i][j];
              c = NF_MMA(a[s & 1][i][PART_A[x]], b[s & 1][j][PART_B[x]], c);
            }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += small[i][j];
  finish_sums<AKC, BKC>(p, acc, m0, n0, wm, wn, kbeg, kend, lane);
  if constexpr (DW) {
    if (by == 0) __syncthreads();
  }
  wide_epilogue<BM, TM, TN, EPI>(p, acc, bias, m0, n0, wm, wn, lane, bz);
}

// How a tile is worked on: waves that load and multiply, with or without the
// second set of fragments, or loading waves of their own.
enum WideForm { WIDE_PLAIN, WIDE_AHEAD, WIDE_ROLES };

// The problems of a launch: several in the tendencies, one elsewhere (a small
// launch waits for its arguments).
template <int EPI>
struct WideArgs {
  static constexpr bool DW = EPI == EPI_DW_PARTIAL || EPI == EPI_DW_SGD;
  static constexpr int MAX = DW ? GEMM_GROUP_MAX : 1;
  int total, per, n;
  int start[MAX + 1];                      // first workgroup of each problem
  GemmParamsT<float> p[MAX];
};

// Workgroup b runs on XCD b mod 8.  An XCD takes consecutive tiles (the grid
// is padded to 8 runs of `per`), in bands of 8 tile rows, so that the tiles
// it works on at one time share their operands in its L2.  (No division where
// there is one tile row and one piece: the chain of five cost a small launch
// about as much as its products.)
template <int BM, int BN, int WM, int WN, int FORM, bool AKC, bool BKC, bool AV, bool BV, int EPI>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * (FORM == WIDE_ROLES ? 192 : 64), FORM == WIDE_ROLES ? 6 : 1)
wide_kernel(const WideArgs<EPI> g) {
  __shared__ __attribute__((aligned(16))) char lds[FORM == WIDE_ROLES ? wide_lds(BM, BN, WIDE_ROLES_BK, 3)
                                                                : wide_lds(BM, BN, WIDE_KI, 2)];
  const int b = (blockIdx.x & 7) * g.per + (blockIdx.x >> 3);
  if (b >= g.total) return;
  int q = 0;
  if constexpr (WideArgs<EPI>::DW) {
#pragma unroll
    for (int i = 1; i < GEMM_GROUP_MAX; ++i) q += (i < g.n && b >= g.start[i]);
  }
  const GemmParamsT<float>& p = g.p[q];
  int r = b - (WideArgs<EPI>::DW ? g.start[q] : 0), bz = 0;
  const int mt = (p.M + BM - 1) / BM, nt = (p.N + BN - 1) / BN;
  if constexpr (EPI == EPI_DW_PARTIAL || EPI == EPI_FWD_PIECE || EPI == EPI_BWD_PIECE) {
    bz = r / (mt * nt);
    r -= bz * (mt * nt);
    bz = __builtin_amdgcn_readfirstlane(bz);
  }
  int bx = 0, by = r;
  if (mt > 1) {
    const int band = mt > 8 ? r / (8 * nt) : 0;
    const int inb = r - band * (8 * nt), bh = min(8, mt - band * 8);
    by = inb / bh;
    bx = band * 8 + inb - by * bh;
  }
  if constexpr (FORM == WIDE_ROLES)
    wide_tile_roles<BM, BN, WM, WN, 2 * (BM / WM) * (BN / WN), AKC, BKC, AV, BV, EPI>(p, bx, by, bz, lds);
  else
    wide_tile<BM, BN, WM, WN, FORM == WIDE_AHEAD, AKC, BKC, AV, BV, EPI>(p, bx, by, bz, lds);
}

template <int BM, int BN, int WM, int WN, int FORM, bool AKC, bool BKC, bool AV, bool BV, int EPI>
static hipError_t launch_one(const GemmGroupT<float>& g, const int* nsplit, hipStream_t s) {
  WideArgs<EPI> a;
  constexpr int MAX = WideArgs<EPI>::MAX;
  a.n = g.n;
  a.start[0] = 0;
  for (int q = 0; q < MAX; ++q) {
    a.p[q] = g.p[q];
    a.start[q + 1] = a.start[q];
    if (q < g.n)
      a.start[q + 1] += ((g.p[q].M + BM - 1) / BM) * ((g.p[q].N + BN - 1) / BN) * nsplit[q];
  }
  a.total = a.start[MAX];
  a.per = (a.total + 7) / 8;
  return launch_k(wide_kernel<BM, BN, WM, WN, FORM, AKC, BKC, AV, BV, EPI>, dim3(8 * a.per),
                  (BM / WM) * (BN / WN) * (FORM == WIDE_ROLES ? 192 : 64), 0, s, a);
}

template <int BM, int BN, int WM, int WN, int FORM>
static hipError_t wide_dispatch(int epi, bool av, const GemmGroupT<float>& g, const int* nsplit,
                                hipStream_t s) {
#define NF_CASE(E, AKC, BKC, AV) \
  if (epi == E && av == AV)      \
    return launch_one<BM, BN, WM, WN, FORM, AKC, BKC, AV, true, E>(g, nsplit, s);
  // forward: A = activations [m][k], B(k, n) = W[n][k]
  NF_CASE(EPI_FWD_STASH, true, true, true)
  NF_CASE(EPI_FWD_OUT, true, true, true)
  if constexpr (BM < 256) {
    NF_CASE(EPI_FWD_STASH, true, true, false)
    NF_CASE(EPI_FWD_DELTA, true, true, true)
    NF_CASE(EPI_FWD_DELTA, true, true, false)
    NF_CASE(EPI_FWD_OUT, true, true, false)
    NF_CASE(EPI_FWD_PIECE, true, true, true)
    NF_CASE(EPI_FWD_PIECE, true, true, false)
  }
  // backward: A = delta [m][k], B(k, n) = W[k][n]
  NF_CASE(EPI_BWD, true, false, true)
  if constexpr (BM < 256) {
    NF_CASE(EPI_BWD_PIECE, true, false, true)
  }
  // tendencies: A(m, k) = delta[k][m], B(k, n) = activations[k][n], read one
  // value at a time, so any row pitch will do
  NF_CASE(EPI_DW_SGD, false, false, true)
  NF_CASE(EPI_DW_PARTIAL, false, false, true)
#undef NF_CASE
  return hipErrorInvalidValue;
}

}  // namespace nf
