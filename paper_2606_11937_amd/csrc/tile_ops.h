// tile_ops.h -- gfx950 device bodies of the four tile operations (Methods,
// "Tiled Cholesky Decomposition": POTRF, TRSM, SYRK, GEMM).  Both schedules
// call exactly these bodies, so they produce bit-identical factors.
//
// Every body runs on one workgroup of TC_THREADS = 256 threads (4 wave64s).
// Matrices are row-major with leading dimension lda; only lower-triangle
// entries are written.  Blocks on the diagonal are read in whole pairs and
// rows, and what lies above the diagonal is dropped or feeds nothing on or
// below it.
//
// The contraction core is v_mfma_f64_16x16x4_f64 (FP64 matrix cores).  Its
// operand/result lane layout, measured on gfx950 with one-hot inputs:
//   A (16 x 4):  lane l holds A[l % 16][l / 16]
//   B (4 x 16):  lane l holds B[l / 16][l % 16]
//   D (16 x 16): lane l, item q holds D[4 q + l / 16][l % 16]
// All three tile products here are of the "NT" form X Y^T with X and Y both
// row-major with the contraction index contiguous, so A and B fragments are
// loaded the same way: lane (r = l % 16, s = l / 16) reads four consecutive
// doubles k0 + 4s .. k0 + 4s + 3 of row r, and MFMA number m of a 16-wide k
// chunk consumes element m.  The contraction order inside one output entry is
// therefore fixed (chunk by chunk; within a chunk, MFMA m sums k0+m, k0+4+m,
// k0+8+m, k0+12+m) and identical for every entry and both schedules.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define TC_THREADS 256

typedef double tc_v4d __attribute__((ext_vector_type(4)));
typedef double tc_d2 __attribute__((ext_vector_type(2), aligned(8)));

// Broadcast lane 0's value to the whole wave as a uniform (scalar) value.
// Values read from LDS that steer loops or branches containing barriers go
// through these, so the compiler sees the control flow as uniform and keeps
// every wave's barrier sequence identical to the source.
// Thread index behind a compiler-only barrier.  Tile bodies derive their
// lane offsets from it, so the persistent kernel recomputes them at the start
// of each body instead of hoisting them out of its unit loop, where they would
// stay live (and spill) across the other bodies.
__device__ __forceinline__ int tc_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ int32_t tc_uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t tc_uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(uint64_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double tc_uniform(double v) {
  const int64_t b = tc_uniform((int64_t)__builtin_bit_cast(int64_t, v));
  return __builtin_bit_cast(double, b);
}

__device__ __forceinline__ tc_v4d tc_mfma(double a, double b, tc_v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// c - a b: FP64 MFMAs take the sign of A as an instruction modifier
__device__ __forceinline__ tc_v4d tc_mfma_neg(double a, double b, tc_v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
}

// Stores of a unit's results.  SHARED: by the persistent schedules, whose
// units are read by workgroups of the same launch on other XCDs: a
// device-scope store goes through the XCD's L2 to memory, so a finished unit
// needs no write-back of that L2 before it is published (see tc_unit_stored).
// Every body takes the choice from its caller, without a default: an ordinary
// store in a persistent unit would be read stale only now and then.
template <bool SHARED, class V>
__device__ __forceinline__ void tc_st(V* p, V v) {
  if constexpr (SHARED)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}
template <bool SHARED>
__device__ __forceinline__ void tc_st2(double* p, double x, double y) {
  // one 16-byte store: in halves, each half went to memory by itself
  if constexpr (SHARED) {
    const tc_d2 v = {x, y};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
  } else {
    *(tc_d2*)p = tc_d2{x, y};
  }
}

// Four consecutive doubles of one row.
struct tc_q4 {
  tc_d2 lo, hi;
};
__device__ __forceinline__ double tc_el(const tc_q4& q, int m) {
  return m == 0 ? q.lo.x : m == 1 ? q.lo.y : m == 2 ? q.hi.x : q.hi.y;
}

// ---------------------------------------------------------------------------
// SYRK / GEMM update of one output block (the trailing-update tile ops):
//   C[r][c] -= sum_{t < kd} PA[r][t] * PB[c][t]     0 <= r < mr, 0 <= c < mc
// restricted to r >= c when `diag` (a block on the matrix diagonal, SYRK).
// mr, mc <= 128.  Wave w computes the 64 x 64 quadrant (w & 1, w >> 1) with
// 4 x 4 MFMA accumulators.
//
// Operands are staged through LDS in 16-wide k chunks, two stages deep, with
// direct-to-LDS buffer loads (16 bytes per lane, no registers involved).
// LDS layout of one operand tile: 128 rows x 8 slots of 16 bytes (two k
// values); slot j of row r sits at position j ^ (r & 7) of its row, which
// keeps the 128-bit fragment reads of the MFMAs free of bank conflicts.  A
// direct-to-LDS load writes lane i's 16 bytes to slot i of a 64-slot window,
// so each lane fetches the global element that belongs in its slot.  The
// buffer resource spans exactly the block's mr (mc) rows: rows beyond them
// read as zero and are never stored.
//
// Rows of B are staged in the order of tc_pair_row, so that a lane's results
// of column blocks j and j + 1 (j even) are neighbours in C, which is then
// read and written 16 bytes a lane, 256 consecutive bytes of a row at a time.
// Against 8 bytes a lane: a unit with K = 128 .. 384 in the batched launch
// 46.5 -> 44.0 us, alone 24 -> 22.5 us; fork-join at order 32768 unchanged.
//
// Fragment registers roll half a chunk ahead: the high halves (k steps 2, 3)
// of chunk c are read while the MFMAs of its low halves run; the barrier that
// publishes chunk c+1 sits in the middle of chunk c; the low halves of chunk
// c+1 are read while the MFMAs of chunk c's high halves run.  One 64-register
// fragment set and a 64 KB stage pair let two workgroups share a CU.
// ---------------------------------------------------------------------------
#define TC_UPD_STAGES 2
// The swizzle below is conflict-free only relative to a bank-period-aligned
// base, and the 128-bit reads need 16-byte alignment: the stages are placed
// on a 512-byte boundary wherever the struct is declared (alone, or inside the
// persistent kernel's union next to other shared variables).
struct alignas(512) TcUpdSmem {
  double tile[TC_UPD_STAGES][2][128 * 16];  // [stage][A|B][row * 16 + slot * 2 + e]
};

typedef __attribute__((address_space(3))) void tc_lds_void;
typedef double tc_d2a16 __attribute__((ext_vector_type(2), aligned(16)));

__device__ __forceinline__ int tc_swz(int r) { return r & 7; }

// Rows [0, mr) of a block at p as a buffer: one 32-bit offset a lane, and
// accesses past the last row read zero or are dropped.  SHARED as in tc_st.
struct TcRows {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ TcRows(double* p, int64_t lda, int mr)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)tc_uniform((int64_t)p), (short)0,
                                            (int)(tc_uniform((int32_t)mr) * tc_uniform(lda) * 8), 0x00020000)) {}
  // at byte o + s of the block; s < 1024 and the same in all lanes
  __device__ __forceinline__ tc_d2 ld2(unsigned o, unsigned s) const {
    return __builtin_bit_cast(tc_d2, __builtin_amdgcn_raw_buffer_load_b128(r, o, s, 0));
  }
  // Stores without a branch: a lane whose `keep` is false stores nothing.  A
  // 16-byte store takes its whole offset from the lane: with a scalar part
  // the compiler leaves no wait state before the data registers are written
  // again, and here the last lanes of a row then stored the new contents.
  template <bool SHARED>
  __device__ __forceinline__ void st2(bool keep, unsigned o, unsigned s, tc_d2 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, keep ? o + s : 0xFFFFF000u, 0,
                                           SHARED ? 16 : 0);
  }
  template <bool SHARED>
  __device__ __forceinline__ void st1(bool keep, unsigned o, unsigned s, double v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, keep ? o : 0xFFFFF000u, s, SHARED ? 16 : 0);
  }
};

// The row of B (and column of C) that LDS row 16 i + r of its 64 holds.
__device__ __forceinline__ int tc_pair_row(int i, int r) { return 32 * (i >> 1) + 2 * r + (i & 1); }

template <bool SHARED>
__device__ __forceinline__ void tc_update_block(double* __restrict__ C, const double* __restrict__ PA,
                                                const double* __restrict__ PB, int64_t lda, int mr, int mc,
                                                int kd, bool diag, TcUpdSmem& sm) {
  const int tid = tc_tid();
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int wm = w & 1, wn = w >> 1;
  // waves with nothing to store still stage operands and take part in barriers
  const bool active = !(diag && wn > wm) && wm * 64 < mr && wn * 64 < mc;
  const int r16 = lane & 15, s2 = (lane >> 4) * 2;

  // --- staging: waves 0,1 fetch A rows, waves 2,3 B rows; load q of wave w
  //     fills LDS slots [(w*8+q)*64, +64) = rows (w&1)*64 + q*8 .. +8.
  //     The operand, its row count and the LDS window depend on the wave
  //     only: taken as scalars, the buffer resource and the LDS base sit in
  //     scalar registers (a resource in vector registers would turn every
  //     load into a loop over the distinct values the lanes hold).
  const int ws = tc_uniform((int32_t)w);
  const int nrow = ws < 2 ? tc_uniform((int32_t)mr) : tc_uniform((int32_t)mc);
  const double* src = (const double*)tc_uniform((int64_t)(ws < 2 ? PA : PB));
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)src, (short)0, (int)((int64_t)nrow * tc_uniform(lda) * 8), 0x00020000);
  const bool isb = ws >= 2;
  const int rl0 = (w & 1) * 64 + (isb ? 2 : 1) * (lane >> 3);
  const int kl0 = (lane & 7) ^ (lane >> 3);
  const unsigned vof0 = (unsigned)(rl0 * lda * 8 + 16 * kl0);
  auto rowof = [&](int q) { return isb ? tc_pair_row(q >> 1, 8 * (q & 1)) : 8 * q; };  // from rl0
  auto stage_load = [&](int st, int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc,
          (tc_lds_void*)((char __attribute__((address_space(3)))*)(tc_lds_void*)&sm.tile[st][0][0] +
                         (ws * 8 + q) * 1024),
          16, vof0 + (unsigned)rowof(q) * (unsigned)(tc_uniform(lda) * 8), (unsigned)(k0 * 8), 0, 0);
  };
  // the ragged last chunk (kd % 16 != 0): ordinary guarded loads, zero past
  // kd or past the block's rows, stored where the direct loads would put them
  auto stage_tail = [&](int st, int k0) {
    const double* gb = w < 2 ? PA : PB;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = rl0 + rowof(q);
      const int k = k0 + 2 * kl0;
      const double* src = gb + (int64_t)(r < nrow ? r : 0) * lda + k;
      tc_d2 v;
      v.x = (r < nrow && k < kd) ? src[0] : 0.0;
      v.y = (r < nrow && k + 1 < kd) ? src[1] : 0.0;
      *(tc_d2*)(&sm.tile[st][0][0] + ((w * 8 + q) * 64 + lane) * 2) = v;
    }
  };
  auto stage = [&](int st, int c, int nfull) {
    if (c < nfull) stage_load(st, c * 16); else stage_tail(st, c * 16);
  };
  // fragment half h (k = 4s + 2h, 4s + 2h + 1) of row-block i of operand t
  // (0 = A rows wm*64.., 1 = B rows wn*64..)
  auto rd = [&](int st, int t, int i, int h) -> tc_d2 {
    const int r = (t == 0 ? wm : wn) * 64 + i * 16 + r16;
    const tc_d2a16 v = *(const tc_d2a16*)(&sm.tile[st][t][r * 16] + 2 * ((s2 + h) ^ tc_swz(r)));
    tc_d2 o;
    o.x = v.x;
    o.y = v.y;
    return o;
  };

  tc_v4d acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = tc_v4d{0.0, 0.0, 0.0, 0.0};

  // (s_waitcnt encodings: 0x0F70 = vmcnt(0); 0x0070 = vmcnt(0) lgkmcnt(0);
  //  expcnt and unnamed counters at their maxima)
  const int nfull = kd >> 4;
  const int nch = (kd + 15) >> 4;
  tc_d2 La[4], Lb[4], Ha[4], Hb[4];
  if (nch > 0) stage(0, 0, nfull);
  if (nch > 1) stage(1, 1, nfull);
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();
  if (active && nch > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      La[i] = rd(0, 0, i, 0);
      Lb[i] = rd(0, 1, i, 0);
    }
  }
  auto high = [&](int st) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      Ha[i] = rd(st, 0, i, 1);
      Hb[i] = rd(st, 1, i, 1);
    }
  };
  auto products = [&](const tc_d2(&fa)[4], const tc_d2(&fb)[4]) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = tc_mfma(m ? fa[i].y : fa[i].x, m ? fb[j].y : fb[j].x, acc[i][j]);
  };
  for (int c = 0; c + 1 < nch; ++c) {
    const int st = c & 1;
    if (active) {
      high(st);
      products(La, Lb);
    }
    // chunk c+1 has landed and this wave's reads of chunk c are complete;
    // a plain barrier (a fenced one would also wait for unrelated traffic)
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    if (c + 2 < nch) stage(st, c + 2, nfull);  // chunk c's stage is free now
    if (active) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        La[i] = rd(st ^ 1, 0, i, 0);
        Lb[i] = rd(st ^ 1, 1, i, 0);
      }
      products(Ha, Hb);
    }
  }
  if (!active) return;

  // the last chunk, and C -= acc on the stored part, in 16-row groups (32
  // registers of C each).  A block of 128 columns reads its C values
  // unconditionally (rows past mr read as zero and are not stored; for a
  // diagonal block the entries above the diagonal are read and left alone):
  // half of group 0 before the last half chunk's products, the rest and group
  // 1 behind them, groups 2 and 3 as groups 0 and 1 are subtracted, and no
  // store before the last load, as loads and stores of a wave complete in
  // order: two memory round trips instead of five.  Measured: the batched
  // launch of 4096 matrices 30.3 -> 29.7 ms, order 32768 187.8 -> 185.7 ms.
  // (All of group 0 ahead takes registers that the persistent kernels spill.)
  // Other blocks read from clamped positions, one group ahead of the stores.
  const int orow = lane >> 4, ocol = 2 * (lane & 15);
  const bool pairs = mc == 128;
  const TcRows cr(C, lda, mr);
  const unsigned c4 = (unsigned)(4 * tc_uniform(lda) * 8);
  const unsigned c0 = (unsigned)((wm * 64 + orow) * lda * 8 + (wn * 64 + ocol) * 8);
  // offset of the lane's first row of group i, made anew for each use: kept,
  // the 16 of them take the registers that the groups need
  auto first = [&](int i) {
    unsigned o = c0 + 4 * i * c4;
    asm volatile("" : "+v"(o));
    return o;
  };
  auto cload = [&](tc_d2(&v)[8], int i, int q0 = 0, int q1 = 4) {
    unsigned o = first(i) + q0 * c4;
#pragma unroll
    for (int q = q0; q < q1; ++q, o += c4) {
      v[2 * q] = cr.ld2(o, 0);
      v[2 * q + 1] = cr.ld2(o, 256);
    }
  };
  tc_d2 v0[8], v1[8];
  if (nch > 0) {
    high((nch - 1) & 1);
    products(La, Lb);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (pairs) cload(v0, 0, 0, 2);
  __builtin_amdgcn_sched_barrier(0);
  if (nch > 0) products(Ha, Hb);
  __builtin_amdgcn_sched_barrier(0);
  if (pairs) {
    auto sub = [&](tc_d2(&v)[8], int i) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          tc_d2& x = v[2 * q + j / 2];
          x.x = x.x - acc[i][j][q];
          x.y = x.y - acc[i][j + 1][q];
        }
    };
    // a diagonal block stores the pairs below the diagonal; those on it lose
    // their second element, and are stored last, as a branch between the
    // groups would let the compiler move the subtractions behind it
    const int below = (wm - wn) * 64 + orow - ocol;  // r - c of the lane's first pair
    auto cstore = [&](const tc_d2(&v)[8], int i) {
      unsigned o = first(i);
#pragma unroll
      for (int q = 0; q < 4; ++q, o += c4)
#pragma unroll
        for (int j = 0; j < 4; j += 2)
          cr.st2<SHARED>(!diag || below + 16 * i + 4 * q - 16 * j > 0, o, 128 * j, v[2 * q + j / 2]);
    };
    auto cstore1 = [&](const tc_d2(&v)[8], int i) {
      unsigned o = first(i);
#pragma unroll
      for (int q = 0; q < 4; ++q, o += c4)
#pragma unroll
        for (int j = 0; j < 4; j += 2)
          cr.st1<SHARED>(below + 16 * i + 4 * q - 16 * j == 0, o, 128 * j, v[2 * q + j / 2].x);
    };
    tc_d2 v2[8], v3[8];
    cload(v0, 0, 2, 4);
    cload(v1, 1);
    __builtin_amdgcn_sched_barrier(0);
    sub(v0, 0);
    __builtin_amdgcn_sched_barrier(0);
    cload(v2, 2);
    __builtin_amdgcn_sched_barrier(0);
    sub(v1, 1);
    __builtin_amdgcn_sched_barrier(0);
    cload(v3, 3);
    __builtin_amdgcn_sched_barrier(0);
    cstore(v0, 0);
    cstore(v1, 1);
    __builtin_amdgcn_sched_barrier(0);
    sub(v2, 2);
    cstore(v2, 2);
    sub(v3, 3);
    cstore(v3, 3);
    if (diag) {
      cstore1(v0, 0);
      cstore1(v1, 1);
      cstore1(v2, 2);
      cstore1(v3, 3);
    }
  } else {
    // ragged: the same pipeline, loads from clamped (in-block) positions,
    // stores guarded
    double cv[2][16];
    auto cload = [&](double(&v)[16], int i) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = wm * 64 + i * 16 + 4 * q + orow;
        const double* rp = C + (int64_t)(r < mr ? r : mr - 1) * lda;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = wn * 64 + 32 * (j >> 1) + ocol + (j & 1);
          v[4 * q + j] = rp[c < mc ? c : mc - 1];
        }
      }
    };
    auto cstore = [&](const double(&v)[16], int i) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = wm * 64 + i * 16 + 4 * q + orow;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = wn * 64 + 32 * (j >> 1) + ocol + (j & 1);
          if (r < mr && c < mc && (!diag || r >= c))
            tc_st<SHARED>(C + (int64_t)r * lda + c, v[4 * q + j] - acc[i][j][q]);
        }
      }
    };
    cload(cv[0], 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i + 1 < 4) cload(cv[(i + 1) & 1], i + 1);
      __builtin_amdgcn_sched_barrier(0);
      cstore(cv[i & 1], i);
    }
  }
}

// ---------------------------------------------------------------------------
// Division and lane reads used by the substitutions.
// ---------------------------------------------------------------------------

// x / d from the correctly rounded reciprocal r = 1 / d and one residual
// correction (Markstein's method): q0 = x r, e = x - q0 d (exact with an
// FMA), q = q0 + e r.  The result is exact whenever x / d is representable
// and otherwise within one unit in the last place of the rounded quotient.
// It takes three dependent operations instead of a full division.
__device__ __forceinline__ double tc_div_rcp(double x, double d, double r) {
  const double q0 = x * r;
  const double e = __builtin_fma(-q0, d, x);
  return __builtin_fma(e, r, q0);
}

__device__ __forceinline__ double tc_readlane(double v, int l) {
  const int64_t b = __builtin_bit_cast(int64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)(uint64_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)((uint64_t)b >> 32), l);
  return __builtin_bit_cast(double, (int64_t)(((uint64_t)hi << 32) | lo));
}

// Orders this wave's LDS writes before its later reads of them from other
// lanes (LDS operations of one wave complete in order; the fences keep the
// compiler from moving them).
__device__ __forceinline__ void tc_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Row broadcasts.  A 16-lane row of the wave holds one 16 x 16 block, lane r
// its row r; column k of the block's factor is then lane k's register.  The
// FP64 multiply-add takes that register straight from lane k through its
// data-parallel operand (row_newbcast:k), one instruction where two lane
// reads and an FMA take three: a lone wave issues one vector instruction per
// 6 cycles here (measured: 6.0 cycles for a dependent FP64 FMA, 6.0 for this
// broadcasting one, 26 for two lane reads and an FMA), so the instruction
// count is what these chains cost.  Written as assembly because the compiler
// emits a move for the broadcast; each block starts with the two wait states
// a broadcast operand needs after a vector write (the compiler's hazard pass
// does not look into assembly).  No operand is ever an MFMA result (those go
// through LDS first), and the whole wave must be active.
// ---------------------------------------------------------------------------
#define TC_BC_ " row_newbcast:%[k"
#define TC_BCM_ "] row_mask:0xf bank_mask:0xf\n\t"
#define TC_FMB_(i) "v_fmac_f64_dpp %" #i ", -%[s], %[x]" TC_BC_ #i TC_BCM_

// v[K0 + t] -= (src of lane K0 + t) * x for t < N, N <= 8
template <int K0, int N>
__device__ __forceinline__ void tc_fmac_bcast8(double (&v)[16], double src, double x) {
  static_assert(N >= 0 && N <= 8 && K0 + N <= 16, "group of columns");
  if constexpr (N == 8) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2) TC_FMB_(3) TC_FMB_(4) TC_FMB_(5) TC_FMB_(6) TC_FMB_(7)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2]), "+&v"(v[K0 + 3]), "+&v"(v[K0 + 4]), "+&v"(v[K0 + 5]),
          "+&v"(v[K0 + 6]), "+&v"(v[K0 + 7])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2), [k3] "i"(K0 + 3), [k4] "i"(K0 +
          4), [k5] "i"(K0 + 5), [k6] "i"(K0 + 6), [k7] "i"(K0 + 7));
  } else if constexpr (N == 7) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2) TC_FMB_(3) TC_FMB_(4) TC_FMB_(5) TC_FMB_(6)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2]), "+&v"(v[K0 + 3]), "+&v"(v[K0 + 4]), "+&v"(v[K0 + 5]),
          "+&v"(v[K0 + 6])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2), [k3] "i"(K0 + 3), [k4] "i"(K0 +
          4), [k5] "i"(K0 + 5), [k6] "i"(K0 + 6));
  } else if constexpr (N == 6) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2) TC_FMB_(3) TC_FMB_(4) TC_FMB_(5)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2]), "+&v"(v[K0 + 3]), "+&v"(v[K0 + 4]), "+&v"(v[K0 + 5])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2), [k3] "i"(K0 + 3), [k4] "i"(K0 +
          4), [k5] "i"(K0 + 5));
  } else if constexpr (N == 5) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2) TC_FMB_(3) TC_FMB_(4)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2]), "+&v"(v[K0 + 3]), "+&v"(v[K0 + 4])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2), [k3] "i"(K0 + 3), [k4] "i"(K0 +
          4));
  } else if constexpr (N == 4) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2) TC_FMB_(3)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2]), "+&v"(v[K0 + 3])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2), [k3] "i"(K0 + 3));
  } else if constexpr (N == 3) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1) TC_FMB_(2)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1]), "+&v"(v[K0 + 2])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1), [k2] "i"(K0 + 2));
  } else if constexpr (N == 2) {
    asm("s_nop 1\n\t" TC_FMB_(0) TC_FMB_(1)
        : "+&v"(v[K0]), "+&v"(v[K0 + 1])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0), [k1] "i"(K0 + 1));
  } else if constexpr (N == 1) {
    asm("s_nop 1\n\t" TC_FMB_(0)
        : "+&v"(v[K0])
        : [s] "v"(src), [x] "v"(x), [k0] "i"(K0));
  }
}
// v[k] -= (src of lane k) * x for k = K0 .. 15
template <int K0>
__device__ __forceinline__ void tc_fmac_bcast(double (&v)[16], double src, double x) {
  if constexpr (K0 < 8) {
    tc_fmac_bcast8<K0, 8>(v, src, x);
    tc_fmac_bcast8<K0 + 8, 8 - K0>(v, src, x);
  } else if constexpr (K0 < 16) {
    tc_fmac_bcast8<K0, 16 - K0>(v, src, x);
  }
}
// lane K's value of v in every lane of its row
template <int K>
__device__ __forceinline__ double tc_bcast(double v) {
  double o;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1" TC_BC_ "0" TC_BCM_ : "=&v"(o) : "v"(v), [k0] "i"(K));
  return o;
}

// ---------------------------------------------------------------------------
// LDS images of 16 x 16 blocks.  A block row is 128 bytes: eight 16-byte
// slots of two doubles.  Slot s of row r sits at position s ^ (r & 7) of the
// row (the swizzle of the update kernel), so that one slot read by 16 rows,
// or whole rows read by 8 lanes, spread over the banks.  `rs` is the row
// stride in doubles of the array the block sits in.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int tc_bo(int r, int c, int rs) { return r * rs + ((((c >> 1) ^ r) & 7) << 1) + (c & 1); }

// Row r of a block (16 doubles), as eight 16-byte accesses.
__device__ __forceinline__ void tc_row_get(const double* blk, int r, int rs, double v[16]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const tc_d2a16 p = *(const tc_d2a16*)(blk + r * rs + ((s ^ (r & 7)) << 1));
    v[2 * s] = p.x;
    v[2 * s + 1] = p.y;
  }
}
__device__ __forceinline__ void tc_row_put(double* blk, int r, int rs, const double v[16]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    tc_d2a16 p;
    p.x = v[2 * s];
    p.y = v[2 * s + 1];
    *(tc_d2a16*)(blk + r * rs + ((s ^ (r & 7)) << 1)) = p;
  }
}
// MFMA operand fragment of lane (r, s): row r, columns 4 s .. 4 s + 3.
__device__ __forceinline__ tc_q4 tc_frag_get(const double* blk, int r, int s, int rs) {
  const tc_d2a16 a = *(const tc_d2a16*)(blk + r * rs + (((2 * s) ^ (r & 7)) << 1));
  const tc_d2a16 b = *(const tc_d2a16*)(blk + r * rs + (((2 * s + 1) ^ (r & 7)) << 1));
  tc_q4 q;
  q.lo = tc_d2{a.x, a.y};
  q.hi = tc_d2{b.x, b.y};
  return q;
}
// A block in the MFMA result layout: lane l, item q is element (4 q + l / 16, l % 16).
__device__ __forceinline__ tc_v4d tc_acc_get(const double* blk, int lane, int rs) {
  tc_v4d a;
#pragma unroll
  for (int q = 0; q < 4; ++q) a[q] = blk[tc_bo(4 * q + (lane >> 4), lane & 15, rs)];
  return a;
}
__device__ __forceinline__ void tc_acc_put(double* blk, int lane, int rs, tc_v4d a) {
#pragma unroll
  for (int q = 0; q < 4; ++q) blk[tc_bo(4 * q + (lane >> 4), lane & 15, rs)] = a[q];
}
// c - X Y^T for 16 x 16 blocks and K = 16: x, y are the fragments of lane
// (l % 16, l / 16) of X and Y, c is in the result layout.  MFMA m sums the
// k = 4 s + m of the four lane groups s, so the contraction order is fixed.
__device__ __forceinline__ tc_v4d tc_nt16(const tc_q4& x, const tc_q4& y, tc_v4d c) {
#pragma unroll
  for (int m = 0; m < 4; ++m) c = tc_mfma_neg(tc_el(x, m), tc_el(y, m), c);
  return c;
}

// 1 / x from the hardware estimate and two Newton-Raphson steps
// (r <- r + r (1 - x r)); within one unit in the last place.
__device__ __forceinline__ double tc_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// ---------------------------------------------------------------------------
// Forward substitution X <- X L^{-T} of 16 rows of X against a factored
// 16 x 16 block L, on the matrix cores, with X in the layout of a transposed
// MFMA result: lane l, item q holds X[l % 16][4 q + l / 16].  Item q, taken as
// the B operand (4 x 16) of an FP64 MFMA, is X[:, 4 q .. 4 q + 3]^T, and so is
// the first item of the MFMA's result, so the rows never change lanes.
// Four columns (a quarter q) at a time: with N the strictly lower part of the
// quarter's 4 x 4 diagonal block and R the reciprocals of its pivots,
//   y <- R a,  then three times  y <- R (a - N y),
// after which component t is r_t (a_t - sum_{k<t} l_tk x_k) for every t < 4:
// component t takes its final value in round t, from final components only
// (N is strictly lower), so this is the substitution itself, not an iteration
// that converges.  Each round is one v_mfma_f64_4x4x4 (four 4 x 4 products,
// one per four rows of X) and one multiply.  The later quarters of the block
// then receive the product of the finished one, one such MFMA each.
// Per 16 columns a wave issues 18 of these MFMAs (17.5 cycles each; 29 when
// one waits for the other) and 16 multiplies.  The form it replaces, one row
// per lane, took 120 multiply-adds of 6 cycles with three lanes in four idle
// or repeating, and matrix and vector FP64 instructions of one wave do not
// overlap (4 MFMAs and 32 FMAs take 473 cycles, alone 257 and 181).
// ---------------------------------------------------------------------------
// Lane l's operands: n[e], e = q' (q' + 1) / 2 + q, is L[4 q' + l % 4][4 q + l / 16]
// (zero on and above the diagonal when q' == q); r[q] = 1 / L[j][j], j = 4 q + l / 16.
struct TcMicro {
  double n[10];
  double r[4];
};

__device__ __forceinline__ double tc_mfma4_neg(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 1);
}

// NS independent 16-row blocks side by side.
template <int NS>
__device__ __forceinline__ void tc_subst16(tc_v4d (&x)[NS], const TcMicro& o) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * (q + 1) / 2 + q;
    double y[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) y[t] = x[t][q] * o.r[q];
#pragma unroll
    for (int it = 0; it < 3; ++it) {
#pragma unroll
      for (int t = 0; t < NS; ++t) y[t] = tc_mfma4_neg(o.n[e], y[t], x[t][q]);
#pragma unroll
      for (int t = 0; t < NS; ++t) y[t] = y[t] * o.r[q];
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) x[t][q] = y[t];
#pragma unroll
    for (int p = q + 1; p < 4; ++p)
#pragma unroll
      for (int t = 0; t < NS; ++t) x[t][p] = tc_mfma4_neg(o.n[p * (p + 1) / 2 + q], y[t], x[t][p]);
  }
}

// ---------------------------------------------------------------------------
// TRSM work unit: X <- X L^{-T} for mr <= 128 rows of a tile (I, J), I > J,
// with L = L_JJ (td x td, factored).  Left-looking over 16-column blocks b:
// X[:, b] -= X[:, c] L_bc^T for every block c < b (MFMA, K = 16), then
// substitution against L_bb.
// Rows are independent: a wave owns 16 of them (a strip) with its column
// blocks in registers, in the layout above; a finished block is the B operand
// of the products as it stands.  L passes through LDS in operand order, so
// that each operand read is a conflict-free 16 bytes per lane: 67 KB, two
// workgroups on a CU.
// Step b needs only block row b of L and block b of X.  All of them are
// loaded at the start, in that order, and block row b goes from registers to
// LDS in front of step b, so what the later steps need arrives behind the
// earlier ones (a CU alone takes in about 20 bytes a cycle here, 7000 cycles
// for L and 64 rows of X; loads issued three steps ahead instead waited
// behind the stores of the steps between, 12.7 against 11.9 us).
// Bound by the FP64 matrix pipe of one SIMD: 112 MFMAs of 64 cycles and 8
// substitutions (about 800 cycles each) per strip, 17000 cycles of the 28000
// that 64 rows take alone on a CU.  In-kernel time of one workgroup: 11.9 us
// for 64 rows (23.5 us with one row per lane in the substitution and the
// operands of L from global memory), 20.8 us for 128 (43.6; 40 with two of
// them on every CU and their rows in HBM).
// ---------------------------------------------------------------------------
struct alignas(16) TcTrsmSmem {
  double op[28][256];     // L_bc, c < b, at b (b - 1) / 2 + c: [q / 2][lane][q % 2] = L_bc[lane % 16][4 q + lane / 16]
  double dg[8][5][16][2];  // TcMicro::n of the diagonal blocks: [b][e / 2][4 (lane / 16) + lane % 4][e % 2]
  double rcp[128];        // reciprocals of the pivots
};

// Lane row g of the wave (16 lanes) and one of two registers change places:
// bit 1 (wide) or bit 0 of g against the register.
__device__ __forceinline__ void tc_swap_rows(double& a, double& b, bool wide) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (wide) {
      const auto r = __builtin_amdgcn_permlane32_swap(x[h], y[h], false, false);
      x[h] = r[0];
      y[h] = r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(x[h], y[h], false, false);
      x[h] = r[0];
      y[h] = r[1];
    }
  }
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
// Between the substitution's layout (lane row g, item m: column 4 m + g) and
// the strip's in memory.  It is read with four consecutive columns a lane
// (two adjacent 16-byte loads; pairs 8 columns apart, as below, were 7 %
// slower a unit) and written with columns 2 g, 2 g + 1, 2 g + 8 and 2 g + 9
// in lane row g, so that a 16-byte store of the wave covers 64 consecutive
// bytes of every row.  (With four consecutive columns a lane there too and
// device-scope stores of 8 bytes, each touched every fourth 8 bytes: 512 of
// these units at a time took 70 us each in the batched launch, 42 us this
// way; the launch of 4096 matrices with solves 34.5 -> 30.4 ms.)
__device__ __forceinline__ tc_v4d tc_strip_out(tc_v4d v) {
  double a = v[0], b = v[1], c = v[2], d = v[3];
  tc_swap_rows(a, b, true);
  tc_swap_rows(c, d, true);
  tc_swap_rows(a, b, false);
  tc_swap_rows(c, d, false);
  return tc_v4d{a, b, c, d};
}
__device__ __forceinline__ tc_v4d tc_strip_in(tc_v4d v) {
  double a = v[0], b = v[1], c = v[2], d = v[3];
  tc_swap_rows(a, c, true);
  tc_swap_rows(b, d, true);
  tc_swap_rows(a, b, false);
  tc_swap_rows(c, d, false);
  return tc_v4d{a, b, c, d};
}

// Column block j of a strip (rows [0, mr) of X, mr <= 16) in those two forms:
// lane (r, g) takes columns 16 j + 4 g .. + 3 of row r in, and gives 16 j +
// 2 g, + 1, + 8 and + 9 out.  Rows past mr and columns past td read clamped
// positions (selected to zero where they matter).
__device__ __forceinline__ tc_v4d tc_strip_get(const double* __restrict__ X, int64_t lda, int mr, int td, int j,
                                               int lane) {
  const int r16 = lane & 15, c = 16 * j + 4 * (lane >> 4);
  const int rc = r16 < mr ? r16 : (mr > 0 ? mr - 1 : 0);
  const double* p = X + (int64_t)rc * lda;
  if (td == 128) {
    const tc_d2 lo = *(const tc_d2*)(p + c), hi = *(const tc_d2*)(p + c + 2);
    return tc_v4d{lo.x, lo.y, hi.x, hi.y};
  }
  tc_v4d a;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int k = c + m;
    a[m] = p[k < td ? k : td - 1];
    a[m] = k < td ? a[m] : 0.0;
  }
  return a;
}
template <bool SHARED>
__device__ __forceinline__ void tc_strip_put(double* __restrict__ X, int64_t lda, int mr, int td, int j, int lane,
                                             tc_v4d a) {
  const int r16 = lane & 15, c = 16 * j + 2 * (lane >> 4);
  if (r16 >= mr) return;
  double* g = X + (int64_t)r16 * lda + c;
  if (td == 128) {
    tc_st2<SHARED>(g, a[0], a[1]);
    tc_st2<SHARED>(g + 8, a[2], a[3]);
  } else {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int k = (m & 1) + 4 * (m & 2);
      if (c + k < td) tc_st<SHARED>(g + k, a[m]);
    }
  }
}

// What a thread holds of L between its loads and their way into LDS: pass k
// covers blocks 2 k and 2 k + 1 (waves 0-1 and 2-3; row r, columns 2 s and
// 2 s + 1 of the block).  A full block reads whole 16-byte pairs (those of a
// diagonal block reach above the diagonal and are dropped at the store); a
// ragged one reads from clamped positions on or below the diagonal and
// selects afterwards, so no load sits in a branch of its own.  Rows past td
// are those of the identity.
struct TcTrsmStage {
  tc_d2 v[14], d[4];
  double piv;
};
__device__ __forceinline__ tc_d2 tc_stage_pair(const double* __restrict__ L, int64_t lda, int td, int R, int C) {
  if (td == 128) return *(const tc_d2*)(L + (int64_t)R * lda + C);
  const int Rc = R < td ? R : td - 1, C0 = C < Rc ? C : Rc, C1 = C + 1 < Rc ? C + 1 : Rc;
  tc_d2 v;
  v.x = L[(int64_t)Rc * lda + C0];
  v.y = L[(int64_t)Rc * lda + C1];
  v.x = R < td ? v.x : 0.0;
  v.y = R < td ? v.y : 0.0;
  return v;
}
__device__ __forceinline__ void tc_stage_load(const double* __restrict__ L, int64_t lda, int td, int k,
                                              TcTrsmStage& st) {
  const int tid = tc_tid(), hi = tc_uniform((int32_t)(tid >> 7)), r = (tid >> 3) & 15, s = tid & 7;
  const int p = 2 * k + hi;
  int bi = 1;
#pragma unroll
  for (int q = 2; q < 8; ++q) bi += p >= q * (q - 1) / 2;
  const int bj = p - bi * (bi - 1) / 2;
  st.v[k] = tc_stage_pair(L, lda, td, 16 * bi + r, 16 * bj + 2 * s);
}
__device__ __forceinline__ void tc_stage_put(TcTrsmSmem& sm, int k, const TcTrsmStage& st) {
  const int tid = tc_tid(), hi = tc_uniform((int32_t)(tid >> 7)), r = (tid >> 3) & 15, s = tid & 7;
  // columns c = 2 s and c + 1 lie in quarter s / 2 at c % 4 and c % 4 + 1
  double* g = sm.op[2 * k + hi] + (s >> 2) * 128 + (((2 * s) & 3) * 16 + r) * 2 + ((s >> 1) & 1);
  g[0] = st.v[k].x;
  g[32] = st.v[k].y;
}
__device__ __forceinline__ void tc_stage_diag(const double* __restrict__ L, int64_t lda, int td, TcTrsmStage& st) {
  const int tid = tc_tid(), hi = tc_uniform((int32_t)(tid >> 7)), r = (tid >> 3) & 15, s = tid & 7;
  const int i = tid & 127;
  st.piv = L[(int64_t)(i < td ? i : td - 1) * (lda + 1)];
  st.piv = i < td ? st.piv : 1.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c0 = 16 * (2 * k + hi);
    st.d[k] = tc_stage_pair(L, lda, td, c0 + r, c0 + 2 * s);
  }
}
__device__ __forceinline__ void tc_stage_diag_put(TcTrsmSmem& sm, const TcTrsmStage& st) {
  const int tid = tc_tid(), hi = tc_uniform((int32_t)(tid >> 7)), r = (tid >> 3) & 15, s = tid & 7;
  const int qr = r >> 2, qc = s >> 1, k4 = (2 * s) & 3;
  const int e = qr * (qr + 1) / 2 + qc;
  double* g = &sm.dg[0][0][0][0] + ((e >> 1) * 16 + 4 * k4 + (r & 3)) * 2 + (e & 1);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (qc <= qr) {
      g[(2 * k + hi) * 160] = 2 * s < r ? st.d[k].x : 0.0;
      g[(2 * k + hi) * 160 + 8] = 2 * s + 1 < r ? st.d[k].y : 0.0;
    }
  }
  if (tid < 128) sm.rcp[tid] = 1.0 / st.piv;
}
// passes that hold block row b's last block
__host__ __device__ constexpr int tc_stage_end(int b) { return (b * (b + 1) / 2 + 1) / 2; }

// Step B of a strip.  FIRST: the workgroup's first strips, whose steps also
// move block row B of L into LDS (all waves, one barrier).
template <int B, bool FIRST, bool SHARED>
__device__ __forceinline__ void tc_trsm_step(double* __restrict__ X, int64_t lda, int mr, int td, int nbk, int lane,
                                             tc_v4d (&x)[8], const TcTrsmStage& st, TcTrsmSmem& sm) {
  const int s4 = lane >> 4;
  if constexpr (FIRST) {
    if constexpr (B == 0) tc_stage_diag_put(sm, st);
    if constexpr (B > 0) {
#pragma unroll
      for (int k = tc_stage_end(B - 1); k < tc_stage_end(B); ++k) tc_stage_put(sm, k, st);
    }
    __syncthreads();
  }
  TcMicro o;
#pragma unroll
  for (int t = 0; t < 5; ++t) {
    const tc_d2a16 p = *(const tc_d2a16*)&sm.dg[B][t][4 * s4 + (lane & 3)][0];
    o.n[2 * t] = p.x;
    o.n[2 * t + 1] = p.y;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) o.r[q] = sm.rcp[16 * B + 4 * q + s4];
  tc_v4d y[1] = {tc_strip_in(x[B])};
#pragma unroll
  for (int c = 0; c < B; ++c) {
    const double* f = sm.op[B * (B - 1) / 2 + c] + 2 * lane;
    const tc_d2a16 lo = *(const tc_d2a16*)f, hi = *(const tc_d2a16*)(f + 128);
    y[0] = tc_mfma_neg(lo.x, x[c][0], y[0]);
    y[0] = tc_mfma_neg(lo.y, x[c][1], y[0]);
    y[0] = tc_mfma_neg(hi.x, x[c][2], y[0]);
    y[0] = tc_mfma_neg(hi.y, x[c][3], y[0]);
  }
  tc_subst16(y, o);
  x[B] = y[0];
  tc_strip_put<SHARED>(X, lda, mr, td, B, lane, tc_strip_out(y[0]));
  if constexpr (B + 1 < 8) {
    if (B + 1 < nbk) tc_trsm_step<B + 1, FIRST, SHARED>(X, lda, mr, td, nbk, lane, x, st, sm);
  }
}

// A TRSM unit, or the mr <= 64 rows of half a unit as a workgroup of its own
// (each row's arithmetic is the same): wave w takes the strips w and w + 4.
template <bool SHARED>
__device__ __forceinline__ void tc_trsm_rows(double* __restrict__ X, const double* __restrict__ L, int64_t lda,
                                             int mr_in, int td_in, TcTrsmSmem& sm) {
  const int mr = tc_uniform((int32_t)mr_in), td = tc_uniform((int32_t)td_in);
  const int tid = tc_tid(), lane = tid & 63;
  const int w = tc_uniform((int32_t)(tid >> 6));
  const int nbk = (td + 15) >> 4;
  // rows of the strip at r0; a wave without one runs along on row 0 and stores nothing
  auto rows = [&](int r0) { return mr - r0 < 16 ? (mr > r0 ? mr - r0 : 0) : 16; };
  double* X0 = X + (16 * w < mr ? (int64_t)(16 * w) * lda : 0);
  tc_v4d x[8];
  TcTrsmStage st;
  tc_stage_diag(L, lda, td, st);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    x[b] = tc_strip_get(X0, lda, rows(16 * w), td, b, lane);
#pragma unroll
    for (int k = b > 0 ? tc_stage_end(b - 1) : 0; k < tc_stage_end(b); ++k) tc_stage_load(L, lda, td, k, st);
    __builtin_amdgcn_sched_barrier(0);
  }
  tc_trsm_step<0, true, SHARED>(X0, lda, rows(16 * w), td, nbk, lane, x, st, sm);
  if (16 * w + 64 < mr) {
    asm volatile("" ::: "memory");  // operands are read from LDS again, not kept in registers
    double* X1 = X0 + 64 * lda;
#pragma unroll
    for (int b = 0; b < 8; ++b) x[b] = tc_strip_get(X1, lda, rows(16 * w + 64), td, b, lane);
    tc_trsm_step<0, false, SHARED>(X1, lda, rows(16 * w + 64), td, nbk, lane, x, st, sm);
  }
}

// ---------------------------------------------------------------------------
// POTRF work unit: in-place lower Cholesky of the td x td diagonal tile D
// (td <= 128).  The lower triangle is copied once into LDS as packed 16 x 16
// blocks (block (i, j), j <= i, at index i (i + 1) / 2 + j), factored there
// right-looking over 16-column blocks b, and copied back once:
//   1. diagonal block (b, b): unblocked factorization in registers by wave 0
//      (lane i holds row i; right-looking over the block's columns, the
//      POTRF definition on the block; a column's entries reach the other
//      lanes as broadcast operands of the FMAs);
//   2. blocks (i, b), i > b: forward substitution against L_bb (tc_subst16):
//      wave 0 takes block b + 1, waves 1 .. 3 two of the others each;
//   3. blocks (i, j), b < j <= i: A_ij -= L_ib L_jb^T (MFMA, K = 16).
// In step 3 wave 0 updates only block (b+1, b+1), straight from the registers
// of its own substitution, and then factors it (step 1 of b+1) while waves
// 1..3 update the other blocks.
// In-kernel time of one workgroup with a 128 x 128 tile: 22.2 us (43.0 us
// with two lane reads per broadcast, the library square root, a substitution
// with one row per thread and predicated loads; 24.0 us with the whole tile
// copied in before the first pivot and out after the last).  What bounds it:
// the 16 pivots of a diagonal block are one wave's chain of about 210 cycles
// each, 27000 of the 53000 cycles.
// A pivot d <= 0 or NaN stops the factorization: returns the 0-based in-tile
// column, else -1 (the tile is then left partly factored).
// ---------------------------------------------------------------------------
struct alignas(16) TcPotrfSmem {
  double blk[36][256];  // packed lower triangle
  double rcp[16];       // reciprocals of the current diagonal block's pivots
  int fail;
};

__device__ __forceinline__ int tc_pk(int i, int j) { return i * (i + 1) / 2 + j; }

// The packed blocks move in halves of 8 rows x 8 slots, one 16-byte pair per
// lane.  A full tile moves whole pairs: those of a diagonal block reach above
// the diagonal on the way in (entries that never feed one on or below it) and
// are masked on the way out.  A ragged tile reads from clamped positions on
// or below the diagonal and selects when it writes to LDS (zero past td), so
// all loads are in flight together.
__device__ __forceinline__ tc_d2 tc_half_ld(const double* __restrict__ D, int64_t lda, int td, int R, int C) {
  if (td == 128) return *(const tc_d2*)(D + (int64_t)R * lda + C);
  const int Rc = R < td ? R : td - 1, C0 = C < Rc ? C : Rc, C1 = C + 1 < Rc ? C + 1 : Rc;
  tc_d2 v;
  v.x = D[(int64_t)Rc * lda + C0];
  v.y = D[(int64_t)Rc * lda + C1];
  return v;
}
__device__ __forceinline__ double* tc_half_at(TcPotrfSmem& sm, int p, int half, int lane) {
  const int r = 8 * half + (lane >> 3), s = lane & 7;
  return sm.blk[p] + r * 16 + ((s ^ (r & 7)) << 1);
}
__device__ __forceinline__ void tc_half_put(TcPotrfSmem& sm, int p, int half, int lane, int td, int R, int C,
                                            tc_d2 v) {
  tc_d2a16 x;
  x.x = td == 128 || (R < td && C <= R) ? v.x : 0.0;
  x.y = td == 128 || (R < td && C + 1 <= R) ? v.y : 0.0;
  *(tc_d2a16*)tc_half_at(sm, p, half, lane) = x;
}

// Lower triangle of D into the packed blocks: wave 0 only the first diagonal
// block, which it factors while waves 1 .. 3 load the other 35.
__device__ __forceinline__ void tc_pk_load(const double* __restrict__ D, int64_t lda, int td, TcPotrfSmem& sm, int wu,
                                           int lane) {
  const int r8 = lane >> 3, c2 = 2 * (lane & 7);
  if (wu == 0) {
    const tc_d2 a = tc_half_ld(D, lda, td, r8, c2), b = tc_half_ld(D, lda, td, 8 + r8, c2);
    tc_half_put(sm, 0, 0, lane, td, r8, c2, a);
    tc_half_put(sm, 0, 1, lane, td, 8 + r8, c2, b);
    tc_wave_sync();
    return;
  }
  // halves h = wu - 1 + 3 k of blocks 1 + h / 2
  auto at = [&](int h, int& R, int& C) {
    const int p = 1 + (h >> 1);
    int bi = 1;
#pragma unroll
    for (int q = 2; q < 8; ++q) bi += p >= q * (q + 1) / 2;
    R = 16 * bi + 8 * (h & 1) + r8;
    C = 16 * (p - bi * (bi + 1) / 2) + c2;
  };
  if (td == 128) {
    tc_d2 v[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      int R, C;
      at(wu - 1 + 3 * k < 70 ? wu - 1 + 3 * k : 69, R, C);
      v[k] = *(const tc_d2*)(D + (int64_t)R * lda + C);
    }
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      const int h = wu - 1 + 3 * k < 70 ? wu - 1 + 3 * k : 69;
      tc_half_put(sm, 1 + (h >> 1), h & 1, lane, 128, 0, 0, v[k]);
    }
  } else {  // six at a time
    const int nbk = (td + 15) >> 4;
    const int nh = nbk * (nbk + 1) - 2;
#pragma unroll 1
    for (int h0 = wu - 1; h0 < nh; h0 += 18) {
      tc_d2 v[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        int R, C;
        at(h0 + 3 * k < nh ? h0 + 3 * k : nh - 1, R, C);
        v[k] = tc_half_ld(D, lda, td, R, C);
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int h = h0 + 3 * k < nh ? h0 + 3 * k : nh - 1;
        int R, C;
        at(h, R, C);
        tc_half_put(sm, 1 + (h >> 1), h & 1, lane, td, R, C, v[k]);
      }
    }
  }
}

// Block column c of the factor back to D, halves wv, wv + nw, ...
template <bool SHARED>
__device__ __forceinline__ void tc_pk_store_col(double* __restrict__ D, int64_t lda, int td, TcPotrfSmem& sm, int c,
                                                int nbk, int wv, int nw, int lane) {
  const int r8 = lane >> 3, c2 = 2 * (lane & 7);
#pragma unroll 1
  for (int h = wv; h < 2 * (nbk - c); h += nw) {
    const int i = c + (h >> 1);
    const int R = 16 * i + 8 * (h & 1) + r8, C = 16 * c + c2;
    double* g = D + (int64_t)R * lda + C;
    const tc_d2a16 x = *(const tc_d2a16*)tc_half_at(sm, tc_pk(i, c), h & 1, lane);
    if (td == 128 && i != c) {
      tc_st2<SHARED>(g, x.x, x.y);
    } else if (R < td) {
      if (C <= R) tc_st<SHARED>(g, x.x);
      if (C + 1 <= R) tc_st<SHARED>(g + 1, x.y);
    }
  }
}

// Pivot J of the diagonal block held one row per lane (the same in every
// 16-lane row of the wave), and the trailing update a_ik -= l_ij l_kj.  The
// square root and its reciprocal come from one hardware estimate of
// 1 / sqrt(d) (5e-8): a third-order step for the reciprocal root (the binomial
// series of (1 - e)^(-1/2) to e^2), then one residual correction each for the
// root and for 1 / root (Markstein's method).  In the range the caller checks,
// root and reciprocal are the bits of sqrt(d) and of 1 / sqrt(d): 420,000
// pivots are compared in tests/test_gpu_pivot_root.py (two octaves, all
// squares up to 60000^2, their neighbours, exponents 2^-698 .. 2^1000).  70
// cycles of one wave against about 150 for the two library sequences.  m collects
// the smallest high word of a pivot; a pivot of zero, infinity or NaN turns
// every later one of the block into NaN.
#define TC_PIV_LO ((1023 - 700) << 20)  // 2^-700
template <int J>
__device__ __forceinline__ void tc_diag_steps(double (&a)[16], double (&s)[16], double (&r)[16], int32_t& m) {
  const double d = tc_bcast<J>(a[J]);
  const int32_t dh = (int32_t)(__builtin_bit_cast(uint64_t, d) >> 32);
  m = dh < m ? dh : m;
  const double y0 = __builtin_amdgcn_rsq(d);
  const double e = __builtin_fma(-(d * y0), y0, 1.0);
  const double y = __builtin_fma(y0 * e, __builtin_fma(e, 0.375, 0.5), y0);
  const double s0 = d * y;
  s[J] = __builtin_fma(__builtin_fma(-s0, s0, d), 0.5 * y, s0);
  r[J] = __builtin_fma(y, __builtin_fma(-s[J], y, 1.0), y);
  a[J] = a[J] * r[J];
  tc_fmac_bcast<J + 1>(a, a[J], a[J]);
  if constexpr (J + 1 < 16) tc_diag_steps<J + 1>(a, s, r, m);
}

// Step 1 on diagonal block b (nb valid columns, column offset c0 in the
// tile) by the calling wave: factors the block in place, leaves the
// reciprocals of its pivots in rcp, and records the first failing pivot in
// fail.  Columns past nb take a unit pivot.  Entries above the diagonal are
// updated too; they never feed an entry on or below it.
// A pivot below 2^-700 (so any that is not positive) or not finite sends the
// block through the plain form below, from its untouched image in LDS.
__device__ __forceinline__ void tc_pk_diag(TcPotrfSmem& sm, int b, int nb, int c0) {
  const int lane = tc_tid() & 63, r16 = lane & 15;
  double* blk = sm.blk[tc_pk(b, b)];
  double a[16], s[16], r[16];
  tc_row_get(blk, r16, 16, a);
  if (nb < 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = (r16 == k && k >= nb) ? 1.0 : a[k];
  }
  int32_t m = INT32_MAX;
  tc_diag_steps<0>(a, s, r, m);
  if (__builtin_expect(tc_uniform((int32_t)(m >= TC_PIV_LO && s[15] == s[15])) != 0, 1)) {
    if (lane < nb) tc_row_put(blk, lane, 16, a);
    tc_wave_sync();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      blk[tc_bo(j, j, 16)] = s[j];
      sm.rcp[j] = r[j];
    }
    return;
  }
  int bad = -1;
#pragma unroll 1
  for (int j = 0; j < 16; ++j) {
    const double d = j < nb ? blk[tc_bo(j, j, 16)] : 1.0;
    if (bad < 0 && !(d > 0.0)) bad = j;
    const double ljj = sqrt(d), rj = tc_rcp(ljj);
    if (lane == 0) sm.rcp[j] = rj;
    if (j >= nb) continue;
    const double l = blk[tc_bo(r16, j, 16)] * rj;
    tc_wave_sync();
    if (lane < 16 && lane >= j) blk[tc_bo(lane, j, 16)] = lane == j ? ljj : l;
    tc_wave_sync();
#pragma unroll 1
    for (int k = j + 1; k < nb; ++k)
      if (lane < 16 && lane >= k)
        blk[tc_bo(lane, k, 16)] = __builtin_fma(-l, blk[tc_bo(k, j, 16)], blk[tc_bo(lane, k, 16)]);
    tc_wave_sync();
  }
  if (lane == 0 && bad >= 0) sm.fail = c0 + bad;
}

// LOAD: the tile is read from D; otherwise it is in sm.blk already (complete
// for every thread).
template <bool LOAD, bool SHARED>
__device__ __forceinline__ int tc_potrf_body(double* __restrict__ D, int64_t lda, int td_in, TcPotrfSmem& sm) {
  const int td = tc_uniform((int32_t)td_in);
  const int tid = tc_tid(), lane = tid & 63, w = tid >> 6;
  const int wu = tc_uniform((int32_t)w);
  const int r16 = lane & 15, s4 = lane >> 4;
  const int nbk = (td + 15) >> 4;
  if (tid == 0) sm.fail = -1;
  if constexpr (LOAD) tc_pk_load(D, lda, td, sm, wu, lane);
  if (wu == 0) tc_pk_diag(sm, 0, td < 16 ? td : 16, 0);
  __syncthreads();
  int fail = tc_uniform((int32_t)sm.fail);
  for (int b = 0; fail < 0 && b + 1 < nbk; ++b) {
    // 2. the blocks below diagonal block b
    tc_v4d x[2];
    {
      TcMicro o;
      const double* db = sm.blk[tc_pk(b, b)];
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q <= p; ++q) {
          const double v = db[tc_bo(4 * p + (lane & 3), 4 * q + s4, 16)];
          o.n[p * (p + 1) / 2 + q] = (p > q || (lane & 3) > s4) ? v : 0.0;
        }
#pragma unroll
      for (int q = 0; q < 4; ++q) o.r[q] = sm.rcp[4 * q + s4];
      // wave 0: block b + 1; wave w: blocks b + 2 w and b + 2 w + 1
      const int i0 = wu == 0 ? b + 1 : b + 2 * wu, i1 = i0 + 1;
      double* x0 = sm.blk[tc_pk(i0 < nbk ? i0 : b, b)];
      double* x1 = sm.blk[tc_pk(i1 < nbk ? i1 : b, b)];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[0][q] = x0[tc_bo(r16, 4 * q + s4, 16)];
        x[1][q] = x1[tc_bo(r16, 4 * q + s4, 16)];
      }
      if (wu != 0 && i1 < nbk) {
        tc_subst16(x, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          x0[tc_bo(r16, 4 * q + s4, 16)] = x[0][q];
          x1[tc_bo(r16, 4 * q + s4, 16)] = x[1][q];
        }
      } else if (i0 < nbk) {
        tc_v4d y[1] = {x[0]};
        tc_subst16(y, o);
        x[0] = y[0];
#pragma unroll
        for (int q = 0; q < 4; ++q) x0[tc_bo(r16, 4 * q + s4, 16)] = x[0][q];
      }
    }
    __syncthreads();
    // 3. the trailing blocks, numbered u = ii (ii + 1) / 2 + jj for block
    //    (b + 1 + ii, b + 1 + jj), jj <= ii; u = 0 is the next diagonal block
    if (wu == 0) {
      double* cb = sm.blk[tc_pk(b + 1, b + 1)];
      tc_v4d c = tc_acc_get(cb, lane, 16);
#pragma unroll
      for (int q = 0; q < 4; ++q) c = tc_mfma_neg(x[0][q], x[0][q], c);
      tc_acc_put(cb, lane, 16, c);
      tc_wave_sync();
      const int c1 = 16 * (b + 1);
      tc_pk_diag(sm, b + 1, td - c1 < 16 ? td - c1 : 16, c1);
    } else {
      // block rows b + ii, ii = 2 .. m: ii blocks each.  Wave w takes rows
      // m + 1 - w and m - 6 + w (where they are at least 2), which splits the
      // 27 blocks of b = 0 into nine each and the rest within one or two.
      const int m = nbk - 1 - b;
#pragma unroll 1
      for (int h = 0; h < 2; ++h) {
        const int ii = h == 0 ? m + 1 - wu : m - 6 + wu;
        if (ii < 2) continue;
        const tc_q4 xi = tc_frag_get(sm.blk[tc_pk(b + ii, b)], r16, s4, 16);
        double* cb = sm.blk[tc_pk(b + ii, b + 1)];  // the row's blocks are consecutive
        tc_q4 y = tc_frag_get(sm.blk[tc_pk(b + 1, b)], r16, s4, 16);
        tc_v4d c = tc_acc_get(cb, lane, 16);
#pragma unroll 1
        for (int j = 1; j <= ii; ++j) {
          const tc_q4 yj = y;
          const tc_v4d cj = c;
          if (j < ii) {  // the next block's operands, behind this one's products
            y = tc_frag_get(sm.blk[tc_pk(b + j + 1, b)], r16, s4, 16);
            c = tc_acc_get(cb + j * 256, lane, 16);
          }
          tc_acc_put(cb + (j - 1) * 256, lane, 16, tc_nt16(xi, yj, cj));
        }
      }
      // block column b - 2, final since step b - 2, goes back to D here,
      // where these waves wait for wave 0 anyway
      if (b >= 2) tc_pk_store_col<SHARED>(D, lda, td, sm, b - 2, nbk, wu - 1, 3, lane);
    }
    __syncthreads();
    fail = tc_uniform((int32_t)sm.fail);
  }
  if (fail >= 0) return fail;  // (the tile is left partly factored)
  for (int c = nbk > 3 ? nbk - 3 : 0; c < nbk; ++c) tc_pk_store_col<SHARED>(D, lda, td, sm, c, nbk, wu, 4, lane);
  return -1;
}

template <bool SHARED>
__device__ __forceinline__ int tc_potrf_tile(double* __restrict__ D, int64_t lda, int td, TcPotrfSmem& sm) {
  return tc_potrf_body<true, SHARED>(D, lda, td, sm);
}

// ---------------------------------------------------------------------------
// SYRK update of a full 128 x 128 diagonal block, C -= P P^T for P of 128
// rows and kd columns (kd a positive multiple of 16), lower triangle only;
// POTRF: the updated block goes to LDS instead of memory and is factored
// there, so it is neither written nor read back in between (returns the
// failing column or -1).
// The general update gives each wave a 64 x 64 quadrant: on a diagonal block
// one wave idles and two do six tiles of sixteen for nothing.  Here wave w
// takes tile rows w and 7 - w of the lower triangle's 36 16 x 16 tiles, nine
// tiles each, 36 MFMAs per 16-wide k chunk instead of 64.  Only one operand is
// staged (16 KB a chunk), so four stages fit where the general update has two
// and loads run three chunks ahead.  C is read behind the last chunk's
// products.  Each entry's products are summed in the order of the general
// update, so the bits are the same.
// Alone on a CU, kd = 128: 13.1 us (20.2 us as a general update; 18400 cycles
// of MFMAs, 7.7 us); with the POTRF 32.0 us (20.2 + 22.2 us as two bodies).
// ---------------------------------------------------------------------------
template <bool POTRF, bool SHARED>
__device__ __forceinline__ int tc_syrk_block(double* __restrict__ C, const double* __restrict__ P, int64_t lda, int kd,
                                             TcUpdSmem& sm, TcPotrfSmem& pm) {
  const int tid = tc_tid(), lane = tid & 63;
  const int wu = tc_uniform((int32_t)(tid >> 6));
  const int r16 = lane & 15, s4 = lane >> 4;
  double* const st0 = &sm.tile[0][0][0];
  // staging: wave w fetches rows 32 w .. 32 w + 31, eight a load
  const double* src = (const double*)tc_uniform((int64_t)P);
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)(128 * tc_uniform(lda) * 8), 0x00020000);
  const int rl0 = wu * 32 + (lane >> 3);
  const unsigned vof0 = (unsigned)(rl0 * lda * 8 + 16 * ((lane & 7) ^ tc_swz(rl0)));
  const unsigned rowstep = (unsigned)(8 * lda * 8);
  auto stage = [&](int c) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc,
          (tc_lds_void*)((char __attribute__((address_space(3)))*)(tc_lds_void*)st0 + (c & 3) * 16384 +
                         (wu * 4 + q) * 1024),
          16, vof0 + q * rowstep, (unsigned)(c * 128), 0, 0);
  };
  auto frag = [&](int c, int i) { return tc_frag_get(st0 + (c & 3) * 2048 + i * 256, r16, s4, 16); };
  const int nch = kd >> 4;
  const int ra = 7 - wu;  // the wave's tile rows: ra (tiles 0 .. ra) and wu (tiles 0 .. wu)
  tc_v4d acc[8], acd[4];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = tc_v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 4; ++j) acd[j] = tc_v4d{0.0, 0.0, 0.0, 0.0};
  auto products = [&](int c) {
    const tc_q4 fa = frag(c, ra), fd = frag(c, wu);
    tc_q4 f[2];
    f[0] = frag(c, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j <= ra) {
        if (j < 7) f[(j + 1) & 1] = frag(c, j + 1);  // (one more than the last tile needs, at most)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[j] = tc_mfma(tc_el(fa, m), tc_el(f[j & 1], m), acc[j]);
        if (j < 4 && j <= wu) {
#pragma unroll
          for (int m = 0; m < 4; ++m) acd[j & 3] = tc_mfma(tc_el(fd, m), tc_el(f[j & 1], m), acd[j & 3]);
        }
      }
    }
  };
  // chunk c has landed when at most the loads of c + 1 and c + 2 are
  // outstanding (s_waitcnt encodings: 0x0F78 = vmcnt(8), 0x0F74 = vmcnt(4),
  // 0x0F70 = vmcnt(0)); the barrier behind the wait publishes it.  It also
  // frees chunk c - 1's stage, so each wave first waits for its LDS reads
  // (0xC07F = lgkmcnt(0)): the last fragment read may have no product that
  // would wait for it, and nothing else keeps a product in front of a barrier
  auto publish = [] {
    asm volatile("" ::: "memory");  // no LDS read moves across the barrier
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  stage(0);
  if (nch > 1) stage(1);
  if (nch > 2) stage(2);
  for (int c = 0; c < nch - 1; ++c) {
    if (c + 2 < nch) __builtin_amdgcn_s_waitcnt(0x0F78); else __builtin_amdgcn_s_waitcnt(0x0F74);
    publish();
    if (c + 3 < nch) stage(c + 3);
    products(c);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  publish();
  tc_v4d cv[8], cd[4];
  auto cload = [&](int i, int j) {
    const double* p = C + (int64_t)(16 * i + s4) * lda + 16 * j + r16;
    tc_v4d v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[(int64_t)(4 * q) * lda];
    return v;
  };
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j <= ra) cv[j] = cload(ra, j);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j <= wu) cd[j] = cload(wu, j);
  products(nch - 1);
  if constexpr (POTRF) {
    __syncthreads();  // every wave is done with the stages, which the packed blocks overlay
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j <= ra) tc_acc_put(pm.blk[tc_pk(ra, j)], lane, 16, cv[j] - acc[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j <= wu) tc_acc_put(pm.blk[tc_pk(wu, j)], lane, 16, cd[j] - acd[j]);
    __syncthreads();
    return tc_potrf_body<false, SHARED>(C, lda, 128, pm);
  } else {
    auto cstore = [&](int i, int j, tc_v4d v) {
      double* p = C + (int64_t)(16 * i + s4) * lda + 16 * j + r16;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i > j || 4 * q + s4 >= r16) tc_st<SHARED>(p + (int64_t)(4 * q) * lda, v[q]);
    };
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j <= ra) cstore(ra, j, cv[j] - acc[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j <= wu) cstore(wu, j, cd[j] - acd[j]);
    return -1;
  }
}
