// Device helpers shared by the kernels: bf16 conversion, the AdamW update, and what turns a
// gradient value (or four of them) into its destination.
#ifndef CHUNKFT_DEVICE_H
#define CHUNKFT_DEVICE_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace chunkft {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at any dword
typedef unsigned int u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));   // 8 bytes at any bf16
#define LDS_PTR(T) __attribute__((address_space(3))) T*
#define GLOBAL_PTR(T) __attribute__((address_space(1))) T*

// Compile-time loop: the body sees its index as a constant, so register arrays
// indexed by it never fall back to scratch memory.
template <int I> struct IntC { static constexpr int value = I; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IntC<I>{});
    static_for<N, I + 1>(f);
  }
}

// LDS transpose read issued as opaque assembly: the compiler must not know that
// it reads LDS, or it would wait for every outstanding global->LDS load before
// it.  The counterpart is that waiting for its result is also done by hand,
// and that no branch may lie between a read and its wait.
template <int OFF>
__device__ __forceinline__ bf16x4 lds_tr_read(unsigned addr) {
  bf16x4 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  return r;
}
// s_waitcnt vmcnt(N) alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, others "no wait")
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float bf16_bits_to_f32(unsigned short b) {
  return __uint_as_float(((unsigned int)b) << 16);
}

template <typename T> __device__ __forceinline__ float load_as_f32(const T* p);
template <> __device__ __forceinline__ float load_as_f32<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_as_f32<unsigned short>(const unsigned short* p) {
  return bf16_bits_to_f32(*p);
}

// One AdamW update in fp32 (Algorithm 1 lines 19-21).  Every path that updates
// state goes through this function so that fused and un-fused calls agree bit
// for bit; contraction is written out (the file is built with -ffp-contract=off).
// The last line is theta - lr * (m_hat / (sqrt(v_hat) + eps) + wd * theta).
__device__ __forceinline__ void adamw_update(float g, float& theta, float& m, float& v,
                                             const AdamWConsts& c) {
  const float m_new = fmaf(c.beta1, m, c.one_minus_beta1 * g);
  const float v_new = fmaf(c.beta2, v, c.one_minus_beta2 * (g * g));
  const float m_hat = m_new * c.inv_bias1;
  const float v_hat = v_new * c.inv_bias2;
  // v_sqrt_f32 and v_rcp_f32 are accurate to 1 ulp: far inside the 1e-5 the update is held to,
  // and an order of magnitude fewer instructions than the correctly rounded sequences
  const float step = fmaf(m_hat, __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(v_hat) + c.eps), c.weight_decay * theta);
  theta = fmaf(-c.lr, step, theta);
  m = m_new;
  v = v_new;
}

// Turn one gradient value into its destination.  i = chunk-local index,
// flat = element index in the tensor, slab = token slab of a split call.
template <int MODE>
__device__ __forceinline__ void emit(const Sinks& s, int64_t E, int32_t slab, int64_t i,
                                     int64_t flat, float val) {
  if constexpr (MODE == EMIT_STORE) {
    s.g[i] = val;
  } else if constexpr (MODE == EMIT_ACCUM) {
    s.g[i] += val;
  } else if constexpr (MODE == EMIT_PARTIAL) {
    s.ws[(int64_t)slab * s.ws_pitch + i] = val;
  } else {
    float th = s.master[i], mm = s.m[i], vv = s.v[i];
    adamw_update(val, th, mm, vv, s.c);
    s.master[i] = th;
    s.m[i] = mm;
    s.v[i] = vv;
    if (s.w_kind == W_BF16) ((unsigned short*)s.W)[flat] = f32_to_bf16_rne(th);
    else if (s.w_kind == W_F32) ((float*)s.W)[flat] = th;
  }
}

// Four consecutive gradient values at once.  The 16-byte fp32 accesses work at
// any 4-byte alignment but stream about 15% faster when 16-byte aligned, whereas
// the 8-byte bf16 store costs next to nothing at 2-byte alignment: callers align
// their groups of four to the fp32 arrays.  Pointers are already offset to the
// first of the four elements.
struct Vec4Sink {
  float* g;        // EMIT_STORE / EMIT_ACCUM / EMIT_PARTIAL destination
  float* master;
  float* m;
  float* v;
  void* W;         // low-precision copy (bf16 or fp32) or nullptr
};

// Chunk state and gradients are streamed: read once, written once, never reused
// by the same kernel, and far larger than the caches.  All these accesses carry
// the non-temporal hint.
struct State4 {
  f32x4_u th, mm, vv;
};

template <int MODE>
__device__ __forceinline__ State4 load_state4(const Vec4Sink& d) {
  State4 st;
  if constexpr (MODE == EMIT_ACCUM) {
    st.th = __builtin_nontemporal_load((const f32x4_u*)d.g);
  } else if constexpr (MODE == EMIT_ADAMW) {
    st.th = __builtin_nontemporal_load((const f32x4_u*)d.master);
    st.mm = __builtin_nontemporal_load((const f32x4_u*)d.m);
    st.vv = __builtin_nontemporal_load((const f32x4_u*)d.v);
  }
  return st;
}

constexpr int kNonTemporal = 2;   // the nt bit in the cache policy of a buffer access

__device__ __forceinline__ void update4(f32x4_u val, State4& st, const AdamWConsts& c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float t = st.th[e], a = st.mm[e], b = st.vv[e];
    adamw_update(val[e], t, a, b, c);
    st.th[e] = t; st.mm[e] = a; st.vv[e] = b;
  }
}

__device__ __forceinline__ u32x2_a2 pack_bf16(f32x4_u x) {
  u32x2_a2 pk;
  pk[0] = (unsigned int)f32_to_bf16_rne(x[0]) | ((unsigned int)f32_to_bf16_rne(x[1]) << 16);
  pk[1] = (unsigned int)f32_to_bf16_rne(x[2]) | ((unsigned int)f32_to_bf16_rne(x[3]) << 16);
  return pk;
}

template <int MODE>
__device__ __forceinline__ void finish4(const Vec4Sink& d, int w_kind, const AdamWConsts& c, f32x4_u val,
                                        State4 st) {
  if constexpr (MODE == EMIT_STORE || MODE == EMIT_PARTIAL) {
    // the gradient is read again by the next kernel (AdamW or the slab reduction):
    // a plain store lets the 256 MB memory-side cache keep it
    *(f32x4_u*)d.g = val;
  } else if constexpr (MODE == EMIT_ACCUM) {
    st.th += val;
    *(f32x4_u*)d.g = st.th;
  } else {
    update4(val, st, c);
    __builtin_nontemporal_store(st.th, (f32x4_u*)d.master);
    __builtin_nontemporal_store(st.mm, (f32x4_u*)d.m);
    __builtin_nontemporal_store(st.vv, (f32x4_u*)d.v);
    if (w_kind == W_BF16) {
      __builtin_nontemporal_store(pack_bf16(st.th), (u32x2_a2*)d.W);
    } else if (w_kind == W_F32) {
      __builtin_nontemporal_store(st.th, (f32x4_u*)d.W);
    }
  }
}

// Workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets one contiguous run of work
// items so that tiles sharing dY rows / X columns meet in the same L2.  Returns -1 for the
// padding workgroups at the end of the grid.
__device__ __forceinline__ int xcd_work_item(int n_items) {
  const int per_xcd = (n_items + 7) >> 3;
  const int item = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  return item < n_items ? item : -1;
}

}  // namespace chunkft
#endif
