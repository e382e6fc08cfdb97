// bf16 weight gradient of layers whose rows are not 16-byte pieces (a width, a height, a stride or a base
// that is no multiple of 8 elements): the kernels with 16-byte LDS loads cannot fetch them.
//
// The operands come through registers instead: 16 bytes per lane at any 2-byte address, two slabs of 32
// tokens ahead, then into LDS, from where the transpose reads and the 32x32x16 MFMAs take them as in the
// aligned kernel (the slots of a token row are XOR-swizzled so that the four tokens of a half-wave's read
// fall on different banks).  A wave owns 64 x 64 of the tile; a workgroup is WM x WN waves side by side
// times WK groups that share the slab's tokens between them (their sums are added in group order when the
// tile leaves).  Several workgroups share a compute unit, so that the loads, the barriers and the store
// phase of one run under the MFMAs of another.
#include "tiles.h"

namespace chunkft {

namespace {

typedef unsigned int u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));   // 16 bytes at any bf16
typedef short i16x4 __attribute__((ext_vector_type(4)));

template <int WM_, int WN_, int WK_, bool UNDER_ = true>
struct RaggedCfg {
  static constexpr bool UNDER = UNDER_;                           // the next slab is stored between the two steps of a slab, else behind them
  static constexpr int WM = WM_, WN = WN_, WK = WK_, BM = 64 * WM, BN = 64 * WN;
  static constexpr int GT = 64 * WM * WN, NT = GT * WK;           // threads of a group, of the workgroup
  static constexpr int BK = 32;
  static constexpr int A_BYTES = BK * BM * 2, B_BYTES = BK * BN * 2, SLAB_BYTES = A_BYTES + B_BYTES;
  static constexpr int NA = A_BYTES / 16 / GT, NB = B_BYTES / 16 / GT;   // 16-byte pieces per thread and slab
  static constexpr int PITCH = BN + 4, HALF = BM / 2;             // the tile leaves in two halves
  static constexpr size_t STAGE_BYTES = (size_t)WK * HALF * PITCH * 4, RING_BYTES = (size_t)WK * 2 * SLAB_BYTES;
  static constexpr size_t LDS_BYTES = STAGE_BYTES > RING_BYTES ? STAGE_BYTES : RING_BYTES;
};

// 16-byte slot of token k that holds logical slot s, in an image of `rows` rows (256 or 128 bytes per token)
template <int ROWS>
__device__ __forceinline__ int swizzle(int s, int k) {
  return ROWS == 128 ? s ^ ((k & 3) << 2) : s ^ (((k >> 1) & 1) << 2);
}

template <class C, bool CLAMP, int MODE>
__global__ __launch_bounds__(C::NT, C::WK == 1 && MODE != EMIT_ADAMW ? 3 : 2) void wgrad_ragged_kernel(const TileGrid q) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int item = xcd_work_item(q.n_items);
  if (item < 0) return;
  const WgradProblem& p = q.p;
  const Place w = place_of<C::BM, C::BN>(q, item);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int group = wave / (C::WM * C::WN), in_group = wave % (C::WM * C::WN);
  const int wm = in_group / C::WN, wn = in_group % C::WN, gtid = (int)threadIdx.x % C::GT;
  // every group does the same number of slabs (the barriers are the workgroup's, see slab_ready); tokens past a group's
  // share or past the end count as zeros of both operands (with zeros in dY alone an infinity in X times them would
  // be NaN)
  const int tokens = (int)(w.k_end - w.k_begin);
  const int nk = ((tokens + C::BK - 1) / C::BK + C::WK - 1) / C::WK;
  const int64_t k0 = w.k_begin + (int64_t)group * nk * C::BK;
  const int64_t last_t = w.k_end - 1;
  unsigned char* const mine = lds + group * (2 * C::SLAB_BYTES);

  // A thread's pieces of an operand lie a whole number of tokens apart: piece i is the thread's first one
  // plus i * TA (TB) tokens, so that a load is a scalar base plus a per-lane offset that never changes.
  constexpr int TA = C::GT / (C::BM / 8), TB = C::GT / (C::BN / 8);
  const int ka = gtid / (C::BM / 8), sa = gtid % (C::BM / 8), kb = gtid / (C::BN / 8), sb = gtid % (C::BN / 8);
  const int64_t lda2 = p.lddy * 2, ldb2 = p.ldx * 2;
  const unsigned ca = (unsigned)((w.row_b + sa * 8) * 2), cb = (unsigned)((w.col_b + sb * 8) * 2);
  const unsigned va = ca + (unsigned)ka * (unsigned)lda2, vb = cb + (unsigned)kb * (unsigned)ldb2;
  auto load = [&](u32x4_t (&a)[C::NA], u32x4_t (&b)[C::NB], int kt) {
    const int64_t t0 = k0 + (int64_t)kt * C::BK;
    if constexpr (CLAMP) {                    // element by element, 64-bit addresses, rows and columns past the end too
      auto piece = [&](const unsigned short* token, int64_t first, int64_t last) {
        unsigned int h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = token[first + e < last ? first + e : last];
        return u32x4_t{h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16};
      };
#pragma unroll
      for (int i = 0; i < C::NA; ++i) {
        const int64_t t = t0 + ka + i * TA;
        a[i] = piece((const unsigned short*)p.dY + (t < last_t ? t : last_t) * p.lddy, w.row_b + sa * 8, p.out - 1);
      }
#pragma unroll
      for (int i = 0; i < C::NB; ++i) {
        const int64_t t = t0 + kb + i * TB;
        b[i] = piece((const unsigned short*)p.X + (t < last_t ? t : last_t) * p.ldx, w.col_b + sb * 8, p.in - 1);
      }
    } else if (t0 + C::BK <= w.k_end) {
      const char* const ga = (const char*)p.dY + t0 * lda2;
      const char* const gb = (const char*)p.X + t0 * ldb2;
#pragma unroll
      for (int i = 0; i < C::NA; ++i) a[i] = *(const u32x4_a2*)(ga + i * TA * lda2 + va);
#pragma unroll
      for (int i = 0; i < C::NB; ++i) b[i] = *(const u32x4_a2*)(gb + i * TB * ldb2 + vb);
    } else {                                  // tokens past the end: the last one, both sides zeroed when they are stored
      const int64_t tl = t0 < last_t ? t0 : last_t;
      const int left = (int)(last_t - tl);
      const char* const ga = (const char*)p.dY + tl * lda2;
      const char* const gb = (const char*)p.X + tl * ldb2;
#pragma unroll
      for (int i = 0; i < C::NA; ++i) {
        const int k = ka + i * TA < left ? ka + i * TA : left;
        a[i] = *(const u32x4_a2*)(ga + (ca + (unsigned)k * (unsigned)lda2));
      }
#pragma unroll
      for (int i = 0; i < C::NB; ++i) {
        const int k = kb + i * TB < left ? kb + i * TB : left;
        b[i] = *(const u32x4_a2*)(gb + (cb + (unsigned)k * (unsigned)ldb2));
      }
    }
  };
  // Tokens past the end become zeros in registers, in slabs that are cut (64 x 128 and 64 x 64 tiles: no slower than without
  // the zeros in X).  On the 128 x 128 tile that form costs the fused call 6 % (4097 x 4095, 2048 tokens: 219 -> 233 us); there dY
  // is selected piece by piece and X overwritten behind its stores (224 us).  The gradient alone: 112 us in each form.
  auto store = [&](u32x4_t (&a)[C::NA], u32x4_t (&b)[C::NB], int kt) {
    unsigned char* const dst = mine + (kt & 1) * C::SLAB_BYTES;
    const int64_t t0 = k0 + (int64_t)kt * C::BK;
    const bool cut = t0 + C::BK > w.k_end;
    const u32x4_t zeros = {0u, 0u, 0u, 0u};
    if constexpr (C::WK > 1) {
      if (cut) {
        const int left = (int)(w.k_end - t0);
#pragma unroll
        for (int i = 0; i < C::NA; ++i)
          if (ka + i * TA >= left) a[i] = zeros;
#pragma unroll
        for (int i = 0; i < C::NB; ++i)
          if (kb + i * TB >= left) b[i] = zeros;
      }
    }
    auto slot_a = [&](int k) { return (u32x4_t*)(dst + k * (C::BM * 2) + swizzle<C::BM>(sa, k) * 16); };
    auto slot_b = [&](int k) { return (u32x4_t*)(dst + C::A_BYTES + k * (C::BN * 2) + swizzle<C::BN>(sb, k) * 16); };
#pragma unroll
    for (int i = 0; i < C::NA; ++i) {
      if (C::WK == 1 && t0 + ka + i * TA > last_t) a[i] = zeros;
      *slot_a(ka + i * TA) = a[i];
    }
#pragma unroll
    for (int i = 0; i < C::NB; ++i) *slot_b(kb + i * TB) = b[i];
    if (C::WK == 1 && cut) {
#pragma unroll
      for (int i = 0; i < C::NB; ++i)
        if (t0 + kb + i * TB > last_t) *slot_b(kb + i * TB) = zeros;
    }
  };

  // transpose reads: in a block of 16 lanes lane j names 4 rows of token j / 4 and receives the 4 tokens of
  // row j; lanes 0-31 take tokens 0-7 of a 16-token step, lanes 32-63 tokens 8-15
  const int blk = lane >> 4, i16 = lane & 15;
  const int tr_k = (blk >> 1) * 8 + (i16 >> 2), low = (blk & 1) * 2 + ((i16 & 3) >> 1), sub = (i16 & 1) * 8;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto frag = [&](const unsigned char* image, int pitch, int slot0, int ks, auto rowsc) {
    constexpr int ROWS = decltype(rowsc)::value;
    bf16x4 h[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = ks * 16 + u * 4 + tr_k;
      const unsigned char* src = image + k * pitch + (swizzle<ROWS>(slot0, k) + low) * 16 + sub;
      h[u] = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(i16x4))(uintptr_t)(unsigned)(uintptr_t)src));
    }
    return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // `between` runs between the two 16-token steps: the loop stores the next slab there, under the matrix instructions of
  // the second step (behind them the barrier waited for the LDS writes: fused call, 12 Mi elements of 32003 x 4096 at 1536
  // tokens 119 -> 113 us, 7 Mi of 2705 x 2907 at 1024 tokens 89 -> 83; in front of the first step, or with the fragments of both
  // steps read at once, 114 - 116 and 83 - 84).
  auto multiply = [&](int kt, auto&& between) {
    const unsigned char* const src = mine + (kt & 1) * C::SLAB_BYTES;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = frag(src, C::BM * 2, wm * 8 + i * 4, ks, IntC<C::BM>{});
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = frag(src + C::A_BYTES, C::BN * 2, wn * 8 + j * 4, ks, IntC<C::BN>{});
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      if (ks == 0) between();
    }
  };

  u32x4_t a0[C::NA], a1[C::NA], b0[C::NB], b1[C::NB];
  // The first slabs of a group that has no token in them are not fetched: with few tokens that was most of the call (17 x 29,
  // one token 7.1 -> 4.3 us; 535 x 29, 6 tokens 7.9 -> 5.0).  In the loop the same test costs 3 % at 1024 tokens.
  auto begin_with = [&](u32x4_t (&a)[C::NA], u32x4_t (&b)[C::NB], int kt) {
    if (C::WK < 4 || k0 + (int64_t)kt * C::BK < w.k_end) {
      load(a, b, kt);
    } else {
#pragma unroll
      for (int i = 0; i < C::NA; ++i) a[i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < C::NB; ++i) b[i] = u32x4_t{0u, 0u, 0u, 0u};
    }
  };
  // A slab is in LDS for those who read it.  A group of one wave has its slabs to itself, and LDS serves a wave's accesses in the order
  // they are issued: there only the compiler has to keep that order.  With the workgroup's barrier each of the four waves of a 64 x 64
  // tile waited for the slowest one's loads in every slab (1 Mi elements of 32003 x 4096, 2047 tokens, gradient / fused call 22.5 / 28.0 us, without
  // 19.8 / 24.8; 1001 x 1003, 5000 tokens, 32.9 / 42.8 and 31.0 / 39.9).
  auto slab_ready = [&] {
    if constexpr (C::GT == 64) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  };
  begin_with(a0, b0, 0);
  begin_with(a1, b1, 1);                            // past the end: clamped, never multiplied
  store(a0, b0, 0);
  slab_ready();
  int kt = 0;
  for (; kt + 2 < nk; kt += 2) {
    load(a0, b0, kt + 2);
    multiply(kt, [&] { if constexpr (C::UNDER) store(a1, b1, kt + 1); });
    if constexpr (!C::UNDER) store(a1, b1, kt + 1);
    slab_ready();
    load(a1, b1, kt + 3);                     // may be past the end: clamped, never multiplied
    multiply(kt + 1, [&] { if constexpr (C::UNDER) store(a0, b0, kt + 2); });
    if constexpr (!C::UNDER) store(a0, b0, kt + 2);
    slab_ready();
  }
  multiply(kt, [] {});
  if (kt + 1 < nk) {
    store(a1, b1, kt + 1);
    slab_ready();
    multiply(kt + 1, [] {});
  }

  // register v of a block is row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32; half h of the tile is
  // block row h of every wave
  float* const staged = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();                          // the slabs (the rows of the other half) have been read
    float* const dst = staged + (group * C::HALF + wm * 32 + (lane >> 5) * 4) * C::PITCH + wn * 64 + (lane & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) dst[((v >> 2) * 8 + (v & 3)) * C::PITCH + j * 32] = acc[h][j][v];
    __syncthreads();
    emit_rows<MODE, C::HALF, C::BN, C::PITCH, C::NT, C::WK>(q, w, staged, [h](int rr) { return rr / 32 * 64 + h * 32 + rr % 32; });
  }
}

template <class C, bool CLAMP, int MODE>
int launch_kernel(const TileGrid& q, hipStream_t st) {
  const int err = raise_lds_limit<&wgrad_ragged_kernel<C, CLAMP, MODE>>(C::LDS_BYTES);
  if (err != 0) return err;
  hipLaunchKernelGGL((wgrad_ragged_kernel<C, CLAMP, MODE>), dim3((q.n_items + 7) / 8 * 8), dim3(C::NT), C::LDS_BYTES, st, q);
  return (int)hipGetLastError();
}

template <class C, bool CLAMP>
int launch_cfg(const WgradProblem& p, int mode, const Sinks& s, hipStream_t st) {
  TileGrid q;
  if (!fill_grid<C::BM, C::BN>(q, p, s, 1)) return (int)hipErrorInvalidValue;
  switch (mode) {
    case EMIT_STORE: return launch_kernel<C, CLAMP, EMIT_STORE>(q, st);
    case EMIT_ACCUM: return launch_kernel<C, CLAMP, EMIT_ACCUM>(q, st);
    case EMIT_PARTIAL: return launch_kernel<C, CLAMP, EMIT_PARTIAL>(q, st);
    default: return launch_kernel<C, CLAMP, EMIT_ADAMW>(q, st);
  }
}

// The update on the 64 x 128 tile, the slab stored behind both steps: the loop is slower, but the kernel's epilogue streams the state a little
// faster where rows of the state are whole 16-byte pieces, and up to 512 tokens that decides.  Fused call in us, stored between / behind: 4 Mi elements
// of 32003 x 4096 1 token 25.9 / 25.0, 256 tokens 29.6 / 28.5, 512 tokens 35.2 / 34.4; of 50257 x 768 256 tokens 30.3 / 29.3, 512 tokens 36.2 /
// 35.1, 768 tokens 38.1 / 39.0; 16 Mi 256 tokens 96.5 / 94.5, 32 Mi 512 tokens 192.0 / 189.1.  On other rows neither is ahead up to 256 tokens
// (4 Mi of 2705 x 2907 128 tokens 35.1 / 34.8, 16 Mi of 31999 x 4100 40 tokens 125.5 / 128.4) and the first beyond (4 Mi of 4097 x 4095
// 420 tokens 43.4 / 44.4).
int launch_update_behind(const WgradProblem& p, const Sinks& s, hipStream_t st) {
  typedef RaggedCfg<1, 2, 2, false> C;
  TileGrid q;
  if (!fill_grid<C::BM, C::BN>(q, p, s, 1)) return (int)hipErrorInvalidValue;
  return launch_kernel<C, false, EMIT_ADAMW>(q, st);
}

}  // namespace

// Which tile (times: gradient / fused call; a scalar-FMA tile was here before, 807 us on the first):
//   32003 x 4096, 16 Mi elements, 1024 tokens: 64 x 128 in two token groups 75 / 123 us, 128 x 128 71 / 139,
//   64 x 64 in four token groups 103 / 143;
//   4097 x 4095, 2048 tokens: 155 / 212, 112 / 224, 193 / 257 us;
//   2705 x 2907, 1.5 Mi elements, 1024 tokens (115 tiles of 128 x 128): 16.6 / 32.8, 19.7 / 42.5, 16.3 / 27.7 us;
//   32003 x 4096, 12 Mi elements, 1536 tokens: 80 / 121, 67 / 118 us;
//   1001 x 1003, 1024 tokens (64 tiles): 15.4 / 26.4, 20.3 / 45.6, 12.2 / 18.7 us.
// (Before the slab was stored between the steps and the waves of a 64 x 64 tile went without the barrier; since then 70 / 123, 98 / 204, 14.8 /
// 26.5, 66 / 111 and 10.0 / 17.1 us for the tiles chosen.)
// The update's streams (82 us of the 123) run under the loops of the other workgroups of a compute unit, of
// which the 64 x 128 tile leaves more room for; with more tokens the loop decides, and the larger tile reads
// its operands fewer times.  Every mode of a call takes the same tile: the order of the sum is the same.
int launch_wgrad_ragged(const WgradProblem& p, int mode, const Sinks& s, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  const int64_t rows = (p.end - 1) / p.in - p.begin / p.in + 1;
  const bool near = p.out + 32 * p.lddy < (int64_t(1) << 31) && p.in + 32 * p.ldx < (int64_t(1) << 31);   // byte offsets of a slab in 32 bits
  if (p.out < 64 || p.in < 64 || !near) return launch_cfg<RaggedCfg<1, 1, 4>, true>(p, mode, s, st);
  const bool few = ceil_div(rows, 128) * ceil_div(p.in, 128) * p.S <= device_compute_units();
  if (few || p.in < 128) return launch_cfg<RaggedCfg<1, 1, 4>, false>(p, mode, s, st);
  if (p.kslab <= 1024 || p.out < 128) {
    if (mode == EMIT_ADAMW && p.in % 8 == 0 && p.kslab <= 512) return launch_update_behind(p, s, st);
    return launch_cfg<RaggedCfg<1, 2, 2>, false>(p, mode, s, st);
  }
  return launch_cfg<RaggedCfg<2, 2, 1>, false>(p, mode, s, st);
}

}  // namespace chunkft
