// Weight gradient of an fp32 layer on the fp32 matrix instruction (32x32x2: fp32 products, fp32 sums).
//
// Both operands have the contraction index (the token) outermost, and that is what this instruction
// wants: a lane holds ONE token's value of its row (column).  So there is nothing to transpose, and a wave
// that takes 1 x TN blocks gives lane l the columns TN * (l % 32) ... + TN - 1: TN consecutive floats.
//
// A workgroup is WK waves on ONE 32 x 32 TN tile, each taking a contiguous WK-th of the slab's tokens;
// their partial tiles meet in LDS and are added in wave order while the tile leaves row by row, 16 bytes
// per lane.  Splitting the tokens instead of the tile inside the workgroup keeps the tile small: the
// number of tiles, and not the size of a layer, decides whether the compute units are filled and how even
// the last round is; and as no wave needs another's operands there is no barrier in the loop.  A wave
// alone can keep its matrix core busy (an instruction takes 64 cycles); what bounds the kernel is how fast
// the operands reach the compute unit.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "tiles.h"

namespace chunkft {

namespace {

template <int TN_, int WK_>
struct F32Cfg {
  static constexpr int TN = TN_, WK = WK_, BM = 32, BN = 32 * TN, NT = 64 * WK;
  static constexpr int ROW_STEP = 1;
  static constexpr int U = 8;                       // two-token steps whose operands are loaded together
  static constexpr int PITCH = BN + 4;              // staged row: 16-byte aligned, rows shifted by 4 banks
  static constexpr size_t LDS_BYTES = (size_t)WK * BM * PITCH * 4;
};

template <int TN_, int WK_, int NS_>
struct F32RingCfg {
  static constexpr int TN = TN_, WK = WK_, BM = 32, BN = 32 * TN, NT = 64 * WK;
  static constexpr int ROW_STEP = 4;                // tiles begin at whole 16-byte pieces of dY
  static constexpr int KS = 8, U = KS / 2, NS = NS_;
  static constexpr int A_BYTES = KS * BM * 4, B_BYTES = KS * BN * 4, SLAB_BYTES = A_BYTES + B_BYTES;
  static constexpr int L = 1 + TN;                  // 1 KB loads per slab
  static constexpr int PITCH = BN + 4;
  static constexpr size_t STAGE_BYTES = (size_t)WK * BM * PITCH * 4, RING_BYTES = (size_t)WK * NS * SLAB_BYTES;
  static constexpr size_t LDS_BYTES = STAGE_BYTES > RING_BYTES ? STAGE_BYTES : RING_BYTES;
};

// N consecutive floats: in registers, and in memory at any dword
template <int N> struct FloatN {
  typedef float reg __attribute__((ext_vector_type(N)));
  typedef float mem __attribute__((ext_vector_type(N), aligned(4)));
};
template <> struct FloatN<1> { typedef float reg, mem; };
__device__ __forceinline__ float element(float v, int) { return v; }
template <class V> __device__ __forceinline__ float element(V v, int i) { return v[i]; }

template <class C>
__device__ __forceinline__ void clear(f32x16 (&acc)[C::TN]) {
#pragma unroll
  for (int j = 0; j < C::TN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
}

template <class C>
__device__ __forceinline__ void mma(f32x16 (&acc)[C::TN], float a, typename FloatN<C::TN>::reg b) {
#pragma unroll
  for (int j = 0; j < C::TN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, element(b, j), acc[j], 0, 0, 0);
}

// The waves' partial tiles meet in LDS and leave row by row.
template <class C, int MODE>
__device__ __forceinline__ void finish_tile(const TileGrid& q, const Place& w, const f32x16 (&acc)[C::TN],
                                            float* staged, int wave, int lane) {
  // register v of block j is row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column TN * (lane % 32) + j
  float* const mine = staged + wave * (C::BM * C::PITCH) + C::TN * (lane & 31);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    float* dst = mine + ((v >> 2) * 8 + (lane >> 5) * 4 + (v & 3)) * C::PITCH;
#pragma unroll
    for (int j = 0; j < C::TN; ++j) dst[j] = acc[j][v];
  }
  __syncthreads();
  emit_rows<MODE, C::BM, C::BN, C::PITCH, C::NT, C::WK>(q, w, staged, [](int rr) { return rr; });
}

// Operands straight from memory: any alignment, any size.
template <class C, int MODE>
__global__ __launch_bounds__(C::NT) void wgrad_f32_kernel(const TileGrid q) {
  extern __shared__ __attribute__((aligned(16))) float staged[];        // [WK][BM][PITCH]
  typedef typename FloatN<C::TN>::reg VB;
  const int item = xcd_work_item(q.n_items);
  if (item < 0) return;
  const WgradProblem& p = q.p;
  const Place w = place_of<C::BM, C::BN>(q, item);
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int steps = (int)((w.k_end - w.k_begin + 1) >> 1);
  const int per_wave = (steps + C::WK - 1) / C::WK;
  const int step0 = wave * per_wave < steps ? wave * per_wave : steps;
  const int step1 = step0 + per_wave < steps ? step0 + per_wave : steps;
  const int64_t t_last = w.k_end - 1;

  int64_t ra = w.row_b + (lane & 31), cb = w.col_b + C::TN * (lane & 31);
  ra = ra < p.out ? ra : p.out - 1;
  if constexpr (C::TN == 1) cb = cb < p.in ? cb : p.in - 1;
  const float* const pa = (const float*)p.dY + ra;
  const float* const pb = (const float*)p.X + cb;
  f32x16 acc[C::TN];
  clear<C>(acc);

  auto load = [&](float (&a)[C::U], VB (&b)[C::U], int s) {              // steps s ... s + U - 1, all complete
    const int64_t t = w.k_begin + 2 * (int64_t)s + half;
    const float* qa = pa + t * p.lddy;
    const float* qb = pb + t * p.ldx;
#pragma unroll
    for (int u = 0; u < C::U; ++u) {
      a[u] = qa[(int64_t)(2 * u) * p.lddy];
      b[u] = *(const typename FloatN<C::TN>::mem*)(qb + (int64_t)(2 * u) * p.ldx);
    }
  };
  auto mma_all = [&](const float (&a)[C::U], const VB (&b)[C::U]) {
#pragma unroll
    for (int u = 0; u < C::U; ++u) mma<C>(acc, a[u], b[u]);
  };

  // the wave's tokens: whole groups of U steps, the loads of a group in flight under the
  // instructions of the one before; then what is left
  const bool odd_end = ((w.k_end - w.k_begin) & 1) != 0 && step1 == steps;   // the last step holds one token
  const int n_full = (step1 - step0 - (odd_end ? 1 : 0)) / C::U;
  int s = step0;
  if (n_full > 0) {
    float a0[C::U], a1[C::U];
    VB b0[C::U], b1[C::U];
    load(a0, b0, s);
    int g = 0;
    for (; g + 2 < n_full; g += 2) {
      load(a1, b1, s + C::U);
      __builtin_amdgcn_sched_barrier(0);
      mma_all(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      load(a0, b0, s + 2 * C::U);
      __builtin_amdgcn_sched_barrier(0);
      mma_all(a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      s += 2 * C::U;
    }
    if (g + 1 < n_full) {
      load(a1, b1, s + C::U);
      __builtin_amdgcn_sched_barrier(0);
      mma_all(a0, b0);
      mma_all(a1, b1);
      s += 2 * C::U;
    } else {
      mma_all(a0, b0);
      s += C::U;
    }
  }
  for (; s < step1; s += C::U) {                                      // fewer than U steps, or U with one token short
    float a[C::U];
    VB b[C::U];
#pragma unroll
    for (int u = 0; u < C::U; ++u) {
      const int64_t t = w.k_begin + 2 * (int64_t)(s + u) + half;
      const int64_t tc = t < t_last ? t : t_last;                     // past the end: the last token, zeroed below
      a[u] = pa[tc * p.lddy];
      b[u] = *(const typename FloatN<C::TN>::mem*)(pb + tc * p.ldx);
    }
#pragma unroll
    for (int u = 0; u < C::U; ++u) {
      if (s + u >= step1) break;
      if (w.k_begin + 2 * (int64_t)(s + u) + half > t_last) {
        a[u] = 0.f;
        b[u] = VB{};
      }
      mma<C>(acc, a[u], b[u]);
    }
  }
  finish_tile<C, MODE>(q, w, acc, staged, wave, lane);
}

// Operands through LDS, in a ring that belongs to one wave (no barrier in the loop): slabs of 8 tokens,
// 16 bytes per lane straight into LDS.  The rows of dY and X must be 16-byte pieces.
// (The LDS reads are opaque assembly for the same reason as the transpose reads of the bf16 kernel: the
// compiler must not wait for the loads in flight; the wait for their results is written out.)
template <int N, int OFF>
__device__ __forceinline__ typename FloatN<N>::reg lds_read(unsigned addr) {
  typename FloatN<N>::reg r;
  if constexpr (N == 1) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  else if constexpr (N == 2) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
  return r;
}

template <class C, int MODE>
__global__ __launch_bounds__(C::NT, 2) void wgrad_f32_ring_kernel(const TileGrid q) {
  extern __shared__ __attribute__((aligned(1024))) float staged[];
  typedef typename FloatN<C::TN>::reg VB;
  const int item = xcd_work_item(q.n_items);
  if (item < 0) return;
  const WgradProblem& p = q.p;
  const Place w = place_of<C::BM, C::BN>(q, item);
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int slabs = (int)((w.k_end - w.k_begin + C::KS - 1) / C::KS);
  const int per_wave = (slabs + C::WK - 1) / C::WK;
  const int s0 = wave * per_wave < slabs ? wave * per_wave : slabs;
  const int s1 = s0 + per_wave < slabs ? s0 + per_wave : slabs;
  const int nk = s1 - s0;
  const int64_t k0 = w.k_begin + (int64_t)s0 * C::KS;
  const int valid = (int)((k0 + (int64_t)nk * C::KS < w.k_end ? k0 + (int64_t)nk * C::KS : w.k_end) - k0);   // tokens of this wave

  // ---- memory -> LDS: load j of an operand holds its tokens j * TPL ... + TPL - 1, lane l the 16-byte
  // piece l % LPT of token l / LPT; the source is a scalar base that moves one slab per fetch plus a
  // per-lane offset that never changes
  constexpr int LPT_A = C::BM / 4, LPT_B = C::BN / 4, TPL_B = 64 / LPT_B;
  const unsigned lda = (unsigned)(p.lddy * 4), ldb = (unsigned)(p.ldx * 4);
  const unsigned va = (unsigned)(lane / LPT_A) * lda + (unsigned)(w.row_b + lane % LPT_A * 4) * 4u;
  const unsigned vb = (unsigned)(lane / LPT_B) * ldb + (unsigned)(w.col_b + lane % LPT_B * 4) * 4u;
  const char* ga = (const char*)p.dY + k0 * p.lddy * 4;
  const char* gb = (const char*)p.X + k0 * p.ldx * 4;
  const unsigned ring = (unsigned)(uintptr_t)staged + wave * (C::NS * C::SLAB_BYTES);
  int fetched = 0;
  auto to_lds = [&](const char* base, unsigned voff, unsigned soff, unsigned dst) {
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (LDS_PTR(void))(uintptr_t)dst, 16, (int)voff, (int)soff, 0, 0);
  };
  auto fetch = [&](int slot) {                             // slab `fetched` into ring slot `slot`
    const unsigned dst = ring + slot * C::SLAB_BYTES;
    const int left = valid - fetched * C::KS;              // tokens past the end step back to the last one
    if (left >= C::KS) {
      to_lds(ga, va, 0, dst);
#pragma unroll
      for (int j = 0; j < C::TN; ++j) to_lds(gb, vb, (unsigned)(j * TPL_B) * ldb, dst + C::A_BYTES + j * 1024);
    } else {
      const int ta = lane / LPT_A < left ? lane / LPT_A : left - 1;
      to_lds(ga, (unsigned)ta * lda + (unsigned)(w.row_b + lane % LPT_A * 4) * 4u, 0, dst);
#pragma unroll
      for (int j = 0; j < C::TN; ++j) {
        const int t = j * TPL_B + lane / LPT_B, tc = t < left ? t : left - 1;
        to_lds(gb, (unsigned)tc * ldb + (unsigned)(w.col_b + lane % LPT_B * 4) * 4u, 0, dst + C::A_BYTES + j * 1024);
      }
    }
    ga += (int64_t)C::KS * p.lddy * 4;
    gb += (int64_t)C::KS * p.ldx * 4;
    ++fetched;
  };

  // ---- LDS -> registers: step u of a slab is tokens 2u, 2u + 1, the lane's is 2u + lane / 32
  const unsigned ra = ring + half * (C::BM * 4) + (lane & 31) * 4;
  const unsigned rb = ring + C::A_BYTES + half * (C::BN * 4) + (lane & 31) * (C::TN * 4);
  auto read = [&](float (&a)[C::U], VB (&b)[C::U], int slot) {
    const unsigned so = slot * C::SLAB_BYTES;
    static_for<C::U>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      a[u] = lds_read<1, u * 2 * C::BM * 4>(ra + so);
      b[u] = lds_read<C::TN, u * 2 * C::BN * 4>(rb + so);
    });
  };
  auto landed = [&](float (&a)[C::U], VB (&b)[C::U]) {         // the reads have returned
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])::"memory");
  };
  f32x16 acc[C::TN];
  clear<C>(acc);
  float a0[C::U], a1[C::U];
  VB b0[C::U], b1[C::U];
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < C::NS; ++i)
      if (i < nk) fetch(i);
    if (nk >= C::NS) wait_vmcnt<(C::NS - 1) * C::L>(); else wait_vmcnt<0>();
    read(a0, b0, 0);
    landed(a0, b0);
    // one slab: refill the slot whose reads have returned, make sure the next slab is there and request its
    // operands, multiply
    auto slab = [&](int k, float (&a)[C::U], VB (&b)[C::U], float (&an)[C::U], VB (&bn)[C::U]) {
      if (k + C::NS < nk) {
        fetch(k % C::NS);
        wait_vmcnt<(C::NS - 1) * C::L>();
      } else {
        wait_vmcnt<0>();
      }
      if (k == nk - 1 && (valid % C::KS) != 0) {
#pragma unroll
        for (int u = 0; u < C::U; ++u)
          if (k * C::KS + 2 * u + half >= valid) {
            a[u] = 0.f;
            b[u] = VB{};
          }
      }
      // no branch between the reads and their wait: the compiler must not move registers that are in flight
      // (behind the last slab they re-read an old slot, for nothing)
      __builtin_amdgcn_sched_barrier(0);
      read(an, bn, (k + 1) % C::NS);
#pragma unroll
      for (int u = 0; u < C::U; ++u) mma<C>(acc, a[u], b[u]);
      __builtin_amdgcn_sched_barrier(0);
      landed(an, bn);
    };
    for (int k = 0; k < nk; k += 2) {
      slab(k, a0, b0, a1, b1);
      if (k + 1 < nk) slab(k + 1, a1, b1, a0, b0);
    }
  }
  __syncthreads();                                         // the rings become the staging area
  finish_tile<C, MODE>(q, w, acc, staged, wave, lane);
}

template <class C> constexpr bool is_ring = false;
template <int TN, int WK, int NS> constexpr bool is_ring<F32RingCfg<TN, WK, NS>> = true;

template <auto Kern, class C>
int launch_kernel(const TileGrid& q, hipStream_t st) {
  const int err = raise_lds_limit<Kern>(C::LDS_BYTES);
  if (err != 0) return err;
  hipLaunchKernelGGL(Kern, dim3((q.n_items + 7) / 8 * 8), dim3(C::NT), C::LDS_BYTES, st, q);
  return (int)hipGetLastError();
}

template <class C, int MODE>
int launch_mode(const TileGrid& q, hipStream_t st) {
  if constexpr (is_ring<C>) return launch_kernel<&wgrad_f32_ring_kernel<C, MODE>, C>(q, st);
  else return launch_kernel<&wgrad_f32_kernel<C, MODE>, C>(q, st);
}

template <class C>
int launch_cfg(const WgradProblem& p, int mode, const Sinks& s, hipStream_t st) {
  TileGrid q;
  if (!fill_grid<C::BM, C::BN>(q, p, s, C::ROW_STEP) || (int64_t)(q.n_items + 7) / 8 * 8 * C::NT > kMaxLaunchThreads) {
    // more tiles than a launch can count: narrow layers of very many rows (128 Mi rows of up to 32 columns in 32 x 32
    // tiles of 1024 threads) go in pieces
    const int64_t most = countable_run(p.in, p.S, C::BM, C::BN, C::NT);
    if (most >= p.end - p.begin) return (int)hipErrorInvalidValue;
    return in_pieces(p, s, most, [&](const WgradProblem& piece, const Sinks& to) { return launch_cfg<C>(piece, mode, to, st); });
  }
  switch (mode) {
    case EMIT_STORE: return launch_mode<C, EMIT_STORE>(q, st);
    case EMIT_ACCUM: return launch_mode<C, EMIT_ACCUM>(q, st);
    case EMIT_PARTIAL: return launch_mode<C, EMIT_PARTIAL>(q, st);
    default: return launch_mode<C, EMIT_ADAMW>(q, st);
  }
}

// Rows of dY and X in whole 16-byte pieces, and the byte offsets of a slab of 8 tokens in 32 bits.
bool ring_ok(const WgradProblem& p) {
  const auto a16 = [](const void* x) { return (reinterpret_cast<uintptr_t>(x) & 15u) == 0; };
  return p.in % 4 == 0 && p.out % 4 == 0 && p.ldx % 4 == 0 && p.lddy % 4 == 0 && a16(p.X) && a16(p.dY) &&
         p.out + 8 * p.lddy < (int64_t(1) << 30) && p.in + 8 * p.ldx < (int64_t(1) << 30);
}

}  // namespace

// Which kernel and tile (times on 4096 x 4096, 8 Mi elements from mid-row, 1024 tokens, gradient / fused call;
// 112 us are the instructions alone, the scalar-FMA kernel that was here before needed 490 us fused):
//   - 16-byte rows go through the LDS ring, 32 x 64 tiles of four waves (139 / 157 us; 64 x 64 tiles 170 / 184,
//     64 x 128 189 / 213: fewer bytes per flop, but a 34 KB staging area over 24 KB of ring and 69 registers let four
//     workgroups share a compute unit, which evens out the rounds and puts the AdamW stream of one under the
//     loop of another; two slabs of ring are as good as four, for the same reason);
//   - other rows straight to registers, 32 x 128 tiles (200 / 212 us; 64 x 64: 222 / 227, 32 x 64: 367): the
//     vector cache serves 8 - 11 bytes per clock to such loads against 24 to the 16-byte LDS loads, so the
//     lanes' loads must be wide;
//   - when 32 x 64 tiles do not give every compute unit one (768 x 768, 2048 tokens, 50000 elements = 36
//     tiles), 32 x 32 tiles of 8 (ring) or 16 (registers) waves: 13 / 25 us against 24 / 37 us; level at 252
//     tiles (23 against 24 us), slower from 512 (14.5 against 12.9 us).
int launch_wgrad_f32(const WgradProblem& p, int mode, const Sinks& s, void* stream) {
  const hipStream_t st = (hipStream_t)stream;
  const int64_t rows = (p.end - 1) / p.in - p.begin / p.in + 1;
  const bool few = ceil_div(rows, 32) * ceil_div(p.in, 64) * p.S <= device_compute_units();
  if (p.out >= 32 && p.in >= 64 && ring_ok(p))
    return few ? launch_cfg<F32RingCfg<1, 8, 3>>(p, mode, s, st) : launch_cfg<F32RingCfg<2, 4, 2>>(p, mode, s, st);
  if (few || p.in < 128) return launch_cfg<F32Cfg<1, 16>>(p, mode, s, st);
  return launch_cfg<F32Cfg<4, 4>>(p, mode, s, st);
}

}  // namespace chunkft
