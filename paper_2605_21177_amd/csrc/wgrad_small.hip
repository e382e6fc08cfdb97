// bf16 weight gradient in small tiles, for chunks that the large tiles leave most of the compute units
// without work on (takes_small_tiles, shape.cpp, says which and what both sides measured).
//
// Four waves, each a 32 x 32 part of a 64 x 64 tile, slabs of BK tokens in a ring of NS, moved by
// 16-byte LDS loads and taken out by transpose reads as in the kernel with the large tiles, and every element
// is summed over the tokens in the same order as there.  The rows a chunk begins and ends in are part of the
// tiles (masked as they leave) instead of an extra block.
//
// A workgroup alone on its compute unit is a chain of one LDS latency and one barrier per slab (about 400
// cycles for 32 tokens: all steps of a slab are read at once, under the MFMAs of the slab before; read step by
// step it was 480); with four to a compute unit the LDS loads bound it, 27 bytes per clock.  A 128 x 128 tile of 64 x 64
// per wave has half the loads but waits longer per slab: 44 against 27 us for 80 tiles at 4096 tokens.
// A ring of six slabs is slower than four (fewer workgroups per compute unit: 22 against 18 us at 4 Mi).
#include "slab_offset.h"
#include "tiles.h"

namespace chunkft {

namespace {

template <int NS_, int BK_>
struct SmallCfg {
  static constexpr int NS = NS_, BM = 64, BN = 64, BK = BK_, KS = BK / 16, NT = 256;
  static constexpr int IMAGE = BK * BM * 2, SLAB_BYTES = 2 * IMAGE;     // dY image, X image behind it
  static constexpr int LPW = IMAGE / 1024 / 4;                          // 1 KB loads of one image per wave
  static constexpr int SLOTS = BM / 8, TPL = 64 / SLOTS;                // 16-byte slots per token, tokens per load
  static constexpr int PITCH = BN + 4;
  static constexpr size_t STAGE_BYTES = (size_t)BM * PITCH * 4, RING_BYTES = (size_t)NS * SLAB_BYTES;
  static constexpr size_t LDS_BYTES = STAGE_BYTES > RING_BYTES ? STAGE_BYTES : RING_BYTES;
};

// Which 16-byte slot of token k holds logical slot s (64-byte groups XORed so that the four tokens of a
// half-wave's transpose read fall on different banks).
__device__ __forceinline__ int swizzle(int s, int k) { return s ^ (((k >> 1) & 1) << 2); }

template <class C, int MODE>
__global__ __launch_bounds__(C::NT, 2) void wgrad_small_kernel(const TileGrid q) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int item = xcd_work_item(q.n_items);
  if (item < 0) return;
  const WgradProblem& p = q.p;
  const Place w = place_of<C::BM, C::BN>(q, item);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave >> 1, wn = wave & 1;
  const int tokens = (int)(w.k_end - w.k_begin);
  const int nk = (tokens + C::BK - 1) / C::BK;

  // ---- memory -> LDS.  A load is TPL tokens; load j of wave v holds tokens (v * LPW + j) * TPL ...  The source is
  // a scalar base, advanced one slab per fetch, plus a per-lane offset.  Rows and columns past the tensor
  // re-read the tile's first ones, tokens past the end the last one (zeroed in registers).
  const unsigned lda = (unsigned)(p.lddy * 2), ldb = (unsigned)(p.ldx * 2);
  const int tk = lane / C::SLOTS, slot = swizzle(lane % C::SLOTS, tk);
  const int64_t ra = w.row_b + slot * 8, cb = w.col_b + slot * 8;
  const unsigned ca = (unsigned)(ra < p.out ? ra : w.row_b) * 2u, cbo = (unsigned)(cb < p.in ? cb : w.col_b) * 2u;
  const char* ga = (const char*)p.dY + w.k_begin * p.lddy * 2;
  const char* gb = (const char*)p.X + w.k_begin * p.ldx * 2;
  const unsigned base = (unsigned)(uintptr_t)lds;
  int fetched = 0;
  auto to_lds = [&](const char* src, unsigned voff, unsigned soff, unsigned dst) {
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, -1, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (LDS_PTR(void))(uintptr_t)dst, 16, (int)voff, (int)soff, 0, 0);
  };
  auto fetch = [&]() {
    const unsigned dst = base + (unsigned)(fetched % C::NS) * C::SLAB_BYTES;
    const int left = tokens - fetched * C::BK;
#pragma unroll
    for (int j = 0; j < C::LPW; ++j) {
      const int load = wave * C::LPW + j;
      const LoadOffset oa = slab_offset(ca, lda, load * C::TPL, tk, left, C::BK);
      const LoadOffset ob = slab_offset(cbo, ldb, load * C::TPL, tk, left, C::BK);
      to_lds(ga, oa.lane, oa.scalar, dst + load * 1024);
      to_lds(gb, ob.lane, ob.scalar, dst + C::IMAGE + load * 1024);
    }
    ga += (int64_t)C::BK * p.lddy * 2;
    gb += (int64_t)C::BK * p.ldx * 2;
    ++fetched;
  };

  // ---- LDS -> registers (transpose reads; lanes 0-31 tokens 0-7 of a 16-token step, lanes 32-63 tokens 8-15)
  const int blk = lane >> 4, i16 = lane & 15;
  const int tr_k = (blk >> 1) * 8 + (i16 >> 2), low = (blk & 1) * 2 + ((i16 & 3) >> 1), sub = (i16 & 1) * 8;
  const unsigned addr_a = base + tr_k * (C::BM * 2) + (swizzle(wm * 4, tr_k) + low) * 16 + sub;
  const unsigned addr_b = base + C::IMAGE + tr_k * (C::BN * 2) + (swizzle(wn * 4, tr_k) + low) * 16 + sub;
  // the operands of a slab: per 16-token step the tokens +0..3 and +4..7 of the lane's eight
  // (four tokens on, a token's swizzle is the same)
  struct Operands {
    bf16x4 a[2 * C::KS], b[2 * C::KS];
  } r0, r1;
  auto read = [&](Operands& r, int slab) {
    const unsigned so = (unsigned)(slab % C::NS) * C::SLAB_BYTES;
    static_for<C::KS>([&](auto ksc) {
      constexpr int ks = decltype(ksc)::value, u = 2 * ks;
      r.a[u] = lds_tr_read<ks * 16 * C::BM * 2>(addr_a + so);
      r.a[u + 1] = lds_tr_read<(ks * 16 + 4) * C::BM * 2>(addr_a + so);
      r.b[u] = lds_tr_read<ks * 16 * C::BN * 2>(addr_b + so);
      r.b[u + 1] = lds_tr_read<(ks * 16 + 4) * C::BN * 2>(addr_b + so);
    });
  };
  auto landed = [&](Operands& r) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < 2 * C::KS; ++i) asm volatile("" : "+v"(r.a[i]), "+v"(r.b[i])::"memory");   // no use before the wait
  };
  auto mask = [&](Operands& r, int slab) {                               // tokens past the end
    if (slab == nk - 1 && (tokens % C::BK) != 0) {
      const int kv = tokens - slab * C::BK - (lane >> 5) * 8;
#pragma unroll
      for (int u = 0; u < 2 * C::KS; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (u / 2 * 16 + (u & 1) * 4 + e >= kv) {
            r.a[u][e] = (__bf16)0.f;
            r.b[u][e] = (__bf16)0.f;
          }
    }
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  auto multiply = [&](const Operands& r) {
#pragma unroll
    for (int u = 0; u < 2 * C::KS; u += 2)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(r.a[u], r.a[u + 1], 0, 1, 2, 3, 4, 5, 6, 7),
                                                    __builtin_shufflevector(r.b[u], r.b[u + 1], 0, 1, 2, 3, 4, 5, 6, 7), acc, 0, 0, 0);
  };

  // ---- the whole ring in flight; then per slab its one barrier (every wave holds slab kt in registers and has seen
  // its own loads of slab kt + 1 land), the loads of slab kt + NS into the freed slot, the reads of slab kt + 1 under
  // the MFMAs of slab kt.  (The reads behind the last slab take an old slot, for nothing: no branch may lie
  // between a read and its wait.)
  constexpr int L = 2 * C::LPW;
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
    if (s < nk) fetch();
  if (nk >= C::NS) wait_vmcnt<(C::NS - 1) * L>(); else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  read(r0, 0);
  landed(r0);
  auto slab = [&](int kt, Operands& r, Operands& next) {
    mask(r, kt);
    if (kt + C::NS - 1 < nk) wait_vmcnt<(C::NS - 2) * L>(); else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (kt + C::NS < nk) fetch();
    __builtin_amdgcn_sched_barrier(0);
    read(next, kt + 1);
    multiply(r);
    __builtin_amdgcn_sched_barrier(0);
    landed(next);
  };
  for (int kt = 0; kt < nk; kt += 2) {
    slab(kt, r0, r1);
    if (kt + 1 < nk) slab(kt + 1, r1, r0);
  }

  // register v of a wave's block is row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32
  float* const staged = reinterpret_cast<float*>(lds);
  __syncthreads();
  float* const dst = staged + (wm * 32 + (lane >> 5) * 4) * C::PITCH + wn * 32 + (lane & 31);
#pragma unroll
  for (int v = 0; v < 16; ++v) dst[((v >> 2) * 8 + (v & 3)) * C::PITCH] = acc[v];
  __syncthreads();
  emit_rows<MODE, C::BM, C::BN, C::PITCH, C::NT, 1>(q, w, staged, [](int rr) { return rr; });
}

template <class C, int MODE>
int launch_kernel(const TileGrid& q, hipStream_t st) {
  const int err = raise_lds_limit<&wgrad_small_kernel<C, MODE>>(C::LDS_BYTES);
  if (err != 0) return err;
  hipLaunchKernelGGL((wgrad_small_kernel<C, MODE>), dim3((q.n_items + 7) / 8 * 8), dim3(C::NT), C::LDS_BYTES, st, q);
  return (int)hipGetLastError();
}

template <class C>
int launch_cfg(const WgradProblem& p, int mode, const Sinks& s, hipStream_t st) {
  TileGrid q;
  if (!fill_grid<C::BM, C::BN>(q, p, s, 8)) return (int)hipErrorInvalidValue;
  switch (mode) {
    case EMIT_STORE: return launch_kernel<C, EMIT_STORE>(q, st);
    case EMIT_ACCUM: return launch_kernel<C, EMIT_ACCUM>(q, st);
    case EMIT_PARTIAL: return launch_kernel<C, EMIT_PARTIAL>(q, st);
    default: return launch_kernel<C, EMIT_ADAMW>(q, st);
  }
}

}  // namespace

// Slabs of 64 tokens halve the barriers and the chains of a token count; up to 256 tokens the slabs of 32 start sooner
// (fused call, 32- / 64-token slabs: 0.25 Mi elements at 256 tokens 6.9 / 7.5 us, 1 Mi 9.0 / 9.3; 1024 tokens: 0.5 Mi
// 12.3 / 11.6, 1 Mi 16.7 / 15.6; 2048 tokens: 1 Mi 23.9 / 22.1; 4096 tokens: 0.5 Mi in two slabs 25.3 / 23.6).
int launch_wgrad_small(const WgradProblem& p, int mode, const Sinks& s, void* stream) {
  if (p.kslab <= 256) return launch_cfg<SmallCfg<4, 32>>(p, mode, s, (hipStream_t)stream);
  return launch_cfg<SmallCfg<2, 64>>(p, mode, s, (hipStream_t)stream);
}

}  // namespace chunkft
