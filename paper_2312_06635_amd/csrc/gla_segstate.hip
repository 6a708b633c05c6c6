// gla_segstate.hip -- the state-only pass of segmented sequences (bf16): the
// states that each segment adds at the inner boundaries, which gla_segment.hip
// then joins,
//       R <- gamma_n R + Y_n^T Z_n
// with Y = K (.) Gamma, Z = V over the chunks in order, or (reverse) Y = Q (.)
// Lambda, Z = dO backwards.
//
// A workgroup owns 64 value columns of one segment; wave (fw, cw) of its 2 FW
// holds features [fw KP/FW, (fw + 1) KP/FW) x columns 32 cw .. +32 of R as 32x32
// fp32 accumulators (FW = 4 where the width divides, so that two waves per
// SIMD cover each other's LDS reads; else 2).  With no output to form, a chunk is one pass over its Y
// and Z tiles, copied straight into LDS three deep and read with transpose
// reads; gamma's row travels with them (loaded per lane it would take as much
// of the load path as both tiles).  On 4 heads x 16384 steps in 8 segments (d_k
// 256, d_v 512) the pass takes 54 us, with 4 waves 74; running the full pass
// for its states took 92 us forward and 100 us in reverse.
#include "gla_common.hpp"
#include "gla_launch.hpp"

namespace gla {

namespace {

constexpr int kCols = 64;   // value columns per workgroup
constexpr int NB = 3;       // buffers

typedef float f16v __attribute__((ext_vector_type(16)));

struct SegArgs {
  const void *Y, *Z;
  const float *gam;
  const float *R0;  // [BH][K][V] the sequence's initial state (reverse: dS_T), nullable
  float *Rseg;      // [BH][nseg - 1][K][V]
  int BH, T, K, V, C, N, ntiles;
  int nseg, Ns;     // segments per head, chunks per segment
};

template <int KP, int CP> struct SegLayout {
  static constexpr int RBY = KP <= 64 ? 128 : (KP <= 128 ? 256 : 512);  // bytes of a key-tile row
  static constexpr int RBZ = 2 * kCols;
  static constexpr int FW = KP % 128 == 0 ? 4 : 2, threads = 128 * FW;
  static constexpr size_t y = (size_t)CP * RBY, z = (size_t)CP * RBZ, g = 1024;  // (256 features of gamma)
  static constexpr size_t offZ = NB * y, offG = offZ + NB * z, total = offG + NB * g;
};

// Chunk swizzles (16-byte chunks of a row): a 32-lane phase of the transpose
// reads touches 64 bytes of rows r .. r + 3, r a multiple of 8, and the
// swizzles give them disjoint banks.  Only the low four row bits enter, so a
// 16-row step is a plain offset, and 64-byte column steps are XORs.
template <int RB> struct RowSwz {
  static __device__ __forceinline__ int swz(int row) {
    if constexpr (RB >= 256) return ((row & 3) << 2) | ((row >> 2) & 3);
    else return (((row >> 1) & 1) << 2) | (((row >> 3) & 1) << 1);
  }
};

// Lane base of a transposed fragment: lane (g, j), g = l / 32, is to get X[r0 +
// 8g + i][c0 + j]; each transpose read returns, to lane L of a 16-lane block,
// element L % 4 of the 4-vector loaded by lane 4m + L / 4 (m = 0..3).
template <int RB> __device__ __forceinline__ int tr32_base(int x4) {
  const int l = lane_id(), L = l & 15, jh = (l >> 4) & 1, g = l >> 5;
  const int row = 8 * g + (L >> 2) + x4, ch = 2 * jh + ((L & 3) >> 1);
  return row * RB + ((ch ^ RowSwz<RB>::swz(row)) << 4) + 8 * (L & 1);
}
// Fragment at row offset (bytes) rowoff, byte column cb (a multiple of 64).
__device__ __forceinline__ bf16x8 ld_tr(const char *tile, int b0, int b1, int rowoff, int cb) {
  const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(tile + rowoff + (b0 ^ cb)));
  const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(tile + rowoff + (b1 ^ cb)));
  return __builtin_bit_cast(bf16x8, s8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
}

template <int KP, int CP, bool REV>
__global__ void __launch_bounds__((SegLayout<KP, CP>::threads)) segstate_kernel(SegArgs a) {
  using L = SegLayout<KP, CP>;
  constexpr int FW = L::FW, kTh = L::threads;
  constexpr int NFT = KP / (32 * FW);  // 32-feature state tiles per wave
  constexpr int NU = CP / 16;    // 16-row steps of the update
  constexpr int RBY = L::RBY, RBZ = L::RBZ, esz = 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  int id, tile;
  xcd_map(blockIdx.x, a.BH * (a.nseg - 1), a.ntiles, id, tile);
  // (forward every segment but the last, reverse every one but the first)
  const int e = id % (a.nseg - 1);
  const SegMap sm = seg_map(id / (a.nseg - 1), e + (REV ? 1 : 0), a.T, a.C, a.N, a.Ns);
  const int w = wave_id() & (2 * FW - 1), l = lane_id(), cw = w & 1, fw = w >> 1, g2 = l >> 5, j2 = l & 31;
  const int K = a.K, V = a.V, C = a.C, N = sm.N, v0 = tile * kCols, col = v0 + 32 * cw + j2;
  const int64_t KV = (int64_t)K * V;
  auto elem = [&](int i, int r) {  // byte offset of state element r of tile i (past d_k or d_v: out of range)
    const int f = 32 * (fw * NFT + i) + 8 * (r >> 2) + 4 * g2 + (r & 3);
    return f < K && col < V ? (uint32_t)((f * V + col) * 4) : 0x80000000u;
  };

  // the sequence's own initial state at its first segment, else zero
  const float *R0 = a.R0 && sm.seg == (REV ? a.nseg - 1 : 0) ? a.R0 + sm.head * KV : nullptr;
  f16v R[NFT];
  {
    const auto rs = make_rsrc(R0 ? R0 : a.gam, R0 ? (uint32_t)(KV * 4) : 0u);
#pragma unroll
    for (int i = 0; i < NFT; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(rs, elem(i, r), 0, 0);
        R[i][r] = __builtin_bit_cast(float, x);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  const char *Yh = (const char *)a.Y + sm.row0 * K * esz, *Zh = (const char *)a.Z + (sm.row0 * V + v0) * esz;
  const float *Gh = a.gam + sm.chunk0 * K;
  TileDma<CP, RBY, kTh, RowSwz<RBY>> dy;
  TileDma<CP, RBZ, kTh, RowSwz<RBZ>> dz;
  dy.init(w, K * esz, C, K * esz);
  dz.init(w, V * esz, C, (V - v0) * esz);
  const uint32_t lds0 = lds_address(smem);
  constexpr int D = decltype(dy)::NV + decltype(dz)::NV + 1;  // vector memory operations of a wave per chunk
  auto copy_tiles = [&](int it) {  // chunk it (past the last: the last again) into buffer it % NB
    const int n = REV ? N - 1 - min(it, N - 1) : min(it, N - 1), t0 = n * C;
    const uint32_t b = it % NB;
    dy.load(Yh + (int64_t)t0 * K * esz, rsrc_bytes((int64_t)(sm.rows - t0) * K * esz), lds0 + b * (uint32_t)L::y, w);
    dz.load(Zh + (int64_t)t0 * V * esz, rsrc_bytes(((int64_t)(sm.rows - t0) * V - v0) * esz), lds0 + (uint32_t)L::offZ + b * (uint32_t)L::z, w);
    // gamma, by every wave alike (features past d_k: 0)
    const uint64_t base = (uint64_t)(Gh + (int64_t)n * K);
    const u32x4 rs = u32x4{(uint32_t)base, (uint32_t)(base >> 32) & 0xFFFFu, (uint32_t)(K * 4), 0x00020000u};
    const uint32_t m = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)L::offG + b * (uint32_t)L::g);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(m), "v"((uint32_t)l * 16u), "s"(rs) : "m0", "memory");
  };
  const int by0 = tr32_base<RBY>(0), by1 = tr32_base<RBY>(4), bz0 = tr32_base<RBZ>(0), bz1 = tr32_base<RBZ>(4);

#pragma unroll
  for (int p = 0; p < NB - 1; ++p) copy_tiles(p);
  dma_wait<D * (NB - 2)>();
  __syncthreads();
  for (int it = 0; it < N; ++it) {
    const int b = it % NB;
    const char *sY = smem + b * L::y, *sZ = smem + L::offZ + b * L::z;
    const float *sG = (const float *)(smem + L::offG + b * L::g) + 32 * fw * NFT + 4 * g2;
    copy_tiles(it + NB - 1);  // (its buffer was last read before the previous barrier)
#pragma unroll
    for (int i = 0; i < NFT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 x = *(const f4 *)(sG + 32 * i + 8 * q);
#pragma unroll
        for (int r = 0; r < 4; ++r) R[i][4 * q + r] *= x[r];
      }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const bf16x8 z = ld_tr(sZ, bz0, bz1, 16 * u * RBZ, 64 * cw);
#pragma unroll
      for (int i = 0; i < NFT; ++i)
        R[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_tr(sY, by0, by1, 16 * u * RBY, 64 * (fw * NFT + i)), z, R[i], 0, 0, 0);
    }
    // the next chunk's tiles have landed: only later chunks' copies are younger
    dma_wait<D * (NB - 2)>();
    __syncthreads();
  }
  dma_wait();  // (no copy outlives the workgroup's LDS)

  const auto rs = make_rsrc(a.Rseg + ((int64_t)sm.head * (a.nseg - 1) + e) * KV, (uint32_t)(KV * 4));
#pragma unroll
  for (int i = 0; i < NFT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = R[i][r];
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), rs, elem(i, r), 0, 0);
    }
}

template <int KP, int CP, bool REV> hipError_t launch_sp(const SegArgs &a, hipStream_t st) {
  // once per instantiation (thread-safe static initialisation), at the maximum
  static const hipError_t attr = hipFuncSetAttribute((const void *)segstate_kernel<KP, CP, REV>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
  (void)attr;
  const size_t lds = SegLayout<KP, CP>::total;
  const int threads = SegLayout<KP, CP>::threads;
  hipLaunchKernelGGL((segstate_kernel<KP, CP, REV>), dim3(a.BH * (a.nseg - 1) * a.ntiles),
                     dim3(threads), lds, st, a);
  return hipGetLastError();
}

template <bool REV> hipError_t dispatch_sp(const Shape &s, const SegArgs &a, hipStream_t st) {
  const int KP = (s.K + 63) / 64 * 64;
#define GLA_SP_CASE(kp) \
  if (KP == kp) return s.C <= 32 ? launch_sp<kp, 32, REV>(a, st) : launch_sp<kp, 64, REV>(a, st);
  GLA_SP_CASE(64) GLA_SP_CASE(128) GLA_SP_CASE(192) GLA_SP_CASE(256)
#undef GLA_SP_CASE
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_seg_pass(const Shape &s, const Segs &sg, bool rev, const void *z, const float *R0, const Work &w,
                           hipStream_t st) {
  SegArgs a{};
  a.BH = s.BH; a.T = s.T; a.K = s.K; a.V = s.V; a.C = s.C; a.N = s.N;
  a.ntiles = (s.V + kCols - 1) / kCols;
  a.nseg = sg.n; a.Ns = sg.Ns;
  a.Y = rev ? w.Qt : w.Kt;
  a.Z = z; a.gam = w.gam; a.R0 = R0; a.Rseg = rev ? w.dSseg : w.Sseg;
  return rev ? dispatch_sp<true>(s, a, st) : dispatch_sp<false>(s, a, st);
}

}  // namespace gla
