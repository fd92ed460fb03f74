// bf16 MFMA GEMMs of the Llama projections on gfx950 (v_mfma_f32_16x16x32_bf16,
// fp32 accumulation):  Y[M, N] = X[M, K] . W[N, K]^T  + fused epilogue.
//
// Operand convention.  The MFMA computes D = A . B with A 16x32 (rows = output
// features n, i.e. W rows) and B 32x16 (columns = activation rows m).  Lane l
// supplies A[l%16][8(l/16) .. 8(l/16)+7] and B[8(l/16) .. +7][l%16] and
// receives D[4(l/16) + i][l%16], i = 0..3: four consecutive output features of
// one activation row, so every epilogue store is a contiguous 16-byte (fp32)
// or 8-byte (bf16) vector.
//
// W is stored in exactly that A-operand order (packed_offset in common.h): a
// 16 x 32 tile of W is 1 KiB, lane l's 16 bytes at offset 16l, so a wave
// loading an A operand from HBM issues one contiguous 1 KiB read.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace metro {

__device__ __forceinline__ f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

__device__ __forceinline__ float silu_f32(float z) { return z / (1.0f + expf(-z)); }

// Epilogue for one 16x16 accumulator tile: lane holds features n .. n+3 of row m.
template <int EPI>
__device__ __forceinline__ void store_tile(f32x4 v, int m, int n, float* __restrict__ outf, int ldo) {
  float4* p = reinterpret_cast<float4*>(outf + static_cast<size_t>(m) * ldo + n);
  if (EPI == kEpiStoreF32) {
    *p = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    float4 o = *p;
    o.x += v[0];
    o.y += v[1];
    o.z += v[2];
    o.w += v[3];
    *p = o;
  }
}

// gate/up tiles of the same 16 features -> bf16(silu(gate) * up)
__device__ __forceinline__ void store_swiglu(f32x4 gt, f32x4 up, int m, int j, uint16_t* __restrict__ outb,
                                             int ldo) {
  uint2 o;
  o.x = pack_bf16x2(silu_f32(gt[0]) * up[0], silu_f32(gt[1]) * up[1]);
  o.y = pack_bf16x2(silu_f32(gt[2]) * up[2], silu_f32(gt[3]) * up[3]);
  *reinterpret_cast<uint2*>(outb + static_cast<size_t>(m) * ldo + j) = o;
}

// ---------------------------------------------------------------------------
// Skinny GEMM (M <= 16*MT, decode batches).  Streaming W from HBM is the cost,
// and every W row tile needs the activation rows of its k range, so each wave
// owns NT row tiles (16*NT rows of W) to keep those activation reads well
// below the W bytes.  A workgroup of NW waves owns the 16*NT rows and a k
// slice (grid.y = KS slices); wave w takes the 128-wide k blocks w, w+NW, ...
// of the slice.  A block is 4 packed 16 x 32 tiles per row tile, i.e. 4 KiB
// contiguous in W, read as four 1 KiB wave loads.
// Partial tiles of the NW waves are summed through LDS in wave order; with
// KS > 1 the slice sums go to part[slice][m][n] and the consumer kernel adds
// the slices (in slice order) where it reads the result.
// ---------------------------------------------------------------------------
// Where the QKV epilogue stores one row: its q, its KV page and its key there.
struct RowOut {
  uint16_t *q, *page;
  int key;
};
__device__ __forceinline__ RowOut row_out(int m, int slot, const RopeKV& rk) {
  return {rk.q + static_cast<size_t>(m) * (rk.nq * rk.hd), rk.kv + kv_offset(slot / kPage, 0, rk.nkv, 0, 0, rk.hd, 0),
          slot % kPage};
}

// q / k / v of one row for dims d0 .. d0+3 (a; d0 % 4 == 0) and d0+half .. (b) of
// a head; c: cos and sin of dims d0 .. d0+3 at its position (not read for v).
// In a K tile the 4 dims are consecutive elements, in a V^T tile 16 bytes apart;
// half (a multiple of 32) dims on is 16 * half elements on in both.
__device__ __forceinline__ void store_rope_kv(f32x4 a, f32x4 b, const float4 (&c)[2], const RowOut& o, int head, int d0,
                                              const RopeKV& rk) {
  const int hd = rk.hd, half = hd / 2;
  if (head < rk.nq + rk.nkv) {
    const float cs[8] = {c[0].x, c[0].y, c[0].z, c[0].w, c[1].x, c[1].y, c[1].z, c[1].w};
    f32x4 ra, rb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // (which product is rounded is fixed, so that every kernel gives the same bits)
      ra[i] = fmaf(a[i], cs[2 * i], -(b[i] * cs[2 * i + 1]));
      rb[i] = fmaf(b[i], cs[2 * i], a[i] * cs[2 * i + 1]);
    }
    const bool q = head < rk.nq;
    uint16_t* dst = q ? o.q + head * hd + d0 : o.page + (head - rk.nq) * (kPage * hd) + k_tile_offset(o.key, d0);
    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(ra[0], ra[1]), pack_bf16x2(ra[2], ra[3]));
    *reinterpret_cast<uint2*>(dst + (q ? half : 16 * half)) =
        make_uint2(pack_bf16x2(rb[0], rb[1]), pack_bf16x2(rb[2], rb[3]));
  } else {
    uint16_t* dst = o.page + (head - rk.nq) * (kPage * hd) + vt_tile_offset(d0, o.key);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dst[8 * i] = f32_to_bf16(a[i]);
      dst[16 * half + 8 * i] = f32_to_bf16(b[i]);
    }
  }
}

// cos and sin of dims d0 .. d0+3 (d0 % 4 == 0) at a position
__device__ __forceinline__ void load_rope(float4 (&c)[2], int pos, int d0, const RopeKV& rk) {
  const float4* p = reinterpret_cast<const float4*>(rk.rope + static_cast<size_t>(pos) * (rk.hd / 2) + d0);
  c[0] = p[0];
  c[1] = p[1];
}

template <int MT, int NT, int EPI, int PF, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_skinny_kernel(const uint16_t* __restrict__ X, int ldx,
                                                              const uint16_t* __restrict__ W, int Kp, int M, int N,
                                                              float* __restrict__ outf, uint16_t* __restrict__ outb,
                                                              int ldo, float* __restrict__ part, RopeKV rk) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16 * NT;
  const int KS = gridDim.y, slice = blockIdx.y;
  const int kslice = Kp / KS, k0 = slice * kslice;

  f32x4 acc[NT][MT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // packed tile (n0/16 + nt, k0/32) of W, this lane's chunk
  const uint16_t* wrow[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    wrow[nt] = W + (static_cast<size_t>(n0 / 16 + nt) * (Kp / 32) + k0 / 32) * 512 + lane * 8;
  const uint16_t* xrow[MT];
  bool xok[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = mt * 16 + r;
    xok[mt] = m < M;
    xrow[mt] = X + static_cast<size_t>(xok[mt] ? m : 0) * ldx + k0 + 8 * g;
  }

  // the wave's k blocks are wave, wave + NW, ...; PF of them are in flight in a
  // register ring whose slots are refilled right after use (clamped, so every
  // load is unconditional and each block waits only for its own loads)
  const int nkb = kslice / 128;
  const int nb = wave < nkb ? (nkb - wave + NW - 1) / NW : 0;
  if (nb > 0) {
    uint4 wv[PF][NT][4], xv[PF][MT][4];
    auto load = [&](int sl, int j) {
      const int k = (wave + NW * j) * 128;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) wv[sl][nt][i] = *reinterpret_cast<const uint4*>(wrow[nt] + (k / 32 + i) * 512);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          xv[sl][mt][i] = xok[mt] ? *reinterpret_cast<const uint4*>(xrow[mt] + k + 32 * i) : make_uint4(0, 0, 0, 0);
    };
#pragma unroll
    for (int sl = 0; sl < PF; ++sl) load(sl, min(sl, nb - 1));
    for (int base = 0; base < nb; base += PF) {
#pragma unroll
      for (int sl = 0; sl < PF; ++sl) {
        const int it = base + sl;
        if (it < nb) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = mfma16(wv[sl][nt][i], xv[sl][mt][i], acc[nt][mt]);
        }
        if (PF > 1) load(sl, min(it + PF, nb - 1));
        else if (it + 1 < nb) load(sl, it + 1);
      }
    }
  }

  __shared__ f32x4 red[NW][NT * MT][kWave];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[wave][nt * MT + mt][lane] = acc[nt][mt];
  __syncthreads();

  const int m_lane = r;  // activation row within a 16-row tile
  const int n_lane = 4 * g;
  if (EPI == kEpiSwiGLU) {
    // Tile nt holds the gate (rows 0..7) and up (rows 8..15) projections of
    // features 8 (n0/16 + nt) .. +7: lane l < 32 has gate rows 4(l/16) .. +3
    // and lane l + 32 the matching up rows, which a 32-lane swap brings together.
    for (int t = wave; t < NT * MT; t += NW) {
      f32x4 sum = red[0][t][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += red[w][t][lane];
      f32x4 gt, up;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i]), __float_as_uint(sum[i]), false, false);
        gt[i] = __uint_as_float(pr[0]);  // from lane l % 32
        up[i] = __uint_as_float(pr[1]);  // from lane l % 32 + 32
      }
      const int nt = t / MT, mt = t % MT;
      const int m = mt * 16 + m_lane;
      if (lane < 32 && m < M) store_swiglu(gt, up, m, 8 * (n0 / 16 + nt) + n_lane, outb, ldo);
    }
  } else if (EPI == kEpiRopeKV) {
    // Tile nt holds dims 8j .. 8j+7 (rows 0..7) and the matching dims of the
    // head's second half (rows 8..15) of one head, j = its 16-row tile within
    // the head: as for SwiGLU, a 32-lane swap brings each pair together.
    for (int t = wave; t < NT * MT; t += NW) {
      f32x4 sum = red[0][t][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += red[w][t][lane];
      f32x4 a, b;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i]), __float_as_uint(sum[i]), false, false);
        a[i] = __uint_as_float(pr[0]);  // dim d (lane l % 32)
        b[i] = __uint_as_float(pr[1]);  // dim d + hd/2 (lane l % 32 + 32)
      }
      const int nt = t / MT, mt = t % MT;
      const int m = mt * 16 + m_lane;
      const int f0 = n0 + nt * 16, head = f0 / rk.hd, d0 = 8 * ((f0 % rk.hd) / 16) + n_lane;
      if (lane < 32 && m < M) {
        float4 c[2];
        if (head < rk.nq + rk.nkv) load_rope(c, rk.pos[m], d0, rk);
        store_rope_kv(a, b, c, row_out(m, rk.slot[m], rk), head, d0, rk);
      }
    }
  } else {
    for (int t = wave; t < NT * MT; t += NW) {
      f32x4 sum = red[0][t][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += red[w][t][lane];
      const int nt = t / MT, mt = t % MT;
      const int m = mt * 16 + m_lane;
      if (m >= M) continue;
      if (KS > 1)
        store_tile<kEpiStoreF32>(sum, m, n0 + nt * 16 + n_lane, part + static_cast<size_t>(slice) * M * N, N);
      else
        store_tile<EPI>(sum, m, n0 + nt * 16 + n_lane, outf, ldo);
    }
  }
}

// out[m, n] (=|+=) sum over slices of part[s][m][n], in slice order
template <int EPI>
__global__ __launch_bounds__(256) void reduce_parts_kernel(const float* __restrict__ part, int KS, int M, int N,
                                                           float* __restrict__ out, int ldo) {
  const int64_t n4 = static_cast<int64_t>(M) * N / 4;
  for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < n4; e += static_cast<int64_t>(gridDim.x) * 256) {
    const int m = static_cast<int>((4 * e) / N), n = static_cast<int>((4 * e) % N);
    float4 s = reinterpret_cast<const float4*>(part)[e];
    for (int k = 1; k < KS; ++k) {
      const float4 v = reinterpret_cast<const float4*>(part + static_cast<size_t>(k) * M * N)[e];
      s.x += v.x;
      s.y += v.y;
      s.z += v.z;
      s.w += v.w;
    }
    float4* o = reinterpret_cast<float4*>(out + static_cast<size_t>(m) * ldo + n);
    if (EPI == kEpiAddF32) {
      const float4 x = *o;
      s.x += x.x;
      s.y += x.y;
      s.z += x.z;
      s.w += x.w;
    }
    *o = s;
  }
}

// ---------------------------------------------------------------------------
// Tiled GEMM of 4 waves, one per SIMD (2 x 2, each 16 TN rows of W x 16 TM
// activation rows of v_mfma_f32_16x16x32_bf16), for more than 32 rows.
//
// What bounds it: for prefill chunks the chip's power limit, which it reaches
// with random operands, so the energy per flop counts as much as the stalls;
// for batches of up to about 256 rows the stream of W.
//  - 16x16x32 instead of 32x32x16 MFMAs: the accumulators are read and written
//    half as often (a loop of nothing but MFMAs on random data: 2125 against
//    1862 TFLOP/s).
//  - 128 x 128 per wave: 128 KiB of LDS reads per 64-wide k step of a 256 x 256
//    tile, against 192 KiB for 8 waves of 64 x 128.
//  - a wave alone on its SIMD has nobody to cover its stalls: each memory
//    instruction rides behind an MFMA, fragments are read one chunk ahead, and
//    operands are requested two to three chunks ahead.
// Ring: 4 chunks of 32-wide k for W (operand order, copied as is), 3 stages of
// 64-wide k for X (whole cache lines; row r keeps its 16-byte chunk c in slot
// c ^ r % 8, which keeps the fragment reads free of bank conflicts); for
// 256 x 256 tiles all 160 KiB.  Chunk c: its MFMAs, the fragments of c + 1, the
// requests of W chunk c + 4 into the slot just freed and of half an X stage,
// then a barrier (chunk c + 2 has landed, c + 1 is in registers everywhere).
// Measured, 8 waves of 64 x 128 with 32x32x16 MFMAs before: 8B gate/up at
// M = 8192 1634 -> 1352 us (1424 TFLOP/s), down 822 -> 649 us (1482), QKV 358
// -> 289 us, 70B gate/up 6281 -> 5062 us (1520).
// ---------------------------------------------------------------------------
template <int TN_, int TM_>
struct TileShape {
  static constexpr int TN = TN_, TM = TM_;  // 16 x 16 tiles per wave
  static constexpr int NTH = 256, BN = 32 * TN, BM = 32 * TM;
  static constexpr int WS = 4, XS = 3;
  static constexpr int LW = TN / 2;                     // W loads per wave and chunk
  static constexpr int LX0 = TM / 2, LX1 = TM - LX0;    // X loads per wave: first, second half of a stage
  static constexpr int kLds = WS * BN * 4 + XS * BM * 8;  // 16-byte units
  static constexpr int OCC = kLds * 16 <= 80 * 1024 ? 2 : 1;  // workgroups per CU that its registers must allow
  static_assert(TN % 4 == 0 && TM >= 2, "the waves share each chunk evenly");
};

// Big: for prefill chunks.  Mid: for batches of 65 to a few hundred rows; 80
// KiB of LDS, so two workgroups share a CU where there are enough.  Wide: for
// wide products at up to 256 rows when 128 x 128 tiles would be too many for
// one round: against 256 x 256 tiles it does no matrix work on absent rows at
// M <= 128 and gives twice the workgroups at M = 129..256.  Against the former
// 8-wave kernels of these tile sizes (32x32x16 MFMAs): 8B gate/up at M = 128 /
// 200 / 256 50.8 / 75.2 / 83.1 -> 49.6 / 63.8 / 68.0 us, down at M = 200 45.3 ->
// 42.2, O at M = 800 41.1 -> 36.6; 70B gate/up at M = 128 194 -> 172, QKV 56.5
// -> 47.3; 70B down and QKV at M = 129 .. 384 from 2% slower to 9% faster.
using BigTile = TileShape<8, 8>;
using MidTile = TileShape<4, 4>;
using WideTile = TileShape<8, 4>;
// Small: 33 to 64 rows.  The decode kernel's waves each read the activations of
// their k blocks from L2, at 64 rows as many bytes as the weights; here the
// four waves share them through LDS.  Us at M = 40 / 64, decode kernel -> this:
// 8B QKV 21.8 / 26.0 -> 16.2 / 16.7, O 15.8 / 18.7 -> 13.6 / 14.5, gate/up 47.9 /
// 49.3 -> 43.3 / 43.6, down 30.6 / 34.3 -> 27.6 / 28.0, LM head 213 / 240 -> 195 /
// 207; 70B QKV 51.9 / 60.4 -> 40.3 / 41.9.  At 25 and 32 rows the two are within
// 4% (8B O 12.4 against 12.9), and the decode kernel keeps those, as it does the
// products that leave these tiles too few (small_tile_splits).
using SmallTile = TileShape<4, 2>;

// Grouped tile order: consecutive tiles sweep groups of GM m-tiles, m fastest
// within a group, so that the blocks in flight cover a compact patch of tiles
// and share their W and X tiles through the caches.  256-row tiles are visited
// in groups of 4 (32 consecutive 256 x 256 tiles, the CUs of one XCD, cover 4 x
// 8); all others, and the tiles of a last round that is cut in k slices, are
// counted in groups of 16.
constexpr int kTailGroupM = 16;
template <class S>
constexpr int kGroupM = S::TN * S::TM > 32 ? 4 : kTailGroupM;

template <class S, int GM>
__device__ __forceinline__ void tile_origin(int t, int M, int N, int& m0, int& n0) {
  const int mt = (M + S::BM - 1) / S::BM, nt = (N + S::BN - 1) / S::BN;
  const int group = t / (GM * nt);
  const int first_m = group * GM;
  const int gm = min(mt - first_m, GM);
  const int in = t % (GM * nt);
  n0 = (in / gm) * S::BN;
  m0 = (first_m + in % gm) * S::BM;
}

// Tile t of the first `full` tiles in the order of groups of 16, visited in the
// kernel's own order.  Which tiles the last round cuts in k slices decides how
// their fp32 sums are grouped, so that set does not follow the order in which
// the others are visited.  A whole group of 16 holds four whole groups of 4; of
// the group that the last round cuts, the first rows may have one column more.
template <class S>
__device__ __forceinline__ void full_tile_origin(int t, int full, int M, int N, int& m0, int& n0) {
  constexpr int GM = kGroupM<S>;
  const int mt = (M + S::BM - 1) / S::BM, nt = (N + S::BN - 1) / S::BN;
  const int whole = full / (kTailGroupM * nt), first = whole * kTailGroupM * nt;
  if (GM == kTailGroupM || t < first) {
    tile_origin<S, GM>(t, M, N, m0, n0);
    return;
  }
  const int h = min(mt - whole * kTailGroupM, kTailGroupM);
  const int cols = (full - first) / h, more = (full - first) % h;
  t -= first;
  int r = 0, gm = min(h, GM);
  for (;;) {
    const int n = gm * cols + min(max(more - r, 0), gm);
    if (t < n || r + gm >= h) break;
    t -= n;
    r += gm;
    gm = min(h - r, GM);
  }
  n0 = (t / gm) * S::BN;
  m0 = (whole * kTailGroupM + r + t % gm) * S::BM;
}

// Workgroups are handed to the 8 XCDs in turn (workgroup b to XCD b % 8), and
// each XCD has its own L2.  Work item of workgroup b (of `total`) such that
// every XCD gets a contiguous run of the work list: in tile_origin order the
// row tiles that read the same W columns are neighbours, so they run on one
// XCD and share its L2 instead of each fetching W through the fabric.  In the
// model (agent trace, 8B, with 8-wave 128 x 128 tiles) this gained 2.5%.
__device__ __forceinline__ int xcd_contiguous(int b, int total) {
  constexpr int kXcds = 8;
  const int q = total / kXcds, r = total % kXcds, x = b % kXcds, s = b / kXcds;
  return x * q + min(x, r) + s;
}

// c += a . b with the accumulator held in place in AGPRs: 64 of these fill the
// AGPR half of the register file, and left to itself the compiler's register
// allocation moves them about inside the loop (430 moves per 128 MFMAs).  The
// compiler does not see these MFMAs' hazards: an accumulator is touched once
// per chunk, and no chunk ends without drained_barrier, behind which the
// accumulators may be read (tests/test_gemm_accumulators.py checks the code).
__device__ __forceinline__ void mfma16_acc(f32x4& c, uint4 a, uint4 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(as_bf16x8(a)), "v"(as_bf16x8(b)));
}
// The same with a direct load into LDS bytes lds_base + INC + 16 * lane behind
// it; the MFMA is the wait state between the M0 write and the load.
template <int INC>
__device__ __forceinline__ void mfma16_acc_load(f32x4& c, uint4 a, uint4 b, const void* base, uint32_t off,
                                                uint32_t lds_base) {
  asm volatile(
      "s_add_u32 m0, %3, %4\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %5, %6"
      : "+a"(c)
      : "v"(as_bf16x8(a)), "v"(as_bf16x8(b)), "s"(lds_base), "n"(INC), "v"(off), "s"(base)
      : "memory", "m0", "scc");
}
// All of the wave's LDS reads are in, its last MFMA has left its accumulator
// readable (8 wait states), and every other wave is as far.
__device__ __forceinline__ void drained_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 7\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Epilogues go through the wave's share of LDS, 32 activation rows at a time,
// so that global accesses cover whole cache lines (the accumulators hold 4
// columns of 16 rows each).  Row r keeps its 16-byte chunk c in slot c ^ r.
//
// fp32: 2 or 4 whole rows of the wave's columns per access; the residual of
// the next 32 rows is loaded meanwhile.
template <class S, int EPI>
__device__ __forceinline__ void tile_epilogue_f32(const f32x4 (&acc)[S::TN][S::TM], uint4* buf, int mw, int nw, int m0,
                                                  int n0, int lane, int M, int N, int KS, int slice, int unit,
                                                  float* __restrict__ outf, int ldo, float* __restrict__ part) {
  constexpr int TN = S::TN, TM = S::TM, CH = 4 * TN;  // 16-byte chunks per row
  constexpr int RPI = 64 / CH, NI = 32 / RPI;         // rows per access, accesses per 32 rows
  const int r16 = lane & 15, g = lane >> 4;
  const int col = lane % CH, sub = lane / CH;
  const bool raw = KS > 1;
  float* out = outf;
  int ld = ldo, mb = mw, nb = nw + 4 * col;
  const bool nok = nb < N;
  const int mok = min(M - mw, 16 * TM);  // rows of the wave's tile
  nb = min(nb, N - 4);
  if (unit >= 0) {
    out = part + static_cast<size_t>(unit) * S::BM * S::BN;
    ld = S::BN;
    mb -= m0;
    nb -= n0;
  } else if (raw) {
    out = part + static_cast<size_t>(slice) * M * N;
    ld = N;
  }
  float* const base = out + static_cast<size_t>(mb) * ld + nb;
  const bool add = EPI == kEpiAddF32 && !raw;
  float4 res[2][NI];
  auto load_res = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NI; ++t)
      res[q & 1][t] =
          *reinterpret_cast<const float4*>(base + static_cast<ptrdiff_t>(min(32 * q + RPI * t + sub, mok - 1)) * ld);
  };
  if (EPI == kEpiAddF32) {
    if (add) load_res(0);
  }
#pragma unroll
  for (int q = 0; q < (TM + 1) / 2; ++q) {
#pragma unroll
    for (int j = 0; j < 2 && 2 * q + j < TM; ++j)
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int r = 16 * j + r16;
        buf[r * CH + ((4 * i + g) ^ (r % CH))] = __builtin_bit_cast(uint4, acc[i][2 * q + j]);
      }
    if (EPI == kEpiAddF32) {
      if (add && 2 * q + 2 < TM) load_res(q + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < (2 * q + 1 < TM ? NI : NI / 2); ++t) {
      const int r = RPI * t + sub;
      float4 v = __builtin_bit_cast(float4, buf[r * CH + (col ^ (r % CH))]);
      if (EPI == kEpiAddF32) {
        if (add) {
          v.x += res[q & 1][t].x;
          v.y += res[q & 1][t].y;
          v.z += res[q & 1][t].z;
          v.w += res[q & 1][t].w;
        }
      }
      if (nok && 32 * q + r < mok) *reinterpret_cast<float4*>(base + static_cast<size_t>(32 * q + r) * ld) = v;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The halves of two 16-row blocks of W brought together: lanes 0-31 get rows
// 0-7 (lo) and the matching rows 8-15 (hi) of block x, lanes 32-63 of block y.
__device__ __forceinline__ void pair_halves(f32x4 x, f32x4 y, f32x4& lo, f32x4& hi) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[r]), __float_as_uint(y[r]), false, false);
    lo[r] = __uint_as_float(p[0]);
    hi[r] = __uint_as_float(p[1]);
  }
}

// SwiGLU: the wave's 8 TN outputs per row (16 TN bytes)
template <class S>
__device__ __forceinline__ void tile_epilogue_swiglu(const f32x4 (&acc)[S::TN][S::TM], uint4* buf, int mw, int nw,
                                                     int lane, int M, int N, uint16_t* __restrict__ outb, int ldo) {
  constexpr int TN = S::TN, TM = S::TM, CH = TN;  // 16-byte chunks per row
  constexpr int RPI = 64 / CH, NI = 32 / RPI;
  const int r16 = lane & 15, g = lane >> 4;
  const int col = lane % CH, sub = lane / CH;
  uint2* const buf8 = reinterpret_cast<uint2*>(buf);
  const bool nok = nw + 16 * col < N;
#pragma unroll
  for (int q = 0; q < (TM + 1) / 2; ++q) {
#pragma unroll
    for (int j = 0; j < 2 && 2 * q + j < TM; ++j)
#pragma unroll
      for (int i = 0; i < TN; i += 2) {
        f32x4 gt, up;
        pair_halves(acc[i][2 * q + j], acc[i + 1][2 * q + j], gt, up);
        const int r = 16 * j + r16, c = i + (g >> 1);
        uint2 o;
        o.x = pack_bf16x2(silu_f32(gt[0]) * up[0], silu_f32(gt[1]) * up[1]);
        o.y = pack_bf16x2(silu_f32(gt[2]) * up[2], silu_f32(gt[3]) * up[3]);
        buf8[(r * CH + (c ^ (r % CH))) * 2 + (g & 1)] = o;
        __builtin_amdgcn_sched_barrier(0);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < (2 * q + 1 < TM ? NI : NI / 2); ++t) {
      const int r = RPI * t + sub, m = mw + 32 * q + r;
      const uint4 v = buf[r * CH + (col ^ (r % CH))];
      if (nok && m < M) {
        uint2* p = reinterpret_cast<uint2*>(outb + static_cast<size_t>(m) * ldo + nw / 2 + 8 * col);
        p[0] = make_uint2(v.x, v.y);  // (rows of the output are 8-byte aligned)
        p[1] = make_uint2(v.z, v.w);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// RoPE and the KV cache write.  A 16-row block of W holds 8 dims of a head's
// first half, then the matching 8 of its second half (rotate-half interleave),
// so two neighbouring blocks, which are of one head, are paired like gate and up.
// A wave has nobody to cover its waits here, and each pair's rotation hangs on two
// dependent loads (position, cos and sin): all slots and positions are loaded at
// once, and the cos and sin of 16 rows while the 16 before them are stored.
// (One pair at a time, loads and all, before -> now, us of the whole product at
// 2000 rows: K 256, N 512 33.6 -> 25.6; K 1024, N 1536 54.9 -> 39.6; K 4096, N
// 6144 107 -> 95.)
template <class S>
__device__ __forceinline__ void tile_epilogue_rope_kv(const f32x4 (&acc)[S::TN][S::TM], int mw, int nw, int lane, int M,
                                                      int N, const RopeKV& rk) {
  constexpr int TM = S::TM, NP = S::TN / 2;
  const int r16 = lane & 15, g = lane >> 4;
  int slot[TM], pos[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = min(mw + 16 * j + r16, M - 1);
    slot[j] = rk.slot[m];
    pos[j] = rk.pos[m];
  }
  float4 c[2][NP][2];
  // pair p: its head, and this lane's first dim
  const int shift = 31 - __builtin_clz(rk.hd);  // (head dims are powers of two)
  auto head = [&](int p) __attribute__((always_inline)) { return (nw + 32 * p) >> shift; };
  auto dim = [&](int p) __attribute__((always_inline)) {
    return 8 * (((nw + 32 * p) & (rk.hd - 1)) / 16 + (g >> 1)) + 4 * (g & 1);
  };
  auto load = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (nw + 32 * p < N && head(p) < rk.nq + rk.nkv) load_rope(c[j & 1][p], pos[j], dim(p), rk);
  };
  load(0);
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    if (j + 1 < TM) load(j + 1);
    __builtin_amdgcn_sched_barrier(0);
    const int m = mw + 16 * j + r16;
    const RowOut o = row_out(m, slot[j], rk);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      f32x4 x, y;
      pair_halves(acc[2 * p][j], acc[2 * p + 1][j], x, y);
      if (m < M && nw + 32 * p < N) store_rope_kv(x, y, c[j & 1][p], o, head(p), dim(p), rk);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// index of the direct load that rides behind MFMA u of nm (nd of them spread
// evenly behind odd MFMAs), nd if none
constexpr int load_behind(int u, int nm, int nd) {
  for (int l = 0; l < nd; ++l)
    if ((l * nm / nd | 1) == u) return l;
  return nd;
}

// Work of one workgroup.  Without a tail split the grid's tiles x k slices
// (slice-major list, tiles in tile_origin order) are spread over the XCDs by
// xcd_contiguous.  With one (tail_split = S > 1), the last tiles in the order of
// groups of 16, which would leave most CUs idle in the final round, are cut into
// S k slices each: workgroup tail_first + u takes slice u % S of tile tail_first
// + u / S and stores its fp32 sums to part[u][BM][BN] for
// gemm_tail_fixup_kernel; workgroups x < tail_first take the other tiles over
// all of K.
// In tile_origin order 32 consecutive 256 x 256 tiles (one XCD's CUs) cover 4 x
// 8 of them, so an XCD's L2 fetches 12 operand tiles per k step; the list in
// grid order made that 18 (8B gate/up at M = 8192 1506 -> 1479 us).
template <class S, int EPI>
__global__ __launch_bounds__(S::NTH, S::OCC) void gemm_tiled_kernel(const uint16_t* __restrict__ X, int ldx,
                                                              const uint16_t* __restrict__ W, int Kp, int M, int N,
                                                              float* __restrict__ outf, uint16_t* __restrict__ outb,
                                                              int ldo, float* __restrict__ part, int tail_first,
                                                              int tail_split, RopeKV rk) {
  constexpr int TN = S::TN, TM = S::TM, WS = S::WS, LW = S::LW, LX0 = S::LX0, LX1 = S::LX1;
  __shared__ uint4 lds[S::kLds];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave >> 1, wm = wave & 1;
  const int r16 = lane & 15, g = lane >> 4;

  int KS = gridDim.y, slice = blockIdx.y, unit = -1;
  int m0, n0;
  if (tail_split > 1 && static_cast<int>(blockIdx.x) >= tail_first) {
    unit = blockIdx.x - tail_first;
    KS = tail_split;
    slice = unit % tail_split;
    tile_origin<S, kTailGroupM>(tail_first + unit / tail_split, M, N, m0, n0);
  } else if (tail_split > 1) {
    full_tile_origin<S>(xcd_contiguous(blockIdx.x, tail_first), tail_first, M, N, m0, n0);
  } else {
    const int i = xcd_contiguous(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    slice = i / gridDim.x;
    tile_origin<S, kGroupM<S>>(i % gridDim.x, M, N, m0, n0);
  }
  const int kspan = Kp / KS, k0 = slice * kspan;
  const int nc = kspan / 32;  // chunks (a multiple of 4)

  // The wave's share of every W chunk (16-row tiles) and X stage (blocks of 8
  // rows).  Rows past N or M re-read the last valid row: finite values whose
  // products only reach outputs that are not stored.
  const char* const wbase =
      reinterpret_cast<const char*>(W + (static_cast<size_t>(n0 / 16) * (Kp / 32) + k0 / 32) * 512);
  const char* const xbase = reinterpret_cast<const char*>(X + static_cast<size_t>(m0) * ldx + k0);
  uint32_t woff[LW], xoff[TM];
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int rt = min(LW * wave + j, N / 16 - 1 - n0 / 16);
    woff[j] = static_cast<uint32_t>(rt) * (Kp / 32) * 1024 + lane * 16;
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int u = TM * wave + j;
    const int row = min(8 * u + (lane >> 3), M - 1 - m0);
    xoff[j] = (static_cast<uint32_t>(row) * ldx + 8 * ((lane & 7) ^ (lane >> 3))) * 2;
  }
  const uint32_t wlds = lds_address(lds) + wave * LW * 1024;
  const uint32_t xlds = lds_address(lds + WS * S::BN * 4) + wave * TM * 1024;
  constexpr uint32_t kWSlot = S::BN * 64, kXSlot = S::BM * 128;  // bytes of a W chunk, an X stage

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const uint32_t wfrag = wn * TN * 1024 + lane * 16;
  const int xrow = wm * TM * 16 + r16;
  const uint32_t xfrag = WS * kWSlot + (xrow >> 3) * 1024 + (xrow & 7) * 128 + 16 * (g ^ (xrow & 7));
  const char* const ldsb = reinterpret_cast<const char*>(lds);
  uint4 a[2][TN], b[2][TM];
  // the u-th fragment, in order of first use, of the chunk (odd: second half of
  // its stage) at ring offsets wo, xo
  auto read_frag = [&](int u, int odd, uint32_t wo, uint32_t xo) __attribute__((always_inline)) {
    if (u >= 1 && u <= TM) {
      b[odd][u - 1] = *reinterpret_cast<const uint4*>(ldsb + ((xfrag ^ (64 * odd)) + xo) + (u - 1) * 2048);
    } else {
      const int i = u == 0 ? 0 : u - TM;
      a[odd][i] = *reinterpret_cast<const uint4*>(ldsb + (wfrag + wo) + i * 1024);
    }
  };

  auto load_w = [&](int c, int j) __attribute__((always_inline)) {
    lds_load16s(wbase + c * 1024, woff[j], wlds + c * kWSlot + j * 1024);
  };
  auto load_x = [&](int s, int j) __attribute__((always_inline)) {
    lds_load16s(xbase + min(s, nc / 2 - 1) * 128, xoff[j], xlds + s * kXSlot + j * 1024);
  };
#pragma unroll
  for (int j = 0; j < LW; ++j) load_w(0, j);
#pragma unroll
  for (int j = 0; j < TM; ++j) load_x(0, j);
#pragma unroll
  for (int j = 0; j < LW; ++j) load_w(1, j);
#pragma unroll
  for (int j = 0; j < TM; ++j) load_x(1, j);
#pragma unroll
  for (int c = 2; c < 4; ++c)
#pragma unroll
    for (int j = 0; j < LW; ++j) load_w(c, j);
#pragma unroll
  for (int j = 0; j < LX0; ++j) load_x(2, j);
  wait_vmcnt<3 * LW + TM + LX0>();
  lds_barrier();
#pragma unroll
  for (int u = 0; u < TN + TM; ++u) read_frag(u, 0, 0, 0);
  wait_vmcnt<2 * LW + TM + LX0>();
  drained_barrier();

  // One chunk, in fragment set P = parity of the chunk: its MFMAs, the
  // fragments of the next chunk (ring offsets wo, xo), the loads of a W chunk
  // (from wsrc to ring offset wd) and of half an X stage (xsrc, xd); then the
  // barrier behind which the chunk after the next has landed: the loads of the
  // last two chunks, and the X half before them if that chunk continues its
  // stage, are younger.  At most one memory instruction per MFMA: a burst of
  // LDS reads would back up and hold the wave's next MFMA.
  auto chunk = [&](auto par, uint32_t wo, uint32_t xo, const char* wsrc, uint32_t wd, const char* xsrc,
                   uint32_t xd) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value, NM = TN * TM, ND = LW + (P ? LX0 : LX1);
    constexpr int RS = 2 * (TN + TM) <= NM ? 2 : 1;
    static_assert(RS * (TN + TM) <= NM && 2 * ND <= NM, "the memory instructions fit behind the MFMAs");
    [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
      (([&]() __attribute__((always_inline)) {
         constexpr int i = U / TM, j = (i & 1) ? TM - 1 - U % TM : U % TM;
         // the direct loads spread over the chunk, behind odd MFMAs; the reads behind the first ones
         constexpr int l = load_behind(U, NM, ND);
         if constexpr (l < LW)
           mfma16_acc_load<l * 1024>(acc[i][j], a[P][i], b[P][j], wsrc, woff[l], wd);
         else if constexpr (l < ND)
           mfma16_acc_load<((P ? 0 : LX0) + l - LW) * 1024>(acc[i][j], a[P][i], b[P][j], xsrc,
                                                            xoff[(P ? 0 : LX0) + l - LW], xd);
         else
           mfma16_acc(acc[i][j], a[P][i], b[P][j]);
         if constexpr (U % RS == 0 && U / RS < TN + TM) read_frag(U / RS, P ^ 1, wo, xo);
         __builtin_amdgcn_sched_barrier(0);
       }()),
       ...);
    }(std::make_integer_sequence<int, NM>{});
    wait_vmcnt<2 * LW + TM + (P ? LX0 : 0)>();
    drained_barrier();
  };
  // Requests past the last chunk re-read it into slots that are no longer
  // needed (the caches hold it), and the last fragments read are never used:
  // so every chunk is the same code and the same counts.
  uint32_t wo = 0, x0 = 0, x1 = kXSlot, x2 = 2 * kXSlot;
  for (int c = 0; c < nc; c += 2) {
    const int s = c >> 1, last = nc - 1;
    chunk(std::integral_constant<int, 0>{}, wo + kWSlot, x0, wbase + min(c + 4, last) * 1024, wlds + wo,
          xbase + min(s + 2, last >> 1) * 128, xlds + x2);
    chunk(std::integral_constant<int, 1>{}, wo ^ (2 * kWSlot), x1, wbase + min(c + 5, last) * 1024,
          wlds + wo + kWSlot, xbase + min(s + 3, last >> 1) * 128, xlds + x0);
    wo ^= 2 * kWSlot;
    const uint32_t x = x0;
    x0 = x1;
    x1 = x2;
    x2 = x;
  }
  wait_vmcnt<0>();
  drained_barrier();
  const int mw = m0 + wm * TM * 16, nw = n0 + wn * TN * 16;
  uint4* const buf = lds + wave * (S::kLds / 4);
  if constexpr (EPI == kEpiRopeKV) {  // launched without k slices
    tile_epilogue_rope_kv<S>(acc, mw, nw, lane, M, N, rk);
  } else if constexpr (EPI == kEpiSwiGLU) {
    if (KS > 1)
      tile_epilogue_f32<S, kEpiStoreF32>(acc, buf, mw, nw, m0, n0, lane, M, N, KS, slice, unit, outf, ldo, part);
    else
      tile_epilogue_swiglu<S>(acc, buf, mw, nw, lane, M, N, outb, ldo);
  } else {
    tile_epilogue_f32<S, EPI>(acc, buf, mw, nw, m0, n0, lane, M, N, KS, slice, unit, outf, ldo, part);
  }
}

// Tail tiles of a product split by gemm_tiled_kernel: out (=|+=) the sum of
// each tile's `split` slice sums, added in slice order.  Workgroup (t, y)
// covers rows 4y .. 4y+3 of tail tile t, a thread 4 consecutive columns.
template <class S, int EPI>
__global__ __launch_bounds__(256) void gemm_tail_fixup_kernel(const float* __restrict__ part, int tail_first,
                                                              int split, int M, int N, float* __restrict__ out,
                                                              int ldo) {
  constexpr int kCols = S::BN / 4;  // threads per tile row
  static_assert(256 % kCols == 0 && S::BM % (256 / kCols) == 0, "rows of a tile split evenly");
  const int i = blockIdx.y * (256 / kCols) + threadIdx.x / kCols;
  const int j = 4 * (threadIdx.x % kCols);
  int m0, n0;
  tile_origin<S, kTailGroupM>(tail_first + blockIdx.x, M, N, m0, n0);
  const int m = m0 + i, n = n0 + j;
  if (m >= M || n >= N) return;
  const float* p = part + static_cast<size_t>(blockIdx.x) * split * S::BM * S::BN + i * S::BN + j;
  float4 a = *reinterpret_cast<const float4*>(p);
  for (int sl = 1; sl < split; ++sl) {
    const float4 v = *reinterpret_cast<const float4*>(p + static_cast<size_t>(sl) * S::BM * S::BN);
    a.x += v.x;
    a.y += v.y;
    a.z += v.z;
    a.w += v.w;
  }
  store_tile<EPI>(f32x4{a.x, a.y, a.z, a.w}, m, n, out, ldo);
}

// The same for the gate/up product: a tile's BN rows of W are BN/16 blocks of
// 8 gate rows then the 8 matching up rows; output column j of the tile (of
// BN/2) takes gate row 16(j/8) + j%8 and up row 16(j/8) + 8 + j%8, summed over
// the slices in slice order, then out_bf16[m][n0/2 + j] = bf16(silu(gate) *
// up).  Workgroup (t, y) covers rows 8y .. 8y+7 of tail tile t, a thread 4
// consecutive output columns.
template <class S>
__global__ __launch_bounds__(256) void gemm_tail_fixup_swiglu_kernel(const float* __restrict__ part, int tail_first,
                                                                     int split, int M, int N,
                                                                     uint16_t* __restrict__ out, int ldo) {
  constexpr int kCols = S::BN / 8;  // threads per tile row (4 of the BN/2 output columns each)
  static_assert(256 % kCols == 0 && S::BM % (256 / kCols) == 0, "rows of a tile split evenly");
  const int i = blockIdx.y * (256 / kCols) + threadIdx.x / kCols;
  const int j = 4 * (threadIdx.x % kCols);
  const int wg = 16 * (j / 8) + j % 8;  // gate row of output column j within the tile
  int m0, n0;
  tile_origin<S, kTailGroupM>(tail_first + blockIdx.x, M, N, m0, n0);
  const int m = m0 + i;
  if (m >= M || n0 + wg >= N) return;
  const float* p = part + static_cast<size_t>(blockIdx.x) * split * S::BM * S::BN + i * S::BN + wg;
  float4 g = *reinterpret_cast<const float4*>(p);
  float4 u = *reinterpret_cast<const float4*>(p + 8);
  for (int sl = 1; sl < split; ++sl) {
    const float* q = p + static_cast<size_t>(sl) * S::BM * S::BN;
    const float4 gv = *reinterpret_cast<const float4*>(q);
    const float4 uv = *reinterpret_cast<const float4*>(q + 8);
    g.x += gv.x;
    g.y += gv.y;
    g.z += gv.z;
    g.w += gv.w;
    u.x += uv.x;
    u.y += uv.y;
    u.z += uv.z;
    u.w += uv.w;
  }
  store_swiglu(f32x4{g.x, g.y, g.z, g.w}, f32x4{u.x, u.y, u.z, u.w}, m, n0 / 2 + j, out, ldo);
}

// ---------------------------------------------------------------------------

constexpr int kSkinnyPF = 1;                // k blocks in flight per wave
constexpr int kSkinnyWaves = 8;             // waves per workgroup (k split inside it)

// Row tiles per wave of the decode kernel: 4 (64 rows) amortises the
// activation reads best, but for short, narrow products (QKV-sized) 2 tiles
// and twice the workgroups finish sooner (11.0 vs 12.9 us at N=6144, K=4096),
// and the gate/up product, which cannot split K, takes 7 where that makes the
// workgroups a multiple of the 256 CUs (448 -> 256 at the 8B shape: 46.3 ->
// 42.5 us).
static int skinny_tiles(int N, int Kp, int epilogue) {
  if (epilogue == kEpiSwiGLU && (N / 16) % (7 * 256) == 0) return 7;
  if (N % 64) return 2;
  return N <= 8192 && Kp <= 4096 ? 2 : 4;
}

// Decode kernel: workgroups split K while fewer than `target` cover the
// product; slices stay multiples of 128, and the slice sums (ks * M * N fp32,
// written and read again) stay within a quarter of the weight bytes (N * Kp
// bf16), i.e. 8 * ks * M <= Kp.
static int gemm_k_splits(int blocks, int target, int M, int Kp) {
  int ks = 1;
  while (blocks * ks < target && ks < 8 && (Kp / (2 * ks)) % 128 == 0 && 8 * (2 * ks) * M <= Kp) ks *= 2;
  return ks;
}

// Tiled kernels: the most k slices (a power of two up to 8, slices multiples
// of 128) whose workgroups still fit one round of the CUs, with slice sums up
// to half the weight bytes (4 * ks * M <= Kp).  Cache-cold, sum included, us for
// 1 / 2 / 4 / 8 slices of 128 x 128 tiles: 8B O at M = 80 35.4 / 23.1 / 18.0 /
// 16.0, at M = 200 36.2 / 24.6 / 20.3 / 23.7, at M = 301 35.8 / 25.9 / 28.6 / 31.7
// (the rule: 8, 4, 2); 8B down at M = 200 113.8 / 65.0 / 42.5 / 45.6 (4); 70B down
// at M = 128 257 / 149 / 105 (4).  Two workgroups of these tiles fit a CU, and
// with a long K a second round's worth of slices can pay: 8B down at M = 301 2
// slices 65.7, 8 62.1; 70B down at M = 200 2 slices 155.9, 4 143.3.
static int tiled_k_splits(int tiles, int cus, int M, int Kp) {
  int ks = 1;
  while (ks < 8 && tiles * (2 * ks) <= cus && (Kp / (2 * ks)) % 128 == 0 && 4 * (2 * ks) * M <= Kp) ks *= 2;
  return ks;
}

// Compute units of the current device (256 on MI355X), cached per device.
static int device_cus() {
  static int cache[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cache[dev] = n;
  }
  return cache[dev];
}

// k slices with which a product of 33 to 64 rows runs as 128 x 64 tiles, 0 if
// the decode kernel takes it.  A tile's workgroup goes through its k slice by
// itself, where the decode kernel puts eight waves on one, so the tiles pay
// while they occupy more than half of the CUs.  In the model, us per launch at
// 33 / 48 / 64 rows, decode kernel against tiles: 192 workgroups (3072 x 3072)
// 12.3 / 13.0 / 13.5 against 9.4 / 9.3 / 9.9; 128 (2048 x 2048) 6.6 / 6.7 / 7.5
// against 7.3 / 7.4 / 7.7, (3072 x 16384, gate/up) 24.8 / 26.2 / 28.3 against
// 32.4 / 30.8 / 31.6; 64 (11008 x 4096) 31.2 / 32.3 / 36.6 against 45.4 / 45.9 /
// 47.0; with no workspace to hold slices, 32 (4096 x 4096) 17.7 / 18.3 / 22.0
// against 33.2 / 33.2 / 33.7, 120 (5120 x 15360) 33.6 / 35.6 / 40.2 against 43.8 /
// 44.5 / 46.2, 136 (4096 x 17408) 47.8 / 51.2 / 56.3 against 37.0 / 37.2 / 38.0.
// Under 4M weights (8 MB) both are bound by latency.
static int small_tile_splits(int M, int N, int Kp, bool split, int64_t part_cap) {
  if (M <= kSkinnyMaxRows || static_cast<int64_t>(N) * Kp < (1 << 22)) return 0;
  const int cus = device_cus(), tiles = (N + SmallTile::BN - 1) / SmallTile::BN;
  int ks = split ? tiled_k_splits(tiles, cus, M, Kp) : 1;
  while (ks > 1 && static_cast<int64_t>(ks) * M * N > part_cap) ks /= 2;
  return 2 * tiles * ks > cus ? ks : 0;
}

// Kernel choice: decode batches (up to 64 rows) the decode kernel or the Small
// tile (small_tile_splits); then 128 x 128 tiles (more blocks) for narrow
// products, and for wide ones up to 192 rows while their tiles number at most
// the CUs; else 256 x 128 tiles for wide products up to 128 rows, or up to 256
// while they number at most the CUs, and for narrow products of up to 128 rows
// that 128 x 128 tiles leave mostly idle; 256 x 256 tiles for the rest and for
// long prefill chunks.
// Cache-cold, us as 128 x 128 / 256 x 128 / 256 x 256 tiles (the last two with
// their last round cut where that applies).  Wide products: 8B gate/up at M =
// 128 48.4 / 58.1 / 58.3, 192 68.9 / 60.5 / 63.7, 256 76.9 / 66.8 / 74.7, 301 97.0
// / 95.1 / 73.1; 70B gate/up at M = 128 181.8 / 168.0 / 170.3, 200 263 / 238 / 191;
// a head of 32000 at M = 128 51.9 / 74.6 / 75.5, 192 73.4 / 67.5 / 78.5; of 128256
// at M = 128 233.9 / 220.3 / 224.2, 192 299 / 286 / 238.  Narrow products: O at M =
// 1000 40.9 / 44.7 / 50.9, 1100 52.1 / 65.4 / 55.6; QKV at M = 1000 66.5 / 54.4 /
// 60.6, 1100 64.7 / 54.1 / 63.1.  kMidMaxRows suits O; with the longer K of 8B
// down 256 x 256 tiles and a cut last round are ahead from about 600 rows (117.7 /
// 104.8 / 81.6; at 1000 130 / 114 / 104), as for 70B QKV from 160 (66.4 / 63.5 /
// 49.9), which the rule does not use.
GemmPlan plan_gemm(int M, int N, int Kp, int epilogue, int64_t part_cap) {
  GemmPlan p{GemmKind::kBig, 4, 1, 1, 0};
  const bool can_split = part_cap > 0;
  const bool split = can_split && epilogue != kEpiSwiGLU && M <= kSplitMaxRows;
  if (M <= 64) {
    if (const int ks = small_tile_splits(M, N, Kp, split, part_cap)) {
      p.kind = GemmKind::kSmall;
      p.ks = ks;
    } else {
      p.kind = GemmKind::kSkinny;
      p.nt = skinny_tiles(N, Kp, epilogue);
      if (split) p.ks = gemm_k_splits(N / (16 * p.nt), p.nt == 2 ? 512 : 256, M, Kp);
    }
    while (p.ks > 1 && static_cast<int64_t>(p.ks) * M * N > part_cap) p.ks /= 2;
    return p;
  }
  auto tiles_of = [&](int bn, int bm) { return ((N + bn - 1) / bn) * ((M + bm - 1) / bm); };
  const int mid_tiles = tiles_of(MidTile::BN, MidTile::BM), wide_tiles = tiles_of(WideTile::BN, WideTile::BM);
  const int cus = device_cus();
  if (N >= 16384) {  // wide products: gate/up and the LM head
    if (M <= 192 && mid_tiles <= cus)
      p.kind = GemmKind::kMid;
    else if (M <= WideTile::BM || (M <= 2 * WideTile::BM && wide_tiles <= cus))
      p.kind = GemmKind::kWide;
    else
      p.kind = GemmKind::kBig;
  } else {
    p.kind = M <= kMidMaxRows ? GemmKind::kMid : GemmKind::kBig;
  }
  // SwiGLU of a short K: most of a 256 x 256 tile's time is then its epilogue
  // (expf and a division per output), one wave per SIMD, where two 128 x 128
  // workgroups per CU cover each other.  Us, former 8-wave kernel / 256 x 256 /
  // 128 x 128 tiles: K 128, N 1376, M 2000 12.5 / 15.8 / 9.1; K 256, N 5632, M 4000
  // 40.6 / 43.6 / 24.6; K 768, N 2816, M 4000 26.7 / 28.2 / 22.3; from K 1024 on
  // 256 x 256 tiles are no slower than that kernel, and ahead where N is wide
  // (N 11264, M 1100 36.4 / 29.5 / 32.4).
  if (p.kind == GemmKind::kBig && epilogue == kEpiSwiGLU && Kp <= 768) p.kind = GemmKind::kMid;
  // Products narrower than a 256-row tile, of which much would be absent rows of
  // W (former kernel / 256 x 256: K 384, N 32, M 2001 13.0 / 17.4 us; 256 x 128, M
  // 128 8.4 / 10.2).
  if (p.kind == GemmKind::kBig && N < BigTile::BN) p.kind = GemmKind::kMid;
  const int kind_tiles = p.kind == GemmKind::kMid    ? mid_tiles
                         : p.kind == GemmKind::kWide ? wide_tiles
                                                     : tiles_of(BigTile::BN, BigTile::BM);
  if (split) p.ks = tiled_k_splits(kind_tiles, cus, M, Kp);
  // Narrow products of up to 128 rows whose 128 x 128 tiles fill under three
  // quarters of the CUs even with k slices take 256 x 128 tiles when those
  // reach at least as many workgroups (70B QKV at M=128: 40 tiles x 4 slices
  // 46.9 us, 80 x 2 of 128 x 128 47.8; at M=80 42.1 against 43.1).
  if (split && p.kind == GemmKind::kMid && M <= WideTile::BM && N >= WideTile::BN &&
      4 * mid_tiles * p.ks < 3 * cus) {
    const int wks = tiled_k_splits(wide_tiles, cus, M, Kp);
    if (wide_tiles * wks >= mid_tiles * p.ks) {
      p.kind = GemmKind::kWide;
      p.ks = wks;
    }
  }
  const int bn = p.kind == GemmKind::kMid ? MidTile::BN : p.kind == GemmKind::kWide ? WideTile::BN : BigTile::BN;
  const int bm = p.kind == GemmKind::kMid ? MidTile::BM : p.kind == GemmKind::kWide ? WideTile::BM : BigTile::BM;
  const int tiles = tiles_of(bn, bm);
  while (p.ks > 1 && static_cast<int64_t>(p.ks) * M * N > part_cap) p.ks /= 2;  // slice sums fit the workspace
  // Last round of 256-row tiles (one workgroup per CU): with r tiles left for
  // C CUs, cut each into S k slices (S a power of two, r * S <= C, slices
  // multiples of 128), so that round takes 1/S of a tile's time; the fixup
  // kernel adds the slices.
  if (p.kind != GemmKind::kMid && p.ks == 1 && can_split) {
    const int r = tiles % cus;
    int sp = 1;
    while (r > 0 && sp < 8 && r * (2 * sp) <= cus && (Kp / (2 * sp)) % 128 == 0) sp *= 2;
    if (sp > 1 && static_cast<int64_t>(r) * sp * bm * bn <= part_cap) {
      p.tail_split = sp;
      p.tail_first = tiles - r;
    }
  }
  return p;
}


template <int MT, int NT, int EPI>
static void launch_skinny(const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N, float* outf,
                          uint16_t* outb, int ldo, float* part, int ks, hipStream_t s) {
  // 7 row tiles: 4 waves, so that the cross-wave reduction buffer fits in LDS
  constexpr int NW = NT == 7 ? 4 : kSkinnyWaves;
  launch_kernel((gemm_skinny_kernel<MT, NT, EPI, kSkinnyPF, NW>), dim3(N / (16 * NT), ks), dim3(NW * 64), 0, s, X,
                ldx, W, Kp, M, N, outf, outb, ldo, part, RopeKV{});
}

template <int NT, int EPI>
static void launch_skinny_m(const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N, float* outf,
                            uint16_t* outb, int ldo, float* part, int ks, hipStream_t s) {
  if (M <= 16)
    launch_skinny<1, NT, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, ks, s);
  else if (M <= 32)
    launch_skinny<2, NT, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, ks, s);
  else
    launch_skinny<4, NT, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, ks, s);
}

template <class S, int EPI>
static void launch_tiled(const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N, float* outf,
                         uint16_t* outb, int ldo, float* part, int ks, hipStream_t s, int tail_split = 1,
                         int tail_first = 0) {
  const int tiles = ((N + S::BN - 1) / S::BN) * ((M + S::BM - 1) / S::BM);
  const int blocks = tail_split > 1 ? tail_first + (tiles - tail_first) * tail_split : tiles;
  launch_kernel((gemm_tiled_kernel<S, EPI>), dim3(blocks, ks), dim3(S::NTH), 0, s, X, ldx, W, Kp, M, N, outf, outb, ldo,
                part, tail_first, tail_split, RopeKV{});
  if (tail_split > 1) {
    if constexpr (EPI == kEpiSwiGLU)
      launch_kernel((gemm_tail_fixup_swiglu_kernel<S>), dim3(tiles - tail_first, S::BM / (2048 / S::BN)),
                    dim3(256), 0, s, part, tail_first, tail_split, M, N, outb, ldo);
    else
      launch_kernel((gemm_tail_fixup_kernel<S, EPI>), dim3(tiles - tail_first, S::BM / (1024 / S::BN)), dim3(256),
                    0, s, part, tail_first, tail_split, M, N, outf, ldo);
  }
}

// go with the smallest of LO .. HI that is at least tm (HI if none is)
template <int LO, int HI, class Go>
static void at_least(int tm, Go&& go) {
  if constexpr (LO < HI) {
    if (tm > LO) return at_least<LO + 1, HI>(tm, go);
  }
  go(std::integral_constant<int, LO>{});
}

// Row blocks of 32 TM rows: as many as the kind's full blocks would be, evened
// out, so that no block works on many absent rows (M = 301: 2 x 160 instead of
// 2 x 256).  LO: the least TM built.
template <class S, int LO, class Go>
static void even_rows(int M, Go&& go) {
  const int blocks = (M + S::BM - 1) / S::BM;
  at_least<LO, S::TM>(((M + blocks - 1) / blocks + 31) / 32, go);
}

template <int EPI>
static hipError_t launch_epi(const GemmPlan& p, const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N,
                             float* outf, uint16_t* outb, int ldo, float* part, hipStream_t s) {
  switch (p.kind) {
    case GemmKind::kSkinny:
      if (p.nt == 7)
        launch_skinny_m<7, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s);
      else if (p.nt == 4)
        launch_skinny_m<4, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s);
      else
        launch_skinny_m<2, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s);
      break;
    case GemmKind::kSmall:
      launch_tiled<SmallTile, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s);
      break;
    case GemmKind::kMid:
      even_rows<MidTile, 3>(M, [&](auto tm) {
        launch_tiled<TileShape<MidTile::TN, tm>, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s);
      });
      break;
    case GemmKind::kWide:
      even_rows<WideTile, 3>(M, [&](auto tm) {
        launch_tiled<TileShape<WideTile::TN, tm>, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s,
                                                       p.tail_split, p.tail_first);
      });
      break;
    case GemmKind::kBig:
      even_rows<BigTile, 5>(M, [&](auto tm) {
        launch_tiled<TileShape<BigTile::TN, tm>, EPI>(X, ldx, W, Kp, M, N, outf, outb, ldo, part, p.ks, s,
                                                      p.tail_split, p.tail_first);
      });
      break;
  }
  return hipGetLastError();
}

// The tiled kernel reaches the rows of a block by 32-bit byte offsets from the
// block's first element (they are 32 bits wide in the load itself).
static bool offsets_fit(const GemmPlan& p, int M, int ldx, int Kp) {
  if (p.kind == GemmKind::kSkinny) return true;  // 64-bit pointers
  const bool big = p.kind == GemmKind::kBig;
  const int bn = big || p.kind == GemmKind::kWide ? BigTile::BN : MidTile::BN;
  const int bm = big ? BigTile::BM : p.kind == GemmKind::kSmall ? SmallTile::BM : MidTile::BM;
  constexpr int64_t kMax = int64_t{1} << 32;
  return 2ll * ldx * std::min(M, bm) <= kMax && 2ll * Kp * bn <= kMax;
}

hipError_t launch_gemm(const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N, int epilogue,
                       float* out_f32, uint16_t* out_bf16, int ldo, float* part, int64_t part_cap, int* n_parts,
                       hipStream_t s) {
  *n_parts = 0;
  if (M <= 0) return hipSuccess;
  auto run = [&](const GemmPlan& p, int m0, int rows) {
    const uint16_t* x = X + static_cast<size_t>(m0) * ldx;
    const size_t o = static_cast<size_t>(m0) * ldo;
    switch (epilogue) {
      case kEpiStoreF32:
        return launch_epi<kEpiStoreF32>(p, x, ldx, W, Kp, rows, N, out_f32 + o, nullptr, ldo, part, s);
      case kEpiAddF32:
        return launch_epi<kEpiAddF32>(p, x, ldx, W, Kp, rows, N, out_f32 + o, nullptr, ldo, part, s);
      case kEpiSwiGLU:
        return launch_epi<kEpiSwiGLU>(p, x, ldx, W, Kp, rows, N, nullptr, out_bf16 + o, ldo, part, s);
      default:
        return hipErrorInvalidValue;
    }
  };
  const GemmPlan p = plan_gemm(M, N, Kp, epilogue, part != nullptr ? part_cap : 0);
  if (offsets_fit(p, M, ldx, Kp)) {
    if (p.ks > 1) *n_parts = p.ks;
    return run(p, 0, M);
  }
  // rows millions of elements apart: the decode kernel, 64 rows at a time
  hipError_t e = hipSuccess;
  for (int m0 = 0; m0 < M && e == hipSuccess; m0 += 64)
    e = run({GemmKind::kSkinny, skinny_tiles(N, Kp, epilogue), 1, 1, 0}, m0, std::min(64, M - m0));
  return e;
}

// Decode kernel: 2 row tiles per wave, 4 waves, K whole: 14.4 us at M=25,
// N=6144, K=4096 (with 4 k slices the product alone takes 13.1 us, but the slice
// sums then cost a RoPE kernel of 5.2 us).  128 x 64 tiles and the RoPE kernel
// cost less once K is kOwnSumMinK or more.  In the model, us per layer at 33 / 48
// / 64 rows, fused against product + RoPE: K 2048, N 6144 13.2 / 13.4 / 15.4
// against 14.2 / 14.5 / 15.2; 2560, 7680 17.9 / 18.1 / 19.5 against 17.7 / 19.2 /
// 19.0; 3072, 9216 27.8 / 29.7 / 34.8 against 25.0 / 25.1 / 25.2; 4096, 6144
// 23.6 / 22.9 / 24.4 against 21.2 / 20.9 / 21.9.
bool gemm_rope_kv_fused(int M, int N, int Kp, int64_t part_cap) {
  if (M <= kRopeKVMaxRows)
    return Kp < kOwnSumMinK || plan_gemm(M, N, Kp, kEpiStoreF32, part_cap).kind != GemmKind::kSmall;
  return plan_gemm(M, N, Kp, kEpiStoreF32, 0).kind == GemmKind::kBig;
}

bool gemm_slices_pay_a_sum(int M, int Kp) { return M > 64 || (M > kSkinnyMaxRows && Kp >= kOwnSumMinK); }

hipError_t launch_gemm_rope_kv(const uint16_t* X, int ldx, const uint16_t* W, int Kp, int M, int N, const RopeKV& rk,
                               hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if ((M > kRopeKVMaxRows && !gemm_rope_kv_fused(M, N, Kp, 0)) || N != (rk.nq + 2 * rk.nkv) * rk.hd || rk.hd % 32 ||
      (rk.hd & (rk.hd - 1)) || N % 32)
    return hipErrorInvalidValue;
  if (M > kRopeKVMaxRows) {  // 256 x 256 tiles over all of K (no workspace: no split of the last round)
    even_rows<BigTile, 5>(M, [&](auto tm) {
      using S = TileShape<BigTile::TN, tm>;
      const int tiles = ((N + S::BN - 1) / S::BN) * ((M + S::BM - 1) / S::BM);
      launch_kernel((gemm_tiled_kernel<S, kEpiRopeKV>), dim3(tiles, 1), dim3(S::NTH), 0, s, X, ldx, W, Kp, M, N,
                    nullptr, nullptr, 0, nullptr, 0, 1, rk);
    });
    return hipGetLastError();
  }
  constexpr int NT = 2, NW = 4;
  auto go = [&](auto mt) {
    constexpr int MT = decltype(mt)::value;
    launch_kernel((gemm_skinny_kernel<MT, NT, kEpiRopeKV, kSkinnyPF, NW>), dim3(N / (16 * NT), 1), dim3(NW * 64), 0,
                  s, X, ldx, W, Kp, M, N, nullptr, nullptr, 0, nullptr, rk);
  };
  if (M <= 16)
    go(std::integral_constant<int, 1>{});
  else if (M <= 32)
    go(std::integral_constant<int, 2>{});
  else
    go(std::integral_constant<int, 4>{});
  return hipGetLastError();
}

hipError_t launch_reduce_parts(const float* part, int KS, int M, int N, int epilogue, float* out, int ldo,
                               hipStream_t s) {
  const int64_t n4 = static_cast<int64_t>(M) * N / 4;
  const int grid = static_cast<int>(std::min<int64_t>((n4 + 255) / 256, 4096));
  if (epilogue == kEpiAddF32)
    launch_kernel((reduce_parts_kernel<kEpiAddF32>), dim3(grid), dim3(256), 0, s, part, KS, M, N, out, ldo);
  else
    launch_kernel((reduce_parts_kernel<kEpiStoreF32>), dim3(grid), dim3(256), 0, s, part, KS, M, N, out, ldo);
  return hipGetLastError();
}

}  // namespace metro
