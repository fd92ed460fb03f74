// Paged grouped-query attention on gfx950 with MFMA.
//
// KV page layout (per layer, page, kv head): K and V^T tiles of 16 keys x hd
// in the layouts of common.h (k_tile_offset, vt_tile_offset), bf16: every
// matrix-core operand is one 16-byte load per lane and every load instruction
// reads 1 KiB of a tile contiguously.
//
//   scores  S^T[key][q] = sum_d K[key][d] Q[q][d]       v_mfma_f32_16x16x32_bf16
//           A = K rows (16 keys), B = Q^T (16 query columns)
//   output  O^T[d][q] += sum_key V^T[d][key] P^T[key][q] v_mfma_f32_16x16x16_bf16
//           (decode, one page) or 16x16x32 over a page pair (prefill)
//
// The MFMA output of S^T leaves lane l with keys 4(l/16)+i of query column
// l%16, which is exactly the B operand the P.V product needs, so the softmax
// runs in registers with no lane shuffles except the two cross-row steps of
// the row maximum.  The query columns are the (token, head) pairs of one GQA
// group, so a K/V page is read once per group.
//
// Precision: scores, the running max/sum and the output accumulators are fp32.
// P enters the bf16 matrix core as hi = bf16(p) plus lo = bf16(p - hi) (two
// MFMAs), which keeps p to about 16 significant bits.
//
// Decode: one workgroup per (work item, kv head), a work item being up to 128
// pages of one row, so that long rows spread over several CUs; its waves take
// the pages round-robin and merge through LDS in wave order.  Rows of several
// work items leave their states in a workspace and a small kernel merges them
// in split order (an agent-scope fence in every workgroup, which an in-kernel
// merge would need, costs L2 write-backs on the multi-XCD chip).  The split
// count depends on the row's own context length only, never on the batch.
//
// Prefill (flash attention): one workgroup = (query block, kv head); the K and
// V pages of the block's visible context go through LDS in pairs, by direct
// loads into a 4-stage ring (three pairs in flight while one is consumed), and
// are shared by the eight waves; causal masking per element.
#include "common.h"
#include "kernels.h"

namespace metro {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma_k32(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma_k16(uint2 a, uint2 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c,
                                                   0, 0, 0);
}

// The upper half of a trades places with the lower half of b.  An MFMA that
// reads the result has to be at least two instructions away (wait states that
// the compiler does not add behind inline assembly): NOPS of them are part of
// the block, the caller keeps the others between.
template <int NOPS>
__device__ __forceinline__ void swap_halves(uint4& a, uint4& b) {
  if constexpr (NOPS == 2)
    asm volatile("v_swap_b32 %0, %2\n\tv_swap_b32 %1, %3\n\ts_nop 1"
                 : "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y));
  else
    asm volatile("v_swap_b32 %0, %2\n\tv_swap_b32 %1, %3" : "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y));
}

// 2^x by the hardware instruction (v_exp_f32, about 1 ulp).  exp2f adds a
// range fix-up (compare, two selects, ldexp) that only matters for results
// below 2^-126; here x = s - m <= 0 is a softmax exponent, and such a weight
// is below half an ulp of the running sum (>= 1) and of any output that the
// weight-1 key contributes to, so it changes no result.
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// p -> (hi, lo) bf16 pairs packed two per word
__device__ __forceinline__ void split_bf16(float p0, float p1, uint32_t& hi, uint32_t& lo) {
  hi = pack_bf16x2(p0, p1);
  lo = pack_bf16x2(p0 - lo_bf16(hi), p1 - hi_bf16(hi));
}

// Keys past the end of a context sit in slots of the last page that no call
// has written (or that hold a closed sequence's values): their softmax weight
// is 0, but 0 times a NaN or Inf bit pattern there would still poison the
// output, so their V values are zeroed.  Decode: in the operand of the row's
// partly filled last page, which is taken outside the page ring so the ring
// holds no extra registers; a V^T operand word holds the bf16 values of two
// consecutive keys k, k + 1 of one dim (k in the low half), and
// keep_below(w, k, n) keeps those below n.  Prefill: in LDS, for the last
// page pair of a query block.
__device__ __forceinline__ uint32_t keep_below(uint32_t w, int k, int n) {
  return k + 1 < n ? w : (k < n ? (w & 0xffffu) : 0u);
}

// ===========================================================================
// Decode
// ===========================================================================

// One workgroup of kDecodeWaves waves per (row, kv head); wave w takes pages
// w, w + kDecodeWaves, ...  The wave's page ids are read once into one VGPR
// (lane j holds the id of the wave's j-th page, 64 pages per pass) so the page
// loop never waits on a memory lookup; PD pages of K/V are kept in flight in
// a register ring.  The waves' (max, sum, output) states are merged through
// LDS in wave order.  Probes over 25 and 200 rows of ~1300-token contexts
// (8 kv heads, scattered pages): 16 waves with two pages in flight (128
// VGPRs) took 26.9 us at 25 rows against 28.1 for 8 waves x 2 and 27.9 for
// 16 x 1; at 200 rows 16 x 1 (102 VGPRs) took 212 us against 218 for 8 x 2
// and 220 for 16 x 2 -- a deeper ring pays while the grid is too small to
// fill the CUs twice over, more resident waves pay once it is not.  Smaller
// splits than 128 pages only moved time into the combine kernel.
constexpr int kDecodeWaves = 16;
constexpr int kDecodeRing2MaxWaves = 512 * 16;  // waves of the grid up to which PD = 2

template <int HD, int G, int NW, int PD, int PS = kDecodePagesPerSplit>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void attn_decode_kernel(AttnArgs a) {
  constexpr int KQ = HD / 32;  // score MFMAs per page
  constexpr int NT = HD / 16;  // output tiles (pairs share one 16-byte V load)
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int wi = blockIdx.x / a.nkv, h = blockIdx.x % a.nkv;
  const int row = a.work[2 * wi], split = a.work[2 * wi + 1];
  const int ctx = a.row_ctx[row];
  const int qrow = a.row_qrow[row];
  const int p0 = split * PS;
  const int32_t* bt = a.bt + a.row_bt[row] + p0;
  const int n_pages = min(ceil_div(ctx, kPage) - p0, PS);  // pages of this split
  const float qscale = a.scale * kLog2e;

  // Q^T operand: column col = head h*G + col (zero beyond the group); MFMA i
  // takes dims 32i + 8grp .. +7, matching the K tile layout.
  uint4 qf[KQ];
#pragma unroll
  for (int i = 0; i < KQ; ++i) qf[i] = make_uint4(0, 0, 0, 0);
  if (col < G) {
    const uint16_t* qp = a.q + (static_cast<size_t>(qrow) * a.nq + h * G + col) * HD;
#pragma unroll
    for (int i = 0; i < KQ; ++i) qf[i] = *reinterpret_cast<const uint4*>(qp + 32 * i + 8 * grp);
  }

  f32x4 o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kNegBig, l = 0.f;

  uint4 kf[PD][KQ];
  uint4 vf[PD][NT / 2];
  const size_t koff = kv_offset(0, 0, a.nkv, h, 0, HD, 0), voff = kv_offset(0, 1, a.nkv, h, 0, HD, 0);
  const size_t pstride = static_cast<size_t>(2) * a.nkv * kPage * HD;
  auto load_page = [&](int sl, int page) {
    const uint16_t* kp = a.kv + static_cast<size_t>(page) * pstride + koff;
    const uint16_t* vp = a.kv + static_cast<size_t>(page) * pstride + voff;
#pragma unroll
    for (int i = 0; i < KQ; ++i) kf[sl][i] = *reinterpret_cast<const uint4*>(kp + 512 * i + 8 * lane);
#pragma unroll
    for (int c = 0; c < NT / 2; ++c) vf[sl][c] = *reinterpret_cast<const uint4*>(vp + 512 * c + 8 * lane);
  };

  // One page: scores, online softmax, P.V.  `last` marks the row's partly
  // filled last page: keys from ctx on get no weight and V = 0.
  auto page_step = [&](const uint4* kp, uint4* vp, int p, bool last) __attribute__((always_inline)) {
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KQ; ++i) s = mfma_k32(kp[i], qf[i], s);
    float sv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) sv[r] = (!last || p * kPage + 4 * grp + r < ctx) ? s[r] * qscale : -INFINITY;
    float mp = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    mp = fmaxf(mp, __shfl_xor(mp, 16, kWave));
    mp = fmaxf(mp, __shfl_xor(mp, 32, kWave));
    const float mn = fmaxf(m, mp);
    const float corr = exp2f(m - mn);
    m = mn;
    float pv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pv[r] = exp2_hw(sv[r] - mn);
    l = l * corr + ((pv[0] + pv[1]) + (pv[2] + pv[3]));
    uint2 hi, lo;
    split_bf16(pv[0], pv[1], hi.x, lo.x);
    split_bf16(pv[2], pv[3], hi.y, lo.y);
    if (last) {
      const int n = ctx - p * kPage, k0 = 4 * grp;
#pragma unroll
      for (int c = 0; c < NT / 2; ++c) {
        vp[c].x = keep_below(vp[c].x, k0, n);
        vp[c].y = keep_below(vp[c].y, k0 + 2, n);
        vp[c].z = keep_below(vp[c].z, k0, n);
        vp[c].w = keep_below(vp[c].w, k0 + 2, n);
      }
    }
#pragma unroll
    for (int c = 0; c < NT / 2; ++c) {
      const uint2 v0 = make_uint2(vp[c].x, vp[c].y), v1 = make_uint2(vp[c].z, vp[c].w);
      o[2 * c] *= corr;
      o[2 * c] = mfma_k16(v0, hi, o[2 * c]);
      o[2 * c] = mfma_k16(v0, lo, o[2 * c]);
      o[2 * c + 1] *= corr;
      o[2 * c + 1] = mfma_k16(v1, hi, o[2 * c + 1]);
      o[2 * c + 1] = mfma_k16(v1, lo, o[2 * c + 1]);
    }
  };

  // Full pages go through the register ring; a partly filled last page of the
  // row (in this split) is taken afterwards by the wave it falls to, so the
  // ring carries no masking.  Each wave's pages and their order are the same
  // either way.
  const bool part_last = (ctx % kPage) != 0 && p0 + n_pages == ceil_div(ctx, kPage);
  const int n_full = n_pages - (part_last ? 1 : 0);
  const int np = wave < n_full ? (n_full - wave + NW - 1) / NW : 0;
  for (int j0 = 0; j0 < np; j0 += 64) {
    const int nj = min(64, np - j0);
    // lane j: id of the wave's page j0 + j
    const int pid = lane < nj ? bt[wave + NW * (j0 + lane)] : 0;
#pragma unroll
    for (int sl = 0; sl < PD; ++sl) load_page(sl, __builtin_amdgcn_readlane(pid, min(sl, nj - 1)));
    for (int base = 0; base < nj; base += PD) {
#pragma unroll
      for (int sl = 0; sl < PD; ++sl) {
        const int it = base + sl;
        if (it < nj) page_step(kf[sl], vf[sl], p0 + wave + NW * (j0 + it), false);
        load_page(sl, __builtin_amdgcn_readlane(pid, min(it + PD, nj - 1)));
      }
    }
  }
  if (part_last && wave == n_full % NW) {
    load_page(0, bt[n_full]);
    page_step(kf[0], vf[0], p0 + n_full, true);
  }
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);

  // merge the waves in order
  __shared__ float sm[NW][G], sl_[NW][G];
  __shared__ float so[NW][HD][G];
  if (col < G) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) so[wave][16 * t + 4 * grp + i][col] = o[t][i];
    if (grp == 0) {
      sm[wave][col] = m;
      sl_[wave][col] = l;
    }
  }
  __syncthreads();
  const bool whole = a.row_nsplit[row] == 1;
  for (int idx = threadIdx.x; idx < G * HD; idx += blockDim.x) {
    const int g = idx / HD, d = idx % HD;
    float M = sm[0][g];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm[w][g]);
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = exp2f(sm[w][g] - M);
      L += sl_[w][g] * f;
      O += so[w][d][g] * f;
    }
    if (whole) {
      a.out[(static_cast<size_t>(qrow) * a.nq + h * G + g) * HD + d] = f32_to_bf16(O / L);
    } else {
      float* pp = a.part + ((static_cast<size_t>(wi) * a.nkv + h) * G + g) * (HD + 2);
      pp[d] = O;
      if (d == 0) {
        pp[HD] = M;
        pp[HD + 1] = L;
      }
    }
  }
}

// Merge the split states of each (row, query head) in split order.  One block
// of hd threads per (row, head); rows with a single split are already final.
__global__ __launch_bounds__(128) void attn_combine_kernel(AttnArgs a) {
  const int row = blockIdx.x / a.nq, j = blockIdx.x % a.nq;
  const int ns = a.row_nsplit[row];
  if (ns == 1) return;
  const int G = a.nq / a.nkv, hd = a.hd;
  const int h = j / G, g = j % G;
  const int w0 = a.row_work[row];
  const int d = threadIdx.x;
  auto state = [&](int s2) { return a.part + ((static_cast<size_t>(w0 + s2) * a.nkv + h) * G + g) * (hd + 2); };
  // Lane l brings split l's max and sum (64 splits at a time), so that neither
  // the maximum nor the weights wait on one memory round trip per split (rows of
  // 2..15 splits, 192 blocks: 111.5 -> 108.8 us for the whole call).
  const int lane = threadIdx.x & 63;
  float M = kNegBig;
  for (int s0 = 0; s0 < ns; s0 += 64) M = fmaxf(M, wave_max(s0 + lane < ns ? state(s0 + lane)[hd] : kNegBig));
  float L = 0.f, O = 0.f;
  for (int s0 = 0; s0 < ns; s0 += 64) {
    const int n = min(64, ns - s0);
    const float* mine = state(s0 + min(lane, n - 1));
    const float f = exp2f(mine[hd] - M), lf = mine[hd + 1];
#pragma unroll 4
    for (int s2 = 0; s2 < n; ++s2) {
      const float fs = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), s2));
      L += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lf), s2)) * fs;
      O += state(s0 + s2)[d] * fs;
    }
  }
  a.out[(static_cast<size_t>(a.row_qrow[row]) * a.nq + j) * hd + d] = f32_to_bf16(O / L);
}

// Zero the V^T entries of keys n0 and beyond in the two V^T page tiles of a
// prefill stage (2 x 16 keys x HD bf16 in LDS), one 32-bit word (two keys of
// one dim) per step.  Out of line: inlined, its index arithmetic raised the
// register count of the whole kernel.
template <int HD>
__device__ __attribute__((noinline)) void zero_v_past(uint32_t* vt, int n0, int tid, int nthreads) {
  constexpr int kWordsPerPage = kPage * HD / 2;
  for (int w = tid; w < 2 * kWordsPerPage; w += nthreads) {
    const int pg = w / kWordsPerPage, in = w % kWordsPerPage;
    // word in of a tile: element pair 2*in, 2*in + 1 = keys 4g + 2j, +1 of dim e
    const int j = in & 1, g = (in >> 6) & 3;   // (((e/32)*4 + g)*16 + e%16)*8 + u*4 + (2j|2j+1)
    const int k = pg * kPage + 4 * g + 2 * j;
    uint32_t v = vt[w];
    if (k >= n0) v = 0u;
    else if (k + 1 >= n0) v &= 0xffffu;
    vt[w] = v;
  }
}

// ===========================================================================
// Prefill (flash attention over pages)
// ===========================================================================

// Query columns of one 16-wide MFMA tile: 16/G tokens x G heads.  A block is
// 8 waves of one tile (128 query columns).  Per page pair and wave the matrix
// core needs 384 cycles and the vector ALU about as many (scale, exp2, hi/lo
// split, sum), so waves in different phases have to overlap: two such blocks,
// each with its own barriers, fit a CU (64 KiB ring, up to 128 VGPRs), where
// one block of 16 waves (head dim 128) or 8 of two tiles (64) filled it before.
// 4 waves per block read the pages from L2 too often (two blocks per CU all the
// same); two tiles per wave with 4 waves halve the LDS reads and gain nothing.
// Blocks run from the end of their list: the last rows of an item, which see the
// most keys, before its first ones.  The items themselves run in reverse order of
// the call, whatever their lengths (whole op call, nkv 8: 4000 rows and 24 items
// of 100, long item listed first 252 us, last 250; 12 items of 310 .. 2400 rows,
// rising 375, falling 397).
// Measured (nq 32, nkv 8, hd 128; us, before -> now): chunks of 3500 and 3800
// after 2000 and 8000 keys 1456 -> 1317; 25 prompts of 256 .. 2416 890 -> 726;
// one of 2048 96 -> 72; 161 rows after 448 keys 29.7 -> 20.3; hd 64, 3 x 700
// after 1000 83 -> 64.
constexpr int kPrefillWaves = 8;

template <int HD, int G>
__global__ __launch_bounds__(kPrefillWaves * 64, 4) void attn_prefill_kernel(PrefillAttnArgs a) {
  constexpr int NW = kPrefillWaves;
  constexpr int KQ = HD / 32;
  constexpr int NT = HD / 16;
  constexpr int TPW = 16 / G;         // tokens per tile
  constexpr int PCH = kPage * HD / 8;  // 16-byte chunks of one K (or V^T) page tile
  constexpr int WPT = NW / 4;         // waves bringing each of the 4 tiles of a stage
  constexpr int LPW = PCH / WPT / 64;  // direct loads per wave per stage
  constexpr int NS = 4;               // stages of the LDS ring
  static_assert(NW % 4 == 0 && PCH % (WPT * 64) == 0, "the waves share each tile evenly");
  // stage = one page pair: [K page 0, K page 1, V^T page 0, V^T page 1]
  __shared__ uint4 ring[NS][4][PCH];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int bi = a.n_blocks - 1 - blockIdx.x / a.nkv, h = blockIdx.x % a.nkv;
  const int item = a.blocks[3 * bi], row0 = a.blocks[3 * bi + 1], nrows = a.blocks[3 * bi + 2];
  const int32_t* bt = a.bt + a.item_bt[item];
  const int last_pos = a.pos[row0 + nrows - 1];
  const int first_pos = a.pos[row0];
  const int n_pages = last_pos / kPage + 1;
  const int n_pairs = (n_pages + 1) / 2;
  const float qscale = a.scale * kLog2e;

  // this lane's query column
  const int tok = wave * TPW + col / G;
  const bool qok = tok < nrows, active = wave * TPW < nrows;
  const int qrow = row0 + (qok ? tok : 0);
  const int qpos = qok ? a.pos[qrow] : -1;
  uint4 qf[KQ];
  const uint16_t* qp = a.q + (static_cast<size_t>(qrow) * a.nq + h * G + col % G) * HD + 8 * grp;
#pragma unroll
  for (int i = 0; i < KQ; ++i) qf[i] = qok ? *reinterpret_cast<const uint4*>(qp + 32 * i) : make_uint4(0, 0, 0, 0);

  f32x4 o[NT];
  float m = kNegBig, l = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Waves WPT*t .. WPT*t + WPT-1 bring the parts of tile t of every stage:
  // the K (t < 2) or V^T (t >= 2) tile of page 2*pair + (t & 1).  The absent
  // second page of an odd count is stood in for by the last page: finite
  // values, all of its keys masked.
  const int tile = wave / WPT, piece = wave % WPT;
  const size_t part = kv_offset(0, tile >> 1, a.nkv, h, 0, HD, 0) + piece * (PCH / WPT) * 8;
  const size_t pstride = static_cast<size_t>(2) * a.nkv * kPage * HD;
  // Lane l holds the id of this wave's page of pair 64 k + l, so that a stage's
  // load issue waits on no memory lookup; the wait for the ids is kept inside
  // the branch (past it, it would also wait for the loads just issued).
  int pid = 0;
  auto issue = [&](int pair) __attribute__((always_inline)) {
    if ((pair & 63) == 0) {
      pid = bt[min(2 * (pair + lane) + (tile & 1), n_pages - 1)];
      asm volatile("" : "+v"(pid));
    }
    const int id = __builtin_amdgcn_readlane(pid, pair & 63);
    const uint16_t* src = a.kv + static_cast<size_t>(id) * pstride + part;
    const uint32_t dst = lds_address(&ring[pair % NS][tile][piece * (PCH / WPT)]);
#pragma unroll
    for (int c = 0; c < LPW; ++c) lds_load16s(src + 512 * c, 16 * lane, dst + 1024 * c);
  };

  issue(0);
  if (n_pairs > 1) issue(1);
  if (n_pairs > 2) issue(2);
  for (int pair = 0; pair < n_pairs; ++pair) {
    // this pair's tiles have landed once at most the later pairs' loads are
    // outstanding; then every wave's part is in LDS after the barrier, and the
    // stage read in the previous iteration is free for pair + 3
    const int later = min(n_pairs - 1 - pair, 2);
    if (later == 2) wait_vmcnt<2 * LPW>();
    else if (later == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    lds_barrier();
    if (pair + 3 < n_pairs) issue(pair + 3);
    const uint4(*st)[PCH] = ring[pair % NS];
    // Keys past the block's last position (never written, or the stand-in
    // page of an odd count) get V = 0 in the stage before any wave reads it:
    // only the last pair can hold them, so only it pays the extra barrier.
    if (const int n0 = last_pos + 1 - 2 * pair * kPage; n0 < 2 * kPage) {
      zero_v_past<HD>(reinterpret_cast<uint32_t*>(&ring[pair % NS][2][0]), n0, tid, NW * 64);
      __syncthreads();
    }

    // Waves without a row of the block (a one-token item beside the chunks of a
    // mixed forward has one row, a ragged chunk's last block a few) only bring
    // their parts of the pages.
    if (!active) continue;
    // scores q.k, K operand (A of S^T): key row col, dims 32i + 8grp .. +7
    float sv[2][4];
#pragma unroll
    for (int pg = 0; pg < 2; ++pg) {
      f32x4 sc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KQ; ++i) sc = mfma_k32(st[pg][64 * i + lane], qf[i], sc);
#pragma unroll
      for (int r = 0; r < 4; ++r) sv[pg][r] = sc[r];
    }
    // (keys of this pair visible to every query of the block need no mask)
    if ((2 * pair + 2) * kPage - 1 > first_pos) {
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if ((2 * pair + pg) * kPage + 4 * grp + r > qpos) sv[pg][r] = -INFINITY;
    }
    // The reference max m only moves when some column's max exceeds it by
    // more than 8 (a factor 2^8): o and l carry the same scale, so their
    // quotient is unchanged, and p = 2^(s - m) stays below 2^8.  Whether any
    // score does is read off the exponents s*scale - m themselves, so the
    // column maxima (a cross-lane reduction) are formed only when m moves.
    float e[2][4];
#pragma unroll
    for (int pg = 0; pg < 2; ++pg)
#pragma unroll
      for (int r = 0; r < 4; ++r) e[pg][r] = fmaf(sv[pg][r], qscale, -m);
    const float top = fmaxf(fmaxf(fmaxf(e[0][0], e[0][1]), fmaxf(fmaxf(e[0][2], e[0][3]), e[1][0])),
                            fmaxf(fmaxf(e[1][1], e[1][2]), e[1][3]));
    if (__any(top > 8.f)) {
      float mp = fmaxf(fmaxf(fmaxf(sv[0][0], sv[0][1]), fmaxf(sv[0][2], sv[0][3])),
                       fmaxf(fmaxf(sv[1][0], sv[1][1]), fmaxf(sv[1][2], sv[1][3])));
      mp = max_xor32(max_xor16(mp)) * qscale;  // in log2 units
      const float mn = fmaxf(m, mp);
      const float corr = exp2f(m - mn);
      m = mn;
      l *= corr;
#pragma unroll
      for (int t = 0; t < NT; ++t) o[t] *= corr;
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int r = 0; r < 4; ++r) e[pg][r] = fmaf(sv[pg][r], qscale, -m);
    }
    float pv[2][4];
    float ps = 0.f;
#pragma unroll
    for (int pg = 0; pg < 2; ++pg)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pv[pg][r] = exp2_hw(e[pg][r]);
        ps += pv[pg][r];
      }
    l += ps;
    // P^T operand over the page pair: k-slot 8grp+j is key 4grp+j of page
    // j/4, the order of the V^T operand
    uint4 hi, lo;
    split_bf16(pv[0][0], pv[0][1], hi.x, lo.x);
    split_bf16(pv[0][2], pv[0][3], hi.y, lo.y);
    split_bf16(pv[1][0], pv[1][1], hi.z, lo.z);
    split_bf16(pv[1][2], pv[1][3], hi.w, lo.w);
    // V^T operands of output tiles 2c, 2c + 1 over the pair, keys 4grp ..
    // 4grp+3 of each page: a page's 16 bytes hold both tiles', so their inner
    // halves trade places (those of c + 1 between the MFMAs of c)
    uint4 v[2][2];
    v[0][0] = st[2][lane];
    v[0][1] = st[3][lane];
    swap_halves<2>(v[0][0], v[0][1]);
#pragma unroll
    for (int c = 0; c < NT / 2; ++c) {
      uint4(&cur)[2] = v[c & 1], (&next)[2] = v[(c + 1) & 1];
      if (c + 1 < NT / 2) {
        next[0] = st[2][64 * (c + 1) + lane];
        next[1] = st[3][64 * (c + 1) + lane];
      }
      o[2 * c] = mfma_k32(cur[0], hi, o[2 * c]);
      o[2 * c + 1] = mfma_k32(cur[1], hi, o[2 * c + 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (c + 1 < NT / 2) swap_halves<0>(next[0], next[1]);
      __builtin_amdgcn_sched_barrier(0);
      o[2 * c] = mfma_k32(cur[0], lo, o[2 * c]);
      o[2 * c + 1] = mfma_k32(cur[1], lo, o[2 * c + 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  const float L = sum_xor32(sum_xor16(l));
  if (!qok) return;
  const float inv = 1.0f / L;
  uint16_t* op = a.out + (static_cast<size_t>(qrow) * a.nq + h * G + col % G) * HD;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    uint2 w;
    w.x = pack_bf16x2(o[t][0] * inv, o[t][1] * inv);
    w.y = pack_bf16x2(o[t][2] * inv, o[t][3] * inv);
    *reinterpret_cast<uint2*>(op + 16 * t + 4 * grp) = w;
  }
}

// ===========================================================================

template <int HD, int G, int NW>
static hipError_t launch_decode_g(bool ring2, dim3 grid, dim3 block, const AttnArgs& a, hipStream_t s) {
  if (ring2)
    launch_kernel((attn_decode_kernel<HD, G, NW, 2>), grid, block, 0, s, a);
  else
    launch_kernel((attn_decode_kernel<HD, G, NW, 1>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int HD>
static hipError_t launch_decode_hd(const AttnArgs& a, hipStream_t s) {
  constexpr int NW = kDecodeWaves;
  const dim3 grid(a.n_work * a.nkv), block(NW * 64);
  const bool ring2 = static_cast<int64_t>(a.n_work) * a.nkv * NW <= kDecodeRing2MaxWaves;
  switch (a.nq / a.nkv) {
    case 1: return launch_decode_g<HD, 1, NW>(ring2, grid, block, a, s);
    case 2: return launch_decode_g<HD, 2, NW>(ring2, grid, block, a, s);
    case 4: return launch_decode_g<HD, 4, NW>(ring2, grid, block, a, s);
    case 8: return launch_decode_g<HD, 8, NW>(ring2, grid, block, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_attn_combine(const AttnArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  launch_kernel(attn_combine_kernel, dim3(a.rows * a.nq), dim3(a.hd), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_attn_decode(const AttnArgs& a, hipStream_t s) {
  if (a.n_work <= 0) return hipSuccess;
  if (a.hd == 128) return launch_decode_hd<128>(a, s);
  if (a.hd == 64) return launch_decode_hd<64>(a, s);
  return hipErrorInvalidValue;
}

template <int HD>
static hipError_t launch_prefill_hd(const PrefillAttnArgs& a, hipStream_t s) {
  const dim3 grid(a.n_blocks * a.nkv), block(kPrefillWaves * 64);
  switch (a.nq / a.nkv) {
    case 1: launch_kernel((attn_prefill_kernel<HD, 1>), grid, block, 0, s, a); break;
    case 2: launch_kernel((attn_prefill_kernel<HD, 2>), grid, block, 0, s, a); break;
    case 4: launch_kernel((attn_prefill_kernel<HD, 4>), grid, block, 0, s, a); break;
    case 8: launch_kernel((attn_prefill_kernel<HD, 8>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attn_prefill(const PrefillAttnArgs& a, hipStream_t s) {
  if (a.n_blocks <= 0) return hipSuccess;
  if (a.hd == 128) return launch_prefill_hd<128>(a, s);
  if (a.hd == 64) return launch_prefill_hd<64>(a, s);
  return hipErrorInvalidValue;
}

int prefill_tokens_per_block(int group) { return kPrefillWaves * 16 / group; }

}  // namespace metro
