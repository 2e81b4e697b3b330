// Prefill path (M > 16): fp16 MFMA GEMM with the weights dequantised in registers, for gfx950.
//
// Three kernels on one stream:
//  1. gather_cols_kernel: Xp[m, j] = X[m, col_perm[j]] (identity without a permutation), one row through
//     LDS per workgroup (coalesced read, coalesced 16-byte writes), written as contiguous 128x128 blocks so
//     that a GEMM step reads 32 contiguous KiB instead of 128 row pieces K*2 bytes apart (10 % faster
//     GEMM).  A random column gather inside the GEMM would turn every 2-byte element into its own
//     cache-line request for each of the N/128 workgroups that need it; doing it once costs 4*M*K bytes
//     of streaming traffic.
//  2. prefill_fed_kernel: workgroup = one tile row (128 features) x 64 to 256 rows of the batch, eight wavefronts that
//     multiply and four that bring everything in.  K is walked one 128x128 weight tile (= one quantisation
//     group) per step, the tiles of the tile row sorted by width (the order of a sum is free; ranks by
//     ballots over the row's tile descriptors): three loops, each with a straight-line body for its width.  A packed
//     slab is already laid out as an MFMA B operand (lane = weight row-in-16 x k-block of 8): a wavefront
//     reads the words of its 32 output columns from LDS and dequantises them in registers (mask-or
//     into the 0x6400 magic, exact q, then fp16(s*q + z) with one FMA, Appendix B Eq. 11) straight
//     into the B operands of v_mfma_f32_16x16x32_f16; every operand feeds four to eight MFMAs.  Activations, packed
//     words and parameters go from global memory directly into LDS.  The product leaves through LDS in whole 256-byte
//     row segments.
//     prefill_mixed_kernel: whole rounds of its 256-row workgroups, and smaller ones on the last tile rows.
//     prefill_kernel: 128 x 128 outputs, four wavefronts that do all of this themselves, two workgroups per CU; for the
//     few numbers of workgroups that suit it better.
//  3. scatter_cols_kernel (only with a row permutation): the GEMM writes the product in reordered
//     row order into the workspace, then Y[m, row_perm[i]] = Yt[m, i] is done one row through LDS.
//     Scattering 2-byte results straight from the GEMM epilogue leaves half-written cache lines all
//     over Y and doubled the kernel time.
#include <cstdlib>
#include <type_traits>

#include "sfmp_device.h"
#include "sfmp_internal.h"
#include "sfmp_schedule.h"

namespace sfmp {

// -------------------------------------------------------------------------------------------
// column gather / column scatter, one row of fp16 through LDS per workgroup
// -------------------------------------------------------------------------------------------
// A row per workgroup, as many threads as give each the same number of units of 8 columns (see pass_threads).  Several rows per
// workgroup, which share the permutation entries, and 1024 threads whatever K, were 0.3 to 1.4 us longer (this pass alone: 777 x 4096
// 3.7 -> 3.5 us, 2048 x 4096 8.5 -> 7.1, 2048 x 28672 53.9 -> 51.9).  Stored past the caches it takes 35 of those 52 us, but the product,
// which reads it next, becomes as much longer (64 x 4096 -> 14336 even 4 % in all).
__global__ __launch_bounds__(1024) void gather_cols_kernel(const _Float16* __restrict__ X,
                                                           const int32_t* __restrict__ col_perm,
                                                           _Float16* __restrict__ Xp, int K) {
  // Output layout: blocks of 128 rows x 128 columns, each block contiguous (32 KiB), block (mt, tc) at
  // (mt * K/128 + tc) * 16384 elements: the GEMM then reads one contiguous block per step instead of 128
  // row pieces K*2 bytes apart.
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const _Float16* row = reinterpret_cast<const _Float16*>(lds_raw);
  const int64_t m = blockIdx.x;
  const int units = K / 8, threads = (int)blockDim.x;
  const uint4* src = reinterpret_cast<const uint4*>(X + m * K);
  for (int i = threadIdx.x; i < units; i += threads) reinterpret_cast<uint4*>(lds_raw)[i] = src[i];
  __syncthreads();
  const int64_t ntc = K / kTile;
  _Float16* const dst = Xp + (m / kTile) * ntc * (kTile * kTile) + (m % kTile) * kTile;
  for (int i = threadIdx.x; i < units; i += threads) {
    int4 c0 = int4{8 * i, 8 * i + 1, 8 * i + 2, 8 * i + 3}, c1 = int4{8 * i + 4, 8 * i + 5, 8 * i + 6, 8 * i + 7};
    if (col_perm) {  // (no permutation: the pass only changes the layout)
      c0 = reinterpret_cast<const int4*>(col_perm)[2 * i];
      c1 = reinterpret_cast<const int4*>(col_perm)[2 * i + 1];
    }
    union {
      _Float16 h[8];
      uint4 u;
    } v;
    v.h[0] = row[c0.x];
    v.h[1] = row[c0.y];
    v.h[2] = row[c0.z];
    v.h[3] = row[c0.w];
    v.h[4] = row[c1.x];
    v.h[5] = row[c1.y];
    v.h[6] = row[c1.z];
    v.h[7] = row[c1.w];
    *reinterpret_cast<uint4*>(dst + (int64_t)(i / 16) * (kTile * kTile) + (i % 16) * 8) = v.u;
  }
}

// Y[m, row_perm[i]] = Yt[m, i].  PAST: the result is stored past the caches (see stores_past_caches).
template <bool PAST>
__global__ __launch_bounds__(1024) void scatter_cols_kernel(const _Float16* __restrict__ Yt,
                                                           const int32_t* __restrict__ row_perm,
                                                           _Float16* __restrict__ Y, int N) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  _Float16* row = reinterpret_cast<_Float16*>(lds_raw);
  const int64_t m = blockIdx.x;
  const uint4* src = reinterpret_cast<const uint4*>(Yt + m * N);
  for (int i = threadIdx.x; i < N / 8; i += (int)blockDim.x) {
    const int4 c0 = reinterpret_cast<const int4*>(row_perm)[2 * i];
    const int4 c1 = reinterpret_cast<const int4*>(row_perm)[2 * i + 1];
    union {
      _Float16 h[8];
      uint4 u;
    } v;
    v.u = src[i];
    row[c0.x] = v.h[0];
    row[c0.y] = v.h[1];
    row[c0.z] = v.h[2];
    row[c0.w] = v.h[3];
    row[c1.x] = v.h[4];
    row[c1.y] = v.h[5];
    row[c1.z] = v.h[6];
    row[c1.w] = v.h[7];
  }
  __syncthreads();
  u32x4* dst = reinterpret_cast<u32x4*>(Y + m * N);
  for (int i = threadIdx.x; i < N / 8; i += (int)blockDim.x) {
    const u32x4 v = reinterpret_cast<const u32x4*>(row)[i];
    if constexpr (PAST)
      __builtin_nontemporal_store(v, dst + i);
    else
      dst[i] = v;
  }
}

// Y[m, row_perm[i]] (or Y[m, i]) = fp16( sum over the K ranges, in range order, of partial[ks][m][i] ): the second
// half of a split-K product, one row through LDS per workgroup.
template <int KS>  // K ranges: ksplit rounded up to 2, 4 or 8
__global__ __launch_bounds__(1024) void reduce_split_kernel(const float* __restrict__ partial, int ksplit, int M,
                                                            const int32_t* __restrict__ row_perm,
                                                            _Float16* __restrict__ Y, int N) {
  // (1024 threads, and eight loads of a thread issued before the sums - the ranges of one column group, or of two or
  // four: with few rows there are few workgroups, and a chain of dependent round trips per thread made this pass
  // longer than the GEMM)
  extern __shared__ __align__(16) unsigned char lds_raw[];
  _Float16* row = reinterpret_cast<_Float16*>(lds_raw);
  const int64_t m = blockIdx.x;
  constexpr int U = 8 / KS;
  for (int i0 = threadIdx.x; i0 < N / 4; i0 += 1024 * U) {
    floatx4 v[U][KS];
    int4 c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + 1024 * u, N / 4 - 1);
      c[u] = row_perm ? reinterpret_cast<const int4*>(row_perm)[i] : int4{4 * i, 4 * i + 1, 4 * i + 2, 4 * i + 3};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        v[u][ks] = ks < ksplit ? *reinterpret_cast<const floatx4*>(partial + ((int64_t)ks * M + m) * N + 4 * i)
                               : floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      floatx4 s = v[u][0];
#pragma unroll
      for (int ks = 1; ks < KS; ++ks) s += v[u][ks];  // range order; the ranges past ksplit add zeros
      if (i0 + 1024 * u < N / 4) {
        row[c[u].x] = (_Float16)s[0];
        row[c[u].y] = (_Float16)s[1];
        row[c[u].z] = (_Float16)s[2];
        row[c[u].w] = (_Float16)s[3];
      }
    }
  }
  __syncthreads();
  uint4* dst = reinterpret_cast<uint4*>(Y + m * N);
  for (int i = threadIdx.x; i < N / 8; i += 1024) dst[i] = reinterpret_cast<const uint4*>(row)[i];
}

// -------------------------------------------------------------------------------------------
// dequant + MFMA GEMM
// -------------------------------------------------------------------------------------------
struct PrefillParams {
  const _Float16* Xp;  // staged activations, columns in reordered order, as contiguous 128x128 blocks (mt, tc)
  const uint8_t* s2;
  const uint8_t* s3;
  const uint8_t* s4;
  const int32_t* index;  // the whole block-index table
  const _Float16* scales;
  const _Float16* zeros;
  _Float16* Yt;  // [M, N], rows of Wt in reordered order
  int32_t M, N, ntr, ntc, n_mtiles;
  int32_t gshift;  // log2(group / 128): tile column tc uses parameter row tc >> gshift
  int32_t ksplit;  // K ranges (1 = the whole K in one workgroup; prefill_fed_kernel only)
  WorkItems items;  // the order of the work items (prefill_fed_kernel only)
  float* partial;  // ksplit > 1: fp32 partial products [ksplit][M][N], rows of Wt in reordered order
};
static_assert(sizeof(PrefillParams) <= 128, "two 64-byte lines of arguments (with a third calls of 11 us took 0.1 us longer)");

constexpr int kPrefillMaxTiles = 224 * 2;  // K <= 57344

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// 16 bytes per lane from global memory straight into LDS at lds_base + 16*lane.  Written as inline
// assembly so that the compiler's wait-count bookkeeping does not see it: the kernel orders these
// loads itself (they complete in issue order with the ordinary loads around them).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is named as clobbered on purpose
__device__ __forceinline__ void load_to_lds_16(u32x4 rsrc, uint32_t soffset, uint32_t byte_offset, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %0, %2 offen lds" ::"s"(rsrc), "v"(byte_offset), "s"(soffset),
               "s"(lds_base)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// 256-byte LDS rows of the activation block: 16-byte unit u of row r is stored at position u ^ (r % 16).  The 16
// rows that one quarter of a wavefront reads for an MFMA operand then hit 16 different positions (all 64
// banks once), and the position does not depend on the 16-row block, so operand addresses of a lane differ
// by multiples of 4096 bytes: immediate offsets.
__device__ __forceinline__ int swz(int row, int unit) { return unit ^ (row & 15); }

// One MFMA B operand in registers: the 16 weight rows {8i + sigma} x the 32 columns of k-step KAPPA of a
// slab, dequantised exactly: q from the 0x6400 magic (1024 + q*2^p) by one exact FMA, then
// fp16(s*q + z) by one FMA (Appendix B Eq. 11, a single rounding).  `magic` is 0x64006400 held in a
// vector register so that mask-and-or is one instruction (two literals do not fit into one).
template <int B, int KAPPA>
__device__ __forceinline__ half8 dequant_operand(const uint32_t* w, half2_ s2, half2_ z2, uint32_t magic) {
  uint32_t op[4][4];
  unpack_slab<B>(w, op);  // the other k-steps are dead code here and shared between the four calls
  constexpr int p = step_pos<B>(KAPPA);
  const _Float16 inv = (_Float16)(1.0f / (float)(1 << p));
  const _Float16 off = (_Float16)(-1024.0f / (float)(1 << p));
  const half2_ inv2 = {inv, inv}, off2 = {off, off};
  union {
    half2_ h[4];
    half8 v;
  } out;
#pragma unroll
  for (int reg = 0; reg < 4; ++reg) {
    union {
      uint32_t u;
      half2_ h;
    } t;
    t.u = op[KAPPA][reg] | magic;
    const half2_ q = __builtin_elementwise_fma(t.h, inv2, off2);  // exact: q in [0, 15]
    out.h[reg] = __builtin_elementwise_fma(q, s2, z2);            // one rounding
  }
  return out.v;
}

// Lays out the tiles of tile row tr in the order of the K reduction: seq[position] = (slot << 9) | tile column; end2, end3 = the
// positions of the first 3-bit and the first 4-bit tile.
// Sorted by width (first all 2-bit tiles, then the 3-bit, then the 4-bit ones, each in ascending column order; the order
// of a sum is free): three loops, each with a straight-line body for its width.  The sequence is laid out from the tile
// descriptors of the row (slot << 2 | width - 2, one per tile column), whose address depends on the arguments alone:
// ranks by ballots, per 64 columns, instead of the row's runs in the CSR part of the table, which are a dependent trip to
// memory later.
template <int THREADS>
__device__ __forceinline__ void lay_out_tiles(const PrefillParams& p, const int tr, int2* counts, int& end2, int& end3, int32_t* seq) {
  const int32_t* desc = p.index + 3 + (int64_t)tr * p.ntc;
  constexpr int kPer = (kPrefillMaxTiles + THREADS - 1) / THREADS;
  constexpr int kChunks = kPer * (THREADS / kWave);
  static_assert(kPrefillMaxTiles <= kPer * THREADS, "one descriptor per thread and pass");
  int32_t d[kPer];
  uint64_t is2[kPer], is3[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = (int)threadIdx.x + u * THREADS;
    d[u] = e < p.ntc ? desc[e] : 3;
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    is2[u] = __ballot((d[u] & 3) == 0);
    is3[u] = __ballot((d[u] & 3) == 1);
    if ((threadIdx.x % kWave) == 0) counts[(int)threadIdx.x / kWave + u * (THREADS / kWave)] = int2{__popcll(is2[u]), __popcll(is3[u])};
  }
  __syncthreads();
  int2 before[kPer] = {};
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int2 n = counts[c];
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (c < (int)threadIdx.x / kWave + u * (THREADS / kWave)) before[u].x += n.x, before[u].y += n.y;
    end2 += n.x, end3 += n.y;
  }
  end2 = __builtin_amdgcn_readfirstlane(end2);
  end3 = end2 + __builtin_amdgcn_readfirstlane(end3);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = (int)threadIdx.x + u * THREADS;  // = tile column
    if (e < p.ntc) {
      // Each tile row walks its runs from a slightly different starting point: the workgroups of one XCD all read the
      // same activation rows, and 256-byte pieces at the same tile column of rows K*2 bytes apart sit in the same L2
      // channel, so workgroups marching exactly in step would all queue at one channel.  The starting points lie
      // within 8 tiles of each other, no further: the workgroups that share an M block then sweep the tile columns
      // together, in ascending order inside a run, and an activation block that one of them has brought into
      // the XCD's L2 is still there for the others.  (With starting points spread over the whole run, as they
      // were at first, every workgroup streamed its M block by itself as soon as that no longer fitted in L2:
      // 6.9 GB fetched per call on 28672 -> 8192 at M = 2048 instead of 1.9 GB, 1003 us instead of 901.)
      const uint64_t below = (1ull << (threadIdx.x % kWave)) - 1;
      const int rank2 = before[u].x + __popcll(is2[u] & below), rank3 = before[u].y + __popcll(is3[u] & below);
      const uint32_t bw = (uint32_t)(d[u] & 3) + 2;
      const int lo = bw == 2 ? 0 : bw == 3 ? end2 : end3;
      const int n = (bw == 2 ? end2 : bw == 3 ? end3 : p.ntc) - lo;
      const int rank = bw == 2 ? rank2 : bw == 3 ? rank3 : e - rank2 - rank3;
      const int back = rank - (int)((uint32_t)((tr * 5) % 8) % (uint32_t)n);
      const int pos = lo + (back < 0 ? back + n : back);
      const uint32_t slot = (uint32_t)d[u] >> 2;
      seq[pos] = (int32_t)(slot << 9) | e;
    }
  }
}

// G64: group length 64 - a tile column has two (scale, zero) pairs per row, one for its k-steps 0-1 and one for 2-3.
// BF16: scales and zeros are bfloat16.  An instantiation each: decided at run time, both conversions were computed and one
// chosen, in a 128-row step 12 of 138 to 152 vector instructions with fp16 parameters and 6 with bf16 ones, at group length
// 64 26 and 16 of 159 to 173 (a branch instead costs 2 % of the large calls, at the synchronisation point).
template <bool G64, bool BF16>
__global__ __launch_bounds__(256, 2) void prefill_kernel(const PrefillParams p) {
  // 128 x 128 outputs, four wavefronts of all 128 rows x two slabs each: a dequantised B operand feeds MI MFMAs
  constexpr int BM = 128, MI = BM / 16, NS = 2;
  constexpr int kRowsPerPass = 256 / 16, kPasses = BM / kRowsPerPass;
  constexpr uint32_t kBufBytes = BM * 256;
  __shared__ __align__(16) unsigned char Xs[2 * kBufBytes];  // activation blocks
  __shared__ int32_t seq[kPrefillMaxTiles];  // the tiles of this tile row, width-sorted: (slot << 9) | tc
  __shared__ int2 counts[8];  // 2-bit and 3-bit tiles per 64 tile columns

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // Work items (tile row, M block) are numbered with the M blocks innermost, and block b (which runs on XCD
  // b % 8) takes item b.  With a multiple of 8 M blocks an XCD always sees the same M blocks (their activation
  // rows stay in its L2), and in any case the blocks that run at the same time need the same weight tiles, so
  // a tile comes from HBM once per XCD, not once per M block.  (Every XCD works for any number of M blocks.)
  const int mt = (int)blockIdx.x % p.n_mtiles;
  const int tr = (int)blockIdx.x / p.n_mtiles;
  const int m0 = mt * BM;
  const int e_last = p.ntc - 1;

  int end2 = 0, end3 = 0;  // positions of the first 3-bit and of the first 4-bit tile
  lay_out_tiles<256>(p, tr, counts, end2, end3, seq);
  __syncthreads();

  const int wn = wave;  // this wavefront: slabs NS*wn .. NS*wn+NS-1
  floatx4 acc[MI][NS];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int xrow = tid / 16, xunit = tid % 16;  // + kRowsPerPass*pass rows
  const int i16 = lane % 16, kb = lane / 16;
  uint32_t magic;
  asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(magic));

  // The activation block goes from global memory straight into LDS (no staging registers).  A 16-byte
  // LDS-DMA load of a wavefront fills 1024 contiguous bytes = four 256-byte rows, lane l -> row l/16,
  // 16-byte position l%16; the swizzle is applied on the global side: position u of row r receives
  // unit u ^ (r%16).
  uint32_t xoff[kPasses];  // byte offsets from Xp + m0*K + tc*128
#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    const int row = xrow + kRowsPerPass * i;
    xoff[i] = 2u * (uint32_t)(row * kTile + swz(row, xunit) * 8);
  }
  // block (mt, tc) of the staged activations starts at (mt * ntc + tc) * 16384 elements; rows past M of the last
  // row block are never written and feed only output rows that are never stored
  const _Float16* xbase = p.Xp + (int64_t)(m0 / kTile) * p.ntc * (kTile * kTile) + (m0 % kTile) * kTile;
  const uint64_t xb64 = (uint64_t)xbase;
  const uint32_t xbytes = (uint32_t)p.ntc * (uint32_t)(kTile * kTile * 2);  // of the row block
  const uint32_t xs_base = (uint32_t)(uintptr_t)(lptr_t)Xs;
  // copies [first, last) of a block into buffer `buf`
  auto issue_x_part = [&](const BlockRequest& x, int buf, int first, int last) __attribute__((always_inline)) {
    const u32x4 rsrc = {(uint32_t)xb64, (uint32_t)(xb64 >> 32), x.records, 0x00020000u};
    const uint32_t dst = xs_base + (uint32_t)buf * kBufBytes + wave * 1024;
#pragma unroll
    for (int i = first; i < last; ++i) load_to_lds_16(rsrc, x.offset, xoff[i], dst + i * (kRowsPerPass * 256));
  };
  // block of tile position e into the buffer that block `like` uses (like = e mod 2, except for the idle
  // loads past the end)
  auto issue_x = [&](int e, int like) __attribute__((always_inline)) {
    const uint32_t tc = (uint32_t)(__builtin_amdgcn_readfirstlane(seq[e]) & 511);
    issue_x_part(block_request(tc << 15, xbytes, true), like & 1, 0, kPasses);
  };
  // operand read addresses: row 16*i + i16, unit 4*kappa + kb -> byte offset aoff[kappa] + 4096*i
  uint32_t aoff[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) aoff[k] = (uint32_t)(i16 * 256 + swz(i16, 4 * k + kb) * 16);

  // Packed weights of one tile for this wavefront: one load of 4*b bytes per slab and lane, whatever the
  // width (equal load counts on the three paths keep the compiler's wait counts exact), plus NS
  // consecutive fp16 scales and zeros (rows 8*i16 + NS*wn + 0..NS-1 of the tile).
  constexpr int NG = G64 ? 2 : 1;  // parameter pairs per row and tile column
  struct SZ {
    uint32_t s[NG][NS / 2], z[NG][NS / 2];
  };
  auto issue_sz = [&](int tc, SZ& rsz) __attribute__((always_inline)) {
    const int64_t off = (int64_t)(G64 ? 2 * tc : tc >> p.gshift) * p.N + (int64_t)tr * 128 + 8 * i16 + NS * wn;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int q = 0; q < NS / 2; ++q) {
        rsz.s[g][q] = reinterpret_cast<const uint32_t*>(p.scales + off + (int64_t)g * p.N)[q];
        rsz.z[g][q] = reinterpret_cast<const uint32_t*>(p.zeros + off + (int64_t)g * p.N)[q];
      }
  };
  // width known at compile time (the next tile belongs to the same run): no branch around the loads, so
  // they land in place and nothing waits for them before the next step
  auto issue_w_static = [&](auto btag, int e, u32x4 (&rw)[NS], SZ& rsz) __attribute__((always_inline)) {
    constexpr int B = decltype(btag)::value;
    const int32_t d = __builtin_amdgcn_readfirstlane(seq[e]);
    const uint8_t* stream = B == 2 ? p.s2 : B == 3 ? p.s3 : p.s4;
    const uint8_t* src = stream + (int64_t)(d >> 9) * (2048 * B) + (NS * wn) * (256 * B) + lane * (4 * B);
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      if constexpr (B == 4) {
        rw[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + q * 1024));
      } else if constexpr (B == 3) {
        const uint32_t* s3 = reinterpret_cast<const uint32_t*>(src + q * 768);  // 4-byte aligned: three dwords, merged
        rw[q][0] = __builtin_nontemporal_load(s3);
        rw[q][1] = __builtin_nontemporal_load(s3 + 1);
        rw[q][2] = __builtin_nontemporal_load(s3 + 2);
      } else {
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(src + q * 512));
        rw[q][0] = v[0];
        rw[q][1] = v[1];
      }
    }
    issue_sz(d & 511, rsz);
  };
  // width decided at run time (near the end of a run, where the tile two steps ahead has another width):
  // the same load sequence for every width, the words a narrower width does not have re-read its last
  // word.  No branch around the loads, so they land in place.
  auto issue_w_generic = [&](int e, u32x4 (&rw)[NS], SZ& rsz) __attribute__((always_inline)) {
    const int32_t d = __builtin_amdgcn_readfirstlane(seq[e]);
    const int bw = e < end2 ? 2 : e < end3 ? 3 : 4;
    const uint8_t* stream = bw == 2 ? p.s2 : bw == 3 ? p.s3 : p.s4;
    const uint8_t* src = stream + (int64_t)(d >> 9) * (2048 * bw) + (NS * wn) * (256 * bw) + lane * (4 * bw);
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const uint32_t* s = reinterpret_cast<const uint32_t*>(src + q * (256 * bw));
      const uint32_t v0 = __builtin_nontemporal_load(s), v1 = __builtin_nontemporal_load(s + 1),
                     v2 = __builtin_nontemporal_load(s + min(2, bw - 1)), v3 = __builtin_nontemporal_load(s + bw - 1);
      rw[q] = u32x4{v0, v1, v2, v3};
    }
    issue_sz(d & 511, rsz);
  };

  u32x4 fw[NS];  // landing registers of the next tile's packed words
#pragma unroll
  for (int q = 0; q < NS; ++q) fw[q] = u32x4{0u, 0u, 0u, 0u};
  SZ fsz;

  // ---- the software pipeline -------------------------------------------------------------------------
  // State between steps: w / s2 / z2 = packed words, scales, zeros of tile e; a0 / b0 = the MFMA operands
  // of its k-step 0; in flight: activation block e+1 (into the other LDS buffer) and the weights of tile
  // e+1 (into fw).  A step runs four groups; in each the MFMAs of one k-step are interleaved with the LDS
  // reads and the dequantisation of the next one (an MFMA occupies the matrix pipe for 16 cycles but the
  // issue port for 4).  Between the third and the fourth group sits the only synchronisation point: all
  // operand reads of block e have returned, block e+1 and tile e+1 have landed, a barrier, and the loads of
  // e+2 start; the fourth group then already prepares k-step 0 of tile e+1.
  u32x4 w[NS];
  half2_ s2[NG][NS], z2[NG][NS];
  half8 a0[MI], a1[MI], b0[NS], b1[NS];

  auto read_a = [&](int buf, auto ktag, half8(&a)[MI]) __attribute__((always_inline)) {
    const unsigned char* base = Xs + buf * kBufBytes + aoff[decltype(ktag)::value];
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = *reinterpret_cast<const half8*>(base + i * 4096);
  };
  auto make_b = [&](auto btag, auto ktag, half8(&b)[NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const uint32_t words[4] = {w[j][0], w[j][1], w[j][2], w[j][3]};
      constexpr int g = G64 ? decltype(ktag)::value / 2 : 0;  // k-steps 0-1 / 2-3 = columns 0-63 / 64-127
      b[j] = dequant_operand<decltype(btag)::value, decltype(ktag)::value>(words, s2[g][j], z2[g][j], magic);
    }
  };
  auto make_b_any = [&](int e, auto ktag, half8(&b)[NS]) __attribute__((always_inline)) {
    if (e < end2)
      make_b(std::integral_constant<int, 2>{}, ktag, b);
    else if (e < end3)
      make_b(std::integral_constant<int, 3>{}, ktag, b);
    else
      make_b(std::integral_constant<int, 4>{}, ktag, b);
  };
  auto mfmas = [&](const half8(&a)[MI], const half8(&b)[NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NS; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < MI * NS; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
    }
  };
  // Synchronisation point.  Loads complete in issue order and X(e+1) was issued before W(e+1): the wait
  // the compiler puts in front of the moves out of the landing registers also covers the LDS-DMA loads of
  // block e+1.  No operand read may still be in the LDS queue when the barrier opens this step's buffer
  // for overwriting.
  auto take_w = [&]() __attribute__((always_inline)) {
    SZ rsz;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      w[i] = fw[i];
      asm volatile("" : "+v"(w[i]));
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int i = 0; i < NS / 2; ++i) {
        rsz.s[g][i] = fsz.s[g][i];
        rsz.z[g][i] = fsz.z[g][i];
        asm volatile("" : "+v"(rsz.s[g][i]), "+v"(rsz.z[g][i]));
      }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        union {
          uint32_t u;
          _Float16 h[2];
        } sv, zv;
        sv.u = rsz.s[g][j / 2];
        zv.u = rsz.z[g][j / 2];
        _Float16 sh = sv.h[j % 2], zh = zv.h[j % 2];
        if constexpr (BF16) {  // bfloat16 = top half of a float; the dequantisation runs in fp16
          sh = (_Float16)__uint_as_float((j % 2 ? sv.u >> 16 : sv.u & 0xFFFFu) << 16);
          zh = (_Float16)__uint_as_float((j % 2 ? zv.u >> 16 : zv.u & 0xFFFFu) << 16);
        }
        s2[g][j] = half2_{sh, sh};
        z2[g][j] = half2_{zh, zh};
      }
  };
  auto sync_and_issue = [&](int e, auto in_run, auto btag) __attribute__((always_inline)) {
    take_w();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // past the end the last tile is loaded again, into the idle buffer and the landing registers: same
    // load count on every path
    const int nn = min(e + 2, e_last);
    issue_x(nn, e);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(in_run)::value)
      issue_w_static(btag, nn, fw, fsz);
    else
      issue_w_generic(nn, fw, fsz);
    __builtin_amdgcn_sched_barrier(0);
  };
  const std::integral_constant<int, 0> k0;
  const std::integral_constant<int, 1> k1;
  const std::integral_constant<int, 2> k2;
  const std::integral_constant<int, 3> k3;

  // in_run: tiles e+1 and e+2 have the same width B as tile e
  auto step = [&](auto btag, auto in_run, int e) __attribute__((always_inline)) {
    // Two workgroups share a CU.  A wavefront inside the three groups that only compute is served before one that is
    // at the synchronisation point or in the group right after it (whose loads have just been issued): the matrix
    // pipe waits less on the other workgroup's bookkeeping (2-4 % measured, same box).
    __builtin_amdgcn_s_setprio(1);
    mfmas(a0, b0);
    read_a(e & 1, k1, a1);
    make_b(btag, k1, b1);
    interleave();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(a1, b1);
    read_a(e & 1, k2, a0);
    make_b(btag, k2, b0);
    interleave();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(a0, b0);
    read_a(e & 1, k3, a1);
    make_b(btag, k3, b1);
    interleave();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    sync_and_issue(e, in_run, btag);
    mfmas(a1, b1);
    read_a((e + 1) & 1, k0, a0);
    if constexpr (decltype(in_run)::value) {
      make_b(btag, k0, b0);
      interleave();
      __builtin_amdgcn_sched_barrier(0);
    } else {
      interleave();
      __builtin_amdgcn_sched_barrier(0);
      make_b_any(min(e + 1, e_last), k0, b0);
    }
  };

  const std::integral_constant<bool, true> in_run;
  const std::integral_constant<bool, false> run_ends;
  const std::integral_constant<int, 2> b2;
  const std::integral_constant<int, 3> b3;
  const std::integral_constant<int, 4> b4;
  // prologue: the first tile lands, then its k-step 0 is prepared while the second is on its way
  issue_x(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue_w_generic(0, fw, fsz);
  __builtin_amdgcn_sched_barrier(0);
  sync_and_issue(-1, std::integral_constant<bool, false>{}, k0);
  read_a(0, k0, a0);
  make_b_any(0, k0, b0);
  __builtin_amdgcn_sched_barrier(0);

  int e = 0;
  for (; e + 2 < end2; ++e) step(b2, in_run, e);
  for (; e < end2; ++e) step(b2, run_ends, e);
  for (; e + 2 < end3; ++e) step(b3, in_run, e);
  for (; e < end3; ++e) step(b3, run_ends, e);
  for (; e + 2 < p.ntc; ++e) step(b4, in_run, e);
  for (; e < p.ntc; ++e) step(b4, run_ends, e);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the idle loads of the last two steps
  // epilogue: the block goes through LDS (the activation buffers are free now) so that it leaves in whole
  // row segments: acc[i][j][r] = C[16i + 4kb + r][8*i16 + NS*wn + j], the NS values j of
  // a lane being consecutive columns.
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();  // every wavefront's idle loads have landed and its operand reads returned
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * i + 4 * kb + r;
      union {
        _Float16 h[NS];
        uint32_t u[NS / 2];
      } o;
#pragma unroll
      for (int j = 0; j < NS; ++j) o.h[j] = (_Float16)acc[i][j][r];
      uint32_t* dst = reinterpret_cast<uint32_t*>(Xs + row * 256 + (8 * i16 + NS * wn) * 2);
#pragma unroll
      for (int q = 0; q < NS / 2; ++q) dst[q] = o.u[q];
    }
  __syncthreads();
  _Float16* ybase = p.Yt + (int64_t)m0 * p.N + (int64_t)tr * 128;
#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    const int row = xrow + kRowsPerPass * i;
    const u32x4 v = *reinterpret_cast<const u32x4*>(Xs + row * 256 + xunit * 16);
    if (m0 + row < p.M) *reinterpret_cast<u32x4*>(ybase + (int64_t)row * p.N + xunit * 8) = v;
  }
}

// 16 bytes per lane of lane_mask from a full address per lane straight into LDS at lds_base + 16*lane.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lanes_to_lds_16(uint64_t vaddr, uint32_t lds_base, uint64_t lane_mask) {
  uint64_t saved;
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %3\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(vaddr), "s"(lds_base), "s"(lane_mask)
      : "memory", "m0");
}
#pragma clang diagnostic pop

// A workgroup owns one tile row and BM rows of the batch.  Eight wavefronts multiply, each MI x 16 rows by 32 columns (two
// slabs): KG = 2 - two K groups of four, each with half of the workgroup's tiles and its own buffers, their fp32 sums added in
// LDS at the end, BM = 16 MI; KG = 1 - two row groups of four on the same tiles, BM = 32 MI.  Four further wavefronts make all
// requests to memory: two bring the activations, in half blocks of 64 columns, two the packed words and parameters, one tile a
// slot.
// Why: one wavefront that requests, waits, dequantises and multiplies cannot overlap these with itself (with one workgroup of
// four per CU a 128-row tile took 2350 cycles for 1024 of matrix instructions), and every copy that it issues stops it
// while the copies of the other wavefronts are taken in (64 bytes a cycle and CU): the same loop with the copies in the multiplying
// wavefronts took 20 % longer at 777 x 4096 -> 4096 and its copies cost 11 of 48 us; here they cost 3.  The requests of words
// and of activations are separate wavefronts because requests complete in order: with one kind behind the other a step waited
// for the words, which come from further away (45.3 -> 41.7 thousand cycles for 16 steps).  Three buffers and slots cover
// 2 half steps and 2 tiles of latency.  What bounds it now: vector and matrix instructions share the issue of a SIMD (measured
// with two wavefronts and n vector instructions per 16x16x32 instruction: max(17.4, 4.3 n + 8.7) cycles), n is 2.1 at MI = 7
// and falls with MI; a step of two tiles takes 2100, 2550, 2640, 2760 cycles at MI = 4, 6, 7, 8 (128 MI of matrix instructions
// per wavefront and step, twice 256 MI per SIMD), 3300 pass before the tiles are laid out, 3600 until the first data is there
// and 4500 at the end.  With several full rounds of workgroups the chip's power limit lowers the clock instead (2048 x 28672 -> 8192:
// pipe 0.73 busy at 1.51 GHz); 2048 x 4096 -> 14336 loses half of its fourth round first (0.55 busy at 1.78 GHz).
// Whole calls back to back, the kernels before (whose wavefronts did all of this themselves) -> now: 777 x 4096 -> 4096 49.1 -> 37.7 us,
// 200 x 14336 -> 4096 (group length 64) 47.7 -> 39.3, 64 x 4096 -> 14336 22.6 -> 20.6, 2048 x 4096 -> 14336 266.7 -> 248.6 (a tail of smaller
// workgroups since, see PrefillMixed), 2048 x 28672 -> 8192 884.8 -> 818.0.
// MI = 8 reaches the 168 registers of 12 wavefronts.  prefill_fed_kernel<8, 1> spills 1 of them, 3 and 9 at group length 64 (fp16 and bf16
// parameters; there with reloads inside the tile loops), <8, 2> 7 and 2, 9 and 11; prefill_mixed_kernel<8>, which is both, 10 and 3, 14 and 20,
// <4> as many as <8, 1>.  The choice of the form does not know of it: calls with a tail gain as much at group length 64 (see choose_prefill_tail).
// Not better: 32x32x16 instructions (the words of two slabs exchanged between rows of 16 lanes): 2770 cycles where 16x16x32
// takes 2550, and 290 us instead of 253 on 2048 x 4096 -> 14336, where the clock falls further; the order of every phase fixed
// by hand (spills at 168 registers).
constexpr int kFedThreads = 768;
template <int MI, int KG, bool G64>
constexpr uint32_t fed_lds_bytes() { return KG * 3 * (16 * MI * (2 / KG) * 128 + (G64 ? 1024 : 512) + 8192); }

template <int MI, int KG, bool G64, bool BF16>
__device__ __forceinline__ void fed_body(const PrefillParams& p, const Place place, unsigned char* const lds, int32_t* const seq, int2* const counts) {
  constexpr int NB = 3, WS = 3, NS = 2, MG = 2 / KG, BM = 16 * MI * MG, kConsumers = 512, kThreads = kFedThreads;
  constexpr uint32_t kBuf = BM * 128;              // half a block: BM rows x 64 columns
  constexpr uint32_t kPar = G64 ? 1024 : 512;      // scales and zeros of a tile (twice at group length 64)
  constexpr uint32_t kSlot = kPar + 8192;          // and its packed words
  constexpr uint32_t kLds = KG * (NB * kBuf + WS * kSlot);
  // the end: sums of the K groups on their way to each other, then the rows
  constexpr uint32_t kOut = KG == 2 ? 8 * MI * 1024 : 0;
  static_assert(kOut + BM * (KG == 2 ? 512 : 256) <= kLds && kLds == fed_lds_bytes<MI, KG, G64>(), "the rows fit in the buffers");

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ks = place.ks, mt = place.mt, tr = place.tr;
  const int m0 = mt * BM;
  const int ranges = p.ksplit * KG;
  auto first_of = [&](int range) __attribute__((always_inline)) { return (int)((uint32_t)(range * p.ntc) / (uint32_t)ranges); };
  const int longest = (p.ntc + ranges - 1) / ranges;  // tiles of the longest share

  int end2 = 0, end3 = 0;
  lay_out_tiles<kThreads>(p, tr, counts, end2, end3, seq);
  __syncthreads();
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lptr_t)lds;

  if (wave >= kConsumers / kWave) {
    // ---- the wavefronts that bring everything in: two the activations, two the packed words and parameters, so that
    // neither waits for the other's requests (they complete in order)
    const int pw = (wave - kConsumers / kWave) % 2;
    int e0[KG], e1[KG];
#pragma unroll
    for (int g = 0; g < KG; ++g) e0[g] = first_of(ks * KG + g), e1[g] = first_of(ks * KG + g + 1) - 1;
    auto desc = [&](int g, int t) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(seq[min(e0[g] + t, e1[g])]); };
    auto wait_and_meet = [&](auto n) __attribute__((always_inline)) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(n)::value) : "memory");
      __builtin_amdgcn_s_barrier();
    };
    if (wave < kConsumers / kWave + 2) {
      // Copies of a half block: 8 rows x 128 bytes each, copy c (rows 8c ..) by wavefront c % 2.  Position u of row r receives
      // unit u ^ (r / 2 % 8).
      constexpr int C = BM / 16;
      const uint32_t xlane = (uint32_t)(lane / 8) * 256 + (uint32_t)(((lane & 7) ^ ((4 * pw + lane / 16) & 7)) * 16);
      const StagedRows<BM> staged(p.M, m0, (uint32_t)p.ntc * (uint32_t)(kTile * kTile * 2));
      const uint64_t xb64 = (uint64_t)p.Xp + (uint64_t)staged.base;
      // (a workgroup's rows may reach past the last block of 128: no request for a block that is not there)
      uint32_t xso[C], xrec[C];  // offset of a copy's rows, records
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const BlockRequest rows = staged.copy(8 * (2 * c + pw));
        xso[c] = rows.offset;
        xrec[c] = rows.records;
      }
      auto half_block = [&](int h, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < KG; ++g) {
          const bool wanted = e0[g] + (h >> 1) <= e1[g];  // (past the end: requests of nothing)
          const uint32_t so = ((uint32_t)(desc(g, h >> 1) & 511) << 15) + (uint32_t)(h & 1) * 128;
          const uint32_t dst = lds_base + (uint32_t)g * (NB * kBuf) + (uint32_t)buf * kBuf + (uint32_t)pw * 1024;
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const BlockRequest x = block_request(so + xso[c], xrec[c], wanted);
            const u32x4 rsrc = {(uint32_t)xb64, (uint32_t)(xb64 >> 32), x.records, 0x00020000u};
            load_to_lds_16(rsrc, x.offset, xlane, dst + c * 2048);
          }
        }
      };
      // (the first half block alone: behind the bursts of all workgroups' further requests it arrived 3000 cycles later)
      half_block(0, 0);
      wait_and_meet(std::integral_constant<int, 0>{});
      half_block(1, 1);
      half_block(2, 2);
      int buf = 0;
      for (int h = 0; h < 2 * longest; ++h) {
        // half block h has been read; h + 1 has landed once only h + 2 is outstanding
        wait_and_meet(std::integral_constant<int, KG * C>{});
        half_block(h + 3, buf);
        buf = buf == 2 ? 0 : buf + 1;
      }
    } else {
      // KG == 2: a wavefront per K group; else half of the words each
      constexpr int kWords = KG == 2 ? 8 : 4, kReq = kWords + 1;
      const int g = KG == 2 ? pw : 0;
      const int first = KG == 2 ? 0 : pw * 4096;
      const uint32_t lane16 = (uint32_t)(first + lane * 16);
      // parameters: 16 bytes per lane, [scales 256 bytes | zeros 256 bytes] per parameter row
      constexpr int kParLanes = (G64 ? 64 : 32) / (KG == 2 ? 1 : 2);
      const int pl = (KG == 2 ? 0 : pw * kParLanes) + lane % kParLanes;
      const uint64_t par_lane = ((pl & 16) ? (uint64_t)p.zeros : (uint64_t)p.scales) + (uint64_t)(tr * 256 + (pl & 15) * 16) +
                                (uint64_t)(pl >> 5) * (uint64_t)(2 * p.N);
      const uint64_t par_mask = kParLanes == 64 ? ~0ull : (1ull << (kParLanes % 64)) - 1;
      auto words = [&](int t, int slot) __attribute__((always_inline)) {
        const int32_t d = desc(g, t);
        const int e = min(e0[g] + t, e1[g]);  // (past the end: the last tile again)
        const uint32_t bw = e < end2 ? 2u : e < end3 ? 3u : 4u;
        const uint64_t src = (bw == 2 ? (uint64_t)p.s2 : bw == 3 ? (uint64_t)p.s3 : (uint64_t)p.s4) + (uint64_t)((uint32_t)d >> 9) * (2048u * bw);
        const u32x4 rsrc = {(uint32_t)src, (uint32_t)(src >> 32) & 0xFFFFu, 2048u * bw, 0x00020000u};
        const uint32_t dst = lds_base + KG * (NB * kBuf) + (uint32_t)(g * WS + slot) * kSlot;
        const uint32_t tc = (uint32_t)d & 511u;
        load_lanes_to_lds_16(par_lane + (uint64_t)((G64 ? 2 * tc : tc >> p.gshift) * (uint32_t)(2 * p.N)), dst + (KG == 2 ? 0 : pw * (kParLanes * 16)), par_mask);
#pragma unroll
        for (int c = 0; c < kWords; ++c) load_to_lds_16(rsrc, 0u, lane16 + c * 1024, dst + kPar + first + c * 1024);
      };
      words(0, 0);
      wait_and_meet(std::integral_constant<int, 0>{});
      words(1, 1);
      words(2, 2);
      int slot = 0;
      for (int t = 0; t < longest; ++t) {
        // the words of tile t have been read; those of t + 1 have landed once only t + 2 is outstanding
        wait_and_meet(std::integral_constant<int, kReq>{});
        words(t + 3, slot);
        slot = slot == 2 ? 0 : slot + 1;
        __builtin_amdgcn_s_barrier();
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  } else {
    // ---- the wavefronts that multiply
    const int kg = KG > 1 ? wave / 4 : 0, wm = KG > 1 ? 0 : wave / 4, wn = wave % 4;
    const int i16 = lane % 16, kb = lane / 16;
    const int e_first = first_of(ks * KG + kg), e_end = first_of(ks * KG + kg + 1), e_last = e_end - 1;
    const unsigned char* const Xs = lds + kg * (NB * kBuf);
    const unsigned char* const Ws = lds + KG * (NB * kBuf) + kg * (WS * kSlot);
    uint32_t magic;
    asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(magic));
    uint32_t aoff[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) aoff[k] = (uint32_t)((16 * MI * wm + i16) * 128 + (((4 * k + kb) ^ (i16 >> 1)) * 16));
    // a: the operands of this k-step, replaced by the next one's as the last matrix instruction that reads them is issued; b[1]
    // is made while b[0] is multiplied and the other way round; wnext: the words of the next tile
    half8 a[MI], b[NS];
    u32x4 w[NS], wnext[NS];
    constexpr int NG = G64 ? 2 : 1;
    uint32_t rs[NG], rz[NG];
    half2_ s2[NS], z2[NS];
    floatx4 acc[MI][NS];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NS; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto read_a = [&](auto ktag, int buf, int i) __attribute__((always_inline)) {
      a[i] = *reinterpret_cast<const half8*>(Xs + (uint32_t)buf * kBuf + aoff[decltype(ktag)::value & 1] + i * 2048);
    };
    auto read_w = [&](auto in_run, auto btag, int e, int slot) __attribute__((always_inline)) {
      constexpr int B = decltype(btag)::value;
      const unsigned char* base = Ws + (uint32_t)slot * kSlot;
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        if constexpr (decltype(in_run)::value) {
          const uint32_t* s = reinterpret_cast<const uint32_t*>(base + kPar + (NS * wn + j) * (256 * B) + lane * (4 * B));
          if constexpr (B == 4)
            wnext[j] = *reinterpret_cast<const u32x4*>(s);
          else if constexpr (B == 3)
            wnext[j] = u32x4{s[0], s[1], s[2], 0u};
          else {
            const u32x2 v = *reinterpret_cast<const u32x2*>(s);
            wnext[j] = u32x4{v[0], v[1], 0u, 0u};
          }
        } else {
          const int bw = e < end2 ? 2 : e < end3 ? 3 : 4;
          const uint32_t* s = reinterpret_cast<const uint32_t*>(base + kPar + (NS * wn + j) * (256 * bw) + lane * (4 * bw));
          wnext[j] = u32x4{s[0], s[1], s[min(2, bw - 1)], s[bw - 1]};
        }
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        rs[g] = *reinterpret_cast<const uint32_t*>(base + g * 512 + (8 * i16 + NS * wn) * 2);
        rz[g] = *reinterpret_cast<const uint32_t*>(base + g * 512 + 256 + (8 * i16 + NS * wn) * 2);
      }
    };
    auto convert = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        union {
          uint32_t u;
          _Float16 h[2];
        } sv, zv;
        sv.u = rs[g];
        zv.u = rz[g];
        _Float16 sh = sv.h[j], zh = zv.h[j];
        if constexpr (BF16) {
          sh = (_Float16)__uint_as_float((j ? sv.u >> 16 : sv.u & 0xFFFFu) << 16);
          zh = (_Float16)__uint_as_float((j ? zv.u >> 16 : zv.u & 0xFFFFu) << 16);
        }
        s2[j] = half2_{sh, sh};
        z2[j] = half2_{zh, zh};
      }
    };
    auto make_b = [&](auto btag, auto ktag, int j) __attribute__((always_inline)) {
      const uint32_t words[4] = {w[j][0], w[j][1], w[j][2], w[j][3]};
      b[j] = dequant_operand<decltype(btag)::value, decltype(ktag)::value>(words, s2[j], z2[j], magic);
    };
    const std::integral_constant<int, 0> k0;
    const std::integral_constant<int, 1> k1;
    const std::integral_constant<int, 2> k2;
    const std::integral_constant<int, 3> k3;
    const std::integral_constant<bool, true> yes;
    const std::integral_constant<bool, false> no;
    const std::integral_constant<int, 2> b2;
    const std::integral_constant<int, 3> b3;
    const std::integral_constant<int, 4> b4;
    auto make_first_any = [&](int e) __attribute__((always_inline)) {
      if (e < end2)
        make_b(b2, k0, 0);
      else if (e < end3)
        make_b(b3, k0, 0);
      else
        make_b(b4, k0, 0);
    };
    auto interleave = [&](auto nds_tag, auto nv_tag) __attribute__((always_inline)) {
      constexpr int nds = decltype(nds_tag)::value, nv = decltype(nv_tag)::value, per = (nv + MI - 1) / MI;
#pragma unroll
      for (int g = 0; g < MI; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (g < nds) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (per > 0) __builtin_amdgcn_sched_group_barrier(0x002, per, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // Synchronisation point, once per half block: everything that this wavefront reads of it has returned
    auto sync = [&]() __attribute__((always_inline)) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    int xb = 0, slot = 0;
    auto ring3 = [](int v) __attribute__((always_inline)) { return v >= 3 ? v - 3 : v; };
    auto tile_step = [&](auto btag, auto in_run, int e) __attribute__((always_inline)) {
      const int bufA = xb, bufB = ring3(xb + 1), bufN = ring3(xb + 2);
      const int slot1 = ring3(slot + 1);
      auto phase = [&](auto ktag, auto jtag) __attribute__((always_inline)) {
        constexpr int k = decltype(ktag)::value, j = decltype(jtag)::value;
        constexpr bool last = k == 3 && j == 1;  // the operand made here belongs to the next tile
        constexpr int kn = (k + 1) % 4;
        const std::integral_constant<int, kn> knext;
        const int bufn = kn == 0 ? bufN : kn == 1 ? bufA : bufB;
        if constexpr (k == 2 && j == 1) read_w(in_run, btag, min(e + 1, e_last), slot1);
        if constexpr (G64 && k == 1 && j == 1) convert(1);
        if constexpr (last) {
#pragma unroll
          for (int q = 0; q < NS; ++q) w[q] = wnext[q];
          convert(0);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[j], acc[i][j], 0, 0, 0);
        if constexpr (j == 1) {
#pragma unroll
          for (int i = 0; i < MI; ++i) read_a(knext, bufn, i);
        }
        const std::integral_constant<int, j == 1 ? MI : 0> ds;
        if constexpr (j == 0) {
          make_b(btag, ktag, 1);
          interleave(ds, std::integral_constant<int, 14>{});
        } else if constexpr (!last || decltype(in_run)::value) {
          make_b(btag, knext, 0);
          interleave(ds, std::integral_constant<int, last ? 22 : 14>{});
        } else {
          interleave(ds, std::integral_constant<int, 0>{});
        }
        if constexpr (k % 2 == 1 && j == 0) sync();
      };
      phase(k0, k0);
      phase(k0, k1);
      phase(k1, k0);
      phase(k1, k1);
      phase(k2, k0);
      phase(k2, k1);
      phase(k3, k0);
      phase(k3, k1);
      if constexpr (!decltype(in_run)::value) make_first_any(min(e + 1, e_last));
      xb = bufN;
      slot = slot1;
    };
    __builtin_amdgcn_s_barrier();  // the first half block and the first words have landed
    asm volatile("" ::: "memory");
    read_w(no, k0, e_first, 0);
#pragma unroll
    for (int q = 0; q < NS; ++q) w[q] = wnext[q];
#pragma unroll
    for (int i = 0; i < MI; ++i) read_a(k0, 0, i);
    convert(0);
    make_first_any(e_first);
    __builtin_amdgcn_sched_barrier(0);
    const int r2 = min(max(end2, e_first), e_end), r3 = min(max(end3, e_first), e_end);
    int e = e_first;
    for (; e + 1 < r2; ++e) tile_step(b2, yes, e);
    for (; e < r2; ++e) tile_step(b2, no, e);
    for (; e + 1 < r3; ++e) tile_step(b3, yes, e);
    for (; e < r3; ++e) tile_step(b3, no, e);
    for (; e + 1 < e_end; ++e) tile_step(b4, yes, e);
    for (; e < e_end; ++e) tile_step(b4, no, e);
    // every wavefront of the workgroup passes the same number of barriers
    for (int n = e_end - e_first; n < longest; ++n) {
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // acc[i][j][r] = C[16*MI*wm + 16i + 4kb + r][8*i16 + 2*wn + j].  Two K groups: the first adds up rows r = 0, 1 of every four,
    // the second 2, 3, so that each gives away half of its sums through LDS and not all of them.
    constexpr int kOwn = 4 / KG;
    float own[MI][kOwn][NS];
    if constexpr (KG == 2) {
      unsigned char* const give = lds + ((kg ^ 1) * 4 + wn) * (MI * 1024) + lane * 16;
      const unsigned char* const take = lds + (kg * 4 + wn) * (MI * 1024) + lane * 16;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const floatx4 lo = {acc[i][0][0], acc[i][1][0], acc[i][0][1], acc[i][1][1]};
        const floatx4 up = {acc[i][0][2], acc[i][1][2], acc[i][0][3], acc[i][1][3]};
        *reinterpret_cast<floatx4*>(give + i * 1024) = kg == 0 ? up : lo;
#pragma unroll
        for (int q = 0; q < 4; ++q) own[i][q / 2][q % 2] = kg == 0 ? lo[q] : up[q];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const floatx4 t = *reinterpret_cast<const floatx4*>(take + i * 1024);
#pragma unroll
        for (int q = 0; q < 4; ++q) own[i][q / 2][q % 2] += t[q];
      }
    } else {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int q = 0; q < kOwn * 2; ++q) own[i][q / 2][q % 2] = acc[i][q % 2][q / 2];
    }
    // The rows in LDS; the slots of the four wavefronts inside a unit of 8 columns change places by kb, so that the rows of
    // one instruction hit different banks.
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < kOwn; ++q) {
        const int row = 16 * MI * wm + 16 * i + 4 * kb + kOwn * kg + q, at = 4 * i16 + (wn ^ kb);
        if (KG == 1 || p.ksplit == 1) {
          union {
            _Float16 h[2];
            uint32_t u;
          } o;
          o.h[0] = (_Float16)own[i][q][0], o.h[1] = (_Float16)own[i][q][1];
          *reinterpret_cast<uint32_t*>(lds + kOut + row * 256 + at * 4) = o.u;
        } else {
          *reinterpret_cast<float2*>(lds + kOut + row * 512 + at * 8) = float2{own[i][q][0], own[i][q][1]};
        }
      }
  }
  if (KG == 2 && wave >= kConsumers / kWave) __syncthreads();
  __syncthreads();
  constexpr int kRows = kThreads / 16;
  const int prow = tid / 16, pu = tid % 16;
  const unsigned char* const out = lds + kOut;
  for (int row = prow; row < BM && m0 + row < p.M; row += kRows) {
    const int f = (row >> 2) & 3;
    if (KG == 1 || p.ksplit == 1) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(out + row * 256 + pu * 16);
      const u32x4 x = f & 1 ? u32x4{v[1], v[0], v[3], v[2]} : v;
      *reinterpret_cast<u32x4*>(p.Yt + (int64_t)(m0 + row) * p.N + (int64_t)tr * 128 + pu * 8) = f & 2 ? u32x4{x[2], x[3], x[0], x[1]} : x;
    } else {
      const floatx4 v = *reinterpret_cast<const floatx4*>(out + row * 512 + pu * 32), u = *reinterpret_cast<const floatx4*>(out + row * 512 + pu * 32 + 16);
      const floatx4 x = f & 1 ? floatx4{v[2], v[3], v[0], v[1]} : v, y = f & 1 ? floatx4{u[2], u[3], u[0], u[1]} : u;
      float* dst = p.partial + ((int64_t)ks * p.M + m0 + row) * p.N + (int64_t)tr * 128 + 8 * pu;
      reinterpret_cast<floatx4*>(dst)[0] = f & 2 ? y : x;
      reinterpret_cast<floatx4*>(dst)[1] = f & 2 ? x : y;
    }
  }
}

// The arguments that a workgroup needs for its place, in one request: each one that waits for the one before is 0.05 us of a call.
__device__ __forceinline__ Place place_of(WorkItems items, const uint32_t block, const int32_t ntr, const int32_t ksplit) {
  asm volatile("" : "+s"(items.whole), "+s"(items.by_ranges), "+s"(items.by_group), "+s"(items.last.by), "+s"(items.last.inverse));
  return items.place(block, (uint32_t)ntr, (uint32_t)ksplit);
}

// M blocks inside tile rows, as in prefill_kernel, in launches of many rounds eight at a time (see order_of)
template <int MI, int KG, bool G64, bool BF16>
__global__ __launch_bounds__(kFedThreads, 3) void prefill_fed_kernel(const PrefillParams p) {
  __shared__ __align__(16) unsigned char lds[fed_lds_bytes<MI, KG, G64>()];
  __shared__ int32_t seq[kPrefillMaxTiles];
  __shared__ int2 counts[kFedThreads / kWave];
  fed_body<MI, KG, G64, BF16>(p, place_of(p.items, blockIdx.x, p.ntr, p.ksplit), lds, seq, counts);
}

// The same in two forms: whole rounds of workgroups of 256 rows on the first tile rows, and smaller workgroups (MI = 4 or 8 in
// two K groups: 64 or 128 rows) on the last ones, where the large ones would leave part of a round empty.  The tail follows in
// the same launch: a CU takes its first piece of it when it is done with its last large one.
struct PrefillMixed {
  PrefillParams p;      // ntr: tile rows of the large workgroups
  WorkItems tail;       // order of the others
  int32_t tail_ntr;
  uint32_t large;       // number of large workgroups
};
template <int MI, bool G64, bool BF16>
__global__ __launch_bounds__(kFedThreads, 3) void prefill_mixed_kernel(const PrefillMixed m) {
  constexpr uint32_t kLarge = fed_lds_bytes<8, 1, G64>(), kTail = fed_lds_bytes<MI, 2, G64>();
  __shared__ __align__(16) unsigned char lds[kLarge > kTail ? kLarge : kTail];
  __shared__ int32_t seq[kPrefillMaxTiles];
  __shared__ int2 counts[kFedThreads / kWave];
  if (blockIdx.x < m.large) {
    fed_body<8, 1, G64, BF16>(m.p, place_of(m.p.items, blockIdx.x, m.p.ntr, 1), lds, seq, counts);
  } else {
    Place place = place_of(m.tail, blockIdx.x - m.large, m.tail_ntr, 1);
    place.tr += m.p.ntr;
    fed_body<MI, 2, G64, BF16>(m.p, place, lds, seq, counts);
  }
}

static WorkItems order_of(int32_t ntr, int32_t n_mtiles, int32_t ksplit) {
  // Block b runs on XCD b % 8.  With all M blocks inside a tile row every XCD sees every one of them unless their number is a
  // multiple of eight, and from about 20 on a round takes the time of its activations from the memory-side cache (64 KiB per
  // workgroup and tile of 256 rows: 2.15 us a tile where 1.5 are spent multiplying, and prefill_kernel was the faster one by up
  // to 10 %).  In groups of eight an XCD keeps one M block, and its workgroups share what one of them has fetched (prefill_kernel /
  // one order / groups): 8714 x 2176 -> 7936 453 / 475 / 371 us, 5000 x 14336 -> 4096 664 / 731 / 606, 30248 x 1664 -> 13952 2133 / 2250 /
  // 1774, 5000 x 8192 -> 28672 2445 / 2336 / 2157.
  // Not with one round of workgroups, nor with two and up to 16 blocks, where the weights that come once more for every group cost up to
  // 4 %, nor with a multiple of eight (up to 2 %).
  const unsigned blocks = (unsigned)n_mtiles, grid = blocks * (unsigned)ntr * (unsigned)ksplit;
  const bool grouped = blocks % kMGroup != 0 && blocks > (grid > 512 ? kMGroup : 2 * kMGroup) && grid > 256;
  return work_items((unsigned)ntr, blocks, (unsigned)ksplit, grouped);
}

template <int MI, int KG>
static void launch_fed(PrefillParams p, int M, bool g64, bool bf16, hipStream_t stream) {
  constexpr int BM = 16 * MI * (2 / KG);
  p.n_mtiles = (M + BM - 1) / BM;
  const unsigned grid = (unsigned)p.n_mtiles * (unsigned)p.ntr * (unsigned)p.ksplit;
  p.items = order_of(p.ntr, p.n_mtiles, p.ksplit);
  if (g64 && bf16)
    hipLaunchKernelGGL((prefill_fed_kernel<MI, KG, true, true>), dim3(grid), dim3(768), 0, stream, p);
  else if (g64)
    hipLaunchKernelGGL((prefill_fed_kernel<MI, KG, true, false>), dim3(grid), dim3(768), 0, stream, p);
  else if (bf16)
    hipLaunchKernelGGL((prefill_fed_kernel<MI, KG, false, true>), dim3(grid), dim3(768), 0, stream, p);
  else
    hipLaunchKernelGGL((prefill_fed_kernel<MI, KG, false, false>), dim3(grid), dim3(768), 0, stream, p);
}

template <int MI>
static void launch_mixed(PrefillParams p, int M, int tail_rows, bool g64, bool bf16, hipStream_t stream) {
  PrefillMixed m;
  p.ksplit = 1, p.partial = nullptr;  // (both sizes go over the whole K and leave no partial products)
  p.ntr -= tail_rows;
  p.n_mtiles = (M + 255) / 256;
  p.items = order_of(p.ntr, p.n_mtiles, 1);
  const int32_t tail_blocks = (M + 16 * MI - 1) / (16 * MI);
  m.tail = order_of(tail_rows, tail_blocks, 1);
  m.tail_ntr = tail_rows;
  m.large = (uint32_t)p.n_mtiles * (uint32_t)p.ntr;
  m.p = p;
  const dim3 grid(m.large + (unsigned)tail_blocks * (unsigned)tail_rows), threads(kFedThreads);
  if (g64 && bf16)
    hipLaunchKernelGGL((prefill_mixed_kernel<MI, true, true>), grid, threads, 0, stream, m);
  else if (g64)
    hipLaunchKernelGGL((prefill_mixed_kernel<MI, true, false>), grid, threads, 0, stream, m);
  else if (bf16)
    hipLaunchKernelGGL((prefill_mixed_kernel<MI, false, true>), grid, threads, 0, stream, m);
  else
    hipLaunchKernelGGL((prefill_mixed_kernel<MI, false, false>), grid, threads, 0, stream, m);
}

static void launch_plain(PrefillParams p, int M, bool g64, bool bf16, hipStream_t stream) {
  p.n_mtiles = (M + 127) / 128;
  const dim3 grid((unsigned)p.n_mtiles * (unsigned)p.ntr), threads(256);
  if (g64 && bf16)
    hipLaunchKernelGGL((prefill_kernel<true, true>), grid, threads, 0, stream, p);
  else if (g64)
    hipLaunchKernelGGL((prefill_kernel<true, false>), grid, threads, 0, stream, p);
  else if (bf16)
    hipLaunchKernelGGL((prefill_kernel<false, true>), grid, threads, 0, stream, p);
  else
    hipLaunchKernelGGL((prefill_kernel<false, false>), grid, threads, 0, stream, p);
}

// The number of K ranges that the workspace query documents: with few workgroups (blocks of 128 rows, or of 64 where those would
// leave half of the CUs without one) ranges of at least 8 tiles, up to two workgroups per CU, with fp32 partial products and
// a reduction pass in a fixed order.
static int32_t documented_ranges(int32_t N, int32_t K, int32_t M) {
  const int64_t ntr = N / kTile, ntc = K / kTile;
  const int64_t bm = (int64_t)((M + 127) / 128) * ntr <= 128 ? 64 : 128;
  const int64_t blocks = (int64_t)((M + bm - 1) / bm) * ntr;
  int64_t ks = 1;
  if (blocks <= 256) {
    ks = 512 / blocks;
    if (ks > ntc / 8) ks = ntc / 8;
    if (ks > 8) ks = 8;
    if (ks < 3 && ntc < 64) ks = 1;  // two ranges of a short K measured between -5 and +6 %; of a long K +20 %
  }
  return (int32_t)ks;
}

PrefillWorkspace prefill_workspace(int32_t N, int32_t K, int32_t M) {
  const int64_t ks = documented_ranges(N, K, M);
  PrefillWorkspace d;
  d.xperm_bytes = round_up_256((int64_t)((M + kTile - 1) / kTile) * kTile * K * 2);  // whole 128-row blocks
  d.ytmp_bytes = round_up_256(ks > 1 ? ks * (int64_t)M * N * 4 : (int64_t)M * N * 2);
  return d;
}

// Time of a call in us: rounds of workgroups on 256 CUs (one per CU), each the steps of its longest share times the time of a
// step, longer from the second round on (the clock falls), plus start and end; the staging pass, and the last pass over fp16
// rows or over the partial products of the ranges.  A fit to 127748 calls (9000 random shapes, M = 17 ... 2048, K and N from 512
// to 28672, every group length and parameter format, every form and number of ranges of each), which it meets within 5.2 %
// (rms).
static double fed_time_us(int32_t N, int32_t K, int32_t M, int32_t mi, int32_t kg, int32_t ks) {
  const int64_t ntr = N / kTile, ntc = K / kTile, bm = 16 * mi * (2 / kg), groups = (int64_t)kg * ks;
  const int64_t rounds = ((M + bm - 1) / bm * ntr * ks + 255) / 256;
  const double steps = (double)((ntc + groups - 1) / groups);
  const double first = kg == 2 ? 0.535 + 0.087 * mi : 0.49 + 0.083 * mi;
  const double later = kg == 2 ? 0.562 + 0.14 * mi : 0.56 + 0.113 * mi;
  const double mn = (double)M * N * 1e-6, mk = (double)M * K * 1e-6;
  return 8.85 + steps * (first + (double)(rounds - 1) * later) + (double)rounds * (kg == 2 ? 0.167 : 0.06) * mi + 0.904 * mk +
         (ks == 1 ? 1.873 * mn : 0.79 + 3.055 * ks * mn);
}

// The same for prefill_kernel with more than 256 workgroups (two per CU), a fit to 1675 calls (5.8 % rms).
static double plain_time_us(int32_t N, int32_t K, int32_t M) {
  const int64_t per_cu = ((int64_t)((M + 127) / 128) * (N / kTile) + 255) / 256, full = per_cu / 2, rest = per_cu % 2;
  return 11.825 + (double)(K / kTile) * (1.486 + 1.801 * (double)(full - 1) + 1.29 * (double)rest) + 1.292e-6 * M * K + 1.615e-6 * M * N;
}

// The fastest form by these times, in no more ranges than the workspace query documents.  On 6640 random shapes that were in
// no fit this choice is 13.3 % faster than the kernels before it (whose wavefronts all requested and multiplied, in blocks of 64
// and 128 rows; geometric mean; 14.0 % with the fastest form of each), and more than 2 % slower on 0.4 % of them.  prefill_kernel where it is estimated less than 3 % slower: with
// a little more than a multiple of 256 workgroups the last round of the others is nearly empty (631 x 3072 -> 23936, 118.7
// us against 125.6; without it 0.75 % of the shapes are more than 2 % slower), and not beyond the 2048 rows of the fits (on 300
// shapes with 1024 to 32768 rows it was never the faster one by more than 2 %).  One K group where a workgroup has a single tile.
static PrefillForm choose_form(int32_t N, int32_t K, int32_t M, double* time_us) {
  const int64_t ntr = N / kTile, ntc = K / kTile;
  const int32_t most = documented_ranges(N, K, M);
  PrefillForm best = {4, 1, 1};
  double least = -1.0;
  for (int32_t kg = 1; kg <= 2; ++kg)
    for (int32_t mi = 4; mi <= 8; ++mi)
      for (int32_t k = 1; k <= (kg == 1 ? 1 : most); ++k) {
        if (kg == 2 && ntc < (k == 1 ? 2 : 4 * k)) continue;                                         // at least a tile per group
        if (k > 1 && (int64_t)((M + 16 * mi - 1) / (16 * mi)) * ntr * k > 512) continue;  // (not measured)
        if (kg == 1 && M <= 64 && ntc >= 2) continue;                                                // half of the rows not there
        const double t = fed_time_us(N, K, M, mi, kg, k);
        if (least < 0.0 || t < least) least = t, best = PrefillForm{mi, kg, k};
      }
  *time_us = least;
  if (M <= 2048 && (int64_t)((M + 127) / 128) * ntr > 256 && plain_time_us(N, K, M) < 1.03 * least) best = PrefillForm{0, 1, 1};
  return best;
}

PrefillForm choose_prefill_form(int32_t N, int32_t K, int32_t M) {
  double t;
  return choose_form(N, K, M, &t);
}

// Time of a call in several rounds of workgroups of one form: a fit to 809 calls (M = 257 ... 2048, K and N from 512 to 28672,
// more than 256 workgroups of 256 rows), 3.5 and 4.1 % rms where fed_time_us, which has to place every form and K range of the
// shorter ones too, is 8 % off.
static double rounds_time_us(int32_t N, int32_t K, int32_t M, const PrefillForm& f) {
  if (f.mi == 0) return plain_time_us(N, K, M);
  const int64_t bm = 16 * f.mi * (2 / f.kg), rounds = ((M + bm - 1) / bm * (N / kTile) + 255) / 256;
  const double steps = (double)((K / kTile + f.kg - 1) / f.kg), mn = (double)M * N * 1e-6, mk = (double)M * K * 1e-6;
  if (f.kg == 2) return 8.0 + steps * (double)rounds * (0.458 + 0.147 * f.mi) + 1.10 * mk + 2.50 * mn;
  return 10.1 + steps * (0.402 + 0.119 * f.mi + (double)(rounds - 1) * (0.541 + 0.137 * f.mi)) + 1.84 * mk + 1.29 * mn;
}

// Rounds that `pieces` workgroups behind `large` ones take when the large ones fill up to `whole` rounds.  Workgroup b runs on XCD b % 8,
// whose 32 CUs share what falls to it and nothing else: a CU without a large workgroup in the last whole round takes `early` pieces
// meanwhile, of its own XCD only.  (Counted over the chip, 256 pieces beside a few early ones on some of the XCDs passed for one round:
// 1524 x 1792 -> 6784 64.9 us with a tail, 58.9 without; 1354 x 6016 -> 6912 156 and 145.)
static int64_t tail_rounds(int64_t large, int64_t pieces, int64_t whole, int64_t early) {
  int64_t rounds = 0;
  for (int64_t xcd = 0; xcd < 8; ++xcd) {
    const int64_t here = (large + 7 - xcd) / 8, left = (large + pieces + 7 - xcd) / 8 - here - early * (32 * whole - here);
    if (left > 0 && (left + 31) / 32 > rounds) rounds = (left + 31) / 32;
  }
  return rounds;
}

// Whole rounds of 256-row workgroups and a tail of smaller ones (see PrefillMixed).  Up to four whole rounds and 2048 rows, where
// its time was fitted (1000 calls of each tail, 3.3 and 4.0 % rms), and where that is below 0.945 of the form's own: of these calls
// 13 % take it, which are 5.8 % faster in the geometric mean (up to 14 %), and 0.3 % are more than 2 % slower (with 0.97 for 0.945 20 %,
// 4.1 % faster, and 1.5 % slower).  300 other calls that take it, in every format: 6.0 % faster with fp16 and 7.0 % with bf16 parameters, 6.7 and
// 5.8 % at group length 64 (where the merged kernel spills more); 5 to 7 % of them, 0.8 % of all, more than 2 % slower, up to 9 %, nearly
// all with a single whole round of a long K.  2048 x 4096 -> 14336, three and a half rounds, 255.3 -> 245.7 us (252.4 -> 248.1 on another
// machine); 1970 x 13184 -> 4736 302 -> 265; 1442 x 6912 -> 12928 293 -> 270; 510 x 5504 -> 19840 134 -> 118.
PrefillTail choose_prefill_tail(int32_t N, int32_t K, int32_t M) {
  PrefillTail best = {0, 0};
  const int64_t ntr = N / kTile, ntc = K / kTile, blocks = (M + 255) / 256, full = blocks * ntr / 256;
  if (M <= 256 || M > 2048 || full == 0 || full > 4 || blocks * ntr % 256 == 0 || ntc < 4) return best;
  // the last tile rows, those that do not fit in the whole rounds
  const int64_t rows = ntr - 256 * full / blocks, steps = (ntc + 1) / 2;
  const double mn = (double)M * N * 1e-6, mk = (double)M * K * 1e-6;
  const PrefillForm one = choose_prefill_form(N, K, M);
  if (one.ksplit != 1) return best;  // (never: K ranges are for 256 workgroups and fewer, of at most 128 rows)
  double least = 0.945 * rounds_time_us(N, K, M, one);
  for (int32_t mi = 4; mi <= 8; mi += 4) {
    const int64_t pieces = (M + 16 * mi - 1) / (16 * mi) * rows;
    const double rounds = (double)tail_rounds(blocks * (ntr - rows), pieces, full, mi == 4 ? 2 : 1);
    const double t = mi == 4 ? 10.55 + (double)ntc * (1.436 + 1.669 * (double)(full - 1)) + rounds * (1.125 * (double)steps + 1.82) + 1.51 * mk + 1.33 * mn
                             : 10.19 + (double)ntc * (1.249 + 1.655 * (double)(full - 1)) + rounds * (1.812 * (double)steps + 3.55) + 1.95 * mk + 1.33 * mn;
    if (t < least) least = t, best = PrefillTail{mi, (int32_t)rows};
  }
  return best;
}

double matrix_core_time_us(int32_t N, int32_t K, int32_t M) {
  double t;
  choose_form(N, K, M, &t);
  return t;
}

static int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    note_hip_error(what, hipGetErrorString(e));
    return SFMP_ERR_HIP;
  }
  return SFMP_OK;
}

// Threads of a workgroup that permutes a row of `columns`: up to 1024, the units of 8 columns evenly among them; with fewer rows
// than two workgroups per CU as many as there are units (57 x 25856 -> 4352 30.8 us with 1024 threads, 31.3 with 832; staging passes of 150 rows
// of 8320 to 28672 columns 0.1 us shorter, 300 to 2048 rows within 1 % either way but 1000 x 8320, 29.2 and 29.9).
static unsigned pass_threads(int32_t columns, int32_t rows) {
  const int32_t units = columns / 8, each = rows < 512 ? 1 : (units + 1023) / 1024;
  const int32_t threads = ((units + each - 1) / each + kWave - 1) / kWave * kWave;
  return (unsigned)(threads < 1024 ? threads : 1024);
}

// Of the un-permute pass: 256 from 512 rows on up to 10240 columns.  256 -> pass_threads, calls with K = 512 of 1024 to 28672 columns: up to
// 420 rows never longer and shorter from 3072 columns on (150 x 8192 12.6 -> 12.3 us, 300 x 14336 19.4 -> 19.0, 200 x 28672 25.1 -> 22.9); from 520
// rows on longer by up to 3 % between 6144 and 10240 columns (520 x 6144 16.8 -> 17.2, 520 x 10240 22.5 -> 23.2, 777 x 6144 20.3 -> 20.7), within
// noise up to 20480 and shorter beyond (1024 x 28672 73.8 -> 71.3, 2048 x 28672 154.8 -> 149.5).
int32_t scatter_threads(int32_t N, int32_t M) { return M >= 512 && N <= 10240 ? 256 : (int32_t)pass_threads(N, M); }

// Does the un-permute pass store its result past the caches?  A call alone is 0 to 2 us shorter for it at any size, but whatever
// reads the result next then takes it from memory: it counts what the two take together.  That is shorter once the result and the
// product before the un-permute, which this pass reads, do not fit in the 256 MiB of the memory-side cache together.  The call
// followed by an addition to another matrix / by a multiplication in place, past the caches -> through them: 777 x 2048 -> 14336 (22 MB)
// 77.6 -> 77.3 / 75.9 -> 75.3 us, 2048 x 4096 -> 4096 followed by a product with its result 108.0 -> 106.6, 2048 x 4096 -> 14336 (59 MB) 275.7 -> 274.4 /
// 267.4 -> 265.3, 2048 x 512 -> 28672 (117 MB) 211 -> 216 / 186 -> 183; 16384 x 1024 -> 4096 (134 MB) 294 -> 309 / 266 -> 279, 4096 x 1024 ->
// 28672 (235 MB) 467 -> 491 / 440 -> 449, the call alone 335 -> 373.
bool stores_past_caches(int32_t N, int32_t M) { return 2 * ((int64_t)M * N * 2) >= (int64_t)256 << 20; }

int launch_prefill(const GemmArgs& a, void* stream) {
  const sfmp_layout_t* L = a.L;
  const int64_t xperm_bytes = prefill_workspace(L->N, L->K, a.M).xperm_bytes;
  const PrefillForm form = choose_prefill_form(L->N, L->K, a.M);
  // the staging / scatter passes hold one fp16 row in LDS (K <= 57344 fits)
  if (((a.row_perm || form.ksplit > 1) && (int64_t)L->N * 2 > 160 * 1024) ||
      L->K / kTile > kPrefillMaxTiles)
    return SFMP_ERR_SHAPE;
  const void* reduce_fn = form.ksplit <= 2   ? reinterpret_cast<const void*>(&reduce_split_kernel<2>)
                          : form.ksplit <= 4 ? reinterpret_cast<const void*>(&reduce_split_kernel<4>)
                                             : reinterpret_cast<const void*>(&reduce_split_kernel<8>);
  if (form.ksplit > 1) {
    if (int e = allow_full_lds(reduce_fn, "hipFuncSetAttribute(reduce)")) return e;
  }
  const bool past = stores_past_caches(L->N, a.M);
  const void* scatter_fn = past ? reinterpret_cast<const void*>(&scatter_cols_kernel<true>) : reinterpret_cast<const void*>(&scatter_cols_kernel<false>);
  if (form.ksplit == 1 && a.row_perm) {
    if (int e = allow_full_lds(scatter_fn, "hipFuncSetAttribute(scatter)")) return e;
  }
  // activations -> workspace: column permutation applied (if any), 128x128 blocks each contiguous
  _Float16* Xp = (_Float16*)a.workspace;
  {
    const void* fn = reinterpret_cast<const void*>(&gather_cols_kernel);
    if (int e = allow_full_lds(fn, "hipFuncSetAttribute(gather)")) return e;
    const _Float16* Xa = (const _Float16*)a.X;
    const int32_t* cp = a.col_perm;
    int Ka = L->K;
    void* kargs[] = {&Xa, &cp, &Xp, &Ka};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)a.M), dim3(pass_threads(L->K, a.M)), kargs, (size_t)L->K * 2, (hipStream_t)stream);
    if (e != hipSuccess) {
      note_hip_error("sfmp_gemm activation staging launch", hipGetErrorString(e));
      return SFMP_ERR_HIP;
    }
    if (int e2 = check_launch("sfmp_gemm activation staging launch")) return e2;
  }
  _Float16* Yt = a.row_perm ? (_Float16*)((char*)a.workspace + xperm_bytes) : (_Float16*)a.Y;
  PrefillParams p;
  p.Xp = Xp;
  p.s2 = a.s2;
  p.s3 = a.s3;
  p.s4 = a.s4;
  p.index = a.index;
  p.scales = (const _Float16*)a.scales;
  p.zeros = (const _Float16*)a.zeros;
  p.Yt = Yt;
  p.M = a.M;
  p.N = L->N;
  p.ntr = L->N / kTile;
  p.ntc = L->K / kTile;
  p.gshift = L->group == 512 ? 2 : L->group == 256 ? 1 : 0;
  p.n_mtiles = 0;
  p.items = WorkItems{};
  p.ksplit = form.ksplit;
  p.partial = form.ksplit > 1 ? (float*)((char*)a.workspace + xperm_bytes) : nullptr;
  const bool g64 = L->group == 64, bf16 = L->scale_format == SFMP_SCALE_BF16;
  const hipStream_t s = (hipStream_t)stream;
  const PrefillTail tail = choose_prefill_tail(L->N, L->K, a.M);
  switch (tail.mi ? tail.mi - 8 : 8 * form.kg + form.mi) {
    case -4: launch_mixed<4>(p, a.M, tail.tile_rows, g64, bf16, s); break;
    case 0: launch_mixed<8>(p, a.M, tail.tile_rows, g64, bf16, s); break;
    case 8: launch_plain(p, a.M, g64, bf16, s); break;
    case 12: launch_fed<4, 1>(p, a.M, g64, bf16, s); break;
    case 13: launch_fed<5, 1>(p, a.M, g64, bf16, s); break;
    case 14: launch_fed<6, 1>(p, a.M, g64, bf16, s); break;
    case 15: launch_fed<7, 1>(p, a.M, g64, bf16, s); break;
    case 16: launch_fed<8, 1>(p, a.M, g64, bf16, s); break;
    case 20: launch_fed<4, 2>(p, a.M, g64, bf16, s); break;
    case 21: launch_fed<5, 2>(p, a.M, g64, bf16, s); break;
    case 22: launch_fed<6, 2>(p, a.M, g64, bf16, s); break;
    case 23: launch_fed<7, 2>(p, a.M, g64, bf16, s); break;
    case 24: launch_fed<8, 2>(p, a.M, g64, bf16, s); break;
    default: return SFMP_ERR_SHAPE;
  }
  if (int e = check_launch("sfmp_gemm prefill launch")) return e;
  if (form.ksplit > 1) {
    const float* partial = p.partial;
    int ks = form.ksplit, Ma = a.M, Na = L->N;
    const int32_t* rp = a.row_perm;
    _Float16* Y = (_Float16*)a.Y;
    void* kargs[] = {&partial, &ks, &Ma, &rp, &Y, &Na};
    hipError_t e = hipLaunchKernel(reduce_fn, dim3((unsigned)a.M), dim3(1024), kargs, (size_t)L->N * 2, (hipStream_t)stream);
    if (e != hipSuccess) {
      note_hip_error("sfmp_gemm split-K reduction launch", hipGetErrorString(e));
      return SFMP_ERR_HIP;
    }
    if (int e = check_launch("sfmp_gemm split-K reduction launch")) return e;
  } else if (a.row_perm) {
    const dim3 grid((unsigned)a.M), threads((unsigned)scatter_threads(L->N, a.M));
    if (past)
      hipLaunchKernelGGL(scatter_cols_kernel<true>, grid, threads, (size_t)L->N * 2, s, (const _Float16*)Yt, a.row_perm, (_Float16*)a.Y, (int)L->N);
    else
      hipLaunchKernelGGL(scatter_cols_kernel<false>, grid, threads, (size_t)L->N * 2, s, (const _Float16*)Yt, a.row_perm, (_Float16*)a.Y, (int)L->N);
    if (int e = check_launch("sfmp_gemm row scatter launch")) return e;
  }
  return SFMP_OK;
}

}  // namespace sfmp
