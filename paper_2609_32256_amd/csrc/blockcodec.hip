// Per-block fixed-length codec of the retained store's Q_eps codes (Section
// 2.2, L2 "error-bounded byte compression"; Section "Composite reduction":
// the reductions of deduplication and of the codec multiply).  Applied to the
// codes themselves, so decoding gives back exactly the Q_eps reconstruction and
// the score bound eps * ||q||_1 is unchanged.
//
// Format.  A block is 32 consecutive codes of a row.  Codes map to unsigned
// values by zigzag (u = 2q for q >= 0, -2q - 1 for q < 0); a block is stored
// with the bit width w of its largest u (0 for an all-zero block) as w 32-bit
// words in bit-plane order: bit j of word t is bit t of code j.  Per block one
// width byte; per row one 64-bit word offset (row_off[r], rows + 1 entries);
// blocks of a row and rows follow each other.
//
// One lane holds one block.  A block's 32 b-bit fields are exactly b words of the
// code stream, and its planes are w words, so a lane reads and writes whole
// words; in between the 32 codes sit NW-bit fields side by side in NW registers
// (NW = 8, 16 or 32, the smallest that holds b bits), where zigzag takes a few
// operations per word and the planes are an NW x NW bit transpose of every field
// at once.  That is about 7 operations a code where one lane per code and one
// ballot (or shuffle) per plane took about 70: those kernels were bound by the
// vector ALU (23,969 x 768 codes of 8 bits: widths 57 us, pack 49 us, decode and
// expansion 85 us each); these take 7, 14, 19 and 16 us, the decode at 4.8 TB/s.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lam_internal.h"

namespace lam {
namespace {

// A buffer resource over the words [base, base + words): loads past the end
// read as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const uint32_t* base, uint32_t words) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(base), (short)0, (int)(words * 4u), 0x00020000);
}

constexpr int kBlkThreads = 256;   // a workgroup holds whole rows: kBlkThreads / nb of them (nb = D / 32 <= 128)

constexpr int field_bits(int b) { return b <= 8 ? 8 : b <= 16 ? 16 : 32; }

// v in every NW-bit field of a word
template <int NW>
constexpr uint32_t rep(uint32_t v) {
  return NW == 8 ? v * 0x01010101u : NW == 16 ? v * 0x00010001u : v;
}

// the rows and blocks of this workgroup; thread t holds block t of them
struct BlkSpan {
  int64_t r0;
  int nrows, cnt;
  __device__ __forceinline__ BlkSpan(int64_t rows, int nb) {
    const int rpw = kBlkThreads / nb;
    r0 = (int64_t)blockIdx.x * rpw;
    nrows = (int)min((int64_t)rpw, rows - r0);
    cnt = nrows * nb;
  }
};

// Transposes the NW x NW bit matrix of every field: afterwards bit k of field f
// of word t is what bit t of field f of word k was.  Code f * NW + k sits in field
// f of word k, so the result's word t is plane t (bit j of it is bit t of code
// j); the transpose is its own inverse.
template <int NW>
__device__ __forceinline__ void bit_transpose(uint32_t (&a)[NW]) {
#pragma unroll
  for (int s = NW / 2; s >= 1; s >>= 1) {
    const uint32_t m = s == 16  ? 0x0000ffffu
                       : s == 8 ? 0x00ff00ffu
                       : s == 4 ? 0x0f0f0f0fu
                       : s == 2 ? 0x33333333u
                                : 0x55555555u;   // bits whose index has bit s clear
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      if (k & s) continue;
      const uint32_t x = a[k], y = a[k + s];
      a[k] = (x & m) | ((y << s) & ~m);
      a[k + s] = ((x >> s) & m) | (y & ~m);
    }
  }
}

// The zigzag codes of a block from its B words of the code stream.
template <int B>
__device__ __forceinline__ void load_zigzag(const uint32_t* __restrict__ src, uint32_t (&a)[field_bits(B)]) {
  constexpr int NW = field_bits(B);
  constexpr uint32_t kMask = B == 32 ? 0xffffffffu : (1u << B) - 1u;
  uint32_t w[B + 1];
  __builtin_memcpy(w, src, 4 * B);   // (word aligned: the device takes wide loads at any word)
  w[B] = 0u;
#pragma unroll
  for (int k = 0; k < NW; ++k) a[k] = 0u;
#pragma unroll
  for (int c = 0; c < 32; ++c) {
    const int bit = c * B, wi = bit >> 5, off = bit & 31;
    const uint32_t u = (off + B > 32 ? __builtin_amdgcn_alignbit(w[wi + 1], w[wi], (uint32_t)off) : w[wi] >> off) & kMask;
    a[c % NW] |= u << (c / NW * NW);
  }
  // u = 2q, or -2q - 1 = ~(2q) within the field for q < 0 (u < 2^B)
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const uint32_t sign = (a[k] >> (B - 1)) & rep<NW>(1u);
    a[k] = ((a[k] << 1) & rep<NW>(kMask & ~1u)) ^ (sign * kMask);
  }
}

// Back to two's complement over the whole NW-bit field.
template <int NW>
__device__ __forceinline__ void unzigzag_fields(uint32_t (&a)[NW]) {
  constexpr uint32_t kField = NW == 32 ? 0xffffffffu : (1u << (NW & 31)) - 1u;
#pragma unroll
  for (int k = 0; k < NW; ++k)
    a[k] = ((a[k] >> 1) & rep<NW>(kField >> 1)) ^ ((a[k] & rep<NW>(1u)) * kField);
}

// Exclusive prefix sum of v over the workgroup's threads; *total: the sum.
__device__ __forceinline__ uint32_t group_prefix(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wt[kBlkThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = (uint32_t)__shfl_up((int)x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) wt[wave] = x;
  __syncthreads();
  uint32_t base = 0u, all = 0u;
#pragma unroll
  for (int w = 0; w < kBlkThreads / 64; ++w) {
    const uint32_t t = wt[w];
    base += w < wave ? t : 0u;
    all += t;
  }
  *total = all;
  return base + x - v;
}

// Pass 1: block widths (the bit length of the OR of a block's zigzag codes) and
// the rows' word counts.
template <int B>
__global__ __launch_bounds__(kBlkThreads) void k_blk_widths(const uint32_t* __restrict__ codes, int64_t rows, int nb,
                                                            uint8_t* __restrict__ widths,
                                                            uint32_t* __restrict__ row_words) {
  constexpr int NW = field_bits(B);
  __shared__ uint32_t ws[kBlkThreads];
  const BlkSpan sp(rows, nb);
  const int t = threadIdx.x;
  if (t < sp.cnt) {
    const int64_t g = sp.r0 * nb + t;
    uint32_t a[NW];
    load_zigzag<B>(codes + g * B, a);
    uint32_t o = 0u;
#pragma unroll
    for (int k = 0; k < NW; ++k) o |= a[k];
    if (NW <= 16) o |= o >> 16;
    if (NW == 8) o |= o >> 8;
    if (NW < 32) o &= (1u << (NW & 31)) - 1u;
    const uint32_t w = o ? 32u - (uint32_t)__clz((int)o) : 0u;
    widths[g] = (uint8_t)w;
    ws[t] = w;
  }
  __syncthreads();
  if (t < sp.nrows) {
    uint32_t total = 0u;
    for (int k = 0; k < nb; ++k) total += ws[t * nb + k];
    row_words[sp.r0 + t] = total;
  }
}

// Exclusive scan of row word counts into row offsets (two small
// kernels: per-chunk scans, and the add of the chunk totals before).
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 4;
constexpr int kScanChunk = kScanThreads * kScanPer;

__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t* warp_tot, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) warp_tot[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t acc = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
      const uint64_t t = warp_tot[w];
      warp_tot[w] = acc;
      acc += t;
    }
    *total = acc;
  }
  __syncthreads();
  return warp_tot[wave] + x - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_chunks(const uint32_t* __restrict__ in, int64_t n,
                                                              uint64_t* __restrict__ out, uint64_t* __restrict__ sums) {
  __shared__ uint64_t wt[kScanThreads / 64];
  __shared__ uint64_t tot;
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
  uint32_t v[kScanPer];
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanPer; ++i) {
    v[i] = base + i < n ? in[base + i] : 0u;
    s += v[i];
  }
  uint64_t x = block_exclusive_scan(s, wt, &tot);
#pragma unroll
  for (int i = 0; i < kScanPer; ++i) {
    if (base + i < n) out[base + i] = x;
    x += v[i];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Adds the totals of the chunks before: a workgroup's 256 rows lie in one chunk
// (nchunks <= kScanChunk totals, a strided sum per workgroup).  The last one
// writes the number of words to out[n] and to the host.
__global__ __launch_bounds__(256) void k_scan_add(uint64_t* __restrict__ out, int64_t n,
                                                  const uint64_t* __restrict__ sums,
                                                  unsigned long long* __restrict__ words_host) {
  __shared__ unsigned long long part[4];
  const int t = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * 256 + t;
  const int c = (int)((int64_t)blockIdx.x * 256 / kScanChunk);
  unsigned long long x = 0ull;
  for (int k = t; k < c; k += 256) x += sums[k];
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  if ((t & 63) == 0) part[t >> 6] = x;
  __syncthreads();
  const uint64_t base = part[0] + part[1] + part[2] + part[3];
  if (i < n && c > 0) out[i] += base;
  if (blockIdx.x == gridDim.x - 1 && t == 0) {
    out[n] = base + sums[c];
    *words_host = base + sums[c];
  }
}
static_assert(kScanChunk % 256 == 0, "k_scan_add's workgroups stay within a chunk");

// Pass 2: a lane transposes its block's codes into planes and puts its w planes
// into the workgroup's run of words in LDS (the rows follow each other in the
// data, so the run is contiguous there too), which is then stored coalesced.
// Nothing is written when the encoding has more than cap words.
template <int B>
__global__ __launch_bounds__(kBlkThreads) void k_blk_pack(const uint32_t* __restrict__ codes, int64_t rows, int nb,
                                                          const uint8_t* __restrict__ widths,
                                                          const uint64_t* __restrict__ row_off,
                                                          uint32_t* __restrict__ data, uint64_t cap) {
  constexpr int NW = field_bits(B);
  __shared__ uint32_t run[kBlkThreads * B];   // (w <= B: zigzag codes are below 2^B)
  if (row_off[rows] > cap) return;
  const BlkSpan sp(rows, nb);
  const int t = threadIdx.x;
  const int64_t g = sp.r0 * nb + t;
  uint32_t a[NW];
  uint32_t w = 0u;
  if (t < sp.cnt) {
    w = widths[g];
    load_zigzag<B>(codes + g * B, a);
    bit_transpose<NW>(a);
  }
  uint32_t total;
  const uint32_t pre = group_prefix(w, &total);
#pragma unroll
  for (int k = 0; k < B; ++k)
    if ((uint32_t)k < w) run[pre + k] = a[k];
  __syncthreads();
  uint32_t* dst = data + row_off[sp.r0];
  for (uint32_t i = t; i < total; i += kBlkThreads) dst[i] = run[i];
}

// A lane's planes, transposed back and unzigzagged: the codes in two's
// complement NW-bit fields.  Planes past the width read as zero (an offset past
// the workgroup's run).
template <int NW>
__device__ __forceinline__ void load_blocks(const BlkSpan& sp, int nb, const uint8_t* __restrict__ widths,
                                            const uint64_t* __restrict__ row_off, const uint32_t* __restrict__ data,
                                            uint32_t (&a)[NW]) {
  const int t = threadIdx.x;
  const uint32_t w = t < sp.cnt ? widths[sp.r0 * nb + t] : 0u;
  const uint64_t off = row_off[sp.r0];
  uint32_t total;
  const uint32_t pre = group_prefix(w, &total);
  const __amdgpu_buffer_rsrc_t rs = words_rsrc(data + off, total);
#pragma unroll
  for (int k = 0; k < NW; ++k)
    a[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (uint32_t)k < w ? (pre + k) * 4u : 0xfffffff0u, 0, 0);
  bit_transpose<NW>(a);
  unzigzag_fields<NW>(a);
}

// Decode to x_hat = float32(float64(q * s)): the fields go through LDS so that a
// wave's float4 stores are consecutive (a field row is padded by four words:
// 16-byte reads, spread over the banks).
template <int NW>
__global__ __launch_bounds__(kBlkThreads) void k_blk_decode(const uint8_t* __restrict__ widths,
                                                            const uint64_t* __restrict__ row_off,
                                                            const uint32_t* __restrict__ data, int64_t rows, int nb,
                                                            double s, float* __restrict__ xhat) {
  constexpr int kLd = NW + 4;
  __shared__ __attribute__((aligned(16))) uint32_t fld[kBlkThreads * kLd];
  const BlkSpan sp(rows, nb);
  const int t = threadIdx.x;
  uint32_t a[NW];
  load_blocks<NW>(sp, nb, widths, row_off, data, a);
#pragma unroll
  for (int k = 0; k < NW; k += 4)
    *reinterpret_cast<uint4*>(&fld[t * kLd + k]) = make_uint4(a[k], a[k + 1], a[k + 2], a[k + 3]);
  __syncthreads();
  float* dst = xhat + sp.r0 * nb * 32;
  for (int i = t; i < sp.cnt * 8; i += kBlkThreads) {
    const int blk = i >> 3, c = (i & 7) * 4;   // codes c .. c + 3 of the block
    const uint4 f = *reinterpret_cast<const uint4*>(&fld[blk * kLd + c % NW]);
    const int sh = 32 - NW - c / NW * NW;      // field to the word's top, then sign-extended down
    const int32_t q0 = (int32_t)(f.x << sh) >> (32 - NW), q1 = (int32_t)(f.y << sh) >> (32 - NW);
    const int32_t q2 = (int32_t)(f.z << sh) >> (32 - NW), q3 = (int32_t)(f.w << sh) >> (32 - NW);
    const float v[4] = {(float)((double)q0 * s), (float)((double)q1 * s), (float)((double)q2 * s),
                        (float)((double)q3 * s)};
    __builtin_memcpy(dst + (int64_t)i * 4, v, 16);   // (xhat is word aligned, no more is asked of it)
  }
}

// Back to the B-bit code stream: a lane packs its block's B words, which go
// through LDS (odd row length) to coalesced stores.
template <int B>
__global__ __launch_bounds__(kBlkThreads) void k_blk_expand(const uint8_t* __restrict__ widths,
                                                            const uint64_t* __restrict__ row_off,
                                                            const uint32_t* __restrict__ data, int64_t rows, int nb,
                                                            uint32_t* __restrict__ codes) {
  constexpr int NW = field_bits(B);
  constexpr uint32_t kMask = B == 32 ? 0xffffffffu : (1u << B) - 1u;
  constexpr int kLd = B | 1;
  __shared__ uint32_t out[kBlkThreads * kLd];
  const BlkSpan sp(rows, nb);
  const int t = threadIdx.x;
  uint32_t a[NW];
  load_blocks<NW>(sp, nb, widths, row_off, data, a);
  uint32_t w[B + 1];
#pragma unroll
  for (int k = 0; k <= B; ++k) w[k] = 0u;
#pragma unroll
  for (int c = 0; c < 32; ++c) {
    const int bit = c * B, wi = bit >> 5, off = bit & 31;
    const uint32_t u = (a[c % NW] >> (c / NW * NW)) & kMask;
    w[wi] |= u << off;
    if (off + B > 32) w[wi + 1] |= u >> (32 - off);
  }
#pragma unroll
  for (int k = 0; k < B; ++k) out[t * kLd + k] = w[k];
  __syncthreads();
  uint32_t* dst = codes + sp.r0 * nb * B;
  for (int i = t; i < sp.cnt * B; i += kBlkThreads) dst[i] = out[i / B * kLd + i % B];
}

// Launches f<B> for the runtime width b in [1, 32].
template <int B = 1, class F>
void for_width(int b, F&& f) {
  if (b == B) return f(std::integral_constant<int, B>{});
  if constexpr (B < 32) for_width<B + 1>(b, f);
}

unsigned blk_grid(int64_t rows, int nb) {
  const int rpw = kBlkThreads / nb;
  return (unsigned)((rows + rpw - 1) / rpw);
}

}  // namespace

lam_status block_encode(lam_ctx* ctx, lam_store* st, lam_block_stats* out) {
  const int D = st->dim;
  const int nb = D / 32;
  const int64_t m = st->size;
  const int b = st->q.bits;
  const int64_t nchunks = (m + kScanChunk - 1) / kScanChunk;
  LAM_CHECK(nchunks <= kScanChunk, LAM_EINVAL, "store too large for the block codec's scan");
  if (!st->blk_w) {
    LAM_HIP(hipMalloc(&st->blk_w, (size_t)st->capacity * nb));
    LAM_HIP(hipMalloc(&st->blk_row_off, (size_t)(st->capacity + 1) * 8));
  }
  LAM_TRY(ctx->scratch[kScratchBlocks].ensure((size_t)m * 4 + (size_t)(nchunks + 1) * 8 + 64));
  uint32_t* row_words = ctx->scratch[kScratchBlocks].as<uint32_t>();
  uint64_t* sums = reinterpret_cast<uint64_t*>(ctx->scratch[kScratchBlocks].as<char>() + (((size_t)m * 4 + 7) & ~7ull));
  const dim3 grid(blk_grid(m, nb)), block(kBlkThreads);
  auto pack = [&]() -> lam_status {
    ProfScope ps(ctx, "store_block_pack");
    for_width(b, [&](auto B) {
      hipLaunchKernelGGL(k_blk_pack<B.value>, grid, block, 0, ctx->stream, st->codes, m, nb, st->blk_w,
                         st->blk_row_off, st->blk_data, st->blk_cap / 4);
    });
    LAM_HIP(hipGetLastError());
    return LAM_OK;
  };
  ctx->flags_host->blk_words = 0;
  // the data buffer holds what the encoding needs and no more.  A pack into the
  // buffer of an earlier encoding is queued before the count is known (it writes
  // nothing if that is too small), so that the device does not idle meanwhile.
  if (m > 0) {
    {
      ProfScope ps(ctx, "store_block_encode");
      for_width(b, [&](auto B) {
        hipLaunchKernelGGL(k_blk_widths<B.value>, grid, block, 0, ctx->stream, st->codes, m, nb, st->blk_w, row_words);
      });
      LAM_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_scan_chunks, dim3((unsigned)nchunks), dim3(kScanThreads), 0, ctx->stream, row_words, m,
                         st->blk_row_off, sums);
      hipLaunchKernelGGL(k_scan_add, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, ctx->stream, st->blk_row_off,
                         m, sums, &ctx->flags_host_dev->blk_words);
      LAM_HIP(hipGetLastError());
    }
    if (st->blk_data) LAM_TRY(pack());
  } else {
    LAM_HIP(hipMemsetAsync(st->blk_row_off, 0, sizeof(uint64_t), ctx->stream));   // (the call waits: it is never captured)
  }
  LAM_HIP(hipStreamSynchronize(ctx->stream));
  const uint64_t words = ctx->flags_host->blk_words;   // written by k_scan_add
  if (words * 4 > st->blk_cap || !st->blk_data) {
    if (st->blk_data) LAM_HIP(hipFree(st->blk_data));
    st->blk_data = nullptr;
    st->blk_cap = 0;
    const uint64_t need = std::max<uint64_t>(words * 4, 4);
    LAM_HIP(hipMalloc(&st->blk_data, need));
    st->blk_cap = need;
    if (m > 0) LAM_TRY(pack());
  }
  st->blk_rows = m;
  st->blk_words = words;
  if (out) {
    lam_block_stats s{};
    s.rows = m;
    s.blocks = m * nb;
    s.data_bytes = words * 4;
    s.meta_bytes = (uint64_t)m * nb + (uint64_t)(m + 1) * 8;
    s.total_bytes = s.data_bytes + s.meta_bytes;
    const double ncodes = (double)m * D;
    s.bits_per_code = ncodes > 0 ? 8.0 * (double)s.total_bytes / ncodes : 0.0;
    s.plain_bits = b;
    s.codec_ratio = s.bits_per_code > 0 ? 32.0 / s.bits_per_code : 0.0;
    s.composite_ratio = s.total_bytes > 0 ? (double)st->n_seen * D * 4.0 / (double)s.total_bytes : 0.0;
    *out = s;
  }
  return LAM_OK;
}

lam_status block_decode(lam_ctx* ctx, const lam_store* st, float* xhat, uint32_t* codes_out) {
  const int64_t m = st->blk_rows;
  if (m <= 0) return LAM_OK;
  ProfScope ps(ctx, xhat ? "store_block_decode" : "store_block_expand");
  const int nb = st->dim / 32, b = st->q.bits;
  const dim3 grid(blk_grid(m, nb)), block(kBlkThreads);
  if (xhat) {
    auto* kernel = b <= 8 ? k_blk_decode<8> : b <= 16 ? k_blk_decode<16> : k_blk_decode<32>;
    hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, st->blk_w, st->blk_row_off, st->blk_data, m, nb,
                       st->q.step, xhat);
  } else {
    for_width(b, [&](auto B) {
      hipLaunchKernelGGL(k_blk_expand<B.value>, grid, block, 0, ctx->stream, st->blk_w, st->blk_row_off,
                         st->blk_data, m, nb, codes_out);
    });
  }
  LAM_HIP(hipGetLastError());
  return LAM_OK;
}

}  // namespace lam
