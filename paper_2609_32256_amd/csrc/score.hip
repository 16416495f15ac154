// Retrieval scoring against the quantized store, dequantized on the fly, with
// top-k per query and the per-query bound eps * ||q||_1 (Hoelder applied to
// the per-coordinate bound of Q_eps, Appendix "Rank invariance, in full").
//
// score(j, y) = s * sum_d q_j,d * code_y,d  (s = 2 eps), i.e. q_j . x_hat_y with
// the exact dequantized row: a binary64 sum, rounded once to float32, in a store
// of more than 4,096 rows; an fp32 sum of the query's fp16 hi and lo parts, of
// every row, in a smaller one (k_dense).
//
// In a larger store the matrix units find the few rows that can be in a query's
// top-k.  A scan
// forms H, the score from fp16 operands: the query's fp16 part h (each query
// scaled by a power of two 2^e_j, max |q| into [2^14, 2^15)) times the codes,
// unpacked from their b-bit words straight into fp16 LDS slabs (no dequantized
// copy exists in HBM) and accumulated in fp32 by v_mfma_f32_32x32x16_f16.  Codes
// of values below 2^11 are exact in fp16; of wider ones the scan takes the top
// 12 bits.  Where every code fits 8 bits the full scan multiplies bytes instead
// (the query rounded to 127ths of its largest entry, twice the matrix rate),
// unless the sample shows that the wider error bound would let too many rows
// through.  A per-query bound err on |H - score| (see k_score_prep) turns the
// k-th best H into a threshold; the rows above it are scored exactly and the k
// best by (score desc, id asc) are the answer.  See score_topk_impl for the
// plan.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "lam_internal.h"
#include "mfma_tile.h"
#include "wave.h"

namespace lam {
namespace {

// (S_QLO shares a slot: a call takes the byte parts or, for a small store, the lo parts)
enum ScoreScratch { S_QHI = 7, S_QMETA, S_PART, S_CAND, S_Q8, S_QLO = S_Q8 };

enum QKind : int {
  kScanned = 0,    // the scan finds the candidates
  kInvalid = 1,    // the query holds NaN/Inf
  kUnscanned = 2,  // its scales leave float32's normal range (a tiny query): the exact pass answers it
  kZero = 3,       // every score is 0: the first k rows
};

struct QMeta {
  float osc;     // float32(s * 2^(sh - e)): multiplies the raw accumulator
                 // (small stores: negative where the scale is -osc 2^-126)
  float bound;   // eps * ||q||_1 rounded up, or NaN for an invalid query
  int kind;      // a QKind
  float err;     // >= |H + c - score| for every store row, c a constant of the query (rounded up)
  float osc8;    // the same two for the byte scan: float32(s * qs), qs = max|q| / 127
  float err8;
};

__device__ __forceinline__ bool normal_f32(float x) { return x >= 0x1p-126f && x <= 3.402823466e38f; }

// Queries that share the choice of the scan's operands: the columns of the
// larger tile, which are multiplied by one instruction stream.
constexpr int kPrecQueries = 256;

__device__ __forceinline__ float ru32(double d) {
  float f = (float)d;
  if ((double)f < d) f = __uint_as_float(__float_as_uint(f) + 1u);   // d >= 0 here
  return f;
}

__device__ __forceinline__ float rd32(double d) {
  float f = (float)d;
  if ((double)f > d) f = nextafterf(f, -INFINITY);
  return f;
}

// Per query: its fp16 part and the meta block.  err bounds the difference
// between a score H of the scan and the exact one S (with a constant of the
// query left out: only differences between rows of one query matter), both
// against T = s sum_d q_d code_d, in score units.  With h = fp16 part * 2^-e in
// the query's own units and, for codes taken without their low sh bits,
// code = 2^sh top + low, low in [0, 2^sh - 1]:
//   h:         |s 2^sh sum_d (q_d - h_d) top_d| <= ||q - h||_2 R (Cauchy-Schwarz;
//              ||q - h||_2 is computed here in binary64), R >= s 2^sh ||top||;
//   low bits:  s sum_d q_d low_d = c + (at most s (2^sh - 1) / 2 sqrt(D) ||q||);
//              trunc = s (2^sh - 1) / 2 sqrt(D);
//   fp32 sum:  g = 2 (D + 64) 2^-24 of s 2^sh sum |h_d top_d| <= (||q|| + ||q - h||) R
//              (two roundings per addition, in any order);
//   scalings:  osc and the final product, 2^-24 each, or 2^-150 where the
//              product is subnormal;
//   S:         the rescoring sums in binary64 and rounds once to float32 (2^-24,
//              or 2^-150 where S is subnormal).
// |H + c - S| <= ||q - h|| R + trunc ||q|| + (g + 2^-21)(||q|| + ||q - h||) R + 2^-149.
// The byte scan (q8 not NULL; codes of at most 8 bits, so trunc = 0) has h = qs
// rint(q / qs) and exact int32 sums: err8 = (||q - h|| + 2^-21 (||q|| + ||q - h||)) R + 2^-149.
// Both hold for scales osc and osc8 that are normal float32 values (2^-24) and a
// finite 2^e; a query that has another (max|q| below about 2^-105) is not
// scanned.  Sample and byte scan differ in their scale, so an error of one of
// them would not cancel in the comparison with the threshold.
// qmax: the largest |q| taken (a query row above it, or holding NaN/Inf, is
// invalid).  cand_cnt, done: this query's candidate count and finished
// workgroups of the exact pass, n_flag the number of flagged queries, and coarse,
// a flag per kPrecQueries queries (see k_sample_thr), start at zero (the buffers
// may hold anything from an earlier call).
__global__ __launch_bounds__(256) void k_score_prep(const float* __restrict__ q, int64_t nq, int D, double step_f,
                                                    double eps, double R, double trunc, float qmax,
                                                    _Float16* __restrict__ qhi, int8_t* __restrict__ q8,
                                                    QMeta* __restrict__ meta, uint32_t* __restrict__ cand_cnt,
                                                    uint32_t* __restrict__ done, uint32_t* __restrict__ n_flag,
                                                    uint32_t* __restrict__ coarse) {
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= nq) return;
  if (lane == 0) {
    cand_cnt[j] = 0u;
    done[j] = 0u;
    if (j == 0) *n_flag = 0u;
    if (j % kPrecQueries == 0) coarse[j / kPrecQueries] = 0u;
  }
  const float* p = q + j * D;
  float mx = 0.0f;
  double l1 = 0.0, l2 = 0.0;
  bool bad = false;
  // D <= 1,024: the row is loaded once as float4 pieces held in registers (all
  // loads in flight together; the resource ends at the row, so pieces past it
  // read as zero), and both passes below work from them
  constexpr int kVec = 4;
  const bool vec = D <= 256 * kVec;
  float4 v4[kVec];
  {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, vec ? D * 4 : 0, 0x00020000);
#pragma unroll
    for (int u = 0; u < kVec; ++u)
      v4[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)(u * 256 + lane * 4) * 4u, 0, 0));
  }
  auto take1 = [&](float v) {
    const float a = fabsf(v);
    bad |= !(a <= qmax);
    mx = fmaxf(mx, a);
    l1 += (double)a;
    l2 = fma((double)v, (double)v, l2);
  };
  if (vec) {
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const int d = u * 256 + lane * 4;
      if (d >= D) break;
      take1(v4[u].x);
      take1(v4[u].y);
      take1(v4[u].z);
      take1(v4[u].w);
    }
  } else {
    for (int d = lane; d < D; d += 64) take1(p[d]);
  }
  mx = wave_max_f32(mx);
  l1 = wave_sum_f64(l1);
  l2 = wave_sum_f64(l2);
  bad = __ballot(bad) != 0ull;
  int e = 0;
  if (!bad && mx > 0.0f) e = min(127, 14 - ilogbf(mx));   // max |q| 2^e in [2^14, 2^15), where 2^e is finite
  const float sc = ldexpf(1.0f, e);
  const double isc = ldexp(1.0, -e);
  double dh2 = 0.0;   // ||q - h||^2
  auto part = [&](float x, _Float16& h) {
    h = (_Float16)(bad ? 0.0f : x * sc);     // exact power-of-two scaling
    const double r = bad ? 0.0 : (double)x - (double)(float)h * isc;   // exact in binary64
    dh2 = fma(r, r, dh2);
  };
  const float qs = bad ? 0.0f : mx * (1.0f / 127.0f);
  const float iqs = qs > 0x1p-120f ? 1.0f / qs : 0.0f;   // (else all bytes 0, err8 ||q|| R)
  double db2 = 0.0;   // ||q - qs rint(q / qs)||^2
  auto byte = [&](float x) {
    const float v = bad ? 0.0f : fminf(fmaxf(rintf(x * iqs), -127.0f), 127.0f);
    const double r = bad ? 0.0 : (double)x - (double)v * (double)qs;
    db2 = fma(r, r, db2);
    return (uint32_t)(int)v & 255u;
  };
  if (vec) {
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const int d = u * 256 + lane * 4;
      if (d >= D) break;
      const float c[4] = {v4[u].x, v4[u].y, v4[u].z, v4[u].w};
      _Float16 h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) part(c[i], h[i]);
      uint2 ph;
      __builtin_memcpy(&ph, h, 8);
      *reinterpret_cast<uint2*>(qhi + j * D + d) = ph;
      if (q8)
        *reinterpret_cast<uint32_t*>(q8 + j * D + d) =
            byte(c[0]) | (byte(c[1]) << 8) | (byte(c[2]) << 16) | (byte(c[3]) << 24);
    }
  } else {
    for (int d = lane; d < D; d += 64) {
      part(p[d], qhi[j * D + d]);
      if (q8) q8[j * D + d] = (int8_t)byte(p[d]);
    }
  }
  dh2 = wave_sum_f64(dh2);
  if (q8) db2 = wave_sum_f64(db2);
  if (lane == 0) {
    QMeta m{};
    m.osc = (float)ldexp(step_f, -e);
    // (a binary64 sum of D non-negative terms is below the exact one by at most
    // (D - 1) 2^-53 relative, in any order; products and sqrt add 2^-53 each)
    const double up = 1.0 + (double)(D + 4) * 0x1p-52;
    m.bound = bad ? __builtin_nanf("") : ru32(eps * l1 * up);
    const double g = 2.0 * (double)(D + 64) * 0x1p-24;
    const double qn = sqrt(l2) * up;
    const double dh = sqrt(dh2) * up;
    const double E = dh * R + trunc * qn + (g + 0x1p-21) * (qn + dh) * R + 0x1p-149;
    m.err = bad ? 0.0f : ru32(E * (1.0 + 0x1p-20));
    m.osc8 = (float)(step_f * (double)qs);
    const double db = sqrt(db2) * up;
    m.err8 = bad ? 0.0f : ru32(((db + 0x1p-21 * (qn + db)) * R + 0x1p-149) * (1.0 + 0x1p-20));
    const bool fits = mx >= 0x1p-113f && normal_f32(m.osc) && (!q8 || normal_f32(m.osc8));
    m.kind = bad ? kInvalid : mx == 0.0f ? kZero : fits ? kScanned : kUnscanned;
    meta[j] = m;
  }
}


struct ScoreArgs {
  const uint32_t* codes;
  int64_t n;                 // store rows
  int D;
  int sh;                    // low bits of a code that the scan leaves out (codes of more than 12 bits)
  int64_t row_words;         // D * b / 32
  const _Float16* qhi;
  const int8_t* q8;          // byte scan: the queries' byte parts
  const uint32_t* coarse;    // byte scan: flags of kPrecQueries queries that take the fp16 scan
  const QMeta* meta;
  int64_t nq;
  int nqt;                   // query tiles of this launch
  int64_t tile_end;          // store tiles [0, tile_end) scanned by this launch
  float* part_s;             // sample pass: [nq][entries]
  int sample_tiles;          // sample pass: store tiles with entries of their own (later tiles fold onto them)
  const float* thr;          // filter pass: per-query threshold (fp16 scan), then the byte scan's
  float* cand_s;             // filter pass: [nq][cap] scores and rows
  int32_t* cand_r;
  uint32_t* cand_cnt;
  uint32_t cap;
};

typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// Code e (a compile-time constant) of the b-bit codes that start at bit 0 of v;
// a word past the codes is read only for a field that straddles into it.
template <int B>
__device__ __forceinline__ int32_t code_at(const uint32_t* v, int e) {
  const int bit = e * B, wi = bit >> 5, off = bit & 31;
  uint32_t u = v[wi] >> off;
  if (off + B > 32) u |= v[wi + 1] << (32 - off);
  return (int32_t)(u << (32 - B)) >> (32 - B);
}

// The 16 b-bit codes of half `h` of a group of 32 to fp16 (without their low
// sh bits when B > 12).  w: the words that hold them, (B + 1) / 2 words from word
// h * (B / 2) of the group; for odd widths the upper half starts at bit 16 of
// its first word.  Byte codes take an exact shortcut, two codes per step: the
// byte c + 128 (c XOR 0x80) becomes the low byte of the fp16 bit pattern 0x6400 |
// byte, which is the value 1024 + c + 128 exactly; one packed fp16 subtraction
// of 1152 leaves c.
template <int B>
__device__ __forceinline__ void unpack16(const uint32_t (&w)[(B + 1) / 2], int h, int sh, _Float16* __restrict__ out) {
  constexpr int NW = (B + 1) / 2;
  if constexpr (B == 8) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const uint32_t x = w[i] ^ 0x80808080u;
      // bytes 0..3 of the selection come from x, 4..7 from the constant 0x64646464
      const uint32_t lo = __builtin_amdgcn_perm(0x64646464u, x, 0x04010400u);
      const uint32_t hi = __builtin_amdgcn_perm(0x64646464u, x, 0x04030402u);
      const half2v off = {(_Float16)1152.0f, (_Float16)1152.0f};
      const half2v a = __builtin_bit_cast(half2v, lo) - off;
      const half2v b = __builtin_bit_cast(half2v, hi) - off;
      out[4 * i + 0] = a.x;
      out[4 * i + 1] = a.y;
      out[4 * i + 2] = b.x;
      out[4 * i + 3] = b.y;
    }
  } else {
    uint32_t v[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      if constexpr ((B & 1) != 0) v[i] = __builtin_amdgcn_alignbit(i + 1 < NW ? w[i + 1] : 0u, w[i], h ? 16u : 0u);
      else v[i] = w[i];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      int32_t c = code_at<B>(v, e);
      if constexpr (B > 12) c >>= sh;
      out[e] = (_Float16)(short)c;   // |c| <= 2^11
    }
  }
}

// NW consecutive words at byte offset voff + soff of the buffer in the widest
// pieces (16, 8, then 4 bytes; multi-dword buffer loads need 4-byte alignment
// only), so that a lane asks for its bytes in one to three requests.
template <int NW>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, uint32_t (&cw)[NW]) {
#pragma unroll
  for (int i = 0; i + 4 <= NW; i += 4) {
    const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + i * 4u, soff, 0));
    cw[i] = v.x;
    cw[i + 1] = v.y;
    cw[i + 2] = v.z;
    cw[i + 3] = v.w;
  }
  constexpr int r = NW & ~3;
  if constexpr ((NW & 2) != 0) {
    const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff + r * 4u, soff, 0));
    cw[r] = v.x;
    cw[r + 1] = v.y;
  }
  if constexpr ((NW & 1) != 0)
    cw[NW - 1] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, voff + (NW - 1) * 4u, soff, 0);
}

// ------------------------------------------------------------------ thresholds
constexpr int kCandCap = 4096;   // candidate buffer entries per query
constexpr int kNoAllocMaxQ = 256;   // queries of one allocation-free scoring call

// A lower bound, within 2^-15 relative, of the k-th largest of a wave's order
// keys (R per lane, 0 for none): the top 24 bits of it, found bit by bit from
// the top, one ballot and one scalar bit count per lane register and bit, so
// the cost does not depend on k.  (Sorted per-lane lists and k rounds of the
// best head: 8.5 us for 1,024 queries of 128 keys at k = 10, 41 us for 300
// queries of up to 7,360 at k = 50; the threshold kernel built on this: 6.8 us
// and, for 736 keys, 13 us.)  0 when fewer than k keys
// are set.  nr: the registers in use (uniform).
template <int R>
__device__ __forceinline__ uint32_t wave_kth_floor(const uint32_t (&key)[R], int nr, int k) {
  uint32_t T = 0u;
  for (int bit = 31; bit >= 8; --bit) {
    const uint32_t c = T | (1u << bit);
    int n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < nr) n += __popcll(__ballot(key[r] >= c));
    T = n >= k ? c : T;
  }
  return T;
}

// The score that a floor of order keys stands for, within float32's finite range
// from above, so that an error bound can be taken off it (a row whose score
// overflows has a larger one); -inf for the keys below every finite score,
// whose low bits wave_kth_floor drops.
__device__ __forceinline__ double floor_score(uint32_t T) {
  constexpr float kMax = 3.402823466e38f;
  return T < f2ord(-kMax) ? -INFINITY : fmin((double)ord2f(T), (double)kMax);
}

// One wave per query: the threshold of the filter pass from the sample's
// entries (scores of distinct rows): the k-th best, lowered by 2 err, so that
// no row of the final top-k falls below it in hi-only terms.  Beyond 1,024
// entries several share a key as their maximum: the k-th best key is then
// still the score of k distinct rows, only a little lower.
// With a byte scan to follow (coarse not NULL) also its threshold, T - err -
// err8, and the choice between the two scans: if more than most_above keys reach
// it (see byte_scan_keys), the query's group of kPrecQueries takes the fp16 scan.  That happens where scores lie close
// together for the byte scan's error (8e-3 ||q|| R for a Gaussian query), or
// where single entries dominate the query, which widens that error.
constexpr int kThrKeys = 16;   // keys per lane
// The rows above the threshold from which the fp16 scan is the faster one, by the
// launch's 128 x 128 tiles: where few tiles run, the candidates' stores and the
// longer selection are not hidden behind other tiles; where many do, bytes lead
// until the candidates near the buffer's size.  Whole calls, fp16 : bytes, us, at
// 8-bit codes (queries x rows x dimension, top-k, rows above):
//   196 tiles  128 x 25,000 x 1,024  k 10, 233  62 : 60    k 20, 348  68 : 75
//   469        128 x 60,000 x 768    k  1,  60  54 : 52    k 10, 520  70 : 75
//   588        300 x 25,000 x 1,024  k 10, 233  74 : 69    k 20, 397  82 : 87
//   939        300 x 40,000 x 1,024  k 10, 373  84 : 78    k 20, 737  93 : 101
//   1,565      600 x 40,000 x 768    k 10, 399  95 : 83    k 50, 846 125 : 128
//   1,565      600 x 40,000 x 384    k 10, 272  74 : 70    k 20, 454  81 : 87
//   2,346      300 x 100,000 x 768   k  1, 176 105 : 82    k 10, 771 119 : 113
//   3,910      600 x 100,000 x 1,024 k  1, 308 195 : 137   k 10, 1,066 220 : 179
//   6,256      1,024 x 100,000 x 768, 1,024 to 2,048 rows 252 : 200, about 3,500 251 : 247
// Over 228 such calls this rule costs 0.3 % against the better scan of each, bytes
// throughout 3.0 %, fp16 throughout 4.2 %.
constexpr double byte_scan_limit(int64_t tiles) { return tiles < 768 ? 256.0 : tiles < 2048 ? 448.0 : 2048.0; }

// The same as a number of the sample's keys: a share f of keys above a threshold,
// each the best of `per` rows, means n (-ln(1 - f)) / per rows above it.  (Below
// nkeys: when every key is above, perhaps every row is.)
int byte_scan_keys(int64_t tiles, int64_t n, int nkeys, double per) {
  return std::min(nkeys - 1, (int)(nkeys * -std::expm1(-byte_scan_limit(tiles) * per / (double)n)));
}

__global__ __launch_bounds__(256) void k_sample_thr(int64_t nq, int entries, int folded, int k,
                                                    const float* __restrict__ ps, const QMeta* __restrict__ meta,
                                                    float* __restrict__ thr, uint32_t* __restrict__ coarse,
                                                    int most_above) {
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= nq) return;
  const float* s = ps + j * (int64_t)entries;
  const QMeta m = meta[j];
  // folded: the sample shared entries and left order codes
  auto code = [&](int e) { return folded ? __float_as_uint(s[e]) : f2ord(s[e] + 0.0f); };
  uint32_t key[kThrKeys];
#pragma unroll
  for (int r = 0; r < kThrKeys; ++r) key[r] = lane + r * 64 < entries ? code(lane + r * 64) : 0u;
  for (int e0 = 64 * kThrKeys; e0 < entries; e0 += 64 * kThrKeys)
#pragma unroll
    for (int r = 0; r < kThrKeys; ++r)
      if (e0 + lane + r * 64 < entries) key[r] = max(key[r], code(e0 + lane + r * 64));
  const uint32_t T = wave_kth_floor<kThrKeys>(key, min(kThrKeys, (entries + 63) / 64), k);
  const double t = floor_score(T);
  if (lane == 0) thr[j] = m.kind != kScanned ? __builtin_nanf("") : rd32(t - 2.0 * (double)m.err);
  if (!coarse) return;
  const float t8 = rd32(t - (double)m.err - (double)m.err8);
  if (lane == 0) thr[nq + j] = m.kind != kScanned ? __builtin_nanf("") : t8;
  int above = 0;
  const uint32_t o8 = f2ord(t8);
#pragma unroll
  for (int r = 0; r < kThrKeys; ++r) above += __popcll(__ballot(key[r] >= o8));
  // (a plain store: every writer stores the same; atomics on one word took 10 us
  // when all of 1,024 queries set it)
  if (lane == 0 && m.kind == kScanned && above > most_above) coarse[j / kPrecQueries] = 1u;
}

// ------------------------------------------------------------------ filter pass on the screen's pipeline
using FilterTile = Tile<2, 4, 2, 1, 4>;
// 256 x 256 (store rows x queries), sixteen waves of 64 x 64 held to 128
// registers, one workgroup per CU: half the code and query loads per flop of
// FilterTile; for the filter pass of stores with many tiles
using FilterTileL = Tile<4, 4, 2, 2, 4>;
static_assert(kPrecQueries % FilterTileL::BN == 0 && kPrecQueries % FilterTile::BN == 0, "a tile's queries share their operands");
constexpr int kMaxBits = 22;       // code widths that can be scored
constexpr int kFilterGroupQ = 8;   // query tiles per group in the tile order
constexpr int kSampleEntries = 4;  // entries per query and 128-row store tile of the sample pass
constexpr int64_t kSampleTiles = 2048;   // sample tiles with entries of their own (later ones share them)
constexpr int64_t kFilterLargeMinTiles = 1024;   // large filter tiles from this many per launch

// The threshold plan's filter pass (hi-only scores H): one C::BM x C::BN tile
// (store rows x queries) per workgroup, each wave 64 rows x 32 TJ queries (2 x
// TJ tiles of v_mfma_f32_32x32x16_f16); K-slabs of 64 through two LDS stages,
// one barrier per slab, every load issued three slabs before its LDS store
// (SETS = 3) or one (SETS = 1, for the large tile).  Four threads share a
// row's 64-code slab (16 codes each: B / 2 words, or the (B + 1) / 2 that hold
// them), so every wave unpacks.  Codes are unpacked straight to fp16 (exact
// for B <= 12); the queries' hi part is loaded in 16-byte pieces.  The slab
// loop takes D at run time, six slabs (both LDS stages, all three register
// sets) per trip: the offsets of a slab are one scalar, and loads past the
// last slab fall outside the buffer bound (no memory touched).  Tile order:
// groups of 8 query tiles against every store tile, query tile fastest, each
// XCD a contiguous range, so an XCD holds its query tiles in L2 while the codes
// stream past.  Every row with H >= the query's threshold is appended to its
// candidate buffer.  The tile loop's latency bounds the small launches: 1,024
// queries x 23,969 rows x 768 at 8 bits take 53.8 us in fp16 (twelve slabs) and
// 37.7 us in bytes (six); 300 x 120,001 x 384, 81.6 and 62.8 us (106 us in a
// one-stage fp16 kernel with two waves' worth of loads in flight, whose sample
// pass took 54 us, here 13).  4,096 x 361,802 x 768 in bytes: 1.68 ms.
// kSample (FilterTile only): the sample pass of the threshold plan over store
// tiles [0, tile_end) (all of them whole) instead: per query and tile, the best
// H of each of the four lanes holding the query (disjoint sets of 32 rows) at
// entries [4 t, 4 t + 4) of the query's list, t the tile (modulo sample_tiles:
// beyond those, tiles share entries as their maximum, order-encoded).  The
// k-th best of these entries is the H of k distinct rows, so at most the
// sample's k-th best H: a valid base for the threshold (lower only where
// several of the best rows share a lane).
// a.nqt and a.tile_end count tiles of this kernel's size.
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));

// The scan's operands: fp16 codes and queries (64 columns in the 128 bytes of a
// row's slab), or bytes (128 columns).
struct OpF16 {
  typedef floatx16 Acc;
  static constexpr int kCols = 64;
  template <int B>
  static constexpr int kWords = (B + 1) / 2;   // code words per thread and slab
  static __device__ __forceinline__ Acc mfma(half8 x, half8 y, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, c, 0, 0, 0);
  }
};
struct OpI8 {
  typedef intx16 Acc;
  static constexpr int kCols = 128;
  template <int B>
  static constexpr int kWords = B;
  static __device__ __forceinline__ Acc mfma(half8 x, half8 y, Acc c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(intx4, x), __builtin_bit_cast(intx4, y), c, 0, 0,
                                                 0);
  }
};

// The 32 b-bit codes of a group (B words; every code fits 8 bits) to bytes.
template <int B>
__device__ __forceinline__ void unpack_bytes(const uint32_t (&w)[B], uint32_t (&out)[8]) {
  if constexpr (B == 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = w[i];
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t c0 = (uint32_t)code_at<B>(w, 4 * i), c1 = (uint32_t)code_at<B>(w, 4 * i + 1);
      const uint32_t c2 = (uint32_t)code_at<B>(w, 4 * i + 2), c3 = (uint32_t)code_at<B>(w, 4 * i + 3);
      // bytes 0..3 of a selection come from its second operand, 4..7 from the first
      out[i] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(c3, c2, 0x0c0c0400u), __builtin_amdgcn_perm(c1, c0, 0x0c0c0400u),
                                     0x05040100u);
    }
  }
}

// acc <- the raw scores of one C::BM x C::BN tile: store rows [rbase, rbase +
// rows) against queries [qbase, qbase + qrows).
template <class C, class Op, int B, int SETS>
__device__ __forceinline__ void scan_tile(const ScoreArgs& a, int64_t rbase, int rows, int64_t qbase, int qrows,
                                          _Float16* lds, typename Op::Acc (&acc)[C::TI][C::TJ]) {
  static_assert(SETS == 1 || SETS == 3, "one or three register sets");
  static_assert(C::kThreads == 4 * C::BM, "four threads per row");
  constexpr bool kBytes = Op::kCols == 128;
  constexpr int kES = kBytes ? 1 : 2;   // bytes per query element
  const int tid = threadIdx.x, wave = tid >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  auto sa = [&](int i) -> _Float16* { return lds + i * ((C::BM + C::BN) * kLdk); };
  auto sb = [&](int i) -> _Float16* { return lds + i * ((C::BM + C::BN) * kLdk) + C::BM * kLdk; };
#pragma unroll
  for (int x = 0; x < C::TI; ++x)
#pragma unroll
    for (int y = 0; y < C::TJ; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0;
  const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.codes + rbase * a.row_words), (short)0, (int)(rows * a.row_words * 4), 0x00020000);
  const char* qb = kBytes ? reinterpret_cast<const char*>(a.q8) : reinterpret_cast<const char*>(a.qhi);
  const __amdgpu_buffer_rsrc_t rsQ = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(qb + qbase * a.D * kES), (short)0, qrows * a.D * kES, 0x00020000);
  // this thread's share of a slab: 16 codes (fp16) or 32 (bytes) of row tid / 4,
  // and kPerB 16-byte pieces of the queries; byte offsets of slab 0
  constexpr int kNW = Op::template kWords<B>;
  const int urow = tid >> 2, upart = tid & 3;
  const int w0 = kBytes ? upart * B : (upart >> 1) * B + (upart & 1) * (B / 2);
  const uint32_t voc = urow < rows ? (uint32_t)(urow * a.row_words + w0) * 4u : kOffOOB;
  uint32_t voq[C::kPerB];
#pragma unroll
  for (int q = 0; q < C::kPerB; ++q) {
    const int c = tid + C::kThreads * q;
    voq[q] = (c >> 3) < qrows ? (uint32_t)((c >> 3) * a.D * kES + (c & 7) * 16) : kOffOOB;
  }
  // columns k0 + cc (codes) and k0 + cq (queries) must lie inside the row (D is
  // a multiple of 32, so the last slab may be partly empty)
  const int cc = kBytes ? upart * 32 : (upart >> 1) * 32, cq = (tid & 7) * (16 / kES);
  auto load = [&](int s, uint32_t (&cw)[kNW], uint4 (&qv)[C::kPerB]) {
    const int k0 = s * Op::kCols;
    load_words<kNW>(rsC, k0 + cc < a.D ? voc : kOffOOB, (uint32_t)(s * (Op::kCols / 32) * B) * 4u, cw);
#pragma unroll
    for (int q = 0; q < C::kPerB; ++q)
      qv[q] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(rsQ, k0 + cq < a.D ? voq[q] : kOffOOB, (uint32_t)k0 * kES, 0));
  };
  auto store = [&](int st, const uint32_t (&cw)[kNW], const uint4 (&qv)[C::kPerB]) {
    _Float16* dst = sa(st) + urow * kLdk + upart * 16;
    if constexpr (kBytes) {
      uint32_t o[8];
      unpack_bytes<B>(cw, o);
      *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<uint4*>(dst + 8) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
      _Float16 h[16];
      unpack16<B>(cw, upart & 1, a.sh, h);
      *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(h);
      *reinterpret_cast<uint4*>(dst + 8) = *reinterpret_cast<const uint4*>(h + 8);
    }
    slab_store_n<C::kPerB>(sb(st), qv, C::kThreads);
  };
  auto compute = [&](int st) {
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      half8 fa[C::TI], fb[C::TJ];
#pragma unroll
      for (int t = 0; t < C::TI; ++t) fa[t] = frag_load(sa(st), wm * C::TI * 32 + t * 32, kk);
#pragma unroll
      for (int t = 0; t < C::TJ; ++t) fb[t] = frag_load(sb(st), wn * C::TJ * 32 + t * 32, kk);
#pragma unroll
      for (int x = 0; x < C::TI; ++x)
#pragma unroll
        for (int y = 0; y < C::TJ; ++y) acc[x][y] = Op::mfma(fa[x], fb[y], acc[x][y]);
    }
  };
  const int S = (a.D + Op::kCols - 1) / Op::kCols;
  if constexpr (SETS == 3) {
    uint32_t cw[3][kNW];
    uint4 qv[3][C::kPerB];
#pragma unroll
    for (int u = 0; u < 3; ++u) load(u, cw[u], qv[u]);
    store(0, cw[0], qv[0]);
    load(3, cw[0], qv[0]);
    __syncthreads();
    for (int s = 0; s < S; s += 6) {
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        compute(u & 1);
        if (s + u + 1 >= S) break;
        const int v = (u + 1) % 3;
        store((u + 1) & 1, cw[v], qv[v]);
        load(s + u + 4, cw[v], qv[v]);
        __syncthreads();
      }
    }
  } else {
    uint32_t cw[kNW];
    uint4 qv[C::kPerB];
    load(0, cw, qv);
    store(0, cw, qv);
    load(1, cw, qv);
    __syncthreads();
    for (int s = 0; s < S; s += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        compute(u);
        if (s + u + 1 >= S) break;
        store(u ^ 1, cw, qv);
        load(s + u + 2, cw, qv);
        __syncthreads();
      }
    }
  }
}

// The filter's epilogue: every row with H = osc * acc at or above the query's
// threshold goes to its candidate buffer.
template <class C, class Acc>
__device__ __forceinline__ void filter_append(const ScoreArgs& a, int64_t rbase, int rows, int wm,
                                              const int64_t (&j)[C::TJ], const bool (&jv)[C::TJ],
                                              const float (&th)[C::TJ], const float (&osc)[C::TJ],
                                              const Acc (&acc)[C::TI][C::TJ]) {
  const int lane = threadIdx.x & 63;
  // a tile whose store rows are all valid needs no per-element row test
  const bool full = rows == C::BM;
#pragma unroll
  for (int y = 0; y < C::TJ; ++y) {
    // the tile's largest raw accumulator first (osc >= 0)
    auto amx = acc[0][y][0];
    if (full) {
#pragma unroll
      for (int x = 0; x < C::TI; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) amx = max(amx, acc[x][y][r]);
    } else {
      bool any = false;
#pragma unroll
      for (int x = 0; x < C::TI; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool in = wm * C::TI * 32 + x * 32 + acc_row(r, lane) < rows;
          amx = in ? (any ? max(amx, acc[x][y][r]) : acc[x][y][r]) : amx;
          any |= in;
        }
      if (!any) continue;
    }
    const bool hot = jv[y] && (float)amx * osc[y] >= th[y];
    if (__ballot(hot) == 0ull || !hot) continue;
    uint32_t c = 0u;
#pragma unroll
    for (int x = 0; x < C::TI; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        c += (wm * C::TI * 32 + x * 32 + acc_row(r, lane) < rows && (float)acc[x][y][r] * osc[y] >= th[y]) ? 1u : 0u;
    uint32_t idx = atomicAdd(&a.cand_cnt[j[y]], c);
#pragma unroll
    for (int x = 0; x < C::TI; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl_ = wm * C::TI * 32 + x * 32 + acc_row(r, lane);
        const float sc = (float)acc[x][y][r] * osc[y];
        if (rl_ < rows && sc >= th[y]) {
          if (idx < a.cap) {
            a.cand_s[j[y] * a.cap + idx] = sc;
            a.cand_r[j[y] * a.cap + idx] = (int)(rbase + rl_);
          }
          ++idx;
        }
      }
  }
}

enum { kFilter = 0, kSample = 1, kFilterBytes = 2 };

template <class C, int B, int MODE, int SETS>
__global__ __launch_bounds__(C::kThreads, C::kMinWaves) void k_filter(ScoreArgs a) {
  static_assert(MODE != kSample || (C::BM == kTB && C::TJ == 1), "the sample pass runs on 128-row tiles of one query block");
  __shared__ _Float16 lds[C::kLdsHalves];
  const int64_t nt = a.tile_end;   // store tiles of this pass (tile_begin = 0)
  // 32-bit index arithmetic: the host keeps the grid (nqt * nt) below 2^31
  const uint32_t logical = (uint32_t)xcd_remap32((int)blockIdx.x, (int)(a.nqt * nt));
  const uint32_t per = (uint32_t)(kFilterGroupQ * nt);
  const uint32_t g = logical / per;
  const uint32_t l = logical - g * per;
  const uint32_t gsize = (uint32_t)min(kFilterGroupQ, a.nqt - (int)g * kFilterGroupQ);
  const int qt = (int)(g * kFilterGroupQ + l % gsize);
  const int64_t rbase = (int64_t)(l / gsize) * C::BM;
  const int rows = (int)min<int64_t>(C::BM, a.n - rbase);
  const int64_t qbase = (int64_t)qt * C::BN;
  const int qrows = (int)min<int64_t>(C::BN, a.nq - qbase);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  if constexpr (MODE == kFilterBytes) {
    if (a.coarse[qbase / kPrecQueries] == 0u) {
      int64_t j[C::TJ];
      bool jv[C::TJ];
      float th[C::TJ], osc[C::TJ];
#pragma unroll
      for (int y = 0; y < C::TJ; ++y) {
        j[y] = qbase + wn * C::TJ * 32 + y * 32 + (lane & 31);
        jv[y] = j[y] < a.nq;
        th[y] = jv[y] ? a.thr[a.nq + j[y]] : 0.0f;
        osc[y] = jv[y] ? a.meta[j[y]].osc8 : 0.0f;
      }
      intx16 acc[C::TI][C::TJ];
      scan_tile<C, OpI8, B, (B <= 8 ? SETS : 1)>(a, rbase, rows, qbase, qrows, lds, acc);
      filter_append<C>(a, rbase, rows, wm, j, jv, th, osc, acc);
      return;
    }
  }
  // this lane's queries and their thresholds, loaded before the GEMM
  int64_t j[C::TJ];
  bool jv[C::TJ];
  float th[C::TJ], osc[C::TJ];
#pragma unroll
  for (int y = 0; y < C::TJ; ++y) {
    j[y] = qbase + wn * C::TJ * 32 + y * 32 + (lane & 31);
    jv[y] = j[y] < a.nq;
    th[y] = (jv[y] && MODE != kSample) ? a.thr[j[y]] : 0.0f;
    osc[y] = jv[y] ? a.meta[j[y]].osc : 0.0f;
  }

  floatx16 acc[C::TI][C::TJ];
  scan_tile<C, OpF16, B, SETS>(a, rbase, rows, qbase, qrows, lds, acc);
  if constexpr (MODE == kSample) {
    // this lane's best H over its 32 rows
    float best = -INFINITY;
#pragma unroll
    for (int x = 0; x < C::TI; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) best = fmaxf(best, acc[x][0][r]);
    if (jv[0]) {
      const int tile = (int)(l / gsize);
      const int64_t o = j[0] * ((int64_t)a.sample_tiles * kSampleEntries) +
                        (tile % a.sample_tiles) * kSampleEntries + wm * 2 + (lane >> 5);
      // (osc > 0; folded entries were set to order code 0 and are read as such)
      if (nt <= a.sample_tiles) a.part_s[o] = best * osc[0];
      else atomicMax(reinterpret_cast<uint32_t*>(a.part_s) + o, f2ord(best * osc[0]));
    }
    return;
  }
  filter_append<C>(a, rbase, rows, wm, j, jv, th, osc, acc);
}

// large: the filter pass on FilterTileL (a.nqt and a.tile_end in its tiles).
// Codes of more than 14 bits keep one slab of loads in flight (three sets of
// their words do not fit in the registers).
template <int B, int MODE>
lam_status launch_filter(int b, bool large, int64_t grid, hipStream_t st, const ScoreArgs& a) {
  if (b == B) {
    if constexpr (MODE == kFilter || MODE == kFilterBytes) {
      if (large) {
        hipLaunchKernelGGL((k_filter<FilterTileL, B, MODE, 1>), dim3((unsigned)grid), dim3(FilterTileL::kThreads), 0,
                           st, a);
        LAM_HIP(hipGetLastError());
        return LAM_OK;
      }
    }
    hipLaunchKernelGGL((k_filter<FilterTile, B, MODE, (B <= 14 ? 3 : 1)>), dim3((unsigned)grid),
                       dim3(FilterTile::kThreads), 0, st, a);
    LAM_HIP(hipGetLastError());
    return LAM_OK;
  }
  if constexpr (B < (MODE == kFilterBytes ? 12 : kMaxBits)) return launch_filter<B + 1, MODE>(b, large, grid, st, a);
  set_error("scoring supports codes of at most %d bits (got %d)", kMaxBits, b);
  return LAM_ESTATE;
}

// ------------------------------------------------------------------ rescoring
constexpr int kRescoreThreads = 256;
constexpr int kRescoreLanes = 8;     // lanes per rescored row

// q . code over the groups of 32 codes g = sl, sl + 8, ... of a row (words at
// w), in binary64: one lane's share.  Products of a float32 and a code of at
// most 22 bits are exact in binary64.
template <int B>
__device__ __forceinline__ double lane_dot(const uint32_t* __restrict__ w, const float* __restrict__ q, int ngroups,
                                           int sl) {
  double acc = 0.0;
  for (int g = sl; g < ngroups; g += kRescoreLanes) {
    uint32_t cw[B];
#pragma unroll
    for (int i = 0; i < B; ++i) cw[i] = w[g * B + i];
    float qv[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) qv[e] = q[g * 32 + e];
#pragma unroll
    for (int e = 0; e < 32; ++e) acc = fma((double)qv[e], (double)code_at<B>(cw, e), acc);
  }
  return acc;
}

// The key of a row's score, ordered by (score desc, row asc): larger is better.
__device__ __forceinline__ unsigned long long score_key(double acc, double step, uint32_t row) {
  return ((unsigned long long)f2ord((float)(acc * step) + 0.0f) << 32) | (unsigned long long)(~row);
}

// Descending bitonic sort of P keys in LDS (P a power of two) by the workgroup.
__device__ __forceinline__ void sort_keys(unsigned long long* keys, uint32_t P) {
  for (uint32_t size = 2; size <= P; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < P; i += kRescoreThreads) {
        const uint32_t l = i ^ stride;
        if (l > i) {
          const unsigned long long x = keys[i], y = keys[l];
          const bool desc = (i & size) == 0;
          if (desc ? (x < y) : (x > y)) {
            keys[i] = y;
            keys[l] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}

// The best k of any number of keys: keys above the k-th found so far are
// appended to a buffer of N, which is sorted and cut back to k when the next
// step might not fit.
constexpr int kTopKeys = 1024;   // the selections' buffer

template <int N>
struct TopBuf {
  unsigned long long keys[N];
  unsigned long long floor;   // keys up to it are not in the top k
  uint32_t cnt;
};

// Called by the whole workgroup; ends with a barrier.
template <int N>
__device__ __forceinline__ void topbuf_clear(TopBuf<N>& b) {
  if (threadIdx.x == 0) {
    b.cnt = 0u;
    b.floor = 0ull;
  }
  __syncthreads();
}

template <int N>
__device__ __forceinline__ void topbuf_push(TopBuf<N>& b, unsigned long long key) {
  if (key > b.floor) b.keys[atomicAdd(&b.cnt, 1u)] = key;
}

// Called by the whole workgroup past a barrier: room for `room` more keys.
template <int N>
__device__ __forceinline__ void topbuf_cut(TopBuf<N>& b, int k, uint32_t room) {
  const uint32_t c = b.cnt;
  __syncthreads();   // every thread has the same count before any pushes again
  if (c + room <= (uint32_t)N) return;
  for (uint32_t i = c + threadIdx.x; i < (uint32_t)N; i += kRescoreThreads) b.keys[i] = 0ull;
  __syncthreads();
  sort_keys(b.keys, N);
  if (threadIdx.x == 0) {
    b.cnt = min(c, (uint32_t)k);
    b.floor = c >= (uint32_t)k ? b.keys[k - 1] : 0ull;
  }
  __syncthreads();
}

// The same by one wave (all its lanes), which alone touches b meanwhile: LDS
// operations of a wave complete in order, so the steps need no barrier.
template <int N>
__device__ __forceinline__ void topbuf_cut_wave(TopBuf<N>& b, int k, uint32_t room) {
  const uint32_t c = b.cnt, lane = threadIdx.x & 63u;
  if (c + room <= (uint32_t)N) return;
  auto step = []() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  for (uint32_t i = c + lane; i < (uint32_t)N; i += 64) b.keys[i] = 0ull;
  step();
#pragma unroll 1   // (unrolled, the steps' addresses and masks take every register)
  for (uint32_t size = 2; size <= (uint32_t)N; size <<= 1) {
#pragma unroll 1
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
#pragma unroll
      for (uint32_t t = 0; t < (uint32_t)N / 2; t += 64) {
        const uint32_t p = t + lane, i = 2 * p - (p & (stride - 1)), l = i | stride;   // pair p of this stride
        const unsigned long long x = b.keys[i], y = b.keys[l];
        const bool swap = (i & size) == 0 ? x < y : x > y;
        b.keys[i] = swap ? y : x;
        b.keys[l] = swap ? x : y;
      }
      step();
    }
  }
  if (lane == 0) {
    b.cnt = min(c, (uint32_t)k);
    b.floor = c >= (uint32_t)k ? b.keys[k - 1] : 0ull;
  }
  step();
}

// The exact score of row t of a list of m rows in LDS, by the eight lanes of
// slot t % 32; true for the lane that holds the key.
template <int B>
__device__ __forceinline__ bool rescore_row(uint32_t t, uint32_t m, const int32_t* rows, const float* __restrict__ qj,
                                            double step, const uint32_t* __restrict__ codes, int64_t row_words, int D,
                                            unsigned long long& key) {
  const int sl = (int)threadIdx.x % kRescoreLanes;
  double acc = 0.0;
  if (t < m) acc = lane_dot<B>(codes + (int64_t)rows[t] * row_words, qj, D / 32, sl);
  for (int o = kRescoreLanes / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);   // within the row's lanes
  if (t >= m || sl != 0) return false;
  key = score_key(acc, step, (uint32_t)rows[t]);
  return true;
}

// One workgroup per query: the selection among the candidates and the exact
// scores.  With h_k the k-th best hi-only score H of the candidates, every row
// of the final top-k has H >= h_k - 2 err (k rows have S >= h_k - err, and
// |H - S| <= err), so those candidates are rescored from the codes and the
// float32 query, summed in binary64 and rounded once to float32, and the k
// best by (S desc, row asc) are the answer.  Any lower bound of h_k serves:
// wave 0 takes the one of wave_kth_floor (beyond 1,024 candidates several
// share a key as their maximum), which costs the same for every k.  Up to 1,024
// such rows are sorted at once; more (many near-equal scores) go through the
// buffer in steps of 256 candidates.  An overflowed candidate buffer, or a query
// that is not scanned, flags the query for the exact pass.  Also writes the bound, NaN outputs for an invalid
// query, and (-inf, -1) past the candidates.  Eight lanes share a rescored row
// (32 rows in flight per workgroup); a lane takes whole groups of 32 codes (B
// words).
template <int B>
__global__ __launch_bounds__(kRescoreThreads) void k_select_rescore(
    int64_t nq, uint32_t cap, int k, const uint32_t* __restrict__ cnt, const float* __restrict__ cs,
    const int32_t* __restrict__ cr, const QMeta* __restrict__ meta, const int64_t* __restrict__ ids,
    const float* __restrict__ q, double step, const uint32_t* __restrict__ codes, int64_t row_words, int D,
    float* __restrict__ out_s, int64_t* __restrict__ out_i, float* __restrict__ bound, uint32_t* __restrict__ n_flag,
    uint32_t* __restrict__ flagged, const uint32_t* __restrict__ coarse) {
  constexpr int kCap = kTopKeys;
  __shared__ int32_t rows[kCap];
  __shared__ TopBuf<kTopKeys> buf;
  __shared__ uint32_t m_sh;
  __shared__ float thr_sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t j = blockIdx.x;
  if (j >= nq) return;
  const uint32_t c = cnt[j];
  const QMeta mj = meta[j];
  const float err = coarse && coarse[j / kPrecQueries] == 0u ? mj.err8 : mj.err;   // of the scan that ran
  if (tid == 0 && bound) bound[j] = mj.bound;
  if (mj.kind == kInvalid) {
    for (int t = tid; t < k; t += kRescoreThreads) {
      out_s[j * k + t] = __builtin_nanf("");
      out_i[j * k + t] = -1;
    }
    return;
  }
  if (mj.kind == kZero) {   // (a store on this path has more than k rows)
    for (int t = tid; t < k; t += kRescoreThreads) {
      out_s[j * k + t] = 0.0f;
      out_i[j * k + t] = ids[t];
    }
    return;
  }
  if (mj.kind == kUnscanned || c > cap) {   // left to the exact pass
    if (tid == 0) flagged[atomicAdd(n_flag, 1u)] = (uint32_t)j;
    return;
  }
  const int kk = (int)min((uint32_t)k, c);
  for (int t = kk + tid; t < k; t += kRescoreThreads) {   // fewer candidates than k
    out_s[j * k + t] = -INFINITY;
    out_i[j * k + t] = -1;
  }
  if (kk == 0) return;
  // every thread's first two candidates for the threshold test below, loaded
  // while wave 0 selects
  float fs[2];
  int fr[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t i = (uint32_t)(tid + u * kRescoreThreads);
    fs[u] = i < c ? cs[j * cap + i] : 0.0f;
    fr[u] = i < c ? cr[j * cap + i] : 0;
  }
  if (wave == 0) {
    uint32_t key[kThrKeys];
#pragma unroll
    for (int r = 0; r < kThrKeys; ++r) {
      const uint32_t i = (uint32_t)(lane + r * 64);
      key[r] = i < c ? f2ord(cs[j * cap + i] + 0.0f) : 0u;
    }
    for (uint32_t e0 = 64 * kThrKeys; e0 < c; e0 += 64 * kThrKeys)
#pragma unroll
      for (int r = 0; r < kThrKeys; ++r) {
        const uint32_t i = e0 + (uint32_t)(lane + r * 64);
        if (i < c) key[r] = max(key[r], f2ord(cs[j * cap + i] + 0.0f));
      }
    const uint32_t T = wave_kth_floor<kThrKeys>(key, (int)min((uint32_t)kThrKeys, (c + 63u) / 64u), kk);
    if (lane == 0) {
      thr_sh = rd32(floor_score(T) - 2.0 * (double)err);
      m_sh = 0u;
    }
  }
  __syncthreads();
  const float thr = thr_sh;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    if ((uint32_t)(tid + u * kRescoreThreads) < c && fs[u] >= thr) {
      const uint32_t p = atomicAdd(&m_sh, 1u);
      if (p < (uint32_t)kCap) rows[p] = fr[u];
    }
  }
  for (uint32_t i = tid + 2 * kRescoreThreads; i < c; i += kRescoreThreads) {
    if (cs[j * cap + i] >= thr) {
      const uint32_t p = atomicAdd(&m_sh, 1u);
      if (p < (uint32_t)kCap) rows[p] = cr[j * cap + i];
    }
  }
  __syncthreads();
  const uint32_t m = m_sh;
  const float* qj = q + j * D;
  const uint32_t slot = (uint32_t)(tid / kRescoreLanes);
  constexpr uint32_t kSlots = kRescoreThreads / kRescoreLanes;
  unsigned long long key;
  if (m <= (uint32_t)kCap) {
    for (uint32_t t0 = 0; t0 < m; t0 += kSlots)
      if (rescore_row<B>(t0 + slot, m, rows, qj, step, codes, row_words, D, key)) buf.keys[t0 + slot] = key;
    uint32_t P = 1u;
    while (P < m) P <<= 1;
    for (uint32_t i = m + tid; i < P; i += kRescoreThreads) buf.keys[i] = 0ull;   // padding
    __syncthreads();
    sort_keys(buf.keys, P);
  } else {
    topbuf_clear(buf);
    for (uint32_t i0 = 0; i0 < c; i0 += kRescoreThreads) {
      if (tid == 0) m_sh = 0u;
      __syncthreads();
      const uint32_t i = i0 + (uint32_t)tid;
      if (i < c && cs[j * cap + i] >= thr) rows[atomicAdd(&m_sh, 1u)] = cr[j * cap + i];
      __syncthreads();
      const uint32_t mi = m_sh;
      for (uint32_t t0 = 0; t0 < mi; t0 += kSlots)
        if (rescore_row<B>(t0 + slot, mi, rows, qj, step, codes, row_words, D, key)) topbuf_push(buf, key);
      __syncthreads();
      topbuf_cut(buf, k, kRescoreThreads);
    }
    topbuf_cut(buf, k, kTopKeys);   // sorts what is left
  }
  for (int t = tid; t < kk; t += kRescoreThreads) {
    out_s[j * k + t] = ord2f((uint32_t)(buf.keys[t] >> 32));
    out_i[j * k + t] = ids[~(uint32_t)(buf.keys[t] & 0xffffffffull)];
  }
}

// The exact pass over the flagged queries (those whose candidates overflowed, or
// that are not scanned): a work item is a group of up to four flagged queries
// and a range of store rows, all scored exactly.  Eight lanes
// share four rows at a time, 128 rows per step: a code is unpacked and converted
// to binary64 once for the group's queries, and a query's value read from LDS
// (in binary64) once for the four rows.  A range's best k go to the queries' candidate
// buffers (no longer needed), and the last of a
// group's workgroups merges them the same way.  Launched always; without
// flagged queries every workgroup returns after one load.
// A call of 128 queries against 361,802 rows, D = 768, top-10, of which 1, 8 or
// all are flagged by 5,000 equal rows: 0.36, 0.52 and 2.6 ms (one query per work
// item and 885 rows per range: 0.39, 1.01 and 13.9 ms; sorted per-lane lists
// behind an fp16 scan of the whole 128-query tile: 0.99, 1.27 and 9.1 ms).  128
// flagged of 300 against 60,000 x 384, top-50: 0.84 ms (2.45; lists 40 ms); 1,000
// of 1,000 against 30,000 x 768: 1.9 ms (19; lists 1.35 ms, the one case found
// where their fp16 products were faster than the binary64 ones here).
constexpr int kExactRows = 4;      // rows per slot and step
constexpr int kExactQueries = 4;   // flagged queries per work item
constexpr int kExactPerCU = 3;     // workgroups that a CU holds at the usual code widths
constexpr int kExactKeys = 256;    // >= 64 + one step's rows
constexpr int kExactStep = kRescoreThreads / kRescoreLanes * kExactRows;

// LDS doubles per group of 32 columns: a column's Q values side by side, groups
// padded to distinct banks.
constexpr int exact_ld(int Q) { return 32 * Q + (Q == 1 ? 1 : 2); }

// (double)c for any int32, by the exponent of 2^52: an exclusive-or and a
// subtraction, where v_cvt_f64_i32 takes four times as long as either.
__device__ __forceinline__ double exact_f64(int32_t c) {
  return __hiloint2double(0x43300000, c ^ (int32_t)0x80000000) - 0x1.000008p52;
}

// Sums of N values over the eight lanes of a slot: while a lane holds several it
// hands half of them over at each step, so lane sl ends with max(1, N / 8)
// sums, those from index exact_first(N, sl).
template <int N, int O>
__device__ __forceinline__ void oct_sums(double* v, int sl) {
  if constexpr (O > 0) {
    if constexpr (N > 1) {
      const bool up = (sl & O) != 0;
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const double give = up ? v[i] : v[i + N / 2];
        v[i] = (up ? v[i + N / 2] : v[i]) + __shfl_xor(give, O);
      }
      oct_sums<N / 2, O / 2>(v, sl);
    } else {
      v[0] += __shfl_xor(v[0], O);
      oct_sums<1, O / 2>(v, sl);
    }
  }
}

// The rows [r0, r1) against the Q queries in qs (nq of them real), into their
// buffers.
template <int B, int Q>
__device__ __forceinline__ void exact_range(const uint32_t* __restrict__ codes, int64_t row_words, int64_t n, int64_t r0,
                                            int64_t r1, int ngroups, const double* qs, double step, int k, int nq,
                                            TopBuf<kExactKeys>* buf) {
  constexpr int kSlots = kRescoreThreads / kRescoreLanes;
  constexpr int N = Q * kExactRows, kMine = N >= kRescoreLanes ? N / kRescoreLanes : 1;
  static_assert(kRescoreLanes == 8 && (N == 4 || N == 16), "sums over eight lanes");
  const int slot = (int)threadIdx.x / kRescoreLanes, sl = (int)threadIdx.x % kRescoreLanes;
  for (int64_t r = r0; r < r1; r += kExactStep) {
    double acc[N];   // query u, row v at u * kExactRows + v
    const uint32_t* w[kExactRows];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.0;
#pragma unroll
    for (int v = 0; v < kExactRows; ++v)
      w[v] = codes + min(r + v * kSlots + slot, n - 1) * row_words;   // (a row past the range is not used)
    for (int g = sl; g < ngroups; g += kRescoreLanes) {
      uint32_t cw[kExactRows][B];
#pragma unroll
      for (int v = 0; v < kExactRows; ++v)
#pragma unroll
        for (int i = 0; i < B; ++i) cw[v][i] = w[v][g * B + i];
      const double* qg = qs + g * exact_ld(Q);
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        double qe[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) qe[u] = qg[e * Q + u];
#pragma unroll
        for (int v = 0; v < kExactRows; ++v) {
          const double c = exact_f64(code_at<B>(cw[v], e));
#pragma unroll
          for (int u = 0; u < Q; ++u) acc[u * kExactRows + v] = fma(qe[u], c, acc[u * kExactRows + v]);
        }
      }
    }
    oct_sums<N, kRescoreLanes / 2>(acc, sl);
    // the lane's sums: with 16 of them two each, with 4 one for two lanes
    const int first = N == 16 ? sl * 2 : sl >> 1;
    if (N == 16 || (sl & 1) == 0) {
#pragma unroll
      for (int i = 0; i < kMine; ++i) {
        const int u = (first + i) / kExactRows;
        const int64_t row = r + (int64_t)((first + i) % kExactRows) * kSlots + slot;
        if (row < r1 && u < nq) topbuf_push(buf[u], score_key(acc[i], step, (uint32_t)row));
      }
    }
    __syncthreads();
    if ((int)threadIdx.x >> 6 < Q) topbuf_cut_wave(buf[threadIdx.x >> 6], k, kExactStep);
    __syncthreads();
  }
}

template <int B>
__global__ __launch_bounds__(kRescoreThreads, B <= 13 ? kExactPerCU : 2) void k_exact(
    int64_t n, uint32_t cap, int k, const int64_t* __restrict__ ids,
    const float* __restrict__ q, double step, const uint32_t* __restrict__ codes, int64_t row_words, int D,
    float* __restrict__ cs, int32_t* __restrict__ cr, uint32_t* __restrict__ done, const uint32_t* __restrict__ n_flag,
    const uint32_t* __restrict__ flagged, float* __restrict__ out_s, int64_t* __restrict__ out_i) {
  const uint32_t nf = *n_flag;
  if (nf == 0u) return;
  extern __shared__ __attribute__((aligned(16))) double qs[];   // the group's queries (exact_ld per 32 columns)
  __shared__ TopBuf<kExactKeys> buf[kExactQueries];
  __shared__ bool last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ngroups = D / 32;
  // ranges of at least two steps whose lists fit the candidate buffer; groups
  // only where they leave every CU kExactPerCU workgroups, and then no more
  // ranges than give it four times that (every range costs its lists' sorts)
  constexpr uint64_t kFill = (uint64_t)kExactPerCU * 256;
  const uint64_t most = min((uint64_t)(cap / (uint32_t)k), ((uint64_t)n + 2 * kExactStep - 1) / (2 * kExactStep));
  const uint32_t per = (uint64_t)nf * most >= kExactQueries * kFill ? kExactQueries : 1u;
  const uint64_t groups = ((uint64_t)nf + per - 1) / per;
  const int splits = (int)min(most, (4 * kFill + groups - 1) / groups);
  const int64_t rows_per_split = (n + splits - 1) / splits;
  const uint64_t items = groups * (uint64_t)splits;
  for (uint64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const uint32_t* fl = flagged + it / (uint64_t)splits * per;
    const int nq = (int)min(per, nf - (uint32_t)(fl - flagged));
    const int sp = (int)(it % (uint64_t)splits);
    const int64_t r0 = sp * rows_per_split, r1 = min(n, r0 + rows_per_split);
    const int Q = nq == 1 ? 1 : kExactQueries;
    for (int u = 0; u < Q; ++u) {
      const float* qj = q + (int64_t)fl[min(u, nq - 1)] * D;   // (a place without a query repeats the last)
      for (int d = tid; d < D; d += kRescoreThreads) qs[(d >> 5) * exact_ld(Q) + (d & 31) * Q + u] = (double)qj[d];
      topbuf_clear(buf[u]);
    }
    if (nq == 1)
      exact_range<B, 1>(codes, row_words, n, r0, r1, ngroups, qs, step, k, nq, buf);
    else
      exact_range<B, kExactQueries>(codes, row_words, n, r0, r1, ngroups, qs, step, k, nq, buf);
    if (wave < nq) {
      topbuf_cut_wave(buf[wave], k, kExactKeys);   // sorts what is left
      const int64_t j = fl[wave];
      if (lane < k) {
        const unsigned long long key = lane < (int)buf[wave].cnt ? buf[wave].keys[lane] : 0ull;
        cs[j * cap + sp * k + lane] = __uint_as_float((uint32_t)(key >> 32));
        cr[j * cap + sp * k + lane] = (int32_t)(uint32_t)key;
      }
    }
    // release this range's keys, count it (on the group's first query), and let
    // the group's last range acquire all of them
    __threadfence();
    __syncthreads();
    if (tid == 0) last = atomicAdd(&done[fl[0]], 1u) == (uint32_t)(splits - 1);
    __syncthreads();
    if (!last) continue;
    __threadfence();
    // a wave merges one query's ranges
    for (int u = 0; u < nq; ++u) topbuf_clear(buf[u]);
    if (wave < nq) {
      TopBuf<kExactKeys>& b = buf[wave];
      const int64_t j = fl[wave];
      constexpr int kAhead = 8;   // keys per lane loaded together
      for (int t0 = 0; t0 < splits * k; t0 += 64 * kAhead) {
        unsigned long long key[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
          const int64_t t = j * cap + min(t0 + a * 64 + lane, splits * k - 1);
          key[a] = ((unsigned long long)__float_as_uint(cs[t]) << 32) | (unsigned long long)(uint32_t)cr[t];
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
          if (t0 + a * 64 + lane < splits * k) topbuf_push(b, key[a]);
          topbuf_cut_wave(b, k, 64);
        }
      }
      topbuf_cut_wave(b, k, kExactKeys);
      if (lane < k) {   // (a flagged query has more than k rows)
        out_s[j * k + lane] = ord2f((uint32_t)(b.keys[lane] >> 32));
        out_i[j * k + lane] = ids[~(uint32_t)(b.keys[lane] & 0xffffffffull)];
      }
    }
    __syncthreads();
  }
}
static_assert(kExactKeys >= 64 + kExactStep, "a cut leaves room for a step");

// The rows scored exactly: arguments shared by the selection and the exact pass.
struct ExactArgs {
  int64_t nq, n;
  uint32_t cap;
  int k;
  uint32_t* cnt;
  float* cs;
  int32_t* cr;
  const QMeta* meta;
  const int64_t* ids;
  const float* q;
  double step;
  const uint32_t* codes;
  int64_t row_words;
  int D;
  float* out_s;
  int64_t* out_i;
  float* bound;
  uint32_t *n_flag, *flagged, *done;
  const uint32_t* coarse;   // byte scan: the flags of the queries that took the fp16 scan (else NULL)
};

// The selection, or the exact pass over the flagged queries.
template <int B>
lam_status launch_exact(int b, bool select, hipStream_t st, const ExactArgs& a) {
  if (b == B) {
    if (select)
      hipLaunchKernelGGL((k_select_rescore<B>), dim3((unsigned)a.nq), dim3(kRescoreThreads), 0, st, a.nq, a.cap, a.k,
                         a.cnt, a.cs, a.cr, a.meta, a.ids, a.q, a.step, a.codes, a.row_words, a.D, a.out_s, a.out_i,
                         a.bound, a.n_flag, a.flagged, a.coarse);
    else
      hipLaunchKernelGGL((k_exact<B>), dim3(1024), dim3(kRescoreThreads), (size_t)(a.D / 32) * exact_ld(kExactQueries) * 8, st, a.n, a.cap, a.k, a.ids, a.q, a.step, a.codes, a.row_words, a.D,
                         a.cs, a.cr, a.done, a.n_flag, a.flagged, a.out_s, a.out_i);
    LAM_HIP(hipGetLastError());
    return LAM_OK;
  }
  if constexpr (B < kMaxBits) return launch_exact<B + 1>(b, select, st, a);
  set_error("scoring supports codes of at most %d bits (got %d)", kMaxBits, b);
  return LAM_ESTATE;
}

__global__ __launch_bounds__(256) void k_fill_zero(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ------------------------------------------------------------------ small stores
// A store of at most kCandCap rows is scored whole: k_dense forms every score
// in fp32 from the query's fp16 hi and lo parts (q 2^e = hi + lo + r, |r| <=
// 2^-22 |q 2^e|), and k_select_dense takes the k best, so that the call is three
// launches.  Codes of more than 12 bits enter as their two exact fp16 halves,
// c = 2^11 (c >> 11) + (c & 2047): 2D columns (the high halves, then the low
// ones) against the query [2^11 q, q].
struct DenseArgs {
  const uint32_t* codes;
  int64_t n;
  int D;                // columns of a row; the scan has D or 2 D
  int64_t row_words;
  const _Float16* qhi;  // [nq][D or 2 D]
  const _Float16* qlo;
  const QMeta* meta;    // osc, bound and kind
  int64_t nq;
  int nqt;
  float* scores;        // [nq][ld]
  int ld;
};

// One wave per query: hi and lo parts of its D columns, or of [2^11 q, q] (wide).
__global__ __launch_bounds__(256) void k_dense_prep(const float* __restrict__ q, int64_t nq, int D, int wide,
                                                    double s, double eps, _Float16* __restrict__ qhi,
                                                    _Float16* __restrict__ qlo, QMeta* __restrict__ meta) {
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= nq) return;
  const float* p = q + j * D;
  const int cols = wide ? 2 * D : D;
  const float up11 = wide ? 2048.0f : 1.0f;
  float mx = 0.0f;
  double l1 = 0.0;
  bool bad = false;
  for (int d = lane * 4; d < D; d += 256) {
    const float4 v = *reinterpret_cast<const float4*>(p + d);
    const float c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a = fabsf(c[i] * up11);
      bad |= !(a <= 3.402823466e38f);
      mx = fmaxf(mx, a);
      l1 += (double)fabsf(c[i]);
    }
  }
  mx = wave_max_f32(mx);
  l1 = wave_sum_f64(l1);
  bad = __ballot(bad) != 0ull;
  int e = 0;
  if (!bad && mx > 0.0f) e = 14 - ilogbf(mx);   // the largest entry times 2^e in [2^14, 2^15)
  for (int d = lane * 4; d < cols; d += 256) {   // (D is a multiple of 32: four columns are of one half)
    const float4 v = *reinterpret_cast<const float4*>(p + (d < D ? d : d - D));
    const float f = d < D ? up11 : 1.0f;
    const float c[4] = {v.x * f, v.y * f, v.z * f, v.w * f};
    _Float16 h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = bad ? 0.0f : ldexpf(c[i], e);   // exact (2^e itself may overflow)
      h[i] = (_Float16)x;
      l[i] = (_Float16)(x - (float)h[i]);
    }
    uint2 ph, pl;
    __builtin_memcpy(&ph, h, 8);
    __builtin_memcpy(&pl, l, 8);
    *reinterpret_cast<uint2*>(qhi + j * cols + d) = ph;
    *reinterpret_cast<uint2*>(qlo + j * cols + d) = pl;
  }
  if (lane == 0) {
    QMeta m{};
    // s 2^-e, times 2^126 and negative where float32 could not hold it as a normal value
    const bool far = ilogb(s) - e < -120;
    m.osc = fminf((float)ldexp(s, far ? 126 - e : -e), 3.402823466e38f);
    if (far) m.osc = -m.osc;
    m.bound = bad ? __builtin_nanf("") : ru32(eps * l1 * (1.0 + (double)(cols + 4) * 0x1p-52));
    m.kind = bad ? kInvalid : kScanned;
    meta[j] = m;
  }
}

// One 128 x 128 tile (store rows x queries) per workgroup of four waves, each
// 128 rows x 32 queries; one LDS stage (codes, hi, lo) is refilled between two
// barriers while the next slab's loads are in flight in registers.  Two threads
// unpack a row's slab, a group of 32 codes each.
template <int B>
__global__ __launch_bounds__(kWG, 2) void k_dense(DenseArgs a) {
  constexpr bool kWide = B > 12;
  __shared__ __attribute__((aligned(16))) _Float16 lds[3 * kTB * kLdk];
  _Float16* sc = lds;
  _Float16* sh = lds + kTB * kLdk;
  _Float16* sl = lds + 2 * kTB * kLdk;
  const int qt = (int)blockIdx.x % a.nqt;
  const int64_t rbase = (int64_t)(blockIdx.x / a.nqt) * kTB;
  const int rows = (int)min<int64_t>(kTB, a.n - rbase);
  const int64_t qbase = (int64_t)qt * kTB;
  const int qrows = (int)min<int64_t>(kTB, a.nq - qbase);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int urow = threadIdx.x >> 1, uhalf = threadIdx.x & 1;
  const int cols = kWide ? 2 * a.D : a.D;
  const int64_t j = qbase + wave * 32 + (lane & 31);
  const float osc = j < a.nq ? a.meta[j].osc : 0.0f;
  floatx16 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
  const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.codes + rbase * a.row_words), (short)0, (int)(rows * a.row_words * 4), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsH = tile_rsrc(a.qhi + qbase * cols, qrows, cols);
  const __amdgpu_buffer_rsrc_t rsL = tile_rsrc(a.qlo + qbase * cols, qrows, cols);
  const int G = a.D / 32;   // groups of a row; group g + G of the scan holds group g's low halves
  auto load_slab = [&](int k0, uint32_t (&cw)[B], uint4 (&rh)[4], uint4 (&rl)[4]) {
    const int g = k0 / 32 + uhalf;
    const bool ok = urow < rows && k0 + 32 * uhalf < cols;
    const uint32_t w0 = (uint32_t)(urow * a.row_words + (int64_t)(kWide && g >= G ? g - G : g) * B);
    load_words<B>(rsC, ok ? w0 * 4u : kOffOOB, 0u, cw);
    slab_load_n<4>(rsH, qrows, cols, k0, cols, rh, kWG);
    slab_load_n<4>(rsL, qrows, cols, k0, cols, rl, kWG);
  };
  const int S = (cols + kBK - 1) / kBK;
  uint32_t cw[B];
  uint4 rh[4], rl[4];
  load_slab(0, cw, rh, rl);
  for (int s = 0; s < S; ++s) {
    __syncthreads();   // every wave is done with the previous slab
    {
      const bool low = kWide && 2 * s + uhalf >= G;
      _Float16 h[32];
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        int32_t c = code_at<B>(cw, e);
        if (kWide) c = low ? (c & 2047) : (c >> 11);
        h[e] = (_Float16)(short)c;
      }
      _Float16* dst = sc + urow * kLdk + uhalf * 32;
#pragma unroll
      for (int i = 0; i < 32; i += 8) *reinterpret_cast<uint4*>(dst + i) = *reinterpret_cast<const uint4*>(h + i);
    }
    slab_store_n<4>(sh, rh, kWG);
    slab_store_n<4>(sl, rl, kWG);
    __syncthreads();
    load_slab((s + 1) * kBK, cw, rh, rl);   // past the last slab: zeros, no memory touched
    __builtin_amdgcn_sched_barrier(0);      // issue the loads before the MFMAs
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      const half8 bh = frag_load(sh, wave * 32, kk);
      const half8 bl = frag_load(sl, wave * 32, kk);
      half8 fa[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) fa[t] = frag_load(sc, t * 32, kk);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[t], bh, acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[t], bl, acc[t], 0, 0, 0);
    }
  }
  if (j >= a.nq) return;
  // this lane's rows, four consecutive ones per store (ld covers whole tiles)
  float* o = a.scores + j * a.ld + rbase;
  auto put = [&](float sa, float sb) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(o + t * 32 + acc_row(4 * g, lane)) =
            make_float4(acc[t][4 * g] * sa * sb, acc[t][4 * g + 1] * sa * sb, acc[t][4 * g + 2] * sa * sb,
                        acc[t][4 * g + 3] * sa * sb);
  };
  if (osc >= 0.0f) put(osc, 1.0f);
  else put(-osc, 0x1p-126f);
}

template <int B>
lam_status launch_dense(int b, dim3 grid, hipStream_t st, const DenseArgs& a) {
  if (b == B) {
    hipLaunchKernelGGL((k_dense<B>), grid, dim3(kWG), 0, st, a);
    LAM_HIP(hipGetLastError());
    return LAM_OK;
  }
  if constexpr (B < kMaxBits) return launch_dense<B + 1>(b, grid, st, a);
  set_error("scoring supports codes of at most %d bits (got %d)", kMaxBits, b);
  return LAM_ESTATE;
}

// One workgroup per query: the k best of the n <= kCandCap scores, held 16 per
// thread.  The largest of the waves' own k-th best is a lower bound of the
// k-th best of all; what reaches it is sorted (through the buffer in steps when
// more than 1,024 tie there).
__global__ __launch_bounds__(kRescoreThreads) void k_select_dense(int64_t nq, int n, int ld, int k,
                                                                  const float* __restrict__ scores,
                                                                  const QMeta* __restrict__ meta,
                                                                  const int64_t* __restrict__ ids,
                                                                  float* __restrict__ out_s,
                                                                  int64_t* __restrict__ out_i,
                                                                  float* __restrict__ bound) {
  constexpr int kPer = kCandCap / kRescoreThreads;
  static_assert(kPer == kThrKeys, "a wave's keys are one register set");
  __shared__ TopBuf<kTopKeys> buf;
  __shared__ uint32_t floor_sh[kRescoreThreads / 64], cnt_sh[kRescoreThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t j = blockIdx.x;
  if (j >= nq) return;
  const QMeta mj = meta[j];
  if (tid == 0 && bound) bound[j] = mj.bound;
  const bool bad = mj.kind == kInvalid;
  const int kk = bad ? 0 : min(k, n);
  for (int t = kk + tid; t < k; t += kRescoreThreads) {
    out_s[j * k + t] = bad ? __builtin_nanf("") : -INFINITY;
    out_i[j * k + t] = -1;
  }
  if (kk == 0) return;
  uint32_t key[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const int i = tid + r * kRescoreThreads;
    key[r] = i < n ? f2ord(scores[j * ld + i] + 0.0f) : 0u;
  }
  const uint32_t T = wave_kth_floor<kPer>(key, (n + kRescoreThreads - 1) / kRescoreThreads, kk);
  if (lane == 0) floor_sh[wave] = T;
  topbuf_clear(buf);
  uint32_t F = 1u;   // (order code 0 marks no row)
#pragma unroll
  for (int w = 0; w < kRescoreThreads / 64; ++w) F = max(F, floor_sh[w]);
  int c = 0;
#pragma unroll
  for (int r = 0; r < kPer; ++r) c += __popcll(__ballot(key[r] >= F));
  if (lane == 0) cnt_sh[wave] = (uint32_t)c;
  __syncthreads();
  uint32_t m = 0u;
#pragma unroll
  for (int w = 0; w < kRescoreThreads / 64; ++w) m += cnt_sh[w];
  const bool fits = m <= (uint32_t)kTopKeys;
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    if (key[r] >= F)
      topbuf_push(buf, ((unsigned long long)key[r] << 32) | (unsigned long long)(~(uint32_t)(tid + r * kRescoreThreads)));
    if (!fits) {
      __syncthreads();
      topbuf_cut(buf, k, kRescoreThreads);
    }
  }
  __syncthreads();
  if (fits) {
    uint32_t P = 1u;
    while (P < m) P <<= 1;
    for (uint32_t i = m + tid; i < P; i += kRescoreThreads) buf.keys[i] = 0ull;
    __syncthreads();
    sort_keys(buf.keys, P);
  } else {
    topbuf_cut(buf, k, kTopKeys);   // sorts what is left
  }
  for (int t = tid; t < kk; t += kRescoreThreads) {
    out_s[j * k + t] = ord2f((uint32_t)(buf.keys[t] >> 32));
    out_i[j * k + t] = ids[~(uint32_t)(buf.keys[t] & 0xffffffffull)];
  }
}

}  // namespace

// What the scoring passes read of a store: its coded rows (D columns of b-bit
// codes, step s = 2 eps), their ids, R >= s ||code_y|| for every row y, and the
// low bits sh that the scan leaves out so that the rest fits 12 bits.
struct ScoreView {
  int D;
  int b;
  int sh;
  bool bytes;   // every code that occurs fits 8 bits
  int64_t n;
  double step;
  double eps;
  double R;
  const uint32_t* codes;
  const int64_t* ids;
};

namespace {

// R >= ||x_hat_y||: ||x|| from the largest ||x||^2 / 2 of the coded rows
// (float32, rounded up by one part in 2^22) plus ||x_hat - x|| <= eps sqrt(D).
double row_norm_bound(uint32_t hn_max_bits, double eps, int D) {
  float hn;
  std::memcpy(&hn, &hn_max_bits, 4);
  return std::sqrt(2.0 * (double)hn * (1.0 + 0x1p-22)) * (1.0 + 0x1p-50) +
         eps * std::sqrt((double)D) * (1.0 + 0x1p-50);
}

ScoreView store_view(const lam_store* st, const uint32_t* codes) {
  ScoreView v;
  v.D = st->dim;
  v.b = st->q.bits;
  // the width of the codes that occur, which a declared absmax may exceed
  int used = 1;
  while (used < 32 && ((1u << (used - 1)) - 1u) < (uint32_t)st->max_code) ++used;
  v.sh = std::max(0, used - 12);
  v.bytes = used <= 8;
  v.n = st->size;
  v.step = st->q.step;
  v.eps = st->q.eps;
  v.R = row_norm_bound(st->hn_max, st->q.eps, st->dim);
  v.codes = codes ? codes : st->codes;
  v.ids = st->ids;
  return v;
}

}  // namespace

// Scoring plan of a store of more than 4,096 rows (smaller ones: score_dense).
// H: scores of the scan, within err of the exact scores S but for a constant of
// the query.
//   1. theta_j, the k-th best H of disjoint 32-row sets' best over the first S
//      rows (S = k * n / 256, at least 4,096), minus 2 err_j: k distinct rows
//      have S >= theta_j + err_j, so every row of the final top-k has H >=
//      theta_j;
//   2. a full scan appends every row with H >= theta_j to query j's candidate
//      buffer (about k * n / S = 256 entries expected; capacity 4,096).  Where
//      all codes fit 8 bits it multiplies bytes, against theta_j of their own
//      error bound, but for the groups of queries where that would let too
//      many rows through;
//   3. the candidates within 2 err_j of the k-th best H of them are scored
//      exactly and their k best by (S desc, id asc) are the answer
//      (k_select_rescore);
//   4. a query whose buffer overflowed (many equal scores, say) is scored
//      exactly over the whole store (k_exact); launched always, it returns at
//      once when nothing was flagged, so the call stays asynchronous.
namespace {

// Scratch of one scoring call: the context's arena (grown on demand), or a
// fixed region carved in order (the allocation-free entry point).
struct ScoreWork {
  char* base = nullptr;   // fixed region; nullptr: the context arena
  size_t bytes = 0;
  size_t used = 0;
  template <class T>
  lam_status take(lam_ctx* ctx, int slot, size_t need, T** out) {
    if (!base) {
      LAM_TRY(ctx->scratch[slot].ensure(need));
      *out = ctx->scratch[slot].as<T>();
      return LAM_OK;
    }
    const size_t at = (used + 255) & ~(size_t)255;
    LAM_CHECK(at + need <= bytes, LAM_ECAPACITY,
              "scoring needs more than the %zu bytes of the fixed workspace", bytes);
    *out = reinterpret_cast<T*>(base + at);
    used = at + need;
    return LAM_OK;
  }
};

// score_topk of a store of at most kCandCap rows.
lam_status score_dense(lam_ctx* ctx, const ScoreView& st, const float* q, int64_t nq, int32_t k, float* scores,
                       int64_t* ids, float* bound, ScoreWork& w, bool prof) {
  const int64_t ntiles = (st.n + kTB - 1) / kTB;
  const bool wide = st.b > 12;
  const int64_t cols = (wide ? 2 : 1) * (int64_t)st.D;
  DenseArgs a{};
  _Float16 *qhi = nullptr, *qlo = nullptr;
  QMeta* qmeta = nullptr;
  LAM_TRY(w.take(ctx, S_QHI, (size_t)nq * cols * 2, &qhi));
  LAM_TRY(w.take(ctx, S_QLO, (size_t)nq * cols * 2, &qlo));
  LAM_TRY(w.take(ctx, S_QMETA, (size_t)nq * sizeof(QMeta), &qmeta));
  LAM_TRY(w.take(ctx, S_CAND, (size_t)nq * ntiles * kTB * 4, &a.scores));
  a.codes = st.codes;
  a.n = st.n;
  a.D = st.D;
  a.row_words = (int64_t)st.D * st.b / 32;
  a.qhi = qhi;
  a.qlo = qlo;
  a.meta = qmeta;
  a.nq = nq;
  a.nqt = (int)((nq + kTB - 1) / kTB);
  a.ld = (int)(ntiles * kTB);
  {
    ProfScope ps(ctx, "score_prep", prof);
    hipLaunchKernelGGL(k_dense_prep, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, ctx->stream, q, nq, st.D,
                       wide ? 1 : 0, st.step, st.eps, qhi, qlo, qmeta);
    LAM_HIP(hipGetLastError());
  }
  if (ntiles > 0) {
    ProfScope ps(ctx, "score_mfma", prof);
    LAM_TRY(launch_dense<1>(st.b, dim3((unsigned)(a.nqt * ntiles)), ctx->stream, a));
  }
  ProfScope ps(ctx, "score_merge", prof);
  hipLaunchKernelGGL(k_select_dense, dim3((unsigned)nq), dim3(kRescoreThreads), 0, ctx->stream, nq, (int)st.n, a.ld, k,
                     a.scores, qmeta, st.ids, scores, ids, bound);
  LAM_HIP(hipGetLastError());
  return LAM_OK;
}

// score_topk on the workspace w.  Every buffer is taken before the first
// launch, so a workspace that is too small fails with nothing enqueued.  No
// profiling events are recorded unless prof.
lam_status score_topk_impl(lam_ctx* ctx, const ScoreView& st, const float* q, int64_t nq, int32_t k, float* scores,
                           int64_t* ids, float* bound, ScoreWork& w, bool prof) {
  if (nq == 0) return LAM_OK;
  const int D = st.D;
  const int b = st.b;
  const int64_t n = st.n;
  const int nqt = (int)((nq + kTB - 1) / kTB);
  const int64_t ntiles = (n + kTB - 1) / kTB;
  // the passes are one workgroup per (query tile, store tile), indexed in 32 bits
  LAM_CHECK((int64_t)nqt * ntiles < (1LL << 31), LAM_EINVAL, "scoring grid too large");
  if (n <= kCandCap) return score_dense(ctx, st, q, nq, k, scores, ids, bound, w, prof);
  // the sample: the store's first max(4,096, k n / 256) rows, so that at
  // most about k n / sample = 256 rows per query pass the filter (a sample of
  // k n / 1,024 rows let about 1,024 through: the corpus call 2.65-2.71 ->
  // 2.57-2.59 ms, 60 K rows at top-50 265 -> 238 us; k n / 128 was no faster)
  const int64_t sample_rows = std::max<int64_t>(4096, ((int64_t)k * n + 255) / 256);
  const int64_t stiles = std::min<int64_t>(n / kTB, (sample_rows + kTB - 1) / kTB);   // whole tiles
  const int64_t sample_tiles = std::min<int64_t>(stiles, kSampleTiles);
  const int64_t entries = sample_tiles * kSampleEntries;
  const uint32_t cap = (uint32_t)kCandCap;

  // every buffer first
  _Float16* qhi = nullptr;
  QMeta* qmeta = nullptr;
  float* part_s = nullptr;
  float* cand_s = nullptr;
  LAM_TRY(w.take(ctx, S_QHI, (size_t)nq * D * 2, &qhi));
  LAM_TRY(w.take(ctx, S_QMETA, (size_t)nq * sizeof(QMeta), &qmeta));
  const bool bytes = st.bytes && b <= 12;
  int8_t* q8 = nullptr;
  if (bytes) LAM_TRY(w.take(ctx, S_Q8, (size_t)nq * D, &q8));
  LAM_TRY(w.take(ctx, S_PART, (size_t)nq * entries * 4, &part_s));
  LAM_TRY(w.take(ctx, S_CAND, (size_t)nq * cap * 8 + (size_t)nq * 20 + 4 + (size_t)(nq / kPrecQueries + 1) * 4, &cand_s));
  int32_t* cand_r = reinterpret_cast<int32_t*>(cand_s + (size_t)nq * cap);
  uint32_t* cand_cnt = reinterpret_cast<uint32_t*>(cand_r + (size_t)nq * cap);
  float* thr = reinterpret_cast<float*>(cand_cnt + nq);   // two per query
  uint32_t* flagged = cand_cnt + 3 * nq;
  uint32_t* done = cand_cnt + 4 * nq;
  uint32_t* n_flag = cand_cnt + 5 * nq;
  uint32_t* coarse = n_flag + 1;

  {
    ProfScope ps(ctx, "score_prep", prof);
    // the scan's operand s 2^sh top, and what the left-out bits add
    const double two = std::ldexp(1.0, st.sh);
    const double rootD = std::sqrt((double)D) * (1.0 + 0x1p-50);
    const double R = st.R + (two - 1.0) * st.step * rootD;
    const double trunc = 0.5 * (two - 1.0) * st.step * rootD;
    // (a query that the former split form of codes over 12 bits, 2^11 q, could
    // not hold in float32 counts as holding Inf)
    const float qmax = b > 12 ? 3.402823466e38f / 2048.0f : 3.402823466e38f;
    hipLaunchKernelGGL(k_score_prep, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, ctx->stream, q, nq, D,
                       st.step * two, st.eps, R, trunc, qmax, qhi, q8, qmeta, cand_cnt, done, n_flag, coarse);
    LAM_HIP(hipGetLastError());
  }

  ScoreArgs a{};
  a.codes = st.codes;
  a.n = n;
  a.D = D;
  a.sh = st.sh;
  a.row_words = (int64_t)D * b / 32;
  a.qhi = qhi;
  a.q8 = q8;
  a.coarse = coarse;
  a.meta = qmeta;
  a.nq = nq;
  a.nqt = nqt;
  a.part_s = part_s;
  a.thr = thr;
  a.cand_s = cand_s;
  a.cand_r = cand_r;
  a.cand_cnt = cand_cnt;
  a.cap = cap;
  ExactArgs x{nq,    n,      cap,     k,         cand_cnt, cand_s, cand_r, qmeta, st.ids,  q,    st.step, st.codes,
              a.row_words, D, scores, ids, bound, n_flag, flagged, done, bytes ? coarse : nullptr};

  {  // 1. a k-th best score of the sample -> thresholds
    ProfScope ps(ctx, "score_sample", prof);
    a.tile_end = stiles;
    a.sample_tiles = (int)sample_tiles;
    const bool folded = sample_tiles < stiles;
    if (folded) {
      const int64_t ne = nq * entries;
      hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, ctx->stream,
                         reinterpret_cast<uint32_t*>(part_s), ne);
    }
    LAM_TRY((launch_filter<1, kSample>(b, false, (int64_t)nqt * stiles, ctx->stream, a)));
    const int nkeys = (int)std::min<int64_t>(entries, 64 * kThrKeys);
    hipLaunchKernelGGL(k_sample_thr, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, ctx->stream, nq, (int)entries,
                       folded ? 1 : 0, k, part_s, qmeta, thr, bytes ? coarse : nullptr,
                       byte_scan_keys((int64_t)nqt * ntiles, n, nkeys,
                                      32.0 * (double)stiles / (double)sample_tiles * (double)entries / nkeys));
    LAM_HIP(hipGetLastError());
  }
  {  // 2. full scan with the thresholds: 256 x 256 tiles when the launch holds
     //    many of them, else 128 x 128
    ProfScope ps(ctx, "score_mfma", prof);
    const int nqtL = (int)((nq + FilterTileL::BN - 1) / FilterTileL::BN);
    const int64_t ntilesL = (n + FilterTileL::BM - 1) / FilterTileL::BM;
    const bool large = (int64_t)nqtL * ntilesL >= kFilterLargeMinTiles;
    a.nqt = large ? nqtL : nqt;
    a.tile_end = large ? ntilesL : ntiles;
    const int64_t grid = (int64_t)a.nqt * a.tile_end;
    if (bytes) LAM_TRY((launch_filter<1, kFilterBytes>(b, large, grid, ctx->stream, a)));
    else LAM_TRY((launch_filter<9, kFilter>(b, large, grid, ctx->stream, a)));   // (codes of up to 8 bits fit bytes)
  }
  {  // 3. select and rescore
    ProfScope ps(ctx, "score_merge", prof);
    LAM_TRY(launch_exact<1>(b, true, ctx->stream, x));
  }
  {  // 4. the exact pass over flagged queries (returns at once otherwise)
    ProfScope ps(ctx, "score_fallback", prof);
    LAM_TRY(launch_exact<1>(b, false, ctx->stream, x));
  }
  return LAM_OK;
}

// ------------------------------------------------------------------ allocation-free scoring
// Its scratch memory: one array per device, allocated with the code object,
// held until the process ends.  Sized for kNoAllocMaxQ queries of up to 4,096
// dimensions: the query parts (3 D bytes per query, 4 D for a small store), the
// query meta block, the sample's entries and the candidate buffer (kCandCap
// entries of 8 bytes, 20 bytes of counts and flags) -- 80 KB per query, 20 MB
// at the limits.
constexpr size_t kNoAllocBytes = (size_t)32 << 20;
static_assert((size_t)kNoAllocMaxQ * (4 * 4096 + sizeof(QMeta) + (size_t)kSampleTiles * kSampleEntries * 4 +
                                      (size_t)kCandCap * 8 + 20) + 64 + 5 * 256 <= kNoAllocBytes,
              "the workspace holds a call at the limits");

}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kMaxDevices];   // device address of `scratch` on each device (host code must not use its name)
}  // namespace

lam_status noalloc_setup(int device) {
  LAM_CHECK(device >= 0 && device < kMaxDevices, LAM_EINVAL, "device %d beyond the supported %d", device, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (g_noalloc_ptr[device]) return LAM_OK;
  void* p = nullptr;
  LAM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));   // the current device is `device`
  g_noalloc_ptr[device] = p;
  return LAM_OK;
}

lam_status score_topk(lam_ctx* ctx, const lam_store* st, const float* q, int64_t nq, int32_t k, float* scores,
                      int64_t* ids, float* bound, const uint32_t* codes) {
  if (nq == 0) return LAM_OK;
  LAM_CHECK(st->q.bits <= kMaxBits, LAM_ESTATE,
            "scoring supports codes of at most %d bits (store codes have %d); quantize with a larger eps", kMaxBits,
            st->q.bits);
  ScoreWork w;
  const ScoreView v = store_view(st, codes);
  // the passes index (query tile, store tile) in 31 bits, and scratch is held
  // for at most 65,536 queries: more go in several passes
  const int64_t ntiles = std::max<int64_t>(1, (v.n + kTB - 1) / kTB);
  const int64_t most = std::min<int64_t>(65536, ((1LL << 31) - 1) / ntiles * kTB);
  for (int64_t j = 0; j < nq; j += most)
    LAM_TRY(score_topk_impl(ctx, v, q + j * v.D, std::min(most, nq - j), k, scores + j * k, ids + j * k,
                            bound ? bound + j : nullptr, w, true));
  return LAM_OK;
}

lam_status score_topk_noalloc(lam_ctx* ctx, const lam_store* st, const float* q, int64_t nq, int32_t k, float* scores,
                              int64_t* ids, float* bound) {
  LAM_CHECK(nq <= kNoAllocMaxQ, LAM_EINVAL, "the allocation-free call takes at most %d queries (asked %lld)",
            kNoAllocMaxQ, (long long)nq);
  void* p = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    p = ctx->device < kMaxDevices ? g_noalloc_ptr[ctx->device] : nullptr;
  }
  LAM_CHECK(p != nullptr, LAM_ESTATE, "the fixed workspace of device %d was not set up", ctx->device);
  LAM_CHECK(st->q.bits <= 12, LAM_ESTATE,
            "the allocation-free call scores codes of at most 12 bits (store codes have %d)", st->q.bits);
  ScoreWork w;
  w.base = static_cast<char*>(p);
  w.bytes = kNoAllocBytes;
  return score_topk_impl(ctx, store_view(st, nullptr), q, nq, k, scores, ids, bound, w, false);
}

// ------------------------------------------------------------------ certificate
namespace {

// Rank-invariance certificate (Appendix "Rank invariance, in full"): one wave
// per query copies the first k of its top-(k+1) and flags the query when the
// float32 margin between ranks k and k+1 exceeds
//   2 (beta + ||q||_2 delta_hat + e),   e = kappa ||q||_1 (A + eps),
// where e bounds the float32 score's error against the exact dequantized score
// (hi/lo residual 2^-22, float32 accumulation of 2 D terms gamma_2D, output
// scaling 2^-23, all relative to sum |q_d x_hat_d| <= ||q||_1 (A + eps)).  A
// flag therefore implies that the exact margin exceeds 2 (beta + ||q||_2
// delta_hat): no record can cross the rank-k boundary when every score moves
// by at most beta + ||q||_2 delta_hat.  A store with at most k rows certifies
// every valid query (nothing can cross).
__global__ __launch_bounds__(256) void k_certify(int64_t nq, int k, const float* __restrict__ s1,
                                                 const int64_t* __restrict__ i1, const float* __restrict__ b1,
                                                 const float* __restrict__ q, int D, double eps, double dhat,
                                                 double err_per_l1, float* __restrict__ scores,
                                                 int64_t* __restrict__ ids, float* __restrict__ bound,
                                                 uint8_t* __restrict__ cert, float* __restrict__ margin) {
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= nq) return;
  const float* p = q + j * D;
  double l1 = 0.0, l2 = 0.0;
  for (int d = lane; d < D; d += 64) {
    const double v = (double)p[d];
    l1 += fabs(v);
    l2 = fma(v, v, l2);
  }
  for (int o = 32; o > 0; o >>= 1) {
    l1 += __shfl_xor(l1, o);
    l2 += __shfl_xor(l2, o);
  }
  const int64_t o1 = j * (k + 1);
  for (int t = lane; t < k; t += 64) {
    scores[j * k + t] = s1[o1 + t];
    ids[j * k + t] = i1[o1 + t];
  }
  if (lane != 0) return;
  if (bound) bound[j] = b1[j];
  const float sk = s1[o1 + k - 1], sk1 = s1[o1 + k];
  const bool valid = !isnan(b1[j]);   // NaN bound: the query row holds NaN/Inf
  const double m = (i1[o1 + k] < 0) ? INFINITY : (double)sk - (double)sk1;
  // rounded up past its own evaluation error: the binary64 sums of D terms are
  // within (D - 1) 2^-53 relative in any order, the few products and the
  // square root add 2^-53 each
  const double thr = 2.0 * (eps * l1 + sqrt(l2) * dhat + err_per_l1 * l1) * (1.0 + (double)(D + 8) * 0x1p-52);
  cert[j] = (valid && m > thr) ? 1 : 0;
  if (margin) margin[j] = valid ? (float)m : __builtin_nanf("");
}

}  // namespace

lam_status score_certify(lam_ctx* ctx, const lam_store* st, const float* q, int64_t nq, int32_t k, float* scores,
                         int64_t* ids, float* bound, uint8_t* certified, float* margin) {
  if (nq == 0) return LAM_OK;
  const int K1 = k + 1;
  const size_t per = (size_t)K1 * (4 + 8);
  LAM_TRY(ctx->scratch[kScratchCertify].ensure((size_t)nq * per + (size_t)nq * 4 + 64));
  char* base = ctx->scratch[kScratchCertify].as<char>();
  int64_t* i1 = reinterpret_cast<int64_t*>(base);
  float* s1 = reinterpret_cast<float*>(base + (size_t)nq * K1 * 8);
  float* b1 = s1 + (size_t)nq * K1;
  LAM_TRY(score_topk(ctx, st, q, nq, K1, s1, i1, b1));
  // error bound of the float32 score per unit of ||q||_1: kappa (A + eps).
  // It is stated for float32 sums of hi and lo query parts, and for codes of
  // more than 12 bits for the sums of their two halves (twice the terms, and
  // sum |q'_d' x_hat'_d'| <= ||q||_1 (A + eps + 2^12 s)), which is what a store of
  // at most 4,096 rows returns; the binary64 sums of a larger one, rounded once,
  // are far inside it.
  const bool wide = st->q.bits > 12;
  const double Dt = (wide ? 2.0 : 1.0) * st->dim;
  const double u = std::ldexp(1.0, -24);
  const double g2d = 2.0 * Dt * u / (1.0 - 2.0 * Dt * u);
  const double kappa = 1.01 * (std::ldexp(1.0, -22) + g2d + std::ldexp(1.0, -23));
  const double mag = (double)st->q.absmax + st->q.eps + (wide ? 4096.0 * st->q.step : 0.0);
  const double err_per_l1 = kappa * mag;
  hipLaunchKernelGGL(k_certify, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, ctx->stream, nq, k, s1, i1, b1, q,
                     st->dim, st->q.eps, st->delta_hat_run, err_per_l1, scores, ids, bound, certified, margin);
  LAM_HIP(hipGetLastError());
  return LAM_OK;
}

}  // namespace lam
