// Convolution as an implicit GEMM whose reduction is split over the waves of
// a workgroup, for launches that are too small to be bound by anything but
// latency (an implicit-GEMM routine; NHWC with C % 8 == 0 or NC8HW8, all
// element types; NCHW in fp32).
//
// The tiled implicit GEMMs move each reduction step of a tile through LDS:
// fill, wait, barrier, read, compute.  At a small batch their few workgroups
// walk a long chain of such steps (72 for a 256-channel 3x3 layer) at 0.3 us
// each, whatever the arithmetic.  Here every wave owns the whole output tile
// of 16 FM pixels x 16 FN channels and a contiguous part of the reduction: it
// loads its operands straight from global memory into MFMA registers (no
// LDS, no barrier, D steps in flight per wave), and the NW waves' partial
// sums meet once in LDS at the end, where bias, residual and activation are
// applied.  The chain is NW times shorter and never waits for another wave.
// A step moves FM + FN KB for FM FN MFMAs per wave, so the L2-to-register
// path (about 125 B/ns per CU) bounds larger launches: those stay with the
// LDS tiles, which share a tile's operands among the waves.  Measured as block
// means against the fastest other routine, bf16: 512 channels 3x3 at 7 x 7, batch
// 1, 11.2 -> 5.8 us; 128 at 28 x 28, 9.0 -> 5.3; 256 at 14 x 14, batch 8, stride
// 2, 11.6 -> 9.1; ResNet-18 at batch 1, 177 -> 120 us per inference.
//
// The reduction index runs over 16-byte chunks (8 channels of a 16-bit type,
// 4 of fp32) of the taps, in the order of the prepared filter [Kp][R][S][C8],
// four chunks per step: lane l holds chunk l / 16 of row l % 16, for both
// operands.  The filter is laid out once in that order (ksplit_pack): a
// step's 16 rows are 1 KB in lane order, zero past the filter's rows and
// chunks, so a wave's load is one contiguous run (8 cache lines, where the
// rows of [Kp][R][S][C8] touch 16).  An fp32 step is four 4-wide MFMAs; element e of the four lane
// groups' chunks forms the reduction of the e-th.  The chunk's tap and
// channel block come from an exact fp32 division, so channel counts need not
// be multiples of the step.  In NCHW a chunk's four channels are four 4-byte loads
// from their planes (channels past C read as zero), which coalesce over the
// lanes' pixels, and the outputs go out element by element along the pixels;
// small nets in fp32 stay in NCHW, where two converters would cost more than a
// layer.  A projected shortcut (PJ) appends the steps of its own
// tensor and filter.
#include "gemm_common.hpp"
#include "kcommon.hpp"
#include "launch.hpp"

#include <algorithm>

namespace sn {
namespace k {

struct KsArgs {
  const void* x;
  const void* w;
  const float* bias;
  const void* res;  // residual in the output's layout, or null
  void* y;
  int M, Ng, PQ, Q, Ks;
  int H, W, Cs, stride, pad, S;
  int CBc, KCH, steps;      // chunks per tap, chunks of the reduction, steps of four chunks
  int HW8;                  // NC8HW8: elements between channel blocks
  int Kp;                   // bias entries
  int act, tiles_m, tiles_n;
  int round_sum;            // round the sum to the type before adding the residual
  float inv_pq, inv_q, inv_cb, inv_s;
  long long x_elems, w_bytes, y_bytes;
  // projected shortcut
  const void* x2;
  const void* w2;
  int H2, W2, Cs2, stride2, KCH2, steps2, HW8_2;
  long long x2_elems, w2_bytes;
};

// One step's MFMAs of a 16 x 16 block: 32 reduction elements of a 16-bit
// type, 16 of fp32.
template <typename T>
__device__ __forceinline__ f32x4 ks_mma(u32x4 w, u32x4 x, f32x4 c) {
  if constexpr (sizeof(T) == 2) {
    typedef typename Mfma<T>::frag frag;
    return Mfma<T>::run(__builtin_bit_cast(frag, w), __builtin_bit_cast(frag, x), c);
  } else {
    const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) c = Mfma<float>::run(wf[e], xf[e], c);
    return c;
  }
}

// K1: a 1x1 convolution without padding (no taps to decode)
template <typename T, int L, int FM, int FN, int NW, int D, bool K1, bool PJ>
__global__ __launch_bounds__(64 * NW) void conv_ksplit_kernel(KsArgs a) {
  static_assert(L != NCHW || (sizeof(T) == 4 && !PJ), "NCHW: fp32 without a projected shortcut");
  constexpr int ES = sizeof(T), CE = 16 / ES;  // bytes and elements per chunk
  constexpr int BM = 16 * FM, BN = 16 * FN;
  constexpr int RP = BN + 4;                   // staging row pitch (floats)
  __shared__ __attribute__((aligned(16))) float red[NW * BM * RP];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int mt, nt;
  tile_of(blockIdx.x, a.tiles_m, a.tiles_n, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, a.x_elems * ES);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.w, a.w_bytes);
  const __amdgpu_buffer_rsrc_t rx2 = make_rsrc(PJ ? a.x2 : a.x, PJ ? a.x2_elems * ES : 0);
  const __amdgpu_buffer_rsrc_t rw2 = make_rsrc(PJ ? a.w2 : a.w, PJ ? a.w2_bytes : 0);

  const int row = lane & 15, grp = lane >> 4;
  // per pixel block: element offset of the window's first pixel and its
  // coordinates (rows past M: no window position is inside the image)
  int xbase[FM], h0[FM], w0[FM], x2base[FM];
  bool mok[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + i * 16 + row;
    mok[i] = m < a.M;
    const int img = sdiv(m, a.inv_pq), pq = m - img * a.PQ;
    const int p = sdiv(pq, a.inv_q), q = pq - p * a.Q;
    h0[i] = mok[i] ? p * a.stride - a.pad : -(1 << 20);
    w0[i] = q * a.stride - a.pad;
    if constexpr (L == NC8) xbase[i] = (img * (a.Cs >> 3) * a.H + p * a.stride - a.pad) * (a.W * 8) + w0[i] * 8;
    else if constexpr (L == NCHW) xbase[i] = (img * a.Cs * a.H + p * a.stride - a.pad) * a.W + w0[i];
    else xbase[i] = ((img * a.H + p * a.stride - a.pad) * a.W + w0[i]) * a.Cs;
    if constexpr (PJ) {
      const int h2 = p * a.stride2, w2 = q * a.stride2;
      if constexpr (L == NC8) x2base[i] = (img * (a.Cs2 >> 3) * a.H2 + h2) * (a.W2 * 8) + w2 * 8;
      else x2base[i] = ((img * a.H2 + h2) * a.W2 + w2) * a.Cs2;
    }
  }
  // the lane's byte of step 0 in each filter block of 16 rows
  unsigned wofs[FN], w2ofs[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    wofs[j] = (unsigned)(n0 / 16 + j) * (unsigned)a.steps * 1024u + lane * 16u;
    if constexpr (PJ) w2ofs[j] = (unsigned)(n0 / 16 + j) * (unsigned)a.steps2 * 1024u + lane * 16u;
  }

  const int plane = a.H * a.W;  // NCHW: elements between channels
  // offset of chunk cc of a pixel's channels
  auto chunk_off = [&](int cc, int hw8) {
    if constexpr (L == NCHW) return cc * CE * plane;
    else if constexpr (L == NC8) return CE == 8 ? cc * hw8 : (cc >> 1) * hw8 + (cc & 1) * 4;
    else return cc * CE;
  };
  auto load = [&](int t, int t1, u32x4 (&fa)[FM], u32x4 (&fb)[FN]) {
    if (!PJ || t < a.steps) {
      const int qk = t * 4 + grp;
      const bool in = t < t1 && qk < a.KCH;
      int r = 0, s = 0, cc = qk;
      if constexpr (!K1) {
        const int tap = sdiv(qk, a.inv_cb);
        cc = qk - tap * a.CBc;
        r = sdiv(tap, a.inv_s);
        s = tap - r * a.S;
      }
      const int d = (K1 ? 0 : (r * a.W + s) * (L == NC8 ? 8 : L == NCHW ? 1 : a.Cs)) + chunk_off(cc, a.HW8);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, t < t1 ? (int)(wofs[j] + t * 1024u) : (int)kOOB, 0, 0);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const bool ok = K1 ? in && mok[i]
                           : in && (unsigned)(h0[i] + r) < (unsigned)a.H && (unsigned)(w0[i] + s) < (unsigned)a.W;
        if constexpr (L == NCHW) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            fa[i][e] = __builtin_amdgcn_raw_buffer_load_b32(
                rx, ok && cc * 4 + e < a.Cs ? (int)((unsigned)(xbase[i] + d + e * plane) * ES) : (int)kOOB, 0, 0);
        } else {
          fa[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? (int)((unsigned)(xbase[i] + d) * ES) : (int)kOOB, 0, 0);
        }
      }
    } else {
      const int qk = (t - a.steps) * 4 + grp;
      const bool in = t < t1 && qk < a.KCH2;
      const int d = chunk_off(qk, a.HW8_2);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j] = __builtin_amdgcn_raw_buffer_load_b128(
            rw2, t < t1 ? (int)(w2ofs[j] + (t - a.steps) * 1024u) : (int)kOOB, 0, 0);
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i] = __builtin_amdgcn_raw_buffer_load_b128(
            rx2, in && mok[i] ? (int)((unsigned)(x2base[i] + d) * ES) : (int)kOOB, 0, 0);
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the wave's contiguous part of the steps; steps past it load zeros
  const int total = a.steps + (PJ ? a.steps2 : 0);
  const int per = (total + NW - 1) / NW;
  const int t0 = min(wave * per, total), t1 = min(t0 + per, total);
  u32x4 fa[D][FM], fb[D][FN];
#pragma unroll
  for (int d = 0; d < D; ++d) load(t0 + d, t1, fa[d], fb[d]);

  // the thread's outputs (NCHW: see the end): quads of four channels, e = tid + 64 NW u;
  // consecutive threads on consecutive addresses (NHWC: a pixel's channels;
  // NC8HW8: the pixels of a channel block).  The residual is loaded here, under
  // the reduction: after it, a load's latency would be most of the epilogue.
  constexpr int NQ = L == NCHW ? 0 : (BM * BN / 4 + 64 * NW - 1) / (64 * NW);
  constexpr bool ALL = BM * BN / 4 % (64 * NW) == 0;  // every thread has NQ quads
  const bool vec = L == NC8 || a.Ks % 4 == 0;
  const T* __restrict__ res = reinterpret_cast<const T*>(a.res);
  constexpr int NQA = NQ ? NQ : 1;
  int qm[NQA], qn[NQA];
  unsigned qo[NQA];  // element offset, or kOOB
  f32x4 rq[NQA];     // the residual's 8 or 16 bytes
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const int e = tid + 64 * NW * u;
    if constexpr (L == NC8) {
      qm[u] = (e >> 1) % BM;
      qn[u] = (e >> 1) / BM * 8 + (e & 1) * 4;
    } else {
      qm[u] = e / (BN / 4);
      qn[u] = e % (BN / 4) * 4;
    }
    const int m = m0 + qm[u], n = n0 + qn[u];
    unsigned o;
    if constexpr (L == NC8) {
      const int img = sdiv(m, a.inv_pq), pq = m - img * a.PQ;
      o = (unsigned)(((img * (a.Ks >> 3) + (n >> 3)) * a.PQ + pq) * 8 + (n & 7));
    } else {
      o = (unsigned)(m * a.Ks + n);
    }
    qo[u] = (ALL || e < BM * BN / 4) && m < a.M && n < a.Ng ? o : kOOB;
    rq[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  if (NQ && res && vec) {
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(res, a.y_bytes);
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int off = qo[u] == kOOB ? (int)kOOB : (int)(qo[u] * ES);
      if constexpr (ES == 4) {
        rq[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, off, 0, 0));
      } else {
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rr, off, 0, 0));
        __builtin_memcpy(&rq[u], &v, 8);
      }
    }
  }
  for (int t = t0; t < t1; t += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = ks_mma<T>(fb[d][j], fa[d][i], acc[i][j]);
      load(t + D + d, t1, fa[d], fb[d]);
    }
  }

  // partial sums: pixel i * 16 + (lane & 15), channels j * 16 + (lane >> 4) * 4 + v
  float* const mine = red + wave * BM * RP;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      *reinterpret_cast<f32x4*>(mine + (i * 16 + row) * RP + j * 16 + grp * 4) = acc[i][j];
  __syncthreads();

  T* __restrict__ y = reinterpret_cast<T*>(a.y);
  if constexpr (L == NCHW) {  // consecutive threads on consecutive pixels of a channel
    for (int e = tid; e < BM * BN; e += 64 * NW) {
      const int mm = e % BM, m = m0 + mm, nn = e / BM, n = n0 + nn;
      if (m >= a.M || n >= a.Ng) continue;
      float s = red[mm * RP + nn];
#pragma unroll
      for (int v = 1; v < NW; ++v) s += red[(v * BM + mm) * RP + nn];
      const int img = sdiv(m, a.inv_pq), pq = m - img * a.PQ;
      const unsigned o = (unsigned)((img * a.Ks + n) * a.PQ + pq);
      s += a.bias[n];
      if (res) s += to_f(res[o]);
      y[o] = from_f<T>(act_f(s, a.act));
    }
  }
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    if (qo[u] == kOOB) continue;
    const int n = n0 + qn[u];
    f32x4 s = *reinterpret_cast<const f32x4*>(red + qm[u] * RP + qn[u]);
#pragma unroll
    for (int v = 1; v < NW; ++v) s += *reinterpret_cast<const f32x4*>(red + (v * BM + qm[u]) * RP + qn[u]);
    T* const yp = y + qo[u];
    T out[4], rt[4];
    __builtin_memcpy(rt, &rq[u], 4 * ES);
    if (vec) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        // the padded channels of NC8HW8 have a bias of zero (Kp entries)
        float f = s[v] + a.bias[n + v];
        if (a.round_sum) f = to_f(from_f<T>(f));
        if (res) f += to_f(rt[v]);
        out[v] = from_f<T>(act_f(f, a.act));
      }
      __builtin_memcpy(__builtin_assume_aligned(yp, 4 * ES), out, 4 * ES);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (n + v >= a.Ng) break;
        float f = s[v] + a.bias[n + v];
        if (a.round_sum) f = to_f(from_f<T>(f));
        if (res) f += to_f(res[qo[u] + v]);
        yp[v] = from_f<T>(act_f(f, a.act));
      }
    }
  }
}

// ------------------------------------------------------------------ host
size_t ksplit_packed_bytes(int kp, size_t row_bytes) {
  return (size_t)((kp + 15) / 16) * ((row_bytes / 16 + 3) / 4) * 1024;
}

void ksplit_pack(const void* w, int kp, size_t row_bytes, void* out) {
  const int nch = (int)(row_bytes / 16), steps = (nch + 3) / 4;
  const char* src = static_cast<const char*>(w);
  char* dst = static_cast<char*>(out);
  for (int kb = 0; kb < (kp + 15) / 16; ++kb)
    for (int t = 0; t < steps; ++t)
      for (int l = 0; l < 64; ++l, dst += 16) {
        const int k = kb * 16 + (l & 15), q = t * 4 + (l >> 4);
        if (k < kp && q < nch) __builtin_memcpy(dst, src + (size_t)k * row_bytes + (size_t)q * 16, 16);
        else __builtin_memset(dst, 0, 16);
      }
}

// The time of a launch, in us: a base plus, per round of 256 workgroups, a cost
// per reduction step and one per tile.  A wave-split tile's step is eight
// 16-element steps, one per wave, and its rounds are whole; the LDS tile's is 32
// elements, its later rounds overlap (tiles / 256, at least one), and its steps
// also wait for one another.  In NCHW both load element by element; a pointwise
// layer's steps read new lines every time, where taps read those of their
// neighbours again, and take a wave-split tile up to twice as long.  red counts the
// channels rounded up to 8.  Fitted to
// 2147 convolutions, each run on the four kernels: 1x1 to 7x7 at stride 1 and 2, 3 to 512
// channels to 4 to 512, 4 to 240000 pixels, in the three layouts (rms error 7 to
// 12 %).  The LDS tile is taken unless a wave-split tile is expected below 0.9 of
// it.  Against the LDS tile alone the picks are 1.69 (NCHW) and 1.58 times faster in the
// geometric mean, 0.8 and 1.3 % from the fastest of the four, and of the 2147 one
// is slower than the LDS tile by more than 3 % (1x1, 80 -> 10 channels, 47526 pixels, 6 %).
// LDS tile -> pick: 512 channels 3x3 at 7 x 7, 103 -> 12.3 us; in NCHW 16 channels
// 3x3/2 at 32 x 32, 10.3 -> 5.1; 64 at 2 x 28 x 28, 28.0 -> 9.2.
static int ksplit_pick_f32(int layout, bool k1, long long m, int k, long long red, bool lds_ok) {
  struct Fit {
    int fm, fn;
    double base[2], step[2], tile[2];  // taps, pointwise
  };
  static const Fit vec[] = {{1, 1, {3.17, 3.08}, {0.22, 0.38}, {1.35, 0.82}},
                            {2, 1, {2.87, 2.97}, {0.39, 0.41}, {1.23, 0.99}},
                            {2, 2, {2.82, 2.71}, {0.61, 0.73}, {2.06, 1.78}}};
  static const Fit nchw[] = {{1, 1, {3.18, 2.83}, {0.30, 0.63}, {1.57, 1.28}},
                             {2, 1, {3.96, 3.03}, {0.63, 0.89}, {1.31, 1.68}},
                             {2, 2, {3.85, 3.27}, {0.87, 1.28}, {2.33, 2.11}}};
  double best = 1e30;
  int pick = 0;
  if (lds_ok) {
    const double r = std::max(1.0, (double)(((m + 63) / 64) * ((k + 63) / 64)) / 256.0), s = (double)((red + 31) / 32);
    best = layout == NCHW ? 0.9 * (3.28 + r * (0.84 * s + 0.83) + 0.45 * s)
                          : 0.9 * (3.11 + r * (0.63 * s + 0.90) + 0.17 * s);
  }
  const double s = (double)((red + 15) / 16) / 8.0;
  for (const Fit& f : layout == NCHW ? nchw : vec) {
    const long long wg = ((m + 16 * f.fm - 1) / (16 * f.fm)) * ((k + 16 * f.fn - 1) / (16 * f.fn));
    const double t = f.base[k1] + (double)((wg + 255) / 256) * (f.step[k1] * s + f.tile[k1]);
    if (t < best) {
      best = t;
      pick = f.fm * 8 + f.fn;
    }
  }
  return pick;
}

bool ksplit_applicable(int dtype, int layout, int n, int c, int h, int w, int r, int s, int stride, int pad, int k,
                       int c2) {
  const long long p = (h + 2 * pad - r) / stride + 1, q = (w + 2 * pad - s) / stride + 1, es = dtype == 0 ? 4 : 2;
  const long long c8 = (c + 7) / 8 * 8, kp = (k + 7) / 8 * 8, k2 = (c2 + 7) / 8 * 8;
  if (!(layout == NC8 || (layout == NHWC && c % 8 == 0 && c2 % 8 == 0) || (layout == NCHW && dtype == 0 && c2 == 0)))
    return false;
  // exact fp32 index divisions (pixels, reduction chunks) and 32-bit byte
  // offsets into every tensor
  const long long nch = (long long)r * s * (c8 * es / 16);
  return n * p * q + p * q < (1 << 20) && nch + c8 < (1 << 20) && r * s < (1 << 20) &&
         n * c8 * h * w * es < (long long)kOOB &&
         ksplit_packed_bytes((int)kp, (size_t)(r * s * c8 * es)) < kOOB && n * kp * p * q * es < (long long)kOOB &&
         ksplit_packed_bytes((int)kp, (size_t)(k2 * es)) < kOOB;
}

int ksplit_tile_f32(int layout, int n, int c, int h, int w, int r, int s, int stride, int pad, int k, int c2) {
  if (!ksplit_applicable(0, layout, n, c, h, w, r, s, stride, pad, k, c2)) return 0;
  const long long p = (h + 2 * pad - r) / stride + 1, q = (w + 2 * pad - s) / stride + 1;
  return ksplit_pick_f32(layout, r == 1 && s == 1 && pad == 0, n * p * q, k, (long long)r * s * ((c + 7) / 8 * 8) + c2,
                         !c2);
}

template <typename T, int L, int FM, int FN, int NW, int D>
static void ks_go(KsArgs a, bool k1, hipStream_t st) {
  a.tiles_m = (a.M + 16 * FM - 1) / (16 * FM);
  a.tiles_n = (a.Ng + 16 * FN - 1) / (16 * FN);
  const dim3 grid(a.tiles_m * a.tiles_n), block(64 * NW);
  if constexpr (L == NCHW) {
    check(!a.x2, "wave-split kernel: no projected shortcut in NCHW");
    if (k1) SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, true, false>), grid, block, 0, st, a);
    else SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, false, false>), grid, block, 0, st, a);
  } else if (a.x2) {
    if (k1) SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, true, true>), grid, block, 0, st, a);
    else SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, false, true>), grid, block, 0, st, a);
  } else {
    if (k1) SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, true, false>), grid, block, 0, st, a);
    else SN_LAUNCH((conv_ksplit_kernel<T, L, FM, FN, NW, D, false, false>), grid, block, 0, st, a);
  }
}

template <typename T, int L>
static void ks_tile(int fm, int fn, int nw, const KsArgs& a, bool k1, hipStream_t st) {
#define KG(FM_, FN_, NW_, D_)                       \
  if (fm == FM_ && fn == FN_ && nw == NW_) {        \
    ks_go<T, L, FM_, FN_, NW_, D_>(a, k1, st);      \
    return;                                         \
  }
  KSPLIT_CONFIGS(KG)
#undef KG
  check(false, "wave-split tile not instantiated");
}

void conv_ksplit(int dtype, int fm, int fn, int nw, const ConvArgs& c, hipStream_t st) {
  check(c.xd.layout == c.yd.layout && c.yd.n == c.xd.n && c.yd.h == (c.xd.h + 2 * c.pad - c.r) / c.stride + 1 &&
            c.yd.w == (c.xd.w + 2 * c.pad - c.s) / c.stride + 1 &&
            ksplit_applicable(dtype, c.xd.layout, c.xd.n, c.xd.c, c.xd.h, c.xd.w, c.r, c.s, c.stride, c.pad, c.yd.c,
                              c.x2 ? c.x2d.c : 0),
        "wave-split kernel: one layout, C % 8 == 0 in NHWC, fp32 in NCHW, tensors below 2 GiB");
  const int es = dtype == 0 ? 4 : 2, ce = 16 / es;
  KsArgs a{};
  a.x = c.x;
  check(c.wks, "wave-split kernel: the filter in its order");
  a.w = c.wks;
  a.bias = c.bias;
  a.res = c.res;
  a.y = c.y;
  a.PQ = c.yd.h * c.yd.w;
  a.M = c.yd.n * a.PQ;
  a.Q = c.yd.w;
  a.Ks = c.yd.cs;
  a.Ng = c.yd.layout == NC8 ? c.yd.cs : c.yd.c;
  a.H = c.xd.h;
  a.W = c.xd.w;
  a.Cs = c.xd.cs;
  a.stride = c.stride;
  a.pad = c.pad;
  a.S = c.s;
  const int c8 = (c.xd.c + 7) / 8 * 8;
  a.CBc = c8 / ce;
  a.KCH = c.r * c.s * a.CBc;
  a.steps = (a.KCH + 3) / 4;
  a.HW8 = a.H * a.W * 8;
  a.Kp = (c.yd.c + 7) / 8 * 8;
  a.act = c.act;
  a.round_sum = c.round_sum;
  a.inv_pq = 1.f / (float)a.PQ;
  a.inv_q = 1.f / (float)a.Q;
  a.inv_cb = 1.f / (float)a.CBc;
  a.inv_s = 1.f / (float)a.S;
  a.x_elems = (long long)c.xd.n * c.xd.cs * c.xd.h * c.xd.w;
  a.y_bytes = (long long)c.yd.n * c.yd.cs * c.yd.h * c.yd.w * es;
  a.w_bytes = (long long)ksplit_packed_bytes(a.Kp, (size_t)c.r * c.s * c8 * es);
  if (c.x2) {
    check(c.w2ks && c.x2d.layout == c.xd.layout && c.x2d.n == c.xd.n && (c.x2d.h - 1) / c.stride2 + 1 == c.yd.h &&
              (c.x2d.w - 1) / c.stride2 + 1 == c.yd.w &&
              (long long)c.x2d.n * c.x2d.cs * c.x2d.h * c.x2d.w * es < (long long)kOOB,
          "wave-split kernel: the projected shortcut's shape or layout");
    const int k2 = (c.x2d.c + 7) / 8 * 8;
    a.x2 = c.x2;
    a.w2 = c.w2ks;
    a.H2 = c.x2d.h;
    a.W2 = c.x2d.w;
    a.Cs2 = c.x2d.cs;
    a.stride2 = c.stride2;
    a.KCH2 = k2 / ce;
    a.steps2 = (a.KCH2 + 3) / 4;
    a.HW8_2 = a.H2 * a.W2 * 8;
    a.x2_elems = (long long)c.x2d.n * c.x2d.cs * c.x2d.h * c.x2d.w;
    a.w2_bytes = (long long)ksplit_packed_bytes(a.Kp, (size_t)k2 * es);
  }
  const bool k1 = c.r == 1 && c.s == 1 && c.pad == 0;
  const bool nc8 = c.xd.layout == NC8;
  if (dtype == 0) {
    if (nc8) ks_tile<float, NC8>(fm, fn, nw, a, k1, st);
    else if (c.xd.layout == NCHW) ks_tile<float, NCHW>(fm, fn, nw, a, k1, st);
    else ks_tile<float, NHWC>(fm, fn, nw, a, k1, st);
  } else if (dtype == 1) {
    if (nc8) ks_tile<f16, NC8>(fm, fn, nw, a, k1, st);
    else ks_tile<f16, NHWC>(fm, fn, nw, a, k1, st);
  } else {
    if (nc8) ks_tile<bf16, NC8>(fm, fn, nw, a, k1, st);
    else ks_tile<bf16, NHWC>(fm, fn, nw, a, k1, st);
  }
}

}  // namespace k
}  // namespace sn
