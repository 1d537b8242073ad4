// Legendre step on the matrix cores (FP32 contraction, FP64 recurrence) for
// groups of 16 channels: per m the parity-folded sums of Eq. (14)/(26) and
// Eq. (24) are dense products
//   analysis:  a[l, col]   = sum_p lambda_lm(z_p) X_{E/O}[p, col]   (K = ring pairs)
//   synthesis: S[p, col]   = sum_l lambda_lm(z_p) a[l, col]         (K = l)
// with col = (channel, re/im), 32 columns.  Both take their FP32 products as BF16
// partial products (below) with v_mfma_f32_32x32x16_bf16: lane j holds
// A[j % 32][8 (j / 32) + e] and B[8 (j / 32) + e][j % 32], e = 0..7, and the
// 32 x 32 accumulator holds D[i][j] in lane j + 32 ((i / 4) % 2), register
// 4 (i / 8) + i % 4.
//
// lambda is produced by the FP64 recurrence of Eq. (16) on mu = lambda / c
// (tables.hip) with lanes running rings; in the synthesis that is already the
// A layout (rows = rings, K = l), in the analysis the values go through a
// wave-private LDS tile to become rows = l, K = rings.
#include <type_traits>

#include "common.h"

namespace shtx {

typedef float f32x16 __attribute__((ext_vector_type(16)));
// FP32 products on the BF16 matrix cores.  An FP32 value is the sum of three
// BF16 values, x = h + m + l with each part the rounding of what the ones
// before it leave (8 bits each, 24 in all: exact where l does not fall below
// the BF16 range, see below), and a product of two such values is taken as the six
// partial products hh + hm + mh + hl + lh + mm.  The three left out are at most
// 2^-24 of it, one FP32 rounding (2^-27.5 in the root mean square of random
// factors); leaving out any other adds 2.5e-6 and more to the sums' relative l2
// error.  All partial products are exact in FP32 and are added in FP32 by the
// matrix core, 16 terms of K to a rounding (the FP32 instruction: 2): random
// operands, K 2048, relative l2 of the sums against FP64, 6.8e-7 with the parts,
// 8.4e-7 with the FP32 instruction.  Six v_mfma_f32_32x32x16_bf16 take 192 cycles
// for what eight v_mfma_f32_32x32x2_f32 take 512, and the vector ALU issues beside
// them (beside FP32 matrix instructions it does not: both use its multipliers).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x16 mfma_bf(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                  0, 0);
}
// The three BF16 parts of two values in words i of p[0..2], x0 in bits 0-15 (the
// words are opaque to the compiler, which would round the low halves a second
// time by themselves).  What a part leaves, x - part, is exact; DOT forms it as
// a two-term dot product with (-1, 0) or (0, -1) instead of a shift or mask and
// a subtraction: fewer instructions, each longer.  Analysis 2.22 -> 2.18 ms
// with it, synthesis 1.69 -> 1.78 (Nside 1024 L 2047 B 16).
__device__ __forceinline__ float dot_bf(uint32_t a, uint32_t b, float c) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
template <bool DOT, typename V> __device__ __forceinline__ void split3(float x0, float x1, V (&p)[3], int i) {
  uint32_t h = pack_bf16x2(x0, x1), m;
  asm("" : "+v"(h));
  float r0, r1;
  if constexpr (DOT) {
    uint32_t n0 = 0x0000bf80u, n1 = 0xbf800000u;
    asm("" : "+s"(n0), "+s"(n1));  // in registers: a literal operand would be repeated in both halves
    r0 = dot_bf(h, n0, x0);
    r1 = dot_bf(h, n1, x1);
    m = pack_bf16x2(r0, r1);
    asm("" : "+v"(m));
    r0 = dot_bf(m, n0, r0);
    r1 = dot_bf(m, n1, r1);
  } else {
    r0 = x0 - __uint_as_float(h << 16);
    r1 = x1 - __uint_as_float(h & 0xffff0000u);
    m = pack_bf16x2(r0, r1);
    asm("" : "+v"(m));
    r0 -= __uint_as_float(m << 16);
    r1 -= __uint_as_float(m & 0xffff0000u);
  }
  p[0][i] = h;
  p[1][i] = m;
  p[2][i] = pack_bf16x2(r0, r1);
}
// c += a b for operands in three parts, small products first
__device__ __forceinline__ void mfma_split(const u32x4 (&a)[3], const u32x4 (&b)[3], f32x16 &c) {
  constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
  for (int k = 0; k < 6; ++k) c = mfma_bf(a[ia[k]], b[ib[k]], c);
}
// the same for two left operands, alternating (no product waits for the one
// before it)
__device__ __forceinline__ void mfma_split2(const u32x4 (&a0)[3], const u32x4 (&a1)[3], const u32x4 (&b)[3],
                                            f32x16 &c0, f32x16 &c1) {
  constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    c0 = mfma_bf(a0[ia[k]], b[ib[k]], c0);
    c1 = mfma_bf(a1[ia[k]], b[ib[k]], c1);
  }
}

// Range.  A part below 2^-133, the smallest BF16 value, is lost, so an operand of
// less than 2^-109 would not keep its 24 bits, and one that rounds to 2^128 would
// have an infinite part.  So the callers hand over halves of the channels' operands
// (spectra, coefficients), and the kernels multiply a column of them, and with it its
// sums, by kTinyScale until the first value of kTinyBelow or more arrives.  From then
// on values below 2^-109 lose what is under 2^-134, 2^-70 of that value, where lambda
// is taken as zero below 2^-64.  The scaled operands are below 1 and, where not zero,
// at least 2^-86.  In ordinary data the first operands of a wave take all its columns
// past kTinyBelow (the adjoint's coefficients, which carry the weight 4 pi / Npix, past
// 2^-64 but not 2^-40); a wave with a column that stays below it (tiny values, a zero
// channel) takes 3% longer (Nside 1024 L 2047 B 16, calls: analysis 2.91 -> 3.00 ms,
// synthesis 2.68 -> 2.77).
constexpr float kTinyBelow = 0x1p-64f;
constexpr float kTinyScale = 0x1p64f, kTinyUndo = 0x1p-64f;
// The scale of a lane's column (kTinyScale or 1) after the operands x(0) .. x(n - 1) of
// this lane, and what its sums so far have to be multiplied by.  Four of the operands
// show it in ordinary data.
template <int n, typename F> __device__ __forceinline__ float tiny_step(F x, float &scale) {
  float big = fmaxf(fmaxf(fabsf(x(0)), fabsf(x(n / 4))), fmaxf(fabsf(x(n / 2)), fabsf(x(3 * n / 4))));
  if (!__all(scale == 1.f || big >= kTinyBelow)) {
#pragma unroll
    for (int i = 0; i < n; ++i) big = fmaxf(big, fabsf(x(i)));
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(big), __float_as_uint(big), false, false);
    big = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));  // of both lanes of the column
  }
  const float undo = scale != 1.f && big >= kTinyBelow ? kTinyUndo : 1.f;
  scale *= undo;
  return undo;
}

// Word 3 of a raw buffer resource on gfx9-family GPUs (untyped 32-bit
// loads, no swizzle).
constexpr int kBufferWord3 = 0x00020000;
constexpr int kSubL = 64;       // l's per LDS sub-tile (two per block)
constexpr int kTileRS = 64 + 4; // row stride of the LDS tile in floats
constexpr int kRedRS = 32 + 1;  // row stride of the cross-wave reduction (reuses the tile)
static_assert(kBlockL * kRedRS <= kSubL * kTileRS, "reduction fits the tile");

// Analysis.  Workgroup = one (m, l0) item of the XCD-grouped block list;
// NW waves take 64-ring slices of every 64 NW-ring chunk; each lane restarts its
// ring's recurrence from the block checkpoint, writes 64 lambdas per sub-tile
// into its wave's LDS tile [l][ring], and the wave multiplies the tile (rows =
// even or odd l) with the ring spectra E or O, split once per slice and held in
// registers.  The NW waves' partial sums are added through LDS at the end.
// NW = 1 or 2 (launch choice): smaller workgroups than four waves measured
// faster at every size (more of them, a shorter cross-wave reduction and
// barriers over fewer waves).
//
// Bound by the vector ALU at two waves per SIMD (256 VGPRs: 64 of sums, 96 of
// split spectra), and by power: the card runs it at about 2.0 GHz, FP32 matrix
// instructions in its place at 2.3.  Timing copies (Nside 1024 L 2047 B 16, 2.2
// ms): without the recurrence 1.6 ms, without the matrix instructions 1.75,
// without splitting lambda 1.9, without splitting the spectra 2.0.  FP32 matrix
// instructions took 2.35 ms (Nside 512 L 1535 B 12 0.80 -> 0.72 ms, Nside 256
// L 767 B 64 0.52 -> 0.46, Nside 128 L 301 B 5 0.028 -> 0.025).
template <int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_legendre_fwd_mfma(Tables tb, int B, const double *__restrict__ coefA, const float2 *__restrict__ XE,
                        const float2 *__restrict__ XO, float2 *__restrict__ alm, float f0, float fm, int accum) {
  const int b0 = 16 * blockIdx.y;  // channel group of this row of the grid
  __shared__ float tile[NW * kSubL * kTileRS];
  const int g = blockIdx.x;
  const int x = g & 7, k = g >> 3;
  const int i0 = tb.ck_xoff[x];
  if (k >= tb.ck_xoff[x + 1] - i0) return;  // uniform across the workgroup
  const int item = i0 + k;
  const int2 it = tb.ck_items[item];
  const int m = it.x, l0 = it.y;
  const int L = tb.lmax, M = L + 1, Rp = tb.npairs;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), j = tid & 63;
  const int h = j >> 5, col = j & 31;
  // columns beyond the batch read channel B-1 (finite data; their outputs are not stored)
  const int colc = (b0 + (col >> 1)) < B ? col : 2 * (B - 1 - b0) + (col & 1);
  // floats per ring pair in X; the fast load path needs 32 of them in 32 bits
  const size_t rowf = (size_t)M * B * 2;
  const bool fast_rows = rowf * 32 * sizeof(float) < (size_t)0x7fffffff;
  // the block's recurrence coefficients through the constant address space:
  // wave-uniform scalar loads (rows past lmax, never stored, read other columns
  // or the table's padding)
  typedef __attribute__((address_space(4))) const double cdouble;
  const cdouble *Ag = (const cdouble *)coefA + (m * (2 * L + 1 - m) / 2 + l0);  // nalm < 2^31
  float *tw = tile + w * kSubL * kTileRS;
  const float *xe_f = reinterpret_cast<const float *>(XE);
  const float *xo_f = reinterpret_cast<const float *>(XO);

  f32x16 acc[4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[a][r] = 0.f;
  // the scale of this lane's column (the imaginary ones of m = 0 are not used)
  float scale = m == 0 && (col & 1) ? 1.f : kTinyScale;
  int tiny = 2;  // uniform: 0 no column of the wave is scaled, 1 some are, 2 and nothing is summed yet

  // this lane's ring per chunk: recurrence start (kBlockL: not
  // active in this block), checkpoint and z, fetched one chunk ahead
  auto fetch_ring = [&](int q, int &t0, double2 &v, double &z) {
    const bool qok = q < Rp;
    t0 = qok ? (int)tb.ck_t[(size_t)item * Rp + q] : kBlockL;
    v = qok ? tb.ck_v[(size_t)item * Rp + q] : make_double2(0.0, 0.0);
    z = qok ? tb.rp_z[q] : 0.0;
  };
  int t0n;
  double2 vn;
  double zn;
  fetch_ring(w * 64 + j, t0n, vn, zn);
  for (int c0 = 0; c0 < Rp; c0 += 64 * NW) {
    const int t0 = t0n;
    const double2 v = vn;
    const double z = zn;
    // wait for this chunk's values here: the recurrence below then waits for
    // no load, while the spectrum loads issued before it are in flight
    asm volatile("" ::"v"(t0), "v"(v.x), "v"(v.y), "v"(z));
    fetch_ring(c0 + 64 * NW + w * 64 + j, t0n, vn, zn);
    if (__all(t0 >= kBlockL)) continue;  // no ring of this slice is active here
    // last start offset of the wave: later groups need no injection selects;
    // first start offset: a half block before it holds only zero lambdas
    int tx = t0 < kBlockL ? t0 : -1, tn = t0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      tx = max(tx, __shfl_xor(tx, o));
      tn = min(tn, __shfl_xor(tn, o));
    }
    const int tlast = __builtin_amdgcn_readfirstlane(tx);
    const int tfirst = __builtin_amdgcn_readfirstlane(tn);
    // B operands: K step s, element e of lane half h is ring c0 + 64 w + 16 s +
    // 8 h + e; FP32 values here, split after the recurrence that covers the loads
    float xf[2][32];             // [E, O][8 s + e]
    const int rw = c0 + w * 64;  // first ring of this wave's slice (uniform)
    if (fast_rows && rw + 64 <= Rp) {
      // buffer loads: one resource per slice (uniform base), the lane's byte
      // offset (half, column) in a VGPR and the ring's row offset in an SGPR, so
      // no per-load vector address arithmetic (offsets < 2^32 by fast_rows)
      const unsigned voff = (unsigned)(h * 8 * rowf + colc) * 4u;
      const size_t o0 = ((size_t)rw * M + m) * B * 2 + (size_t)b0 * 2;
      const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float *>(xe_f + o0), 0, 0xffffffff, kBufferWord3);
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float *>(xo_f + o0), 0, 0xffffffff, kBufferWord3);
#pragma unroll
      for (int s = 0; s < 32; ++s) {
        const unsigned so = (unsigned)((16 * (s >> 3) + (s & 7)) * rowf) * 4u;
        xf[0][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(re, voff, so, 0));
        xf[1][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ro, voff, so, 0));
      }
    } else {
      // rings beyond the last pair read the last pair (their lambda is zero)
#pragma unroll
      for (int s = 0; s < 32; ++s) {
        const int r = min(rw + 16 * (s >> 3) + 8 * h + (s & 7), Rp - 1);
        const size_t o = (((size_t)r * M + m) * B + b0) * 2 + colc;
        xf[0][s] = xe_f[o];
        xf[1][s] = xo_f[o];
      }
    }
    // issue the loads here, ahead of the recurrence (left alone, the compiler
    // sinks them to their first use after it and their latency is exposed)
    asm volatile("" ::: "memory");
    double prv = 0.0, cur = 0.0;
    // 64 steps of the recurrence from l0 + base, one lambda per lane per step
    // into the tile (rows: the half block's 32 even l, then its 32 odd l)
    auto recurrence = [&](int base) {
      double Ac[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) Ac[u] = Ag[base + u];
#pragma unroll 1
      for (int t8 = 0; t8 < kSubL / 8; ++t8) {
        const int tb8 = base + t8 * 8;
        // the next group's coefficients, once this group's have arrived (scalar
        // loads complete out of order: a wait for one is a wait for all)
        double An[8];
        int ta = tb8 + 8;
        asm volatile("" : "+s"(ta) : "s"(Ac[7]));
#pragma unroll
        for (int u = 0; u < 8; ++u) An[u] = Ag[ta + u];
        __builtin_amdgcn_sched_barrier(0);
        float *trow = tw + t8 * 4 * kTileRS + j;
        // rows l > lmax only feed output rows that are never stored
        if (tb8 <= tlast) {  // uniform: some ring starts in this group
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const double nx = fma(Ac[u] * z, cur, -prv);
            if (u == 0) {
              const bool inj = (tb8 == t0);
              prv = inj ? v.x : cur;
              cur = inj ? v.y : nx;
            } else {
              prv = cur;
              cur = nx;
            }
            trow[((u & 1) * 32 + (u >> 1)) * kTileRS] = (float)cur;
          }
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const double nx = fma(Ac[u] * z, cur, -prv);
            prv = cur;
            cur = nx;
            trow[((u & 1) * 32 + (u >> 1)) * kTileRS] = (float)cur;
          }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) Ac[u] = An[u];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    u32x4 xs[2][4][3];  // [E, O][K step][part]
    // contraction: rows l0 + 64 hb + 2 i (E) and + 1 (O); K = 4 steps of 16
    // rings, summed over the slice from zero and then added: products of a
    // smooth spectrum's leading parts repeat from ring to ring, and so would
    // the rounding of adding them to a long sum
    auto contract = [&](f32x16 &ce, f32x16 &co) {
      const float *rows = tw + col * kTileRS + h * 8;
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        f32x16 sum = {};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          u32x4 a[3];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float4 v4 = *reinterpret_cast<const float4 *>(rows + par * 32 * kTileRS + 16 * s + 4 * i);
            split3<true>(v4.x, v4.y, a, 2 * i);
            split3<true>(v4.z, v4.w, a, 2 * i + 1);
          }
          mfma_split(a, xs[par][s], sum);
        }
        f32x16 &c = par ? co : ce;
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] += sum[r];
        __builtin_amdgcn_sched_barrier(0);  // one parity's operands at a time (registers)
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // half blocks with no lambda are left out: every ring of the wave starts
    // after the first (the recurrence state stays zero until its start), or
    // every l of the second is beyond lmax (output rows that are never stored)
    const bool first = tfirst < kSubL;
    if (first) recurrence(0);
    if (tiny) {
      const float undo = tiny_step<64>([&](int i) { return xf[i & 1][i >> 1]; }, scale);
      if (tiny == 1 && __any(undo != 1.f)) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[a][r] *= undo;
      }
      tiny = __any(scale != 1.f) ? 1 : 0;
      if (tiny) {
#pragma unroll
        for (int s = 0; s < 32; ++s) {
          xf[0][s] *= scale;
          xf[1][s] *= scale;
        }
      }
    }
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) split3<true>(xf[par][8 * s + 2 * i], xf[par][8 * s + 2 * i + 1], xs[par][s], i);
        __builtin_amdgcn_sched_barrier(0);
      }
    if (first) contract(acc[0], acc[1]);
    if (l0 + kSubL <= L) {
      recurrence(kSubL);
      contract(acc[2], acc[3]);
    }
  }
  // sum the waves' partial tiles, red[w][l - l0][col] (row stride
  // kRedRS: the reads below walk l, conflict-free), and write the caller's
  // layout alm[b][idx(l, m)] = f_m c_lm a (Im = 0 for m = 0), or add to it
  __syncthreads();
  float *red = tile;
  const float unscale = scale != 1.f ? kTinyUndo : 1.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int hb = a >> 1, par = a & 1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r >> 2) + 4 * h + (r & 3);
      const int lrel = hb * kSubL + 2 * i + par;
      red[(w * kBlockL + lrel) * kRedRS + col] = unscale * acc[a][r];
    }
  }
  __syncthreads();
  const double *Cn = tb.coefC + alm_idx(m, m, L) - m;
  const size_t nalm = nalm_of(L);
  const size_t base = alm_idx(l0, m, L);
  const float f = (m == 0) ? f0 : fm;
  for (int e = tid; e < 16 * kBlockL; e += 64 * NW) {
    const int c = e / kBlockL, lrel = e % kBlockL;  // a wave walks 64 consecutive l of one channel
    const int l = l0 + lrel;
    if (l > L || b0 + c >= B) continue;
    float re = 0.f, im = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      re += red[(ww * kBlockL + lrel) * kRedRS + 2 * c];
      im += red[(ww * kBlockL + lrel) * kRedRS + 2 * c + 1];
    }
    const float g = f * (float)Cn[l];
    float2 v = make_float2(g * re, (m == 0) ? 0.f : g * im);
    float2 *dst = alm + (size_t)(b0 + c) * nalm + base + lrel;
    if (accum) {
      const float2 o = *dst;
      v.x += o.x;
      v.y += o.y;
    }
    *dst = v;
  }
}

// Synthesis.  Workgroup = one wave = (m, chunk of 64 ring pairs), one ring
// per lane, NC groups of 16 channels.  Per 32 steps of l every lane advances
// its ring's recurrence by 32 values, splits them and packs the 16 even and
// the 16 odd ones into the words of the A operands: v_permlane32_swap gives
// the 32-ring halves (lanes 0-31 the first 8 values of one parity, lanes
// 32-63 the last 8 of the same 32 rings), so no ring's recurrence is computed
// twice.  The B operands a[l][col] come as FP32 rows of the coefficient slab
// (L1/L2), loaded before the recurrence that hides their latency and split
// after it.  The recurrence coefficients are wave-uniform scalar loads, one
// group of 8 ahead.  No LDS, no barriers, and every wave starts at its own
// rings' first non-negligible l.  Workgroups are dealt so that all chunks
// of eight consecutive m run on one XCD (consecutive workgroups go to
// consecutive XCDs): they share the a_m slabs in L2.  A wave writes, per ring
// pair, whole [m][batch] rows of the synthesis spectra (32 consecutive floats
// per ring: one 128-byte line at 16 channels).  The slab holds half of each
// coefficient; the sums are doubled as they are stored.
//
// Bound by the vector ALU: per group of 32 l some 400 vector instructions
// (recurrence 72, conversions 32, splitting of lambda 176 and of the rows 88,
// half exchanges 24) beside 24 matrix instructions.  Timing copies (Nside 1024
// L 2047 B 16, 1.72 ms): without the matrix instructions 1.31 ms, without
// splitting lambda 1.35, without splitting the rows 1.52, without the half
// exchanges 1.65.  FP32 matrix instructions in this place took 2.03 ms (Nside
// 512 L 1535 B 12 0.67 -> 0.52 ms; Nside 256 L 767 B 64, two channel groups per
// wave, 0.40 -> 0.30 ms).  One group of channels runs three waves per SIMD
// (167 VGPRs; 1.88 ms with two), two groups two (253 VGPRs).
constexpr int kInvRings = 64;

template <int NC>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NC == 1 ? 3 : 2, NC == 1 ? 3 : 2)))
    k_legendre_inv_mfma(Tables tb, int B, int bg, const double *__restrict__ coefA, const float2 *__restrict__ ALMT,
                        SynLayout lay, float2 *__restrict__ GN, float2 *__restrict__ GS) {
  const int b0 = bg + 16 * NC * blockIdx.y;  // first channel of this row of the grid
  const int L = tb.lmax, Rp = tb.npairs;
  const int nch = (Rp + kInvRings - 1) / kInvRings;
  const int g = blockIdx.x;
  const int x = g & 7, q = g >> 3;
  // XCD x takes the octets x, x+8, ... of m; within an octet, m-major then chunk
  const int oct = x + 8 * (q / (8 * nch));
  const int r8 = q % (8 * nch);
  const int m = 8 * oct + r8 / nch;
  const int chunk = r8 % nch;
  if (m > L) return;  // uniform
  const int j = threadIdx.x;
  const int h = j >> 5, col = j & 31;
  const int p = chunk * kInvRings + j;
  const bool pok = p < Rp;
  const double z = pok ? tb.rp_z[p] : 0.0;
  const int ls = pok ? tb.seed_l[(size_t)m * Rp + p] : L + 1;
  const double2 sd = pok ? tb.seed_v[(size_t)m * Rp + p] : make_double2(0.0, 0.0);
  // first l any ring of the chunk needs (m + 8j, like every seed)
  int wh = ls;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) wh = min(wh, __shfl_xor(wh, o));
  const int wl = __builtin_amdgcn_readfirstlane(wh);
  if (wl > L && __all(!pok || m >= ring_orders(tb.rp_mtop[p]))) return;  // zero spectra, which the ring FFT does not read
  f32x16 acc[NC][4];
#pragma unroll
  for (int n = 0; n < NC; ++n)
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[n][a][r] = 0.f;
  // A[l] of this m through the constant address space: wave-uniform indices
  // become scalar loads into SGPRs
  // (32-bit index arithmetic keeps the address on the scalar unit; nalm < 2^31)
  typedef __attribute__((address_space(4))) const double cdouble;
  const int aoff = m * (2 * L + 1 - m) / 2;  // alm_idx(m, m, L) - m
  const cdouble *Ag = (const cdouble *)coefA + aoff;
  // B operands of the group from lq: lane (h, col) takes rows lq + 16 h + 2 e
  // + parity, e = 0..7.  The slab of column m is a buffer resource that ends
  // after row lmax: rows past it read as zero and need no mask (the bounds check
  // covers the VGPR offset, the lane's, plus the SGPR offset, the row's, which
  // stays within the resource).
  // Channels past the batch read channel B-1 (finite data, not stored).
  const float *ag = reinterpret_cast<const float *>(ALMT) + (size_t)aoff * B * 2;
  const unsigned rowb = 8u * (unsigned)B;  // bytes per row; (lmax + 1) rows of one m are below 2^32 bytes
  const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(ag), 0, (int)((unsigned)(L + 1) * rowb), kBufferWord3);
  unsigned vo[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    const int c = min(b0 + 16 * n + (col >> 1), B - 1);
    vo[n] = 16u * h * rowb + 8u * c + 4u * (col & 1);
  }
  float scale[NC];   // of this lane's columns (the imaginary ones of m = 0 are zero)
  bool tiny = true;  // some column of the wave is scaled (uniform)
#pragma unroll
  for (int n = 0; n < NC; ++n) scale[n] = m == 0 && (col & 1) ? 1.f : kTinyScale;
  double prv = 0.0, cur = 0.0;
  // One group of 32 steps from l = lq; ac holds A_l of its first 8 steps and
  // receives those of the next group's.  TAIL: the group holds l > lmax, whose
  // coefficients are taken as zero (the recurrence stays finite there and
  // meets zero rows of B).  CHECK: columns may be scaled (a test of `tiny` in the
  // loop without it took 2.5% more).
  auto group = [&](int lq, double (&ac)[8], auto tail, auto check) {
    constexpr bool TAIL = decltype(tail)::value, CHECK = decltype(check)::value;
    float bf[NC][2][8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        const int row = lq + 2 * e + par;
        const unsigned so = (unsigned)(TAIL ? min(row, L + 1) : row) * rowb;
#pragma unroll
        for (int n = 0; n < NC; ++n)
          bf[n][par][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ar, vo[n], so, 0));
      }
    asm volatile("" ::: "memory");  // issued here, ahead of the recurrence
    uint32_t w[2][3][8];            // [parity][part][pair of l]
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int l8 = lq + 8 * s;
      double an[8];
      int la = l8 + 8;
      if (la > L) la = l8;
      asm volatile("" : "+s"(la) : "s"(ac[7]));
#pragma unroll
      for (int u = 0; u < 8; ++u) an[u] = Ag[la + u];
      __builtin_amdgcn_sched_barrier(0);  // issued here, a group of 8 ahead of their use
      // a ring's state is exactly zero before its seed, so the seed enters as a
      // 0/1 factor on two fused multiply-adds (no selects, no branch)
      const double f = (l8 == ls) ? 1.0 : 0.0;
      float lam[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double a = !TAIL || l8 + u <= L ? ac[u] : 0.0;
        const double nx = fma(a * z, cur, -prv);
        if (u == 0) {
          prv = fma(f, sd.x, cur);
          cur = fma(f, sd.y, nx);
        } else {
          prv = cur;
          cur = nx;
        }
        lam[u] = f64_to_f32(cur);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int par = 0; par < 2; ++par)
          split3<false>(lam[4 * i + par], lam[4 * i + 2 + par], w[par], 2 * s + i);
#pragma unroll
      for (int u = 0; u < 8; ++u) ac[u] = an[u];
    }
    if (CHECK && tiny) {
      bool any = false;
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        const float undo = tiny_step<16>([&](int i) { return bf[n][i & 1][i >> 1]; }, scale[n]);
        if (lq != wl && __any(undo != 1.f)) {
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[n][a][r] *= undo;
        }
        any |= scale[n] != 1.f;
      }
      tiny = __any(any);
      if (tiny) {
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            bf[n][0][e] *= scale[n];
            bf[n][1][e] *= scale[n];
          }
      }
    }
#pragma unroll
    for (int par = 0; par < 2; ++par) {
      __builtin_amdgcn_sched_barrier(0);
      u32x4 a0[3], a1[3];  // rings 0-31 and 32-63 of the chunk
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto r = __builtin_amdgcn_permlane32_swap(w[par][k][i], w[par][k][i + 4], false, false);
          a0[k][i] = r[0];
          a1[k][i] = r[1];
        }
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        u32x4 b[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) split3<false>(bf[n][par][2 * i], bf[n][par][2 * i + 1], b, i);
        mfma_split2(a0, a1, b, acc[n][par], acc[n][2 + par]);
      }
    }
  };
  if (wl <= L) {
    double ac[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ac[u] = Ag[wl + u];
    int lq = wl;
#pragma unroll 1
    for (; tiny && lq + 31 <= L; lq += 32) group(lq, ac, std::false_type{}, std::true_type{});
#pragma unroll 1
    for (; lq + 31 <= L; lq += 32) group(lq, ac, std::false_type{}, std::false_type{});
    if (lq <= L) group(lq, ac, std::true_type{}, std::true_type{});
  }
  float *gn = reinterpret_cast<float *>(GN);
  float *gs = reinterpret_cast<float *>(GS);
  const size_t ringf = (size_t)lay.ns * lay.M * lay.G * 2;  // floats per ring pair
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    const int c = b0 + 16 * n + (col >> 1);
    if (c >= B) continue;
    const size_t cofs = lay.idx(0, c, m) * 2 + (col & 1);
    const float out = scale[n] != 1.f ? 2.f * kTinyUndo : 2.f;  // (the coefficients came halved)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = 8 * (r >> 2) + 4 * h + (r & 3);
        const int pr = chunk * kInvRings + hh * 32 + i;
        if (pr >= Rp) continue;
        const size_t o = (size_t)pr * ringf + cofs;
        gn[o] = out * (acc[n][2 * hh][r] + acc[n][2 * hh + 1][r]);
        gs[o] = out * (acc[n][2 * hh][r] - acc[n][2 * hh + 1][r]);
      }
    }
  }
}

bool mfma_fwd_supported(const Tables &tb) { return tb.nitems > 0; }

hipError_t launch_legendre_fwd_mfma(const Tables &tb, int B, const float2 *XE, const float2 *XO, float2 *alm, double f0,
                                    double fm, int accum, hipStream_t st) {
  // grid: 8 XCD groups x the longest group
  int longest = 0;
  {
    // item counts per XCD group follow from the same enumeration as k_items
    const int L = tb.lmax;
    for (int xg = 0; xg < 8; ++xg) {
      int c = 0;
      for (int m = xg; m <= L; m += 8) c += (L - m + kBlockL) / kBlockL;
      longest = c > longest ? c : longest;
    }
  }
  // all 16-channel groups in one launch (one tail instead of one per group);
  // one wave per workgroup from 2048 ring pairs (Nside 1024 B 16: 2.30 ms
  // against 2.33 with two waves and 2.43 with four), two below (Nside 512
  // B 16: 0.401 ms against 0.414 with one and 0.411 with four)
  const dim3 grid(8 * longest, (B + 15) / 16);
  if (tb.npairs >= 2048)
    hipLaunchKernelGGL(k_legendre_fwd_mfma<1>, grid, dim3(64), 0, st, tb, B, tb.coefA, XE, XO, alm, (float)f0,
                       (float)fm, accum);
  else
    hipLaunchKernelGGL(k_legendre_fwd_mfma<2>, grid, dim3(128), 0, st, tb, B, tb.coefA, XE, XO, alm, (float)f0,
                       (float)fm, accum);
  return hipGetLastError();
}

hipError_t launch_legendre_inv_mfma(const Tables &tb, int B, const float2 *ALMT, SynLayout lay, float2 *GN,
                                    float2 *GS, hipStream_t st) {
  const int nch = (tb.npairs + kInvRings - 1) / kInvRings;
  const int noct = (tb.lmax + 1 + 7) / 8;
  const int per_xcd = ((noct + 7) / 8) * 8 * nch;  // octets per XCD x 8 m x chunks
  // pairs of 16-channel groups share a wave's recurrence, then one group; where
  // the waves do not fill the chip, each group has its own (B 17, whole call:
  // Nside 64 L 127 54 us as a pair, 50 as two groups of FP32 products)
  const int n32 = tb.npairs > 256 ? (B + 15) / 32 : 0;
  if (n32 > 0)
    hipLaunchKernelGGL(k_legendre_inv_mfma<2>, dim3(8 * per_xcd, n32), dim3(64), 0, st, tb, B, 0, tb.coefA, ALMT, lay,
                       GN, GS);
  if (32 * n32 < B)
    hipLaunchKernelGGL(k_legendre_inv_mfma<1>, dim3(8 * per_xcd, (B - 32 * n32 + 15) / 16), dim3(64), 0, st, tb, B, 32 * n32, tb.coefA, ALMT,
                       lay, GN, GS);
  return hipGetLastError();
}

}  // namespace shtx
