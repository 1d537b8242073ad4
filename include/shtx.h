/*
 * shtx -- spherical harmonic transforms on HEALPix RING grids for AMD
 * Instinct MI355X (gfx950).  C ABI of libshtx.so.
 *
 * The library computes, for real maps on the HEALPix grid (Sec. III-A of the
 * paper: Npix = 12 nside^2 pixels on 4 nside - 1 iso-latitude rings, RING
 * pixel order north to south, Sec. III-B) and complex spherical harmonic
 * coefficients a_lm, 0 <= m <= l <= lmax:
 *
 *   map2alm  (analysis, Eq. (1) / Eq. (26) with equal weights W = 4 pi/Npix)
 *       a_lm = (4 pi / Npix) sum_p f_p conj(Y_lm(theta_p, phi_p))
 *   alm2map  (synthesis, Eq. (2) / Eq. (24))
 *       f_p = sum_l sum_{-l<=m<=l} a_lm Y_lm(theta_p, phi_p),
 *             a_{l,-m} = (-1)^m conj(a_lm)
 *   map2alm_backward / alm2map_backward: the adjoints of the two transforms
 *       (Sec. III-F: the synthesis' adjoint is the conjugate transpose of
 *       its matrix, the analysis' adjoint the synthesis scaled by the
 *       quadrature weights) in the
 *       convention of PyTorch complex autograd (grad = dL/dRe + i dL/dIm) on
 *       the m >= 0 storage:
 *       map2alm_backward(G) = (4 pi/Npix) alm2map(G'),  G'_l0 = Re G_l0,
 *                             G'_lm = G_lm / 2 (m > 0)
 *       alm2map_backward(g) = unit-weight analysis sum of g, times 2 for m > 0,
 *                             Im of m = 0 set to 0.
 * Y_lm is orthonormal (Eq. (8)-(9)) with the Condon-Shortley sign (-1)^m of
 * Eq. (15) taken once.  Each transform is a per-ring FFT (Eq. (13)) followed
 * by the Legendre sum (Eq. (14)) with lambda_lm generated by the three-term
 * recurrence of Eq. (16) in FP64 on the device.
 *
 * Layouts (all contiguous, caller-owned, device memory):
 *   map  [batch][12 nside^2]        RING order; double (F64), float (F32) or
 *                                   bfloat16 bits as uint16 (BF16)
 *   alm  [batch][nalm] complex      interleaved (re, im); complex128 for F64,
 *                                   complex64 for F32 and BF16;
 *                                   nalm = (lmax+1)(lmax+2)/2,
 *                                   idx(l,m) = m (2 lmax + 1 - m)/2 + l.
 *   Output Im(a_l0) is written as 0; input Im(a_l0) is ignored.
 *   Alignment: map pointers 16-byte aligned (8-byte for BF16), alm pointers
 *   aligned to their complex element (16 / 8 bytes); SHTX_ERR_ARG otherwise.
 *
 * Streams: `stream` is a hipStream_t (NULL = the default stream).  Every
 * transform call only validates its arguments on the host and enqueues
 * kernels on `stream`; it never allocates, frees or synchronises.  Outputs
 * are overwritten, never accumulated into; inputs and outputs must not alias.
 * Concurrent calls on different streams need distinct workspaces; a table
 * buffer may be shared by any number of concurrent calls once built.
 *
 * Non-finite values stay in their channel.  There an infinite or NaN pixel
 * makes the coefficients that its ring contributes to non-finite, and an
 * infinite or NaN coefficient a_lm the pixels of every ring where lambda_lm
 * counts; which of them are infinite and which NaN is not specified.  Rings
 * where no lambda_l'm of its order m, l' <= lmax, reaches some 2^-64 take none of
 * that order, so such a coefficient leaves their pixels finite.
 *
 * Errors: arguments are checked before anything is launched; a failed check
 * returns a status code and launches nothing.  A launch failure returns
 * SHTX_ERR_HIP; a fault inside a kernel surfaces at the caller's next
 * synchronisation.
 */
#ifndef SHTX_H
#define SHTX_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Element type of maps (alm use the complex type of the compute precision). */
typedef enum {
  SHTX_F64 = 0,  /* double maps, complex128 alm, FP64 arithmetic */
  SHTX_F32 = 1,  /* float maps, complex64 alm, FP32 ring FFT and contraction,
                    FP64 Legendre recurrence */
  SHTX_BF16 = 2  /* bfloat16 maps, complex64 alm, FP32 arithmetic; accepted by
                    map2alm and map2alm_backward only */
} shtx_dtype;

typedef enum {
  SHTX_OK = 0,
  SHTX_ERR_ARG = 1,          /* invalid argument (null pointer, bad size, ...) */
  SHTX_ERR_UNSUPPORTED = 2,  /* valid but not supported (nside > 2048, BF16
                                synthesis, ...) */
  SHTX_ERR_WORKSPACE = 3,    /* work_bytes below shtx_workspace_bytes() */
  SHTX_ERR_HIP = 4,          /* a HIP runtime call or launch failed */
  SHTX_ERR_TABLES = 5,       /* tables pointer not built for (nside, lmax) */
  SHTX_ERR_SCRATCH = 6       /* request larger than the fixed scratch of
                                shtx_map2alm_noalloc */
} shtx_status;

/* Version of this ABI (major*10000 + minor*100 + patch). */
int shtx_version(void);

/* Static description of a status code (host memory, never freed). */
const char *shtx_status_string(int status);

/*
 * Resident tables for one (nside, lmax): ring-pair geometry, recurrence
 * coefficients, FP64 Legendre seeds at each ring's first non-negligible l,
 * and the roots of unity of every ring length.  Size in bytes, or 0 when
 * (nside, lmax) is invalid.  nside must be a power of two in [1, 2048];
 * 0 <= lmax <= 8191.
 */
size_t shtx_tables_bytes(int nside, int lmax);

/*
 * Compute the tables into `tables` (device memory of at least
 * shtx_tables_bytes(nside, lmax) bytes, 256-byte aligned) by kernels enqueued
 * on `stream`, and register the pointer for (nside, lmax).  The tables are
 * ready for any call ordered after this one on `stream` (or after the caller
 * synchronises it).  The caller owns the memory; building again over the same
 * pointer re-registers it.
 */
int shtx_tables_build(int nside, int lmax, void *tables, size_t tables_bytes, void *stream);

/*
 * Legendre work of the pruned triangle: the sums of Eq. (14) and (24)
 * restricted to the l where the normalised Legendre function of Eq. (15)-(16)
 * is not negligible (a restriction of this library, not of the paper):
 * *executed = sum over m = 0..lmax and ring pairs p of (lmax + 1 - l_s), with
 * l_s the first l the kernels evaluate for (m, p) (lmax + 1 when none), and
 * *full = (lmax+1)(lmax+2)/2 * (2 nside) (every (l, m, p) triple).  Waits for
 * `stream` (the tables' build stream), then copies the seed table to host
 * memory: a set-up query, not for hot loops.  SHTX_ERR_TABLES when `tables`
 * is not registered; SHTX_ERR_ARG for null outputs.
 */
int shtx_tables_work(const void *tables, long long *executed, long long *full, void *stream);

/* Forget the registration of a table buffer (before the caller frees it). */
int shtx_tables_release(const void *tables);

/* Bytes of scratch device memory a transform call needs: two spectrum
   buffers of (lmax+1) * 2 nside * B' complex values, B' = batch rounded up to
   whole channel slices of the ring FFT (at most 15 more), and the
   coefficients in the kernels' layout (for BF16 maps, the larger of that and
   the analysis' BF16 spectra in matrix-operand order: 2 x ceil(batch/16) x
   (lmax+1) x ceil(2 nside/8) x 512 bytes).  0 if invalid or nside > 2048. */
size_t shtx_workspace_bytes(int nside, int lmax, int batch, int dtype);

/*
 * Forward transform map2alm: map [batch][Npix] -> alm [batch][nalm].
 * `tables` must have been built for (nside, lmax); `work` must hold at least
 * shtx_workspace_bytes(nside, lmax, batch, dtype) bytes (256-byte aligned).
 */
int shtx_map2alm(int nside, int lmax, int batch, int dtype, const void *map, void *alm, const void *tables,
                 void *work, size_t work_bytes, void *stream);

/*
 * map2alm with quadrature weights per ring instead of the equal pixel weight
 * 4 pi / Npix (the ring weights of Sec. IV-A, which lower the round-trip
 * error):  a_lm = sum_r w_r sum_(j in ring r) f_j conj(Y_lm).  ring_weights
 * is device memory of 2 nside doubles (8-byte aligned), one per ring pair:
 * entry p weights the north ring p + 1 (1-based, from the pole) and its
 * mirror 4 nside - 1 - p, entry 2 nside - 1 the equator ring; the values are
 * the caller's (no weight data ships with the library).  Otherwise as
 * shtx_map2alm; a null or misaligned ring_weights is SHTX_ERR_ARG.
 */
int shtx_map2alm_weighted(int nside, int lmax, int batch, int dtype, const void *map, void *alm,
                          const double *ring_weights, const void *tables, void *work, size_t work_bytes,
                          void *stream);

/*
 * map2alm of maps in NESTED order (map_nest [batch][Npix], the hierarchical
 * order of Sec. III-B): the same transform as shtx_map2alm of the RING-ordered
 * maps, with the layout conversion fused into the ring FFT's loads (each ring
 * pixel read at its NESTED index from a RING -> NESTED table among the
 * resident tables) instead of a separate reorder pass; the coefficients are
 * bit-identical to shtx_nest2ring followed by shtx_map2alm.  Arguments,
 * workspace and errors as shtx_map2alm.
 */
int shtx_map2alm_nested(int nside, int lmax, int batch, int dtype, const void *map_nest, void *alm,
                        const void *tables, void *work, size_t work_bytes, void *stream);

/*
 * map2alm with one quadrature weight per pixel (the pixel weights of Sec.
 * IV-A): a_lm = sum_p w_p f_p conj(Y_lm(p)).  pixel_weights is device memory
 * of 12 nside^2 doubles in RING order (16-byte aligned), the caller's values
 * (no weight data ships with the library).  Otherwise as shtx_map2alm; a null
 * or misaligned pixel_weights is SHTX_ERR_ARG.
 */
int shtx_map2alm_pixel_weighted(int nside, int lmax, int batch, int dtype, const void *map, void *alm,
                                const double *pixel_weights, const void *tables, void *work, size_t work_bytes,
                                void *stream);

/*
 * Stored-lambda analysis (the paper's precomputed Legendre tensor, Sec.
 * III-G, Eq. (28), kept resident in device memory for a hot (nside, lmax)
 * instead of streamed from the host): the BF16 Legendre operands of the BF16
 * matrix-core analysis, written once into a caller-owned table and then read
 * by shtx_map2alm_stored instead of being recomputed by the FP64 recurrence.
 * Only the pruned triangle's tiles are stored (64 l x 128 ring pairs of BF16
 * per tile, after a per-block offset table): about 7 GB at nside 1024,
 * lmax 2047.
 *   shtx_lambda_table_bytes: size of that table for a registered tables
 *     buffer (reads the tables back to the host after waiting for `stream`:
 *     a set-up query);
 *   shtx_lambda_table_build: writes the table into `lam` (device memory,
 *     256-byte aligned, at least that size; SHTX_ERR_WORKSPACE otherwise)
 *     with a synchronous copy and a kernel on `stream`, and registers it for
 *     `tables`;
 *   shtx_lambda_table_release: forgets the registration (before the caller
 *     frees the memory).
 * shtx_map2alm_stored: map2alm of BF16 maps (dtype SHTX_BF16 only, else
 * SHTX_ERR_UNSUPPORTED) through the BF16 matrix-core analysis with lambda read
 * from `lam` (built for `tables`, else SHTX_ERR_TABLES); bit-identical to
 * shtx_map2alm's BF16 matrix-core path.  Other arguments as shtx_map2alm.
 * Neither nside above 2048 nor tables without recurrence checkpoints are
 * supported (SHTX_ERR_UNSUPPORTED).
 */
int shtx_lambda_table_bytes(const void *tables, size_t *bytes, void *stream);
int shtx_lambda_table_build(const void *tables, void *lam, size_t lam_bytes, void *stream);
int shtx_lambda_table_release(const void *lam);
int shtx_map2alm_stored(int nside, int lmax, int batch, int dtype, const void *map, void *alm, const void *tables,
                        const void *lam, void *work, size_t work_bytes, void *stream);

/*
 * Allocation-free map2alm, for callers that cannot allocate device memory
 * (code under HIP graph capture, tight serving loops, harnesses that forbid
 * hipMalloc): the same transform and kernels as shtx_map2alm, with its
 * scratch (the spectrum buffers) in a fixed array of
 * SHTX_NOALLOC_SCRATCH_BYTES inside the library instead of a caller
 * workspace.  The library holds one such array per device until the process
 * ends; this call allocates and frees nothing.  Requests whose spectra need
 * more (2 x (lmax+1) x 2 nside x B' complex values, B' as for
 * shtx_workspace_bytes, plus for BF16 maps their operand-order copy sized
 * there) return SHTX_ERR_SCRATCH and launch nothing; e.g.
 * nside 256, lmax 511, 8 FP32 channels fits, nside 1024 does not.  Every call
 * on one device shares that device's array: calls that overlap in time on one
 * device (different streams or host threads without ordering) race on it and
 * give undefined results; calls ordered on one stream are safe.  Other
 * arguments and errors as shtx_map2alm.
 */
#define SHTX_NOALLOC_SCRATCH_BYTES (64u << 20)
size_t shtx_noalloc_scratch_bytes(void);
int shtx_map2alm_noalloc(int nside, int lmax, int batch, int dtype, const void *map, void *alm, const void *tables,
                         void *stream);

/* Inverse transform alm2map: alm [batch][nalm] -> map [batch][Npix].
   dtype F64 or F32. */
int shtx_alm2map(int nside, int lmax, int batch, int dtype, const void *alm, void *map, const void *tables,
                 void *work, size_t work_bytes, void *stream);

/*
 * Iterative refinement of map2alm (Eq. (4)-(5)): a^0 = A f, then niter times
 * a <- a + A (f - S a), with A the analysis and S the synthesis of this
 * library (niter + 1 forward and niter inverse transforms; niter = 3 is the
 * usual setting).  dtype F64 or F32; 0 <= niter <= 64 (SHTX_ERR_ARG
 * otherwise).  `work` must hold shtx_iter_workspace_bytes() bytes: the
 * transform workspace followed by one residual map.  `map` is only read.
 */
size_t shtx_iter_workspace_bytes(int nside, int lmax, int batch, int dtype);
int shtx_map2alm_iter(int nside, int lmax, int batch, int dtype, const void *map, void *alm, int niter,
                      const void *tables, void *work, size_t work_bytes, void *stream);

/*
 * The same refinement with the weighted analysis A_w (Sec. IV-A's quadrature
 * weight schemes; Eq. (4) with W the weights): a = A_w f, then niter times
 * a <- a + A_w (f - S a).  ring_weights: 2 nside doubles per ring pair as for
 * shtx_map2alm_weighted, or null; pixel_weights: 12 nside^2 doubles in RING
 * order as for shtx_map2alm_pixel_weighted, or null.  Both null: equal weights
 * (shtx_map2alm_iter); pixel weights alone: ring weight 1; both: their
 * product.  Device memory, 8- and 16-byte aligned (SHTX_ERR_ARG otherwise).
 * Workspace and other arguments as shtx_map2alm_iter.
 */
int shtx_map2alm_iter_weighted(int nside, int lmax, int batch, int dtype, const void *map, void *alm, int niter,
                               const double *ring_weights, const double *pixel_weights, const void *tables,
                               void *work, size_t work_bytes, void *stream);

/* Adjoint of map2alm: grad_alm [batch][nalm] -> grad_map [batch][Npix]
   (BF16 writes a bfloat16 gradient map from complex64 grad_alm). */
int shtx_map2alm_backward(int nside, int lmax, int batch, int dtype, const void *grad_alm, void *grad_map,
                          const void *tables, void *work, size_t work_bytes, void *stream);

/* Adjoint of alm2map: grad_map [batch][Npix] -> grad_alm [batch][nalm].
   dtype F64 or F32. */
int shtx_alm2map_backward(int nside, int lmax, int batch, int dtype, const void *grad_map, void *grad_alm,
                          const void *tables, void *work, size_t work_bytes, void *stream);

/*
 * Pixel order conversion between RING and NESTED (the hierarchical order of
 * the HEALPix grid of Sec. III-A: pixel p = f nside^2 + interleave(x, y) of
 * base pixel f, face coordinates x in the even and y in the odd bits; the
 * paper benchmarks this remapping alongside the transforms).  Maps are
 * [batch][12 nside^2] in device memory, elements of the dtype's size (F64 8,
 * F32 4, BF16 2 bytes; copied bit for bit), aligned to that size.  nside is a
 * power of two in [1, 8192], batch >= 1.  `map_nest` / `map_ring` must not
 * overlap (SHTX_ERR_ARG).  Enqueued on `stream`; no allocation, no
 * synchronisation; no tables needed.
 */
int shtx_nest2ring(int nside, int batch, int dtype, const void *map_nest, void *map_ring, void *stream);
int shtx_ring2nest(int nside, int batch, int dtype, const void *map_ring, void *map_nest, void *stream);

/*
 * Any-to-any pixel layout conversion through face coordinates (Sec. III-B,
 * Fig. 3-4: source -> (x, y, f) -> target, with face f = 0..11 and
 * 0 <= x, y < nside inside the face).  Layout codes:
 *   SHTX_LAYOUT_RING     the RING order of the transforms;
 *   SHTX_LAYOUT_NESTED   f nside^2 + interleave(x, y) (x in the even bits);
 *   SHTX_LAYOUT_FLAT + 2 origin + clockwise   (origin 0..3 = S, E, N, W;
 *                        clockwise 0 or 1): f nside^2 + r nside + c, each
 *                        face an image whose column axis c runs from the
 *                        origin corner towards the next corner
 *                        counter-clockwise (S -> E -> N -> W, seen from
 *                        outside with north up) and row axis r towards the
 *                        previous one; clockwise exchanges c and r.  Face
 *                        corners S = (x, y) = (0, 0), E = (nside-1, 0),
 *                        N = (nside-1, nside-1), W = (0, nside-1): origin S
 *                        counter-clockwise is c = x, r = y.  The paper names
 *                        the flat layout's reference corner and orientation
 *                        without a formula; this is this library's reading.
 * Maps, dtypes, sizes and errors as shtx_nest2ring (an unknown layout code is
 * SHTX_ERR_ARG); src_layout == dst_layout copies.
 */
#define SHTX_LAYOUT_RING 0
#define SHTX_LAYOUT_NESTED 1
#define SHTX_LAYOUT_FLAT 2
int shtx_reorder(int nside, int batch, int dtype, int src_layout, int dst_layout, const void *in, void *out,
                 void *stream);

/*
 * Spectral resize: alm_in [batch][nalm(lmax_in)] -> alm_out
 * [batch][nalm(lmax_out)] (layout of the transforms), a_lm copied bit for bit
 * for l <= min(lmax_in, lmax_out) and zero for lmax_in < l <= lmax_out: the
 * truncation or zero extension of a band-limited spectrum (with an analysis
 * at one nside and a synthesis at another, a change of resolution: the
 * regridding of Sec. IV-D).  dtype F64 (complex128) or F32
 * (complex64); 0 <= lmax <= 8191; batch >= 1; the buffers must not overlap
 * (SHTX_ERR_ARG).  Enqueued on `stream`; no allocation, no tables needed.
 */
int shtx_alm_resize(int lmax_in, int lmax_out, int batch, int dtype, const void *alm_in, void *alm_out,
                    void *stream);

/*
 * Stage timing (for benchmarks and profiling).  While enabled, every kernel
 * launch of later transform calls is bracketed by HIP events recorded on the
 * call's stream; shtx_profile_read synchronises those events and returns the
 * summed GPU time and launch count of one stage.  Stages:
 *   0 ring FFT (analysis), 1 Legendre (analysis, writes the caller's
 *   coefficient layout), 2 coefficient input layout, 3 Legendre (synthesis),
 *   4 ring FFT (synthesis), 5 BF16 analysis spectra rewritten in matrix
 *   operand order (BF16 maps on the matrix cores, before stage 1).
 * Not meant for concurrent use from several host threads.
 */
int shtx_profile_enable(int on);
int shtx_profile_reset(void);
int shtx_profile_read(int stage, double *total_ms, long long *launches);
const char *shtx_stage_name(int stage);

#ifdef __cplusplus
}
#endif

#endif /* SHTX_H */
