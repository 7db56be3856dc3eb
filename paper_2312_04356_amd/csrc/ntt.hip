// Negacyclic NTT over RNS limbs for N >= 4096 (gfx950).
//
// Same transform as the LDS-staged generic kernels (forward Cooley-Tukey stages
// m = 1..N/2 with psi^rev(m+i), inverse Gentleman-Sande with psi^-rev(h+i) and
// N^-1), organised for registers:
//   * N = N1 * 4096.  The first log2(N1) stages couple words with equal index
//     mod 4096: one thread owns a whole column of N1 words (coalesced loads at
//     stride 4096, twiddles uniform across the wavefront) - no LDS at all.
//   * The last 12 stages stay inside a 4096-word tile: 512 threads own 8 words each
//     and run 4 rounds of 3 radix-2 stages in registers; between rounds the tile goes
//     through LDS once.  Global loads and stores are fully coalesced.
// Which words a thread holds outside its rounds:
//   across the block (forward in, inverse out): tid + 512 k;
//   across its wave (forward out, inverse in): wv8(tid) + 64 k, wv8 = 512 wave + lane.
#include <algorithm>

#include "internal.h"

namespace nj {

constexpr int kT = 4096;
constexpr int kNT = 256;

// FP64 values between passes, stored in a word's place
__device__ __forceinline__ double b2d(uint64_t x) { return __longlong_as_double((long long)x); }
__device__ __forceinline__ uint64_t d2b(double x) { return (uint64_t)__double_as_longlong(x); }

// Rounds are lazy in both directions: no correction inside, centred reductions (reduce_c)
// where the bound asks for one.  With t < 2^50 the lazy product of a word below B t in
// magnitude lies within (1/2 + 3B/8) t (the quotient estimate is off by at most 1/2 + 3
// ulp-relative errors of a value below B 2^50).
//   Forward: the bound grows 1/2 -> 1.19 -> 2.13 -> 3.43 -> 5.22 -> 7.68 over 5 stages from
//   centred words (1 -> 7.01 over 4 from canonical ones).
//   Inverse: sums double, 1/2 -> 1 -> 2 -> 4 -> 8 from centred words (products of
//   differences stay below 3.5).
// So every intermediate is an integer below 2^53 (8 t + 32 < 2^53 for t <= 2^50 - 4),
// computed exactly.  A butterfly costs 9 to 9.5 FP64 operations, rounds included, in either
// direction.  Words travel between the passes of one transform as FP64 values, centred;
// what leaves a transform is canonical.

// orders a wave's LDS writes before its own later reads (no other wave is waited for)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------- tile passes: 512 threads, 8 words each
//
// 4 rounds of 3 stages.  Round 0 (strides 2048..512) holds words tid + 512 k; after it a wave
// owns 512 contiguous words and the rest needs no barrier: round 1 (256..64) wv8(tid) + 64 k,
// round 2 (32..8) 64 (tid >> 3) + (tid & 7) + 8 k, round 3 (4..1) 8 tid + k.  The twiddles of
// rounds 0 and 1 are the same for a whole wave: scalar loads.  The LDS tile is padded by one
// word every 8: every access pattern above then spreads over all banks.
// Eight words leave registers for what else a kernel reads or sums through the transform, all of
// it requested before, and 8 waves per SIMD by LDS where it reads little.  Against 256 threads
// of 16 words in 3 rounds of 4 stages (one LDS exchange less): a conv at level 1, N = 2^16, 158
// against 169 us, conv + CoeffToSlot at N = 2^14 685 / 733, one rotation at level 23 113 / 117,
// a batch of 11 32.8 / 33.2 ms.
constexpr int kNT8 = 512;
__device__ __forceinline__ int pad8(int x) { return x + (x >> 3); }
__device__ __forceinline__ int wv8(int tid) { return ((tid & ~63) << 3) | (tid & 63); }

// Twiddles of one tile's forward pass for blocks that transform many limbs of one prime and
// tile, so that the transform waits for no vector memory operation: round 2's staged in LDS
// (stage st: entry (g, i) of 64 2^st, g = tid >> 3, at 64 (2^st - 1) + (g << st) + i), round 3's 7
// of each thread in its registers.
constexpr int kTw8R2 = 64 * 7;

__device__ __forceinline__ void load_twiddles8(double *tws, double tw3[7], const double *W, int tile, int logN1, int N,
                                               int tid)
{
    if (tid < kTw8R2) {
        const int st = tid < 64 ? 0 : tid < 192 ? 1 : 2, mm = N / (2 * (32 >> st));
        tws[tid] = W[mm + tile * (mm >> logN1) + tid - 64 * ((1 << st) - 1)];
    }
#pragma unroll
    for (int st = 0; st < 3; st++) {
        const int mm = N / (2 * (4 >> st));
#pragma unroll
        for (int i = 0; i < (1 << st); i++) tw3[(1 << st) - 1 + i] = W[mm + tile * (mm >> logN1) + (tid << st) + i];
    }
}

// one forward stage of a 3-stage round (st 0..2) on 8 words; tw(i): the stage's twiddle i
template <typename F>
__device__ __forceinline__ void ct8(double v[8], int st, Mod m, F tw)
{
    const int step = 4 >> st;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        if (k & step) continue;
        const double U = v[k], V = mul_lazy(v[k + step], tw(k >> (3 - st)), m);
        v[k] = U + V;
        v[k + step] = U - V;
    }
}
__device__ __forceinline__ void reduce8(double v[8], Mod m)
{
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = reduce_c(v[k], m);
}

// The last 12 forward stages of one tile from centred words tid + 512 k, left in s at
// pad8, below 2.2 t: the bound grows 1/2 -> 1.19 -> 2.13 -> 3.43 -> 5.22 -> 7.68 over 5
// stages, so words are reduced after stages 5 and 10 only.  No other wave may still be
// reading s on entry; on return a thread may read its words wv8(tid) + 64 k.  `mid` runs
// after the one barrier.
template <typename F>
__device__ __forceinline__ void tile_forward8(double v[8], double *s, const double *tws, const double tw3[7], int tid,
                                              int tile, int logN1, const double *W, int N, Mod m, F mid)
{
    const ConstTab<double> C = const_tab(W);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = tid >> 3;
    double *sb = s + pad8(tid), *sw = s + pad8(wv8(tid)), *s2 = s + 72 * g + (tid & 7), *s3 = s + 9 * tid;
    auto uni = [&](int t, int hi) {  // twiddles of stride t in block hi of that stride's round
        const int mm = N / (2 * t);
        return C + mm + tile * (mm >> logN1) + hi;
    };
#pragma unroll
    for (int st = 0; st < 3; st++) {
        const auto w = uni(2048 >> st, 0);
        ct8(v, st, m, [&](int i) { return w[i]; });
    }
#pragma unroll
    for (int k = 0; k < 8; k++) sb[576 * k] = v[k];
    __syncthreads();
    mid();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = sw[72 * k];
#pragma unroll
    for (int st = 0; st < 3; st++) {
        const auto w = uni(256 >> st, wave << st);
        if (st == 2) reduce8(v, m);
        ct8(v, st, m, [&](int i) { return w[i]; });
    }
#pragma unroll
    for (int k = 0; k < 8; k++) sw[72 * k] = v[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = s2[9 * k];
#pragma unroll
    for (int st = 0; st < 3; st++) ct8(v, st, m, [&](int i) { return tws[64 * ((1 << st) - 1) + (g << st) + i]; });
#pragma unroll
    for (int k = 0; k < 8; k++) s2[9 * k] = v[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = s3[k];
#pragma unroll
    for (int st = 0; st < 3; st++) {
        if (st == 1) reduce8(v, m);
        ct8(v, st, m, [&](int i) { return tw3[(1 << st) - 1 + i]; });
    }
#pragma unroll
    for (int k = 0; k < 8; k++) s3[k] = v[k];
    wave_sync();
}

// one inverse stage of a 3-stage round (st 2..0) on 8 words
template <typename F>
__device__ __forceinline__ void gs8(double v[8], int st, Mod m, F tw)
{
    const int step = 4 >> st;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        if (k & step) continue;
        const double U = v[k], V = v[k + step];
        v[k] = U + V;
        v[k + step] = mul_lazy(U - V, tw(k >> (3 - st)), m);
    }
}

// The first 12 inverse stages of one tile from centred words wv8(tid) + 64 k to centred
// words tid + 512 k (sums 1/2 -> 4 over a round).  No other wave may still be reading s.
__device__ __forceinline__ void tile_inverse8(double v[8], double *s, int tid, int tile, int logN1, const double *W,
                                              int N, Mod m)
{
    const ConstTab<double> C = const_tab(W);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = tid >> 3;
    double *sb = s + pad8(tid), *sw = s + pad8(wv8(tid)), *s2 = s + 72 * g + (tid & 7), *s3 = s + 9 * tid;
    auto at = [&](int t, int hi) {
        const int hh = N / (2 * t);
        return hh + tile * (hh >> logN1) + hi;
    };
#pragma unroll
    for (int k = 0; k < 8; k++) sw[72 * k] = v[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = s3[k];
#pragma unroll
    for (int st = 2; st >= 0; st--) {
        const double *w = W + at(4 >> st, tid << st);
        gs8(v, st, m, [&](int i) { return w[i]; });
    }
    reduce8(v, m);
#pragma unroll
    for (int k = 0; k < 8; k++) s3[k] = v[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = s2[9 * k];
#pragma unroll
    for (int st = 2; st >= 0; st--) {
        const double *w = W + at(32 >> st, g << st);
        gs8(v, st, m, [&](int i) { return w[i]; });
    }
    reduce8(v, m);
#pragma unroll
    for (int k = 0; k < 8; k++) s2[9 * k] = v[k];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = sw[72 * k];
#pragma unroll
    for (int st = 2; st >= 0; st--) {
        const auto w = C + at(256 >> st, wave << st);
        gs8(v, st, m, [&](int i) { return w[i]; });
    }
    reduce8(v, m);
#pragma unroll
    for (int k = 0; k < 8; k++) sw[72 * k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = sb[576 * k];
#pragma unroll
    for (int st = 2; st >= 0; st--) {
        const auto w = C + at(2048 >> st, 0);
        gs8(v, st, m, [&](int i) { return w[i]; });
    }
    reduce8(v, m);
}

// rows pass: last 12 stages on 4096-word tiles.  grid (N/4096, limbs).  part: the forward's
// input and the inverse's output are FP64 words of the pass beside it (a column pass, or a
// kernel that does its work); else the tile is the whole transform, N = 4096.
template <bool INV>
__global__ __launch_bounds__(kNT8) void k_ntt_tile(uint64_t *data, const uint64_t *src, LimbTab lt, int part,
                                                   const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[INV ? 1 : kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12;
    const int limb = blockIdx.y, pidx = lt.pidx[limb], tile = blockIdx.x, tid = threadIdx.x;
    const PrimeInfo pi = info[pidx];
    const Mod m = pi.m;
    const size_t off = (size_t)lt.off[limb] * N + (size_t)tile * kT;
    const uint64_t *in = src ? src + (size_t)lt.soff[limb] * N + (size_t)tile * kT : data + off;
    const double *W = tw + (size_t)pidx * N;
    const int w0 = wv8(tid);
    double v[8];
    if (!INV) {
        uint64_t *out = data + off + w0;
        double tw3[7];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint64_t x = in[tid + 512 * k];
            v[k] = part ? b2d(x) : reduce_c(u2d(x), m);
        }
        load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
        tile_forward8(v, s, tws, tw3, tid, tile, logN1, W, N, m, [] {});
#pragma unroll
        for (int k = 0; k < 8; k++) out[64 * k] = d2u(corr(reduce_c(s[pad8(w0) + 72 * k], m), m));
    } else {
        uint64_t *out = data + off + tid;
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = reduce_c(u2d(in[w0 + 64 * k]), m);
        tile_inverse8(v, s, tid, tile, logN1, W, N, m);
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = part ? d2b(v[k]) : d2u(corr(mul_lazy(v[k], pi.ninv, m), m));
    }
}

// Rings of one tile (N = 4096) have no column pass, and their launches are a few blocks each:
// what bounds them is the chain of launches, so the basis conversion runs inside the kernels
// that transform its result.  v = words tid + 512 k of sum_a x_a hat[a n_out] mod t, centred: x_a
// the canonical words of limb a of `in` ([m][N], scaled by launch_intt_tiles), m <= 8.
__device__ __forceinline__ void tile_convert(double v[8], const uint64_t *in, int m, const double *hat, int n_out,
                                             Mod mo, int tid)
{
    constexpr int kA = 4;  // limbs requested at once
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = 0.0;
#pragma unroll 1
    for (int a = 0; a < m; a += kA) {
        uint64_t x[kA][8];
        double h[kA];
#pragma unroll
        for (int i = 0; i < kA; i++) {
            const int ai = min(a + i, m - 1);
            h[i] = a + i < m ? const_tab(hat)[ai * n_out] : 0.0;
#pragma unroll
            for (int k = 0; k < 8; k++) x[i][k] = in[(size_t)ai * kT + tid + 512 * k];
        }
#pragma unroll
        for (int i = 0; i < kA; i++) {
            if (a + i >= m) break;
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] += mul_lazy(u2d(x[i][k]), h[i], mo);  // 8 products within 7/8 t
        }
    }
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = reduce_c(v[k], mo);
}

// Requests the words of step q = z ND + j of a key inner product (job z, digit j) of one
// tile into LDS (xb, in memory order): the extended digit's tile ([ND][ne][N], as it came out
// of its column pass), or for the job's own limb the tile that X -> X^g reads (it moves whole
// tiles).  Straight to LDS, so no registers are held while they are under way: 16 bytes per
// lane, or 4 where ANY8 allows a polynomial of the caller's, only known to be 8-byte aligned,
// to start at an odd word (the digits and summed jobs' polynomials lie in the library's
// scratch, whole limbs from its start).
template <int ND, bool ANY8>
__device__ __forceinline__ void ip_request_x(const KeyJobs &kj, const IpRow &r, int q, int tile, int tid, int logN,
                                             double *xb)
{
    using lds = __attribute__((address_space(3))) void *;
    const size_t N = (size_t)1 << logN;
    const int z = q / ND, j = q - z * ND;
    const uint64_t *p = j == r.own ? kj.d[z] + r.t * N + (galois_src2(tile * kT, kj.g[z], logN) & ~(kT - 1))
                                   : kj.ext[z] + (j * r.ne + r.t) * N + tile * kT;
    const auto rs = buf_rsrc(p, 8u * kT);
    const uint32_t c0 = 4096u * __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    if (!ANY8 || ((uintptr_t)p & 15) == 0) {
#pragma unroll
        for (int i = 0; i < 4; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds)(xb + (c0 + 1024u * i) / 8u), 16, 16u * lane,
                                                     c0 + 1024u * i, 0, 0);
    } else {
#pragma unroll 1
        for (int i = 0; i < 16; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds)(xb + (c0 + 256u * i) / 8u), 4, 4u * lane, c0 + 256u * i,
                                                     0, 0);
    }
}

// Key inner products fused with the forward tile pass of the extended digits (N >=
// 8192).  The key switch is of tau_g(d_z), g = kj.g[z]: at output limb t, digit j of
// job z is either the job's own limb d_z[t] read through X -> X^g (evaluation form) or
// the converted limb ext_z[j][t] of tau_g(d_z), which arrives with only its column
// pass applied: the block finishes that tile's transform in LDS and
// multiplies it by the key words at once, so extended digits are never stored in
// evaluation form.  Grid (outputs, N/4096, l+1+alpha-skip): grid row 0 is limb 0, row r > 0
// limb r + skip (skip = l - 1: only Q limbs 0 and l and the special primes, what a
// rescale followed by a drop to level 0 reads).  Output o =
// blockIdx.x, u_base + o 2 ne N, is (accumulate ? itself : 0) + the sum of the jobs o per ..
// (SUM; else job o alone): outputs vary fastest, so those sharing keys read each key tile
// close together in time.  After each job the
// running sums take at most ND <= 4 lazy terms on a reduced value.
// A block works through its (job, digit) steps one after another, and both the memory
// stream (32 KB of digit and 64 KB of key words a step) and the transform take most of a
// step, so they have to overlap: the b half of a step's key words is requested before its
// transform, the next step's digit words, straight to LDS, as soon as this step's have left
// it.  8 words per thread leave room for that in 128 registers (4 waves per SIMD, two blocks
// per CU by LDS), but not for the a half, which is requested after the transform (before it:
// 18 registers spilled, 259 us); with 16 words per thread at 2 waves per SIMD it spills.  7 giant steps at level 23 of N =
// 2^16 (704 MB of keys, 352 MB of digits): 258 us with 256 threads and neither request
// ahead, 236 this way, when the memory stream alone takes 228; one key switch at level 20
// 48 and 39 us.  Non-temporal key words and digits: 216 and 33 us.
template <int ND, bool SUM, bool NT>
__global__ __launch_bounds__(kNT8, 4) void k_ntt_ip(KeyJobs kj, int per, uint64_t *u_base, int accumulate, int level,
                                                 int L, int alpha, int nq, const double *tw, const PrimeInfo *info,
                                                 int logN, uint64_t *pout, const double *itw, int skip)
{
    __shared__ double s[kT + kT / 8];
    __shared__ __align__(16) double xb[kT];
    __shared__ double tws[kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12;
    const int t = blockIdx.z == 0 ? 0 : (int)blockIdx.z + skip, tile = blockIdx.y, tid = threadIdx.x;
    const int pidx = t <= level ? t : nq + (t - level - 1);
    const Mod m = info[pidx].m;
    const double *W = tw + (size_t)pidx * N;
    const IpRow r = ip_row(t, level, L, alpha);
    const uint32_t t0 = (uint32_t)tile * kT;
    const int wl = wv8(tid);
    double *sw = s + pad8(wl);
    const size_t w0 = t0 + wl;
    const int z0 = SUM ? (int)blockIdx.x * per : (int)blockIdx.x, z1 = z0 + (SUM ? per : 1);
    uint64_t *u = u_base + (size_t)blockIdx.x * 2 * r.ne * N;
    const size_t o0 = r.t * N + w0, o1 = (r.ne + r.t) * N + w0;
    const int q0 = z0 * ND, q1 = z1 * ND;
    double tw3[7], a0[8], a1[8];
    load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
    ip_request_x<ND, !SUM>(kj, r, q0, tile, tid, logN, xb);
    if (accumulate) {
#pragma unroll
        for (int k = 0; k < 8; k++) a0[k] = u2d(u[o0 + 64 * k]), a1[k] = u2d(u[o1 + 64 * k]);
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++) a0[k] = 0.0, a1[k] = 0.0;
    }
#pragma unroll 1
    for (int q = q0; q < q1; q++) {
        const int z = q / ND, j = q - z * ND;
        // key [ND][2][nk][N]: words of row kl of digit j, b half then a half
        const auto key = buf_rsrc(kj.key[z], 8u * (uint32_t)(2 * ND * r.nk) * (uint32_t)N);
        const uint32_t vb = 8u * ((uint32_t)(j * 2 * r.nk + r.kl) * (uint32_t)N + (uint32_t)w0),
                       va = vb + 8u * (uint32_t)(r.nk * N);
        uint64_t kb[8], ka[8];
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's words of step q are in xb
        __syncthreads();                     // every wave's are, and the previous step's have been read out of s
        const bool own = j == r.own;
        double x[8];
        if (own) {  // these words are the job's own limb's
            const uint64_t *xu = (const uint64_t *)xb;
            const uint32_t g = kj.g[z], gb = gal_base((int)w0, g, logN);
#pragma unroll
            for (int k = 0; k < 8; k++) x[k] = u2d(xu[gal_at(gb, 64 * k, g, logN) & (kT - 1)]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) x[k] = xb[tid + 512 * k];
        }
#pragma unroll
        for (int k = 0; k < 8; k++) kb[k] = buf_ld<NT>(key, vb, 512u * k);
        auto next = [&]() {
            if (q + 1 < q1) ip_request_x<ND, !SUM>(kj, r, q + 1, tile, tid, logN, xb);
        };
        if (own) {
#pragma unroll
            for (int k = 0; k < 8; k++) sw[72 * k] = x[k];  // read back by this thread alone
            __syncthreads();
            next();
        } else {
            tile_forward8(x, s, tws, tw3, tid, tile, logN1, W, N, m, next);
        }
#pragma unroll
        for (int k = 0; k < 8; k++) ka[k] = buf_ld<NT>(key, va, 512u * k);
#pragma unroll
        for (int k = 0; k < 8; k++) {  // |x| < 2.2 t: products within 1.33 t, at most 4 on a centred sum
            const double xv = sw[72 * k];
            a0[k] += mul_lazy(xv, u2d(kb[k]), m);
            a1[k] += mul_lazy(xv, u2d(ka[k]), m);
        }
        if (j == ND - 1) reduce8(a0, m), reduce8(a1, m);
    }
    if (pout && t > level) {  // special-prime rows: on to ModDown's inverse transform
        uint64_t *out = pout + ((size_t)2 * blockIdx.x * alpha + (t - level - 1)) * N + t0 + tid;
        const double *iW = itw + (size_t)pidx * N;
        tile_inverse8(a0, s, tid, tile, logN1, iW, N, m);
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = d2b(a0[k]);
        __syncthreads();
        tile_inverse8(a1, s, tid, tile, logN1, iW, N, m);
        out += (size_t)alpha * N;
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = d2b(a1[k]);
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        u[o0 + 64 * k] = d2u(corr(a0[k], m));
        u[o1 + 64 * k] = d2u(corr(a1[k], m));
    }
}

// Key inner products on the ring of one tile (N = 4096).  One compute unit takes 1.6 us for
// one tile's transform alone, so every (job, limb, digit) is a block of its own: k_conv_ip
// converts the digit to its limb (kj.ext[z]: the [l+1][N] words of tau_g(d_z), canonical and
// scaled; the own limb is d_z[t] read through X -> X^g), transforms it and multiplies it by
// both key halves, into part [job][digit][2][ne][N] (lazy FP64 words); k_ip_reduce adds the
// products up, special-prime rows on through ModDown's inverse transform.  grid (jobs, ne, digits).
// A rotation's key switch is 4 launches this way.  What bounds it is their round trips to memory
// (about 2 us each from a cold L2, a block alone on its compute unit): 512 threads of 8 words,
// everything a block reads requested at once.  One rotation at level 7 (4 digits): 29.3 us; 47.8
// with the general kernels (8 launches), 45 with k_ntt_ip, which works through the digits one
// after another, 59 with 256 threads of 16 words.  CoeffToSlot with lazy giant steps (28 of them
// summed): a step 373 us, 525 with the general kernels, 662 with k_ntt_ip.
struct IpTiles {
    const double *hat[4];  // digit j's conversion table [m_j][n_out_j]
};
__global__ __launch_bounds__(kNT8, 4) void k_conv_ip(KeyJobs kj, IpTiles it, uint64_t *part, int level, int L,
                                                     int alpha, int nq, const double *tw, const PrimeInfo *info)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    constexpr int logN = 12;
    const int z = blockIdx.x, t = blockIdx.y, j = blockIdx.z, tid = threadIdx.x, w0 = wv8(tid);
    const int pidx = t <= level ? t : nq + (t - level - 1);
    const IpRow r = ip_row(t, level, L, alpha);
    const double *W = tw + (size_t)pidx * kT;
    double v[8], tw3[7];
    const uint64_t *kp = kj.key[z] + ((size_t)j * 2 * r.nk + r.kl) * kT + w0, *kq = kp + r.nk * kT;
    uint64_t kb[8], ka[8];
#pragma unroll
    for (int k = 0; k < 8; k++) kb[k] = kp[64 * k], ka[k] = kq[64 * k];
    const Mod m = info[pidx].m;
    if (j == r.own) {
        const uint64_t *d = kj.d[z] + (size_t)t * kT;
        const uint32_t g = kj.g[z], gb = gal_base(w0, g, logN);
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = u2d(d[gal_at(gb, 64 * k, g, logN)]);
    } else {
        const int a0 = j * alpha, mj = min(alpha, level + 1 - a0);
        load_twiddles8(tws, tw3, W, 0, 0, kT, tid);
        tile_convert(v, kj.ext[z] + (size_t)a0 * kT, mj, it.hat[j] + (t < a0 ? t : t - mj), level + 1 + alpha - mj,
                        m, tid);
        tile_forward8(v, s, tws, tw3, tid, 0, 0, W, kT, m, [] {});
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = s[pad8(wv8(tid)) + 72 * k];
    }
    uint64_t *o = part + (((size_t)z * gridDim.z + j) * 2 * r.ne + t) * kT + w0;
#pragma unroll
    for (int k = 0; k < 8; k++) {  // |v| < 2.2 t: within 1.33 t
        o[64 * k] = d2b(mul_lazy(v[k], u2d(kb[k]), m));
        o[r.ne * kT + 64 * k] = d2b(mul_lazy(v[k], u2d(ka[k]), m));
    }
}

// u_z = (accumulate ? u_z : 0) + the sum of n parts (n = digits, times the jobs where one sum
// is wanted); with pout the special-prime rows go through their inverse transform to row
// (2 z + p) alpha + a of pout instead, canonical and scaled.  grid (sums, 2 ne).
__global__ __launch_bounds__(kNT8, 4) void k_ip_reduce(const uint64_t *part, int n, uint64_t *u_base, int accumulate,
                                                    int level, int alpha, int nq, const PrimeInfo *info,
                                                    uint64_t *pout, const double *itw, const double *scale)
{
    __shared__ double s[kT + kT / 8];
    const int ne = level + 1 + alpha, z = blockIdx.x, row = blockIdx.y, p = row >= ne, t = row - p * ne;
    const int pidx = t <= level ? t : nq + (t - level - 1), tid = threadIdx.x;
    const size_t o = (size_t)row * kT + wv8(tid), stride = (size_t)2 * ne * kT;
    const uint64_t *in = part + (size_t)z * n * stride + o;
    uint64_t *u = u_base + z * stride + o;
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = accumulate ? u2d(u[64 * k]) : 0.0;
    const Mod m = info[pidx].m;
#pragma unroll 1
    for (int i = 0; i < n; i += 4) {  // 4 parts requested at once
        uint64_t x[4][8];
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int k = 0; k < 8; k++) x[q][k] = in[min(i + q, n - 1) * stride + 64 * k];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            if (i + q >= n) break;
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] += b2d(x[q][k]);
        }
        reduce8(v, m);  // below t + 4 1.33 t before
    }
    if (!pout || t <= level) {
#pragma unroll
        for (int k = 0; k < 8; k++) u[64 * k] = d2u(corr(v[k], m));
        return;
    }
    const double sc = scale[pidx];
    tile_inverse8(v, s, tid, 0, 0, itw + (size_t)pidx * kT, kT, m);
    uint64_t *out = pout + ((size_t)(2 * z + p) * alpha + (t - level - 1)) * kT + tid;
#pragma unroll
    for (int k = 0; k < 8; k++) out[512 * k] = d2u(corr(mul_lazy(v[k], sc, m), m));
}

// The inverse transform of the ring of one tile, read through X -> X^gt.g[off / L1] when L1 > 0.
// scale: canonical words times the prime's factor, for tile_convert; else FP64 words without
// their N^-1, as the tile pass of a larger ring.  grid (limbs).
__global__ __launch_bounds__(kNT8) void k_intt_tile(uint64_t *data, const uint64_t *src, LimbTab lt, GalTab gt, int L1,
                                                    const double *scale, const double *itw, const PrimeInfo *info)
{
    __shared__ double s[kT + kT / 8];
    constexpr int logN = 12;
    const int limb = blockIdx.x, pidx = lt.pidx[limb], tid = threadIdx.x, w0 = wv8(tid);
    const Mod m = info[pidx].m;
    const uint64_t *in = src ? src + (size_t)lt.soff[limb] * kT : data + (size_t)lt.off[limb] * kT;
    const uint32_t g = L1 ? gt.g[lt.off[limb] / L1] : 1u, gb = gal_base(w0, g, logN);
    const double f = scale ? scale[pidx] : 0.0;
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = reduce_c(u2d(in[gal_at(gb, 64 * k, g, logN)]), m);
    tile_inverse8(v, s, tid, 0, 0, itw + (size_t)pidx * kT, kT, m);
    uint64_t *out = data + (size_t)lt.off[limb] * kT + tid;
#pragma unroll
    for (int k = 0; k < 8; k++) out[512 * k] = scale ? d2u(corr(mul_lazy(v[k], f, m), m)) : d2b(v[k]);
}

// Conversion and transform on the ring of one tile: limb o of digit j of job z into jp.out,
// evaluation form (inputs canonical and scaled).  grid (jobs nd, targets).
__global__ __launch_bounds__(kNT8, 4) void k_conv_tile(BconvShared sh, BconvPtrs jp, const double *tw,
                                                       const PrimeInfo *info)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    const int z = blockIdx.x / sh.nd, j = blockIdx.x % sh.nd, o = blockIdx.y, tid = threadIdx.x;
    if (o >= sh.n_out[j]) return;
    const int pidx = sh.out_pidx[j][o];
    const double *W = tw + (size_t)pidx * kT;
    const Mod m = info[pidx].m;
    double v[8], tw3[7];
    load_twiddles8(tws, tw3, W, 0, 0, kT, tid);
    tile_convert(v, jp.in[z] + (size_t)sh.in_off0[j] * kT, sh.m[j], sh.hat[j] + o, sh.n_out[j], m, tid);
    tile_forward8(v, s, tws, tw3, tid, 0, 0, W, kT, m, [] {});
    uint64_t *out = jp.out[z] + (size_t)sh.out_off[j][o] * kT + wv8(tid);
#pragma unroll
    for (int k = 0; k < 8; k++) out[64 * k] = d2u(corr(reduce_c(s[pad8(wv8(tid)) + 72 * k], m), m));
}

// Decryption's inverse tile pass: limb i of c0 + c1 s (evaluation form, c1 at c0 + half N) enters
// the transform of that limb (a product and a sum per word on the way in instead of two
// passes over memory: 20.3 us instead of 39.1 for the whole call at level 20, N = 2^16, whose
// words take 6.6 us to read and write once).  grid (N/4096, limbs); output as k_ntt_tile<true>'s.
__global__ __launch_bounds__(kNT8) void k_ntt_tile_dec(uint64_t *data, const uint64_t *c0, size_t half, const uint64_t *sk,
                                                      const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    const int N = 1 << logN, logN1 = logN - 12, limb = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
    const PrimeInfo pi = info[limb];
    const Mod m = pi.m;
    const size_t o = (size_t)limb * N + (size_t)tile * kT, w0 = o + wv8(tid);
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; k++)  // within 1.88 t
        v[k] = reduce_c(mul_lazy(u2d(c0[half * N + w0 + 64 * k]), u2d(sk[w0 + 64 * k]), m) + u2d(c0[w0 + 64 * k]), m);
    tile_inverse8(v, s, tid, tile, logN1, tw + (size_t)limb * N, N, m);
    uint64_t *out = data + o + tid;
    if (logN1 == 0) {
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = d2u(corr(mul_lazy(v[k], pi.ninv, m), m));
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = d2b(v[k]);
    }
}

// Special-prime rows of the key inner products of n_jobs jobs whose digits are already
// extended and in evaluation form (job z: [ND][ne][N] at kj.ext[z], read through
// X -> X^g, g = kj.g[z]; a special prime is in no digit, so no own limb): each block
// sums one tile of one half's products over the digits and sends it through the first
// 12 stages of ModDown's inverse transform into row (2 z + p) alpha + a of pout, as
// launch_ntt_ip does with its special-prime rows.  The products never go to memory in
// evaluation form.  Grid (2 jobs, N/4096, alpha): blockIdx.x = 2 z + p, so the two
// halves of one tile, which read the same digit words, are dispatched together.  Key words
// are non-temporal here and in k_key_ip_md, for rotations of one ciphertext, each with a key
// of its own.  Block convs give one key to every input's job and would do a little better
// with cached loads (16 diagonals per block; non-temporal / cached): 8 x 1 blocks at levels 1
// and 23 of N = 2^16 412 / 403 us and 2.40 / 2.32 ms, 4 x 4 395 / 393 us and 2.82 / 2.80 ms; 2
// x 3 blocks of 20 babies at level 11 of N = 2^13 236 / 216 us.
template <int ND>
__global__ __launch_bounds__(kNT8, 4) void k_key_ip_ptile(KeyJobs kj, int level, int L, int alpha, int nq,
                                                         const PrimeInfo *info, int logN, uint64_t *pout,
                                                         const double *itw, const double *scale)
{
    __shared__ double s[kT + kT / 8];
    const int N = 1 << logN, logN1 = logN - 12;
    const int z = blockIdx.x >> 1, p = blockIdx.x & 1, tile = blockIdx.y, a = blockIdx.z, tid = threadIdx.x;
    const int t = level + 1 + a, pidx = nq + a;
    const Mod m = info[pidx].m;
    const IpRow r = ip_row(t, level, L, alpha);
    const uint32_t g = kj.g[z], w0 = (uint32_t)tile * kT + wv8(tid);
    const auto e = buf_rsrc(kj.ext[z], 8u * (uint32_t)(ND * r.ne) * (uint32_t)N);
    const auto key = buf_rsrc(kj.key[z], 8u * (uint32_t)(2 * ND * r.nk) * (uint32_t)N);
    const uint32_t gb = gal_base((int)w0, g, logN);
    uint32_t src[8];
#pragma unroll
    for (int k = 0; k < 8; k++) src[k] = 8u * (uint32_t)gal_at(gb, 64 * k, g, logN);
    double acc[8];
#pragma unroll
    for (int k = 0; k < 8; k++) acc[k] = 0.0;
#pragma unroll
    for (int j = 0; j < ND; j++) {
        const uint32_t xo = 8u * (uint32_t)((j * r.ne + r.t) * N),
                       vk = 8u * ((uint32_t)((j * 2 + p) * r.nk + r.kl) * (uint32_t)N + w0);
#pragma unroll
        for (int k = 0; k < 8; k++)
            acc[k] += mul_lazy(u2d(buf_ld(e, src[k], xo)), u2d(buf_ld<true>(key, vk, 512u * k)), m);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) acc[k] = reduce_c(acc[k], m);
    tile_inverse8(acc, s, tid, tile, logN1, itw + (size_t)pidx * N, N, m);
    uint64_t *out = pout + ((size_t)(2 * z + p) * alpha + a) * N + (size_t)tile * kT + tid;
    if (logN1 == 0) {  // as launch_intt_tiles with its scale
        const double sc = scale[pidx];
#pragma unroll
        for (int k = 0; k < 8; k++) out[512 * k] = d2u(corr(mul_lazy(acc[k], sc, m), m));
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) out[512 * k] = d2b(acc[k]);
}

// Inverse tile pass whose input limbs are read through X -> X^g (the automorphism of a
// key switch folded into ModUp's inverse transform): limb lt[b] is of job off / L1,
// read from src + soff N at the words the Galois element gt.g[job] moves to each
// position.  grid (N/4096, limbs).
__global__ __launch_bounds__(kNT8) void k_ntt_tile_gal(uint64_t *data, const uint64_t *src, LimbTab lt, GalTab gt,
                                                      int L1, const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    const int N = 1 << logN, logN1 = logN - 12;
    const int limb = blockIdx.y, pidx = lt.pidx[limb], tile = blockIdx.x, tid = threadIdx.x;
    const Mod m = info[pidx].m;
    const uint32_t g = gt.g[lt.off[limb] / L1];
    const uint64_t *in = src + (size_t)lt.soff[limb] * N;
    const size_t w0 = (size_t)tile * kT + tid;
    double v[8];
    const uint32_t gb = gal_base(tile * kT + wv8(tid), g, logN);
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = reduce_c(u2d(in[gal_at(gb, 64 * k, g, logN)]), m);
    tile_inverse8(v, s, tid, tile, logN1, tw + (size_t)pidx * N, N, m);
    uint64_t *out = data + (size_t)lt.off[limb] * N + w0;
#pragma unroll
    for (int k = 0; k < 8; k++) __builtin_nontemporal_store(d2b(v[k]), out + 512 * k);
}

// The first log2(N1) forward stages on one column of N1 words, canonical or centred (lazy,
// one centred reduction at the end: at most 4 stages).
template <int N1, typename P>
__device__ __forceinline__ void col_forward(double v[N1], P W, Mod m)
{
#pragma unroll
    for (int mm = 1; mm < N1; mm <<= 1) {
        const int tr = N1 / (2 * mm);
#pragma unroll
        for (int r = 0; r < N1; r++) {
            if (r & tr) continue;
            const double w = W[mm + r / (2 * tr)];
            const double U = v[r], V = mul_lazy(v[r + tr], w, m);
            v[r] = U + V;
            v[r + tr] = U - V;
        }
    }
#pragma unroll
    for (int r = 0; r < N1; r++) v[r] = reduce_c(v[r], m);
}

// The last log2(N1) inverse stages on one column of N1 centred words, uncorrected: at
// most 4 stages, 8 t in magnitude.
template <int N1, typename P>
__device__ __forceinline__ void col_inverse(double v[N1], P W, Mod m)
{
#pragma unroll
    for (int h = N1 / 2; h >= 1; h >>= 1) {
        const int tr = N1 / (2 * h);
#pragma unroll
        for (int r = 0; r < N1; r++) {
            if (r & tr) continue;
            const double w = W[h + r / (2 * tr)];
            const double U = v[r], V = v[r + tr];
            v[r] = U + V;
            v[r + tr] = mul_lazy(U - V, w, m);
        }
    }
}

// columns pass: first log2(N1) stages, one column of N1 words per thread.  grid (4096/256, limbs).
// The forward's results go to the tile pass as centred FP64 values; the inverse ends with
// the factor N^-1 and is canonical.
template <int N1, bool INV>
__global__ __launch_bounds__(kNT) void k_ntt_col(uint64_t *data, const uint64_t *src, LimbTab lt, const double *tw,
                                                 const PrimeInfo *info, int logN)
{
    const int N = 1 << logN;
    const int limb = blockIdx.y, pidx = lt.pidx[limb];
    const PrimeInfo pi = info[pidx];
    const Mod m = pi.m;
    const uint32_t cb = 8u * (blockIdx.x * kNT + threadIdx.x);
    uint64_t *outp = data + (size_t)lt.off[limb] * N;
    const auto in = buf_rsrc(src ? src + (size_t)lt.soff[limb] * N : outp, 8u * N);
    const auto out = buf_rsrc(outp, 8u * N);
    const double *W = tw + (size_t)pidx * N;
    double v[N1];
#pragma unroll
    for (int r = 0; r < N1; r++) {
        const uint64_t x = buf_ld(in, cb, 8u * r * kT);
        v[r] = INV ? b2d(x) : u2d(x);
    }
    if (!INV) {
        col_forward<N1>(v, W, m);
    } else {
        col_inverse<N1>(v, W, m);
#pragma unroll
        for (int r = 0; r < N1; r++) v[r] = reduce(mul_lazy(v[r], pi.ninv, m), m);
    }
#pragma unroll
    for (int r = 0; r < N1; r++) buf_st(out, cb, 8u * r * kT, INV ? d2u(v[r]) : d2b(v[r]));
}

// Basis conversion with the column passes on both sides of it.  Inputs are limbs after
// their inverse tile pass (FP64 words, centred); a block takes 64 columns (N1 words each at
// stride 4096) of (job, digit) blockIdx.z = job * nd + digit:
//   1. wave a < m finishes input limb a's inverse transform on its columns (the last
//      log2(N1) stages and the factor scale[prime] = N^-1 (D/q_a)^-1) and leaves the
//      canonical words in LDS;
//   2. each wave converts to one target after another, y_t = sum_a x_a (D/q_a) mod t, and
//      runs the target's first log2(N1) forward stages before anything is stored.
// So neither the inputs after their column pass nor the converted limbs before theirs go
// to memory.  One wave works on one prime at a time: its constants and twiddles are
// scalar loads.
//
// The sum is kept as an exact pair (S, L): S starts at 2^103 and takes each product
// rounded to a multiple of 2^51 (S stays below 2^104: 8 products below 2^100), L the
// rounding errors, d = S_old - S_new being exact and x h + d an integer below 2^50 in
// magnitude that one fma computes exactly; |L| <= 2^53.  4 operations per product instead
// of the 7 of a modular one, and one reduction at the end: S - 2^103 less its quotient
// times t leaves at most t/2 + 2^51 (the quotient's error times t is below 2^-52 times
// 2^103), plus L centred, an integer below 2^52.
// FP64 issue bounds it (7 giant steps at level 23, N = 2^16: 33 M converted words, about 63
// operations each, 94-98 us at 70% of the FP64 rate; the inverse column pass and a 7
// operation product as launches of their own took 27 + 104 us), latency a single key
// switch (25 us for its 3 digits; 6 + 24 us).  The block's LDS (64 KB at N1 = 16) allows
// two per CU, 4 waves per SIMD; 12 or 16 waves per block with 64 registers were slower.
// Grid (4096/64, target chunks of 8 tpw, jobs nd), wave w of chunk y taking targets
// (y tpw + i) 8 + w.
constexpr int kBcCols = 64, kBcWaves = 8;  // columns per block; waves, and input limbs at most

// step 2's sums for one column of one target: v[r] = sum_a x_a[r] hat[a n_out], centred; x_a's
// rows at x + (a N1 + r) kBcCols, zero for m <= a < MM.  No branch on m inside, so the LDS
// reads of one input are under way while another is being multiplied; all factors are
// loaded first (a scalar load in between would hold up every LDS read issued before it).
template <int MM, int N1>
__device__ __forceinline__ void bconv_sum(double v[N1], const double *x, ConstTab<double> hat, int m, int n_out, Mod mo)
{
    constexpr double kGrid = 10141204801825835211973625643008.0;  // 2^103
    constexpr int kR = N1 < 8 ? N1 : 8;  // rows at a time: 16 pairs at once would spill
    double h[MM];
#pragma unroll
    for (int a = 0; a < MM; a++) h[a] = hat[(a < m ? a : m - 1) * n_out];
#pragma unroll
    for (int r0 = 0; r0 < N1; r0 += kR) {
        double S[kR], L[kR];
#pragma unroll
        for (int r = 0; r < kR; r++) S[r] = kGrid, L[r] = 0.0;
#pragma unroll
        for (int a = 0; a < MM; a++)
#pragma unroll
            for (int r = 0; r < kR; r++) {
                const double xv = x[(a * N1 + r0 + r) * kBcCols], Sn = fma(xv, h[a], S[r]);
                L[r] += fma(xv, h[a], S[r] - Sn);
                S[r] = Sn;
            }
#pragma unroll
        for (int r = 0; r < kR; r++)
            v[r0 + r] = reduce_c(reduce_c(S[r] - kGrid, mo) + reduce_c(L[r], mo), mo);
    }
}

template <int N1>
__global__ __launch_bounds__(kBcCols * kBcWaves, 4) void k_bconv_col(BconvShared sh, BconvPtrs jp, const double *scale,
                                                                     const double *tw, const double *itw,
                                                                     const PrimeInfo *info, int logN, int tpw)
{
    __shared__ double xs[kBcWaves * N1 * kBcCols];
    const int N = 1 << logN;
    const int job = blockIdx.z / sh.nd, j = blockIdx.z % sh.nd;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kBcCols), lane = threadIdx.x % kBcCols;
    const int n_out = sh.n_out[j], m = sh.m[j], o0 = blockIdx.y * tpw * kBcWaves;
    if (o0 >= n_out) return;
    const uint32_t cb = 8u * (blockIdx.x * kBcCols + lane);
    double v[N1];
    if (w >= m) {  // bconv_sum reads 2, 4 or 8 inputs
#pragma unroll
        for (int r = 0; r < N1; r++) xs[(w * N1 + r) * kBcCols + lane] = 0.0;
    } else {
        const int pidx = sh.in_pidx[j][w];
        const Mod mi = info[pidx].m;
        const auto in = buf_rsrc(jp.in[job] + (size_t)(sh.in_off0[j] + w) * N, 8u * N);
#pragma unroll
        for (int r = 0; r < N1; r++) v[r] = b2d(buf_ld(in, cb, 8u * r * kT));
        col_inverse<N1>(v, itw + (size_t)pidx * N, mi);
        const double sc = scale[pidx];
#pragma unroll
        for (int r = 0; r < N1; r++) xs[(w * N1 + r) * kBcCols + lane] = reduce(mul_lazy(v[r], sc, mi), mi);
    }
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < tpw; i++) {
        const int o = o0 + i * kBcWaves + w;
        if (o >= n_out) return;
        const int pq = sh.out_pidx[j][o];
        const Mod mo{const_tab(info)[pq].m.t, const_tab(info)[pq].m.ti};
        const ConstTab<double> hat = const_tab(sh.hat[j]) + o;
        if (m > 4) bconv_sum<8, N1>(v, xs + lane, hat, m, n_out, mo);
        else if (m > 2) bconv_sum<4, N1>(v, xs + lane, hat, m, n_out, mo);
        else bconv_sum<2, N1>(v, xs + lane, hat, m, n_out, mo);
        col_forward<N1>(v, const_tab(tw) + (size_t)pq * N, mo);
        const auto out = buf_rsrc(jp.out[job] + (size_t)sh.out_off[j][o] * N, 8u * N);
#pragma unroll
        for (int r = 0; r < N1; r++) buf_st<true>(out, cb, 8u * r * kT, d2b(v[r]));
    }
}

// The words a ModDown combine adds, summed over the terms of MdSum: canonical, words w0 + 64 k of
// the limb at add (two terms requested at once).
__device__ __forceinline__ void md_sum(double av[8], const uint64_t *add, const MdSum &ms, int w0, int logN, Mod m)
{
#pragma unroll
    for (int k = 0; k < 8; k++) av[k] = 0.0;
#pragma unroll 1
    for (int q = 0; q < ms.n; q += 2) {
        const bool two = q + 1 < ms.n;
        const int q1 = two ? q + 1 : q;
        const uint32_t g0 = ms.g[q], g1 = ms.g[q1], b0 = gal_base(w0, g0, logN), b1 = gal_base(w0, g1, logN);
        uint64_t x[8], y[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            x[k] = add[ms.off[q] + gal_at(b0, 64 * k, g0, logN)];
            y[k] = add[ms.off[q1] + gal_at(b1, 64 * k, g1, logN)];
        }
#pragma unroll
        for (int k = 0; k < 8; k++) av[k] = add_mod(av[k], u2d(x[k]), m);
        if (two) {
#pragma unroll
            for (int k = 0; k < 8; k++) av[k] = add_mod(av[k], u2d(y[k]), m);
        }
    }
}

// ModDown of K key switches, finished inside the forward transform's tile pass.  The
// converted limbs conv [K][2][l+1][N] (coefficient form, column pass already applied)
// are transformed tile by tile and, instead of being stored, combined at once:
// out_z[p][i] = (u_z[p][i] - NTT(conv_z[p][i])) P^-1 (+ c0 of job z read through
// X -> X^g_add[z] for p = 0) (+ the previous out_z when acc; job 0 reads it from acc0
// instead when given), with u_z at u_base + z 2 ne N.  With last_out (one job), the
// blocks of the last limb also run the first 12 stages of its inverse transform on
// the words they wrote and store them at last_out + p N, ready for a rescale.
// grid (N/4096, 2 K (l+1)): limb w = (2 z + p)(l+1) + i.
template <bool CONJ>
__global__ __launch_bounds__(kNT8, 4) void k_ntt_tile_md(const uint64_t *conv, const uint64_t *u_base, MdJobs mj, int acc,
                                                     int level, int ne, const double *pinv, const double *pinvq,
                                                     const double *tw, const PrimeInfo *info, int logN, const uint64_t *acc0,
                                                     uint64_t *last_out, const double *itw, MdConj cj, int skip, int part, MdSum ms)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12, L1 = level + 1, L1e = L1 - skip;
    const int w = blockIdx.y, h = w / L1e, ie = w - h * L1e, i = ie == 0 ? 0 : ie + skip, z = h >> 1, p = h & 1;
    const int tile = blockIdx.x, tid = threadIdx.x;
    const Mod m = info[i].m;
    const double *W = tw + (size_t)i * N;
    const size_t t0 = (size_t)tile * kT;
    const uint64_t *in = conv + ((size_t)h * L1 + i) * N + t0;
    double v[8];
    const int wl = wv8(tid);
    const uint64_t *u = u_base + ((size_t)z * 2 * ne + (size_t)p * ne + i) * N + t0 + wl;
    uint64_t uv[8];  // requested before the transform, in which their latency passes: conv +
                      // CoeffToSlot at N = 2^14 750 -> 734 us
#pragma unroll
    for (int k = 0; k < 8; k++) uv[k] = u[64 * k];
    if (!part) {
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = reduce_c(u2d(in[tid + 512 * k]), m);
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = b2d(in[tid + 512 * k]);
    }
    const uint64_t *add = p == 0 ? mj.add[z] : nullptr;
    double tw3[7];
    load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
    uint64_t av[8];
#pragma unroll
    for (int k = 0; k < 8; k++) av[k] = 0;
    if (add) {
        add += (size_t)i * N;
        if (ms.n) {
            double sum[8];
            md_sum(sum, add, ms, (int)t0 + wl, logN, m);
#pragma unroll
            for (int k = 0; k < 8; k++) av[k] = d2u(sum[k]);
        } else {
            const uint32_t g = mj.g_add[z], gb = gal_base((int)t0 + wl, g, logN);
#pragma unroll
            for (int k = 0; k < 8; k++) av[k] = add[gal_at(gb, 64 * k, g, logN)];
        }
    }
    tile_forward8(v, s, tws, tw3, tid, tile, logN1, W, N, m, [] {});
    uint64_t *out = mj.out[z] + ((size_t)p * L1 + i) * N + t0;
    const uint64_t *prev = acc0 && z == 0 ? acc0 + ((size_t)p * L1 + i) * N + t0 : out;
    const double pv = pinv[i], pvq = pinvq[i];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int x = wl + 64 * k;
        // u in [0, t), s below 2.2 t
        double t = corr(mul_shoup_lazy(reduce_c(u2d(uv[k]) - s[pad8(wl) + 72 * k], m), pv, pvq, m) + u2d(av[k]), m);
        if (acc) t = add_mod(t, u2d(prev[x]), m);
        if (CONJ) {  // the real/imaginary split, as in k_conj_split
            const size_t o = ((size_t)p * L1 + i) * N + t0 + x;
            const double a = u2d(cj.x[o]);
            cj.re[o] = d2u(add_mod(a, t, m));
            double r = mul_canon(sub_mod(a, t, m), W[1], m);
            if ((brev_n((uint32_t)(t0 + x), logN) & 1u) == 0u) r = r == 0.0 ? 0.0 : m.t - r;
            cj.im[o] = d2u(r);
        } else {
            out[x] = d2u(t);
        }
    }
    if (last_out && i == level) {  // the rescale's inverse tile pass of this limb
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = reduce_c(u2d(out[wl + 64 * k]), m);  // this thread's own words
        tile_inverse8(v, s, tid, tile, logN1, itw + (size_t)i * N, N, m);
#pragma unroll
        for (int k = 0; k < 8; k++) last_out[(size_t)p * N + t0 + tid + 512 * k] = d2b(v[k]);
    }
}

// ModDown combine of K key switches from extended evaluation-form digits, with their
// key inner products on the Q limbs computed in the same block (the plain combine of
// k_ntt_tile_md, no accumulation): job z's half p at limb i is the sum over digits j of
// x_j read through X -> X^g (the own limb of kj.d[z] for i's digit, else the extended
// digit j at kj.ext[z]) times the key words, then (that - the converted special-prime
// part, after its tile pass) P^-1 plus add.  The products never go to memory.  Grid
// (N/4096, 2 K (l+1)).
template <int ND>
__global__ __launch_bounds__(kNT8, 4) void k_key_ip_md(const uint64_t *conv, KeyJobs kj, MdJobs mj, int level, int L,
                                                       int alpha, const double *pinv, const double *pinvq,
                                                       const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12, L1 = level + 1;
    const int w = blockIdx.y, h = w / L1, i = w - h * L1, z = h >> 1, p = h & 1;
    const int tile = blockIdx.x, tid = threadIdx.x;
    const Mod m = info[i].m;
    const size_t t0 = (size_t)tile * kT;
    const IpRow r = ip_row(i, level, L, alpha);
    const uint32_t g = kj.g[z], w0 = (uint32_t)t0 + wv8(tid);
    const auto e = buf_rsrc(kj.ext[z], 8u * (uint32_t)(ND * r.ne) * (uint32_t)N);
    const auto dd = buf_rsrc(kj.d[z] + (size_t)i * N, 8u * (uint32_t)N);
    const auto key = buf_rsrc(kj.key[z], 8u * (uint32_t)(2 * ND * r.nk) * (uint32_t)N);
    double a[8];
    {
        const uint32_t gb = gal_base((int)w0, g, logN);
        uint32_t src[8];
#pragma unroll
        for (int k = 0; k < 8; k++) src[k] = 8u * (uint32_t)gal_at(gb, 64 * k, g, logN);
#pragma unroll
        for (int k = 0; k < 8; k++) a[k] = 0.0;
#pragma unroll
        for (int j = 0; j < ND; j++) {
            const uint32_t vk = 8u * ((uint32_t)((j * 2 + p) * r.nk + r.kl) * (uint32_t)N + w0);
            if (j == r.own) {
#pragma unroll
                for (int k = 0; k < 8; k++)
                    a[k] += mul_lazy(u2d(buf_ld(dd, src[k], 0)), u2d(buf_ld<true>(key, vk, 512u * k)), m);
            } else {
                const uint32_t xo = 8u * (uint32_t)((j * r.ne + r.t) * N);
#pragma unroll
                for (int k = 0; k < 8; k++)
                    a[k] += mul_lazy(u2d(buf_ld(e, src[k], xo)), u2d(buf_ld<true>(key, vk, 512u * k)), m);
            }
        }
        reduce8(a, m);
    }
    const uint64_t *add = p == 0 ? mj.add[z] : nullptr;
    uint64_t av[8];
    if (add) {
        const uint32_t ga = mj.g_add[z], gb = gal_base((int)w0, ga, logN);
        add += (size_t)i * N;
#pragma unroll
        for (int k = 0; k < 8; k++) av[k] = add[gal_at(gb, 64 * k, ga, logN)];
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++) av[k] = 0;
    }
    const uint64_t *in = conv + ((size_t)h * L1 + i) * N + t0;
    const double *W = tw + (size_t)i * N;
    double v[8], tw3[7];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = b2d(in[tid + 512 * k]);
    load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
    tile_forward8(v, s, tws, tw3, tid, tile, logN1, W, N, m, [] {});
    uint64_t *out = mj.out[z] + ((size_t)p * L1 + i) * N + w0;
    const double pv = pinv[i], pvq = pinvq[i];
#pragma unroll
    for (int k = 0; k < 8; k++)  // a centred, s below 2.2 t
        out[64 * k] = d2u(corr(mul_shoup_lazy(reduce_c(a[k] - s[pad8(wv8(tid)) + 72 * k], m), pv, pvq, m) + u2d(av[k]), m));
}

// The ModDown combine on the ring of one tile, with its conversion: pc [2 K][alpha][N], the
// special-prime rows after their inverse transform, canonical and scaled.  ND = 0: as
// k_ntt_tile_md (u read, all its options; ND = -1: with MdSum); else the key inner products of ND extended
// evaluation-form digits, as k_key_ip_md.  8 words per thread, everything requested before the
// transform: a block alone on its compute unit waits for each round trip in full.  grid
// 2 K (l+1) blocks.
template <int ND>
__global__ __launch_bounds__(kNT8, ND > 0 ? 2 : 4) void k_md_tile(const uint64_t *pc, const double *hat, const uint64_t *u_base,
                                                     KeyJobs kj, MdJobs mj, int acc, const uint64_t *acc0, int level,
                                                     int L, int alpha, const double *pinv, const double *pinvq,
                                                     const double *tw, const PrimeInfo *info, uint64_t *last_out,
                                                     const double *itw, MdConj cj, MdSum ms)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    constexpr int logN = 12;
    const int L1 = level + 1, w = blockIdx.x, h = w / L1, i = w - h * L1, z = h >> 1, p = h & 1, tid = threadIdx.x;
    const int wl = wv8(tid);
    const IpRow r = ip_row(i, level, L, alpha);
    const Mod m = info[i].m;
    const double *W = tw + (size_t)i * kT;
    double a[8], v[8], tw3[7];
    load_twiddles8(tws, tw3, W, 0, 0, kT, tid);
    if (ND <= 0) {
        const uint64_t *u = u_base + ((size_t)h * r.ne + i) * kT + wl;
#pragma unroll
        for (int k = 0; k < 8; k++) a[k] = u2d(u[64 * k]);
    } else {
        const uint32_t g = kj.g[z], gb = gal_base(wl, g, logN);
        const uint64_t *key = kj.key[z] + ((size_t)p * r.nk + r.kl) * kT + wl;
#pragma unroll
        for (int k = 0; k < 8; k++) a[k] = 0.0;
#pragma unroll
        for (int j = 0; j < ND; j++) {
            const uint64_t *x = j == r.own ? kj.d[z] + (size_t)i * kT : kj.ext[z] + (j * r.ne + i) * kT;
#pragma unroll
            for (int k = 0; k < 8; k++)
                a[k] += mul_lazy(u2d(x[gal_at(gb, 64 * k, g, logN)]), u2d(key[(size_t)j * 2 * r.nk * kT + 64 * k]), m);
        }
        reduce8(a, m);
    }
    const uint64_t *add = p == 0 ? mj.add[z] : nullptr;
    uint64_t av[8];
#pragma unroll
    for (int k = 0; k < 8; k++) av[k] = 0;
    if (add) {
        add += (size_t)i * kT;
        if (ND < 0) {
            double sum[8];
            md_sum(sum, add, ms, wl, logN, m);
#pragma unroll
            for (int k = 0; k < 8; k++) av[k] = d2u(sum[k]);
        } else {
            const uint32_t g = mj.g_add[z], gb = gal_base(wl, g, logN);
#pragma unroll
            for (int k = 0; k < 8; k++) av[k] = add[gal_at(gb, 64 * k, g, logN)];
        }
    }
    tile_convert(v, pc + (size_t)h * alpha * kT, alpha, hat + i, L1, m, tid);
    tile_forward8(v, s, tws, tw3, tid, 0, 0, W, kT, m, [] {});
    const size_t o = ((size_t)p * L1 + i) * kT + wl;
    const uint64_t *prev = acc0 && z == 0 ? acc0 : mj.out[z];
    const double pv = pinv[i], pvq = pinvq[i];
#pragma unroll
    for (int k = 0; k < 8; k++) {  // a in [0, t) or centred, s below 2.2 t
        double t = corr(mul_shoup_lazy(reduce_c(a[k] - s[pad8(wl) + 72 * k], m), pv, pvq, m) + u2d(av[k]), m);
        if (acc) t = add_mod(t, u2d(prev[o + 64 * k]), m);
        if (cj.x) {  // the real/imaginary split, as in k_conj_split
            const double x = u2d(cj.x[o + 64 * k]);
            cj.re[o + 64 * k] = d2u(add_mod(x, t, m));
            double q = mul_canon(sub_mod(x, t, m), W[1], m);
            if ((brev_n((uint32_t)(wl + 64 * k), logN) & 1u) == 0u) q = q == 0.0 ? 0.0 : m.t - q;
            cj.im[o + 64 * k] = d2u(q);
        } else {
            mj.out[z][o + 64 * k] = d2u(t);
        }
        v[k] = reduce_c(t, m);
    }
    if (last_out && i == level) {  // the rescale's inverse tile pass of this limb
        tile_inverse8(v, s, tid, 0, 0, itw + (size_t)i * kT, kT, m);
#pragma unroll
        for (int k = 0; k < 8; k++) last_out[(size_t)p * kT + tid + 512 * k] = d2b(v[k]);
    }
}

// Rescale by q_l and ModRaise, fused into the lifted limbs' transform (N >= 4096).
// k_lift_col: one limb of each polynomial after its inverse tile pass (src [P][N], FP64
// words): its last log2(N1) inverse stages and N^-1, the centred lift into target limbs
// i < n_out and their forward column pass; thread = one column, `per` targets in turn;
// grid (4096/256, ceil(n_out / per), P).
template <int N1>
__global__ __launch_bounds__(kNT) void k_lift_col(const uint64_t *last, int src_pidx, int n_out, int per,
                                                  uint64_t *lifted, const double *tw, const double *itw,
                                                  const PrimeInfo *info, int logN)
{
    const int N = 1 << logN, z = blockIdx.z;
    const uint32_t cb = 8u * (blockIdx.x * kNT + threadIdx.x);
    const Mod ms = info[src_pidx].m;
    const double ninv = info[src_pidx].ninv;
    const auto src = buf_rsrc(last + (size_t)z * N, 8u * N);
    double x[N1];
#pragma unroll
    for (int r = 0; r < N1; r++) x[r] = b2d(buf_ld(src, cb, 8u * r * kT));
    col_inverse<N1>(x, itw + (size_t)src_pidx * N, ms);
    // centred exactly, |x| <= (t_l - 1)/2 < 2^49: after the first reduction |x/t| is below
    // 1/2 + 2/t, the second one's quotient error below 2^-53, and |x|/t at least 1/2t away
    // from 1/2
#pragma unroll
    for (int r = 0; r < N1; r++) x[r] = reduce_c(reduce_c(mul_lazy(x[r], ninv, ms), ms), ms);
    const int i1 = min(n_out, (int)(blockIdx.y + 1) * per);
#pragma unroll 1
    for (int i = blockIdx.y * per; i < i1; i++) {
        const Mod mt{const_tab(info)[i].m.t, const_tab(info)[i].m.ti};
        double v[N1];
#pragma unroll
        for (int r = 0; r < N1; r++) v[r] = reduce_c(x[r], mt);
        col_forward<N1>(v, const_tab(tw) + (size_t)i * N, mt);
        const auto dst = buf_rsrc(lifted + ((size_t)z * n_out + i) * N, 8u * N);
#pragma unroll
        for (int r = 0; r < N1; r++) buf_st(dst, cb, 8u * r * kT, d2b(v[r]));
    }
}

// k_ntt_tile_rs: the lifted limbs' tile pass with the rescale combine as its epilogue,
// out[z][i] = (in[z][i] - NTT(lift)[z][i]) q_l^-1 mod q_i; grid (N/4096, P n_out).
__global__ __launch_bounds__(kNT8) void k_ntt_tile_rs(const uint64_t *lifted, const uint64_t *in, uint64_t *out,
                                                     int level, int n_out, const double *qlinv, const double *qlinvq,
                                                     int nq, const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12;
    const int w = blockIdx.y, z = w / n_out, i = w - z * n_out;
    const int tile = blockIdx.x, tid = threadIdx.x;
    const Mod m = info[i].m;
    const size_t t0 = (size_t)tile * kT;
    const double *W = tw + (size_t)i * N;
    double tw3[7];
    load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
    const uint64_t *src = lifted + (size_t)w * N + t0;
    double v[8];
    if (logN1 == 0) {  // `lifted` is the last limbs after their inverse tile pass: lifted here
        const PrimeInfo pl = info[level];
        const uint64_t *last = lifted + (size_t)z * N;
#pragma unroll
        for (int k = 0; k < 8; k++)
            v[k] = reduce_c(reduce_c(reduce_c(mul_lazy(b2d(last[tid + 512 * k]), pl.ninv, pl.m), pl.m), pl.m), m);
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = b2d(src[tid + 512 * k]);
    }
    const uint64_t *a = in + ((size_t)z * (level + 1) + i) * N + t0 + wv8(tid);
    uint64_t av[8];  // requested before the transform, in which their latency passes: a
                      // mask's product and rescale at level 18, N = 2^16, 65 -> 61.6 us
#pragma unroll
    for (int k = 0; k < 8; k++) av[k] = a[64 * k];
    tile_forward8(v, s, tws, tw3, tid, tile, logN1, W, N, m, [] {});
    uint64_t *o = out + ((size_t)z * n_out + i) * N + t0;
    const double wl = qlinv[level * nq + i], wlq = qlinvq[level * nq + i];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int x = wv8(tid) + 64 * k;
        __builtin_nontemporal_store(d2u(corr(mul_shoup_lazy(reduce_c(u2d(av[k]) - s[pad8(wv8(tid)) + 72 * k], m), wl, wlq, m), m)), o + x);
    }
}

// Sums of rescaled terms (RsTerms).  Rescaling is linear modulo each remaining prime:
// sum_j w_j (k_j x_j - lift_j) q_l^-1, lift_j the centred last limb of k_j x_j, needs one forward
// transform, of sum_j w_j lift_j (an integer below 8 2^49), however many terms there are.  A
// baby-step sum of ModEval (7 terms, Re and Im packed, N = 2^16) is 3 launches instead of
// 36, a layer (activation and StoC1 included) 8.7 ms instead of 11.7.
// k_lift_sum: the terms' last limbs after their inverse tile pass (last [terms][P][N]),
// their last log2(N1) inverse stages with the factor N^-1 k_j, centred and summed, lifted
// into targets i < n_out with their forward column pass; grid as k_lift_col's.
template <int N1>
__global__ __launch_bounds__(kNT) void k_lift_sum(const uint64_t *last, RsTerms rt, int level, int n_polys, int n_out,
                                                  int per, uint64_t *lifted, const double *tw, const double *itw,
                                                  const PrimeInfo *info, int logN)
{
    const int N = 1 << logN, z = blockIdx.z;
    const uint32_t cb = 8u * (blockIdx.x * kNT + threadIdx.x);
    const Mod ms = info[level].m;
    double x[N1];
#pragma unroll
    for (int r = 0; r < N1; r++) x[r] = 0.0;
#pragma unroll 1
    for (int j = 0; j < rt.n; j++) {
        const auto src = buf_rsrc(last + ((size_t)j * n_polys + z) * N, 8u * N);
        double v[N1];
#pragma unroll
        for (int r = 0; r < N1; r++) v[r] = b2d(buf_ld(src, cb, 8u * r * kT));
        col_inverse<N1>(v, const_tab(itw) + (size_t)level * N, ms);
        const double kn = rt.kn[j], w = rt.w[j];
#pragma unroll
        for (int r = 0; r < N1; r++)  // centred exactly, as in k_lift_col
            x[r] = fma(w, reduce_c(reduce_c(mul_lazy(v[r], kn, ms), ms), ms), x[r]);
    }
    const int i1 = min(n_out, (int)(blockIdx.y + 1) * per);
#pragma unroll 1
    for (int i = blockIdx.y * per; i < i1; i++) {
        const Mod mt{const_tab(info)[i].m.t, const_tab(info)[i].m.ti};
        double v[N1];
#pragma unroll
        for (int r = 0; r < N1; r++) v[r] = reduce_c(x[r], mt);
        col_forward<N1>(v, const_tab(tw) + (size_t)i * N, mt);
        const auto dst = buf_rsrc(lifted + ((size_t)z * n_out + i) * N, 8u * N);
#pragma unroll
        for (int r = 0; r < N1; r++) buf_st(dst, cb, 8u * r * kT, d2b(v[r]));
    }
}

// k_ntt_tile_rsum: the lifted sums' tile pass with the combine as its epilogue,
// out[z][i] = (sum_j kw_j x_j[z][i] - NTT(lift)[z][i]) q_l^-1 + c + add; grid (N/4096, P n_out).
// The terms' lazy products stay within 8 7/8 t.
__global__ __launch_bounds__(kNT8) void k_ntt_tile_rsum(const uint64_t *lifted, RsTerms rt, uint64_t *out, int level,
                                                       int n_out, const double *qlinv, const double *qlinvq, int nq,
                                                       const double *tw, const PrimeInfo *info, int logN)
{
    __shared__ double s[kT + kT / 8];
    __shared__ double tws[kTw8R2];
    const int N = 1 << logN, logN1 = logN - 12;
    const int w = blockIdx.y, z = w / n_out, i = w - z * n_out;
    const int tile = blockIdx.x, tid = threadIdx.x, wl = wv8(tid);
    const Mod m = info[i].m;
    const size_t t0 = (size_t)tile * kT;
    const uint64_t *src = lifted + (size_t)w * N + t0;
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = b2d(src[tid + 512 * k]);
    const double *W = tw + (size_t)i * N;
    double tw3[7];
    load_twiddles8(tws, tw3, W, tile, logN1, N, tid);
    tile_forward8(v, s, tws, tw3, tid, tile, logN1, W, N, m, [] {});
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = -reduce_c(s[pad8(wl) + 72 * k], m);
#pragma unroll 1
    for (int j = 0; j < rt.n; j++) {
        const uint64_t *a = rt.src[j] + ((size_t)z * rt.stride[j] + i) * N + t0 + wl;
        const double kw = rt.kw[j][i];
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] += mul_lazy(u2d(a[64 * k]), kw, m);
    }
    uint64_t *o = out + (size_t)w * N + t0 + wl;
    const uint64_t *add = rt.add ? rt.add + (size_t)w * N + t0 + wl : nullptr;
    const double wi = qlinv[level * nq + i], wiq = qlinvq[level * nq + i], cc = z & 1 ? 0.0 : rt.c[i];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        double t = corr(mul_shoup_lazy(reduce_c(v[k], m), wi, wiq, m) + cc, m);
        if (add) t = add_mod(t, u2d(add[64 * k]), m);
        o[64 * k] = d2u(t);
    }
}

template <bool INV>
static hipError_t launch_cols(const nj_ctx *c, int kind, double bytes, int N1, dim3 grid, hipStream_t s,
                              uint64_t *data, const uint64_t *src, const LimbTab &lt, const double *tw,
                              const PrimeInfo *info, int logN)
{
    switch (N1) {
    case 2: return launch(c, kind, bytes, k_ntt_col<2, INV>, grid, dim3(kNT), s, data, src, lt, tw, info, logN);
    case 4: return launch(c, kind, bytes, k_ntt_col<4, INV>, grid, dim3(kNT), s, data, src, lt, tw, info, logN);
    case 8: return launch(c, kind, bytes, k_ntt_col<8, INV>, grid, dim3(kNT), s, data, src, lt, tw, info, logN);
    default: return launch(c, kind, bytes, k_ntt_col<16, INV>, grid, dim3(kNT), s, data, src, lt, tw, info, logN);
    }
}

// N >= 4096: forward = columns then tiles, inverse = tiles then columns.  src (optional)
// is read instead of data by the first pass (limb i at src + soff[i]*N).
hipError_t launch_ntt_fast(const nj_ctx *c, uint64_t *data, const uint64_t *src, const LimbTab &lt, bool inverse,
                           hipStream_t s)
{
    const int N = c->N, N1 = N / kT;
    const double *tw = inverse ? c->d_itw : c->d_tw;
    dim3 gt(N1, lt.n), gc(kT / kNT, lt.n);
    const double bytes = 16.0 * N * lt.n;  // each pass reads and writes every word once
    hipError_t e;
    if (!inverse) {
        if (N1 > 1) {
            e = launch_cols<false>(c, PROF_NTT_COL, bytes, N1, gc, s, data, src, lt, tw, c->d_info, c->log_n);
            if (e != hipSuccess) return e;
            src = nullptr;
        }
        return launch(c, PROF_NTT_TILE, bytes, k_ntt_tile<false>, gt, dim3(kNT8), s, data, src, lt, N1 > 1, tw, c->d_info,
                      c->log_n);
    }
    e = launch(c, PROF_NTT_TILE_INV, bytes, k_ntt_tile<true>, gt, dim3(kNT8), s, data, src, lt, N1 > 1, tw, c->d_info,
               c->log_n);
    if (e != hipSuccess || N1 == 1) return e;
    return launch_cols<true>(c, PROF_NTT_COL_INV, bytes, N1, gc, s, data, nullptr, lt, tw, c->d_info, c->log_n);
}

// c0 + c1 s of a level-`level` ciphertext in coefficient form (N >= 4096)
hipError_t launch_decrypt_fast(const nj_ctx *c, const uint64_t *ct, int level, uint64_t *out, hipStream_t s)
{
    const int N = c->N, N1 = N / kT, L1 = level + 1;
    if (N < kT) return hipErrorInvalidValue;
    hipError_t e = launch(c, PROF_NTT_TILE_INV, 32.0 * N * L1, k_ntt_tile_dec, dim3(N1, L1), dim3(kNT8), s, out, ct,
                          (size_t)L1, c->d_s, c->d_itw, c->d_info, c->log_n);
    if (e != hipSuccess || N1 == 1) return e;
    const LimbTab lt = limbs_q(level);
    return launch_cols<true>(c, PROF_NTT_COL_INV, 16.0 * N * L1, N1, dim3(kT / kNT, L1), s, out, nullptr, lt, c->d_itw,
                             c->d_info, c->log_n);
}

// Inverse tile pass alone, into data from src (N >= 4096): the basis conversion runs the
// column pass.  With gt, the input limbs are read through X -> X^g of their job (off / L1);
// with scale (N = 4096) canonical words times the prime's factor.
hipError_t launch_intt_tiles(const nj_ctx *c, uint64_t *data, const uint64_t *src, const LimbTab &lt, hipStream_t s,
                             const GalTab *gt, int L1, const double *scale)
{
    const int N = c->N, N1 = N / kT;
    if (N1 < 1 || (scale && N1 > 1) || (gt && (!src || L1 < 1))) return hipErrorInvalidValue;
    if (lt.n == 0) return hipSuccess;
    const double bytes = 16.0 * N * lt.n;
    if (N1 == 1)
        return launch(c, PROF_NTT_TILE_INV, bytes, k_intt_tile, dim3(lt.n), dim3(kNT8), s, data, src, lt,
                      gt ? *gt : GalTab{}, gt ? L1 : 0, scale, c->d_itw, c->d_info);
    return gt ? launch(c, PROF_NTT_TILE_INV, bytes, k_ntt_tile_gal, dim3(N1, lt.n), dim3(kNT8), s, data, src, lt, *gt,
                       L1, c->d_itw, c->d_info, c->log_n)
              : launch(c, PROF_NTT_TILE_INV, bytes, k_ntt_tile<true>, dim3(N1, lt.n), dim3(kNT8), s, data, src, lt,
                       1, c->d_itw, c->d_info, c->log_n);
}

// Centred lift of n_polys limbs after their inverse tile pass (prime src_pidx, at src + z N)
// into primes 0..n_out-1 with the column passes on both sides, into out [n_polys][n_out][N]
// (N >= 4096); the tile pass (launch_ntt_tiles, k_ntt_tile_rs) finishes the forward transform.
hipError_t launch_lift_col(const nj_ctx *c, const uint64_t *src, int src_pidx, int n_polys, int n_out, uint64_t *out,
                           hipStream_t s)
{
    const int N = c->N, N1 = N / kT;
    if (N1 < 1 || n_out < 1 || n_polys < 1) return hipErrorInvalidValue;
    // two targets share one inverse column pass: 1, 2, 4 and 8 each measured, mask and HMult
    // best at 1 and 2, a layer and a batch at 2 and 4 (12.59 / 12.50 / 12.52 / 12.68 ms a layer)
    const int per = 2;
    const dim3 g(kT / kNT, (n_out + per - 1) / per, n_polys);
    const double b = 8.0 * N * n_polys * (1 + n_out);
#define NJ_LC(NN)                                                                                                 \
    case NN:                                                                                                      \
        return launch(c, PROF_OTHER, b, k_lift_col<NN>, g, dim3(kNT), s, src, src_pidx, n_out, per, out, c->d_tw, \
                      c->d_itw, c->d_info, c->log_n);
    switch (N1) {
        NJ_LC(1) NJ_LC(2) NJ_LC(4) NJ_LC(8) NJ_LC(16)
    }
#undef NJ_LC
    return hipErrorInvalidValue;
}

// Rescale of P packed level-l polynomials (P = 2 per ciphertext; limbs 0..n_out-1 of
// each kept), N >= 4096: inverse tile pass of the last limbs read in place (into
// last [P][N]), lift fused with the column passes (into lifted [P][n_out][N], which may be
// out: each tile block reads its own lifted words before writing them), tile pass
// fused with the combine.  in must not alias out.
hipError_t launch_rescale_fused(const nj_ctx *c, int level, const uint64_t *in, uint64_t *out, int n_out,
                                uint64_t *last, uint64_t *lifted, hipStream_t s, int n_polys, bool last_tiled)
{
    const int N = c->N, N1 = N / kT;
    if (N1 < 1 || n_out < 1 || n_out > level || n_polys < 1 || n_polys > NJ_MAX_LIMBS) return hipErrorInvalidValue;
    LimbTab lt;
    lt.n = n_polys;
    for (int p = 0; p < n_polys; p++) lt.pidx[p] = level, lt.off[p] = p, lt.soff[p] = p * (level + 1) + level;
    // last_tiled: the last limbs' inverse tile pass already ran (into last)
    hipError_t e = last_tiled ? hipSuccess : launch_intt_tiles(c, last, in, lt, s);
    if (e == hipSuccess && N1 > 1) e = launch_lift_col(c, last, level, n_polys, n_out, lifted, s);
    if (N1 == 1) lifted = last;
    if (e != hipSuccess) return e;
    return launch(c, PROF_OTHER, 8.0 * N * n_polys * n_out * 4.0, k_ntt_tile_rs, dim3(N1, n_polys * n_out), dim3(kNT8),
                  s, lifted, in, out, level, n_out, c->d_qlinv, c->d_qlinvq, c->n_q, c->d_tw, c->d_info, c->log_n);
}

hipError_t launch_rescale_sum(const nj_ctx *c, int level, const RsTerms &rt, uint64_t *out, uint64_t *last,
                              int n_polys, hipStream_t s)
{
    const int N = c->N, N1 = N / kT, P = n_polys, n_out = level;
    if (N1 < 1 || level < 1 || level > 31 || rt.n < 1 || rt.n > NJ_MAX_TERMS || P < 1 || rt.n * P > NJ_MAX_LIMBS)
        return hipErrorInvalidValue;
    double wsum = 0;
    const uint64_t *base = rt.src[0];
    for (int j = 0; j < rt.n; j++) wsum += std::fabs(rt.w[j]), base = std::min(base, rt.src[j]);
    if (wsum > 8) return hipErrorInvalidValue;
    LimbTab lt;
    lt.n = 0;
    for (int j = 0; j < rt.n; j++)
        for (int z = 0; z < P; z++) {
            const size_t d = rt.src[j] - base;  // the terms live in one scratch buffer, whole limbs apart
            if (d % N || d / N > (size_t)1 << 30) return hipErrorInvalidValue;
            lt.pidx[lt.n] = level, lt.off[lt.n] = lt.n, lt.soff[lt.n] = (int)(d / N) + z * rt.stride[j] + level;
            lt.n++;
        }
    hipError_t e = launch_intt_tiles(c, last, base, lt, s);
    if (e != hipSuccess) return e;
    // the inverse column passes are repeated per target chunk: two chunks for many terms,
    // two targets at a time, as launch_lift_col, for one or two.  (For many terms it hardly
    // matters: a layer with 2 targets, 4 targets, a quarter of them, half of them or all of
    // them per block 8.637, 8.624, 8.592, 8.605 and 8.615 ms.)
    const int per = rt.n > 2 ? (n_out + 1) / 2 : 2;
    const dim3 g(kT / kNT, (n_out + per - 1) / per, P);
    const double b = 8.0 * N * P * (rt.n + n_out);
#define NJ_LS(NN)                                                                                                  \
    case NN:                                                                                                       \
        e = launch(c, PROF_OTHER, b, k_lift_sum<NN>, g, dim3(kNT), s, last, rt, level, P, n_out, per, out, c->d_tw, \
                   c->d_itw, c->d_info, c->log_n);                                                                 \
        break;
    switch (N1) {
        NJ_LS(1) NJ_LS(2) NJ_LS(4) NJ_LS(8) NJ_LS(16)
    default: return hipErrorInvalidValue;
    }
#undef NJ_LS
    if (e != hipSuccess) return e;
    return launch(c, PROF_OTHER, 8.0 * N * P * n_out * (2.0 + rt.n + (rt.add ? 1 : 0)), k_ntt_tile_rsum,
                  dim3(N1, P * n_out), dim3(kNT8), s, out, rt, out, level, n_out, c->d_qlinv, c->d_qlinvq, c->n_q,
                  c->d_tw, c->d_info, c->log_n);
}

// Forward tile pass alone (the column pass already applied), N >= 4096.
hipError_t launch_ntt_tiles(const nj_ctx *c, uint64_t *data, const LimbTab &lt, hipStream_t s)
{
    const int N = c->N, N1 = N / kT;
    if (N1 < 1) return hipErrorInvalidValue;
    if (lt.n == 0) return hipSuccess;
    return launch(c, PROF_NTT_TILE, 16.0 * N * lt.n, k_ntt_tile<false>, dim3(N1, lt.n), dim3(kNT8), s, data, nullptr,
                  lt, 1, c->d_tw, c->d_info, c->log_n);
}

// Basis conversion of n_jobs (job, digit) pairs with the column passes on both sides
// (inputs after their inverse tile pass; scale: [n_primes] factor of each input's inverse
// transform), N >= 4096, at most 8 input limbs per digit.  N = 4096: the whole forward
// transform, inputs canonical and scaled.
hipError_t launch_bconv_col(const nj_ctx *c, const BconvShared &sh, const BconvPtrs &jp, int n_jobs,
                            const double *scale, hipStream_t s)
{
    const int N = c->N, N1 = N / kT;
    if (N1 < 1 || n_jobs == 0) return N1 < 1 ? hipErrorInvalidValue : hipSuccess;
    int max_out = 0, mmax = 0;
    double bytes = 0;
    for (int j = 0; j < sh.nd; j++) {
        max_out = std::max(max_out, sh.n_out[j]);
        mmax = std::max(mmax, sh.m[j]);
        bytes += 8.0 * N * (sh.m[j] + sh.n_out[j]) * n_jobs;
    }
    if (mmax > kBcWaves) return hipErrorInvalidValue;
    if (N1 == 1)  // inputs scaled by their inverse transform; outputs in evaluation form
        return launch(c, PROF_BCONV, bytes, k_conv_tile, dim3(n_jobs * sh.nd, max_out), dim3(kNT8), s, sh, jp, c->d_tw,
                      c->d_info);
    // targets per wave: step 1 is half a target's work, so a block takes all targets once
    // there are blocks enough to fill the chip (256 CUs, two blocks each by their LDS: 8
    // digits of one size), and one per wave below that.  N = 2^16, 24 targets: 21 digits
    // 98 us against 107 with one per wave, one key switch's 3 digits 25 us against 31 with 3
    const int chunks = (max_out + kBcWaves - 1) / kBcWaves, wide = kT / kBcCols * n_jobs * sh.nd;
    const int tpw = wide >= 512 ? chunks : 1;
    const dim3 grid(kT / kBcCols, (chunks + tpw - 1) / tpw, n_jobs * sh.nd), blk(kBcCols * kBcWaves);
#define NJ_BC(NN)                                                                                                 \
    case NN:                                                                                                      \
        return launch(c, PROF_BCONV, bytes, k_bconv_col<NN>, grid, blk, s, sh, jp, scale, c->d_tw, c->d_itw,      \
                      c->d_info, c->log_n, tpw);
    switch (N1) {
        NJ_BC(2) NJ_BC(4) NJ_BC(8) NJ_BC(16)
    }
#undef NJ_BC
    return hipErrorInvalidValue;
}

// ModDown combine of K jobs fused into the forward transform of their converted
// limbs (N >= 4096; cols_done: the column pass was already applied, N = 4096: conv is the
// special-prime rows, converted here); same results
// as the transform followed by the combine.
hipError_t launch_ntt_moddown(const nj_ctx *c, int level, int K, uint64_t *conv, const uint64_t *u_base,
                              const MdJobs &mj, int acc, int cols_done, hipStream_t s, const uint64_t *acc0,
                              uint64_t *last_out, const MdConj *conj, int skip, const MdSum *ms)
{
    const int N = c->N, N1 = N / kT, L1 = level + 1, n = 2 * K * (L1 - skip);
    if (N < kT || K < 1 || K > NJ_MAX_JOBS || ((last_out || conj) && K != 1) || (last_out && conj) || skip < 0 ||
        skip > std::max(0, level - 1) || (skip && (!cols_done || last_out || conj)))
        return hipErrorInvalidValue;
    MdConj cj{nullptr, nullptr, nullptr};
    if (conj) cj = *conj;
    MdSum msum;
    msum.n = 0;
    if (ms) msum = *ms;
    if (msum.n < 0 || msum.n > NJ_MAX_GIANT) return hipErrorInvalidValue;
    if (N1 == 1 && cols_done) {
        if (skip || c->alpha > 8) return hipErrorInvalidValue;
        const double b = 8.0 * N * (n * 3.0 + K * L1 * std::max(1, msum.n) + (acc ? n : 0));
#define NJ_MDT(ND)                                                                                                   \
    launch(c, PROF_NTT_MD, b, k_md_tile<ND>, dim3(n), dim3(kNT8), s, conv, c->moddown[level].hat, u_base, KeyJobs{}, \
           mj, acc, acc0, level, c->L, c->alpha, c->d_pinv, c->d_pinvq, c->d_tw, c->d_info, last_out, c->d_itw, cj,  \
           msum)
        return msum.n ? NJ_MDT(-1) : NJ_MDT(0);
#undef NJ_MDT
    }
    if (N1 > 1 && !cols_done) {
        LimbTab lt;
        for (int b = 0; b < n; b += NJ_MAX_LIMBS) {
            lt.n = std::min(NJ_MAX_LIMBS, n - b);
            for (int j = 0; j < lt.n; j++) lt.pidx[j] = (b + j) % L1, lt.off[j] = b + j, lt.soff[j] = 0;
            hipError_t e = launch_cols<false>(c, PROF_NTT_COL, 16.0 * N * lt.n, N1, dim3(kT / kNT, lt.n), s, conv,
                                              nullptr, lt, c->d_tw, c->d_info, c->log_n);
            if (e != hipSuccess) return e;
        }
    }
    const double bytes = 8.0 * N * (n * 3.0 + K * (L1 - skip) * std::max(1, msum.n) + (acc ? n : 0));
    if (conj)
        return launch(c, PROF_NTT_MD, bytes, k_ntt_tile_md<true>, dim3(N1, n), dim3(kNT8), s, conv, u_base, mj, acc,
                      level, L1 + c->alpha, c->d_pinv, c->d_pinvq, c->d_tw, c->d_info, c->log_n, acc0, last_out, c->d_itw, cj, skip,
                      N1 > 1, msum);
    return launch(c, PROF_NTT_MD, bytes, k_ntt_tile_md<false>, dim3(N1, n), dim3(kNT8), s, conv, u_base, mj, acc, level,
                  L1 + c->alpha, c->d_pinv, c->d_pinvq, c->d_tw, c->d_info, c->log_n, acc0, last_out, c->d_itw, cj, skip,
                      N1 > 1, msum);
}

// The plain ModDown combine of K key switches (converted limbs column-passed) with their
// Q-limb key inner products computed inside it from extended evaluation-form digits
// (N >= 4096, 1..4 digits).
hipError_t launch_key_ip_moddown(const nj_ctx *c, int level, int K, const uint64_t *conv, const KeyJobs &kj,
                                 const MdJobs &mj, hipStream_t s)
{
    const int N = c->N, N1 = N / kT, L1 = level + 1, n = 2 * K * L1, nd = n_digits(c, level);
    if (N1 < 1 || K < 1 || K > NJ_MAX_JOBS || nd < 1 || nd > 4) return hipErrorInvalidValue;
    const double bytes = 8.0 * N * (n * (2.0 * nd + 2.0) + K * L1);
#define NJ_IPMD(ND)                                                                                                \
    case ND:                                                                                                       \
        if (N1 == 1)                                                                                               \
            return launch(c, PROF_KEYIP, bytes, k_md_tile<ND>, dim3(n), dim3(kNT8), s, conv, c->moddown[level].hat, \
                          nullptr, kj, mj, 0, nullptr, level, c->L, c->alpha, c->d_pinv, c->d_pinvq, c->d_tw,      \
                          c->d_info, nullptr, c->d_itw, MdConj{nullptr, nullptr, nullptr}, MdSum{});               \
        return launch(c, PROF_KEYIP, bytes, k_key_ip_md<ND>, dim3(N1, n), dim3(kNT8), s, conv, kj, mj, level, c->L, \
                      c->alpha, c->d_pinv, c->d_pinvq, c->d_tw, c->d_info, c->log_n);
    switch (nd) {
        NJ_IPMD(1) NJ_IPMD(2) NJ_IPMD(3) NJ_IPMD(4)
    }
#undef NJ_IPMD
    return hipErrorInvalidValue;
}

// Key inner products of n_jobs jobs (digits of tau_g(d) column-passed only, own limbs
// read from d through X -> X^g) fused with the digits' tile pass; output o sums the jobs
// o per .. o per + per - 1; accumulate: added to the output's previous value.
hipError_t launch_ntt_ip(const nj_ctx *c, int level, const KeyJobs &kj, int n_jobs, uint64_t *u, int per,
                         int accumulate, hipStream_t s, uint64_t *pout, int skip, uint64_t *part)
{
    const int N = c->N, N1 = N / kT, nd = n_digits(c, level), ne = level + 1 + c->alpha;
    if (N1 < 1 || nd < 1 || nd > 4 || n_jobs < 1 || n_jobs > NJ_MAX_JOBS || per < 1 || n_jobs % per ||
        skip < 0 || skip > std::max(0, level - 1))
        return hipErrorInvalidValue;
    for (int z = 0; per > 1 && z < n_jobs; z++)
        if ((uintptr_t)kj.d[z] & 15) return hipErrorInvalidValue;  // (ip_request_x: scratch, always aligned)
    const int n_out = n_jobs / per;
    const double bytes = 8.0 * N * (ne - skip) * (3.0 * nd * n_jobs + 2.0 * n_out * (1 + accumulate));
    if (N1 == 1) {
        if (!part || skip || c->alpha > 8) return hipErrorInvalidValue;
        IpTiles it;
        for (int j = 0; j < nd; j++) it.hat[j] = c->modup[level][j].hat;
        hipError_t e = launch(c, PROF_KEYIP, bytes, k_conv_ip, dim3(n_jobs, ne, nd), dim3(kNT8), s, kj, it, part, level,
                              c->L, c->alpha, c->n_q, c->d_tw, c->d_info);
        if (e != hipSuccess) return e;
        return launch(c, PROF_KEYIP, 16.0 * N * ne * (nd * n_jobs + n_out), k_ip_reduce,
                      dim3(n_out, 2 * ne), dim3(kNT8), s, part, nd * per, u, accumulate, level,
                      c->alpha, c->n_q, c->d_info, pout, c->d_itw, c->d_downscale);
    }
    const dim3 grid(n_out, N1, ne - skip);
    // key words stay in the caches only for the jobs that share them (a batch: 33.3 ms cached,
    // 35.8 non-temporal; giant steps with a key each at N = 2^14: 0.78 and 0.75 ms a step)
    const bool shared = n_out > 1 && kj.key[0] == kj.key[per];
#define NJ_IP_K(ND, SUM, NT)                                                                                         \
    launch(c, PROF_KEYIP, bytes, k_ntt_ip<ND, SUM, NT>, grid, dim3(kNT8), s, kj, per, u, accumulate, level, c->L, \
           c->alpha, c->n_q, c->d_tw, c->d_info, c->log_n, pout, c->d_itw, skip)
#define NJ_IP(ND)                                                                                                   \
    case ND:                                                                                                        \
        return per > 1 ? (shared ? NJ_IP_K(ND, true, false) : NJ_IP_K(ND, true, true))                              \
                       : (shared ? NJ_IP_K(ND, false, false) : NJ_IP_K(ND, false, true));
    switch (nd) {
        NJ_IP(1) NJ_IP(2) NJ_IP(3) NJ_IP(4)
    }
#undef NJ_IP
#undef NJ_IP_K
    return hipErrorInvalidValue;
}

// Special-prime rows of n_jobs key inner products from extended evaluation-form digits,
// through the first 12 stages of ModDown's inverse transform into pout (N >= 4096,
// 1..4 digits, alpha <= 8).
hipError_t launch_key_ip_ptile(const nj_ctx *c, int level, const KeyJobs &kj, int n_jobs, uint64_t *pout,
                               hipStream_t s)
{
    const int N = c->N, N1 = N / kT, nd = n_digits(c, level);
    if (N1 < 1 || nd < 1 || nd > 4 || c->alpha > 8 || n_jobs < 1 || n_jobs > NJ_MAX_JOBS || !pout)
        return hipErrorInvalidValue;
    const double bytes = 8.0 * N * c->alpha * (3.0 * nd + 2.0) * n_jobs;
    const dim3 grid(2 * n_jobs, N1, c->alpha);
#define NJ_PT(ND)                                                                                             \
    case ND:                                                                                                  \
        return launch(c, PROF_KEYIP, bytes, k_key_ip_ptile<ND>, grid, dim3(kNT8), s, kj, level, c->L, c->alpha, \
                      c->n_q, c->d_info, c->log_n, pout, c->d_itw, c->d_downscale);
    switch (nd) {
        NJ_PT(1) NJ_PT(2) NJ_PT(3) NJ_PT(4)
    }
#undef NJ_PT
    return hipErrorInvalidValue;
}

}  // namespace nj
