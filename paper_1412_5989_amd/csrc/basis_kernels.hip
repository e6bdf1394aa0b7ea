// Partner lists of the species determinants, built on the device.
//
// For every determinant x of one species (protons or neutrons):
//   l1(x):  every y with d(x, y) <= 1 (x itself included), any key;
//   l12(x): every y with d(x, y) <= 2 in the keys of x's 2M and Nq parity,
// where d is half the popcount of x XOR y (the number of moved nucleons), each
// in ascending y, so that every key is one contiguous segment.  One wavefront
// takes one x.  The d <= 1 partners are generated: every move of one nucleon
// within the Nq budget is looked up among the determinants of its key (sorted)
// and marked in a bit mask over y, which is read back in order.  The d <= 2
// partners are found by testing the few keys of x's class.  Passes: count (per
// key), offsets, fill with (x, y) placeholders, decode into records (moved
// orbits from __ffsll: particles in x and not in y, holes in y and not in x;
// fermion phase from masked popcounts).
#include <hip/hip_runtime.h>

#include "ci_internal.h"

namespace ci {


namespace {

constexpr int kPartnerWaves = 4;

// descriptor pointers are generic; use them through the global address space
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* glb(const T* p)
{
    return (const __attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* glbw(T* p)
{
    return (__attribute__((address_space(1))) T*)p;
}
// tables that a kernel only reads, read with wavefront-uniform addresses:
// through the constant address space they become scalar loads
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* cst(const T* p)
{
    return (const __attribute__((address_space(4))) T*)p;
}

// number of set bits of the W-word string strictly below orbit k
template <int W>
__device__ __forceinline__ int bits_below(const uint64_t* w, int k)
{
    int c = 0;
#pragma unroll
    for (int t = 0; t < W; t++) {
        const int d = k - t * 64;
        c += __popcll(d >= 64 ? w[t] : (d > 0 ? w[t] & ((1ull << d) - 1) : 0));
    }
    return c;
}

// lowest set orbit of a W-word string (which must have one)
template <int W>
__device__ __forceinline__ int lowest_orbit(const uint64_t* w)
{
    int k = -1;
#pragma unroll
    for (int t = W - 1; t >= 0; t--) k = w[t] ? t * 64 + __ffsll((long long)w[t]) - 1 : k;
    return k;
}

// (selects over the words: a runtime word index would put them in scratch memory)
template <int W>
__device__ __forceinline__ void clear_orbit(uint64_t* w, int k)
{
#pragma unroll
    for (int t = 0; t < W; t++) w[t] &= (k >> 6) == t ? ~(1ull << (k & 63)) : ~0ull;
}

// Record of partner y (local index yl in its key) of determinant x; pc is the
// popcount of x XOR y (0, 2 or 4).
template <int W>
__device__ __forceinline__ uint64_t partner_record(const uint64_t* x, const uint64_t* y, int pc, uint32_t yl)
{
    if (pc == 0) return make_rec(yl, 0, 0, 0, 0, 0, false);
    uint64_t holes[W], parts[W];
#pragma unroll
    for (int t = 0; t < W; t++) {
        holes[t] = y[t] & ~x[t];
        parts[t] = x[t] & ~y[t];
    }
    const int h1 = lowest_orbit<W>(holes), p1 = lowest_orbit<W>(parts);
    if (pc == 2) {
        // orbits of x strictly between the particle and the hole
        const int lo = p1 < h1 ? p1 : h1, hi = p1 < h1 ? h1 : p1;
        const int between = bits_below<W>(x, hi) - bits_below<W>(x, lo + 1);
        return make_rec(yl, 1, h1, p1, 0, 0, between & 1);
    }
    clear_orbit<W>(holes, h1);
    clear_orbit<W>(parts, p1);
    const int h2 = lowest_orbit<W>(holes), p2 = lowest_orbit<W>(parts);
    // phase of a+_p1 a+_p2 a_h2 a_h1 on y: T = y without h1, h2 (= x without p1, p2)
    uint64_t T[W];
#pragma unroll
    for (int t = 0; t < W; t++) T[t] = y[t];
    clear_orbit<W>(T, h1);
    clear_orbit<W>(T, h2);
    const int e = bits_below<W>(y, h1) + bits_below<W>(y, h2) - 1 + bits_below<W>(T, p1) + bits_below<W>(T, p2);
    return make_rec(yl, 2, h1, p1, h2, p2, e & 1);
}

__device__ __forceinline__ int rank_in(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int lane_read(int v, int l) { return __builtin_amdgcn_ds_bpermute(l << 2, v); }
__device__ __forceinline__ int incl_scan64(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef int int2_t __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2_t __attribute__((ext_vector_type(2)));

// The W words of determinant y (16-byte loads where W is even: the table
// starts at a 16-byte multiple).
template <int W>
__device__ __forceinline__ void load_sd(const uint64_t* sd, int64_t y, uint64_t* w)
{
    if constexpr (W % 2 == 0) {
#pragma unroll
        for (int t = 0; t < W; t += 2) {
            const u64x2_t v = *(const __attribute__((address_space(1))) u64x2_t*)(sd + y * W + t);
            w[t] = v.x;
            w[t + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int t = 0; t < W; t++) w[t] = glb(sd)[y * W + t];
    }
}

// Determinants covered by the bit mask of one wavefront (4 KB of LDS); a
// larger species is done in windows of that many, generating the moves again
// for each.
constexpr int kWindow = 32768;

// Testing every determinant against every other cost one wavefront instruction
// per pair and word (10B Nmax = 4, 19704 determinants per species: count 270
// us, fill 309 us; 6Li Nmax = 6, 8980: 126 and 140 us).  The moves of a
// nucleon that the budget allows are few (about as many as the d <= 1
// partners), so looking each up costs X n_sps searches instead of n tests, and
// the d <= 2 candidates of one class are a twentieth of the determinants: 75
// and 83 us (10B), 52 and 60 us (6Li).  Bound by the vector memory pipeline,
// which takes one cycle per lane of the searches' gathers; hence whole
// determinants per 16-byte load and the key's range in one.
template <int W, bool FILL>
__global__ void __launch_bounds__(64 * kPartnerWaves) partner_kernel(PartnerArgs A)
{
    __shared__ uint64_t bits_[kPartnerWaves][kWindow / 64];
    __shared__ int32_t ahead_[kPartnerWaves][FILL ? 1 : kWindow / 64 + 1];
    __shared__ uint8_t occ_[kPartnerWaves][64];
    const int lane = threadIdx.x & 63, wid = uniform(threadIdx.x >> 6);
    const int x = (int)blockIdx.x * kPartnerWaves + wid;
    if (x >= A.nsd) return;
    uint64_t* bits = bits_[wid];
    uint8_t* occ = occ_[wid];
    const int nsd = A.nsd, nk = A.nk;
    const auto sd = cst(A.sd);
    const auto key_off = cst(A.key_off);
    const auto orb = glb(A.orb_qn);
    const int kx = cst(A.sd_key)[x];
    const int mx = cst(A.key_m2)[kx], qx = cst(A.key_nq)[kx];
    const int64_t sb = (int64_t)x * (nk + 1);
    uint64_t xw[W];
    int X = 0;
#pragma unroll
    for (int t = 0; t < W; t++) {
        xw[t] = sd[(int64_t)x * W + t];
        if ((xw[t] >> lane) & 1) occ[X + rank_in(xw[t])] = (uint8_t)(t * 64 + lane);
        X += __popcll(xw[t]);
    }
    wave_fence();

    // the moves p -> h of lane u's nucleon p: the orbits of the shells that
    // the budget leaves it (whole shells, so a prefix of the orbits), holes of
    // x or not
    int p = 0, qp = 0, np = 0;
    if (lane < X) {
        p = occ[lane];
        qp = orb[p];
        const int top = A.budget - qx + 2 * (qp & 255) + ((qp >> 8) & 255);  // highest shell
        np = top < 0 ? 0 : min(A.nsps, (top + 1) * (top + 2) * (top + 3) / 3);
    }
    const int pincl = incl_scan64(np), pstart = pincl - np;
    const int moves = __builtin_amdgcn_readlane(pincl, 63);
    int64_t o1 = FILL ? cst(A.l1_ptr)[x] : 0;
    for (int w0 = 0; w0 < nsd; w0 += kWindow) {
        const int w1 = min(w0 + kWindow, nsd);
        const int nw = (w1 - w0 + 63) / 64;
        for (int i = lane; i < nw; i += 64) bits[i] = 0;
        wave_fence();
        if (lane == 0 && x >= w0 && x < w1) bits[(x - w0) >> 6] = 1ull << ((x - w0) & 63);
        wave_fence();
        for (int c0 = 0; c0 < moves; c0 += 64) {
            const int c = c0 + lane;
            int u = 0;  // the nucleon of move c: the last one that starts at or before it
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (lane_read(pstart, u + step) <= c) u += step;
            const int pu = lane_read(p, u), qu = lane_read(qp, u);
            const int h = c - lane_read(pstart, u);
            if (c >= moves) continue;
            uint64_t yw[W];
            bool free_h = true;
#pragma unroll
            for (int t = 0; t < W; t++) {
                const uint64_t hb = (h >> 6) == t ? 1ull << (h & 63) : 0, pb = (pu >> 6) == t ? 1ull << (pu & 63) : 0;
                free_h = free_h && !(xw[t] & hb);
                yw[t] = (xw[t] | hb) & ~pb;
            }
            if (!free_h) continue;
            // its key, by (Nq, 2M)
            const int qh = orb[h];
            const int kq = qx + 2 * ((qh & 255) - (qu & 255)) + ((qh >> 8) & 255) - ((qu >> 8) & 255) - A.kmap_nq0;
            const int km = (mx + (qh >> 24) - (qu >> 24) - A.kmap_m20) >> 1;
            if (kq < 0 || kq >= A.kmap_nq || km < 0 || km >= A.kmap_m2) continue;
            const int2_t range = glb((const int2_t*)A.kmap)[kq * A.kmap_m2 + km];
            // binary search among the key's determinants, ascending as numbers
            int lo = range.x, hi = range.y;
            bool hit = false;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                uint64_t z[W];
                load_sd<W>(A.sd, mid, z);
                bool less = false, eq = true;
#pragma unroll
                for (int t = 0; t < W; t++) {
                    less = z[t] < yw[t] || (z[t] == yw[t] && less);
                    eq = eq && z[t] == yw[t];
                }
                hit = hit || eq;
                if (eq) lo = hi = mid;
                else if (less) lo = mid + 1;
                else hi = mid;
            }
            if (hit && lo >= w0 && lo < w1)
                __hip_atomic_fetch_or(bits + ((lo - w0) >> 6), 1ull << ((lo - w0) & 63), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        wave_fence();
        if (FILL) {
            // lane i: word i of the mask, its partners in ascending y
            for (int i0 = 0; i0 < nw; i0 += 64) {
                uint64_t m = i0 + lane < nw ? bits[i0 + lane] : 0;
                const int n = __popcll(m), incl = incl_scan64(n);
                int64_t at = o1 + incl - n;
                const int y0 = w0 + (i0 + lane) * 64;
                for (; m; m &= m - 1)
                    glbw(A.l1)[at++] = ((uint64_t)(uint32_t)x << 32) | (uint32_t)(y0 + __ffsll((long long)m) - 1);
                o1 += __builtin_amdgcn_readlane(incl, 63);
            }
        } else {
            // marks ahead of each word, then lane k: the marks of key k
            int32_t* ahead = ahead_[wid];
            int tot = 0;
            for (int i0 = 0; i0 < nw; i0 += 64) {
                const int n = i0 + lane < nw ? __popcll(bits[i0 + lane]) : 0, incl = incl_scan64(n);
                if (i0 + lane < nw) ahead[i0 + lane] = tot + incl - n;
                tot += __builtin_amdgcn_readlane(incl, 63);
            }
            wave_fence();
            auto upto = [&](int y) -> int {  // marks below y
                if (y <= w0) return 0;
                if (y >= w1) return tot;
                const int d = y - w0;
                return ahead[d >> 6] + __popcll(bits[d >> 6] & ((1ull << (d & 63)) - 1));
            };
            for (int k = lane; k < nk; k += 64) {
                int n = upto(glb(A.key_off)[k + 1]) - upto(glb(A.key_off)[k]);
                if (w0 > 0) n += glbw(A.seg1)[sb + k];
                glbw(A.seg1)[sb + k] = n;
            }
        }
    }

    // d <= 2: the keys of x's 2M and Nq parity, 64 candidates at a time
    int64_t o12 = FILL ? cst(A.l12_ptr)[x] : 0;
    for (int k0 = 0; k0 < nk; k0 += 64) {
        const int k = k0 + lane;
        const bool same = k < nk && glb(A.key_m2)[k] == mx && ((glb(A.key_nq)[k] - qx) & 1) == 0;
        int cnt = 0;
        for (uint64_t keys = __ballot(same); keys; keys &= keys - 1) {
            const int kk = uniform(__ffsll((long long)keys) - 1);
            const int y0 = key_off[k0 + kk], y1 = key_off[k0 + kk + 1];
            int n = 0;
#pragma unroll 2
            for (int yb = y0; yb < y1; yb += 64) {
                const int y = yb + lane;
                int pc = 64;
                if (y < y1) {
                    uint64_t yw[W];
                    load_sd<W>(A.sd, y, yw);
                    pc = 0;
#pragma unroll
                    for (int t = 0; t < W; t++) pc += __popcll(xw[t] ^ yw[t]);
                }
                const bool in = pc <= 4;
                const uint64_t m = __ballot(in);
                if (FILL && in) glbw(A.l12)[o12 + n + rank_in(m)] = ((uint64_t)(uint32_t)x << 32) | (uint32_t)y;
                n += __popcll(m);
            }
            if (FILL) o12 += n;
            else if (lane == kk) cnt = n;
        }
        if (!FILL && k < nk) glbw(A.seg12)[sb + k] = cnt;
    }
}

// One lane per partner: the placeholder (x, y) becomes the partner record
// (local index of y, moved orbits, phase, d).  For l12 also records the
// position of x itself inside its own key segment.
template <int W>
__global__ void __launch_bounds__(256) partner_decode(PartnerArgs A, int64_t n1, int64_t n12, unsigned blocks1)
{
    const bool is12 = blockIdx.x >= blocks1;  // the first blocks1 workgroups take l1
    const int64_t t = (int64_t)(blockIdx.x - (is12 ? blocks1 : 0)) * blockDim.x + threadIdx.x;
    if (t >= (is12 ? n12 : n1)) return;
    const auto lst = glbw(is12 ? A.l12 : A.l1);
    const uint64_t ph = lst[t];
    const int x = (int)(ph >> 32), y = (int)(uint32_t)ph;
    uint64_t xw[W], yw[W];
    load_sd<W>(A.sd, x, xw);
    load_sd<W>(A.sd, y, yw);
    int pc = 0;
#pragma unroll
    for (int w = 0; w < W; w++) pc += __popcll(xw[w] ^ yw[w]);
    const int ky = glb(A.sd_key)[y];
    lst[t] = partner_record<W>(xw, yw, pc, (uint32_t)(y - glb(A.key_off)[ky]));
    if (is12 && x == y)
        glbw(A.self12)[x] = (int)(t - glb(A.l12_ptr)[x] - glb(A.seg12)[(int64_t)x * (A.nk + 1) + ky]);
}

// Segment counts -> segment offsets (exclusive scan over the keys of each
// determinant x), in both orders: seg[x][key], read by a wavefront that works
// on one x, and segT[key][x] (null: not wanted), read by one that works on
// neighbouring x in one key.  List lengths into l*_ptr[x + 1].  A workgroup takes kOffDets
// determinants of one of the two lists, a wavefront a quarter of them, lanes
// take keys; the transposed copy goes through LDS so that its stores are
// contiguous too.
constexpr int kOffDets = 32;

__global__ void __launch_bounds__(64 * kPartnerWaves) partner_offsets(PartnerArgs A)
{
    constexpr int kPer = kOffDets / kPartnerWaves;
    __shared__ int32_t tile[kOffDets][65];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xw = (int)blockIdx.x * kOffDets, x0 = xw + w * kPer;
    const bool l12 = blockIdx.y != 0;
    const auto seg = glbw(l12 ? A.seg12 : A.seg1), segT = glbw(l12 ? A.segT12 : A.segT1);
    const auto ptr = glbw(l12 ? A.l12_ptr : A.l1_ptr);
    const int nk = A.nk, nsd = A.nsd;
    int run[kPer] = {};
    for (int k0 = 0; k0 <= nk; k0 += 64) {
        int c[kPer];
#pragma unroll
        for (int i = 0; i < kPer; i++)
            c[i] = (x0 + i < nsd && k0 + lane < nk) ? seg[(int64_t)(x0 + i) * (nk + 1) + k0 + lane] : 0;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            int incl = c[i];
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(incl, o, 64);
                if (lane >= o) incl += u;
            }
            const int off = run[i] + incl - c[i];
            tile[w * kPer + i][lane] = off;
            if (x0 + i < nsd && k0 + lane <= nk) seg[(int64_t)(x0 + i) * (nk + 1) + k0 + lane] = off;
            run[i] += __shfl(incl, 63, 64);
        }
        if (!segT) continue;
        __syncthreads();
        const int m = nk + 1 - k0 < 64 ? nk + 1 - k0 : 64;
        for (int t = threadIdx.x; t < m * kOffDets; t += 64 * kPartnerWaves) {
            const int k = t / kOffDets, x = t % kOffDets;
            if (xw + x < nsd) segT[(int64_t)(k0 + k) * nsd + xw + x] = tile[x][k];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kPer; i++)
        if (lane == 0 && x0 + i < nsd) ptr[x0 + i + 1] = run[i];
    if (xw == 0 && threadIdx.x == 0) ptr[0] = 0;  // so that the inclusive scan of ptr gives offsets
}

}  // namespace

static inline unsigned grid_of(int64_t items) { return (unsigned)((items + kPartnerWaves - 1) / kPartnerWaves); }

template <bool FILL>
static void launch_scan(const PartnerArgs& a, hipStream_t s)
{
    const dim3 g(grid_of(a.nsd)), b(64 * kPartnerWaves);
    switch (a.W) {
        case 1: hipLaunchKernelGGL((partner_kernel<1, FILL>), g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL((partner_kernel<2, FILL>), g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL((partner_kernel<3, FILL>), g, b, 0, s, a); break;
        default: hipLaunchKernelGGL((partner_kernel<4, FILL>), g, b, 0, s, a); break;
    }
}

static void launch_decode(const PartnerArgs& a, int64_t n1, int64_t n12, hipStream_t s)
{
    const unsigned b1 = (unsigned)((n1 + 255) / 256), b12 = (unsigned)((n12 + 255) / 256);
    if (b1 + b12 == 0) return;
    const dim3 g(b1 + b12), b(256);
    switch (a.W) {
        case 1: hipLaunchKernelGGL(partner_decode<1>, g, b, 0, s, a, n1, n12, b1); break;
        case 2: hipLaunchKernelGGL(partner_decode<2>, g, b, 0, s, a, n1, n12, b1); break;
        case 3: hipLaunchKernelGGL(partner_decode<3>, g, b, 0, s, a, n1, n12, b1); break;
        default: hipLaunchKernelGGL(partner_decode<4>, g, b, 0, s, a, n1, n12, b1); break;
    }
}

__global__ void partner_no_sd(PartnerArgs A)
{
    glbw(A.l1_ptr)[0] = 0;
    glbw(A.l12_ptr)[0] = 0;
}

hipError_t launch_partner_count(const PartnerArgs& a, hipStream_t s)
{
    if (a.nsd > 0) {
        launch_scan<false>(a, s);
        hipLaunchKernelGGL(partner_offsets, dim3((unsigned)((a.nsd + kOffDets - 1) / kOffDets), 2),
                           dim3(64 * kPartnerWaves), 0, s, a);
    } else {
        hipLaunchKernelGGL(partner_no_sd, dim3(1), dim3(1), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_partner_fill(const PartnerArgs& a, int64_t n1, int64_t n12, hipStream_t s)
{
    if (a.nsd > 0) {
        launch_scan<true>(a, s);
        launch_decode(a, n1, n12, s);
    }
    return hipGetLastError();
}

}  // namespace ci
