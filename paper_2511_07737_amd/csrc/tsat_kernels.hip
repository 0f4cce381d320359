// tsat_kernels.hip -- gfx950 kernels of the gradient-guided SAT step
// (TurboSAT, arXiv 2511.07737, Sec. III-B and IV-A).
//
// Device data layout (all arrays owned by the host runtime):
//   lit rows   u64 [2V][W]     W = ceil(N/64); row 2v holds B(theta_norm) of
//                              variable v (bit c%64 of word c/64 = candidate c),
//                              row 2v+1 its complement (the negated literal,
//                              Sec. III-A: complete assignments).  Pad bits of
//                              both rows are 0.
//   theta,m,v  f32 [V][N]      logits and AdamW moments.
//   clause     u32 [Cb][k]     literal index 2*var+neg, one array per width k.
//   occurrence u32 stream      per variable: records of clauses where it
//                              occurs positively, then negatively; a record is
//                              (k-1, indices of the other k-1 literal rows).
//   H          u32 [Np][K+1]   per-candidate histogram of R (Np = 64 W).
//   table      f32 [K+1][Np]   dL/dR as a function of R, per candidate.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "tsat.h"
#include "tsat_device.h"
#include "tsat_learned.h"

namespace tsat {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

// c + bit `lane` of the wave-uniform 64-bit mask m, in one VALU op: the mask
// is the carry-in of v_addc, and its bits map one-to-one onto the 64 lanes.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t add_lane_bit(uint32_t c, uint64_t m)
{
    uint32_t r;
    uint64_t co;
    const uint64_t ms = uniform64(m); // a no-op when m already lives in SGPRs
    asm("v_addc_co_u32_e64 %0, %1, %2, 0, %3" : "=v"(r), "=s"(co) : "v"(c), "s"(ms));
    return r;
}

// Wave-uniform load through the scalar cache: the constant address space tells
// the compiler the location is not written by this kernel, so a uniform
// address becomes an s_load.  Only for buffers the kernel does not write.
template <class T>
__device__ __forceinline__ T sload(const T* p)
{
    return *(const __attribute__((address_space(4))) T*)p;
}

// FP64 sum over the 64 lanes without LDS: DPP swaps inside quads, DPP
// rotations inside rows of 16, then the four row sums read from fixed lanes.
// Every call adds in the same order, so the result is deterministic and
// wave-uniform (it lives in SGPRs).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    // every lane has a source lane under these patterns, so no old value is needed
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double readlane_f64(double x, int lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum within each row of 16 lanes (every lane of the row gets it).
__device__ __forceinline__ double row16_sum(double x)
{
    x += dpp_f64<0xB1>(x);  // quad_perm [1,0,3,2]
    x += dpp_f64<0x4E>(x);  // quad_perm [2,3,0,1]
    x += dpp_f64<0x124>(x); // row_ror:4
    x += dpp_f64<0x128>(x); // row_ror:8
    return x;
}

__device__ __forceinline__ double wave_sum(double x)
{
    x = row16_sum(x);
    const double r0 = readlane_f64(x, 0), r1 = readlane_f64(x, 16);
    const double r2 = readlane_f64(x, 32), r3 = readlane_f64(x, 48);
    return (r0 + r1) + (r2 + r3);
}

// Sum of a row held by one wave (lane l: candidates 64 j + l), x[j] a lane's
// terms.  Rows of more than four words are summed in groups of four words,
// group after group: the order in which a team of waves, four words each,
// adds its shares (var_window_team_kernel), so that every kernel forms the
// same sums.
template <int J, class F>
__device__ __forceinline__ double row_sum(F x)
{
    double total = 0.0;
#pragma unroll
    for (int j0 = 0; j0 < J; j0 += 4) {
        double s = 0.0;
#pragma unroll
        for (int j = j0; j < (J < j0 + 4 ? J : j0 + 4); ++j) s += x(j);
        s = wave_sum(s);
        total = j0 == 0 ? s : total + s;
    }
    return total;
}

// Sum over each half wave (lanes 0-31, 32-63), returned to the lanes of that
// half.  A half holding a row of at most 32 values gets the wave_sum value
// of that row alone (there, the other half adds only zeros).
__device__ __forceinline__ double half_sum(double x)
{
    x = row16_sum(x);
    const double r0 = readlane_f64(x, 0), r1 = readlane_f64(x, 16);
    const double r2 = readlane_f64(x, 32), r3 = readlane_f64(x, 48);
    return (__lane_id() < 32u) ? r0 + r1 : r2 + r3;
}

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

// XCD-aware work order.  Workgroups are handed to the eight XCDs round-robin
// (workgroup b runs on XCD b mod 8), each XCD with its own L2.  With `on`
// and a grid that is a multiple of 8, each XCD takes a contiguous eighth of
// the work items, so items that touch the same data (consecutive clauses of
// one instance or community, consecutive variables) share that XCD's L2.
// Without it (or for other grid sizes) the items go round-robin as before.
struct ItemRange {
    uint32_t first, end, stride;
};

__device__ __forceinline__ ItemRange xcd_items(bool on, uint32_t nitems, uint32_t per_block, uint32_t slot)
{
    ItemRange r;
    const uint32_t g = gridDim.x;
    if (on && g % 8u == 0u) {
        const uint32_t x = blockIdx.x % 8u, local = blockIdx.x / 8u;
        const uint32_t share = (nitems + 7u) / 8u;
        const uint32_t b0 = x * share;
        r.first = b0 + local * per_block + slot;
        r.end = b0 + share < nitems ? b0 + share : nitems;
        r.stride = (g / 8u) * per_block;
    } else {
        r.first = blockIdx.x * per_block + slot;
        r.end = nitems;
        r.stride = g * per_block;
    }
    return r;
}

// The forward work unit of this block (grid rounded up to a multiple of 8
// when XCD-aware; surplus blocks get an index >= n and return).
__device__ __forceinline__ uint32_t xcd_unit(bool on, uint32_t n)
{
    const uint32_t g = gridDim.x;
    if (!on || g % 8u != 0u) return blockIdx.x;
    return (blockIdx.x % 8u) * (g / 8u) + blockIdx.x / 8u;
}

// ---------------------------------------------------------------------------
// Forward: R = P A (Eq. 1) as a per-candidate histogram of R.
//
// One thread owns candidate dword d (32 candidates) and a strided set of up
// to CPT clauses of one width bucket.  For each clause it forms the k literal
// dwords and the cumulative masks ge[r] = [R >= r+1] bit-sliced over the 32
// candidates, and adds each mask into a B-plane vertical counter.  At the end
// the counters are read out per candidate into LDS bins, then the block adds
// its bins to the global histogram.
// ---------------------------------------------------------------------------

// Literal dword d of row `code` (2 var + neg).  VR: the rows hold the values
// of the variables only ([V][W2] dwords); a negated literal is the complement.
template <bool VR>
__device__ __forceinline__ uint32_t lit_dword(const uint32_t* __restrict__ bits32, uint32_t code, int W2, int d)
{
    if (VR) return bits32[(size_t)(code >> 1) * W2 + d] ^ (0u - (code & 1u));
    return bits32[(size_t)code * W2 + d];
}

// One work unit of a width-KW bucket: the block's clauses [u.c0, u.c1),
// their literal codes in `codes` (KW per clause), planes of R written to
// `planes` ([clause][plane_P][plane_stride] dwords from clause plane_base)
// when non-null.  lh: the block's LDS counts, [KW][32][DT].
//
// A lane counts dword tid mod DT of the rows; the 64 / DT lanes of a wave
// that share a dword are its slots.  The read-out adds the vertical counters
// of a wave's slots with a bit-sliced adder over log2(slots) lane exchanges,
// after which every lane of a dword holds the wave's totals and extracts its
// share of the 32 candidates: consecutive LDS words, one add per candidate
// and level.  (Every lane extracting all 32 of its candidates and adding
// them to LDS bins shared by its slots took most of a small launch: all
// lanes of a dword hit one bank at a time.)  With the histogram replicas:
// large configuration 255 -> 212 us, 32 ragged instances (4.6e5 variables,
// N = 32) 69 -> 27 us, V = 5e4 and N = 1000 76 -> 43 us, 32 instances of
// V = 200 and N = 64 15.8 -> 10.5 us.
template <int KW, int B, bool VR>
__device__ __forceinline__ void fwd_hist_unit(const FwdArgs& a, const FwdUnit& u, const uint32_t* __restrict__ codes,
                                              uint32_t* planes, int plane_P, int64_t plane_base, uint32_t* lh)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int DT = a.DT, nsl = 64 / DT; // dwords of the tile, slots of a wave
    const int dl = lane % DT, ws = lane / DT, slot = (tid >> 6) * nsl + ws, S = 4 * nsl;
    const int d = blockIdx.y * DT + dl;
    for (int q = tid; q < KW * 32 * DT; q += blockDim.x) lh[q] = 0;
    __syncthreads();
    uint32_t pl[KW][B + 6];
#pragma unroll
    for (int r = 0; r < KW; ++r)
#pragma unroll
        for (int b = 0; b < B + 6; ++b) pl[r][b] = 0;
    if (d < a.Dn && ws < nsl) {
        // this thread's clauses: c0 + it S for it < nit
        const int64_t c0 = u.c0 + slot;
        const int64_t rem = u.c1 - c0;
        const int nit = rem <= 0 ? 0 : (int)(rem < (int64_t)a.CPT * S ? (rem + S - 1) / S : a.CPT);
        // software pipeline over the clauses: while clause it is counted, the
        // literal dwords of clause it + 1 and the literal codes of clause
        // it + 2 are in flight (one memory round trip per clause, not two)
        uint32_t code_nx[KW], x_nx[KW];
#pragma unroll
        for (int q = 0; q < KW; ++q) {
            code_nx[q] = 0u;
            x_nx[q] = 0u;
        }
        if (nit > 0) {
#pragma unroll
            for (int q = 0; q < KW; ++q) x_nx[q] = lit_dword<VR>(a.bits32, codes[c0 * KW + q], a.W2, d);
        }
        if (nit > 1) {
#pragma unroll
            for (int q = 0; q < KW; ++q) code_nx[q] = codes[(c0 + S) * KW + q];
        }
        for (int it = 0; it < nit; ++it) {
            const int64_t c = c0 + (int64_t)it * S;
            uint32_t x[KW];
#pragma unroll
            for (int q = 0; q < KW; ++q) x[q] = x_nx[q];
            if (it + 1 < nit) {
#pragma unroll
                for (int q = 0; q < KW; ++q) x_nx[q] = lit_dword<VR>(a.bits32, code_nx[q], a.W2, d);
            }
            if (it + 2 < nit) {
#pragma unroll
                for (int q = 0; q < KW; ++q) code_nx[q] = codes[(c + 2 * S) * KW + q];
            }
            uint32_t ge[KW];
#pragma unroll
            for (int r = 0; r < KW; ++r) ge[r] = 0;
#pragma unroll
            for (int q = 0; q < KW; ++q) {
#pragma unroll
                for (int r = KW - 1; r >= 1; --r) ge[r] |= ge[r - 1] & x[q];
                ge[0] |= x[q];
            }
            if (a.rbytes) {
                // R of the 32 candidates in bytes, four at a time: the four
                // bits of a plane spread to four bytes by a multiplication
                uint32_t bp[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    bp[p] = 0;
#pragma unroll
                    for (int r = 1 << p; r <= KW; r += 1 << p) bp[p] ^= ge[r - 1];
                }
                uint32_t w[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    w[q] = 0;
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        if ((1 << p) <= KW) w[q] |= (__umul24((bp[p] >> (4 * q)) & 15u, 0x204081u) & 0x01010101u) << p;
                }
                uint4* out = (uint4*)(a.rbytes + (size_t)(plane_base + c) * a.rb_stride + 32u * (uint32_t)d);
                out[0] = make_uint4(w[0], w[1], w[2], w[3]);
                out[1] = make_uint4(w[4], w[5], w[6], w[7]);
            } else if (planes) {
                // R in binary for the backward, plane_P planes: bit p of R is
                // the parity of the masks [R >= m 2^p], m >= 1
                uint32_t* P = planes + (size_t)(plane_base + c) * (size_t)(plane_P * a.plane_stride) + d;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    if (p >= plane_P) break;
                    uint32_t bp = 0;
#pragma unroll
                    for (int r = 1 << p; r <= KW; r += 1 << p) bp ^= ge[r - 1];
                    P[(size_t)p * a.plane_stride] = bp;
                }
            }
#pragma unroll
            for (int r = 0; r < KW; ++r) {
                uint32_t carry = ge[r];
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const uint32_t t = pl[r][b] & carry;
                    pl[r][b] ^= carry;
                    carry = t;
                }
            }
        }
    }
    // the slots' counters, added over windows of `off` slots: a circular
    // window when the slots are a power of two (every lane then ends with
    // the wave's total), else cut at the last slot (slot 0 holds the total)
    const bool pow2 = (nsl & (nsl - 1)) == 0;
#pragma unroll
    for (int st = 0; st < 6; ++st) {
        const int off = 1 << st;
        if (off >= nsl) break; // block-uniform
        const int other = ws + off;
        const bool in = pow2 || other < nsl;
        const int src = (pow2 ? (other & (nsl - 1)) : other) * DT + dl;
#pragma unroll
        for (int r = 0; r < KW; ++r) {
            uint32_t carry = 0;
#pragma unroll
            for (int b = 0; b < B + st; ++b) {
                uint32_t y = __shfl(pl[r][b], in ? src : lane);
                y = in ? y : 0u;
                const uint32_t x = pl[r][b], t = x ^ y;
                pl[r][b] = t ^ carry;
                carry = (t & carry) | (~t & x);
            }
            pl[r][B + st] = carry;
        }
    }
    if (!pow2) {
#pragma unroll
        for (int r = 0; r < KW; ++r)
#pragma unroll
            for (int b = 0; b < B + 6; ++b) pl[r][b] = __shfl(pl[r][b], dl);
    }
    if (d < a.Dn && ws < nsl) {
        for (int p = ws; p < 32; p += nsl) {
#pragma unroll
            for (int r = 0; r < KW; ++r) {
                uint32_t s = 0;
#pragma unroll
                for (int b = 0; b < B + 6; ++b) s |= ((pl[r][b] >> p) & 1u) << b;
                if (s) atomicAdd(&lh[(r * 32 + p) * DT + dl], s);
            }
        }
    }
    __syncthreads();
    uint32_t* H = a.H + ((size_t)u.inst * a.H_reps + blockIdx.x % (uint32_t)a.H_reps) * a.H_stride;
    const uint32_t total = (uint32_t)(u.c1 - u.c0);
    // consecutive lanes add to consecutive words of H (a lane per candidate
    // with its levels in turn touches four lines for one: V = 5e4 and
    // N = 1000, 117 us against 43)
    for (int q = tid; q < 32 * DT * (KW + 1); q += blockDim.x) {
        const int c = q / (KW + 1), r = q - c * (KW + 1), dd = c >> 5;
        const int at = (c & 31) * DT + dd;
        if (blockIdx.y * DT + dd >= a.Dn) break;
        const uint32_t ge = r > 0 ? lh[(r - 1) * 32 * DT + at] : total;
        const uint32_t nx = r < KW ? lh[r * 32 * DT + at] : 0u;
        if (ge != nx) atomicAdd(&H[(size_t)(blockIdx.y * DT * 32 + c) * a.K1 + r], ge - nx);
    }
}

template <int KW, int B, bool VR>
__global__ __launch_bounds__(256) void fwd_hist_kernel(FwdArgs a)
{
    extern __shared__ uint32_t lh[]; // [KW][32][DT]
    if (a.ctrl && a.ctrl->stop) return;
    const uint32_t un = xcd_unit(a.xcd, (uint32_t)a.nunits);
    if (un >= (uint32_t)a.nunits) return;
    const FwdUnit u = a.units[un];
    if (a.ictrl && a.ictrl[u.inst].frozen) return;
    fwd_hist_unit<KW, B, VR>(a, u, a.codes, a.planes, a.plane_P, a.plane_base, lh);
}

// Wide clauses (k > 4): one lane per candidate.  A wave takes a run of
// consecutive clauses of the bucket (their literal indices come through the
// scalar cache), reads for each literal the dword of the row that holds its
// lane's candidate, counts R = the candidate's true literals and adds one to
// the lane's own LDS bin R (no two lanes share a bin, so no conflicts); the
// block then adds its four waves' bins into the global histogram.  Clauses
// are taken G at a time, all their row loads issued before the first wait.
template <int KMAX, int G, bool VR>
__device__ __forceinline__ void fwd_lanes_run(const FwdArgs& a, int k, const uint32_t* codes, int64_t cb, int64_t ce,
                                              int64_t pbase, uint32_t cand, bool live, uint32_t* my)
{
    const uint32_t d = live ? cand >> 5 : 0u, bit = cand & 31u;
    for (int64_t c = cb; c < ce; c += G) { // wave-uniform
        // the codes past a clause's width belong to the next one (the bucket
        // is padded): all loads without a condition between them, the rows
        // past the width replaced by the clause's first
        uint32_t code[G][KMAX], x[G][KMAX];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t* cl = (const uint32_t*)uniform64((uint64_t)(codes + (c + g < ce ? c + g : c) * k));
#pragma unroll
            for (int q = 0; q < KMAX; ++q) code[g][q] = sload(cl + q);
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int q = 0; q < KMAX; ++q) x[g][q] = lit_dword<VR>(a.bits32, q < k ? code[g][q] : code[g][0], a.W2, d);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (c + g >= ce) break;
            uint32_t R = 0;
#pragma unroll
            for (int q = 0; q < KMAX; ++q) R += q < k ? (x[g][q] >> bit) & 1u : 0u;
            if (live) atomicAdd(&my[R], 1u);
            if (a.rbytes) a.rbytes[(size_t)(pbase + c + g) * a.rb_stride + cand] = (uint8_t)R;
        }
    }
}

// A block's clauses share a width; the run is compiled for widths up to 8,
// 16 and 32, so that narrow units keep several clauses in flight next to a
// bucket of wide ones (2e5 mixed clauses up to 24 wide, N = 100: 87 us
// with every unit one clause at a time and codes in vector registers, 24 us
// with the bytes of R written as well).
template <int KMAX, bool VR>
__global__ __launch_bounds__(256) void fwd_hist_lanes_kernel(FwdArgs a)
{
    extern __shared__ uint32_t lh[]; // [4 waves][64 lanes][K1]
    if (a.ctrl && a.ctrl->stop) return;
    const uint32_t un = xcd_unit(a.xcd, (uint32_t)a.nunits);
    if (un >= (uint32_t)a.nunits) return;
    const FwdUnit u = a.units[un];
    if (a.ictrl && a.ictrl[u.inst].frozen) return;
    uint32_t* H = a.H + ((size_t)u.inst * a.H_reps + blockIdx.x % (uint32_t)a.H_reps) * a.H_stride;
    const uint32_t lane = __lane_id(), wave = uniform(threadIdx.x / 64u);
    // KW = 0: the units of every wide bucket in one launch, unit width in pad
    const int K1 = a.K1, k = (int)uniform((uint32_t)(a.KW > 0 ? a.KW : u.pad));
    // from the tables by width in either form: a choice between them and the
    // single bucket's fields becomes one of two addresses, for which every lane
    // copies the arguments to scratch memory (672 bytes)
    const uint32_t* codes = a.wide_codes[k];
    const int64_t pbase = a.wide_base[k];
    const uint32_t cand = blockIdx.y * 64u + lane;
    const bool live = (int)(cand >> 5) < a.Dn;
    uint32_t* my = lh + (wave * 64u + lane) * (uint32_t)K1;
    for (int r = 0; r < K1; ++r) my[r] = 0;
    // this wave's clauses: a quarter of the unit
    const int64_t u0 = (int64_t)uniform64((uint64_t)u.c0), u1 = (int64_t)uniform64((uint64_t)u.c1);
    const int64_t share = (u1 - u0 + 3) / 4;
    const int64_t cb = u0 + (int64_t)wave * share;
    const int64_t ce = cb + share < u1 ? cb + share : u1;
    if (KMAX > 16 && k > 16) fwd_lanes_run<KMAX, 1, VR>(a, k, codes, cb, ce, pbase, cand, live, my);
    else if (KMAX > 8 && k > 8) fwd_lanes_run<(KMAX < 16 ? KMAX : 16), 2, VR>(a, k, codes, cb, ce, pbase, cand, live, my);
    else fwd_lanes_run<8, 4, VR>(a, k, codes, cb, ce, pbase, cand, live, my);
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * K1; e += 256) {
        const int l = e / K1, r = e % K1;
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += lh[(w * 64 + l) * K1 + r];
        const uint32_t cc = blockIdx.y * 64u + (uint32_t)l;
        if (sum && (int)(cc >> 5) < a.Dn) atomicAdd(&H[(size_t)cc * K1 + r], sum);
    }
}

// ---------------------------------------------------------------------------
// SmoothMin (Eq. 4), loss (Eq. 3), dL/dR table, schedule (Sec. IV-A).
// One block per instance (stateless evaluations without a loss: one per 256
// candidates).  Candidate i: H[i][r] (plus the empty clauses in bin 0),
// r0 = min{r : H > 0}, w_r = exp(-tau (r - r0)), D = sum H w,
// S = sum r H w / D, table[r][i] = dS_i (w_r / D)(1 - tau (r - S)).
//
// A latency chain, not work: the exponentials depend on r - r0 alone and are
// formed once per block, the schedule's powers by three waves side by side,
// the histogram replicas are summed by coalesced loads into LDS, and the
// closing reductions take one barrier.  (V = 200, N = 64: 5.2 -> 4.6 us
// with eight replicas to add where there was one; large 9.9 -> 9.7.)
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void smin_kernel(SminArgs a)
{
    __shared__ double s_loss[256];
    __shared__ double s_w[2 * TSAT_MAX_WIDTH + 1]; // exp(-tau x), x = -(K1 - 1) .. K1 - 1
    __shared__ int64_t s_best[4];
    __shared__ int32_t s_bidx[4], s_sat[4];
    extern __shared__ uint32_t s_h[]; // [256][K1 | 1]
    Ctrl* ctrl = a.ctrl;
    if (ctrl && ctrl->stop) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int b = blockIdx.x; // instance
    const int K1 = a.K1, hs = K1 | 1;
    const int64_t t = ctrl ? ctrl->t : 0;
    if (b == 0 && ctrl && a.update) {
        // schedule scalars of the pending update:
        // lr(t) = max(lr_min, lr0 decay^floor((t mod restart)/every))
        const int64_t phase = a.restart > 0 ? t % a.restart : t;
        // assignment mixing at a restart replaces the update and starts a
        // fresh AdamW: the bias corrections count from the next iteration
        const bool mixing = a.mix && a.restart > 0 && t > 0 && phase == 0;
        const double tt = (double)(t - (mixing ? t + 1 : ctrl->t_reset) + 1);
        __syncthreads(); // every thread has read t_reset
        if (tid == 0) {
            const int64_t e = a.every > 0 ? phase / a.every : 0;
            double lr = a.lr0 * pow(a.decay, (double)e);
            if (lr < a.lr_min) lr = a.lr_min;
            ctrl->mixing = mixing ? 1 : 0;
            if (mixing) ctrl->t_reset = t + 1;
            ctrl->lr = lr;
            ctrl->f_decay = (float)(1.0 - lr * a.weight_decay);
            s_loss[0] = lr;
        } else if (tid == 64) {
            s_loss[1] = 1.0 - pow(a.beta1, tt);
        } else if (tid == 128) {
            const double bc2 = 1.0 - pow(a.beta2, tt);
            ctrl->f_isbc2 = (float)(1.0 / sqrt(bc2));
        }
    }
    if (tid >= 192) {
        for (int x = tid - 192; x < 2 * K1 - 1; x += 64) s_w[x] = exp(-a.tau * (double)(x - (K1 - 1)));
    }
    __syncthreads();
    if (tid == 0 && b == 0 && ctrl && a.update) ctrl->f_step = (float)(s_loss[0] / s_loss[1]);
    InstCtrl* ic = a.ictrl ? a.ictrl + b : nullptr;
    if (ic && ic->frozen) return; // nothing accumulated for a frozen instance
    const InstInfo info = a.info[b];
    uint32_t* Hb = a.H + (size_t)b * a.H_reps * a.Np * K1;
    float* tb = a.table ? a.table + (size_t)b * K1 * a.Np : nullptr;
    const size_t ob = (size_t)b * a.N;
    const double* w0 = s_w + (K1 - 1); // w0[x] = exp(-tau x)
    double loss = 0.0;
    int64_t best = -1;
    int32_t bidx = 0x7fffffff, satc = 0x7fffffff;
    // passes of 256 candidates, counted in passes: Np may be close to 2^31
    const int passes = (a.Np - 1) / 256 + 1;
    for (int pass = blockIdx.y; pass < passes; pass += gridDim.y) {
        const int i0 = pass * 256;
        // this pass's histogram rows: the replicas' sum, cleared on the way
        const int rows = min(256, a.Np - i0);
        for (int g = tid; g < rows * K1 / 4; g += 256) { // 16 bytes: rows is a multiple of 64
            uint4* src = (uint4*)(Hb + (size_t)i0 * K1) + g;
            const size_t stride = (size_t)a.Np * K1 / 4;
            uint4 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = q < a.H_reps ? src[q * stride] : make_uint4(0u, 0u, 0u, 0u);
            uint32_t h[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                h[0] += v[q].x;
                h[1] += v[q].y;
                h[2] += v[q].z;
                h[3] += v[q].w;
            }
            if (a.zero_H) {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (q < a.H_reps) src[q * stride] = make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = 4 * g + j, c = e / K1, r = e - c * K1;
                s_h[c * hs + r] = h[j];
                if (a.H_save) a.H_save[(size_t)i0 * K1 + e] = h[j];
                if (a.H_last && i0 + c < a.N)
                    a.H_last[(ob + i0) * K1 + e] = h[j] + (r == 0 ? (uint32_t)info.n_empty : 0u);
            }
        }
        __syncthreads();
        const int i = i0 + tid;
        if (tid < rows && i >= a.N) {
            if (tb)
                for (int r = 0; r < K1; ++r) tb[(size_t)r * a.Np + i] = 0.0f;
        } else if (tid < rows) {
            const uint32_t* h = s_h + tid * hs;
            int r0 = -1;
            for (int r = 0; r < K1; ++r) {
                const uint64_t hr = (uint64_t)h[r] + (r == 0 ? (uint64_t)info.n_empty : 0);
                if (hr > 0) { r0 = r; break; }
            }
            double D = 0.0, num = 0.0;
            if (r0 >= 0) {
                for (int r = 0; r < K1; ++r) {
                    const double hr = (double)h[r] + (r == 0 ? (double)info.n_empty : 0.0);
                    const double w = w0[r - r0];
                    D += hr * w;
                    num += (double)r * hr * w;
                }
            }
            const double S = (r0 >= 0) ? num / D : 0.0;
            const int64_t unsat = (int64_t)h[0] + info.n_empty;
            const int64_t sat = info.C - unsat;
            if (a.S_out) a.S_out[ob + i] = (float)S;
            if (a.S64_out) a.S64_out[ob + i] = S;
            if (a.sat_out) a.sat_out[ob + i] = sat;
            loss += S;
            if (sat > best) { best = sat; bidx = i; }
            if (unsat == 0 && i < satc) satc = i;
            if (tb) {
                // dL/dS_i: given per candidate, or -dloss (Eq. 3 scaled by
                // the upstream gradient of the loss), or -1 (Eq. 3)
                const double up = a.dS ? (double)a.dS[ob + i] : (a.dloss ? -(double)a.dloss[b] : -1.0);
                for (int r = 0; r < K1; ++r) {
                    double tv = 0.0;
                    if (r0 >= 0) tv = up * (w0[r - r0] / D) * (1.0 - a.tau * ((double)r - S));
                    tb[(size_t)r * a.Np + i] = (float)tv;
                }
            }
        }
        __syncthreads(); // the next pass rewrites the rows
    }
    if (!ic && !a.loss_out) return;
    // the loss in a fixed order: lanes tid, tid + 128, tid + 64, tid + 192,
    // then halves of the first wave; the best candidate by count, then index
    s_loss[tid] = loss;
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) {
        const int64_t ob2 = __shfl_xor(best, st);
        const int32_t oi = __shfl_xor(bidx, st), os = __shfl_xor(satc, st);
        if (ob2 > best || (ob2 == best && oi < bidx)) {
            best = ob2;
            bidx = oi;
        }
        satc = min(satc, os);
    }
    if (lane == 0) {
        s_best[wv] = best;
        s_bidx[wv] = bidx;
        s_sat[wv] = satc;
    }
    __syncthreads();
    if (wv != 0) return;
    double l = (s_loss[tid] + s_loss[tid + 128]) + (s_loss[tid + 64] + s_loss[tid + 192]);
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) l += __shfl_down(l, st);
    if (tid != 0) return;
#pragma unroll
    for (int w = 1; w < 4; ++w) {
        if (s_best[w] > best || (s_best[w] == best && s_bidx[w] < bidx)) {
            best = s_best[w];
            bidx = s_bidx[w];
        }
        satc = min(satc, s_sat[w]);
    }
    if (a.loss_out) a.loss_out[b] = (float)(-l);
    if (!ic) return;
    const uint64_t now = __builtin_amdgcn_s_memrealtime();
    if (ic->start_time == 0) ic->start_time = now;
    ic->loss = -l;
    ic->best_cand = bidx;
    ic->best_sat = best;
    ic->witness_pending = 0;
    const bool any_sat = satc != 0x7fffffff;
    if (any_sat && ic->first_sat_step < 0) {
        ic->first_sat_step = t;
        ic->sat_cand = satc;
        ic->sat_time = now;
        ic->witness_pending = 1;
    }
    const bool converged = (double)best > a.conv_frac * (double)info.C;
    if (converged && ic->first_conv_step < 0) {
        ic->first_conv_step = t;
        ic->conv_time = now;
    }
    // stop mode 1: freeze on a satisfying candidate; 2: also on
    // convergence, the hand-off point of Sec. IV-B
    if (a.update && ctrl && ctrl->stop_on_sat && (any_sat || (ctrl->stop_on_sat == 2 && converged))) {
        // freeze: the current bits stay (a witness if satisfied), no more updates
        ic->frozen = 1;
        ic->witness_pending = 0;
        const int nf = atomicAdd(&ctrl->n_frozen, 1) + 1;
        if (nf >= a.n_inst) ctrl->stop = 1;
    }
}

// ---------------------------------------------------------------------------
// Variable-major pass: adjoint (P^T dL/dR with the straight-through
// estimator), Eq. 5 backward, AdamW, Eq. 5 + Eq. 2 re-binarization, pack.
//
// One wave owns one variable row at a time; lane l holds candidates
// 64 j + l, j < J.  The records of the variable are wave-uniform, so the
// clause's other literal rows come in through the scalar cache and their
// bits reach the lanes as carry-in masks.  No atomics: every U_vi is summed
// by the lane that owns it, and the row's reductions stay in the wave.
// ---------------------------------------------------------------------------

enum { OP_STEP = 0, OP_GRAD = 1, OP_ADJ = 2, OP_BINARIZE = 3, OP_NORMBWD = 4 };

struct StepScalars {
    float f_decay, f_step, f_isbc2;
    float b1, b2, omb1, omb2, eps;
};

__device__ __forceinline__ StepScalars load_scalars(const VarArgs& a, int op)
{
    StepScalars c;
    c.f_decay = 1.f;
    c.f_step = 0.f;
    c.f_isbc2 = 1.f;
    if (op == OP_STEP) {
        c.f_decay = a.ctrl->f_decay;
        c.f_step = a.ctrl->f_step;
        c.f_isbc2 = a.ctrl->f_isbc2;
    }
    c.b1 = a.beta1;
    c.b2 = a.beta2;
    c.omb1 = a.one_minus_beta1;
    c.omb2 = a.one_minus_beta2;
    c.eps = a.eps;
    return c;
}

// Eq. 5 clamp of a row mean: |mu| < 1e-12 becomes +-1e-12 (0 -> +1e-12).
__device__ __forceinline__ double clamp_mu(double mu, bool& clamped)
{
    clamped = fabs(mu) < 1e-12;
    return clamped ? ((mu >= 0.0) ? 1e-12 : -1e-12) : mu;
}

// Pack B(theta_norm) of one variable row into its two literal rows: their
// 2 W words are consecutive, lane j < W stores word j of the value row and
// lane W + j of the complement (one store instruction per variable, not 2 W).
template <int J>
__device__ __forceinline__ void write_bits(const VarArgs& a, uint32_t v, uint32_t lane, const float (&th)[J],
                                          const bool (&valid)[J], bool pos)
{
    const int W = a.W;
    uint64_t word = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if (j >= W) break;
        const bool p = valid[j] && (pos ? th[j] > 0.f : th[j] < 0.f);
        const uint64_t bal = ballot64(p);
        const uint64_t vm = ballot64(valid[j]);
        word = (int)lane == j ? bal : word;
        word = (int)lane == W + j ? ~bal & vm : word;
    }
    if (a.lit_rows) { // row v is a literal of its own
        if ((int)lane < W) a.lits_next[(size_t)v * W + lane] = word;
    } else if ((int)lane < 2 * W) {
        a.lits_next[(size_t)(2 * v) * W + lane] = word;
    }
}

// Row loads of theta (and the optimizer moments for the step).  The θ, m, v
// streams are touched once per iteration, so they go non-temporal: they
// then do not push the clause planes and literal rows, which the gathers
// read at random, out of the last-level cache.
template <int J, int OP, bool FULL = false>
__device__ __forceinline__ void load_row(const VarArgs& a, uint32_t v, uint32_t lane, float (&th)[J], float (&mm)[J],
                                         float (&vv)[J], bool (&valid)[J])
{
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = 64 * j + (int)lane;
        valid[j] = FULL || i < a.N; // FULL: N == 64 J, every lane holds a candidate
        const size_t idx = (size_t)v * a.N + i;
        th[j] = (OP != OP_ADJ && valid[j]) ? __builtin_nontemporal_load(a.theta + idx) : 0.f;
        mm[j] = (OP == OP_STEP && valid[j]) ? __builtin_nontemporal_load(a.m + idx) : 0.f;
        vv[j] = (OP == OP_STEP && valid[j]) ? __builtin_nontemporal_load(a.v + idx) : 0.f;
    }
}

// Eq. 5 backward of one variable row: g = U / mu - (sum_i U_i theta_i) /
// (N mu^2) in mean mode (inside the clamp the mean is a constant and the
// second term is dropped), g = U without normalization.  The difference is
// written as the fused operation: left to the compiler, which of the two
// products it fuses depends on the code around, and where the terms cancel
// (one candidate: g is their rounding alone) kernels would disagree.
template <int J>
__device__ __forceinline__ void norm_backward_row(const VarArgs& a, const float (&th)[J], const double (&U)[J],
                                                  double mu, bool clamped, float (&g)[J])
{
    if (a.mode == 1) {
        const double ut = row_sum<J>([&](int j) { return U[j] * (double)th[j]; });
        const double inv_mu = 1.0 / mu;
        const double corr = clamped ? 0.0 : ut * inv_mu * inv_mu * a.inv_n;
#pragma unroll
        for (int j = 0; j < J; ++j) g[j] = (float)__builtin_fma(U[j], inv_mu, -corr);
    } else {
#pragma unroll
        for (int j = 0; j < J; ++j) g[j] = (float)U[j];
    }
}

// Store of one gradient entry: the whole [V][N], or the selected candidates'
// columns only, [V][g_nsel] in their order.
__device__ __forceinline__ void store_g(const VarArgs& a, uint32_t v, uint32_t i, float g)
{
    if (!a.g_slot) {
        a.g_out[(size_t)v * a.N + i] = g;
        return;
    }
    const int32_t q = a.g_slot[i];
    if (q >= 0) a.g_out[(size_t)v * a.g_nsel + q] = g;
}

// Everything after U: stores of U (adjoint op), Eq. 5 backward, stores of g
// (gradient op), AdamW, witness, new row mean, re-binarization (step op).
template <int J, int OP>
__device__ __forceinline__ void var_tail(const VarArgs& a, const StepScalars& c, uint32_t v, uint32_t lane,
                                         float (&th)[J], const float (&mm0)[J], const float (&vv0)[J],
                                         const bool (&valid)[J], double mu, bool clamped, const double (&U)[J],
                                         const uint64_t (&oP)[J], int witness, int wcand, int& bad)
{
    const int N = a.N;
    if (OP == OP_ADJ || OP == OP_GRAD) {
        if (a.U_out) {
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (valid[j]) a.U_out[(size_t)v * N + 64 * j + lane] = (float)U[j];
        }
        if (OP == OP_ADJ) { // without the Eq. 5 normalization the gradient is U
            if (a.g_out) {
#pragma unroll
                for (int j = 0; j < J; ++j)
                    if (valid[j]) store_g(a, v, 64u * j + lane, (float)U[j]);
            }
            return;
        }
    }
    float g[J];
    norm_backward_row<J>(a, th, U, mu, clamped, g);
    if (OP == OP_GRAD) {
        if (a.g_out) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                if (!valid[j]) continue;
                const int i = 64 * j + lane;
                store_g(a, v, (uint32_t)i, g[j]);
            }
        }
        return;
    }
    // AdamW (decoupled weight decay), FP32 with FP64-derived scalars
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const size_t idx = (size_t)v * N + 64 * j + lane;
        float t = th[j] * c.f_decay;
        const float mm = c.b1 * mm0[j] + c.omb1 * g[j];
        const float vv = c.b2 * vv0[j] + c.omb2 * (g[j] * g[j]);
        // hardware square root and reciprocal (1 ulp each)
        const float denom = __builtin_amdgcn_sqrtf(vv) * c.f_isbc2 + c.eps;
        t = t - c.f_step * (mm * __builtin_amdgcn_rcpf(denom));
        th[j] = valid[j] ? t : 0.f;
        if (valid[j]) {
            if (!(__builtin_isfinite(t) && __builtin_isfinite(mm) && __builtin_isfinite(vv))) bad = 1;
            __builtin_nontemporal_store(t, a.theta + idx); // non-temporal: see load_row
            __builtin_nontemporal_store(mm, a.m + idx);
            __builtin_nontemporal_store(vv, a.v + idx);
        }
    }
    if (witness && lane == 0 && !a.lit_rows) a.witness[v] = (uint8_t)((oP[wcand >> 6] >> (wcand & 63)) & 1u);
    bool pos = true;
    if (a.mode == 1) {
        const double mu2 = row_sum<J>([&](int j) { return (double)th[j]; }) * a.inv_n;
        if (lane == 0) a.mu_next[v] = mu2;
        pos = mu2 >= 0.0; // the clamp maps a zero mean to +1e-12
    }
    write_bits<J>(a, v, lane, th, valid, pos);
}

// After a stop (stop_on_sat), the step kernel keeps the next bit buffer and
// row means equal to the current ones so the host's buffer swap stays valid.
__device__ __forceinline__ void copy_bits_on_stop(const VarArgs& a)
{
    const size_t n = (size_t)(a.lit_rows ? 1 : 2) * a.V * a.W; // rows of literals
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) a.lits_next[e] = a.lits_cur[e];
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < (size_t)a.V; e += stride)
        a.mu_next[e] = a.mu_cur[e];
}

// A variable of an instance frozen on a satisfying candidate keeps its bits
// and row mean (the next buffers get the current ones) and is not updated.
template <int J>
__device__ __forceinline__ void keep_variable(const VarArgs& a, uint32_t v, uint32_t lane)
{
    const int W = a.W;
    const int nw = a.lit_rows ? W : 2 * W; // words of the variable's (or literal's) rows
    if (lane < (uint32_t)nw) {
        const size_t e = (size_t)(a.lit_rows ? v : 2 * v) * W + lane;
        a.lits_next[e] = a.lits_cur[e];
    }
    if (lane == 0) a.mu_next[v] = a.mu_cur[v];
}

struct VarInst {
    uint32_t inst;
    bool frozen;
    int witness, wcand;
};

template <int OP>
__device__ __forceinline__ VarInst var_instance(const VarArgs& a, uint32_t v)
{
    VarInst r;
    r.inst = a.var_inst ? sload(a.var_inst + v) : 0u;
    r.frozen = false;
    r.witness = 0;
    r.wcand = 0;
    if (OP == OP_STEP && a.ictrl) {
        const InstCtrl* ic = a.ictrl + r.inst;
        r.frozen = sload(&ic->frozen) != 0;
        r.witness = sload(&ic->witness_pending);
        r.wcand = sload(&ic->sat_cand);
    }
    return r;
}

template <int OP>
__device__ __forceinline__ VarInst instance_state(const VarArgs& a, uint32_t inst)
{
    VarInst r;
    r.inst = inst;
    r.frozen = false;
    r.witness = 0;
    r.wcand = 0;
    if (OP == OP_STEP && a.ictrl) {
        const InstCtrl* ic = a.ictrl + inst;
        r.frozen = sload(&ic->frozen) != 0;
        r.witness = sload(&ic->witness_pending);
        r.wcand = sload(&ic->sat_cand);
    }
    return r;
}

// The update kernel advances the iteration index once all of it has run
// (the next kernel on the stream sees it).
__device__ __forceinline__ void advance_step(const VarArgs& a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctrl->t += 1;
        a.ctrl->updates += 1;
    }
}

// Assignment mixing at a learning-rate restart (the mixing paragraph of
// Sec. IV-A and its equation): in every variable row, each candidate other
// than its instance's best one i* (most satisfied clauses at this
// iteration's forward pass, lower index on ties) becomes the average of
// itself and i*; the AdamW moments restart from zero; the new row means and
// bits follow.  Replaces the gradient step of the iteration; one wave per
// variable, every variable (heavy ones included).
template <int J>
__device__ void mix_rows(const VarArgs& a)
{
    const uint32_t lane = __lane_id(), wpb = blockDim.x / 64u;
    const uint32_t wave0 = uniform(blockIdx.x * wpb + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * wpb);
    const int N = a.N, W = a.W;
    for (uint32_t v = wave0; v < (uint32_t)a.V; v += nwaves) {
        const VarInst vi = var_instance<OP_STEP>(a, v);
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            continue;
        }
        const int32_t best = a.ictrl ? (int32_t)uniform((uint32_t)sload(&a.ictrl[vi.inst].best_cand)) : 0;
        const float* row = a.theta + (size_t)v * N;
        const double star = (double)row[best]; // same address in every lane
        float th[J];
        bool valid[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = 64 * j + (int)lane;
            valid[j] = i < N;
            float x = valid[j] ? __builtin_nontemporal_load(row + i) : 0.f;
            if (valid[j] && i != best) x = (float)(0.5 * ((double)x + star));
            th[j] = x;
            if (valid[j]) {
                const size_t idx = (size_t)v * N + i;
                __builtin_nontemporal_store(x, a.theta + idx);
                __builtin_nontemporal_store(0.f, a.m + idx);
                __builtin_nontemporal_store(0.f, a.v + idx);
            }
        }
        if (vi.witness && lane == 0 && !a.lit_rows) {
            const uint64_t w = a.lits_cur[(size_t)(2 * v) * W + (vi.wcand >> 6)];
            a.witness[v] = (uint8_t)((w >> (vi.wcand & 63)) & 1u);
        }
        bool pos = true;
        if (a.mode == 1) {
            const double mu2 = row_sum<J>([&](int j) { return (double)th[j]; }) * a.inv_n;
            if (lane == 0) a.mu_next[v] = mu2;
            pos = mu2 >= 0.0;
        }
        write_bits<J>(a, v, lane, th, valid, pos);
    }
    advance_step(a);
}

// theta -> row means and literal rows (initialization, set_logits/state).
// A wave takes R consecutive variables, all their loads in flight before the
// first row sum: one row at a time leaves a wave waiting for memory and then
// for the sum's lane exchanges in turn (V = 4e5, N = 256, 410 MB: 207 us at
// R = 1, 136 at R = 4, 3.4 TB/s with the rows written; 8 the same).
template <int J, int R>
__global__ __launch_bounds__(256) void binarize_kernel(VarArgs a)
{
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    for (uint32_t v0 = wave0 * R; v0 < (uint32_t)a.V; v0 += nwaves * R) {
        float th[R][J];
        bool valid[J];
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int i = 64 * j + (int)lane;
                valid[j] = i < a.N;
                th[q][j] = valid[j] && v0 + q < (uint32_t)a.V ? a.theta[(size_t)(v0 + q) * a.N + i] : 0.f;
            }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint32_t v = v0 + q;
            if (R > 1 && v >= (uint32_t)a.V) break; // wave-uniform
            bool pos = true;
            if (a.mode == 1) {
                // the same arithmetic as the update's new row mean, so that a
                // state set from a checkpoint binarizes exactly as the run did
                const double mu = row_sum<J>([&](int j) { return (double)th[q][j]; }) * a.inv_n;
                if (lane == 0) a.mu_next[v] = mu;
                pos = mu >= 0.0;
            } else if (lane == 0) {
                a.mu_next[v] = 1.0;
            }
            write_bits<J>(a, v, lane, th[q], valid, pos);
            if (a.vbits_out || a.assign_out) {
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const bool b = valid[j] && (pos ? th[q][j] > 0.f : th[q][j] < 0.f);
                    const uint64_t bal = ballot64(b);
                    if (a.vbits_out && j < a.W && lane == 0) a.vbits_out[(size_t)v * a.W + j] = bal;
                    if (a.assign_out && valid[j]) a.assign_out[(size_t)v * a.N + 64 * j + lane] = b ? 1.f : 0.f;
                }
            }
        }
    }
}

// Eq. 5 backward of caller arrays (device-pointer API): g from theta and
// dA = dL/d(theta_norm), the gradient the straight-through estimator passes
// through Eq. 2.  The row mean is formed exactly as binarize_kernel forms it.
template <int J>
__global__ __launch_bounds__(256) void norm_backward_kernel(VarArgs a)
{
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    for (uint32_t v = wave0; v < (uint32_t)a.V; v += nwaves) {
        float th[J];
        double U[J];
        bool valid[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = 64 * j + (int)lane;
            valid[j] = i < a.N;
            th[j] = valid[j] ? a.theta[(size_t)v * a.N + i] : 0.f;
            U[j] = valid[j] ? (double)a.dA_in[(size_t)v * a.N + i] : 0.0;
        }
        bool clamped = false;
        const double mu =
            a.mode == 1 ? clamp_mu(row_sum<J>([&](int j) { return (double)th[j]; }) * a.inv_n, clamped) : 1.0;
        float g[J];
        norm_backward_row<J>(a, th, U, mu, clamped, g);
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (valid[j]) a.g_out[(size_t)v * a.N + 64 * j + lane] = g[j];
    }
}

// Generic widths: records (k-1, the other k-1 literal indices), the dL/dR
// table in LDS indexed by R, FP64 accumulation.
template <int J, int OP, bool MULTI>
__global__ __launch_bounds__(256) void var_kernel(VarArgs a)
{
    extern __shared__ float s_tbl[]; // [K1][Np] (one instance)
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    if (!MULTI) {
        const int nt = a.K1 * a.Np;
        for (int q = threadIdx.x; q < nt; q += blockDim.x) s_tbl[q] = a.tbl[q];
        __syncthreads();
    }
    const uint32_t lane = __lane_id();
    // 256-thread blocks: 4 waves each (kept uniform so the compiler holds
    // the variable index in SGPRs and issues scalar loads)
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const int W = a.W, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    const char* lit_base = (const char*)a.lits_cur;
    const uint32_t row_bytes = (uint32_t)W * 8u;
    int bad = 0;

    for (uint32_t v = wave0; v < (uint32_t)a.V; v += nwaves) {
        if (a.heavy && sload(a.heavy + v)) continue; // the chunk kernels own it
        const VarInst vi = var_instance<OP>(a, v);
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            continue;
        }
        const float* tg = a.tbl + (size_t)vi.inst * a.K1 * Np; // this instance's table (MULTI)
        float th[J], mm[J], vv[J];
        bool valid[J];
        load_row<J, OP>(a, v, lane, th, mm, vv, valid);
        bool clamped = false;
        const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
        // own literal rows (buffers carry 16 words of padding: J-word reads stay in bounds)
        const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * W;
        uint64_t oP[J], oN[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            oP[j] = sload(ownp + j);
            oN[j] = sload(ownp + W + j);
        }
        // FP64 accumulation: the error stays at the table's FP32 rounding
        // whatever the variable's degree
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) U[j] = 0.0;
        uint32_t q = sload(a.occ_off + v);
        const uint32_t qm = sload(a.occ_mid + v), qe = sload(a.occ_off + v + 1);
        while (q < qe) {
            const bool neg = q >= qm;
            const uint32_t k1 = sload(a.occ_data + q);
            uint32_t R[J];
#pragma unroll
            for (int j = 0; j < J; ++j) R[j] = add_lane_bit(0u, neg ? oN[j] : oP[j]);
            for (uint32_t e = 0; e < k1; ++e) {
                const uint32_t off = sload(a.occ_data + q + 1 + e) * row_bytes;
                const uint64_t* row = (const uint64_t*)(lit_base + off);
#pragma unroll
                for (int j = 0; j < J; ++j) R[j] = add_lane_bit(R[j], sload(row + j));
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                if (j >= W) break;
                const int ti = R[j] * Np + 64 * j + lane;
                const double val = (double)(MULTI ? tg[ti] : s_tbl[ti]);
                U[j] = neg ? U[j] - val : U[j] + val;
            }
            q += 1 + k1;
        }
        var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// Generic records over the forward's bytes of R (the stores and candidate
// counts without clause planes: clauses wider than 15, or mixed widths at
// N > 256): a record is its clause's index, the wave loads R of its
// candidates (64 bytes per word and record, B records in flight), looks up
// dL/dR in the table and adds in FP64, record by record in var_kernel's order
// and so with its results.  A record's sign multiplies its entry inside the
// fused sum.  What bounds it is latency: a record's row is a random 64 W-byte
// read, hubs are long chains of them (cut into the heavy variables' chunks,
// which run first, beside the other variables).  V = 4e4, 2e5 clauses of
// widths 2 .. 24, N = 100: adjoint 70 us; the row gather 211 + 100 for the
// heavy chunks' launch before it.  16 records in flight and doubled 105 us,
// 4 67.  var_kernel, which gathers the k - 1 other literal
// rows of every record through the scalar cache and counts them, remains for
// stores whose bytes would not fit and with the clause planes off.
template <int J, int B, class T>
__device__ __forceinline__ void bytes_records(const VarArgs& a, uint32_t q, uint32_t qm, uint32_t qe, uint32_t lane,
                                              T table, double (&U)[J])
{
    const int W = a.W;
    const uint32_t stride = 64u * (uint32_t)W;
    // lanes past the candidates read the last one's byte: those beyond the
    // forward's dwords hold nothing
    uint32_t col[J];
#pragma unroll
    for (int j = 0; j < J; ++j) col[j] = min(64u * j + lane, (uint32_t)a.N - 1u);
    for (uint32_t base = q; base < qe; base += 64) { // wave-uniform
        // the next 64 records' clauses in one load, lane by lane
        const uint32_t n = qe - base < 64u ? qe - base : 64u;
        const uint64_t rows = (uint64_t)a.occ_cid[base + min(lane, n - 1u)] * stride;
        const uint32_t rlo = (uint32_t)rows, rhi = (uint32_t)(rows >> 32);
        uint32_t nx[B][J];
        auto load = [&](uint32_t i0) {
#pragma unroll
            for (int i = 0; i < B; ++i) { // past the end: the last record's row again
                const int at = (int)min(i0 + i, n - 1u);
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)rlo, at);
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)rhi, at);
                const uint8_t* row = a.rb + (((uint64_t)hi << 32) | lo);
#pragma unroll
                for (int j = 0; j < J; ++j) nx[i][j] = j < W ? row[col[j]] : 0u;
            }
        };
        load(0);
        for (uint32_t i0 = 0; i0 < n; i0 += B) {
            // the next batch is in flight while this one is added
            uint32_t R[B][J];
#pragma unroll
            for (int i = 0; i < B; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) R[i][j] = nx[i][j];
            if (i0 + B < n) load(i0 + B);
#pragma unroll
            for (int i = 0; i < B; ++i) {
                if (i0 + i >= n) break;
                // +-1 times the entry, fused: the sum itself
                const double sg = base + i0 + i >= qm ? -1.0 : 1.0;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    if (j >= W) break;
                    const double val = (double)table[__umul24(R[i][j], (uint32_t)a.Np) + 64 * j + lane];
                    U[j] = __builtin_fma(sg, val, U[j]);
                }
            }
        }
    }
}

// records in flight per wave
template <int J> constexpr int bytes_batch() { return J <= 2 ? 8 : 16 / J; }

template <int J, int OP, bool MULTI>
__global__ __launch_bounds__(256) void var_bytes_kernel(VarArgs a)
{
    extern __shared__ float s_tbl[]; // [K1][Np] (one instance)
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    if (!MULTI) {
        const int nt = a.K1 * a.Np;
        for (int q = threadIdx.x; q < nt; q += blockDim.x) s_tbl[q] = a.tbl[q];
        __syncthreads();
    }
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const StepScalars c = load_scalars(a, OP);
    int bad = 0;
    // the chunks of the heavy variables first (the longest items), then the
    // variables
    const uint32_t nch = a.heavy ? (uint32_t)a.n_chunks : 0u;
    for (uint32_t it = wave0; it < nch + (uint32_t)a.V; it += nwaves) {
        if (it < nch) {
            const uint32_t v = sload(a.ch_var + it);
            const VarInst vi = var_instance<OP>(a, v);
            double U[J];
#pragma unroll
            for (int j = 0; j < J; ++j) U[j] = 0.0;
            if (!vi.frozen) {
                const uint32_t q = sload(a.ch_rbeg + it), qm = sload(a.cid_mid + v), qe = sload(a.ch_rend + it);
                if constexpr (MULTI) bytes_records<J, bytes_batch<J>()>(a, q, qm, qe, lane, a.tbl + (size_t)vi.inst * a.K1 * a.Np, U);
                else bytes_records<J, bytes_batch<J>()>(a, q, qm, qe, lane, (const float*)s_tbl, U);
            }
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (j < a.W) a.partial[(size_t)it * a.Np + 64 * j + lane] = U[j];
            continue;
        }
        const uint32_t v = it - nch;
        if (a.heavy && sload(a.heavy + v)) continue; // its chunks' sums meet in the tail kernel
        const VarInst vi = var_instance<OP>(a, v);
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            continue;
        }
        float th[J], mm[J], vv[J];
        bool valid[J];
        load_row<J, OP>(a, v, lane, th, mm, vv, valid);
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) U[j] = 0.0;
        const uint32_t q = sload(a.cid_off + v), qm = sload(a.cid_mid + v), qe = sload(a.cid_off + v + 1);
        if constexpr (MULTI) bytes_records<J, bytes_batch<J>()>(a, q, qm, qe, lane, a.tbl + (size_t)vi.inst * a.K1 * a.Np, U);
        else bytes_records<J, bytes_batch<J>()>(a, q, qm, qe, lane, (const float*)s_tbl, U);
        bool clamped = false;
        const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
        const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * a.W;
        uint64_t oP[J];
#pragma unroll
        for (int j = 0; j < J; ++j) oP[j] = OP == OP_STEP ? sload(ownp + j) : 0ull;
        var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// Heavy variables of generic stores.  Chunk kernel: one wave per chunk of a
// heavy variable's records sums their table entries (same arithmetic as the
// generic kernel) into an FP64 partial row.  Tail kernel: one wave per heavy
// variable adds its partials in chunk order and runs the tail.
template <int J, int OP>
__global__ __launch_bounds__(256) void var_heavy_part_kernel(VarArgs a)
{
    if (OP == OP_STEP && (a.ctrl->stop || a.ctrl->mixing)) return; // the main kernel covers both
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const int W = a.W, Np = a.Np;
    const char* lit_base = (const char*)a.lits_cur;
    const uint32_t row_bytes = (uint32_t)W * 8u;
    for (uint32_t ch = wave0; ch < (uint32_t)a.n_chunks; ch += nwaves) {
        const uint32_t v = sload(a.ch_var + ch);
        const VarInst vi = var_instance<OP>(a, v);
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) U[j] = 0.0;
        if (!vi.frozen) {
            const float* tg = a.tbl + (size_t)vi.inst * a.K1 * Np;
            const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * W;
            uint64_t oP[J], oN[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                oP[j] = sload(ownp + j);
                oN[j] = sload(ownp + W + j);
            }
            uint32_t q = sload(a.ch_beg + ch);
            const uint32_t qe = sload(a.ch_end + ch), qm = sload(a.occ_mid + v);
            while (q < qe) {
                const bool neg = q >= qm;
                const uint32_t k1 = sload(a.occ_data + q);
                uint32_t R[J];
#pragma unroll
                for (int j = 0; j < J; ++j) R[j] = add_lane_bit(0u, neg ? oN[j] : oP[j]);
                for (uint32_t e = 0; e < k1; ++e) {
                    const uint32_t off = sload(a.occ_data + q + 1 + e) * row_bytes;
                    const uint64_t* row = (const uint64_t*)(lit_base + off);
#pragma unroll
                    for (int j = 0; j < J; ++j) R[j] = add_lane_bit(R[j], sload(row + j));
                }
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    if (j >= W) break;
                    const double val = (double)tg[R[j] * Np + 64 * j + lane];
                    U[j] = neg ? U[j] - val : U[j] + val;
                }
                q += 1 + k1;
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (j < W) a.partial[(size_t)ch * Np + 64 * j + lane] = U[j];
    }
}

template <int J, int OP>
__global__ __launch_bounds__(256) void var_heavy_tail_kernel(VarArgs a)
{
    if (OP == OP_STEP && (a.ctrl->stop || a.ctrl->mixing)) return; // the main kernel covers both
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const int W = a.W, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    int bad = 0;
    for (uint32_t h = wave0; h < (uint32_t)a.n_heavy; h += nwaves) {
        const uint32_t v = sload(a.hv_var + h);
        const VarInst vi = var_instance<OP>(a, v);
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            continue;
        }
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) U[j] = 0.0;
        const uint32_t c0 = sload(a.hv_chunk + h), c1 = sload(a.hv_chunk + h + 1);
        for (uint32_t ch = c0; ch < c1; ++ch) {
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (j < W) U[j] += a.partial[(size_t)ch * Np + 64 * j + lane];
        }
        float th[J], mm[J], vv[J];
        bool valid[J];
        load_row<J, OP>(a, v, lane, th, mm, vv, valid);
        bool clamped = false;
        const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
        const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * W;
        uint64_t oP[J];
#pragma unroll
        for (int j = 0; j < J; ++j) oP[j] = sload(ownp + j);
        var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
    }
    if (OP == OP_STEP && ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
}

// ---------------------------------------------------------------------------
// Batched scalar-memory gathers.  Scalar loads return out of order, so a
// wave can only wait for all of its outstanding ones at once; the gather of
// a variable's occurrence records is therefore cut into as few batches as
// the scalar registers allow, each one inline-assembly statement that issues
// its loads and waits inside it (the compiler can neither re-issue the loads
// later nor read their registers before they arrive).
// ---------------------------------------------------------------------------

typedef uint32_t sv2 __attribute__((ext_vector_type(2)));
typedef uint32_t sv4 __attribute__((ext_vector_type(4)));
typedef uint32_t sv8 __attribute__((ext_vector_type(8)));
typedef uint32_t sv16 __attribute__((ext_vector_type(16)));

// scalar registers holding the first J 64-bit words of a literal row
template <int J> struct RowVec;
template <> struct RowVec<1> { typedef sv2 T; };
template <> struct RowVec<2> { typedef sv4 T; };
template <> struct RowVec<4> { typedef sv8 T; };

#define TSAT_ROWS8(OPC)                                                                                      \
    asm volatile(OPC " %0, %8, %9\n\t" OPC " %1, %8, %10\n\t" OPC " %2, %8, %11\n\t" OPC " %3, %8, %12\n\t" \
                 OPC " %4, %8, %13\n\t" OPC " %5, %8, %14\n\t" OPC " %6, %8, %15\n\t" OPC " %7, %8, %16\n\t" \
                 "s_waitcnt lgkmcnt(0)"                                                                      \
                 : "=&s"(r[0]), "=&s"(r[1]), "=&s"(r[2]), "=&s"(r[3]), "=&s"(r[4]), "=&s"(r[5]), "=&s"(r[6]),   \
                   "=&s"(r[7])                                                                               \
                 : "s"(base), "s"(off[0]), "s"(off[1]), "s"(off[2]), "s"(off[3]), "s"(off[4]), "s"(off[5]),     \
                   "s"(off[6]), "s"(off[7]))

// eight literal rows at byte offsets off[] from base, in one round trip
template <int J>
__device__ __forceinline__ void smem_rows8(uint64_t base, const uint32_t (&off)[8], typename RowVec<J>::T (&r)[8])
{
    if constexpr (J == 1) TSAT_ROWS8("s_load_dwordx2");
    else if constexpr (J == 2) TSAT_ROWS8("s_load_dwordx4");
    else TSAT_ROWS8("s_load_dwordx8");
}
#undef TSAT_ROWS8

// sixteen words at byte offset off from base, in one round trip
__device__ __forceinline__ sv16 smem_words16(uint64_t base, uint32_t off)
{
    sv16 r;
    asm volatile("s_load_dwordx16 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&s"(r) : "s"(base), "s"(off));
    return r;
}

// The first sixteen code words of a variable's positive and negative
// records, and the record offsets of the next variable, in one round trip.
// Also the FP64 row mean of the variable and the instance index of the next
// variable, so that no other scalar round trip precedes the record batches.
__device__ __forceinline__ void smem_var_start(uint64_t occ, uint32_t off_pos, uint32_t off_neg, uint64_t offs,
                                               uint64_t mids, uint32_t off_next, uint64_t mu_base, uint32_t off_mu,
                                               uint64_t inst_base, sv16& cp, sv16& cn, sv2& rn, uint32_t& mn,
                                               sv2& mu, uint32_t& inst_next)
{
    asm volatile("s_load_dwordx16 %0, %6, %7\n\t"
                 "s_load_dwordx16 %1, %6, %8\n\t"
                 "s_load_dwordx2 %2, %9, %11\n\t"
                 "s_load_dword %3, %10, %11\n\t"
                 "s_load_dwordx2 %4, %12, %13\n\t"
                 "s_load_dword %5, %14, %11\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(cp), "=&s"(cn), "=&s"(rn), "=&s"(mn), "=&s"(mu), "=&s"(inst_next)
                 : "s"(occ), "s"(off_pos), "s"(off_neg), "s"(offs), "s"(mids), "s"(off_next), "s"(mu_base),
                   "s"(off_mu), "s"(inst_base));
}

template <int J>
__device__ __forceinline__ uint64_t row_word(const typename RowVec<J>::T& r, int j)
{
    return (uint64_t)r[2 * j] | ((uint64_t)r[2 * j + 1] << 32);
}

template <int KO>
__device__ __forceinline__ void cum_masks(const uint64_t (&w)[KO], uint64_t (&ge)[KO])
{
#pragma unroll
    for (int o = 0; o < KO; ++o) ge[o] = 0;
#pragma unroll
    for (int e = 0; e < KO; ++e) {
#pragma unroll
        for (int o = KO - 1; o >= 1; --o) ge[o] |= ge[o - 1] & w[e];
        ge[0] |= w[e];
    }
}

template <int J, int KO, int G, int OP, bool FULL>
__device__ __forceinline__ void var_pure_body(const VarArgs& a);

// Uniform-width update kernels.  The batched gather needs its scalar
// registers; the grouped one fits eight waves per SIMD with rows of up to
// four words.  Longer rows hold more than the 64 registers that leaves: at
// eight waves they spill (850 to 900 registers of the step's 16-word rows), so
// they get the registers of four waves (8 words), three, or two for the step
// (16 words).  V = 1e5, 3-SAT, N = 1000: update 5.96 ms at eight waves, 2.02
// at four, 1.76 at three, 1.29 at two; adjoint 0.80, 0.50, 0.51, 0.64;
// N = 300: update 0.88, 0.69 at six, 0.64 at five, 0.36 at four.
template <int J, int OP>
constexpr int pure_waves()
{
    return J <= 4 ? 8 : (J <= 8 ? 4 : (OP == OP_STEP ? 2 : 3));
}

template <int J, int KO, int G, int OP, bool FULL>
__global__ __launch_bounds__(256) void var_pure_kernel(VarArgs a)
{
    var_pure_body<J, KO, G, OP, FULL>(a);
}

template <int J, int KO, int G, int OP, bool FULL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pure_waves<J, OP>(), 8))) void var_pure8_kernel(
    VarArgs a)
{
    var_pure_body<J, KO, G, OP, FULL>(a);
}

// Row-gather update for uniform widths: every clause has the same width
// k = KO + 1 (KO other literals per record, no header).  Occurrences are
// taken G records at a time: all their literal rows are requested through
// the scalar cache before the first wait (the buffers are padded, so the
// loads need no guards; records past the end of the variable are masked
// out).  Per candidate and sign, integer counters c_o = #{occurrences whose
// other literals hold >= o true ones} (o = 1..KO) are accumulated from
// bit-sliced cumulative masks; n_O = c_O - c_{O+1} (c_0 = degree) counts the
// occurrences with exactly O other literals true, so a positive one has
// R = x + O and a negative one R = 1 - x + O (x the candidate's own value),
// and U = sum over r of (positive - negative occurrences with R = r) g[r].
template <int J, int KO, int G, int OP, bool FULL>
__device__ __forceinline__ void var_pure_body(const VarArgs& a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const int W = a.W, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    const char* lit_base = (const char*)a.lits_cur;
    const uint32_t row_bytes = (uint32_t)W * 8u;
    constexpr int K1 = KO + 2; // R in 0..KO+1
    // dL/dR table for the lane's candidates: in lane-private LDS slots for up
    // to four candidate words (registers are kept for the prefetched row)
    constexpr bool GT_LDS = J <= 4;
    __shared__ float s_gt[4][GT_LDS ? K1 * J * 64 : 1];
    float gt[GT_LDS ? 1 : K1][J];
    float* my_gt = s_gt[threadIdx.x / 64u];
    uint32_t gt_inst = 0xffffffffu;
    int bad = 0;
    // G = 4 selects the batched scalar-memory gather (rows of up to four words)
    constexpr bool BATCHED = G == 4 && J <= 4;
    const uint64_t lit_u64 = uniform64((uint64_t)a.lits_cur);
    const uint64_t occ_base = uniform64((uint64_t)a.occ_data);
    const uint64_t offs_base = uniform64((uint64_t)a.occ_off);
    const uint64_t mids_base = uniform64((uint64_t)a.occ_mid);
    // record offsets and instance of the wave's current variable (prefetched
    // one variable ahead), and the state of the last instance seen
    uint32_t b_r0 = 0, b_rm = 0, b_r1 = 0, b_inst = 0;
    const uint64_t mu_base = uniform64((uint64_t)(a.mu_cur ? a.mu_cur : (const double*)a.occ_off));
    const uint64_t inst_base = uniform64((uint64_t)(a.var_inst ? a.var_inst : a.occ_mid));
    VarInst vic = instance_state<OP>(a, 0u);
    if (BATCHED && wave0 < (uint32_t)a.V) {
        b_r0 = sload(a.occ_off + wave0);
        b_rm = sload(a.occ_mid + wave0);
        b_r1 = sload(a.occ_off + wave0 + 1);
        b_inst = a.var_inst ? sload(a.var_inst + wave0) : 0u;
    }

    // theta, m, v of the wave's next variable, loaded one variable ahead so
    // that their latency hides behind the current variable's gather
    constexpr bool PREFETCH = false;
    float th_n[J], mm_n[J], vv_n[J];
    bool valid_n[J];
    if (PREFETCH && wave0 < (uint32_t)a.V) load_row<J, OP, FULL>(a, wave0, lane, th_n, mm_n, vv_n, valid_n);

    for (uint32_t v = wave0; v < (uint32_t)a.V; v += nwaves) {
        float th[J], mm[J], vv[J];
        bool valid[J];
        if constexpr (PREFETCH) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                th[j] = th_n[j];
                mm[j] = mm_n[j];
                vv[j] = vv_n[j];
                valid[j] = valid_n[j];
            }
            if (v + nwaves < (uint32_t)a.V) load_row<J, OP, FULL>(a, v + nwaves, lane, th_n, mm_n, vv_n, valid_n);
        } else {
            load_row<J, OP, FULL>(a, v, lane, th, mm, vv, valid);
        }
        VarInst vi;
        if constexpr (BATCHED) {
            if (a.var_inst && b_inst != vic.inst) vic = instance_state<OP>(a, b_inst);
            vi = vic;
        } else {
            vi = var_instance<OP>(a, v);
        }
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            if (BATCHED) {
                const uint32_t vn = min(v + nwaves, (uint32_t)a.V - 1u);
                b_r0 = sload(a.occ_off + vn);
                b_rm = sload(a.occ_mid + vn);
                b_r1 = sload(a.occ_off + vn + 1);
                b_inst = a.var_inst ? sload(a.var_inst + vn) : 0u;
            }
            continue;
        }
        if (vi.inst != gt_inst) {
            // the dL/dR table of this instance for the lane's candidates
            gt_inst = vi.inst;
            const float* tg = a.tbl + (size_t)vi.inst * K1 * Np;
#pragma unroll
            for (int r = 0; r < K1; ++r)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const float x = (j < W) ? tg[(size_t)r * Np + 64 * j + lane] : 0.f;
                    if constexpr (GT_LDS) my_gt[(r * J + j) * 64 + lane] = x;
                    else gt[r][j] = x;
                }
        }
        bool clamped = false;
        const bool need_mu = !(OP == OP_ADJ || a.mode != 1);
        double mu = 1.0;
        if (!BATCHED && need_mu) mu = clamp_mu(sload(a.mu_cur + v), clamped);
        const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * W;
        uint64_t oP[J];
        if constexpr (BATCHED) {
            // the own row through the vector path, off the scalar round trips
            uint32_t zv;
            asm volatile("v_mov_b32 %0, 0" : "=v"(zv));
#pragma unroll
            for (int j = 0; j < J; ++j) oP[j] = ownp[j + zv];
        } else {
#pragma unroll
            for (int j = 0; j < J; ++j) oP[j] = sload(ownp + j);
        }
        uint32_t cnt[2][KO][J];
#pragma unroll
        for (int sg = 0; sg < 2; ++sg)
#pragma unroll
            for (int o = 0; o < KO; ++o)
#pragma unroll
                for (int j = 0; j < J; ++j) cnt[sg][o][j] = 0;
        const uint32_t r0 = BATCHED ? b_r0 : sload(a.occ_off + v);
        const uint32_t rm = BATCHED ? b_rm : sload(a.occ_mid + v);
        const uint32_t r1 = BATCHED ? b_r1 : sload(a.occ_off + v + 1);
        if constexpr (BATCHED) {
            // record counts per chunk of code words and per batch of eight rows
            constexpr int RPC = 16 / KO, RB = 8 / KO;
            const uint32_t vn = min(v + nwaves, (uint32_t)a.V - 1u);
            sv16 cfirst[2];
            sv2 rn, mub;
            uint32_t mn, inst_n;
            smem_var_start(occ_base, r0 * (uint32_t)(4 * KO), rm * (uint32_t)(4 * KO), offs_base, mids_base,
                           vn * 4u, mu_base, need_mu ? v * 8u : 0u, inst_base, cfirst[0], cfirst[1], rn, mn, mub,
                           inst_n);
            if (need_mu)
                mu = clamp_mu(__longlong_as_double((long long)((uint64_t)mub[0] | ((uint64_t)mub[1] << 32))),
                              clamped);
#pragma unroll
            for (int sg = 0; sg < 2; ++sg) {
                const uint32_t beg = sg ? rm : r0, end = sg ? r1 : rm;
                for (uint32_t c0 = beg; c0 < end; c0 += RPC) {
                    const sv16 ck = (c0 == beg) ? cfirst[sg] : smem_words16(occ_base, c0 * (uint32_t)(4 * KO));
#pragma unroll
                    for (int b = 0; b < (RPC + RB - 1) / RB; ++b) {
                        const uint32_t q0 = c0 + (uint32_t)(b * RB);
                        if (q0 >= end) break; // wave-uniform
                        uint32_t off[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            const int rec = b * RB + t / KO;
                            const bool use = t < RB * KO && rec < RPC && q0 + (uint32_t)(t / KO) < end;
                            off[t] = use ? ck[rec * KO + t % KO] * row_bytes : 0u;
                        }
                        typename RowVec<J>::T rows[8];
                        smem_rows8<J>(lit_u64, off, rows);
#pragma unroll
                        for (int g = 0; g < RB; ++g) {
                            const bool live = b * RB + g < RPC && q0 + (uint32_t)g < end; // wave-uniform
#pragma unroll
                            for (int j = 0; j < J; ++j) {
                                uint64_t wj[KO], ge[KO];
#pragma unroll
                                for (int e = 0; e < KO; ++e) wj[e] = row_word<J>(rows[g * KO + e], j);
                                cum_masks<KO>(wj, ge);
#pragma unroll
                                for (int o = 0; o < KO; ++o)
                                    cnt[sg][o][j] = add_lane_bit(cnt[sg][o][j], live ? ge[o] : 0ull);
                            }
                        }
                    }
                }
            }
            b_r0 = rn[0];
            b_r1 = rn[1];
            b_rm = mn;
            b_inst = a.var_inst ? inst_n : 0u;
        }
        if constexpr (!BATCHED) {
#pragma unroll
        for (int sg = 0; sg < 2; ++sg) {
            const uint32_t beg = sg ? rm : r0, end = sg ? r1 : rm;
            // the codes of the next group are requested with the rows of the
            // current one: one scalar-memory round trip per group
            uint32_t code_next[G][KO];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < KO; ++e) code_next[g][e] = sload(a.occ_data + (size_t)(beg + g) * KO + e);
            for (uint32_t q = beg; q < end; q += G) {
                uint32_t code[G][KO];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < KO; ++e) code[g][e] = code_next[g][e];
                uint64_t w[G][KO][J];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < KO; ++e) {
                        const uint64_t* row = (const uint64_t*)(lit_base + code[g][e] * row_bytes);
#pragma unroll
                        for (int j = 0; j < J; ++j) w[g][e][j] = sload(row + j);
                    }
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < KO; ++e) code_next[g][e] = sload(a.occ_data + (size_t)(q + G + g) * KO + e);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const bool live = q + g < end; // wave-uniform
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        uint64_t wj[KO], ge[KO];
#pragma unroll
                        for (int e = 0; e < KO; ++e) wj[e] = w[g][e][j];
                        cum_masks<KO>(wj, ge);
#pragma unroll
                        for (int o = 0; o < KO; ++o) cnt[sg][o][j] = add_lane_bit(cnt[sg][o][j], live ? ge[o] : 0ull);
                    }
                }
            }
        }
        }
        const uint32_t dp = rm - r0, dn = r1 - rm;
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            // own value of this lane's candidate
            const uint32_t x = BATCHED ? (uint32_t)(oP[j] >> lane) & 1u : add_lane_bit(0u, oP[j]);
            // records with exactly O other literals true, per sign; a
            // positive occurrence has R = x + O, a negative one R = 1 - x + O
            int32_t np[KO + 1], nn[KO + 1];
#pragma unroll
            for (int O = 0; O <= KO; ++O) {
                np[O] = (int32_t)(((O == 0) ? dp : cnt[0][O - 1][j]) - ((O < KO) ? cnt[0][O][j] : 0u));
                nn[O] = (int32_t)(((O == 0) ? dn : cnt[1][O - 1][j]) - ((O < KO) ? cnt[1][O][j] : 0u));
            }
            float u = 0.f;
#pragma unroll
            for (int r = 0; r <= KO + 1; ++r) {
                const int32_t ep = x ? (r >= 1 ? np[r - 1] : 0) : (r <= KO ? np[r] : 0);
                const int32_t en = x ? (r <= KO ? nn[r] : 0) : (r >= 1 ? nn[r - 1] : 0);
                const float t = GT_LDS ? my_gt[(r * J + j) * 64 + lane] : gt[GT_LDS ? 0 : r][j];
                u = fmaf((float)(ep - en), t, u);
            }
            U[j] = (double)u;
        }
        var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// A half of a window's 64-bit word.  The words were stored as such by the same
// lane: without the attribute the compiler may move the loads of halves ahead
// of the stores, as types that cannot alias.
typedef uint32_t __attribute__((may_alias)) half_word;

// Counts of the window gathers.  cnt[r - 1][j] collects, for candidate
// 64 j + lane and level r, (positive - negative records whose clause has
// R >= r) + (negative records): with the positive records' window bits in mp
// and the negative ones' in mn, popc((G & (mp | mn)) ^ mn) = popc(G & mp) +
// |mn| - popc(G & mn), one bitwise operation and one popcount per level and
// dword.  (A popcount per sign, packed in 16-bit halves, took ten
// instructions per level and word; the instruction stream is a large share
// of these kernels' time: V = 4e5, N = 256 gradient 359 -> 326 us, large
// update 1320 -> 1302, N = 1000 update 358 -> 345.)
// T: the window's words, or the dwords of one half of them.
template <int J, int KW, typename T>
__device__ __forceinline__ void count_planes(const T (&b0)[J], const T (&b1)[J], T mp, T mn, uint32_t (&cnt)[KW][J])
{
    const T m = mp | mn;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const T ge[3] = {b0[j] | b1[j], b1[j], b0[j] & b1[j]}; // R >= 1, R >= 2, R = 3
#pragma unroll
        for (int r = 0; r < KW; ++r) {
            const T x = (ge[r] & m) ^ mn;
            if constexpr (sizeof(T) == 8) cnt[r][j] += (uint32_t)__popcll(x);
            else cnt[r][j] += (uint32_t)__popc(x);
        }
    }
}

// the records of one variable in the wave's window (win[(p J + j) 64 + lane])
template <int J, int KW>
__device__ __forceinline__ void count_window(const uint64_t* win, uint32_t lane, uint64_t mp, uint64_t mn,
                                             uint32_t (&cnt)[KW][J])
{
    const uint64_t m = mp | mn;
    if ((uint32_t)(m >> 32) == 0u || (uint32_t)m == 0u) { // wave-uniform
        // they lie in one 32-bit half (most do): count on its dwords only
        const uint32_t hf = (uint32_t)m == 0u ? 1u : 0u;
        const half_word* win32 = reinterpret_cast<const half_word*>(win);
        uint32_t b0[J], b1[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            b0[j] = win32[2 * (j * 64 + lane) + hf];
            b1[j] = win32[2 * ((J + j) * 64 + lane) + hf];
        }
        count_planes<J, KW, uint32_t>(b0, b1, (uint32_t)(mp >> (32u * hf)), (uint32_t)(mn >> (32u * hf)), cnt);
    } else {
        uint64_t b0[J], b1[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            b0[j] = win[j * 64 + lane];
            b1[j] = win[(J + j) * 64 + lane];
        }
        count_planes<J, KW, uint64_t>(b0, b1, mp, mn, cnt);
    }
}

// U of one variable row from these counts: dp / dn are the record counts and
// my_gt the lane-private dL/dR table ([r][j][lane]).  U = sum over r of
// (positive - negative records with R = r) dL/dR[r], in the order of r as in
// the other uniform-width gathers, so that every gather gives identical
// results.
template <int J, int KW>
__device__ __forceinline__ void plane_u(const uint32_t (&cnt)[KW][J], uint32_t dp, uint32_t dn, const float* my_gt,
                                        uint32_t lane, double (&U)[J])
{
#pragma unroll
    for (int j = 0; j < J; ++j) {
        float u = 0.f;
#pragma unroll
        for (int r = 0; r <= KW; ++r) {
            const int32_t d = (int32_t)(r == 0 ? dp : cnt[r - 1][j]) - (int32_t)(r < KW ? cnt[r][j] : dn);
            u = fmaf((float)d, my_gt[(r * J + j) * 64 + lane], u);
        }
        U[j] = (double)u;
    }
}

// Lane-private copy of an instance's dL/dR table, [r][j][lane].
template <int J, int K1>
__device__ __forceinline__ void load_gt(const VarArgs& a, uint32_t inst, float* my_gt, uint32_t lane)
{
    const float* tg = a.tbl + (size_t)inst * K1 * a.Np;
#pragma unroll
    for (int r = 0; r < K1; ++r)
#pragma unroll
        for (int j = 0; j < J; ++j) my_gt[(r * J + j) * 64 + lane] = (j < a.W) ? tg[(size_t)r * a.Np + 64 * j + lane] : 0.f;
}

// ---------------------------------------------------------------------------
// Uniform-width update with the clause-plane gather (widths 2 and 3).
//
// The forward pass leaves R of every clause in binary (two bit planes per
// candidate row), so the adjoint of Sec. III-B needs no other literal rows:
// U_vi = sum over the positive occurrences of dL/dR_i[R_ci] minus the same
// over the negative ones.  Per record the wave gathers one clause's planes
// (2 J words through the scalar cache) and counts, per candidate and sign,
// the records with R >= r as carry-in masks of v_addc; U is formed from the
// exact counts and the dL/dR table.  The rest is the tail shared with the
// other update kernels.
// ---------------------------------------------------------------------------
template <int J, int KW, int OP, bool FULL>
// seven waves per SIMD: the register budget of eight would spill to scratch
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7, 8))) void var_plane_kernel(VarArgs a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    constexpr int G = 2;       // records per scalar-load group
    constexpr int K1 = KW + 1; // R in 0..KW
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t nwaves = uniform(gridDim.x * 4u);
    const int W = a.W, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    const char* plane_base = (const char*)a.planes;
    constexpr uint32_t plane_bytes = 16u * J; // two planes of J words
    __shared__ float s_gt[4][K1 * J * 64];
    float* my_gt = s_gt[threadIdx.x / 64u];
    uint32_t gt_inst = 0xffffffffu;
    int bad = 0;

    for (uint32_t v = wave0; v < (uint32_t)a.V; v += nwaves) {
        const VarInst vi = var_instance<OP>(a, v);
        if (vi.frozen) {
            keep_variable<J>(a, v, lane);
            continue;
        }
        if (vi.inst != gt_inst) {
            gt_inst = vi.inst;
            const float* tg = a.tbl + (size_t)vi.inst * K1 * Np;
#pragma unroll
            for (int r = 0; r < K1; ++r)
#pragma unroll
                for (int j = 0; j < J; ++j)
                    my_gt[(r * J + j) * 64 + lane] = (j < W) ? tg[(size_t)r * Np + 64 * j + lane] : 0.f;
        }
        float th[J], mm[J], vv[J];
        bool valid[J];
        load_row<J, OP, FULL>(a, v, lane, th, mm, vv, valid);
        bool clamped = false;
        const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
        uint32_t cnt[2][KW][J];
#pragma unroll
        for (int sg = 0; sg < 2; ++sg)
#pragma unroll
            for (int r = 0; r < KW; ++r)
#pragma unroll
                for (int j = 0; j < J; ++j) cnt[sg][r][j] = 0;
        const uint32_t r0 = sload(a.occ_off + v), rm = sload(a.occ_mid + v), r1 = sload(a.occ_off + v + 1);
#pragma unroll
        for (int sg = 0; sg < 2; ++sg) {
            const uint32_t beg = sg ? rm : r0, end = sg ? r1 : rm;
            // the clause indices of the next group come with the planes of
            // the current one (the index array is padded past its end)
            uint32_t id_next[G];
#pragma unroll
            for (int g = 0; g < G; ++g) id_next[g] = sload(a.occ_cid + beg + g);
            for (uint32_t q = beg; q < end; q += G) {
                uint32_t id[G];
#pragma unroll
                for (int g = 0; g < G; ++g) id[g] = id_next[g];
                uint64_t w[G][2][J];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint64_t* pl = (const uint64_t*)(plane_base + (size_t)id[g] * plane_bytes);
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int j = 0; j < J; ++j) w[g][p][j] = sload(pl + p * J + j);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) id_next[g] = sload(a.occ_cid + q + G + g);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const bool live = q + g < end; // wave-uniform
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        const uint64_t b0 = live ? w[g][0][j] : 0ull, b1 = live ? w[g][1][j] : 0ull;
                        cnt[sg][0][j] = add_lane_bit(cnt[sg][0][j], b0 | b1); // R >= 1
                        cnt[sg][1][j] = add_lane_bit(cnt[sg][1][j], b1);      // R >= 2
                        if constexpr (KW == 3) cnt[sg][2][j] = add_lane_bit(cnt[sg][2][j], b0 & b1); // R = 3
                    }
                }
            }
        }
        const uint32_t dp = rm - r0, dn = r1 - rm;
        // U as in the other uniform-width gathers (identical results): the
        // sum over r of (positive - negative records with R = r) dL/dR[r]
        const uint64_t* ownp = a.lits_cur + (size_t)(2 * v) * W;
        uint64_t oP[J];
#pragma unroll
        for (int j = 0; j < J; ++j) oP[j] = sload(ownp + j);
        double U[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            float u = 0.f;
#pragma unroll
            for (int r = 0; r <= KW; ++r) {
                const uint32_t p_ge = r == 0 ? dp : cnt[0][r - 1][j], p_gt = r < KW ? cnt[0][r][j] : 0u;
                const uint32_t n_ge = r == 0 ? dn : cnt[1][r - 1][j], n_gt = r < KW ? cnt[1][r][j] : 0u;
                const int32_t d = (int32_t)(p_ge - p_gt) - (int32_t)(n_ge - n_gt);
                u = fmaf((float)d, my_gt[(r * J + j) * 64 + lane], u);
            }
            U[j] = (double)u;
        }
        var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// ---------------------------------------------------------------------------
// Clause-plane update by record windows (uniform widths 2 and 3).
//
// The same counts as var_plane_kernel, gathered through the vector memory
// path: a wave owns a chunk of consecutive variables, whose occurrence
// records are consecutive too, and takes them 64 at a time: lane r loads
// record r's clause index (one coalesced load) and that clause's planes (one
// random 16 J-byte load per lane), then each of the 2 J plane words is
// transposed across the wave (a 64 x 64 bit matrix: afterwards lane l holds,
// per word, one bit per record for candidate 64 j + l).  A variable's counts
// are popcounts of these words under the mask of its records' window bits;
// a variable whose records run past the window takes the next window and
// adds.  Every record is loaded once.  U and the tail are those of
// var_plane_kernel, so the results are identical.
// ---------------------------------------------------------------------------

// 64 x 64 bit-matrix transposes across the wave, E matrices at once: lane i
// holds row i of each (bit c is element (i, c)); afterwards lane c holds
// column c (bit i is element (i, c)).  A transpose exchanges lane-index bit
// k with column-index bit k for k = 5 .. 0, all on the VALU (no LDS round
// trips), every stage applied to the E words before the next:
//  - bit 5 (the 32-bit half of the word): v_permlane32_swap trades the upper
//    lanes' low dwords for the lower lanes' high dwords, which is exactly
//    that exchange;
//  - bit 4: v_permlane16_swap makes the same trade between odd and even
//    16-lane rows, so the 16-bit halves are first moved so that column bit 4
//    selects the dword (one byte permute per dword), swapped, and moved back;
//  - bit 3 (a byte within a 16-bit half): the partner lane i ^ 8 is a
//    rotation of the 16-lane row by 8 (DPP), and one byte permute keeps this
//    lane's bytes and inserts the partner's;
//  - bits 2, 1, 0: the partner's dword arrives through DPP (lane i ^ 4 as
//    two shifts by 4 within the row, each written to half of the banks;
//    i ^ 2 and i ^ 1 as quad permutations); the lane with bit k clear keeps
//    its columns with bit k clear and takes the partner's ones rotated up by
//    2^k, the other keeps the columns with bit k set and takes the partner's
//    rotated down (the wrapped bits fall under the kept mask).
template <int E>
__device__ __forceinline__ void transpose64_n(uint64_t (&x)[E], uint32_t lane)
{
    uint32_t lo[E], hi[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        lo[e] = (uint32_t)x[e];
        hi[e] = (uint32_t)(x[e] >> 32);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const auto r = __builtin_amdgcn_permlane32_swap(lo[e], hi[e], false, false);
        lo[e] = r[0];
        hi[e] = r[1];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        // low halves to lo, high halves to hi; swap; and back
        const uint32_t a = __builtin_amdgcn_perm(hi[e], lo[e], 0x05040100u);
        const uint32_t b = __builtin_amdgcn_perm(hi[e], lo[e], 0x07060302u);
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        lo[e] = __builtin_amdgcn_perm(r[1], r[0], 0x05040100u);
        hi[e] = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
    }
    {
        // bytes (own 0, partner 0, own 2, partner 2) or (partner 1, own 1, partner 3, own 3)
        const uint32_t sel = (lane & 8u) ? 0x03070105u : 0x06020400u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t tl = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo[e], 0x128, 0xF, 0xF, false);
            const uint32_t th = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi[e], 0x128, 0xF, 0xF, false);
            lo[e] = __builtin_amdgcn_perm(tl, lo[e], sel);
            hi[e] = __builtin_amdgcn_perm(th, hi[e], sel);
        }
    }
    {
        const bool up = lane & 4u;
        const uint32_t keep = up ? 0xF0F0F0F0u : 0x0F0F0F0Fu, rot = up ? 4u : 28u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            // banks 0 and 2 of a row read lane i + 4, banks 1 and 3 lane i - 4
            uint32_t tl = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo[e], 0x104, 0xF, 0x5, false);
            tl = (uint32_t)__builtin_amdgcn_update_dpp((int)tl, (int)lo[e], 0x114, 0xF, 0xA, false);
            uint32_t th = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi[e], 0x104, 0xF, 0x5, false);
            th = (uint32_t)__builtin_amdgcn_update_dpp((int)th, (int)hi[e], 0x114, 0xF, 0xA, false);
            lo[e] = (keep & lo[e]) | (~keep & __builtin_amdgcn_alignbit(tl, tl, rot));
            hi[e] = (keep & hi[e]) | (~keep & __builtin_amdgcn_alignbit(th, th, rot));
        }
    }
    {
        const bool up = lane & 2u;
        const uint32_t keep = up ? 0xCCCCCCCCu : 0x33333333u, rot = up ? 2u : 30u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t tl = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo[e], 0x4E, 0xF, 0xF, false); // [2,3,0,1]
            const uint32_t th = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi[e], 0x4E, 0xF, 0xF, false);
            lo[e] = (keep & lo[e]) | (~keep & __builtin_amdgcn_alignbit(tl, tl, rot));
            hi[e] = (keep & hi[e]) | (~keep & __builtin_amdgcn_alignbit(th, th, rot));
        }
    }
    {
        const bool up = lane & 1u;
        const uint32_t keep = up ? 0xAAAAAAAAu : 0x55555555u, rot = up ? 1u : 31u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t tl = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo[e], 0xB1, 0xF, 0xF, false); // [1,0,3,2]
            const uint32_t th = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi[e], 0xB1, 0xF, 0xF, false);
            lo[e] = (keep & lo[e]) | (~keep & __builtin_amdgcn_alignbit(tl, tl, rot));
            hi[e] = (keep & hi[e]) | (~keep & __builtin_amdgcn_alignbit(th, th, rot));
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = ((uint64_t)hi[e] << 32) | lo[e];
}

// Planes of records [w, w + 64) (records at or past `end` read as zero),
// transposed into the wave's LDS window: win[(p J + j) 64 + lane] bit r =
// plane p, word j, candidate bit of record w + r.  Each lane writes its own
// slots; a caller whose lanes read other lanes' slots orders the stores
// before those loads itself.
template <int J>
__device__ __forceinline__ void load_window(const VarArgs& a, uint32_t w, uint32_t end, uint32_t lane, uint64_t* win)
{
    const uint32_t rec = w + lane;
    const bool ok = rec < end;
    const uint32_t id = ok ? a.occ_cid[rec] : 0u;
    const uint4* pl = (const uint4*)a.planes + (size_t)id * J; // 2 J words: [plane][word]
    uint64_t wd[2 * J];
#pragma unroll
    for (int k = 0; k < J; ++k) {
        const uint4 q = ok ? pl[k] : make_uint4(0u, 0u, 0u, 0u);
        wd[2 * k] = ((uint64_t)q.y << 32) | q.x;
        wd[2 * k + 1] = ((uint64_t)q.w << 32) | q.z;
    }
    transpose64_n<2 * J>(wd, lane);
#pragma unroll
    for (int e = 0; e < 2 * J; ++e) win[e * 64 + lane] = wd[e];
}

// Packed planes (N <= 32: plane 0 of a clause in the low dword of one 8-byte
// word, plane 1 in the high one) of records [w, w + 64) (records at or past
// `end` read as zero), transposed into the wave's LDS window: one transpose
// serves both planes, win[c] bit r = plane 0, candidate c of record w + r and
// win[32 + c] bit r = plane 1, candidate c, for c < 32.
__device__ __forceinline__ void load_window_packed(const VarArgs& a, uint32_t w, uint32_t end, uint32_t lane,
                                                   uint64_t* win)
{
    const uint32_t rec = w + lane;
    const bool ok = rec < end;
    const uint32_t id = ok ? a.occ_cid[rec] : 0u;
    const uint2 q = ok ? ((const uint2*)a.planes)[id] : make_uint2(0u, 0u);
    uint64_t wd[1] = {((uint64_t)q.y << 32) | q.x};
    transpose64_n<1>(wd, lane);
    win[lane] = wd[0];
}

// bits [lo, hi) of a 64-bit word, 0 <= lo < hi <= 64
__device__ __forceinline__ uint64_t bit_range(uint32_t lo, uint32_t hi)
{
    const uint64_t below_hi = hi >= 64u ? ~0ull : ((1ull << hi) - 1ull);
    return below_hi & ~((1ull << lo) - 1ull);
}

template <int J, int KW, int OP, bool FULL>
__global__ __launch_bounds__(256) void var_window_kernel(VarArgs a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    constexpr int K1 = KW + 1;     // R in 0..KW
    const uint32_t kChunk = a.chunk; // variables per wave work item
    const uint32_t lane = __lane_id();
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t V = (uint32_t)a.V;
    const int W = a.W;
    const StepScalars c = load_scalars(a, OP);
    // each wave keeps the dL/dR table of the instance at hand (one table
    // shared by the block measured slower: the higher occupancy it allows
    // does not pay)
    __shared__ float s_gt[4][K1 * J * 64];
    __shared__ uint64_t s_win[4][2 * J * 64]; // each wave's transposed record window
    float* my_gt = s_gt[threadIdx.x / 64u];
    uint64_t* my_win = s_win[threadIdx.x / 64u];
    uint32_t gt_inst = 0xffffffffu;
    int bad = 0;
    const uint32_t nchunks = (V + kChunk - 1) / kChunk;

    const ItemRange cr = xcd_items(a.xcd, nchunks, 4u, wave0 % 4u);
    for (uint32_t ch = cr.first; ch < cr.end; ch += cr.stride) {
        const uint32_t vb = ch * kChunk, ve = vb + kChunk < V ? vb + kChunk : V;
        const uint32_t rend = sload(a.occ_off + ve); // end of the chunk's records
        uint32_t w = 0;                              // window [w, w + 64), once loaded
        bool loaded = false;
        for (uint32_t v = vb; v < ve; ++v) {
            const VarInst vi = var_instance<OP>(a, v);
            if (vi.frozen) {
                keep_variable<J>(a, v, lane);
                continue;
            }
            if (vi.inst != gt_inst) {
                gt_inst = vi.inst;
                load_gt<J, K1>(a, vi.inst, my_gt, lane);
            }
            const uint32_t r0 = sload(a.occ_off + v), rm = sload(a.occ_mid + v), r1 = sload(a.occ_off + v + 1);
            uint32_t cnt[KW][J];
#pragma unroll
            for (int r = 0; r < KW; ++r)
#pragma unroll
                for (int j = 0; j < J; ++j) cnt[r][j] = 0;
            for (uint32_t q = r0; q < r1;) { // wave-uniform
                if (!loaded || q - w >= 64u) {
                    w = q;
                    loaded = true;
                    load_window<J>(a, w, rend, lane, my_win);
                }
                const uint32_t hi = r1 < w + 64u ? r1 : w + 64u;
                const uint64_t mp = q < rm ? bit_range(q - w, (hi < rm ? hi : rm) - w) : 0ull;
                const uint64_t mn = hi > rm ? bit_range((q > rm ? q : rm) - w, hi - w) : 0ull;
                count_window<J, KW>(my_win, lane, mp, mn, cnt);
                q = hi;
            }
            float th[J], mm[J], vv[J];
            bool valid[J];
            load_row<J, OP, FULL>(a, v, lane, th, mm, vv, valid);
            bool clamped = false;
            const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
            const uint64_t* ownp = a.lits_cur + (size_t)(a.lit_rows ? v : 2 * v) * W;
            uint64_t oP[J];
#pragma unroll
            for (int j = 0; j < J; ++j) oP[j] = sload(ownp + j);
            double U[J];
            plane_u<J, KW>(cnt, rm - r0, r1 - rm, my_gt, lane, U);
            var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
        }
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// ---------------------------------------------------------------------------
// Window gather for rows of more than four words (256 < N <= 1024): a block
// is a team of ceil(W / 4) waves, each holding four words (256 candidates)
// of the rows, so that a wave keeps the window, table and registers of
// var_window_kernel<4>.  The team takes three consecutive variables at a
// time: every wave requests its share of their rows, counts their records,
// and the two row sums of each variable (Eq. 5 backward, new mean) are added
// over the team in LDS, all three variables between the same two barriers
// (three 358 us, two 376, four 381 before the one-popcount counts).
//
// What bounds it: the theta, m, v streams and a plane row per record (V =
// 5e4, C = 2.05e5, N = 1000: 1.2 GB and 0.16 GB a launch, 345 us = 3.9 TB/s,
// a copy of 5.1).  The row gather of var_pure_kernel, which these sizes take
// without the planes, reads two literal rows of 128 bytes per record through
// the scalar cache, one wave per variable: 660 us.
// ---------------------------------------------------------------------------

// Planes of records [w, w + 64) as load_window<4>, of the four words from
// word0 of clauses holding `words` words per plane.
__device__ __forceinline__ void load_window_part(const VarArgs& a, uint32_t w, uint32_t end, uint32_t lane,
                                                 uint32_t words, uint32_t word0, uint64_t* win)
{
    const uint32_t rec = w + lane;
    const bool ok = rec < end;
    const uint32_t id = ok ? a.occ_cid[rec] : 0u;
    const uint64_t* pl = (const uint64_t*)a.planes + (size_t)id * (2u * words) + word0;
    uint64_t wd[8];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint4 q = ok ? ((const uint4*)(pl + p * words))[k] : make_uint4(0u, 0u, 0u, 0u);
            wd[4 * p + 2 * k] = ((uint64_t)q.y << 32) | q.x;
            wd[4 * p + 2 * k + 1] = ((uint64_t)q.w << 32) | q.z;
        }
    transpose64_n<8>(wd, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) win[e * 64 + lane] = wd[e];
}

template <int KW, int OP>
__global__ __launch_bounds__(256) void var_window_team_kernel(VarArgs a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<16>(a);
        return;
    }
    constexpr int K1 = KW + 1, J = 4;
    constexpr int C = 3; // variables per team pass
    const uint32_t lane = __lane_id();
    const uint32_t wv = uniform(threadIdx.x / 64u), G = blockDim.x / 64u;
    const uint32_t word0 = wv * J; // first word of this wave's share
    const uint32_t V = (uint32_t)a.V;
    const int W = a.W, N = a.N, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    __shared__ float s_gt[4][K1 * J * 64];
    __shared__ uint64_t s_win[4][2 * J * 64];
    __shared__ double s_ut[C][4], s_mu[C][4]; // the waves' shares of the row sums
    float* my_gt = s_gt[wv];
    uint64_t* my_win = s_win[wv];
    uint32_t gt_inst = 0xffffffffu;
    int bad = 0;
    bool valid[J];
#pragma unroll
    for (int j = 0; j < J; ++j) valid[j] = (int)(64u * (word0 + j) + lane) < N;
    const bool sums = OP != OP_ADJ && a.mode == 1;
    const uint32_t nchunks = (V + C - 1) / C;
    for (uint32_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) { // block-uniform
        const uint32_t vb = ch * C, nv = V - vb < C ? V - vb : C;
        const uint32_t rend = sload(a.occ_off + vb + nv);
        float th[C][J], mm[C][J], vv[C][J], g[C][J];
        VarInst vi[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if ((uint32_t)i < nv) vi[i] = var_instance<OP>(a, vb + i);
            else vi[i].frozen = true;
            const size_t row = (size_t)(vb + i) * N + 64u * word0 + lane;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const bool ld = (uint32_t)i < nv && valid[j];
                th[i][j] = (OP != OP_ADJ && ld) ? __builtin_nontemporal_load(a.theta + row + 64 * j) : 0.f;
            }
        }
        uint32_t w = 0;
        bool loaded = false;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if ((uint32_t)i >= nv) break;
            const uint32_t v = vb + i;
            if (vi[i].frozen) {
                if (wv == 0) keep_variable<16>(a, v, lane);
                continue;
            }
            if (vi[i].inst != gt_inst) {
                gt_inst = vi[i].inst;
                const float* tg = a.tbl + (size_t)gt_inst * K1 * Np;
#pragma unroll
                for (int r = 0; r < K1; ++r)
#pragma unroll
                    for (int j = 0; j < J; ++j)
                        my_gt[(r * J + j) * 64 + lane] =
                            (int)word0 + j < W ? tg[(size_t)r * Np + 64u * (word0 + j) + lane] : 0.f;
            }
            const uint32_t r0 = sload(a.occ_off + v), rm = sload(a.occ_mid + v), r1 = sload(a.occ_off + v + 1);
            uint32_t cnt[KW][J];
#pragma unroll
            for (int r = 0; r < KW; ++r)
#pragma unroll
                for (int j = 0; j < J; ++j) cnt[r][j] = 0;
            for (uint32_t q = r0; q < r1;) { // wave-uniform
                if (!loaded || q - w >= 64u) {
                    w = q;
                    loaded = true;
                    load_window_part(a, w, rend, lane, 4u * G, word0, my_win);
                }
                const uint32_t hi = r1 < w + 64u ? r1 : w + 64u;
                const uint64_t mp = q < rm ? bit_range(q - w, (hi < rm ? hi : rm) - w) : 0ull;
                const uint64_t mn = hi > rm ? bit_range((q > rm ? q : rm) - w, hi - w) : 0ull;
                count_window<J, KW>(my_win, lane, mp, mn, cnt);
                q = hi;
            }
            double U[J];
            plane_u<J, KW>(cnt, rm - r0, r1 - rm, my_gt, lane, U);
#pragma unroll
            for (int j = 0; j < J; ++j) g[i][j] = (float)U[j]; // U is a float's value
            if (sums) {
                const double ut = row_sum<J>([&](int j) { return U[j] * (double)th[i][j]; });
                if (lane == 0) s_ut[i][wv] = ut;
            }
        }
        // the moments are requested here, not with theta: held through the
        // counting they cost registers (415 us; 358 this way)
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const size_t row = (size_t)(vb + i) * N + 64u * word0 + lane;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const bool ld = OP == OP_STEP && (uint32_t)i < nv && valid[j];
                mm[i][j] = ld ? __builtin_nontemporal_load(a.m + row + 64 * j) : 0.f;
                vv[i][j] = ld ? __builtin_nontemporal_load(a.v + row + 64 * j) : 0.f;
            }
        }
        if (sums) __syncthreads();
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (vi[i].frozen) continue;
            const uint32_t v = vb + i;
            const size_t row = (size_t)v * N + 64u * word0 + lane;
            if ((OP == OP_ADJ || OP == OP_GRAD) && a.U_out) {
#pragma unroll
                for (int j = 0; j < J; ++j)
                    if (valid[j]) a.U_out[row + 64 * j] = g[i][j];
            }
            if (OP == OP_ADJ) {
                if (a.g_out) {
#pragma unroll
                    for (int j = 0; j < J; ++j)
                        if (valid[j]) store_g(a, v, 64u * (word0 + j) + lane, g[i][j]);
                }
                continue;
            }
            if (a.mode == 1) {
                bool clamped;
                const double mu = clamp_mu(sload(a.mu_cur + v), clamped);
                double ut = s_ut[i][0];
                for (uint32_t k = 1; k < G; ++k) ut = ut + s_ut[i][k];
                const double inv_mu = 1.0 / mu;
                const double corr = clamped ? 0.0 : ut * inv_mu * inv_mu * a.inv_n;
#pragma unroll
                for (int j = 0; j < J; ++j) g[i][j] = (float)__builtin_fma((double)g[i][j], inv_mu, -corr);
            }
            if (OP == OP_GRAD) {
                if (a.g_out) {
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        if (!valid[j]) continue;
                        store_g(a, v, 64u * (word0 + j) + lane, g[i][j]);
                    }
                }
                continue;
            }
            // AdamW as in var_tail
#pragma unroll
            for (int j = 0; j < J; ++j) {
                float t = th[i][j] * c.f_decay;
                const float m2 = c.b1 * mm[i][j] + c.omb1 * g[i][j];
                const float v2 = c.b2 * vv[i][j] + c.omb2 * (g[i][j] * g[i][j]);
                const float denom = __builtin_amdgcn_sqrtf(v2) * c.f_isbc2 + c.eps;
                t = t - c.f_step * (m2 * __builtin_amdgcn_rcpf(denom));
                th[i][j] = valid[j] ? t : 0.f;
                if (valid[j]) {
                    if (!(__builtin_isfinite(t) && __builtin_isfinite(m2) && __builtin_isfinite(v2))) bad = 1;
                    __builtin_nontemporal_store(t, a.theta + row + 64 * j);
                    __builtin_nontemporal_store(m2, a.m + row + 64 * j);
                    __builtin_nontemporal_store(v2, a.v + row + 64 * j);
                }
            }
            if (vi[i].witness && wv == 0 && lane == 0) {
                const uint64_t own = a.lits_cur[(size_t)(2 * v) * W + (vi[i].wcand >> 6)];
                a.witness[v] = (uint8_t)((own >> (vi[i].wcand & 63)) & 1u);
            }
            if (a.mode == 1) {
                const double s2 = row_sum<J>([&](int j) { return (double)th[i][j]; });
                if (lane == 0) s_mu[i][wv] = s2;
            }
        }
        // the next pass writes s_ut only after every wave is past this
        // barrier, and s_mu only after its own first one
        if (sums) __syncthreads();
        if (OP != OP_STEP) continue;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (vi[i].frozen) continue;
            const uint32_t v = vb + i;
            bool pos = true;
            if (a.mode == 1) {
                double mu2 = s_mu[i][0];
                for (uint32_t k = 1; k < G; ++k) mu2 = mu2 + s_mu[i][k];
                mu2 = mu2 * a.inv_n;
                if (wv == 0 && lane == 0) a.mu_next[v] = mu2;
                pos = mu2 >= 0.0; // the clamp maps a zero mean to +1e-12
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint64_t bal = ballot64(valid[j] && (pos ? th[i][j] > 0.f : th[i][j] < 0.f));
                const uint64_t vm = ballot64(valid[j]);
                if (lane == 0 && (int)word0 + j < W) {
                    a.lits_next[(size_t)(2 * v) * W + word0 + j] = bal;
                    a.lits_next[(size_t)(2 * v + 1) * W + word0 + j] = ~bal & vm;
                }
            }
        }
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// ---------------------------------------------------------------------------
// Window gather with two variables per wave (N <= 32, rows of one word):
// lanes 0-31 hold the candidates of the first variable of a pair, lanes
// 32-63 those of the second.  The pair's records are consecutive, so one
// window loop covers both; the forward leaves a clause's two planes packed
// in one 8-byte word, one load and one transpose per record window; every
// lane reads the two transposed words of its candidate (lane mod 32) and
// counts under its own variable's record masks.
// The per-variable work of the tail (two FP64 row sums, the divisions,
// scalar loads, bit packing) is then shared by two rows.  Row sums stay
// within each half in the order of var_tail, where the idle half adds only
// zeros, so the results are those of var_window_kernel.
// ---------------------------------------------------------------------------

// var_tail<1, OP> for two rows, one per half wave (vl: this lane's variable,
// l: its candidate, live: the lane's variable is present and not frozen).
template <int OP>
__device__ __forceinline__ void pair_tail(const VarArgs& a, const StepScalars& c, uint32_t lane, uint32_t vl, uint32_t l,
                                          bool live, float th, float mm0, float vv0, bool valid, double mu,
                                          bool clamped, double U, uint64_t own, int witness, int wcand, int& bad)
{
    const size_t idx = (size_t)vl * a.N + l;
    if (OP == OP_ADJ || OP == OP_GRAD) {
        if (a.U_out && valid) a.U_out[idx] = (float)U;
        if (OP == OP_ADJ) {
            if (a.g_out && valid) store_g(a, vl, l, (float)U);
            return;
        }
    }
    float g;
    if (a.mode == 1) {
        double ut = 0.0;
        ut += U * (double)th;
        ut = half_sum(ut);
        const double inv_mu = 1.0 / mu;
        const double corr = clamped ? 0.0 : ut * inv_mu * inv_mu * a.inv_n;
        g = (float)__builtin_fma(U, inv_mu, -corr);
    } else {
        g = (float)U;
    }
    if (OP == OP_GRAD) {
        if (a.g_out && valid) {
            store_g(a, vl, l, g);
        }
        return;
    }
    float t = th * c.f_decay;
    const float mm = c.b1 * mm0 + c.omb1 * g;
    const float vv = c.b2 * vv0 + c.omb2 * (g * g);
    const float denom = __builtin_amdgcn_sqrtf(vv) * c.f_isbc2 + c.eps;
    t = t - c.f_step * (mm * __builtin_amdgcn_rcpf(denom));
    th = valid ? t : 0.f;
    if (valid) {
        if (!(__builtin_isfinite(t) && __builtin_isfinite(mm) && __builtin_isfinite(vv))) bad = 1;
        __builtin_nontemporal_store(t, a.theta + idx);
        __builtin_nontemporal_store(mm, a.m + idx);
        __builtin_nontemporal_store(vv, a.v + idx);
    }
    double s2 = 0.0;
    s2 += (double)th;
    if (witness && l == 0 && live) a.witness[vl] = (uint8_t)((own >> wcand) & 1u);
    bool pos = true;
    if (a.mode == 1) {
        const double mu2 = half_sum(s2) * a.inv_n;
        if (l == 0 && live) a.mu_next[vl] = mu2;
        pos = mu2 >= 0.0; // the clamp maps a zero mean to +1e-12
    }
    const uint64_t bal = ballot64(valid && (pos ? th > 0.f : th < 0.f));
    const uint64_t vm = ballot64(valid);
    if (l == 0 && live) {
        const uint32_t sh = lane & 32u;
        const uint64_t bp = (bal >> sh) & 0xffffffffull, bm = (vm >> sh) & 0xffffffffull;
        a.lits_next[2 * (size_t)vl] = bp;
        a.lits_next[2 * (size_t)vl + 1] = ~bp & bm;
    }
}

// records of [lo, hi) inside [q, qe) as bits of the window at w (0 if none)
__device__ __forceinline__ uint64_t window_bits(uint32_t lo, uint32_t hi, uint32_t q, uint32_t qe, uint32_t w)
{
    const uint32_t b = lo > q ? lo : q, e = hi < qe ? hi : qe;
    return b < e ? bit_range(b - w, e - w) : 0ull;
}

// Eight waves per SIMD: the compiler then keeps the kernel within 80 SGPRs
// (spilling some scalars to VGPR lanes); at 100 SGPRs it ran 7 (ragged
// 200-instance iteration 2.55 -> 2.46 ms).
template <int KW, int OP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void var_window_pair_kernel(VarArgs a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<1>(a);
        return;
    }
    constexpr int K1 = KW + 1;
    // variables (sixteen pairs) per wave work item: a chunk's last record
    // window is partly used, so longer chunks waste less of the window loads
    // (measured best of 4, 8, 16 and 32)
    constexpr uint32_t kChunk = 32;
    const uint32_t lane = __lane_id();
    const uint32_t h = lane >> 5, l = lane & 31u;
    const uint32_t wave0 = uniform(blockIdx.x * 4u + threadIdx.x / 64u);
    const uint32_t V = (uint32_t)a.V;
    const int N = a.N, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    __shared__ float s_gt[4][K1 * 64];
    __shared__ uint64_t s_win[4][64];
    float* my_gt = s_gt[threadIdx.x / 64u];
    uint64_t* my_win = s_win[threadIdx.x / 64u];
    uint32_t gt_inst0 = 0xffffffffu, gt_inst1 = 0xffffffffu;
    int bad = 0;
    const uint32_t nchunks = (V + kChunk - 1) / kChunk;

    const ItemRange cr = xcd_items(a.xcd, nchunks, 4u, wave0 % 4u);
    for (uint32_t ch = cr.first; ch < cr.end; ch += cr.stride) {
        const uint32_t vb = ch * kChunk, ve = vb + kChunk < V ? vb + kChunk : V;
        const uint32_t rend = sload(a.occ_off + ve);
        // variables of one instance are consecutive: a chunk whose first and
        // last variables share it takes the instance's state once
        const uint32_t inst_b = a.var_inst ? sload(a.var_inst + vb) : 0u;
        const uint32_t inst_e = a.var_inst ? sload(a.var_inst + ve - 1) : 0u;
        const bool one_inst = inst_b == inst_e;
        VarInst ci;
        if (one_inst) ci = instance_state<OP>(a, inst_b);
        uint32_t w = 0;
        bool loaded = false;
        for (uint32_t v0 = vb; v0 < ve; v0 += 2) {
            const uint32_t v1 = v0 + 1;
            const bool has1 = v1 < ve; // wave-uniform
            VarInst i0, i1;
            if (one_inst) {
                i0 = ci;
                i1 = ci;
            } else {
                i0 = var_instance<OP>(a, v0);
                i1 = i0;
                if (has1) i1 = var_instance<OP>(a, v1);
            }
            const bool live0 = !i0.frozen, live1 = has1 && !i1.frozen;
            const uint32_t vl = v0 + h;
            const bool present = h ? has1 : true, live = h ? live1 : live0;
            if (present && !live) { // a frozen variable keeps its bits and row mean
                if (l < 2u) a.lits_next[2 * (size_t)vl + l] = a.lits_cur[2 * (size_t)vl + l];
                if (l == 0u) a.mu_next[vl] = a.mu_cur[vl];
            }
            if (!live0 && !live1) continue;
            if (i0.inst != gt_inst0 || i1.inst != gt_inst1) {
                gt_inst0 = i0.inst;
                gt_inst1 = i1.inst;
                const float* tg = a.tbl + (size_t)(h ? i1.inst : i0.inst) * K1 * Np;
#pragma unroll
                for (int r = 0; r < K1; ++r) my_gt[r * 64 + lane] = tg[(size_t)r * Np + l];
            }
            const uint32_t a0 = sload(a.occ_off + v0), am = sload(a.occ_mid + v0), a1 = sload(a.occ_off + v1);
            uint32_t bm = a1, b1 = a1;
            if (has1) {
                bm = sload(a.occ_mid + v1);
                b1 = sload(a.occ_off + v1 + 1);
            }
            // a frozen variable's records are skipped by empty masks
            const uint32_t pa0 = live0 ? a0 : a1, pam = live0 ? am : a1, pa1 = a1;
            const uint32_t pb0 = live1 ? a1 : b1, pbm = live1 ? bm : b1, pb1 = b1;
            uint32_t cnt[KW][1];
#pragma unroll
            for (int r = 0; r < KW; ++r) cnt[r][0] = 0;
            for (uint32_t q = a0; q < b1;) { // wave-uniform
                if (!loaded || q - w >= 64u) {
                    w = q;
                    loaded = true;
                    load_window_packed(a, w, rend, lane, my_win);
                    // every lane reads slots other lanes wrote: order the LDS
                    // stores before those loads for the compiler and the wave
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
                const uint32_t qe = b1 < w + 64u ? b1 : w + 64u;
                const uint64_t mpa = window_bits(pa0, pam, q, qe, w), mna = window_bits(pam, pa1, q, qe, w);
                const uint64_t mpb = window_bits(pb0, pbm, q, qe, w), mnb = window_bits(pbm, pb1, q, qe, w);
                const uint64_t mp = h ? mpb : mpa, mn = h ? mnb : mna;
                const uint64_t b0[1] = {my_win[l]}, b1[1] = {my_win[32 + l]};
                count_planes<1, KW, uint64_t>(b0, b1, mp, mn, cnt);
                q = qe;
            }
            const bool valid = live && (int)l < N;
            const size_t idx = (size_t)vl * N + l;
            const float th = (OP != OP_ADJ && valid) ? __builtin_nontemporal_load(a.theta + idx) : 0.f;
            const float mm0 = (OP == OP_STEP && valid) ? __builtin_nontemporal_load(a.m + idx) : 0.f;
            const float vv0 = (OP == OP_STEP && valid) ? __builtin_nontemporal_load(a.v + idx) : 0.f;
            bool c0 = false, c1 = false;
            double mu0 = 1.0, mu1 = 1.0;
            if (OP != OP_ADJ && a.mode == 1) {
                mu0 = clamp_mu(sload(a.mu_cur + v0), c0);
                if (has1) mu1 = clamp_mu(sload(a.mu_cur + v1), c1);
            }
            const uint64_t o0 = sload(a.lits_cur + 2 * (size_t)v0);
            const uint64_t o1 = has1 ? sload(a.lits_cur + 2 * (size_t)v1) : 0ull;
            double U[1];
            plane_u<1, KW>(cnt, h ? bm - a1 : am - a0, h ? b1 - bm : a1 - am, my_gt, lane, U);
            pair_tail<OP>(a, c, lane, vl, l, live, th, mm0, vv0, valid, h ? mu1 : mu0, h ? c1 : c0, U[0],
                          h ? o1 : o0, h ? i1.witness : i0.witness, h ? i1.wcand : i0.wcand, bad);
        }
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// ---------------------------------------------------------------------------
// Clause-plane update by record windows for mixed widths (and uniform widths
// 1 and 4 .. 15).
//
// The forward leaves R of every clause in binary in P planes (P = 2 up to
// width 3, else 4), at the clause's global index.  A record is that index.
// As in var_window_kernel a wave takes a chunk of consecutive variables and
// their records 64 at a time: each lane loads one record's P J plane words,
// every word is transposed across the wave into the wave's LDS window, and
// a variable counts, per level r = 1 .. KT and candidate, its positive and
// negative records whose clause has R >= r (the comparison of the P-bit R
// with the constant r, bit-sliced over 64 records, then one popcount).
// U_vi = sum over r of (positive - negative records with R = r) dL/dR_i[r]
// (Sec. III-B: P^T dL/dR with the straight-through estimator), formed from
// these exact counts in the order of r; the tail is the one shared with the
// other update kernels.  A single-instance solver keeps one dL/dR table per
// block, a batch one per wave (the instance at hand).
// ---------------------------------------------------------------------------

// Thermometer of a bit-sliced R = sum_p 2^p pl[p] (P = 2 or 4 planes):
// ge[r - 1] = [R >= r] for r = 1 .. KT, built up bit by bit: the levels of
// the lower q bits give those of q + 1 bits as (new bit) OR (lower levels)
// below 2^q, the new bit itself at 2^q, and (new bit) AND (lower levels)
// above.  All are ORs and ANDs of the planes (no constant-true term), so
// planes masked to a record set give levels masked to that set.
template <int P, int KT, typename T = uint64_t>
__device__ __forceinline__ void thermometer(const T (&pl)[P], T (&ge)[KT])
{
    T lv[15]; // levels 1 .. 2^q - 1 of the lower q bits
    lv[0] = pl[0];
    int n = 1; // 2^q - 1
#pragma unroll
    for (int q = 1; q < P; ++q) {
        const T b = pl[q];
        T nx[15];
#pragma unroll
        for (int r = 1; r <= 15; ++r) {
            if (r > 2 * n + 1) break;
            if (r <= n) nx[r - 1] = b | lv[r - 1];
            else if (r == n + 1) nx[r - 1] = b;
            else nx[r - 1] = b & lv[r - n - 2];
        }
        n = 2 * n + 1;
#pragma unroll
        for (int r = 0; r < 15; ++r)
            if (r < n) lv[r] = nx[r];
    }
#pragma unroll
    for (int r = 0; r < KT; ++r) ge[r] = r < n ? lv[r] : T(0);
}

// Signed level counts of one variable in one window: with the records of
// its positive occurrences in mp and of its negative ones in mn (disjoint),
// popc(mn ^ (G & (mp | mn))) = popc(G & mp) + |mn| - popc(G & mn), so one
// popcount per level gives (positive - negative records with R >= r) + |mn|.
template <int P, int KT, typename T = uint64_t>
__device__ __forceinline__ void count_levels(const T (&pl)[P], T mp, T mn, uint32_t (&cnt)[KT])
{
    const T m = mp | mn;
    T pm[P];
#pragma unroll
    for (int p = 0; p < P; ++p) pm[p] = pl[p] & m;
    T ge[KT];
    thermometer<P, KT, T>(pm, ge);
#pragma unroll
    for (int r = 0; r < KT; ++r) {
        if constexpr (sizeof(T) == 8) cnt[r] += (uint32_t)__popcll(mn ^ ge[r]);
        else cnt[r] += (uint32_t)__popc(mn ^ ge[r]);
    }
}

// Planes of records [w, w + 64) (records at or past `end` read as zero),
// transposed into the wave's window: win[(p J + j) 64 + lane] bit r = plane
// p, word j, candidate bit of record w + r.  Lane-private slots.
template <int J, int P>
__device__ __forceinline__ void load_window_p(const VarArgs& a, uint32_t w, uint32_t end, uint32_t lane, uint64_t* win)
{
    constexpr int Q = P * J / 2; // 16-byte loads per record (P even)
    const uint32_t rec = w + lane;
    const bool ok = rec < end;
    const uint32_t id = ok ? a.occ_cid[rec] : 0u;
    // clauses below narrow_end (widths up to 3) hold two planes (the upper
    // two read as zero), the wider ones four, stored after them
    const bool narrow = P == 2 || id < a.narrow_end;
    const uint4* pl = narrow ? (const uint4*)a.planes + (size_t)id * J
                             : (const uint4*)a.planes + (size_t)a.narrow_end * J + (size_t)(id - a.narrow_end) * Q;
    uint64_t wd[P * J];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const bool ld = ok && (k < J || !narrow);
        const uint4 q = ld ? pl[k] : make_uint4(0u, 0u, 0u, 0u);
        wd[2 * k] = ((uint64_t)q.y << 32) | q.x;
        wd[2 * k + 1] = ((uint64_t)q.w << 32) | q.z;
    }
    // transposed four words at a time: the exchange temporaries of all
    // eight words at once would hold 16 more VGPRs, which cost a wave per
    // SIMD (structured configuration: 108 -> 94 VGPRs, 4 -> 5 waves, update
    // 0.647 -> 0.598 ms)
    constexpr int E = P * J, G = E > 4 ? 4 : E;
#pragma unroll
    for (int g0 = 0; g0 < E; g0 += G) {
        uint64_t part[G];
#pragma unroll
        for (int e = 0; e < G; ++e) part[e] = wd[g0 + e];
        transpose64_n<G>(part, lane);
#pragma unroll
        for (int e = 0; e < G; ++e) win[(g0 + e) * 64 + lane] = part[e];
    }
}

template <int J, int KT, int OP, bool FULL = false>
__global__ __launch_bounds__(256) void var_window_levels_kernel(VarArgs a)
{
    if (OP == OP_STEP && a.ctrl->stop) {
        copy_bits_on_stop(a);
        return;
    }
    if (OP == OP_STEP && a.ctrl->mixing) {
        mix_rows<J>(a);
        return;
    }
    constexpr int P = KT <= 3 ? 2 : 4;
    constexpr uint32_t kChunk = 4; // variables per wave work item
    const uint32_t lane = __lane_id(), wv = threadIdx.x / 64u;
    const uint32_t wave0 = uniform(blockIdx.x * 4u + wv);
    const uint32_t V = (uint32_t)a.V;
    const int W = a.W, K1 = a.K1, Np = a.Np;
    const StepScalars c = load_scalars(a, OP);
    // dynamic LDS: [4][P J 64] u64 windows, then the dL/dR table(s)
    // [KT + 1][J][64] f32 (rows at and past K1 zero), one per block (single
    // instance) or one per wave
    constexpr int KR = KT + 1;
    extern __shared__ uint64_t lds_lv[];
    uint64_t* my_win = lds_lv + (size_t)wv * (P * J * 64);
    float* gt_base = (float*)(lds_lv + 4 * P * J * 64);
    const bool per_wave = a.var_inst != nullptr;
    float* my_gt = gt_base + (per_wave ? (size_t)wv * KR * J * 64 : 0);
    uint32_t gt_inst = 0xffffffffu;
    if (!per_wave) {
        for (int e = threadIdx.x; e < KR * J * 64; e += 256) {
            const int r = e / (J * 64), j = (e / 64) % J, l = e % 64;
            my_gt[e] = (r < K1 && j < W) ? a.tbl[(size_t)r * Np + 64 * j + l] : 0.f;
        }
        __syncthreads();
        gt_inst = 0;
    }
    int bad = 0;
    // work items: the host's variable chunks that fill one record window
    // (fewer windows, so fewer transposes), else four variables each
    const uint32_t nchunks = a.vchunk ? (uint32_t)a.n_vchunk : (V + kChunk - 1) / kChunk;

    const ItemRange cr = xcd_items(a.xcd, nchunks, 4u, wave0 % 4u);
    for (uint32_t ch = cr.first; ch < cr.end; ch += cr.stride) {
        uint32_t vb, ve;
        if (a.vchunk) {
            vb = sload(a.vchunk + 2 * (size_t)ch);
            ve = sload(a.vchunk + 2 * (size_t)ch + 1);
        } else {
            vb = ch * kChunk;
            ve = vb + kChunk < V ? vb + kChunk : V;
        }
        const uint32_t rend = sload(a.cid_off + ve);
        uint32_t w = 0;
        bool loaded = false;
        for (uint32_t v = vb; v < ve; ++v) {
            const VarInst vi = var_instance<OP>(a, v);
            if (vi.frozen) {
                keep_variable<J>(a, v, lane);
                continue;
            }
            if (vi.inst != gt_inst) { // per-wave tables only
                gt_inst = vi.inst;
                const float* tg = a.tbl + (size_t)vi.inst * K1 * Np;
#pragma unroll
                for (int r = 0; r < KR; ++r)
#pragma unroll
                    for (int j = 0; j < J; ++j)
                        my_gt[(r * J + j) * 64 + lane] = (r < K1 && j < W) ? tg[(size_t)r * Np + 64 * j + lane] : 0.f;
            }
            const uint32_t r0 = sload(a.cid_off + v), rm = sload(a.cid_mid + v), r1 = sload(a.cid_off + v + 1);
            // per level r and word j: (positive - negative records with
            // R >= r) + (negative records), summed over the windows
            uint32_t cnt[J][KT];
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < KT; ++r) cnt[j][r] = 0;
            for (uint32_t q = r0; q < r1;) { // wave-uniform
                if (!loaded || q - w >= 64u) {
                    w = q;
                    loaded = true;
                    load_window_p<J, P>(a, w, rend, lane, my_win);
                }
                const uint32_t hi = r1 < w + 64u ? r1 : w + 64u;
                const uint64_t mp = q < rm ? bit_range(q - w, (hi < rm ? hi : rm) - w) : 0ull;
                const uint64_t mn = hi > rm ? bit_range((q > rm ? q : rm) - w, hi - w) : 0ull;
                const uint64_t m = mp | mn;
                if ((uint32_t)(m >> 32) == 0u || (uint32_t)m == 0u) { // wave-uniform
                    // the variable's records in this window lie in one 32-bit
                    // half (most do): count on that half's dwords only
                    const uint32_t hf = (uint32_t)m == 0u ? 1u : 0u;
                    const half_word* win32 = reinterpret_cast<const half_word*>(my_win);
                    const uint32_t mp32 = (uint32_t)(mp >> (32u * hf)), mn32 = (uint32_t)(mn >> (32u * hf));
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        uint32_t pl[P];
#pragma unroll
                        for (int p = 0; p < P; ++p) pl[p] = win32[2 * ((p * J + j) * 64 + lane) + hf];
                        count_levels<P, KT, uint32_t>(pl, mp32, mn32, cnt[j]);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        uint64_t pl[P];
#pragma unroll
                        for (int p = 0; p < P; ++p) pl[p] = my_win[(p * J + j) * 64 + lane];
                        count_levels<P, KT>(pl, mp, mn, cnt[j]);
                    }
                }
                q = hi;
            }
            float th[J], mm[J], vv[J];
            bool valid[J];
            load_row<J, OP, FULL>(a, v, lane, th, mm, vv, valid);
            bool clamped = false;
            const double mu = (OP == OP_ADJ || a.mode != 1) ? 1.0 : clamp_mu(sload(a.mu_cur + v), clamped);
            const uint64_t* ownp = a.lits_cur + (size_t)(a.lit_rows ? v : 2 * v) * W;
            uint64_t oP[J];
#pragma unroll
            for (int j = 0; j < J; ++j) oP[j] = sload(ownp + j);
            // U = sum over r of (positive - negative records with R = r)
            // dL/dR[r]: with D_r = cnt[r - 1] - dn (positive - negative
            // records with R >= r), that difference is D_r - D_(r+1), i.e.
            // dp - cnt[0] at r = 0, cnt[r - 1] - cnt[r] inside and cnt[KT - 1] - dn
            // at r = KT.  Levels above the widest clause width K count nothing
            // (their differences are 0) and meet zero table rows, so every
            // one of the KT + 1 terms can be formed: u gains exactly +0.
            const int32_t dp = (int32_t)(rm - r0), dn = (int32_t)(r1 - rm);
            double U[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                float u = 0.f;
#pragma unroll
                for (int r = 0; r <= KT; ++r) {
                    const int32_t hi = r == 0 ? dp + dn : (int32_t)cnt[j][r - 1];
                    const int32_t lo = r < KT ? (int32_t)cnt[j][r] : dn;
                    u = fmaf((float)(hi - lo - (r == 0 ? dn : 0)), my_gt[(r * J + j) * 64 + lane], u);
                }
                U[j] = (double)u;
            }
            var_tail<J, OP>(a, c, v, lane, th, mm, vv, valid, mu, clamped, U, oP, vi.witness, vi.wcand, bad);
        }
    }
    if (OP == OP_STEP) {
        if (ballot64(bad != 0) && lane == 0) atomicOr(&a.ctrl->nonfinite, 1);
        advance_step(a);
    }
}

// ---------------------------------------------------------------------------
// Forward of the wide clauses (widths 5 .. 15) when the clause planes are on:
// two passes over every wide bucket, one launch each.
//
// fwd_planes_kernel: one thread per (clause, candidate dword): R of 32
// candidates as a bit-sliced binary counter (P = 4 planes: a 1-bit add per
// literal), written as the clause's planes.
// planes_hist_kernel: the histogram of R from those planes: a wave takes 64
// consecutive clauses of a unit, loads their planes (lane r: clause r),
// transposes every plane word across the wave (lane l: candidate 64 j + l,
// bit r: clause r) and counts per level r the clauses with R >= r
// (thermometer of the planes, one popcount per level); H[r] = #(R >= r) -
// #(R >= r + 1).  The block adds its four waves' counts in LDS, then into
// the global histogram (integer atomics, so the result is exact).
// ---------------------------------------------------------------------------

// One work unit of wide clauses (width k <= KMAX): the planes of R of its
// clauses, pipelined like fwd_hist_unit (the literal dwords of the next
// clause and the codes of the one after in flight while a clause is added).
template <int KMAX, bool VR>
__device__ __forceinline__ void fwd_planes_unit(const FwdArgs& a, const FwdUnit& u, int k,
                                                const uint32_t* __restrict__ codes, uint32_t* planes, int64_t base)
{
    const int Dn = a.Dn, S = 256 / Dn;
    const int slot = threadIdx.x / Dn, d = threadIdx.x % Dn;
    if (slot >= S) return;
    const size_t prow = (size_t)4 * a.plane_stride; // dwords of one clause's planes
    const int64_t c0 = u.c0 + slot;
    const int64_t rem = u.c1 - c0;
    const int nit = rem <= 0 ? 0 : (int)((rem + S - 1) / S);
    uint32_t code_nx[KMAX], x_nx[KMAX];
#pragma unroll
    for (int q = 0; q < KMAX; ++q) {
        code_nx[q] = 0u;
        x_nx[q] = 0u;
    }
    if (nit > 0) {
#pragma unroll
        for (int q = 0; q < KMAX; ++q)
            if (q < k) x_nx[q] = lit_dword<VR>(a.bits32, codes[c0 * k + q], a.W2, d);
    }
    if (nit > 1) {
#pragma unroll
        for (int q = 0; q < KMAX; ++q)
            if (q < k) code_nx[q] = codes[(c0 + S) * k + q];
    }
    for (int it = 0; it < nit; ++it) {
        const int64_t c = c0 + (int64_t)it * S;
        uint32_t x[KMAX];
#pragma unroll
        for (int q = 0; q < KMAX; ++q) x[q] = x_nx[q];
        if (it + 1 < nit) {
#pragma unroll
            for (int q = 0; q < KMAX; ++q)
                if (q < k) x_nx[q] = lit_dword<VR>(a.bits32, code_nx[q], a.W2, d);
        }
        if (it + 2 < nit) {
#pragma unroll
            for (int q = 0; q < KMAX; ++q)
                if (q < k) code_nx[q] = codes[(c + 2 * S) * k + q];
        }
        uint32_t r0 = 0, r1 = 0, r2 = 0, r3 = 0; // R < 16: a 4-bit counter per candidate
#pragma unroll
        for (int q = 0; q < KMAX; ++q) {
            const uint32_t c0b = r0 & x[q];
            r0 ^= x[q];
            const uint32_t c1b = r1 & c0b;
            r1 ^= c0b;
            const uint32_t c2b = r2 & c1b;
            r2 ^= c1b;
            r3 ^= c2b;
        }
        uint32_t* P = planes + (size_t)(base + c) * prow + d;
        P[0] = r0;
        P[(size_t)a.plane_stride] = r1;
        P[(size_t)2 * a.plane_stride] = r2;
        P[(size_t)3 * a.plane_stride] = r3;
    }
}

template <int KMAX, bool VR>
__global__ __launch_bounds__(256) void fwd_planes_kernel(FwdArgs a)
{
    if (a.ctrl && a.ctrl->stop) return;
    const uint32_t un = xcd_unit(a.xcd, (uint32_t)a.nunits);
    if (un >= (uint32_t)a.nunits) return;
    const FwdUnit u = a.units[un];
    if (a.ictrl && a.ictrl[u.inst].frozen) return;
    const int k = u.pad;
    fwd_planes_unit<KMAX, VR>(a, u, k, a.wide_codes[k], a.planes, a.wide_base[k]);
}

// Several buckets of a mixed-width store in one launch: with clause planes
// every bucket (at most 256 candidates, so a block's tile is all of them),
// without them those of widths up to 4.  A unit of width
// k <= 4 is a histogram unit of fwd_hist_unit (widths up to 3 write two
// planes from the start of the plane buffer, width 4 four planes in the
// wide region), a wider one a planes unit of fwd_planes_unit; the histogram
// of the wide clauses then comes from planes_hist_kernel.  Small buckets no
// longer run as launches of their own with too few waves to hide latency.
template <int KMAX, bool VR>
__global__ __launch_bounds__(256) void fwd_multi_kernel(FwdArgs a)
{
    extern __shared__ uint32_t lh[]; // [4][32][DT]
    if (a.ctrl && a.ctrl->stop) return;
    const uint32_t un = xcd_unit(a.xcd, (uint32_t)a.nunits);
    if (un >= (uint32_t)a.nunits) return;
    const FwdUnit u = a.units[un];
    if (a.ictrl && a.ictrl[u.inst].frozen) return;
    const int k = u.pad; // block-uniform
    const uint32_t* codes = a.wide_codes[k];
    const int64_t base = a.wide_base[k];
    uint32_t* planes4 = a.planes ? a.planes + a.wide_off : nullptr;
    switch (k) {
    case 1: fwd_hist_unit<1, 8, VR>(a, u, codes, a.planes, 2, base, lh); break;
    case 2: fwd_hist_unit<2, 8, VR>(a, u, codes, a.planes, 2, base, lh); break;
    case 3: fwd_hist_unit<3, 8, VR>(a, u, codes, a.planes, 2, base, lh); break;
    case 4: fwd_hist_unit<4, 8, VR>(a, u, codes, planes4, 4, base, lh); break;
    default: fwd_planes_unit<KMAX, VR>(a, u, k, codes, planes4, base); break;
    }
}

template <int J, int KT>
__global__ __launch_bounds__(256) void planes_hist_kernel(FwdArgs a, int nunits)
{
    if (a.ctrl && a.ctrl->stop) return;
    constexpr int P = 4, Q = P * J / 2; // 16-byte loads per clause
    __shared__ uint32_t s_cnt[J][KT + 1][64]; // the block's counts, summed over its waves
    const uint32_t lane = __lane_id(), wv = threadIdx.x / 64u;
    const int K1 = a.K1;
    uint32_t cnt[J][KT + 1]; // [j][0]: clauses; [j][r]: clauses with R >= r
    int32_t inst = -1;
    for (int e = threadIdx.x; e < J * (KT + 1) * 64; e += 256) (&s_cnt[0][0][0])[e] = 0;
    __syncthreads();
    auto flush = [&](int32_t to) {
        // every wave of the block reaches each flush together: the units
        // of a block are visited in the same order by all its waves
        if (inst >= 0) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r <= KT; ++r) atomicAdd(&s_cnt[j][r][lane], cnt[j][r]);
        }
        __syncthreads();
        if (inst >= 0) {
            uint32_t* H = a.H + ((size_t)inst * a.H_reps + blockIdx.x % (uint32_t)a.H_reps) * a.H_stride;
            for (int e = threadIdx.x; e < J * 64; e += 256) {
                const int j = e / 64, l = e % 64;
                const uint32_t cand = 64u * j + l;
                if ((int)(cand >> 5) >= a.Dn) continue;
#pragma unroll
                for (int r = 0; r <= KT; ++r) {
                    if (r >= K1) break;
                    const uint32_t h = s_cnt[j][r][l] - (r < KT ? s_cnt[j][r + 1][l] : 0u);
                    if (h) atomicAdd(&H[(size_t)cand * K1 + r], h);
                }
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < J * (KT + 1) * 64; e += 256) (&s_cnt[0][0][0])[e] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int r = 0; r <= KT; ++r) cnt[j][r] = 0;
        inst = to;
    };
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int r = 0; r <= KT; ++r) cnt[j][r] = 0;
    const ItemRange ur = xcd_items(a.xcd, (uint32_t)nunits, 1u, 0u);
    for (uint32_t un = ur.first; un < ur.end; un += ur.stride) { // block-uniform
        const FwdUnit u = a.units[un];
        if (a.ictrl && a.ictrl[u.inst].frozen) continue;
        if (u.inst != inst) flush(u.inst);
        const int k = u.pad;
        const int64_t base = a.wide_base[k];
        // planes of clauses [cc, cc + 64) (lane r: clause cc + r; past the
        // unit: zero)
        auto load = [&](int64_t cc, uint64_t (&wd)[P * J]) {
            const int64_t rec = cc + lane;
            const bool ok = rec < u.c1;
            const uint4* pl = (const uint4*)a.planes + (size_t)(base + (ok ? rec : cc)) * Q;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint4 v = ok ? pl[q] : make_uint4(0u, 0u, 0u, 0u);
                wd[2 * q] = ((uint64_t)v.y << 32) | v.x;
                wd[2 * q + 1] = ((uint64_t)v.w << 32) | v.z;
            }
        };
        uint64_t wd_nx[P * J];
        const int64_t cw = u.c0 + 64 * (int64_t)wv;
        if (cw < u.c1) load(cw, wd_nx);
        for (int64_t c = cw; c < u.c1; c += 256) { // wave-uniform
            // the next group's planes are in flight while this one is counted
            uint64_t wd[P * J];
#pragma unroll
            for (int e = 0; e < P * J; ++e) wd[e] = wd_nx[e];
            if (c + 256 < u.c1) load(c + 256, wd_nx);
            const uint32_t n = (uint32_t)((u.c1 - c) < 64 ? (u.c1 - c) : 64);
#pragma unroll
            for (int j = 0; j < J; ++j) {
                // the P plane words of candidate word j, transposed together
                uint64_t pw[P];
#pragma unroll
                for (int p = 0; p < P; ++p) pw[p] = wd[p * J + j];
                transpose64_n<P>(pw, lane);
                uint64_t ge[KT];
                thermometer<P, KT>(pw, ge);
                cnt[j][0] += n;
#pragma unroll
                for (int r = 0; r < KT; ++r) cnt[j][r + 1] += (uint32_t)__popcll(ge[r]);
            }
        }
    }
    flush(-1);
}

// ---------------------------------------------------------------------------
// Clause-major adjoint by atomic scatter (the alternative to the
// variable-major gather of the update kernels, kept for comparison).
//
// One thread per (clause, candidate dword) of one width bucket: R of its 32
// candidates as a bit-sliced binary counter, then for every candidate the
// table entry dL/dR[R] is added into the row of every literal of the clause
// (+1 for x_v, -1 for not-x_v: Sec. III-B's straight-through estimator).
// The block's clauses are consecutive in the lexicographic clause order, so
// their first (smallest) literals fall into a short run of variables: those
// contributions go to an LDS tile of ST variable rows (LDS atomics), flushed
// into U with global atomics at the end; every other contribution is a
// global FP32 atomic.  U must be zero on entry.
// ---------------------------------------------------------------------------

struct ScatterArgs {
    const uint32_t* codes; // [Cb][k]
    int64_t Cb;
    int32_t k, N, Np, K1, Dn;
    const uint32_t* bits32; // literal rows, row stride W2 dwords
    int32_t W2;
    const float* tbl;       // [K1][Np]
    float* U;               // [V][N]
    int32_t V;
    int32_t ST;             // variable rows of the LDS tile
};

__global__ __launch_bounds__(256) void adj_scatter_kernel(ScatterArgs a)
{
    extern __shared__ float lds_sc[]; // [K1][Np] table, then [ST][N] tile
    float* s_tbl = lds_sc;
    float* s_U = lds_sc + (size_t)a.K1 * a.Np;
    const int Dn = a.Dn, S = 256 / Dn;
    const int slot = threadIdx.x / Dn, d = threadIdx.x % Dn;
    const int64_t c0 = (int64_t)blockIdx.x * S;
    for (int e = threadIdx.x; e < a.K1 * a.Np; e += 256) s_tbl[e] = a.tbl[e];
    for (int e = threadIdx.x; e < a.ST * a.N; e += 256) s_U[e] = 0.f;
    // the tile starts at the first variable of the block's first clause
    const uint32_t vlo = a.codes[(size_t)c0 * a.k] >> 1;
    __syncthreads();
    const int64_t c = c0 + slot;
    if (slot < S && c < a.Cb) {
        uint32_t r[6] = {0u, 0u, 0u, 0u, 0u, 0u}; // R <= 32 in binary
        for (int q = 0; q < a.k; ++q) {
            const uint32_t code = a.codes[(size_t)c * a.k + q];
            uint32_t carry = a.bits32[(size_t)code * a.W2 + d];
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const uint32_t t = r[b] & carry;
                r[b] ^= carry;
                carry = t;
            }
        }
        for (int bit = 0; bit < 32; ++bit) {
            const int i = 32 * d + bit;
            if (i >= a.N) break;
            uint32_t R = 0;
#pragma unroll
            for (int b = 0; b < 6; ++b) R |= ((r[b] >> bit) & 1u) << b;
            const float val = s_tbl[(size_t)R * a.Np + i];
            for (int q = 0; q < a.k; ++q) {
                const uint32_t code = a.codes[(size_t)c * a.k + q];
                const uint32_t v = code >> 1;
                const float x = (code & 1u) ? -val : val;
                if (q == 0 && v - vlo < (uint32_t)a.ST) atomicAdd(&s_U[(size_t)(v - vlo) * a.N + i], x);
                else atomicAdd(&a.U[(size_t)v * a.N + i], x);
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < a.ST * a.N; e += 256) {
        const float x = s_U[e];
        const uint32_t v = vlo + (uint32_t)(e / a.N);
        if (x != 0.f && v < (uint32_t)a.V) atomicAdd(&a.U[(size_t)v * a.N + e % a.N], x);
    }
}

hipError_t launch_adj_scatter(const uint32_t* codes, int64_t Cb, int k, int N, int K1, const uint32_t* bits32,
                              int W2, const float* tbl, float* U, int V, hipStream_t st)
{
    if (Cb <= 0 || k <= 0) return hipSuccess;
    ScatterArgs a{};
    a.V = V;
    a.codes = codes;
    a.Cb = Cb;
    a.k = k;
    a.N = N;
    a.Np = 64 * ((N + 63) / 64);
    a.K1 = K1;
    a.Dn = (N + 31) / 32;
    a.bits32 = bits32;
    a.W2 = W2;
    a.tbl = tbl;
    a.U = U;
    const size_t tbl_bytes = (size_t)K1 * a.Np * 4;
    a.ST = (int)std::max<size_t>(1, std::min<size_t>(64, (64 * 1024 - tbl_bytes) / ((size_t)N * 4)));
    const int S = 256 / a.Dn;
    const size_t lds = tbl_bytes + (size_t)a.ST * N * 4;
    hipLaunchKernelGGL(adj_scatter_kernel, dim3((unsigned)((Cb + S - 1) / S)), dim3(256), lds, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------

// Variable bits [V][W] -> literal rows [2V][W] (complement with pad bits 0).
__global__ void expand_kernel(const uint64_t* __restrict__ bits, int64_t V, int W, int N, uint64_t* __restrict__ lits)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= V * W) return;
    const int64_t v = e / W;
    const int j = (int)(e % W);
    const int rem = N - 64 * j;
    const uint64_t vm = rem >= 64 ? ~0ull : ((1ull << rem) - 1ull);
    const uint64_t x = bits[e] & vm;
    lits[(2 * v) * W + j] = x;
    lits[(2 * v + 1) * W + j] = ~x & vm;
}

// Float assignment [V][N] (value > 0.5 = True) -> variable bits [V][W].
// Bound by latency with one word per wave: a wave takes R consecutive words,
// all their loads in flight, and lane q stores word q, so that the words
// leave in one store (V = 1e5, N = 100, 40 MB: 23.7 us with a word per wave,
// 16.0 at R = 4, 16.6 at 8, 16.8 at 16).
template <int R>
__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ assign, int V, int N, int W,
                                                   uint64_t* __restrict__ bits)
{
    const uint32_t lane = __lane_id();
    const int64_t words = (int64_t)V * W;
    const int64_t w0 = ((int64_t)blockIdx.x * 4 + uniform(threadIdx.x / 64u)) * R;
    if (w0 >= words) return;
    int64_t v = w0 / W;
    int j = (int)(w0 - v * W);
    float x[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = 64 * j + (int)lane;
        x[q] = w0 + q < words && i < N ? assign[v * N + i] : 0.f; // 0: False past N
        if (++j == W) j = 0, ++v;
    }
    uint64_t word = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const uint64_t bal = ballot64(x[q] > 0.5f);
        if (lane == (uint32_t)q) word = bal;
    }
    if (lane < (uint32_t)R && w0 + lane < words) bits[w0 + lane] = word;
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) + Box-Muller.
__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = (uint32_t)p1;
        c[2] = n2;
        c[3] = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Element e of the batch draws one Philox block with counter
// (e mod 2^32, e div 2^32, 0x5A17, 0) and key (seed mod 2^32, seed div 2^32):
// words 0 and 1 give N(0,1) by Box-Muller, word 2 a Bernoulli draw.
__device__ __forceinline__ float normal_draw(int64_t e, uint64_t seed, uint32_t* word2)
{
    uint32_t c[4] = {(uint32_t)e, (uint32_t)((uint64_t)e >> 32), 0x5A17u, 0u};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    const double u1 = ((double)c[0] + 0.5) * (1.0 / 4294967296.0);
    const double u2 = ((double)c[1] + 0.5) * (1.0 / 4294967296.0);
    if (word2) *word2 = c[2];
    return (float)(sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}

__global__ void init_normal_kernel(float* __restrict__ theta, int64_t n, uint64_t seed)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    theta[e] = normal_draw(e, seed, nullptr);
}

// Initialisation from a proposal p_v = P(x_v = true), one wave per variable:
// b_vi = [word2 < floor(p_v 2^32)], theta_vi = +|z_vi| where b_vi = 1 and
// -rho_v |z_vi| where b_vi = 0, z_vi the draw of the random initialisation.
// Mean mode (Eq. 5 ahead of Eq. 2) keeps the row mean positive so that the
// normalised signs reproduce b: rho_v = min(1, 0.5 sum_{b=1}|z| / sum_{b=0}|z|),
// and a row without any b = 1 gets b = 1 at candidate v mod N.
__global__ __launch_bounds__(256) void init_proposal_kernel(PropArgs a)
{
    const int lane = threadIdx.x & 63;
    const int32_t v = (int32_t)(blockIdx.x * 4u + (threadIdx.x >> 6));
    if (v >= a.V) return;
    const float pv = a.p[v];
    double pd = pv >= 0.f ? (double)pv : 0.0; // NaN -> 0
    if (pd > 1.0) pd = 1.0;
    const double thr = floor(pd * 4294967296.0);
    const int64_t e0 = (int64_t)v * a.N;
    int forced = -1;
    double rho = 1.0;
    if (a.mode == 1) {
        bool any = false;
        for (int i = lane; i < a.N; i += 64) {
            uint32_t w2;
            (void)normal_draw(e0 + i, a.seed, &w2);
            any |= (double)w2 < thr;
        }
        if (!ballot64(any)) forced = v % a.N;
        double sp = 0.0, sn = 0.0;
        for (int i = lane; i < a.N; i += 64) {
            uint32_t w2;
            const float mag = fabsf(normal_draw(e0 + i, a.seed, &w2));
            if ((double)w2 < thr || i == forced) sp += (double)mag;
            else sn += (double)mag;
        }
        sp = wave_sum(sp);
        sn = wave_sum(sn);
        if (sn > 0.0 && 0.5 * sp / sn < 1.0) rho = 0.5 * sp / sn;
    }
    for (int i = lane; i < a.N; i += 64) {
        uint32_t w2;
        const float mag = fabsf(normal_draw(e0 + i, a.seed, &w2));
        const bool b = (double)w2 < thr || i == forced;
        a.theta[e0 + i] = b ? mag : (float)(-rho * (double)mag);
    }
}

__global__ void copy16_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) dst[e] = src[e];
}

// Bandwidth reference kernels (calibration of the roofline): streams with
// 16-byte non-temporal accesses, four loads per array in flight per thread
// (KIND 0: copy src -> a; KIND 1: three arrays read and written in place,
// the pattern of the optimizer state), or with the update kernels' own
// access pattern (KIND 2: three arrays in place, rows of 256 floats, one
// dword per lane and load, four loads per array in flight).
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));

template <int KIND>
__global__ __launch_bounds__(256) void stream_kernel(uint32_t* __restrict__ a, uint32_t* __restrict__ b,
                                                      uint32_t* __restrict__ c, const uint32_t* __restrict__ src,
                                                      int64_t n4)
{
    const int64_t tiles = (n4 + 1023) / 1024; // 1024 16-byte units per block pass
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        if (KIND == 2) {
            // each wave: four rows of 256 dwords of each array (one 1 KiB row
            // = one 16-byte unit per lane); lane l takes dwords 64 j + l
            const int64_t row0 = t * 16 + (threadIdx.x / 64) * 4;
            const uint32_t l = __lane_id();
            uint32_t x[4][4], y[4][4], z[4][4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t e = (row0 + r) * 256 + 64 * j + l;
                    const bool ok = e < 4 * n4;
                    x[r][j] = ok ? __builtin_nontemporal_load(a + e) : 0u;
                    y[r][j] = ok ? __builtin_nontemporal_load(b + e) : 0u;
                    z[r][j] = ok ? __builtin_nontemporal_load(c + e) : 0u;
                }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t e = (row0 + r) * 256 + 64 * j + l;
                    if (e >= 4 * n4) continue;
                    __builtin_nontemporal_store(x[r][j] ^ y[r][j], a + e);
                    __builtin_nontemporal_store(y[r][j] + z[r][j], b + e);
                    __builtin_nontemporal_store(z[r][j] ^ x[r][j], c + e);
                }
            continue;
        }
        v4u32* A = (v4u32*)a;
        v4u32* B = (v4u32*)b;
        v4u32* Cc = (v4u32*)c;
        const v4u32* S = (const v4u32*)src;
        v4u32 x[4], y[4], z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = t * 1024 + k * 256 + threadIdx.x;
            const bool ok = e < n4;
            const v4u32 zero = {0u, 0u, 0u, 0u};
            if (KIND == 0) {
                x[k] = ok ? __builtin_nontemporal_load(S + e) : zero;
            } else {
                x[k] = ok ? __builtin_nontemporal_load(A + e) : zero;
                y[k] = ok ? __builtin_nontemporal_load(B + e) : zero;
                z[k] = ok ? __builtin_nontemporal_load(Cc + e) : zero;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = t * 1024 + k * 256 + threadIdx.x;
            if (e >= n4) continue;
            if (KIND == 0) {
                __builtin_nontemporal_store(x[k], A + e);
            } else {
                __builtin_nontemporal_store(x[k] ^ y[k], A + e);
                __builtin_nontemporal_store(y[k] + z[k], B + e);
                __builtin_nontemporal_store(z[k] ^ x[k], Cc + e);
            }
        }
    }
}

hipError_t launch_stream(int kind, uint32_t* a, uint32_t* b, uint32_t* c, const uint32_t* src, int64_t n4, int blocks,
                         hipStream_t st)
{
    if (n4 <= 0) return hipSuccess;
    switch (kind) {
    case 0: hipLaunchKernelGGL(stream_kernel<0>, dim3(blocks), dim3(256), 0, st, a, b, c, src, n4); break;
    case 1: hipLaunchKernelGGL(stream_kernel<1>, dim3(blocks), dim3(256), 0, st, a, b, c, src, n4); break;
    default: hipLaunchKernelGGL(stream_kernel<2>, dim3(blocks), dim3(256), 0, st, a, b, c, src, n4); break;
    }
    return hipGetLastError();
}

// dst[r][j] = src[r * src_stride + j] for r < rows, j < w (64-bit words):
// strided rows packed for one contiguous device-to-host copy
__global__ void strided_rows_kernel(const uint64_t* __restrict__ src, int64_t rows, int w, int64_t src_stride,
                                    uint64_t* __restrict__ dst)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * w) return;
    const int64_t r = e / w;
    dst[e] = src[r * src_stride + (e - r * w)];
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, int64_t n, uint32_t val)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = val;
}

// Candidate priority (Sec. IV-B): rank = #{j : sat_j > sat_i or (== and j < i)}.
// order[rank] = i, and slot[i] = rank for the first nsel candidates, else -1.
__global__ __launch_bounds__(256) void rank_kernel(const int64_t* __restrict__ sat, int N, int nsel,
                                                   int32_t* __restrict__ order, int32_t* __restrict__ slot)
{
    __shared__ int64_t s_sat[256];
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int64_t si = i < N ? sat[i] : 0;
    int rank = 0;
    for (int j0 = 0; j0 < N; j0 += 256) {
        __syncthreads();
        if (j0 + (int)threadIdx.x < N) s_sat[threadIdx.x] = sat[j0 + threadIdx.x];
        __syncthreads();
        const int n = min(256, N - j0);
        for (int j = 0; j < n; ++j) rank += (s_sat[j] > si) || (s_sat[j] == si && j0 + j < i);
    }
    if (i >= N) return;
    order[rank] = i;
    slot[i] = rank < nsel ? rank : -1;
}

// ---------------------------------------------------------------------------
// Confident partial assignments (Sec. IV-B): per selected candidate (slot)
// the k eligible variables with the smallest |g| (ties: lower index), in that
// order.  Keys are the IEEE bits of |g|, which order like the values for
// non-negative floats.
//
// A radix select of the k-th smallest key over [V][slots], every slot at
// once and the variables split over the chip: four digit passes (a histogram
// per slot and 8-bit digit), a counting pass (keys below and equal to the
// k-th, per chunk), a collecting pass, and a sort of each slot's k keys.
// The passes read the keys from the last-level cache; what bounds them is
// each launch's latency and its closing adds (eight histogram replicas, one
// per XCD).  V = 2e5, 16 slots, k = 20: four digit passes of 9.9 us, count
// 9.4, collect 14.2, sort 5.8; one block per candidate, walking its column
// of a transposed gradient five times, took 2.2 ms, and the transposed
// store of every candidate's gradient 0.19 ms of the 0.28 ms gradient pass
// (0.09 ms now, storing the selected columns row by row).
// ---------------------------------------------------------------------------

constexpr int kSelTile = 32; // slots of a block

struct SelDigit {
    uint32_t prefix, rank, k; // key digits found so far, rank left among the keys sharing them, keys to take
};

// State of a slot before pass `pass` (0: nothing known): the previous
// pass's histogram scanned for the digit that holds the rank.  Called by a
// whole wave.
__device__ __forceinline__ SelDigit select_state(const SelectArgs& a, int pass, int slot, uint32_t lane)
{
    SelDigit d = {0u, 0u, 0u};
    if (pass == 0) return d;
    if (pass > 1) d = ((const SelDigit*)a.state)[(size_t)(pass - 1) * a.S + slot];
    const uint4* h = (const uint4*)(a.hist + ((size_t)(pass - 1) * 8 * a.S + slot) * 256) + lane;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint4 x = h[(size_t)q * a.S * 64];
        v.x += x.x;
        v.y += x.y;
        v.z += x.z;
        v.w += x.w;
    }
    const uint32_t own = v.x + v.y + v.z + v.w;
    uint32_t incl = own;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const uint32_t y = __shfl_up(incl, st);
        if ((int)lane >= st) incl += y;
    }
    if (pass == 1) d.k = d.rank = min((uint32_t)a.k, (uint32_t)__shfl(incl, 63));
    if (d.k == 0) return d;
    // the lane whose four bins hold the rank, then the bin
    const uint64_t m = ballot64(incl >= d.rank);
    const int at = __ffsll((unsigned long long)m) - 1;
    uint32_t before = incl - own, dig = 0;
    const uint32_t c[3] = {v.x, v.y, v.z};
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (dig == (uint32_t)j && before + c[j] < d.rank) {
            before += c[j];
            ++dig;
        }
    const uint32_t digit = 4u * (uint32_t)at + (uint32_t)__shfl(dig, at);
    d.rank -= (uint32_t)__shfl(before, at);
    d.prefix |= digit << (32 - 8 * pass);
    return d;
}

// The slots of this block: [s0, s0 + n), one slot per lane group of a power
// of two, threads striding the variables of chunk blockIdx.x.
struct SelTile {
    int s0, n, slot, row, rows, v0, v1;
};

__device__ __forceinline__ SelTile select_tile(const SelectArgs& a)
{
    SelTile t;
    t.s0 = blockIdx.y * kSelTile;
    t.n = min(kSelTile, a.S - t.s0);
    int p = 1;
    while (p < t.n) p <<= 1;
    t.slot = threadIdx.x % p;
    t.row = threadIdx.x / p;
    t.rows = 256 / p;
    t.v0 = blockIdx.x * a.chunk;
    t.v1 = min(a.V, t.v0 + a.chunk);
    return t;
}

// f(v, key) over the eligible variables of the tile's chunk for this
// thread's slot, four keys in flight
template <class F>
__device__ __forceinline__ void select_keys(const SelectArgs& a, const SelTile& t, F f)
{
    if (t.slot >= t.n) return;
    for (int v = t.v0 + t.row; v < t.v1; v += 4 * t.rows) {
        uint32_t key[4], o0[4], o1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int w = min(v + q * t.rows, t.v1 - 1);
            key[q] = __float_as_uint(fabsf(a.g[(size_t)w * a.S + t.s0 + t.slot]));
            o0[q] = a.occ_off[w];
            o1[q] = a.occ_off[w + 1];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v + q * t.rows < t.v1 && o1[q] > o0[q]) f(v + q * t.rows, key[q]);
    }
}

__device__ __forceinline__ void select_states(const SelectArgs& a, const SelTile& t, int pass, SelDigit* s_d)
{
    const uint32_t lane = __lane_id();
    for (int s = threadIdx.x / 64; s < t.n; s += 4) {
        const SelDigit d = select_state(a, pass, t.s0 + s, lane);
        if (lane == 0) {
            s_d[s] = d;
            if (blockIdx.x == 0 && pass > 0) ((SelDigit*)a.state)[(size_t)pass * a.S + t.s0 + s] = d;
        }
    }
}

__global__ __launch_bounds__(256) void select_hist_kernel(SelectArgs a, int pass)
{
    __shared__ uint32_t s_hist[kSelTile][256];
    __shared__ SelDigit s_d[kSelTile];
    const SelTile t = select_tile(a);
    for (int e = threadIdx.x; e < t.n * 256; e += 256) (&s_hist[0][0])[e] = 0;
    select_states(a, t, pass, s_d);
    __syncthreads();
    const SelDigit d = s_d[t.slot < t.n ? t.slot : 0];
    const uint32_t mask = pass == 0 ? 0u : ~0u << (32 - 8 * pass);
    const int shift = 24 - 8 * pass;
    if (pass == 0 || d.k > 0)
        select_keys(a, t, [&](int, uint32_t key) {
            if ((key & mask) == d.prefix) atomicAdd(&s_hist[t.slot][(key >> shift) & 255u], 1u);
        });
    __syncthreads();
    uint32_t* H = a.hist + (((size_t)pass * 8 + blockIdx.x % 8u) * a.S + t.s0) * 256;
    for (int e = threadIdx.x; e < t.n * 256; e += 256) {
        const uint32_t c = (&s_hist[0][0])[e];
        if (c) atomicAdd(&H[e], c);
    }
}

// keys below and equal to the k-th, per chunk and slot
__global__ __launch_bounds__(256) void select_count_kernel(SelectArgs a)
{
    __shared__ uint32_t s_c[2][kSelTile];
    __shared__ SelDigit s_d[kSelTile];
    const SelTile t = select_tile(a);
    if (threadIdx.x < 2 * kSelTile) (&s_c[0][0])[threadIdx.x] = 0;
    select_states(a, t, 4, s_d);
    __syncthreads();
    const SelDigit d = s_d[t.slot < t.n ? t.slot : 0];
    uint32_t lt = 0, eq = 0;
    if (d.k > 0)
        select_keys(a, t, [&](int, uint32_t key) {
            lt += key < d.prefix;
            eq += key == d.prefix;
        });
    if (t.slot < t.n) {
        if (lt) atomicAdd(&s_c[0][t.slot], lt);
        if (eq) atomicAdd(&s_c[1][t.slot], eq);
    }
    __syncthreads();
    if ((int)threadIdx.x < t.n) {
        uint2* o = (uint2*)a.count + (size_t)blockIdx.x * a.S + t.s0;
        o[threadIdx.x] = make_uint2(s_c[0][threadIdx.x], s_c[1][threadIdx.x]);
    }
}

// Selected (key, variable) pairs: keys below the k-th take the slots' first
// places (offset by the earlier chunks' counts), the ones equal to it follow
// in the order of the variables until k are taken.
__global__ __launch_bounds__(256) void select_collect_kernel(SelectArgs a)
{
    __shared__ uint32_t s_lt[kSelTile], s_eq[kSelTile]; // keys of earlier chunks
    __shared__ int s_any;
    const SelTile t = select_tile(a);
    const uint2* cnt = (const uint2*)a.count;
    if (threadIdx.x == 0) s_any = 0;
    if (threadIdx.x < kSelTile) s_lt[threadIdx.x] = s_eq[threadIdx.x] = 0;
    __syncthreads();
    if ((int)threadIdx.x < t.n) {
        const uint2 c = cnt[(size_t)blockIdx.x * a.S + t.s0 + threadIdx.x];
        if (c.x | c.y) s_any = 1;
    }
    __syncthreads();
    if (!s_any) return;
    if (t.slot < t.n) {
        uint32_t lt = 0, eq = 0;
        for (int ch = t.row; ch < (int)blockIdx.x; ch += t.rows) {
            const uint2 c = cnt[(size_t)ch * a.S + t.s0 + t.slot];
            lt += c.x;
            eq += c.y;
        }
        if (lt) atomicAdd(&s_lt[t.slot], lt);
        if (eq) atomicAdd(&s_eq[t.slot], eq);
    }
    __syncthreads();
    const SelDigit* state = (const SelDigit*)a.state + (size_t)4 * a.S + t.s0;
    // keys equal to the k-th: a wave per slot, variables in order
    const uint32_t lane = __lane_id();
    for (int s = threadIdx.x / 64; s < t.n; s += 4) {
        const SelDigit d = state[s];
        uint64_t* out = a.sel + (size_t)(t.s0 + s) * a.k + (d.k - d.rank); // keys below the k-th come first
        uint32_t eq = s_eq[s];
        const uint32_t end = eq + cnt[(size_t)blockIdx.x * a.S + t.s0 + s].y;
        if (d.k == 0) continue;
        for (int v = t.v0; v < t.v1 && eq < d.rank && eq < end; v += 64) { // wave-uniform
            const int w = v + (int)lane;
            const bool hit = w < t.v1 && a.occ_off[w + 1] > a.occ_off[w] &&
                             __float_as_uint(fabsf(a.g[(size_t)w * a.S + t.s0 + s])) == d.prefix;
            const uint64_t m = ballot64(hit);
            const uint32_t at = eq + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (hit && at < d.rank) out[at] = ((uint64_t)d.prefix << 32) | (uint32_t)w;
            eq += (uint32_t)__popcll(m);
        }
    }
    const SelDigit d = state[t.slot < t.n ? t.slot : 0];
    if (d.k > 0)
        select_keys(a, t, [&](int v, uint32_t key) {
            if (key < d.prefix)
                a.sel[(size_t)(t.s0 + t.slot) * a.k + atomicAdd(&s_lt[t.slot], 1u)] = ((uint64_t)key << 32) | (uint32_t)v;
        });
}

// bitonic sort of a slot's (key, variable) pairs, padded with max, and the
// literals of the candidate's current values
__global__ __launch_bounds__(256) void select_sort_kernel(SelectArgs a)
{
    extern __shared__ uint64_t sel[]; // [kpow2]
    const int tid = threadIdx.x, kp = a.kpow2, cand = a.order[blockIdx.x];
    const uint32_t k = ((const SelDigit*)a.state)[(size_t)4 * a.S + blockIdx.x].k;
    for (int q = tid; q < kp; q += 256) sel[q] = q < (int)k ? a.sel[(size_t)blockIdx.x * a.k + q] : ~0ull;
    __syncthreads();
    for (int size = 2; size <= kp; size <<= 1)
        for (int stride = size / 2; stride > 0; stride >>= 1) {
            for (int q = tid; q < kp; q += 256) {
                const int p = q ^ stride;
                if (p > q) {
                    const bool up = (q & size) == 0;
                    const uint64_t x = sel[q], y = sel[p];
                    if ((x > y) == up) { sel[q] = y; sel[p] = x; }
                }
            }
            __syncthreads();
        }
    int32_t* out = a.lits_out + (size_t)blockIdx.x * a.k;
    for (int q = tid; q < a.k; q += 256) {
        if (q >= (int)k) { out[q] = 0; continue; }
        const uint32_t v = (uint32_t)(sel[q] & 0xffffffffu);
        const uint64_t w = a.lits[(size_t)(2 * v) * a.W + (cand >> 6)];
        out[q] = ((w >> (cand & 63)) & 1u) ? (int32_t)(v + 1) : -(int32_t)(v + 1);
    }
    if (tid == 0) {
        a.cand_out[blockIdx.x] = cand;
        a.sat_out[blockIdx.x] = a.sat[cand];
    }
}

// ---------------------------------------------------------------------------
// launchers (host side, same translation unit)
// ---------------------------------------------------------------------------

template <int KW, int B, bool VR>
static hipError_t launch_fwd_k(const FwdArgs& a, dim3 grid, hipStream_t st)
{
    const size_t lds = (size_t)a.DT * 32 * KW * sizeof(uint32_t);
    hipLaunchKernelGGL((fwd_hist_kernel<KW, B, VR>), grid, dim3(256), lds, st, a);
    return hipGetLastError();
}

template <bool VR>
static hipError_t launch_fwd_vr(const FwdArgs& a, dim3 grid, hipStream_t st)
{
    switch (a.KW) {
    case 1: return launch_fwd_k<1, 8, VR>(a, grid, st);
    case 2: return launch_fwd_k<2, 8, VR>(a, grid, st);
    case 3: return launch_fwd_k<3, 8, VR>(a, grid, st);
    case 4: return launch_fwd_k<4, 8, VR>(a, grid, st);
    default: {
        const size_t lds = (size_t)4 * 64 * a.K1 * sizeof(uint32_t);
        if (a.KW <= 8) hipLaunchKernelGGL((fwd_hist_lanes_kernel<8, VR>), grid, dim3(256), lds, st, a);
        else if (a.KW <= 16) hipLaunchKernelGGL((fwd_hist_lanes_kernel<16, VR>), grid, dim3(256), lds, st, a);
        else hipLaunchKernelGGL((fwd_hist_lanes_kernel<32, VR>), grid, dim3(256), lds, st, a);
        return hipGetLastError();
    }
    }
}

static unsigned fwd_grid_x(const FwdArgs& a, int nunits)
{
    return a.xcd ? (unsigned)((nunits + 7) / 8 * 8) : (unsigned)nunits;
}

// every wide bucket (widths 5 .. kmax) in one launch: a.KW = 0, unit widths in
// pad.  With clause planes (four per clause, kmax <= 15): the planes pass,
// then the histogram pass over the planes; else the lane-per-candidate kernel.
// the histogram pass over the wide clauses' planes (units of the wide
// buckets, a.planes at the four-plane region)
hipError_t launch_planes_hist(const FwdArgs& a, int kmax, int nunits, hipStream_t st)
{
    const int J = a.plane_stride / 2; // words per plane row
    // each block ends with one atomic add per (candidate, level) into the
    // instance's histogram; those to one address serialize, so fewer blocks
    // (measured on the structured configuration: 512 blocks 81 us, 256 50 us,
    // 128 40 us, of which 19 us without the adds at 256)
    const unsigned hb = (unsigned)std::min(nunits, 128) / 8 * 8 + (nunits < 8 ? (unsigned)nunits : 0u);
    if (J == 1) {
        if (kmax <= 8) hipLaunchKernelGGL((planes_hist_kernel<1, 8>), dim3(hb), dim3(256), 0, st, a, nunits);
        else if (kmax <= 12) hipLaunchKernelGGL((planes_hist_kernel<1, 12>), dim3(hb), dim3(256), 0, st, a, nunits);
        else hipLaunchKernelGGL((planes_hist_kernel<1, 15>), dim3(hb), dim3(256), 0, st, a, nunits);
    } else if (J == 2) {
        if (kmax <= 8) hipLaunchKernelGGL((planes_hist_kernel<2, 8>), dim3(hb), dim3(256), 0, st, a, nunits);
        else if (kmax <= 12) hipLaunchKernelGGL((planes_hist_kernel<2, 12>), dim3(hb), dim3(256), 0, st, a, nunits);
        else hipLaunchKernelGGL((planes_hist_kernel<2, 15>), dim3(hb), dim3(256), 0, st, a, nunits);
    } else {
        if (kmax <= 8) hipLaunchKernelGGL((planes_hist_kernel<4, 8>), dim3(hb), dim3(256), 0, st, a, nunits);
        else if (kmax <= 12) hipLaunchKernelGGL((planes_hist_kernel<4, 12>), dim3(hb), dim3(256), 0, st, a, nunits);
        else hipLaunchKernelGGL((planes_hist_kernel<4, 15>), dim3(hb), dim3(256), 0, st, a, nunits);
    }
    return hipGetLastError();
}

// every bucket in one launch (fwd_multi_kernel): a.units hold the units of
// all widths, the width in pad; LDS for the widest histogram unit (k = 4)
hipError_t launch_fwd_multi(const FwdArgs& a, int kmax, int nunits, int tiles, hipStream_t st)
{
    const dim3 g(fwd_grid_x(a, nunits), (unsigned)tiles);
    const size_t lds = (size_t)a.DT * 32 * 4 * sizeof(uint32_t);
    if (a.vrows) {
        if (kmax <= 8) hipLaunchKernelGGL((fwd_multi_kernel<8, true>), g, dim3(256), lds, st, a);
        else hipLaunchKernelGGL((fwd_multi_kernel<15, true>), g, dim3(256), lds, st, a);
    } else {
        if (kmax <= 8) hipLaunchKernelGGL((fwd_multi_kernel<8, false>), g, dim3(256), lds, st, a);
        else hipLaunchKernelGGL((fwd_multi_kernel<15, false>), g, dim3(256), lds, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_fwd_wide(const FwdArgs& a, int kmax, int nunits, int tiles, hipStream_t st)
{
    if (a.planes && a.plane_P == 4 && kmax <= 15 && a.Dn <= 8) {
        const dim3 g(fwd_grid_x(a, nunits));
        if (a.vrows) {
            if (kmax <= 8) hipLaunchKernelGGL((fwd_planes_kernel<8, true>), g, dim3(256), 0, st, a);
            else hipLaunchKernelGGL((fwd_planes_kernel<15, true>), g, dim3(256), 0, st, a);
        } else {
            if (kmax <= 8) hipLaunchKernelGGL((fwd_planes_kernel<8, false>), g, dim3(256), 0, st, a);
            else hipLaunchKernelGGL((fwd_planes_kernel<15, false>), g, dim3(256), 0, st, a);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_planes_hist(a, kmax, nunits, st);
    }
    const dim3 grid(fwd_grid_x(a, nunits), (unsigned)tiles, 1);
    const size_t lds = (size_t)4 * 64 * a.K1 * sizeof(uint32_t);
    if (a.vrows) {
        if (kmax <= 8) hipLaunchKernelGGL((fwd_hist_lanes_kernel<8, true>), grid, dim3(256), lds, st, a);
        else if (kmax <= 16) hipLaunchKernelGGL((fwd_hist_lanes_kernel<16, true>), grid, dim3(256), lds, st, a);
        else hipLaunchKernelGGL((fwd_hist_lanes_kernel<32, true>), grid, dim3(256), lds, st, a);
    } else {
        if (kmax <= 8) hipLaunchKernelGGL((fwd_hist_lanes_kernel<8, false>), grid, dim3(256), lds, st, a);
        else if (kmax <= 16) hipLaunchKernelGGL((fwd_hist_lanes_kernel<16, false>), grid, dim3(256), lds, st, a);
        else hipLaunchKernelGGL((fwd_hist_lanes_kernel<32, false>), grid, dim3(256), lds, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_fwd(const FwdArgs& a, int nunits, int tiles, hipStream_t st)
{
    const dim3 grid(fwd_grid_x(a, nunits), (unsigned)tiles, 1);
    return a.vrows ? launch_fwd_vr<true>(a, grid, st) : launch_fwd_vr<false>(a, grid, st);
}

// Work units of one single-instance bucket: unit j covers clauses
// [j per, min((j + 1) per, Cb)).
__global__ void fwd_units_kernel(FwdUnit* __restrict__ u, int64_t n, int64_t per, int64_t Cb)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    FwdUnit w;
    w.inst = 0;
    w.pad = 0;
    w.c0 = j * per;
    w.c1 = (j + 1) * per < Cb ? (j + 1) * per : Cb;
    u[j] = w;
}

hipError_t launch_fwd_units(FwdUnit* u, int64_t n, int64_t per, int64_t Cb, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fwd_units_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, u, n, per, Cb);
    return hipGetLastError();
}

// Fixed device memory of the allocation-free forward entry point.  In host
// code the name stands for a host-side shadow: kernels get the device
// address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) uint8_t scratch[TSAT_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch_address(int device, void** out)
{
    static std::mutex mu;
    static void* addr[64] = {};
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

hipError_t launch_smin(const SminArgs& a, hipStream_t st)
{
    // the candidates of an evaluation without a loss or bookkeeping are
    // independent: as many blocks as they fill (a brute-force check has
    // millions)
    const unsigned tiles = (a.ictrl || a.loss_out) ? 1u : (unsigned)std::min(4096, (a.Np - 1) / 256 + 1);
    const size_t lds = (size_t)256 * (a.K1 | 1) * sizeof(uint32_t);
    hipLaunchKernelGGL(smin_kernel, dim3((unsigned)a.n_inst, tiles), dim3(256), lds, st, a);
    return hipGetLastError();
}

template <int J, bool MULTI>
static hipError_t launch_var_jm(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    const size_t lds = MULTI ? 0 : (size_t)a.K1 * a.Np * sizeof(float);
    if (a.rb && op != OP_NORMBWD && op != OP_BINARIZE) {
        switch (op) {
        case OP_STEP: hipLaunchKernelGGL((var_bytes_kernel<J, OP_STEP, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
        case OP_GRAD: hipLaunchKernelGGL((var_bytes_kernel<J, OP_GRAD, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
        default: hipLaunchKernelGGL((var_bytes_kernel<J, OP_ADJ, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
        }
        return hipGetLastError();
    }
    switch (op) {
    case OP_STEP: hipLaunchKernelGGL((var_kernel<J, OP_STEP, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
    case OP_GRAD: hipLaunchKernelGGL((var_kernel<J, OP_GRAD, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
    case OP_ADJ: hipLaunchKernelGGL((var_kernel<J, OP_ADJ, MULTI>), dim3(blocks), dim3(256), lds, st, a); break;
    case OP_NORMBWD: hipLaunchKernelGGL((norm_backward_kernel<J>), dim3(blocks), dim3(256), 0, st, a); break;
    default: {
        // several rows per wave once the variables fill the chip's waves
        // without it (256 CUs of 32); below that the rows run side by side
        constexpr int R = J <= 2 ? 8 : (J == 4 ? 4 : (J == 8 ? 2 : 1));
        const bool many = R > 1 && a.V >= 8192 * R;
        if (many) {
            const unsigned want = (unsigned)((a.V + 4 * R - 1) / (4 * R));
            hipLaunchKernelGGL((binarize_kernel<J, R>), dim3(want), dim3(256), 0, st, a);
        } else {
            hipLaunchKernelGGL((binarize_kernel<J, 1>), dim3(blocks), dim3(256), 0, st, a);
        }
        break;
    }
    }
    return hipGetLastError();
}

template <int J, int OP>
static hipError_t launch_heavy_op(const VarArgs& a, bool tail, int blocks, hipStream_t st)
{
    if (tail) hipLaunchKernelGGL((var_heavy_tail_kernel<J, OP>), dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((var_heavy_part_kernel<J, OP>), dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int J>
static hipError_t launch_heavy(const VarArgs& a, int op, bool tail, int blocks, hipStream_t st)
{
    switch (op) {
    case OP_STEP: return launch_heavy_op<J, OP_STEP>(a, tail, blocks, st);
    case OP_GRAD: return launch_heavy_op<J, OP_GRAD>(a, tail, blocks, st);
    default: return launch_heavy_op<J, OP_ADJ>(a, tail, blocks, st);
    }
}

template <int J>
static hipError_t launch_var_j(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    const bool split = a.heavy && a.n_chunks > 0 && op != OP_BINARIZE && op != OP_NORMBWD;
    if (split && !a.rb) {
        // partial sums of the heavy variables (the byte gather forms them with
        // the light variables), then the light variables, then the heavy tails
        hipError_t e = launch_heavy<J>(a, op, false, std::max(1, std::min((a.n_chunks + 3) / 4, blocks)), st);
        if (e != hipSuccess) return e;
    }
    hipError_t e = a.var_inst ? launch_var_jm<J, true>(a, op, blocks, st) : launch_var_jm<J, false>(a, op, blocks, st);
    if (e != hipSuccess || !split) return e;
    return launch_heavy<J>(a, op, true, std::max(1, std::min((a.n_heavy + 3) / 4, blocks)), st);
}

// resident blocks per CU of the kernel a launch with these arguments would use
template <class K>
static int occupancy_of(K kernel, size_t lds, int threads = 256)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

// the batched gather keeps its scalar registers
template <int J, int KO, int G, int OP, bool FULL>
static auto pure_kernel_ptr()
{
    if constexpr (G == 4 && J <= 4) return &var_pure_kernel<J, KO, G, OP, FULL>;
    else return &var_pure8_kernel<J, KO, G, OP, FULL>;
}

template <int J, int KO, int G, bool FULL>
static hipError_t launch_pure_jkgf(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    switch (op) {
    case OP_STEP: hipLaunchKernelGGL((pure_kernel_ptr<J, KO, G, OP_STEP, FULL>()), dim3(blocks), dim3(256), 0, st, a); break;
    case OP_GRAD: hipLaunchKernelGGL((pure_kernel_ptr<J, KO, G, OP_GRAD, FULL>()), dim3(blocks), dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((pure_kernel_ptr<J, KO, G, OP_ADJ, FULL>()), dim3(blocks), dim3(256), 0, st, a); break;
    }
    return hipGetLastError();
}

template <int J, int KO, int G>
static hipError_t launch_pure_jkg(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    if (a.N == 64 * J) return launch_pure_jkgf<J, KO, G, true>(a, op, blocks, st);
    return launch_pure_jkgf<J, KO, G, false>(a, op, blocks, st);
}

// records per scalar-load group (tuning knob): up to 4 for rows of up to 4
// words, 2 up to 8 words, else 1
static int pure_group(const VarArgs& a, int J)
{
    if (J <= 4 && a.group >= 4) return 4;
    if (J <= 8 && a.group >= 2) return 2;
    return 1;
}

template <int J, int KO>
static hipError_t launch_pure_jk(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    switch (pure_group(a, J)) {
    case 4: return launch_pure_jkg<J, KO, (J <= 4 ? 4 : 1)>(a, op, blocks, st);
    case 2: return launch_pure_jkg<J, KO, (J <= 8 ? 2 : 1)>(a, op, blocks, st);
    default: return launch_pure_jkg<J, KO, 1>(a, op, blocks, st);
    }
}

template <int J>
static hipError_t launch_pure_j(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    switch (a.pure_k) {
    case 2: return launch_pure_jk<J, 1>(a, op, blocks, st);
    case 3: return launch_pure_jk<J, 2>(a, op, blocks, st);
    default: return launch_pure_jk<J, 3>(a, op, blocks, st);
    }
}

template <int J, int KW, int OP, bool FULL>
static auto plane_kernel_ptr(bool window)
{
    return window ? &var_window_kernel<J, KW, OP, FULL> : &var_plane_kernel<J, KW, OP, FULL>;
}

template <int KW>
static hipError_t launch_pair_k(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    switch (op) {
    case OP_STEP: hipLaunchKernelGGL((var_window_pair_kernel<KW, OP_STEP>), dim3(blocks), dim3(256), 0, st, a); break;
    case OP_GRAD: hipLaunchKernelGGL((var_window_pair_kernel<KW, OP_GRAD>), dim3(blocks), dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((var_window_pair_kernel<KW, OP_ADJ>), dim3(blocks), dim3(256), 0, st, a); break;
    }
    return hipGetLastError();
}

// two variables per wave: window gather over packed planes, rows of at most
// 32 candidates (the host sets the flag together with the forward's layout)
static bool pair_rows(const VarArgs& a) { return a.packed != 0; }

template <int J, int KW, bool FULL>
static hipError_t launch_plane_jkf(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    if (J == 1 && pair_rows(a)) return launch_pair_k<KW>(a, op, blocks, st);
    const bool win = a.window != 0;
    switch (op) {
    case OP_STEP: hipLaunchKernelGGL((plane_kernel_ptr<J, KW, OP_STEP, FULL>(win)), dim3(blocks), dim3(256), 0, st, a); break;
    case OP_GRAD: hipLaunchKernelGGL((plane_kernel_ptr<J, KW, OP_GRAD, FULL>(win)), dim3(blocks), dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((plane_kernel_ptr<J, KW, OP_ADJ, FULL>(win)), dim3(blocks), dim3(256), 0, st, a); break;
    }
    return hipGetLastError();
}

template <int J>
static hipError_t launch_plane_j(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    const bool full = a.N == 64 * J;
    if (a.pure_k == 2) return full ? launch_plane_jkf<J, 2, true>(a, op, blocks, st) : launch_plane_jkf<J, 2, false>(a, op, blocks, st);
    return full ? launch_plane_jkf<J, 3, true>(a, op, blocks, st) : launch_plane_jkf<J, 3, false>(a, op, blocks, st);
}

// rows of more than four words: a team of ceil(W / 4) waves per block
template <int KW>
static auto team_kernel_ptr(int op)
{
    return op == OP_STEP ? var_window_team_kernel<KW, OP_STEP>
                         : (op == OP_GRAD ? var_window_team_kernel<KW, OP_GRAD> : var_window_team_kernel<KW, OP_ADJ>);
}

static int team_threads(const VarArgs& a) { return 64 * ((a.W + 3) / 4); }

static hipError_t launch_team(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    const auto k = a.pure_k == 2 ? team_kernel_ptr<2>(op) : team_kernel_ptr<3>(op);
    hipLaunchKernelGGL(k, dim3(blocks), dim3(team_threads(a)), 0, st, a);
    return hipGetLastError();
}

// mixed-width window gather: levels KT >= the widest clause (K1 - 1)
static int levels_of(const VarArgs& a) { return levels_for_width(a.K1 - 1); }

static size_t levels_lds(const VarArgs& a, int J, int KT)
{
    const size_t P = KT <= 3 ? 2 : 4;
    return 4 * P * J * 64 * 8 + (a.var_inst ? 4 : 1) * (size_t)(KT + 1) * J * 64 * 4;
}

template <int J, int KT>
static auto levels_kernel_ptr(int op)
{
    return op == OP_STEP ? var_window_levels_kernel<J, KT, OP_STEP>
                         : (op == OP_GRAD ? var_window_levels_kernel<J, KT, OP_GRAD> : var_window_levels_kernel<J, KT, OP_ADJ>);
}

// the iteration's update with every lane holding a candidate (N = 64 J):
// no per-lane candidate checks
template <int J, int KT>
static auto levels_kernel_full_ptr()
{
    return var_window_levels_kernel<J, KT, OP_STEP, true>;
}

template <int J>
static hipError_t launch_levels_j(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    const int KT = levels_of(a);
    const size_t lds = levels_lds(a, J, KT);
    if (op == OP_STEP && a.N == 64 * J) {
        switch (KT) {
        case 3: hipLaunchKernelGGL((levels_kernel_full_ptr<J, 3>()), dim3(blocks), dim3(256), lds, st, a); break;
        case 4: hipLaunchKernelGGL((levels_kernel_full_ptr<J, 4>()), dim3(blocks), dim3(256), lds, st, a); break;
        case 8: hipLaunchKernelGGL((levels_kernel_full_ptr<J, 8>()), dim3(blocks), dim3(256), lds, st, a); break;
        case 12: hipLaunchKernelGGL((levels_kernel_full_ptr<J, 12>()), dim3(blocks), dim3(256), lds, st, a); break;
        default: hipLaunchKernelGGL((levels_kernel_full_ptr<J, 15>()), dim3(blocks), dim3(256), lds, st, a); break;
        }
        return hipGetLastError();
    }
    switch (KT) {
    case 3: hipLaunchKernelGGL((levels_kernel_ptr<J, 3>(op)), dim3(blocks), dim3(256), lds, st, a); break;
    case 4: hipLaunchKernelGGL((levels_kernel_ptr<J, 4>(op)), dim3(blocks), dim3(256), lds, st, a); break;
    case 8: hipLaunchKernelGGL((levels_kernel_ptr<J, 8>(op)), dim3(blocks), dim3(256), lds, st, a); break;
    case 12: hipLaunchKernelGGL((levels_kernel_ptr<J, 12>(op)), dim3(blocks), dim3(256), lds, st, a); break;
    default: hipLaunchKernelGGL((levels_kernel_ptr<J, 15>(op)), dim3(blocks), dim3(256), lds, st, a); break;
    }
    return hipGetLastError();
}

template <int J>
static int occupancy_levels_j(const VarArgs& a)
{
    const int KT = levels_of(a);
    const size_t lds = levels_lds(a, J, KT);
    switch (KT) {
    case 3: return occupancy_of(levels_kernel_ptr<J, 3>(OP_STEP), lds);
    case 4: return occupancy_of(levels_kernel_ptr<J, 4>(OP_STEP), lds);
    case 8: return occupancy_of(levels_kernel_ptr<J, 8>(OP_STEP), lds);
    case 12: return occupancy_of(levels_kernel_ptr<J, 12>(OP_STEP), lds);
    default: return occupancy_of(levels_kernel_ptr<J, 15>(OP_STEP), lds);
    }
}

hipError_t launch_var(const VarArgs& a, int op, int blocks, hipStream_t st)
{
    // without the Eq. 5 normalization a gradient is the adjoint itself: no
    // theta to read
    if (op == OP_GRAD && a.mode != 1) op = OP_ADJ;
    const bool rowwise = op == OP_BINARIZE || op == OP_NORMBWD; // no gather
    if (a.occ_cid && a.planes && !a.rb && !rowwise && a.W > 4) return launch_team(a, op, blocks, st);
    if (a.occ_cid && a.planes && !a.rb && !rowwise) {
        if (a.pure_k == 2 || a.pure_k == 3) {
            switch (a.W) {
            case 1: return launch_plane_j<1>(a, op, blocks, st);
            case 2: return launch_plane_j<2>(a, op, blocks, st);
            default: return launch_plane_j<4>(a, op, blocks, st);
            }
        }
        switch (a.W) {
        case 1: return launch_levels_j<1>(a, op, blocks, st);
        case 2: return launch_levels_j<2>(a, op, blocks, st);
        default: return launch_levels_j<4>(a, op, blocks, st);
        }
    }
    const bool pure = a.pure_k >= 2 && a.pure_k <= 4 && !rowwise;
    switch (a.W) {
    case 1: return pure ? launch_pure_j<1>(a, op, blocks, st) : launch_var_j<1>(a, op, blocks, st);
    case 2: return pure ? launch_pure_j<2>(a, op, blocks, st) : launch_var_j<2>(a, op, blocks, st);
    case 3: case 4: return pure ? launch_pure_j<4>(a, op, blocks, st) : launch_var_j<4>(a, op, blocks, st);
    case 5: case 6: case 7: case 8: return pure ? launch_pure_j<8>(a, op, blocks, st) : launch_var_j<8>(a, op, blocks, st);
    default: return pure ? launch_pure_j<16>(a, op, blocks, st) : launch_var_j<16>(a, op, blocks, st);
    }
}

template <int J, int KO>
static int occupancy_pure(const VarArgs& a)
{
    switch (pure_group(a, J)) {
    case 4: return occupancy_of(pure_kernel_ptr<J, KO, (J <= 4 ? 4 : 1), OP_STEP, true>(), 0);
    case 2: return occupancy_of(pure_kernel_ptr<J, KO, (J <= 8 ? 2 : 1), OP_STEP, true>(), 0);
    default: return occupancy_of(pure_kernel_ptr<J, KO, 1, OP_STEP, true>(), 0);
    }
}

template <int J>
static int occupancy_j(const VarArgs& a, bool pure)
{
    if (!pure) {
        if (a.rb && a.var_inst) return occupancy_of(var_bytes_kernel<J, OP_STEP, true>, 0);
        if (a.rb) return occupancy_of(var_bytes_kernel<J, OP_STEP, false>, (size_t)a.K1 * a.Np * sizeof(float));
        if (a.var_inst) return occupancy_of(var_kernel<J, OP_STEP, true>, 0);
        return occupancy_of(var_kernel<J, OP_STEP, false>, (size_t)a.K1 * a.Np * sizeof(float));
    }
    switch (a.pure_k) {
    case 2: return occupancy_pure<J, 1>(a);
    case 3: return occupancy_pure<J, 2>(a);
    default: return occupancy_pure<J, 3>(a);
    }
}

int var_occupancy(const VarArgs& a, int op)
{
    const bool rowwise = op == OP_BINARIZE || op == OP_NORMBWD; // no gather
    if (a.occ_cid && a.planes && !a.rb && !rowwise && a.W > 4)
        return occupancy_of(a.pure_k == 2 ? team_kernel_ptr<2>(OP_STEP) : team_kernel_ptr<3>(OP_STEP), 0, team_threads(a));
    if (a.occ_cid && a.planes && !a.rb && !rowwise && a.pure_k != 2 && a.pure_k != 3) {
        switch (a.W) {
        case 1: return occupancy_levels_j<1>(a);
        case 2: return occupancy_levels_j<2>(a);
        default: return occupancy_levels_j<4>(a);
        }
    }
    if (a.occ_cid && a.planes && !a.rb && !rowwise) {
        const bool k2 = a.pure_k == 2, win = a.window != 0;
        if (pair_rows(a))
            return k2 ? occupancy_of(var_window_pair_kernel<2, OP_STEP>, 0) : occupancy_of(var_window_pair_kernel<3, OP_STEP>, 0);
        switch (a.W) {
        case 1: return occupancy_of(k2 ? plane_kernel_ptr<1, 2, OP_STEP, false>(win) : plane_kernel_ptr<1, 3, OP_STEP, false>(win), 0);
        case 2: return occupancy_of(k2 ? plane_kernel_ptr<2, 2, OP_STEP, false>(win) : plane_kernel_ptr<2, 3, OP_STEP, false>(win), 0);
        default: return occupancy_of(k2 ? plane_kernel_ptr<4, 2, OP_STEP, false>(win) : plane_kernel_ptr<4, 3, OP_STEP, false>(win), 0);
        }
    }
    const bool pure = a.pure_k >= 2 && a.pure_k <= 4 && !rowwise;
    switch (a.W) {
    case 1: return occupancy_j<1>(a, pure);
    case 2: return occupancy_j<2>(a, pure);
    case 3: case 4: return occupancy_j<4>(a, pure);
    case 5: case 6: case 7: case 8: return occupancy_j<8>(a, pure);
    default: return occupancy_j<16>(a, pure);
    }
}

hipError_t launch_expand(const uint64_t* bits, int64_t V, int W, int N, uint64_t* lits, hipStream_t st)
{
    const int64_t n = V * W;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(expand_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, bits, V, W, N, lits);
    return hipGetLastError();
}

hipError_t launch_pack(const float* assign, int V, int N, int W, uint64_t* bits, hipStream_t st)
{
    const int64_t words = (int64_t)V * W;
    if (words == 0) return hipSuccess;
    constexpr int R = 4;
    hipLaunchKernelGGL(pack_kernel<R>, dim3((unsigned)((words + 4 * R - 1) / (4 * R))), dim3(256), 0, st, assign, V, N,
                       W, bits);
    return hipGetLastError();
}

hipError_t launch_init_normal(float* theta, int64_t n, uint64_t seed, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(init_normal_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, theta, n, seed);
    return hipGetLastError();
}

hipError_t launch_strided_rows(const uint64_t* src, int64_t rows, int w, int64_t src_stride, uint64_t* dst,
                               hipStream_t st)
{
    const int64_t n = rows * w;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(strided_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, rows, w,
                       src_stride, dst);
    return hipGetLastError();
}

hipError_t launch_copy16(void* dst, const void* src, int64_t n16, int blocks, hipStream_t st)
{
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy16_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (uint4*)dst, (const uint4*)src, n16);
    return hipGetLastError();
}

hipError_t launch_init_proposal(const PropArgs& a, hipStream_t st)
{
    if (a.V <= 0) return hipSuccess;
    hipLaunchKernelGGL(init_proposal_kernel, dim3((unsigned)((a.V + 3) / 4)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t val, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, val);
    return hipGetLastError();
}

hipError_t launch_rank(const int64_t* sat, int N, int nsel, int32_t* order, int32_t* slot, hipStream_t st)
{
    hipLaunchKernelGGL(rank_kernel, dim3((N + 255) / 256), dim3(256), 0, st, sat, N, nsel, order, slot);
    return hipGetLastError();
}

hipError_t launch_select(const SelectArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)a.nchunks, (unsigned)((a.S + kSelTile - 1) / kSelTile));
    for (int pass = 0; pass < 4; ++pass) {
        hipLaunchKernelGGL(select_hist_kernel, grid, dim3(256), 0, st, a, pass);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(select_count_kernel, grid, dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(select_collect_kernel, grid, dim3(256), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(select_sort_kernel, dim3((unsigned)a.S), dim3(256), (size_t)a.kpow2 * sizeof(uint64_t), st, a);
    return hipGetLastError();
}

} // namespace tsat
