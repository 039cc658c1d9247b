// Readout kernels for gfx950, off the propagation loop: a per-generator comparison of two term
// lists (the stated error of an FP32 result against an FP64 one), and expectation values
// <psi|P|psi> = Tr(rho P) with rho = 2^-n prod_j (I + G_j) (paper, eq. (2)) from a device
// statevector: a random vector is projected onto the common +1 eigenspace of the generators,
// one (I + G_j)/2 at a time.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "qimax_internal.h"

namespace qimax {
namespace {

inline uint32_t blocks_for(uint64_t n, uint32_t block) { return (uint32_t)((n + block - 1) / block); }

// ----------------------------------------------------------------------------- compare
// Tiles of one side's segments (each tile inside one segment). For every element of side
// `a`, its key is searched in the same segment of side `b`: matched pairs add (wa - wb)^2,
// unmatched ones wa^2 (the other side's weight is 0). With count_ref set the pass is the
// second one (a = the reference list): it adds every wa^2 to the reference norm and only the
// unmatched elements to the difference. A key on whose side |w| > tau differs is counted.
constexpr int kCmpBlock = 256, kCmpItems = 16, kCmpTile = kCmpBlock * kCmpItems;

template <typename K>
__device__ __forceinline__ uint64_t lower_bound_k(const K* __restrict__ a, uint64_t lo, uint64_t hi, K key) {
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo) / 2;
    if (a[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

template <typename K, typename WA, typename WB>
__global__ void __launch_bounds__(kCmpBlock)
k_compare(const K* __restrict__ ka, const WA* __restrict__ wa, const K* __restrict__ kb, const WB* __restrict__ wb,
          const uint64_t* __restrict__ b_off, const uint64_t* __restrict__ t_begin, const uint64_t* __restrict__ t_end,
          const uint32_t* __restrict__ t_seg, int count_ref, double tau, double* __restrict__ acc,
          unsigned long long* __restrict__ cnt) {
  __shared__ uint64_t rng[2];
  __shared__ double red[2][kCmpBlock / 64];
  __shared__ unsigned long long redc[kCmpBlock / 64];
  const uint32_t t = blockIdx.x, s = t_seg[t];
  const uint64_t a0 = t_begin[t], a1 = t_end[t];
  const uint64_t lo = b_off[s], hi = b_off[s + 1];
  // the part of b's segment that can hold this tile's keys
  if (threadIdx.x == 0) rng[0] = lower_bound_k(kb, lo, hi, ka[a0]);
  if (threadIdx.x == 1) rng[1] = lower_bound_k(kb, lo, hi, ka[a1 - 1]) + 1;
  __syncthreads();
  const uint64_t r0 = rng[0], r1 = min(rng[1], hi);
  double d2 = 0.0, ref2 = 0.0;
  unsigned long long nd = 0;
  for (int r = 0; r < kCmpItems; ++r) {
    const uint64_t i = a0 + (uint64_t)r * kCmpBlock + threadIdx.x;
    if (i >= a1) break;
    const K key = ka[i];
    const double x = (double)wa[i];
    const uint64_t p = lower_bound_k(kb, r0, r1, key);
    const bool hit = p < r1 && kb[p] == key;
    const double y = hit ? (double)wb[p] : 0.0;
    if (count_ref) {
      ref2 += x * x;
      if (!hit) {
        d2 += x * x;
        nd += fabs(x) > tau;
      }
    } else {
      d2 += (x - y) * (x - y);
      nd += (fabs(x) > tau) != (fabs(y) > tau);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    d2 += __shfl_xor(d2, o, 64);
    ref2 += __shfl_xor(ref2, o, 64);
    nd += __shfl_xor(nd, o, 64);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wid] = d2;
    red[1][wid] = ref2;
    redc[wid] = nd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sd = 0.0, sr = 0.0;
    unsigned long long sc = 0;
    for (int w = 0; w < kCmpBlock / 64; ++w) {
      sd += red[0][w];
      sr += red[1][w];
      sc += redc[w];
    }
    atomicAdd(&acc[2 * s], sd);
    if (count_ref) atomicAdd(&acc[2 * s + 1], sr);
    atomicAdd(&cnt[s], sc);
  }
}

// ---------------------------------------------------------------------- statevector
// Basis state index i: qubit q is bit (n-1-q). A Pauli string with x mask xm, z mask zm
// (over those bits) and ny letters Y acts as P|i> = i^ny (-1)^{popcount(i & zm)} |i ^ xm>,
// so (P v)[k] = i^ny (-1)^{popcount((k ^ xm) & zm)} v[k ^ xm].

__device__ __forceinline__ uint64_t mix64(uint64_t x) {  // splitmix64 finaliser
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

__global__ void k_sv_random(double2* __restrict__ v, uint64_t D, uint64_t seed) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= D) return;
  const uint64_t a = mix64(seed ^ (2 * i)), b = mix64(seed ^ (2 * i + 1));
  v[i] = make_double2((double)(a >> 11) * 0x1.0p-53 - 0.5, (double)(b >> 11) * 0x1.0p-53 - 0.5);
}

// A generator's terms [T y/Y, T (y+1)/Y) applied to v by the blocks (., y) of a grid of
// ceil(D / kSvTile) x Y: part y at k = sum over those terms t of c_t (-1)^{popcount(src & z_t)}
// v[src], src = k ^ x_t. Small states have few amplitudes (n = 10: one tile), so the terms are
// split too, over the blocks and over the kSvGroups groups of a block, whose sums meet in LDS: a
// launch of D threads alone left 252 of 256 CUs idle. A wave holds 64 terms, one per lane, and
// reads them back as scalars; a coefficient w i^ny is real or imaginary, so a term costs two
// multiply-adds per amplitude and its kind is the same for the whole wave. v in LDS where it takes
// 32 KB at most (n <= 11).
// Bound by the LDS reads of v (16 KB a term, 128 cycles of a CU at n = 10) and the thirty or so
// vector instructions per term and thread; with one wave per SIMD the two did not overlap. One
// state at n = 10 with 177216 terms in ten generators: 15.3 ms with D threads in all, 0.25 ms with
// 346 blocks of four waves over terms staged in LDS, 0.14 ms here.
constexpr int kSvThreads = 256, kSvItems = 4, kSvTile = kSvThreads * kSvItems, kSvGroups = 4, kSvUnroll = 4;
// generators of fewer take blocks of one group: 5 to 7 us for them against 10 to 11, where four
// groups save 11 to 23 us of 28 to 64 on generators of 20 to 80 thousand terms
constexpr uint64_t kSvManyTerms = 1u << 14;
constexpr uint64_t kSvFewTerms = 16;

// v and the parts lie in slots of D amplitudes: v in slot vs (0 or 1), part y in the y-th of the
// others. With one part the projection is finished here, (v + g) / 2 written to the part's slot, which
// is v's from then on: one launch a generator where it took two (one string of states of three
// terms a generator: n = 11 125 -> 81 us, n = 14 157 -> 96, n = 18 224 -> 136; a thread per amplitude and two
// launches took 122, 147 and 213).
__device__ __forceinline__ uint64_t sv_slot(uint32_t y, uint32_t vs) { return y + (y >= vs ? 1u : 0u); }

constexpr uint32_t kSvLdsQubits = 11;
template <typename K, typename W, bool kLds, int kGroups>
__global__ void __launch_bounds__(kSvThreads * kGroups)
k_sv_apply(const K* __restrict__ keys, const W* __restrict__ w, uint64_t T, uint32_t n, double2* mem, uint32_t vs,
           uint64_t D) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ double2 sums[kGroups > 1 ? kGroups / 2 : 1][kSvTile];
  double2* const sv = (double2*)lds;
  const double2* __restrict__ const v = mem + vs * D;
  double2* __restrict__ const part = mem + sv_slot(blockIdx.y, vs) * D;
  if constexpr (kLds) {
    for (uint32_t i = threadIdx.x; i < (uint32_t)D; i += kSvThreads * kGroups) sv[i] = v[i];
    __syncthreads();
  }
  const uint32_t tid = threadIdx.x % kSvThreads, group = threadIdx.x / kSvThreads, lane = threadIdx.x & 63;
  const uint64_t k0 = (uint64_t)blockIdx.x * kSvTile + tid;
  const uint64_t p = (uint64_t)blockIdx.y * kGroups + group, np = (uint64_t)gridDim.y * kGroups;
  const uint64_t t0 = T * p / np, t1 = T * (p + 1) / np;
  // amplitude i of the thread is kb + 256 i, whose bits 8 and 9 are i's alone: the index of its
  // source is one XOR away from amplitude 0's, and its sign a constant of the term away
  static_assert(kSvThreads == 256 && kSvItems == 4, "an amplitude's bits 8 and 9");
  const uint32_t kb = (uint32_t)k0, mask = (uint32_t)(D - 1);
  double re[kSvItems] = {}, im[kSvItems] = {};
  for (uint64_t c0 = t0; c0 < t1; c0 += 64) {
    const uint32_t nt = __builtin_amdgcn_readfirstlane((uint32_t)min<uint64_t>(64, t1 - c0));
    const uint64_t t = min<uint64_t>(c0 + lane, t1 - 1);
    const K key = keys[t];
    const uint32_t lz = pack_bits((uint64_t)key >> 1), lx = pack_bits((uint64_t)key) ^ lz;  // below 2^30
    const uint32_t ny = (uint32_t)__popc(lx & lz);
    // bit 31 of x: an odd number of Ys; the weight's sign: two Ys more, and that of x & z
    const uint32_t lxo = lx | (ny << 31);
    const double wt = (double)w[t];
    const uint32_t lhi = (uint32_t)__double2hiint(wt) ^ (((ny >> 1) ^ ny) << 31), llo = (uint32_t)__double2loint(wt);
    for (uint32_t u0 = 0; u0 < nt; u0 += kSvUnroll) {
      uint32_t xo[kSvUnroll];
      double2 a[kSvUnroll][kSvItems];
#pragma unroll
      for (int j = 0; j < kSvUnroll; ++j) {
        xo[j] = __builtin_amdgcn_readlane(lxo, min(u0 + j, nt - 1));
        const uint32_t s0 = kb ^ (xo[j] & 0x7FFFFFFFu);
#pragma unroll
        for (int i = 0; i < kSvItems; ++i) {
          const uint32_t src = (s0 ^ (uint32_t)(i * kSvThreads)) & mask;  // (k past D: read, not used)
          a[j][i] = kLds ? sv[src] : v[src];
        }
      }
#pragma unroll
      for (int j = 0; j < kSvUnroll; ++j) {
        if (u0 + j >= nt) break;
        const uint32_t z = __builtin_amdgcn_readlane(lz, u0 + j);
        const uint32_t lo = __builtin_amdgcn_readlane(llo, u0 + j), hi0 = __builtin_amdgcn_readlane(lhi, u0 + j);
        // (-1)^{popcount(src & z)}: of amplitude 0's k per thread, of i for the block (of x: above)
        const uint32_t hi = hi0 ^ ((uint32_t)__popc(kb & z) << 31);
        double ck[kSvItems];
#pragma unroll
        for (int i = 0; i < kSvItems; ++i)
          ck[i] = __hiloint2double((int)(hi ^ ((uint32_t)__popc((uint32_t)(i * kSvThreads) & z) << 31)), (int)lo);
        if (xo[j] >> 31) {
#pragma unroll
          for (int i = 0; i < kSvItems; ++i) {
            re[i] -= ck[i] * a[j][i].y;
            im[i] += ck[i] * a[j][i].x;
          }
        } else {
#pragma unroll
          for (int i = 0; i < kSvItems; ++i) {
            re[i] += ck[i] * a[j][i].x;
            im[i] += ck[i] * a[j][i].y;
          }
        }
      }
    }
  }
#pragma unroll
  for (uint32_t half = kGroups / 2; half > 0; half /= 2) {
    if (group >= half && group < 2 * half) {
#pragma unroll
      for (int i = 0; i < kSvItems; ++i) sums[group - half][tid + i * kSvThreads] = make_double2(re[i], im[i]);
    }
    __syncthreads();
    if (group < half) {
#pragma unroll
      for (int i = 0; i < kSvItems; ++i) {
        re[i] += sums[group][tid + i * kSvThreads].x;
        im[i] += sums[group][tid + i * kSvThreads].y;
      }
    }
    __syncthreads();
  }
  if (group == 0) {
#pragma unroll
    for (int i = 0; i < kSvItems; ++i) {
      const uint64_t k = k0 + (uint64_t)i * kSvThreads;
      if (k >= D) continue;
      if (gridDim.y == 1) {
        const double2 a = kLds ? sv[k] : v[k];
        part[k] = make_double2(0.5 * (a.x + re[i]), 0.5 * (a.y + im[i]));
      } else {
        part[k] = make_double2(re[i], im[i]);
      }
    }
  }
}

// v = (v + g) / 2, the projection (I + G) / 2 applied given g = G v in Y parts: sixteen threads
// per amplitude each add every sixteenth part, then their sums in a fixed order.
constexpr int kSvSumLanes = 16, kSvSumAmps = 256 / kSvSumLanes;
__global__ void __launch_bounds__(256) k_sv_half_sum(double2* mem, uint32_t vs, uint64_t D, uint32_t Y) {
  __shared__ double2 sh[kSvSumLanes][kSvSumAmps];
  const uint32_t ka = threadIdx.x % kSvSumAmps, l = threadIdx.x / kSvSumAmps;
  const uint64_t k = (uint64_t)blockIdx.x * kSvSumAmps + ka;
  double2* __restrict__ const v = mem + vs * D;
  auto part = [&](uint32_t y) -> const double2* { return mem + sv_slot(y, vs) * D; };
  double re = 0.0, im = 0.0;
  if (k < D) {
    uint32_t y = l;
    for (; y + 3 * kSvSumLanes < Y; y += 4 * kSvSumLanes) {  // four loads in flight
      double2 p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = part(y + i * kSvSumLanes)[k];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        re += p[i].x;
        im += p[i].y;
      }
    }
    for (; y < Y; y += kSvSumLanes) {
      const double2 p = part(y)[k];
      re += p.x;
      im += p.y;
    }
  }
  sh[l][ka] = make_double2(re, im);
  __syncthreads();
  if (l == 0 && k < D) {
    for (int i = 1; i < kSvSumLanes; ++i) {
      re += sh[i][ka].x;
      im += sh[i][ka].y;
    }
    const double2 a = v[k];
    v[k] = make_double2(0.5 * (a.x + re), 0.5 * (a.y + im));
  }
}

// Block b of string y: sums over its amplitudes, sum |v|^2, Re sum conj(v) (P v) and Im of it; or with
// zall set (one row) sum |v|^2 and sum |v_i|^2 (1 - 2 bit_q(i)) for every qubit q (<Z_q>,
// unnormalised). acc[(y B + b) A ..] with B blocks a row and A sums a block: the host adds the
// blocks' in order.
constexpr uint32_t kSvMaxQubits = 32;  // statevectors hold at most 2^kSvMaxQubits amplitudes
constexpr int kSvBlock = 256;
__global__ void __launch_bounds__(kSvBlock) k_sv_reduce(const double2* __restrict__ v, uint64_t D, uint32_t n,
                                                       const SvString* __restrict__ str, int zall,
                                                       double* __restrict__ acc) {
  __shared__ double sh[kSvBlock / 64][1 + kSvMaxQubits];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  SvString p{0, 0, 0.0, 0.0};
  if (!zall) p = str[blockIdx.y];
  double nv = 0.0, pr = 0.0, pi = 0.0;
  double zq[kSvMaxQubits];
  const uint32_t nz = zall ? min(n, kSvMaxQubits) : 0u;
#pragma unroll
  for (uint32_t q = 0; q < kSvMaxQubits; ++q) zq[q] = 0.0;
  for (uint64_t i = (uint64_t)blockIdx.x * kSvBlock + threadIdx.x; i < D; i += (uint64_t)gridDim.x * kSvBlock) {
    const double2 a = v[i];
    const double p2 = a.x * a.x + a.y * a.y;
    nv += p2;
    if (zall) {
#pragma unroll
      for (uint32_t q = 0; q < kSvMaxQubits; ++q)
        if (q < nz) zq[q] += ((i >> (n - 1 - q)) & 1u) ? -p2 : p2;
    } else {
      const uint64_t src = i ^ p.x;
      const double2 b = v[src];
      const double sg = (__popcll(src & p.z) & 1) ? -1.0 : 1.0;
      const double br = sg * (p.re * b.x - p.im * b.y), bi = sg * (p.re * b.y + p.im * b.x);  // (P v)[i]
      pr += a.x * br + a.y * bi;
      pi += a.x * bi - a.y * br;
    }
  }
  auto wsum = [](double x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
  };
  nv = wsum(nv);
  if (lane == 0) sh[wid][0] = nv;
  if (zall) {
#pragma unroll
    for (uint32_t q = 0; q < kSvMaxQubits; ++q) {
      const double s = wsum(zq[q]);
      if (lane == 0 && q < nz) sh[wid][1 + q] = s;
    }
  } else {
    pr = wsum(pr);
    pi = wsum(pi);
    if (lane == 0) {
      sh[wid][1] = pr;
      sh[wid][2] = pi;
    }
  }
  __syncthreads();
  const uint32_t nacc = zall ? 1 + nz : 3;
  if (threadIdx.x < nacc) {
    double s = 0.0;
    for (int w = 0; w < kSvBlock / 64; ++w) s += sh[w][threadIdx.x];
    acc[((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * nacc + threadIdx.x] = s;
  }
}

}  // namespace

size_t compare_tile() { return (size_t)kCmpTile; }

// Device memory of qimax_compare_noalloc (the comparison's tile arrays, accumulators and
// counters), held by every GPU the library runs on until the process ends. Host code never
// passes the array's name to a kernel or copy: it uses the address hipGetSymbolAddress
// returns for the current device.
constexpr size_t kCompareScratchBytes = (size_t)4 << 20;
constexpr int kScratchDevices = 64;
static __device__ __align__(256) uint8_t scratch[kCompareScratchBytes];

hipError_t compare_scratch(int device, void** ptr, size_t* bytes) {
  static std::mutex mu;
  static void* addr[kScratchDevices] = {};
  if (device < 0 || device >= kScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = p;
  }
  *ptr = addr[device];
  *bytes = kCompareScratchBytes;
  return hipSuccess;
}

hipError_t launch_compare(int KC, int WPa, int WPb, const void* ka, const void* wa, const void* kb, const void* wb,
                          const uint64_t* b_off, const uint64_t* t_begin, const uint64_t* t_end, const uint32_t* t_seg,
                          uint32_t n_tiles, int count_ref, double tau, double* acc, unsigned long long* cnt,
                          hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
#define QIMAX_CMP(K, WA, WB)                                                                                     \
  k_compare<K, WA, WB><<<n_tiles, kCmpBlock, 0, s>>>((const K*)ka, (const WA*)wa, (const K*)kb, (const WB*)wb, \
                                                      b_off, t_begin, t_end, t_seg, count_ref, tau, acc, cnt)
#define QIMAX_CMP_W(K)                                      \
  do {                                                      \
    if (WPa == 64 && WPb == 64) QIMAX_CMP(K, double, double); \
    else if (WPa == 64) QIMAX_CMP(K, double, float);          \
    else if (WPb == 64) QIMAX_CMP(K, float, double);          \
    else QIMAX_CMP(K, float, float);                          \
  } while (0)
  if (KC == 0) QIMAX_CMP_W(uint32_t);
  else if (KC == 1) QIMAX_CMP_W(uint64_t);
  else QIMAX_CMP_W(unsigned __int128);
#undef QIMAX_CMP_W
#undef QIMAX_CMP
  return hipGetLastError();
}

hipError_t launch_sv_random(void* v, uint64_t D, uint64_t seed, hipStream_t s) {
  k_sv_random<<<blocks_for(D, 256), 256, 0, s>>>((double2*)v, D, seed);
  return hipGetLastError();
}

uint32_t sv_parts(uint64_t T, uint64_t D, size_t limit) {
  // about a block per CU, at least 16 terms for each, and no more parts than `limit` bytes hold
  const uint64_t tiles = (D + kSvTile - 1) / kSvTile;
  const uint64_t y = std::min<uint64_t>({(T + 15) / 16, std::max<uint64_t>(256 / tiles, 1), limit / (D * 16)});
  return (uint32_t)std::max<uint64_t>(y, 1);
}

hipError_t launch_sv_project(int KC, int WP, const void* keys, const void* w, uint64_t T, uint32_t n, void* mem,
                             uint32_t* vs, uint32_t Y, hipStream_t s) {
  const uint64_t D = 1ull << n;
  if (n < 1 || n > 30 || KC > 1 || Y < 1 || Y > 65535 || *vs > 1) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)((D + kSvTile - 1) / kSvTile), Y);
  // (a few terms a thread are read from L2 sooner than the state is staged)
  const bool lds = n <= kSvLdsQubits && T > kSvFewTerms;
  const size_t bytes = lds ? (size_t)D * 16 : 0;
#define QIMAX_SVA_G(K, W, L, G) \
  k_sv_apply<K, W, L, G><<<grid, kSvThreads * G, bytes, s>>>((const K*)keys, (const W*)w, T, n, (double2*)mem, *vs, D)
#define QIMAX_SVA(K, W, L) do { if (T >= kSvManyTerms) QIMAX_SVA_G(K, W, L, kSvGroups); else QIMAX_SVA_G(K, W, L, 1); } while (0)
#define QIMAX_SVA_L(K, W) do { if (lds) QIMAX_SVA(K, W, true); else QIMAX_SVA(K, W, false); } while (0)
  if (KC == 0) {
    if (WP == 64) QIMAX_SVA_L(uint32_t, double); else QIMAX_SVA_L(uint32_t, float);
  } else {
    if (WP == 64) QIMAX_SVA_L(uint64_t, double); else QIMAX_SVA_L(uint64_t, float);
  }
#undef QIMAX_SVA_L
#undef QIMAX_SVA
#undef QIMAX_SVA_G
  if (Y == 1)
    *vs ^= 1u;
  else
    k_sv_half_sum<<<blocks_for(D, kSvSumAmps), 256, 0, s>>>((double2*)mem, *vs, D, Y);
  return hipGetLastError();
}

uint32_t sv_reduce_blocks(uint32_t n, uint32_t rows, bool zall, size_t limit) {
  // eight amplitudes a thread (every <Z_q> at n = 14: one block 45 us, eight 10), and blocks enough for
  // the chip over all rows
  const uint64_t D = 1ull << n, per = 8ull * (zall ? 1 + n : 3) * std::max(rows, 1u);
  return (uint32_t)std::max<uint64_t>(
      std::min<uint64_t>({(D + kSvBlock * 8 - 1) / (kSvBlock * 8), std::max(4096u / std::max(rows, 1u), 1u), 1024,
                          limit / per}), 1);
}

hipError_t launch_sv_reduce(const void* v, uint32_t n, const SvString* str, uint32_t k, uint32_t blocks, double* acc,
                            hipStream_t s) {
  if (k > 65535 || n > kSvMaxQubits || blocks < 1) return hipErrorInvalidValue;
  const bool zall = str == nullptr;
  const uint32_t rows = zall ? 1 : k;
  if (rows == 0) return hipSuccess;
  k_sv_reduce<<<dim3(blocks, rows), kSvBlock, 0, s>>>((const double2*)v, 1ull << n, n, str, zall ? 1 : 0, acc);
  return hipGetLastError();
}

}  // namespace qimax
