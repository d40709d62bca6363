// attn_bwd.hip -- deterministic attention backward for gfx950: the kernels
// around the main kernel, the d = 128 main kernel's instantiation, and the
// launch sequence of a backward call.
//
// bwd_pre  : D = rowsum(dO o O) per query row in fp32 (Algorithm 1, the
//            preprocessing kernel); resets the ordering counters, the work
//            ticket and the error flag (and dQacc for the atomic variant).
// bwd_main : the KV-tile kernels with the ordered dQ reduction: 128-row tiles
//            (bwd_main.h; d = 128 here, d = 64 in attn_bwd_d64.hip), 256-row
//            d = 64 tiles (attn_bwd64w.hip), d = 256 (attn_bwd256.hip).
// bwd_post : atomic variant only: dQ = bf16(s * dQacc).
// bwd_sum_partials : PARTIALS variant: the fixed-order sum of the partials.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "bwd_common.h"
#include "bwd_main.h"

namespace dash {


// ---------------------------------------------------------------- bwd_pre
// Memory-bound: O and dO are read once.  A wave takes U times 64 / TPR rows in
// a row, all their loads issued before the first is used, and writes their D
// and L with one store each.  O, which nothing reads again, is loaded past the
// caches that dO stays in for the main kernel (not beside the atomic variant's
// zeroing of its accumulator: 15.1 us there, 17.6 with it, 919 heads of 192 at d = 64).
// Measured (us, one row per thread -> four): 16 MB of O and dO each 8.1 -> 7.1,
// 67 MB 27.4 -> 22.9 (5.9 TB/s), 134 MB 55.4 -> 53.3.
template <int D, int U, bool ZERO>
__global__ __launch_bounds__(256) void bwd_pre_kernel(BwdArgs a) {
  constexpr int TPR = D / 8;    // threads per row, 8 elements each
  constexpr int RPL = 64 / TPR;  // rows of a wave's load instruction
  static_assert(U <= TPR, "lane c of a row writes row c of its U");
  const unsigned gtid = blockIdx.x * 256u + threadIdx.x;  // (at most 2^24 threads)
  const unsigned nthreads = gridDim.x * 256u;
  const long rows = (long)a.bh * a.n;
  const int l = threadIdx.x & 63, c = l % TPR;
  // the grid covers every row once, except where the number of workgroups is capped
  for (long row0 = (long)(gtid >> 6) * (RPL * U); row0 < rows; row0 += (long)(nthreads >> 6) * (RPL * U)) {
    u32x4 x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      long row = row0 + u * RPL + l / TPR;
      row = row < rows ? row : rows - 1;  // (read, not written)
      x[u] = *(const u32x4*)((const __bf16*)a.dO + row * D + 8 * c);
      const u32x4* o = (const u32x4*)((const __bf16*)a.o + row * D + 8 * c);
      y[u] = ZERO ? *o : __builtin_nontemporal_load(o);
    }
    float mine = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float xf = bf16_to_f32((unsigned short)(x[u][e >> 1] >> (16 * (e & 1))));
        const float yf = bf16_to_f32((unsigned short)(y[u][e >> 1] >> (16 * (e & 1))));
        acc = __builtin_fmaf(xf, yf, acc);
      }
      // butterfly over the TPR lanes of a row: a+b == b+a exactly, so every lane
      // ends with the same bits and the tree is fixed
#pragma unroll
      for (int off = 1; off < TPR; off <<= 1) acc += __shfl_xor(acc, off);
      mine = c == u ? acc : mine;
    }
    const long row = row0 + c * RPL + l / TPR;
    if (c < U && row < rows) {
      a.dvec[row] = mine;
      a.lse2[row] = a.lse[row] * kLog2e;
    }
  }

  const unsigned nctr = (unsigned)a.bh * (unsigned)a.nblk;
  const int init = a.poison ? kPoison : 0;
  for (unsigned i = gtid; i < nctr; i += nthreads) a.counters[(size_t)i * kCtrStride] = init;
  if (gtid == 0) {
    a.ctrl[kCtrlTicket] = 0;
    a.ctrl[kCtrlError] = 0;
    if (a.status) *a.status = 0;
  }
  if (gtid < kMaxXcd) a.ctrl[kCtrlXcdTicket + gtid] = 0;
  // every chain's step table (the same for every head): entry 0 is the number
  // of steps; entry 1 + st is step st, i.e. 64-row block pb of Q tile i with
  // KV tile j, its rank in the block's summation order and whether it is the
  // last one (see pack_step)
  {
    const Geom& G = a.G;
    const int bc = G.bc;
    const unsigned ntab = (unsigned)G.chains * (unsigned)a.step_cap;
    for (unsigned x = gtid; x < ntab; x += nthreads) {
      const int w = (int)(x / (unsigned)a.step_cap), e = (int)(x % (unsigned)a.step_cap);
      const int len = chain_len(G, w) * G.nsub;
      if (e == 0) {
        a.steps[x] = (unsigned)len;
        continue;
      }
      const int st = e - 1;
      if (st >= len) continue;
      int j, i;
      task(G, w, st / G.nsub, &j, &i);
      const int pb = i * G.nsub + st % G.nsub;
      const int rank = rank_of(G, i, j);
      a.steps[x] = (pb * kBlockRows < a.n && j * bc < a.n) ? pack_step(pb, j, rank, rank == contributors(G, i) - 1) : kNoStep;
    }
    // work ticket -> (head, chain); XCD-local placement: one segment of
    // xcd_cap tickets per XCD
    if (a.nxcd > 0) {
      const unsigned nitems = (unsigned)a.nxcd * (unsigned)a.xcd_cap;
      for (unsigned x = gtid; x < nitems; x += nthreads) {
        const int q = (int)(x / (unsigned)a.xcd_cap), t = (int)(x % (unsigned)a.xcd_cap);
        if (t >= xcd_heads(a.bh, a.nxcd, q) * G.chains) continue;
        int bh, w;
        ticket_chain_xcd(G, a.bh, a.nxcd, q, t, &bh, &w);
        a.order[2 * (size_t)x] = bh;
        a.order[2 * (size_t)x + 1] = w;
      }
    } else {
      const unsigned nitems = (unsigned)a.bh * (unsigned)G.chains;
      for (unsigned x = gtid; x < nitems; x += nthreads) {
        int bh, w;
        ticket_chain(G, a.bh, (int)x, &bh, &w);
        a.order[2 * (size_t)x] = bh;
        a.order[2 * (size_t)x + 1] = w;
      }
    }
  }
  if (ZERO) {
    const long n4 = (long)a.bh * a.n * D / 4;
    for (long i = gtid; i < n4; i += (long)nthreads) ((f32x4*)a.dqacc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// ---------------------------------------------------------------- bwd_post
template <int D>
__global__ __launch_bounds__(256) void bwd_post_kernel(BwdArgs a) {
  const long n8 = (long)a.bh * a.n * D / 8;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long)gridDim.x * 256) {
    const f32x4 x = ((const f32x4*)a.dqacc)[2 * i];
    const f32x4 y = ((const f32x4*)a.dqacc)[2 * i + 1];
    const float s = a.scale;
    u32x4 r = {pack_bf16(x[0] * s, x[1] * s), pack_bf16(x[2] * s, x[3] * s), pack_bf16(y[0] * s, y[1] * s),
               pack_bf16(y[2] * s, y[3] * s)};
    ((u32x4*)a.dq)[i] = r;
  }
}

// ---------------------------------------------------------------- bwd_sum_partials
// PARTIALS variant: dQ = bf16(s * sum_j partial_j), the partials of each
// 64-row block added in ascending KV order (the order NAIVE's counters
// enforce, so the result is bitwise NAIVE's).  Partial j of block pb of head
// bh is the register-order block at ((bh * T_c + j) * nblk + pb) * 64 * D; one
// thread per 4 floats, consecutive threads on consecutive 16-byte pieces.
template <int D>
__global__ __launch_bounds__(256) void bwd_sum_partials_kernel(BwdArgs a) {
  constexpr int BM = kBlockRows;
  constexpr int PER = BM * D / 4;  // f32x4 pieces per block
  const long total = (long)a.bh * a.nblk * PER;
  const size_t stride_j = (size_t)a.nblk * BM * D;
  for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
    const int e4 = (int)(idx % PER);
    const long bp = idx / PER;
    const int pb = (int)(bp % a.nblk), bh = (int)(bp / a.nblk);
    // register order: 32 x 32 tile T = 2 * (d block) + (query half) of 1024
    // floats, 1 KB chunk rb of 256 floats, lane l of 4 floats
    const int T = e4 >> 8, rb = (e4 >> 6) & 3, l = e4 & 63;
    const int q = pb * BM + 32 * (T & 1) + (l & 31);
    const int col = 32 * (T >> 1) + 8 * rb + 4 * (l >> 5);
    if (q >= a.n) continue;
    const int c = contributors(a.G, pb / a.G.nsub);
    const f32x4* p = (const f32x4*)(a.dqacc + ((size_t)bh * a.tc * a.nblk + pb) * BM * D) + e4;
    f32x4 s = p[0];
    for (int j = 1; j < c; ++j) s = s + p[j * stride_j / 4];
    const float sc = a.scale;
    u32x2 t = {pack_bf16(s[0] * sc, s[1] * sc), pack_bf16(s[2] * sc, s[3] * sc)};
    *(u32x2*)((__bf16*)a.dq + ((size_t)bh * a.n + q) * D + col) = t;
    if (a.dq_accum) *(f32x4*)(a.dq_accum + ((size_t)bh * a.n + q) * D + col) = s;
  }
}

template <int D>
hipError_t launch_all(const BwdArgs& a, int grid_main, hipStream_t stream) {
  const bool atomic = a.G.sched == S_ATOMIC;
  // four rows per thread from 4096 such workgroups on (d = 64 / 128 / 256: 8.0
  // -> 7.2 us there, 27 -> 23 at 16384); at 2048 both take 5.0 and below that
  // (1024: 4.2-4.6 against 4.3-4.8) more waves are worth more
  const long one = ((long)a.bh * a.n * (D / 8) + 255) / 256;  // workgroups of one row per thread group
  const long four = (one + 3) / 4;
  const dim3 grid((unsigned)(one < 4096 ? one : four < 65536 ? four : 65536));
  if (one < 4096)
    hipLaunchKernelGGL((atomic ? bwd_pre_kernel<D, 1, true> : bwd_pre_kernel<D, 1, false>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((atomic ? bwd_pre_kernel<D, 4, true> : bwd_pre_kernel<D, 4, false>), grid, dim3(256), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.ev_begin) (void)hipEventRecord(a.ev_begin, stream);
  if constexpr (D == 256)
    e = a.G.bc == 128 ? launch_mainw(a, D, grid_main, stream) : launch_main256(a, grid_main, stream);
  else if constexpr (D == 64)
    e = a.G.bc == 256 ? launch_main64w(a, grid_main, stream) : launch_main64(a, grid_main, stream);
  else
    e = a.G.bc == 256 ? launch_mainw(a, D, grid_main, stream) : launch_main<D>(a, grid_main, stream);
  if (e != hipSuccess) return e;
  if (a.ev_end) (void)hipEventRecord(a.ev_end, stream);
  if (atomic) hipLaunchKernelGGL(bwd_post_kernel<D>, dim3(1024), dim3(256), 0, stream, a);
  if constexpr (D <= 128) {
    if (a.G.sched == S_PARTIALS) hipLaunchKernelGGL(bwd_sum_partials_kernel<D>, dim3(4096), dim3(256), 0, stream, a);
    if (a.G.sched == S_SPLIT) (void)launch_dq(a, D, stream);
  }
  return hipGetLastError();
}

hipError_t launch_bwd(const BwdArgs& a, int d, int grid_main, hipStream_t stream) {
  if (d == 64) return launch_all<64>(a, grid_main, stream);
  if (d == 128) return launch_all<128>(a, grid_main, stream);
  return launch_all<256>(a, grid_main, stream);
}

int bwd_main_occupancy(int d) {
  if (d == 64) {
    const int a = main64_occupancy(), b = bwd_main64w_occupancy();
    return a < b ? a : b;
  }
  const int a = d == 128 ? main_occupancy<128>() : bwd_main256_occupancy(), b = bwd_mainw_occupancy(d);
  return a < b ? a : b;
}

}  // namespace dash
