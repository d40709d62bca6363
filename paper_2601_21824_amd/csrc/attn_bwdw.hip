// attn_bwdw.hip -- the backward main kernel with wide KV tiles at head dims 128
// (256 rows) and 256 (128 rows): twice the rows of bwd_main_kernel<128> and
// bwd_main256_kernel, i.e. half the fp32 accumulator traffic and half the Q / dO
// copies per FLOP.
//
// Same method and protocol as bwd_main.h.  Four waves, one per SIMD with all 512
// registers: a wave owns NKB blocks of 32 keys (2 at d = 128, 1 at d = 256) and
// its dK, dV accumulators are exactly the 256 AGPRs, held there by the asm of
// mfma32_acc (the compiler, choosing by itself, puts the MFMA results of S and
// dP there as well and spills).  V rows stay in VGPRs; the K tile (64 KB) is in
// LDS, read as rows for S = Q K^T and transposed for dQ^T = K^T dS^T.
//
// A chain's 64-row block steps are run as two sub-steps of 32 queries, so that S
// and dP take 32 NKB registers, and dQ^T trails one sub-step:
//   phase 1   S, dP of sub-step i          beside: the copies of i + 1
//   phase 2   dQ^T of sub-step i - 1       beside: P of i (exp)
//   phase 3a  dV += P^T dO of i            beside: dS of i, the ordered add and the
//                                          stores of dQ^T of i - 1
//   phase 3b  dK += dS^T Q of i            beside: dS^T of i into LDS, the loads of
//                                          the accumulator slice for dQ^T of i
// Each phase is 16 MFMAs (phase 1: 32).  One workgroup barrier per sub-step: it
// publishes Q / dO of i and dS^T of i - 1 (both double-buffered by the sub-step's
// parity, which is its half h of the block).  The accumulator slice goes to
// registers directly, as the block's 32 queries leave room for it.
//
// What bounds it: the issue of one wave per SIMD.  Of the about 6,000 cycles of a
// sub-step (d = 128, full) the matrix cores are busy 2,560; the wave's 460 VALU
// instructions, its 80 MFMAs among them, are active for about 2,000, its LDS instructions
// for 650, and it waits for about 1,300 (hardware counters over the benchmark's
// launch, at 1.93 GHz).  The LDS reads of phase 1 (128 KB
// per CU) take longer than its MFMAs, and the accumulator's 1 KB device-coherent
// loads and stores cost a wave 100-300 cycles each where they stand close together,
// hence one per 2-4 MFMAs.
//
// Measured (main kernel and bwd_pre, us, narrow tile -> this): d = 128, 32 heads of
// 8192 full 3901 -> 3176 (705 -> 866 TFLOP/s), 64 heads causal 4199 -> 3360; d =
// 256, 8 heads of 32768 causal 28727 -> 15241 (383 -> 721), full 58085 -> 29292.
//
// The order of the sums and the counters are those of bwd_main.h: a block's turn
// is taken before its first half is added and released after its second.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "bwd_common.h"
#include "lds_layout.h"

namespace dash {
namespace {

constexpr int BM = kBlockRows;   // rows of a Q block (one counter)
constexpr int SQ = 32;           // rows of a sub-step
constexpr int NW = 4, NT = 256;  // waves, threads

template <int D>
struct SmemW {
  static constexpr int BC = 32768 / D;  // KV rows per tile: 256 at d = 128, 128 at d = 256
  __bf16 kt[BC * D];                    // K tile [kv][d] (bf_at); between two tiles: store pads of the waves
  __bf16 qs[2][SQ * D];                 // Q rows of sub-step h of a block (bf_at)
  __bf16 dos[2][SQ * D];                // dO rows
  __bf16 dst[2][BC * SQ];               // dS^T [kv][32 q] (dst32_at)
  float ls[2][BM];                      // L * log2(e) of a block's rows, by block parity
  float ds[2][BM];                      // D
  unsigned steps[kMaxChainSteps];       // this chain's blocks (pack_step)
  int poll[NW][64];                     // per wave: the block's counter
  int item;
};

// dK / dV MFMA with the accumulator in AGPRs.  The compiler does not see an MFMA
// here, so its wait states are the caller's: B comes from LDS, A (P^T, dS^T) is
// packed at least one MFMA earlier, and reading c takes acc_settle first.
__device__ inline void mfma32_acc(bf16x8 a, bf16x8 b, f32x16& c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// 20 wait states: more than any MFMA's result takes
__device__ inline void acc_settle(f32x16& c) { asm volatile("s_nop 15\n\ts_nop 3" : "+a"(c)); }

__device__ inline bf16x8 lds16(uint32_t at) { return *(const __attribute__((address_space(3))) bf16x8*)(at); }
__device__ inline f32x4 lds16f(uint32_t at) { return *(const __attribute__((address_space(3))) f32x4*)(at); }
__device__ inline void lds_st8(uint32_t at, u32x2 v) { *(__attribute__((address_space(3))) u32x2*)(at) = v; }
__device__ inline bf16x8 lds_tr2(uint32_t a, uint32_t b) {
  typedef short s16x4 __attribute__((__vector_size__(8)));
  typedef __attribute__((address_space(3))) s16x4* p;
  return as_bf16x8(__builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((p)(a))),
                   __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((p)(b))));
}
// as vm_wait_le with the counts that occur here
__device__ inline void vm_wait_few(int n) {
  if (n >= 16) vm_wait<16>();
  else if (n >= 8) vm_wait<8>();
  else if (n >= 4) vm_wait<4>();
  else vm_wait<0>();
}

template <int D, bool CAUSAL, int MODE, bool STATS = false>
__global__ __launch_bounds__(NT) void bwd_mainw_kernel(BwdArgs a) {
  using SM = SmemW<D>;
  constexpr int BC = SM::BC;
  constexpr int NKB = BC / 128;   // 32-key blocks per wave
  constexpr int KS = D / 16;      // k-steps over d
  constexpr int KSC = BC / 16;    // k-steps over the tile's keys
  constexpr int NB = D / 32;      // 32-column blocks of d
  constexpr int DQT = NB / NW;    // 32 x 32 dQ^T tiles per wave and sub-step
  constexpr int NACC = 4 * DQT;   // its accumulator slice in 1 KB chunks
  constexpr int CPR = D / 8;      // 16-byte chunks per row
  constexpr int QP = SQ * CPR / NT;  // direct copies per thread of a sub-step's Q (or dO) rows
  constexpr int KP = BC * CPR / NT;  // ... of the K tile
  static_assert(QP * 4096 == SQ * D * 2 && KP == 16 && NB * 2 * NKB == 16 && KSC * DQT == 16, "shape");
  __shared__ __attribute__((aligned(1024))) SM sm;

  const Geom G = a.G;
  const int N = a.n;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float c2 = a.scale * kLog2e;
  const uint32_t hbytes = (uint32_t)((size_t)N * D * 2);
  constexpr bool ordered = MODE == kModeOrdered;
  const bool xcd = a.nxcd > 0;
  const int xq = xcd ? xcc_id() : 0;
  const int total = xcd ? (xq < a.nxcd ? xcd_heads(a.bh, a.nxcd, xq) * G.chains : 0) : a.bh * G.chains;
  int* const ticket = &a.ctrl[xcd ? kCtrlXcdTicket + xq : kCtrlTicket];
  const int* const order = a.order + (xcd ? 2 * xq * a.xcd_cap : 0);
  const uint32_t sm_lds = lds_base(&sm);
  auto lds_of = [&](const void* p) { return sm_lds + (uint32_t)((const char*)p - (const char*)&sm); };
  // Shift-type orders: the next contributor to a block reaches it two or more
  // blocks later, so the counter release waits until the next sub-step, when
  // the stores have drained without a wait of their own
  const bool deferred = G.sched == S_SHIFT || G.sched == S_SYMSHIFT;
  bool failed = false;
  WaitStats wst;
  if constexpr (STATS) stats_wave_begin(wst);

  for (;;) {
    if (tid == 0) sm.item = atomicAdd(ticket, 1);
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(sm.item);
    if (item >= total) break;
    const int bh = __builtin_amdgcn_readfirstlane(order[2 * item]);
    const int wch = __builtin_amdgcn_readfirstlane(order[2 * item + 1]);
    const size_t head = (size_t)bh * N * D;
    const auto rq = make_rsrc((const __bf16*)a.q + head, hbytes);
    const auto rk = make_rsrc((const __bf16*)a.k + head, hbytes);
    const auto rdo = make_rsrc((const __bf16*)a.dO + head, hbytes);
    int* ctr_head = a.counters + (size_t)bh * a.nblk * kCtrStride;
    const auto rctr = make_rsrc(ctr_head, (uint32_t)a.nblk * kCtrStride * 4);

    const unsigned* tab = a.steps + (size_t)wch * a.step_cap;
    const int nsteps = __builtin_amdgcn_readfirstlane((int)tab[0]);
    for (int st = tid; st < nsteps; st += NT) sm.steps[st] = tab[1 + st];
    __syncthreads();

    int cur_j = -1;
    bf16x8 vreg[NKB][KS];                       // V rows of the wave's keys (B of dP = dO V^T)
    f32x16 dkacc[NKB][NB], dvacc[NKB][NB];      // in AGPRs
    f32x16 dq[DQT];                             // dQ^T of the sub-step before
    f32x4 old[NACC];                            // its accumulator slice
    // the sub-step before: its block (half h ^ 1), whether there is one, its turn
    int p_pb = 0;
    bool p_valid = false, p_last = false, p_turn = false, p_add = false;
    int rel_pb = -1;   // block whose stores are issued and whose counter this wave still has to advance
    int vm_st = 0;     // vector memory operations since the copies of the coming sub-step
    int bpar = 0;      // parity of the current block (L, D buffers)

    auto step_at = [&](int st) -> unsigned { return __builtin_amdgcn_readfirstlane(sm.steps[st]); };
    auto next_valid = [&](int st) {
      while (st < nsteps && step_at(st) == kNoStep) ++st;
      return st;
    };
    // part k of the Q and dO rows of half h of block pb into buffer h
    auto load_part = [&](int pb, int h, int k) {
      const int t0 = 64 * w + fresh_lane();
      const int r = t0 / CPR + k * (NT / CPR), c = (t0 % CPR) ^ tile_swz<D>(r);
      const uint32_t at = lds_of(&sm.qs[h][0]) + 1024u * w + 4096u * k;
      dma16_pair(rq, rdo, at, at + (uint32_t)sizeof(sm.qs), (uint32_t)((pb * BM + SQ * h + r) * D + 8 * c) * 2, 0);
    };
    auto load_ld = [&](int pb, int par) {  // L * log2(e) and D of a block's rows
      const uint32_t row = (uint32_t)(pb * BM + fresh_lane());
      // padded rows of a ragged last block read L = D = 0 (P = 1 there), and
      // their Q and dO rows read 0: they add nothing to dK and dV
      if (w == 0) dma4(make_rsrc(a.lse2 + (size_t)bh * N, (uint32_t)N * 4), lds_of(&sm.ls[par][0]), row * 4);
      if (w == 1) dma4(make_rsrc(a.dvec + (size_t)bh * N, (uint32_t)N * 4), lds_of(&sm.ds[par][0]), row * 4);
    };
    auto poll_copy = [&](int pb) { dma4_coherent(rctr, lds_of(&sm.poll[w][0]), (uint32_t)pb * kCtrStride * 4); };
    // The accumulator in register order, as bwd_sum_partials reads it: block pb
    // is BM*D floats at pb*BM*D, 32 x 32 tile T = 2 (d block) + (query half) at
    // T*1024, chunk rb of lane l at rb*256 + 4l: row 32 half + l%32 of the block,
    // columns 32 (d block) + 8rb + 4(l/32) .. +3.  Wave w: d blocks w DQT ...
    auto acc_off = [&](int pb, int h, int k) {  // wave-uniform part
      return (uint32_t)(pb * BM * D + (2 * (w * DQT + (k >> 2)) + h) * 1024 + (k & 3) * 256) * 4;
    };
    // An accumulator slice is loaded and stored by straight-line code in every
    // sub-step: where there is nothing to load or store, the descriptor covers 0
    // bytes (loads read 0, stores are dropped).  Behind a branch the compiler
    // loses count of what is in flight and waits for everything, the stores of
    // the chunk before included, at every chunk.
    auto acc_rsrc = [&](bool on) {
      return make_rsrc(a.dqacc + (size_t)bh * a.nblk * BM * D, on ? (uint32_t)a.nblk * BM * D * 4 : 0u);
    };
    auto load_old1 = [&](__amdgpu_buffer_rsrc_t r, int pb, int h, int k, int lane) {
      old[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, 16 * lane, acc_off(pb, h, k), kCoherent));
    };
    auto load_old = [&](int pb, int h, bool add) {
      const int lf = fresh_lane();
      const auto r = acc_rsrc(add);
#pragma unroll
      for (int k = 0; k < NACC; ++k) load_old1(r, pb, h, k, lf);
    };
    auto release = [&]() {
      if (fresh_lane() == 0 && rel_pb >= 0)
        __hip_atomic_fetch_add(ctr_head + (size_t)rel_pb * kCtrStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      rel_pb = -1;
    };
    // chunk k of dQ^T of half h of block pb: added to the slice (the first
    // contributor: as it is) and stored; the last contributor also writes bf16 s*dQ
    auto put = [&](__amdgpu_buffer_rsrc_t r, int pb, int h, bool add, bool last, int k, int lf) {
      const int t = k >> 2, rb = k & 3;
      f32x4 v = {dq[t][4 * rb], dq[t][4 * rb + 1], dq[t][4 * rb + 2], dq[t][4 * rb + 3]};
      if constexpr (MODE == kModePartials) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, 16 * lf, acc_off(pb, h, k), 0);
      } else {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float sum = old[k][x] + v[x];
          v[x] = add ? sum : v[x];
        }
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, 16 * lf, acc_off(pb, h, k), kCoherent);
        if (last) {
          const uint32_t off = (uint32_t)((pb * BM + SQ * h + (lf & 31)) * D + 32 * (w * DQT + t) + 8 * rb + 4 * (lf >> 5));
          st8(make_rsrc((__bf16*)a.dq + head, hbytes), off * 2,
              u32x2{pack_bf16(v[0] * a.scale, v[1] * a.scale), pack_bf16(v[2] * a.scale, v[3] * a.scale)});
          if (a.dq_accum) st16(make_rsrc(a.dq_accum + head, hbytes * 2), off * 4, __builtin_bit_cast(u32x4, v));
        }
      }
    };
    auto put_rsrc = [&](bool on, int j) {
      if constexpr (MODE == kModePartials)
        return make_rsrc(a.dqacc + ((size_t)bh * a.tc + j) * a.nblk * BM * D, on ? (uint32_t)a.nblk * BM * D * 4 : 0u);
      else
        return acc_rsrc(on);
    };
    auto put_all = [&](int pb, int h, bool add, bool last, int j) {
      const int lf = fresh_lane();
      const auto r = put_rsrc(true, j);
#pragma unroll
      for (int k = 0; k < NACC; ++k) put(r, pb, h, add, last, k, lf);
    };
    auto put_partial = [&](int pb, int h, int j) {  // the partials option (debugging)
      const auto rp = make_rsrc(a.partials + ((size_t)bh * a.tc + j) * N * D, hbytes * 2);
      const int lf = fresh_lane();
#pragma unroll
      for (int k = 0; k < NACC; ++k) {
        const int t = k >> 2, rb = k & 3;
        st16(rp, (uint32_t)((pb * BM + SQ * h + (lf & 31)) * D + 32 * (w * DQT + t) + 8 * rb + 4 * (lf >> 5)) * 4,
             __builtin_bit_cast(u32x4, f32x4{dq[t][4 * rb], dq[t][4 * rb + 1], dq[t][4 * rb + 2], dq[t][4 * rb + 3]}));
      }
    };
    auto note_witness = [&](int pb, int rank, int j) {
      if (tid == 0 && a.witness && rank < a.tc) a.witness[((size_t)bh * a.nblk + pb) * a.tc + rank] = j;
    };
    // wait for block pb's turn (rank), late: its early look had not seen it
    auto take_turn = [&](int pb, int rank) {
      if constexpr (STATS) vm_wait<0>();  // time the wait only, not this wave's own loads
      const unsigned long long t0 = STATS ? clock_now() : 0ull;
      const bool ok = wait_turn(ctr_head + (size_t)pb * kCtrStride, NW * rank, a.spin_limit);
      if constexpr (STATS) stats_wait(wst, t0);
      if (!ok) {
        failed = true;
        __hip_atomic_store(&a.ctrl[kCtrlError], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (a.status) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      return ok;
    };

    // dQ^T of half h (its dS^T in dst[h]) = K^T dS^T: A = K^T of this wave's
    // columns, B = dS^T, both by transposed reads; k-step ks covers keys 16ks +
    // 8(l/32) .. +7.  The addresses and the first reads come from the phase before.
    constexpr int DQR = D == 256 ? 2 : 3;  // (a ring of 3 spills at d = 256)
    uint32_t dq_ka[DQT][2], dq_da[2][2];
    bf16x8 dq_fk[DQR][DQT], dq_fd[DQR];
    auto dq_addr = [&](int h, int lf) {
      const int L16 = lf & 15, nh = (lf >> 4) & 1, g = lf >> 5;
      const int row0 = 8 * g + (L16 >> 2), row1 = row0 + 4;
      const int col = 16 * nh + 4 * (L16 & 3);
      const uint32_t kt = lds_of(sm.kt), dst = lds_of(&sm.dst[0][0]) + (uint32_t)(h * BC * SQ * 2);
#pragma unroll
      for (int t = 0; t < DQT; ++t) {
        dq_ka[t][0] = kt + (uint32_t)bf_at<D>(row0, 32 * (w * DQT + t) + col) * 2;
        dq_ka[t][1] = kt + (uint32_t)bf_at<D>(row1, 32 * (w * DQT + t) + col) * 2;
      }
      dq_da[0][0] = dst + (uint32_t)dst32_at(row0, col) * 2;
      dq_da[0][1] = dst + (uint32_t)dst32_at(row1, col) * 2;
#pragma unroll
      for (int e = 0; e < 2; ++e) dq_da[1][e] = dq_da[0][e] ^ 32u;  // odd k-steps: 4 slots of the swizzle
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        asm volatile("" : "+v"(dq_da[0][e]), "+v"(dq_da[1][e]));
#pragma unroll
        for (int t = 0; t < DQT; ++t) asm volatile("" : "+v"(dq_ka[t][e]));
      }
    };
    auto dq_rd = [&](int ks) {
#pragma unroll
      for (int t = 0; t < DQT; ++t) dq_fk[ks % DQR][t] = lds_tr2(dq_ka[t][0] + 16 * ks * D * 2, dq_ka[t][1] + 16 * ks * D * 2);
      dq_fd[ks % DQR] = lds_tr2(dq_da[ks & 1][0] + 16 * ks * SQ * 2, dq_da[ks & 1][1] + 16 * ks * SQ * 2);
    };
    auto dq_run = [&](auto&& extra) {
#pragma unroll
      for (int t = 0; t < DQT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[t][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KSC; ++ks) {
        if (ks + DQR - 1 < KSC) dq_rd(ks + DQR - 1);
#pragma unroll
        for (int t = 0; t < DQT; ++t) {
          __builtin_amdgcn_sched_barrier(0);
          dq[t] = mfma32(dq_fk[ks % DQR][t], dq_fd[ks % DQR], dq[t]);
          __builtin_amdgcn_sched_barrier(0);
          extra(ks * DQT + t);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };

    // the last sub-step's dQ^T at the end of a tile or chain, and its release
    auto flush = [&]() {
      __syncthreads();  // dS^T of every wave
      dq_addr(1, fresh_lane());
#pragma unroll
      for (int ks = 0; ks < DQR - 1; ++ks) dq_rd(ks);
      dq_run([](int) {});
      if (a.partials) put_partial(p_pb, 1, cur_j);
      if (!ordered || p_turn) put_all(p_pb, 1, p_add, p_last, cur_j);  // (its slice was loaded by the last sub-step)
      if constexpr (ordered) {
        rel_pb = p_pb;
        vm_wait<0>();
        release();
      }
      vm_st = 0;
      p_valid = false;
    };
    auto store_dkdv = [&](int j) {
      // every wave is past its dQ^T (the K tile's last reads): its quarter of
      // the tile becomes a store pad, 32 rows at a time
      __syncthreads();
      const auto rdk = make_rsrc((__bf16*)a.dk + head, hbytes);
      const auto rdv = make_rsrc((__bf16*)a.dv + head, hbytes);
      char* pad = (char*)sm.kt + w * 16384;
      const int lf = fresh_lane();
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          acc_settle(dvacc[kb][nb]);
          acc_settle(dkacc[kb][nb]);
        }
        store_block32<D>(rdv, pad, dvacc[kb], 1.f, j * BC + 32 * (NKB * w + kb), lf);
        store_block32<D>(rdk, pad, dkacc[kb], a.scale, j * BC + 32 * (NKB * w + kb), lf);
      }
    };

    int st = next_valid(0);
    if (st < nsteps) {
      const int pb0 = step_at(st) & 0xfff;
#pragma unroll
      for (int k = 0; k < QP; ++k) load_part(pb0, 0, k);
      load_ld(pb0, bpar);
      if (ordered) poll_copy(pb0);
    }
    unsigned e = st < nsteps ? step_at(st) : 0u;

    for (; st < nsteps;) {
      const int pb = e & 0xfff, j = (e >> 12) & 0x1ff, rank = (e >> 21) & 0x3ff;
      const bool last = (e >> 31) != 0;

      if (j != cur_j) {  // new KV tile
        const int lf = fresh_lane();
        const auto rv = make_rsrc((const __bf16*)a.v + head, hbytes);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            vreg[kb][ks] = as_bf16x8(
                ld16(rv, (uint32_t)((j * BC + 32 * (NKB * w + kb) + (lf & 31)) * D + 16 * ks + 8 * (lf >> 5)) * 2));
        if (cur_j >= 0) {  // (the V loads above are on their way meanwhile)
          flush();
          store_dkdv(cur_j);
        }
        cur_j = j;
        __syncthreads();  // every wave is done with its store pad (and, in a new chain, with the K tile)
        {
          const int t0 = 64 * w + lf;
          const uint32_t at = lds_of(sm.kt) + 1024u * w;
#pragma unroll
          for (int k = 0; k < KP; ++k) {
            const int r = t0 / CPR + k * (NT / CPR), c = (t0 % CPR) ^ tile_swz<D>(r);
            dma16(rk, at + 4096u * k, (uint32_t)((j * BC + r) * D + 8 * c) * 2);
          }
        }
        vm_wait<0>();  // published by the barrier at the top of the sub-step
        vm_st = 0;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              dkacc[kb][nb][r] = 0.f;
              dvacc[kb][nb][r] = 0.f;
            }
      }

      int nst = st + 1, pb_next = -1;  // the next block (looked up in the first sub-step)
      unsigned e_next = 0;
      bool turn = !ordered;  // this block's turn

      auto sub_step = [&](auto h_c) {
        constexpr int h = decltype(h_c)::value;
        // this wave's copies of Q / dO (and L, D, the counter) have landed;
        // after the barrier every wave's have, dS^T of the sub-step before is
        // complete, and the other Q / dO buffer is free
        vm_wait_few(vm_st);
        __syncthreads();
        const int lf0 = fresh_lane();
        const int g = lf0 >> 5, lc = lf0 & 31;
        unsigned e_v = 0;
        if constexpr (h == 0) e_v = sm.steps[st + 1 < nsteps ? st + 1 : st];

        // ---- this block's turn: looked up a sub-step ahead of its first half's
        //      slice loads, once more a sub-step later, and waited for at the end
        //      of the second sub-step
        bool look2 = false;
        if (ordered && !failed && !turn) {
          const int v0 = __builtin_amdgcn_readfirstlane(sm.poll[w][0]);
          if (v0 >= NW * rank) {
            turn = true;
            look2 = h == 1;
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
          }
        }
        // dQ^T of the sub-step before is added in this one (phase 3b), and the
        // slice for this one's is loaded behind it
        const bool do_put = h == 0 ? p_valid && p_turn : turn;
        const bool do_load = ordered && turn, add = rank > 0;
        const int d_pb = h == 0 ? p_pb : pb;
        const bool d_last = do_put && (h == 0 ? p_last : last), d_add = h == 0 ? p_add : add;

        // ---- phase 1: S = Q K^T, dP = dO V^T (A = Q / dO rows, B = K rows, all
        //      from LDS; V rows from registers)
        f32x16 s[NKB], dp[NKB];
        {
          constexpr int RING = 3;
          const uint32_t qa = lds_of(&sm.qs[h][0]) + (uint32_t)bf_at<D>(lc, 8 * g) * 2;
          const uint32_t ka = lds_of(sm.kt) + (uint32_t)bf_at<D>(32 * NKB * w + lc, 8 * g) * 2;
          bf16x8 fq[RING], fo[RING], fk[RING][NKB];
          auto rd = [&](int ks) {  // the swizzle leaves the k-step as an XOR of the chunk bits
            fq[ks % RING] = lds16(qa ^ (uint32_t)(ks << 5));
            fo[ks % RING] = lds16((qa ^ (uint32_t)(ks << 5)) + (uint32_t)sizeof(sm.qs));
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) fk[ks % RING][kb] = lds16((ka ^ (uint32_t)(ks << 5)) + 32 * kb * D * 2);
          };
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kb][r] = dp[kb][r] = 0.f;
#pragma unroll
          for (int ks = 0; ks < RING - 1; ++ks) rd(ks);
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            if (ks + RING - 1 < KS) rd(ks + RING - 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
              s[kb] = mfma32(fq[ks % RING], fk[ks % RING][kb], s[kb]);
              dp[kb] = mfma32(fo[ks % RING], vreg[kb][ks], dp[kb]);
            }
            __builtin_amdgcn_sched_barrier(0);
            // the copies of the next sub-step, spread: a wave's 1 KB copies issue
            // back to back only as fast as the CU's four waves together move them
            constexpr int GAP = (KS - 2) / QP;
            if (h == 0) {
              if (ks == 0 && ordered && !turn) poll_copy(pb);
              if (ks % GAP == 1 && ks / GAP < QP) load_part(pb, 1, ks / GAP);
            } else if (pb_next >= 0) {
              if (ks == 0 && ordered) poll_copy(pb_next);
              if (ks == 0) load_ld(pb_next, bpar ^ 1);
              if (ks % GAP == 1 && ks / GAP < QP) load_part(pb_next, 0, ks / GAP);
            }
            if (h == 1 && ks == KS - 3 && look2) load_old(pb, 0, add);
            // phase 2's addresses and first reads
            if (ks == KS - 4) dq_addr(h ^ 1, lf0);
            if (ks >= KS - (DQR - 1)) dq_rd(ks - (KS - (DQR - 1)));
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if constexpr (h == 0) {
          nst = st + 1;
          if (nst < nsteps) {
            e_next = __builtin_amdgcn_readfirstlane(e_v);
            if (e_next == kNoStep) {
              nst = next_valid(nst + 1);
              if (nst < nsteps) e_next = step_at(nst);
            }
          }
          pb_next = nst < nsteps ? (int)(e_next & 0xfff) : -1;
        }
        // deferred release of the block whose second half was stored a sub-step ago
        if (ordered && h == 1 && rel_pb >= 0) {
          vm_wait_few(pb_next >= 0 ? 2 * QP : 0);  // (the copies issued since)
          release();
        }

        // element (kb, r) is query 8(r/4) + 4g + r%4 of the sub-step and key
        // 32 (NKB w + kb) + lc of the tile.  Keys past N need no mask: their
        // K, V rows read as zero, P is at most 1 there and their dK, dV rows are
        // not stored.
        if (CAUSAL && j * BC + 32 * NKB * (w + 1) - 1 > pb * BM + SQ * h) {
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb) {
            const int thr = j * BC + 32 * (NKB * w + kb) + lc - pb * BM - SQ * h - 4 * g;  // masked iff query < thr
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (8 * (r >> 2) + (r & 3) < thr) s[kb][r] = -INFINITY;
          }
        }

        // Phase 3's operand reads (B = dO, Q by transposed reads, rows 16 half +
        // 4g + 0..3 and +8 of d block i / 2, half i % 2); each run's first ones are
        // issued in the phase before
        const int L16 = lf0 & 15, nh = (lf0 >> 4) & 1;
        uint32_t ta0 = lds_of(&sm.qs[h][0]) + (uint32_t)bf_at<D>(4 * g + (L16 >> 2), 16 * nh + 4 * (L16 & 3)) * 2;
        uint32_t ta1 = lds_of(&sm.qs[h][0]) + (uint32_t)bf_at<D>(4 * g + (L16 >> 2) + 8, 16 * nh + 4 * (L16 & 3)) * 2;
        asm volatile("" : "+v"(ta0), "+v"(ta1));
        constexpr int TR = 4;
        bf16x8 tf[TR];
        auto t_rd = [&](auto is_dk, int i) {
          constexpr uint32_t base = decltype(is_dk)::value ? 0u : (uint32_t)sizeof(sm.qs);
          const uint32_t x = (uint32_t)((i >> 1) << 6), at = base + (uint32_t)(16 * (i & 1) * D * 2);
          tf[i % TR] = lds_tr2((ta0 ^ x) + at, (ta1 ^ x) + at);
        };
        using DV = std::false_type;
        using DK = std::true_type;
        auto dvdk_run = [&](auto is_dk, u32x4(&op)[NKB][2], f32x16(&acc)[NKB][NB], auto&& extra) {
#pragma unroll
          for (int i = 0; i < 2 * NB; ++i) {
            if (i + TR - 1 < 2 * NB) t_rd(is_dk, i + TR - 1);
            else if (!decltype(is_dk)::value) t_rd(DK{}, i + TR - 1 - 2 * NB);  // dK's first reads
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
              __builtin_amdgcn_sched_barrier(0);
              mfma32_acc(__builtin_bit_cast(bf16x8, op[kb][i & 1]), tf[i % TR], acc[kb][i >> 1]);
              __builtin_amdgcn_sched_barrier(0);
              extra(i * NKB + kb);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        static_assert((2 * NB) % TR == 0, "dK's first reads continue dV's ring");

        // ---- phase 2: dQ^T of the sub-step before, beside P = exp(S - L)
        u32x4 pbf[NKB][2], dsbf[NKB][2];
        const uint32_t ls_at = lds_of(&sm.ls[0][0]) + (uint32_t)((bpar * BM + SQ * h + 4 * g) * 4);
        const uint32_t ds_at = ls_at + (uint32_t)sizeof(sm.ls);
        f32x4 ld[2], dd[2];
        ld[0] = lds16f(ls_at);
        dq_run([&](int i) {  // slot i: element i of every key block
          if ((i & 3) == 0 && i < 12) ld[((i >> 2) + 1) & 1] = lds16f(ls_at + 32 * ((i >> 2) + 1));
          if (i == 12) dd[0] = lds16f(ds_at);
          if (i >= 13) t_rd(DV{}, i - 13);
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb) {
            s[kb][i] = exp2_unit(__builtin_fmaf(s[kb][i], c2, -ld[(i >> 2) & 1][i & 3]));
            // packed by twos a slot late; the empty asm keeps the work in this slot
            const int q = i - 2;
            if (i >= 2 && (i & 1) == 0) {
              unsigned x = pack_bf16(s[kb][q], s[kb][q + 1]);
              asm volatile("" : "+v"(x));
              pbf[kb][q >> 3][(q & 7) >> 1] = x;
            }
            if (i == 15) {
              unsigned x = pack_bf16(s[kb][14], s[kb][15]);
              asm volatile("" : "+v"(x));
              pbf[kb][1][3] = x;
            }
          }
        });
        if (a.partials && (h == 1 || p_valid)) put_partial(d_pb, h ^ 1, j);

        // ---- phase 3: dV += P^T dO beside dS = P (dP - D), the
        //      ordered add and the stores of dQ^T, then dK += dS^T Q beside the dS^T stores
        //      and the loads of the next slice.  A = P^T, dS^T from registers.
        asm volatile("s_nop 1" ::: "memory");  // two wait states between the packs and their first MFMA
        const int lfp = fresh_lane();
        const auto r_put = put_rsrc(do_put, j);
        const auto r_ld = acc_rsrc(do_load && add);
        constexpr int EV = 16 / NACC;  // slots per chunk
        dvdk_run(DV{}, pbf, dvacc, [&](int i) {  // slot i: element i of every key block
          if ((i & 3) == 0 && i < 12) dd[((i >> 2) + 1) & 1] = lds16f(ds_at + 32 * ((i >> 2) + 1));
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb) {
            dp[kb][i] = s[kb][i] * (dp[kb][i] - dd[(i >> 2) & 1][i & 3]);
            if (i & 1) {
              unsigned x = pack_bf16(dp[kb][i - 1], dp[kb][i]);
              asm volatile("" : "+v"(x));
              dsbf[kb][i >> 3][(i & 7) >> 1] = x;
            }
          }
          if (i % EV == EV - 1) put(r_put, d_pb, h ^ 1, d_add, d_last, i / EV, lfp);
        });
        asm volatile("s_nop 1" ::: "memory");
        const uint32_t dst_w = lds_of(&sm.dst[h][0]);
        dvdk_run(DK{}, dsbf, dkacc, [&](int i) {
          if (i < 4 * NKB) {  // dS^T of key block i / 4, queries 8 (i % 4) + 4g .. +3
            const int kb = i >> 2, rb = i & 3;
            const u32x4 v = dsbf[kb][rb >> 1];
            lds_st8(dst_w + (uint32_t)dst32_at(32 * (NKB * w + kb) + lc, 8 * rb + 4 * g) * 2,
                    (rb & 1) ? u32x2{v[2], v[3]} : u32x2{v[0], v[1]});
          }
          if (ordered && i % EV == EV - 1) load_old1(r_ld, pb, h, i / EV, lfp);
        });
        vm_st = ordered ? 2 * NACC : NACC;  // this sub-step's stores, then loads
        if constexpr (h == 0) {
          if (ordered && p_valid) {
            rel_pb = p_pb;
            if (!deferred) {
              vm_wait_few(NACC);  // the stores (the loads came after)
              release();
            }
          }
        } else {
          if constexpr (ordered) {
            if (!turn && !failed) {
              turn = take_turn(pb, rank);
              if (turn) {
                load_old(pb, 0, add);
                put_all(pb, 0, add, last, j);
                load_old(pb, 1, add);
              }
            }
            if (turn) note_witness(pb, rank, j);
          }
          p_valid = true;
          p_pb = pb;
          p_last = last;
          p_add = add;
          p_turn = turn;
        }
      };
      sub_step(std::integral_constant<int, 0>{});
      sub_step(std::integral_constant<int, 1>{});
      bpar ^= 1;
      st = nst;
      e = e_next;
    }
    if (cur_j >= 0) {
      flush();
      store_dkdv(cur_j);
    }
    __syncthreads();  // sm.item is rewritten by the next ticket
  }
  if constexpr (STATS) stats_wave_end(wst, a.wait_stats, tid & 63);
}

template <int D, bool CAUSAL>
hipError_t launch_mask(const BwdArgs& a, int grid, hipStream_t stream) {
  if constexpr (D == 128) {
    if (a.G.sched == S_PARTIALS) return launch_main_grid(bwd_mainw_kernel<D, CAUSAL, kModePartials>, a, grid, NT, stream);
  }
  if (a.wait_stats) return launch_main_grid(bwd_mainw_kernel<D, CAUSAL, kModeOrdered, true>, a, grid, NT, stream);
  return launch_main_grid(bwd_mainw_kernel<D, CAUSAL, kModeOrdered>, a, grid, NT, stream);
}

template <typename K>
bool resident(K k, int* lo) {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, (const void*)k, NT, 0) != hipSuccess) return false;
  *lo = blocks < *lo ? blocks : *lo;
  return true;
}
template <int D, bool CAUSAL>
bool resident_all(int* lo) {
  bool ok = resident(bwd_mainw_kernel<D, CAUSAL, kModeOrdered>, lo) && resident(bwd_mainw_kernel<D, CAUSAL, kModeOrdered, true>, lo);
  if constexpr (D == 128) ok = ok && resident(bwd_mainw_kernel<D, CAUSAL, kModePartials>, lo);
  return ok;
}

}  // namespace

hipError_t launch_mainw(const BwdArgs& a, int d, int grid_main, hipStream_t stream) {
  if (d == 128) return a.G.causal ? launch_mask<128, true>(a, grid_main, stream) : launch_mask<128, false>(a, grid_main, stream);
  return a.G.causal ? launch_mask<256, true>(a, grid_main, stream) : launch_mask<256, false>(a, grid_main, stream);
}

int bwd_mainw_occupancy(int d) {
  int lo = 1 << 30;
  const bool ok = d == 128 ? resident_all<128, false>(&lo) && resident_all<128, true>(&lo)
                           : resident_all<256, false>(&lo) && resident_all<256, true>(&lo);
  return ok ? lo : 0;
}

}  // namespace dash
