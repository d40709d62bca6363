// Bank-conflict check of the kernels' LDS layouts (host build of
// paper_2601_21824_amd/csrc/lds_layout.h), and of the address arithmetic by
// which the wide-tile backward and the forward reach them (a lane's base address
// with the step entered by XOR or as an offset).
//
// Bank model of gfx950 (measured with the hardware bank-conflict counter on a
// one-wave probe): 64 banks of 4 bytes; 16-byte-per-lane accesses are served
// in lane groups of 16, 8-byte-per-lane accesses in groups of 32; a group
// costs (largest number of distinct dwords that share one bank) - 1 extra
// cycles.  The lane -> (row, column) mappings below are those of the kernels'
// LDS accesses.  Prints one line per pattern; exits 1 if any kernel pattern
// has a conflict or the model does not reproduce the probe's counts.
#include <cstdio>
#include <map>
#include <set>
#include <vector>
#include "lds_layout.h"

using namespace dash;

static int conflicts(const std::vector<long>& byte_addr, int nbytes) {
  const int per = nbytes == 16 ? 16 : nbytes == 8 ? 32 : 64;
  int total = 0;
  for (int g0 = 0; g0 < 64; g0 += per) {
    std::map<long, std::set<long>> bank;
    for (int l = g0; l < g0 + per; ++l)
      for (int b = 0; b < nbytes / 4; ++b) {
        const long dw = byte_addr[l] / 4 + b;
        bank[dw % 64].insert(dw);
      }
    size_t worst = 0;
    for (auto& kv : bank) worst = kv.second.size() > worst ? kv.second.size() : worst;
    total += (int)worst - 1;
  }
  return total;
}

static int failures = 0;
static void expect(const char* what, int got, int want) {
  std::printf("%-58s %4d (expected %d)\n", what, got, want);
  if (got != want) ++failures;
}

template <int D>
static void tile_patterns(const char* name) {
  const int KS = D / 16, NB = D / 32;
  int rows = 0, tr = 0, dma = 0;
  for (int h = 0; h < 2; ++h)
    for (int ks = 0; ks < KS; ++ks) {  // MFMA row operands
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) a[l] = 2L * bf_at<D>(32 * h + (l & 31), 16 * ks + 8 * (l >> 5));
      rows += conflicts(a, 16);
    }
  for (int h = 0; h < 2; ++h)
    for (int k = 0; k < 2 * NB; ++k)  // transposed operands of dV, dK
      for (int dr = 0; dr < 16; dr += 8) {
        std::vector<long> a(64);
        for (int l = 0; l < 64; ++l) {
          const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5, nb = k >> 1, half = k & 1;
          a[l] = 2L * bf_at<D>(32 * h + 16 * half + 4 * g + (L16 >> 2) + dr, 32 * nb + 16 * nh + 4 * (L16 & 3));
        }
        tr += conflicts(a, 8);
      }
  {  // the direct loads land row-major in LDS: each lane's 16 bytes at 16 * lane
    std::vector<long> a(64);
    for (int l = 0; l < 64; ++l) a[l] = 16L * l;
    dma += conflicts(a, 16);
  }
  char buf[96];
  std::snprintf(buf, sizeof buf, "%s row operands (per wave and step)", name);
  expect(buf, rows, 0);
  std::snprintf(buf, sizeof buf, "%s transposed operands (per wave and step)", name);
  expect(buf, tr, 0);
}

static void dst_patterns() {
  int wr = 0, rd = 0;
  for (int w = 0; w < 4; ++w)
    for (int p = 0; p < 8; ++p) {  // dS^T stores, piece p
      std::vector<long> a(64);
      const int qb = p >> 2, half = (p >> 1) & 1, part = p & 1;
      for (int l = 0; l < 64; ++l) a[l] = 2L * dst_at(32 * w + (l & 31), 32 * qb + 16 * half + 8 * part + 4 * (l >> 5));
      wr += conflicts(a, 8);
    }
  for (int ks = 0; ks < 8; ++ks)  // transposed reads for dQ^T
    for (int qc = 0; qc < 64; qc += 32)
      for (int dr = 0; dr < 8; dr += 4) {
        std::vector<long> a(64);
        for (int l = 0; l < 64; ++l) {
          const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5;
          a[l] = 2L * dst_at(16 * ks + 8 * g + (L16 >> 2) + dr, qc + 16 * nh + 4 * (L16 & 3));
        }
        rd += conflicts(a, 8);
      }
  expect("d<=128 dS^T stores (all waves, per step)", wr, 0);
  expect("d<=128 dS^T transposed reads (per wave and step)", rd, 0);
}

// d = 64 kernel with 256-row KV tiles (attn_bwd64w.hip): the Q / dO patterns
// are tile_patterns<64>'s; new are the dS^T stores of 8 waves' worth of rows
// (64 keys per wave), the K tile's transposed reads (A = K^T of dQ^T) and the
// dS^T transposed reads over 256 keys
static void w64_patterns() {
  int wr = 0, rdk = 0, rdd = 0;
  for (int w = 0; w < 4; ++w)
    for (int kb = 0; kb < 2; ++kb)
      for (int p = 0; p < 8; ++p) {
        std::vector<long> a(64);
        const int qb = p >> 2, half = (p >> 1) & 1, part = p & 1;
        for (int l = 0; l < 64; ++l)
          a[l] = 2L * dst_at(64 * w + 32 * kb + (l & 31), 32 * qb + 16 * half + 8 * part + 4 * (l >> 5));
        wr += conflicts(a, 8);
      }
  for (int ks = 0; ks < 16; ++ks)
    for (int blk = 0; blk < 2; ++blk)  // d block of the K^T operand / query half of dS^T
      for (int dr = 0; dr < 8; dr += 4) {
        std::vector<long> k(64), d(64);
        for (int l = 0; l < 64; ++l) {
          const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5;
          const int row = 16 * ks + 8 * g + (L16 >> 2) + dr, col = 32 * blk + 16 * nh + 4 * (L16 & 3);
          k[l] = 2L * bf_at<64>(row, col);
          d[l] = 2L * dst_at(row, col);
        }
        rdk += conflicts(k, 8);
        rdd += conflicts(d, 8);
      }
  expect("d=64 256-row dS^T stores (all waves, per step)", wr, 0);
  expect("d=64 256-row K^T transposed reads (per step, both d blocks)", rdk, 0);
  expect("d=64 256-row dS^T transposed reads (per step, both halves)", rdd, 0);
}

static void d256_patterns() {
  int rows = 0, tr = 0, wr = 0, rd = 0;
  for (int qb = 0; qb < 4; ++qb)
    for (int ks = 0; ks < 8; ++ks) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) a[l] = 2L * q256_at(16 * qb + (l & 15), 32 * ks + 8 * (l >> 4));
      rows += conflicts(a, 16);
    }
  for (int k = 0; k < 32; ++k)
    for (int dr = 0; dr < 32; dr += 16) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) {
        const int lr = l & 15, gq = l >> 4, db = k >> 1, kq = k & 1;
        a[l] = 2L * q256_at(32 * kq + 4 * gq + (lr >> 2) + dr, 16 * db + 4 * (lr & 3));
      }
      tr += conflicts(a, 8);
    }
  for (int w = 0; w < 4; ++w)
    for (int qb = 0; qb < 4; ++qb) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) a[l] = 2L * ds256_at(16 * w + (l & 15), 16 * qb + 4 * (l >> 4));
      wr += conflicts(a, 8);
    }
  for (int kk = 0; kk < 2; ++kk)
    for (int qb = 0; qb < 4; ++qb)
      for (int dr = 0; dr < 8; dr += 4) {
        std::vector<long> a(64);
        for (int l = 0; l < 64; ++l)
          a[l] = 2L * ds256_at(32 * kk + 8 * (l >> 4) + ((l & 15) >> 2) + dr, 16 * qb + 4 * (l & 3));
        rd += conflicts(a, 8);
      }
  expect("d=256 Q/dO row operands (per wave and step)", rows, 0);
  expect("d=256 Q/dO transposed operands (per wave and step)", tr, 0);
  expect("d=256 dS^T stores (all waves, per step)", wr, 0);
  expect("d=256 dS^T transposed reads (per wave and step)", rd, 0);
}

static void same(const char* what, long got, long want) {
  if (got == want) return;
  std::printf("%s: address %ld, expected %ld\n", what, got, want);
  ++failures;
}

// Direct global -> LDS copies of a [rows][D] tile: thread t of 256 writes 16 bytes
// at 16 t (+ 4096 per part) and reads chunk (t % (D/8)) ^ swz(row) of its row.
template <int D>
static void copy_lands(int rows) {
  const int CPR = D / 8;
  for (int p = 0; p < rows * CPR / 256; ++p)
    for (int t = 0; t < 256; ++t) {
      const int row = t / CPR + p * (256 / CPR), c = (t % CPR) ^ tile_swz<D>(row);
      same("direct copy", 16L * t + 4096L * p, 2L * bf_at<D>(row, 8 * c));
    }
}

// bwd_mainw_kernel (attn_bwdw.hip): KV tile of BC = 32768 / D rows, sub-steps of
// 32 queries
template <int D>
static void wide_patterns(const char* name) {
  const int BC = 32768 / D, NKB = BC / 128, NB = D / 32, KS = D / 16;
  int rows = 0, krows = 0, tr = 0, wr = 0, rdk = 0, rdd = 0;
  for (int ks = 0; ks < KS; ++ks) {
    std::vector<long> a(64);
    for (int l = 0; l < 64; ++l) {  // phase 1: Q / dO rows
      a[l] = (2L * bf_at<D>(l & 31, 8 * (l >> 5))) ^ (ks << 5);
      same("wide Q row", a[l], 2L * bf_at<D>(l & 31, 16 * ks + 8 * (l >> 5)));
    }
    rows += conflicts(a, 16);
    for (int w = 0; w < 4; ++w)  // K rows of the wave's key blocks
      for (int kb = 0; kb < NKB; ++kb) {
        for (int l = 0; l < 64; ++l) {
          a[l] = ((2L * bf_at<D>(32 * NKB * w + (l & 31), 8 * (l >> 5))) ^ (ks << 5)) + 32L * kb * D * 2;
          same("wide K row", a[l], 2L * bf_at<D>(32 * (NKB * w + kb) + (l & 31), 16 * ks + 8 * (l >> 5)));
        }
        krows += conflicts(a, 16);
      }
  }
  for (int i = 0; i < 2 * NB; ++i)  // phase 3: transposed Q / dO
    for (int e = 0; e < 2; ++e) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) {
        const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5, row = 4 * g + (L16 >> 2) + 8 * e, col = 16 * nh + 4 * (L16 & 3);
        a[l] = ((2L * bf_at<D>(row, col)) ^ ((i >> 1) << 6)) + 16L * (i & 1) * D * 2;
        same("wide Q column", a[l], 2L * bf_at<D>(row + 16 * (i & 1), col + 32 * (i >> 1)));
      }
      tr += conflicts(a, 8);
    }
  for (int kb = 0; kb < BC / 32; ++kb)  // phase 3: dS^T stores of 32 keys
    for (int rb = 0; rb < 4; ++rb) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) a[l] = 2L * dst32_at(32 * kb + (l & 31), 8 * rb + 4 * (l >> 5));
      wr += conflicts(a, 8);
    }
  for (int ks = 0; ks < BC / 16; ++ks)  // phase 2: dQ^T
    for (int e = 0; e < 2; ++e) {
      std::vector<long> a(64);
      for (int db = 0; db < NB; ++db) {
        for (int l = 0; l < 64; ++l) {
          const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5, row = 8 * g + (L16 >> 2) + 4 * e, col = 16 * nh + 4 * (L16 & 3);
          a[l] = 2L * bf_at<D>(row, 32 * db + col) + 16L * ks * D * 2;
          same("wide K column", a[l], 2L * bf_at<D>(row + 16 * ks, 32 * db + col));
        }
        rdk += conflicts(a, 8);
      }
      for (int l = 0; l < 64; ++l) {
        const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5, row = 8 * g + (L16 >> 2) + 4 * e, col = 16 * nh + 4 * (L16 & 3);
        a[l] = ((2L * dst32_at(row, col)) ^ (32 * (ks & 1))) + 16L * ks * 32 * 2;
        same("wide dS^T", a[l], 2L * dst32_at(row + 16 * ks, col));
      }
      rdd += conflicts(a, 8);
    }
  std::set<long> cells;  // dst32_at keeps 4 queries together and every slot apart
  for (int r = 0; r < BC; ++r)
    for (int q = 0; q < 32; q += 4) cells.insert(dst32_at(r, q));
  same("dst32_at cells", (long)cells.size(), 8L * BC);
  same("dst32_at last cell", *cells.rbegin(), 32L * BC - 4);
  copy_lands<D>(32);
  copy_lands<D>(BC);
  char buf[96];
  std::snprintf(buf, sizeof buf, "%s wide Q/dO row operands (per sub-step)", name);
  expect(buf, rows, 0);
  std::snprintf(buf, sizeof buf, "%s wide K row operands (all waves)", name);
  expect(buf, krows, 0);
  std::snprintf(buf, sizeof buf, "%s wide Q/dO transposed operands", name);
  expect(buf, tr, 0);
  std::snprintf(buf, sizeof buf, "%s wide dS^T stores (all waves)", name);
  expect(buf, wr, 0);
  std::snprintf(buf, sizeof buf, "%s wide K^T transposed reads (all d blocks)", name);
  expect(buf, rdk, 0);
  std::snprintf(buf, sizeof buf, "%s wide dS^T transposed reads", name);
  expect(buf, rdd, 0);
}

// attn_fwd_kernel: K and V tiles of KT rows, in units of 32 keys
template <int D>
static void fwd_patterns(const char* name) {
  const int KT = D == 256 ? 32 : 64;
  int k = 0, v = 0;
  for (int uu = 0; uu < KT / 32; ++uu) {
    for (int ks = 0; ks < D / 16; ++ks) {
      std::vector<long> a(64);
      for (int l = 0; l < 64; ++l) {
        const int g = l >> 5, lc = l & 31;
        a[l] = ((lc * D * 2 + ((g ^ tile_swz<D>(lc)) << 4)) ^ (ks << 5)) + 32L * uu * D * 2;
        same("forward K row", a[l], 2L * bf_at<D>(32 * uu + lc, 16 * ks + 8 * g));
      }
      k += conflicts(a, 16);
    }
    for (int p = 0; p < D / 16; ++p)
      for (int e = 0; e < 2; ++e) {
        std::vector<long> a(64);
        const int half = p / (D / 32), db = p % (D / 32);
        for (int l = 0; l < 64; ++l) {
          const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5, row = 4 * g + (L16 >> 2) + 8 * e;
          const long lane = row * D * 2 + (((2 * nh + ((L16 & 3) >> 1)) ^ tile_swz<D>(row)) << 4) + ((L16 & 1) << 3);
          a[l] = (lane ^ (db << 6)) + (32L * uu + 16 * half) * D * 2;
          same("forward V column", a[l], 2L * bf_at<D>(32 * uu + 16 * half + row, 32 * db + 16 * nh + 4 * (L16 & 3)));
        }
        v += conflicts(a, 8);
      }
  }
  copy_lands<D>(KT);
  char buf[96];
  std::snprintf(buf, sizeof buf, "%s forward K row operands (per tile)", name);
  expect(buf, k, 0);
  std::snprintf(buf, sizeof buf, "%s forward V^T transposed operands (per tile)", name);
  expect(buf, v, 0);
}

static void probe_patterns() {
  // the probe's measured conflict cycles per instruction
  auto rows_at = [](int period) {
    std::vector<long> a(64);
    for (int l = 0; l < 64; ++l) a[l] = 256L * l + 16 * (period ? l % period : 0);
    return a;
  };
  std::vector<long> lin(64);
  for (int l = 0; l < 64; ++l) lin[l] = 16L * l;
  expect("probe: 16-byte reads, linear", conflicts(lin, 16), 0);
  expect("probe: 16-byte reads, 64 rows at one chunk", conflicts(rows_at(0), 16), 60);
  expect("probe: 16-byte reads, chunk = row % 4", conflicts(rows_at(4), 16), 12);
  expect("probe: 16-byte reads, chunk = row % 8", conflicts(rows_at(8), 16), 4);
  expect("probe: 16-byte reads, chunk = row % 16", conflicts(rows_at(16), 16), 0);
  std::vector<long> tr(64);
  for (int l = 0; l < 64; ++l) {  // transposed-read lane pattern without a swizzle
    const int L16 = l & 15, nh = (l >> 4) & 1, g = l >> 5;
    tr[l] = 256L * (4 * g + (L16 >> 2)) + 2 * (16 * nh + 4 * (L16 & 3));
  }
  expect("probe: 8-byte transposed reads, rows unswizzled", conflicts(tr, 8), 6);
}

int main() {
  probe_patterns();
  tile_patterns<128>("d=128 Q/dO");
  tile_patterns<64>("d=64 Q/dO");
  dst_patterns();
  w64_patterns();
  d256_patterns();
  wide_patterns<128>("d=128");
  wide_patterns<256>("d=256");
  fwd_patterns<64>("d=64");
  fwd_patterns<128>("d=128");
  fwd_patterns<256>("d=256");
  std::printf(failures ? "FAIL\n" : "OK\n");
  return failures ? 1 : 0;
}
