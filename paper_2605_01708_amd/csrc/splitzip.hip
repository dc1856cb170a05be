// SplitZip codec for MI355X (gfx950): the C ABI of include/splitzip.h and the host side of its
// kernels.  One translation unit; the kernels live in the headers included below:
//   common.hpp      stream layout, wave scan, agent-scope accesses
//   compress.hpp    dense transform (paper section 3.2 eq. (1), encode table, nibble pack, planes)
//                   fused with escape detection, counting and position-ordered compaction
//                   (appendix "Quad64 Vectorized Encoding" fuses only the counting); two launches
//                   for a tensor or up to 160 of them, one for few chunks
//   decompress.hpp  nibble unpack, decode table, eq. (2), scatter correction in LDS; one
//                   launch per tensor or per batch
//   aux_kernels.hpp calibration histogram (section 3.3), workspace initialisation, traffic probe
//   variants.hpp    the formats of the ablations (top-8 / 3-bit codes, top-15 + sentinel, chunk 256,
//                   absolute positions, E4M3) through one plain set of kernels
//
// Work decomposition (wavefront = 64 lanes): a chunk of 1024 elements (the escape-position
// granule) is owned by one wave; every global access of a wave is one fully coalesced run of 16,
// 8 or 4 bytes per lane; all plane traffic uses non-temporal loads and stores, nothing is re-used.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>
#include <unistd.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "splitzip.h"

namespace {

#include "common.hpp"
#include "compress.hpp"
#include "decompress.hpp"
#include "aux_kernels.hpp"
#include "variants.hpp"

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

uint64_t chunks_of(uint64_t n) { return (n + kChunk - 1) / kChunk; }
bool dtype_ok(int dtype) { return dtype == SPLITZIP_BF16 || dtype == SPLITZIP_FP8_E5M2; }
unsigned exp_values(int dtype) { return dtype == SPLITZIP_BF16 ? 256u : 32u; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// A launch whose arguments are copied once, by the runtime.  Through hipLaunchKernelGGL they are copied to the stack
// before that.  Both copies of a batch call's 3.2 KB take 2 us longer where the source lies badly, and that changed with
// unrelated edits (64 streams of two chunks: 9.4 to 11.7 us a call); without the first, and with arguments that begin
// with a cache line, it is 9.3.  Errors are left to hipGetLastError.
template <typename A>
void launch(void (*kernel)(A), dim3 grid, dim3 block, unsigned lds, hipStream_t st, const A& args) {
  void* params[] = {const_cast<A*>(&args)};
  (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, params, lds, st);
}

// the arguments of a launch of few tensors, which begin those of one of many
template <template <uint32_t> class A>
const A<kBatchFew>& few(const A<kBatchMax>& args) {
  static_assert(offsetof(A<kBatchFew>, item) == offsetof(A<kBatchMax>, item) && alignof(A<kBatchFew>) == alignof(A<kBatchMax>), "one begins the other");
  return reinterpret_cast<const A<kBatchFew>&>(args);
}

// What the tests of the rarely taken paths turn: a staging area and a status area smaller than the workspace has
// (tiles whose records do not fit their slots; batches that take several launches), and the number of groups a
// workgroup of the finishing pass takes, which small launches would leave at one, and the bytes of tile counts the
// finishing pass may read directly before it is given sums instead.  Set through
// splitzip_internal_test_hooks (exported, not declared in splitzip.h); zero in normal use.
// And what the launch rules choose by the sizes of a call, so that every choice can be tested at any size (set through
// splitzip_internal_test_launch): chunks per wave of the compress tiles and of the decoders, and the tiles' order.
struct TestHooks {
  std::atomic<uint64_t> stage_bytes{0};
  std::atomic<uint64_t> status_bytes{0};
  std::atomic<uint32_t> finish_groups{0};
  std::atomic<uint64_t> direct_bytes{0};
  std::atomic<uint32_t> cpt{0};   // 1, 2, 4 or 8
  std::atomic<uint32_t> cpw{0};   // 1, 2, 4 or 8, most_cpw at most
  std::atomic<uint32_t> xcd{0};   // 1: batch launches keep the tiles' own order, 2: they take xcd_order
  std::atomic<uint32_t> short_looks{0};   // how often a workgroup of compress_short_kernel looks for the counts of the others; kNoShort: no such launches
  std::atomic<bool> short_anywhere{false};   // and on streams with a mask as on others
  bool any() const { return stage_bytes || status_bytes || finish_groups || direct_bytes || cpt || xcd; }   // the two-launch path is meant
};
constexpr uint32_t kNoShort = 0xffffffffu;
TestHooks g_hooks;

// Whether more than one element in 16 may have escaped, by the bytes that the caller says it holds beyond the fixed part
// of its streams (three per record): the device alone knows the number.
bool many_escapes(uint64_t bytes_beyond, uint64_t n_elems) { return bytes_beyond * 16 > n_elems * 3; }

// The most chunks per wave that a decompress launch of one stream or of several takes, and that there are kernels for.
constexpr uint32_t most_cpw(int dtype, bool several) { return (dtype == SPLITZIP_BF16 ? 2u : 4u) << (several ? 1 : 0); }

// Chunks per wave of a decompress launch over n_chunks chunks in all; device us per call with one / two / four chunks per
// wave, all of whose planes a wave asks for at once:
//   BF16  2.6 / 3.0 / 3.8 (512 chunks), 4.0 / 4.3 / 4.5 (4096), 5.4 / 4.9 / 5.5 (6144), 6.7 / 6.1 / 5.9 (8192), 8.5 / 7.1 / 7.3
//         (10 240), 9.4 / 8.7 / 7.9 (12 288), 10.8 / 10.4 / 11.2 (14 336), 11.8 / 11.8 / 11.6 (16 384), 13.0 / 13.3 / 14.3 (18 432),
//         16.3 / 16.6 / 16.1 (24 576), 21.2 / 21.4 / 21.2 (32 768), 38.2 / 39.6 / 40.9 (65 536), 75.2 / 74.0 / 76.0 (131 072).
//         Two up to what is resident at once (eight workgroups of eight chunks per CU) and again for long
//         launches, in those of several streams from 32 768 on; in the longest, with fewer workgroups per CU
//         (plan_decompress), 1228 / 1187 / 1246 (2 Mi).  Four, where its workgroups come out as whole rounds of the chip, is up to
//         9 % faster than two and loses as much between (14 336): single calls do not use it.
//   E5M2  2.5 / 2.9 / 3.6 (512), 5.4 / 4.6 / 5.1 (8192), 6.8 / 6.8 / 6.1 (12 288), 8.3 / 8.0 / 7.4 (16 384), 10.9 / 10.8 / 10.5 (24 576),
//         14.0 / 13.0 / 13.3 (32 768), 24.8 / 22.5 / 23.3 (65 536), 45.4 / 40.4 / 41.5 (128 000), 180 / 155.5 / 159.6 (524 288),
//         722 / 636 / 650 and, with fewer workgroups per CU, 619 with four (2 Mi).
// Streams with many escapes keep a wave busy with its chunks' records, one chunk after the other, so the larger pieces
// pay from somewhat longer streams on.  Random words in 15 / 40 % of the places (14 / 37 % escapes for BF16, 8 / 20 % for E5M2):
//   BF16  one 4.8 / 5.8, two 5.9 / 7.6 (4096 chunks); one 7.4 / 8.2, two 7.8 / 9.6 (8192); one 8.9 / 10.5, two 8.4 / 10.5 (9216); one
//         9.8 / 11.2, two 8.6 / 10.7 (10 240); one 14.1 / 16.8, two 12.3 / 18.0 (16 384)
//   E5M2  one 5.7 / 6.7, two 5.8 / 7.1 (8192); one 6.7 / 8.2, two 6.4 / 7.8 (10 240); two 9.6 / 10.4, four 9.6 / 11.3 (16 384); two
//         11.7 / 12.9, four 11.8 / 12.6 (20 480); one 26.7 / 35.7, two 26.5 / 33.1, four 28.9 / 33.2 (65 536)
// Beyond, one chunk would be up to 12 % faster for E5M2 from 16 384 to 24 576 chunks with 8 % escapes, and for long BF16 streams
// it is about as fast as two (131 072 chunks 79.8 and 80.7).
uint32_t pick_decompress_cpw(uint64_t n_chunks, bool several, bool escapes, int dtype, uint64_t cus) {
  if (const uint32_t forced = g_hooks.cpw.load()) return forced < most_cpw(dtype, several) ? forced : most_cpw(dtype, several);
  const uint64_t round = cus * 8;   // workgroups resident at a time
  if (dtype == SPLITZIP_BF16) return (n_chunks >= (escapes ? 9 : 5) * round / 2 && n_chunks <= 8 * round) || n_chunks >= (several ? 16 : 56) * round ? 2u : 1u;
  if (n_chunks >= 40 * round && n_chunks < 512 * round) return 2;
  return n_chunks >= (escapes ? 10 : 8) * round ? 4u : n_chunks >= (escapes ? 5 : 4) * round ? 2u : 1u;
}

// tables must describe one bijection between 16 codes and 16 distinct exponents
bool codebook_ok(const splitzip_codebook* cb, int dtype) {
  if (!cb || cb->dtype != (uint32_t)dtype) return false;
  unsigned members = 0;
  for (unsigned v = 0; v < 256; ++v) {
    if (cb->member[v] > 1) return false;
    if (cb->member[v]) {
      if (v >= exp_values(dtype) || cb->enc[v] > 15 || cb->dec[cb->enc[v]] != v) return false;
      ++members;
    } else if (cb->enc[v] != 0) {
      return false;
    }
  }
  return members == 16;
}

// codebook_ok for the tensors of one call, one after the other.  They share codebooks as a rule, K's and V's by turns: the
// two looked at last are not looked at again (0.08 us each, 64 of them more than the launches of a small batch).
struct CallCodebooks {
  const splitzip_codebook *last = nullptr, *before = nullptr;
  bool ok(const splitzip_codebook* cb, int dtype) {
    if (cb && (cb == last || cb == before)) return true;
    if (!codebook_ok(cb, dtype)) return false;
    before = last;
    last = cb;
    return true;
  }
};

// Somewhere in the tags' range, another place in every process and for every copy of this library.
uint64_t first_call() {
  timespec now;
  clock_gettime(CLOCK_REALTIME, &now);
  const uint64_t x = ((uint64_t)now.tv_sec * 1000000000ull + (uint64_t)now.tv_nsec) ^ (reinterpret_cast<uintptr_t>(&g_hooks) << 20) ^ ((uint64_t)getpid() << 40);
  return x * 0x9e3779b97f4a7c15ull;
}
// The next tensors of a batch that go into one launch, of n: kBatchFew, and more up to kBatchMax as long as the launch's row
// of workgroups per tensor, as long as the longest, leaves no more than 8192 workgroups without a tile of four chunks (2 us).
// most_chunks: of the longest.
template <typename Item>
uint32_t tensors_of_launch(const Item* items, uint32_t n, uint64_t* most_chunks = nullptr) {
  uint64_t all = 0, most = 0;
  uint32_t k = 0;
  for (; k < n && k < kBatchMax; ++k) {
    const uint64_t c = chunks_of(items[k].n_elems), longest = c > most ? c : most;
    if (k >= kBatchFew && longest * (k + 1) - (all + c) > 4 * 8192) break;
    all += c;
    most = longest;
  }
  if (most_chunks) *most_chunks = most;
  return k;
}
// The same for a compress call.  The tensors of a launch share the workspace, which is sized for one of them: the more they are, the less
// has a tile for its records, and tiles whose records outgrow their slots are encoded twice, 16 of them one after another.  So
// more than kBatchFew are for launches where a chunk has room for four records, what the staging area alone leaves each of
// kBatchFew tensors (KV tensors have one or two); others are halved or cut in three.  us per call, BF16, in launches of 64 with slots in the staging
// area alone, of 160 and this way: 160 tensors of 4096 chunks 382 / 386 / 372 (0.12 % escapes), 418 / 479 / 376 (0.25), 523 / 629 / 400 (0.4); of 8192 745 /
// 859 / 742, 812 / 1138 / 769, of 32 768 2972 / 3464 / 2956; 100 of 16 384 (0.25) 1016 / 1170 / 925; E5M2 160 of 8192 (0.25) 457 / 654 / 426.
constexpr uint64_t kRecordsPerChunk = 4;
uint32_t tensors_of_compress(const splitzip_item* items, uint32_t n, uint64_t status_bytes, uint64_t stage_bytes) {
  uint64_t longest;
  const uint32_t k = tensors_of_launch(items, n, &longest);
  const uint64_t chunks = (g_hooks.stage_bytes ? stage_bytes : status_bytes + stage_bytes) / (4 * kRecordsPerChunk);   // that have so much room
  if (k <= kBatchFew || k * longest <= chunks) return k;
  const uint64_t fit = chunks / longest, most = fit > kBatchFew ? fit : kBatchFew, launches = (k + most - 1) / most;
  return (uint32_t)((k + launches - 1) / launches);
}

// The tag of a call of compress_short_kernel: no two calls of a process have the same one.
uint64_t next_call_tag() {
  static std::atomic<uint64_t> calls{first_call()};
  uint64_t tag;
  do tag = calls.fetch_add(1, std::memory_order_relaxed) << kShortTagShift;
  while (!tag);   // what cleared memory holds
  return tag;
}
// How many CUs a launch of so many workgroups that is enqueued now can have, and 0 if it may run more than once: a captured launch is
// replayed with the tag that it was captured with.  Where there are few workgroups, any part of a chip has room for them, and nobody is
// asked: for the current device 0.05 us, for a stream's mask 0.2.
constexpr uint64_t kMostCus = 1024;
uint64_t cus_once(hipStream_t st, uint64_t wgs) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) != hipSuccess) {
    (void)hipGetLastError();   // the legacy stream while another one is captured: the launch will say so itself
    return 0;
  }
  if (s != hipStreamCaptureStatusNone) return 0;
  if (wgs <= 32) return kMostCus;
  const uint64_t all = (uint64_t)cu_count();
  if (!st || g_hooks.short_anywhere) return all;
  uint32_t mask[kMostCus / 32] = {0};
  if (all > kMostCus || hipExtStreamGetCUMask(st, (uint32_t)(all + 31) / 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return all;
  }
  uint64_t cus = 0;
  for (const uint32_t w : mask) cus += (uint64_t)__builtin_popcount(w);
  return cus && cus < all ? cus : all;
}

constexpr uint32_t kShortLooks = 64;   // about 50 us
uint32_t short_looks() {
  const uint32_t forced = g_hooks.short_looks.load();
  return forced ? forced : kShortLooks;
}

// ---------------------------------------------------------------------------
// format variants: host side
// ---------------------------------------------------------------------------

bool variant_ok(const splitzip_variant* v) {
  if (!v || v->dtype > SPLITZIP_FP8_E4M3) return false;
  if (v->code_bits != 3 && v->code_bits != 4) return false;
  if (v->escape_mode > SPLITZIP_ESC_ABS32) return false;
  const uint32_t codes = 1u << v->code_bits;
  const uint32_t kmax = v->escape_mode == SPLITZIP_ESC_SENTINEL ? codes - 1 : codes;
  if (v->k < 1 || v->k > kmax || v->k > v_exp_values(v->dtype)) return false;
  if (v->escape_mode != SPLITZIP_ESC_ABS32 && v->chunk_elems != 256 && v->chunk_elems != 1024) return false;
  if (v->value_bits != 0 && v->value_bits != 8 && v->value_bits != v_exp_bits(v->dtype)) return false;
  return true;
}

// exactly the first k entries of dec are members, with codes 0 .. k-1
bool variant_codebook_ok(const splitzip_codebook* cb, const splitzip_variant* v) {
  if (!cb || cb->dtype != v->dtype) return false;
  unsigned members = 0;
  for (unsigned e = 0; e < 256; ++e) {
    if (cb->member[e] > 1) return false;
    if (cb->member[e]) {
      if (e >= v_exp_values(v->dtype) || cb->enc[e] >= v->k || cb->dec[cb->enc[e]] != e) return false;
      ++members;
    }
  }
  return members == v->k;
}

// the part of VArgs that follows from (n, variant): layout and chunking
void variant_layout(uint64_t n, const splitzip_variant* v, VArgs* a) {
  memset(a, 0, sizeof *a);
  const bool absolute = v->escape_mode == SPLITZIP_ESC_ABS32;
  a->n = n;
  a->dtype = v->dtype; a->code_bits = v->code_bits; a->k = v->k; a->mode = v->escape_mode;
  a->chunk_shift = absolute || v->chunk_elems == 1024 ? 10 : 8;
  a->pos_bytes = v_pos_bytes(v->escape_mode, v->chunk_elems);
  a->val_bits = v->value_bits ? v->value_bits : 8u;
  a->n_chunks = (n + (1ull << a->chunk_shift) - 1) >> a->chunk_shift;
  a->sm_bytes = (n * v_sm_bits(v->dtype) + 7) / 8;
  a->code_bytes = (n * v->code_bits + 7) / 8;
  a->off_tab = kHeaderBytes;
  a->off_sm = a256(kHeaderBytes + (absolute ? 0 : 4 * (a->n_chunks + 1)));
  a->off_code = a->off_sm + a256(a->sm_bytes);
  a->off_pos = a->off_code + a256(a->code_bytes);
  a->n_tiles = (uint32_t)((a->n_chunks + kVScanTile - 1) / kVScanTile);
  if (a->n_tiles == 0) a->n_tiles = 1;
}

// header words of a stream of this call (M and total, words 6..9, are the kernels' business) and the tables
void variant_tables(const splitzip_variant* v, const splitzip_codebook* cb, VArgs* a) {
  memcpy(a->dec, cb->dec, 16);
  for (uint32_t j = v->k; j < 16; ++j) a->dec[j] = 0;
  a->hdr[0] = 0x31505A53u;   // "SZP1"
  a->hdr[1] = 2u | (a->dtype << 16) | (a->code_bits << 24);
  a->hdr[2] = a->mode == SPLITZIP_ESC_ABS32 ? 0u : 1u << a->chunk_shift;
  a->hdr[3] = a->mode | (a->k << 8) | ((a->val_bits == 8 ? 0u : a->val_bits) << 16);
  a->hdr[4] = (uint32_t)a->n;
  a->hdr[5] = (uint32_t)(a->n >> 32);
  for (int i = 0; i < 4; ++i)
    a->hdr[10 + i] = a->dec[4 * i] | (a->dec[4 * i + 1] << 8) | (a->dec[4 * i + 2] << 16) | ((uint32_t)a->dec[4 * i + 3] << 24);
}

#define SPLITZIP_V_DISPATCH2(KERNEL, grid, block, st, args) SPLITZIP_V_DISPATCH3(KERNEL, args, grid, block, st, args)
#define SPLITZIP_V_DISPATCH3(KERNEL, v, grid, block, st, args)                                                     \
  do {                                                                                                             \
    const int key_ = (int)(v).dtype * 2 + ((v).code_bits == 4 ? 1 : 0);                                            \
    switch (key_) {                                                                                                \
      case 0: hipLaunchKernelGGL((KERNEL<SPLITZIP_BF16, 3>), grid, block, 0, st, args); break;                     \
      case 1: hipLaunchKernelGGL((KERNEL<SPLITZIP_BF16, 4>), grid, block, 0, st, args); break;                     \
      case 2: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E5M2, 3>), grid, block, 0, st, args); break;                 \
      case 3: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E5M2, 4>), grid, block, 0, st, args); break;                 \
      case 4: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E4M3, 3>), grid, block, 0, st, args); break;                 \
      default: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E4M3, 4>), grid, block, 0, st, args); break;                \
    }                                                                                                              \
  } while (0)
#define SPLITZIP_V_DISPATCH1(KERNEL, dtype, grid, block, st, args)                                                 \
  do {                                                                                                             \
    switch (dtype) {                                                                                        \
      case SPLITZIP_BF16: hipLaunchKernelGGL((KERNEL<SPLITZIP_BF16>), grid, block, 0, st, args); break;            \
      case SPLITZIP_FP8_E5M2: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E5M2>), grid, block, 0, st, args); break;    \
      default: hipLaunchKernelGGL((KERNEL<SPLITZIP_FP8_E4M3>), grid, block, 0, st, args); break;                   \
    }                                                                                                              \
  } while (0)

template <int DT, int CB>
constexpr auto v_short_one = v_short_kernel<DT, CB, 1>;
template <int DT, int CB>
constexpr auto v_short_two = v_short_kernel<DT, CB, 2>;
// Blocks per wave of v_short_kernel if it takes a tensor of so many blocks, else 0: by the launch's workgroups, as in pick_short.  Its words
// lie in the blocks' slots, 2 KB per tile of four blocks; a tensor of one tile has no words.
uint32_t variant_short(uint64_t blocks, hipStream_t st) {
  if (!blocks || blocks > 2 * kWaves * kShortTiles || g_hooks.short_looks.load() == kNoShort) return 0;
  const uint32_t bpw = blocks <= kWaves * kShortTiles ? 1 : 2;
  const uint64_t cus = cus_once(st, (blocks + bpw * kWaves - 1) / (bpw * kWaves));
  return blocks <= kWaves * cus && bpw == 1 ? 1 : blocks <= 2 * kWaves * cus ? 2 : 0;
}

void launch_v_pack(uint64_t n_elems, hipStream_t st, const VArgs& a) {
  // M is known to the device only: a grid that strides over however many bytes the section has
  uint64_t g = (v_val_bytes(n_elems, a.val_bits) + kThreads - 1) / kThreads;
  const uint64_t cap = (uint64_t)cu_count() * 8;
  if (g > cap) g = cap;
  hipLaunchKernelGGL(v_pack_kernel, dim3((unsigned)g), dim3(kThreads), 0, st, a);
}

template <int DT>
void launch_v_finish(dim3 g, hipStream_t st, const VArgs& a) {
  const dim3 b(kThreads);
  switch (a.pos_bytes) {
    case 0: hipLaunchKernelGGL((v_finish_kernel<DT, 0>), g, b, 0, st, a); break;
    case 1: hipLaunchKernelGGL((v_finish_kernel<DT, 1>), g, b, 0, st, a); break;
    case 2: hipLaunchKernelGGL((v_finish_kernel<DT, 2>), g, b, 0, st, a); break;
    default: hipLaunchKernelGGL((v_finish_kernel<DT, 4>), g, b, 0, st, a); break;
  }
}

constexpr unsigned kVDecodeLdsPad = 13800;   // unused LDS asked for at the launch: seven workgroups of v_decode_kernel per CU

template <int DT, int CB>
void launch_v_decode(unsigned grid, hipStream_t st, uint32_t mode, uint32_t chunk_shift, const VDecodeArgs& a) {
  const dim3 g(grid), b(kThreads);
  if (mode == SPLITZIP_ESC_POS) {
    // Long launches of BF16 under 4-bit codes: seven workgroups per CU instead of eight.  us per call with eight / seven / six:
    // 39.0 / 38.6 / 38.9 (65 536 chunks), 59.2 / 58.1 / 57.8 (98 304), 77.4 / 76.0 / 76.3 (131 072), 300.6 / 294.0 / 294.5 (524 288);
    // 3-bit codes, sentinels and FP8 gain nothing by it (131 072 chunks: 75.3 / 76.1, 75.9 / 79.9, E5M2 50.4 / 50.6), nor do streams
    // with more than one escape in 16 elements (98 304 chunks, 6.6 %: 60.2 / 61.5), by the bytes beyond the fixed part.
    const unsigned pad = DT == SPLITZIP_BF16 && CB == 4 && grid >= 16384u && !many_escapes(a.capacity - a.off_pos, a.n) ? kVDecodeLdsPad : 0u;
    if (chunk_shift == 10) hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_POS, 10>), g, b, pad, st, a);
    else hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_POS, 8>), g, b, 0, st, a);
  } else if (mode == SPLITZIP_ESC_SENTINEL) {
    // By what the caller says it holds beyond the fixed part, a value per escape: more than a quarter of the elements, or
    // half of them where values are packed and take two loads each (32 Mi words of E5M2, top-7, 5 bits: a fifth
    // escaped, 45.1 us and 52.8 this way; about half 57.8 and 58.3; all that random words make escape 62.5 and 60.4).
    const uint64_t values = (a.capacity - a.off_pos) * 8 / a.val_bits;
    const bool many = values > (a.val_bits == 8 ? a.n / 4 : a.n / 2);
    if (many && chunk_shift == 10) hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_SENTINEL, 10, true>), g, b, 0, st, a);
    else if (many) hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_SENTINEL, 8, true>), g, b, 0, st, a);
    else if (chunk_shift == 10) hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_SENTINEL, 10>), g, b, 0, st, a);
    else hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_SENTINEL, 8>), g, b, 0, st, a);
  } else {
    hipLaunchKernelGGL((v_decode_kernel<DT, CB, SPLITZIP_ESC_ABS32, 10>), g, b, 0, st, a);
  }
}

}  // namespace

extern "C" {

int splitzip_version(void) { return 1; }


// ---- format variants ---------------------------------------------------------

int splitzip_variant_supported(const splitzip_variant* v) { return variant_ok(v) ? 1 : 0; }

size_t splitzip_variant_total_bytes(uint64_t n_elems, uint64_t n_escapes, const splitzip_variant* v) {
  if (!variant_ok(v) || (n_elems >> 32)) return 0;
  VArgs a;
  variant_layout(n_elems, v, &a);
  return a.off_pos + a256(a.pos_bytes * n_escapes) + v_val_bytes(n_escapes, a.val_bits);
}

size_t splitzip_variant_compress_bound(uint64_t n_elems, const splitzip_variant* v) {
  return splitzip_variant_total_bytes(n_elems, n_elems, v);
}

size_t splitzip_variant_workspace_bytes(uint64_t n_elems, const splitzip_variant* v) {
  if (!variant_ok(v) || (n_elems >> 32)) return 0;
  VArgs a;
  variant_layout(n_elems, v, &a);
  const uint64_t n_blocks = (n_elems + kVBlock - 1) / kVBlock;
  return a256(4 * a.n_chunks + 4) + a256(4 * (a.n_chunks + 1)) + a256(4 * (uint64_t)a.n_tiles) +
         a256(4ull * kVSlotCap * n_blocks) +         // the blocks' slots of staged escape records
         (a.val_bits == 8 ? 0 : a256(n_elems));   // values narrower than a byte are packed from whole bytes kept here
}

int splitzip_variant_codebook_from_dec(const uint8_t* dec, const splitzip_variant* v, splitzip_codebook* out) {
  if (!dec || !out || !variant_ok(v)) return SPLITZIP_ERR_INVALID_ARG;
  memset(out, 0, sizeof *out);
  out->dtype = v->dtype;
  for (uint32_t j = 0; j < v->k; ++j) {
    if (dec[j] >= v_exp_values(v->dtype) || out->member[dec[j]]) return SPLITZIP_ERR_INVALID_ARG;
    out->dec[j] = dec[j];
    out->enc[dec[j]] = (uint8_t)j;
    out->member[dec[j]] = 1;
  }
  return SPLITZIP_OK;
}

int splitzip_variant_calibrate(const void* h_sample, uint64_t n_elems, const splitzip_variant* v,
                               splitzip_codebook* out, uint64_t* hist_out) {
  if (!out || !variant_ok(v) || (n_elems && !h_sample)) return SPLITZIP_ERR_INVALID_ARG;
  uint64_t hist[256] = {0};
  if (v->dtype == SPLITZIP_BF16) {
    const uint16_t* p = static_cast<const uint16_t*>(h_sample);
    for (uint64_t i = 0; i < n_elems; ++i) hist[(p[i] >> 7) & 0xff]++;
  } else {
    const uint8_t* p = static_cast<const uint8_t*>(h_sample);
    const unsigned shift = v->dtype == SPLITZIP_FP8_E5M2 ? 2 : 3, mask = v->dtype == SPLITZIP_FP8_E5M2 ? 0x1f : 0xf;
    for (uint64_t i = 0; i < n_elems; ++i) hist[(p[i] >> shift) & mask]++;
  }
  if (hist_out) memcpy(hist_out, hist, sizeof hist);
  // the ranking of splitzip_codebook_from_hist, cut at k
  const unsigned nv = v_exp_values(v->dtype);
  uint8_t top[16];
  unsigned filled = 0;
  for (unsigned e = 0; e < nv; ++e) {
    unsigned at = filled;
    while (at > 0 && hist[top[at - 1]] < hist[e]) --at;
    if (at >= 16) continue;
    const unsigned last = filled < 16 ? filled : 15;
    for (unsigned i = last; i > at; --i) top[i] = top[i - 1];
    top[at] = (uint8_t)e;
    if (filled < 16) ++filled;
  }
  return splitzip_variant_codebook_from_dec(top, v, out);
}

int splitzip_variant_compress(const void* d_in, uint64_t n_elems, const splitzip_variant* v,
                              const splitzip_codebook* cb, void* d_out, size_t out_capacity, void* d_workspace,
                              size_t workspace_bytes, splitzip_sizes* d_sizes, void* stream) {
  if (!variant_ok(v) || !variant_codebook_ok(cb, v) || !d_out || !d_sizes || !d_workspace || (n_elems && !d_in))
    return SPLITZIP_ERR_INVALID_ARG;
  if (!aligned16(d_in) || !aligned16(d_out) || !aligned16(d_workspace) || (reinterpret_cast<uintptr_t>(d_sizes) & 7u))
    return SPLITZIP_ERR_INVALID_ARG;
  if (n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
  if (out_capacity < splitzip_variant_total_bytes(n_elems, 0, v) ||
      workspace_bytes < splitzip_variant_workspace_bytes(n_elems, v))
    return SPLITZIP_ERR_CAPACITY;

  VArgs a;
  variant_layout(n_elems, v, &a);
  a.in = static_cast<const uint8_t*>(d_in);
  a.out = static_cast<uint8_t*>(d_out);
  a.capacity = out_capacity;
  a.sizes = d_sizes;
  a.counts = static_cast<uint32_t*>(d_workspace);
  uint8_t* ws = static_cast<uint8_t*>(d_workspace);
  a.offs = v->escape_mode == SPLITZIP_ESC_ABS32 ? reinterpret_cast<uint32_t*>(ws + a256(4 * a.n_chunks + 4))
                                                : reinterpret_cast<uint32_t*>(a.out + a.off_tab);
  a.tile_sums = reinterpret_cast<uint32_t*>(ws + a256(4 * a.n_chunks + 4) + a256(4 * (a.n_chunks + 1)));
  const uint64_t blocks = (n_elems + kVBlock - 1) / kVBlock;
  a.slots = reinterpret_cast<uint32_t*>(ws + a256(4 * a.n_chunks + 4) + a256(4 * (a.n_chunks + 1)) + a256(4 * (uint64_t)a.n_tiles));
  a.val_stage = reinterpret_cast<uint8_t*>(a.slots) + a256(4ull * kVSlotCap * blocks);
  variant_tables(v, cb, &a);
  a.escape_code = v->escape_mode == SPLITZIP_ESC_SENTINEL ? (1u << v->code_bits) - 1u : 0u;

  const hipStream_t st = static_cast<hipStream_t>(stream);
  const unsigned grid = (unsigned)((blocks + kWaves - 1) / kWaves);
  // A tensor of up to kVDirectSums workgroups needs no launch between the two passes (64 MiB of BF16: 4.7 us and the
  // gap in front of it); the sums of the workgroups lie where the absolute mode has its one word at [n_chunks] and
  // the other modes nothing.
  a.wg_sums = reinterpret_cast<uint32_t*>(ws + a256(4 * a.n_chunks + 4));
  const bool direct = grid <= kVDirectSums;
  a.sums = direct ? a.wg_sums : a.tile_sums;
  a.n_sums = direct ? grid : a.n_tiles;
  a.sum_shift = direct ? 2u + (10u - a.chunk_shift) : 10u;
  a.ahead = v->k <= 8 ? 64u : 16u;   // a top-8 codebook leaves about 60 records per block, a larger one one or two
  if (const uint32_t bpw = variant_short(blocks, st)) {
    VShortArgs sa;
    sa.a = a;
    sa.short_words = reinterpret_cast<uint64_t*>(a.slots);
    sa.tag = next_call_tag();
    sa.looks = short_looks();
    sa.tiles = (unsigned)((blocks + bpw * kWaves - 1) / (bpw * kWaves));
    if (bpw == 1) SPLITZIP_V_DISPATCH3(v_short_one, a, dim3(sa.tiles), dim3(kThreads), st, sa);
    else SPLITZIP_V_DISPATCH3(v_short_two, a, dim3(sa.tiles), dim3(kThreads), st, sa);
    if (a.val_bits != 8) launch_v_pack(n_elems, st, a);
    return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
  }
  if (grid) SPLITZIP_V_DISPATCH2(v_dense_kernel, dim3(grid), dim3(kThreads), st, a);
  if (!direct) hipLaunchKernelGGL(v_tile_sum_kernel, dim3(a.n_tiles), dim3(1024), 0, st, a);
  const unsigned fgrid = (unsigned)((blocks + kVFinishBlocks - 1) / kVFinishBlocks);
  const dim3 fg(fgrid ? fgrid : 1u);
  switch (a.dtype) {
    case SPLITZIP_BF16: launch_v_finish<SPLITZIP_BF16>(fg, st, a); break;
    case SPLITZIP_FP8_E5M2: launch_v_finish<SPLITZIP_FP8_E5M2>(fg, st, a); break;
    default: launch_v_finish<SPLITZIP_FP8_E4M3>(fg, st, a); break;
  }
  if (grid && a.val_bits != 8) launch_v_pack(n_elems, st, a);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

int splitzip_variant_decompress(const void* d_comp, size_t comp_bytes, uint64_t n_elems, const splitzip_variant* v,
                                const splitzip_codebook* cb, void* d_out, splitzip_sizes* d_sizes, void* stream) {
  if (!variant_ok(v) || !variant_codebook_ok(cb, v) || !d_comp || (n_elems && !d_out)) return SPLITZIP_ERR_INVALID_ARG;
  if (!aligned16(d_comp) || !aligned16(d_out) || (reinterpret_cast<uintptr_t>(d_sizes) & 7u))
    return SPLITZIP_ERR_INVALID_ARG;
  if (n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
  if (comp_bytes < splitzip_variant_total_bytes(n_elems, 0, v)) return SPLITZIP_ERR_CAPACITY;

  VArgs l;
  variant_layout(n_elems, v, &l);
  variant_tables(v, cb, &l);
  VDecodeArgs a;
  a.in = static_cast<const uint8_t*>(d_comp);
  a.out = static_cast<uint8_t*>(d_out);
  a.sizes = d_sizes;
  a.capacity = comp_bytes;
  a.n = (uint32_t)n_elems;
  a.n_chunks = (uint32_t)l.n_chunks;
  a.k = l.k;
  a.val_bits = l.val_bits;
  a.off_pos = l.off_pos;
  a.tab = reinterpret_cast<const uint32_t*>(a.in + l.off_tab);
  a.sm = n_elems ? a.in + l.off_sm : a.in;
  a.code = n_elems ? a.in + l.off_code : a.in;
  a.sm_last = n_elems ? (uint32_t)(a256(l.sm_bytes) - v_sm_bits(l.dtype) / 8 * 4 - 4) : 0u;   // a load is 8 bytes of 8-bit fields, 4 of narrower ones
  a.code_last = n_elems ? (uint32_t)(a256(l.code_bytes) - 4) : 0u;
  a.pos = a.in + l.off_pos;
  memcpy(a.hdr, l.hdr, sizeof a.hdr);
  memcpy(a.dec, l.dec, sizeof a.dec);

  const hipStream_t st = static_cast<hipStream_t>(stream);
  const uint64_t blocks = (n_elems + kVBlock - 1) / kVBlock;
  const unsigned grid = blocks ? (unsigned)((blocks + kWaves - 1) / kWaves) : 1u;
  switch ((int)l.dtype * 2 + (l.code_bits == 4 ? 1 : 0)) {
    case 0: launch_v_decode<SPLITZIP_BF16, 3>(grid, st, l.mode, l.chunk_shift, a); break;
    case 1: launch_v_decode<SPLITZIP_BF16, 4>(grid, st, l.mode, l.chunk_shift, a); break;
    case 2: launch_v_decode<SPLITZIP_FP8_E5M2, 3>(grid, st, l.mode, l.chunk_shift, a); break;
    case 3: launch_v_decode<SPLITZIP_FP8_E5M2, 4>(grid, st, l.mode, l.chunk_shift, a); break;
    case 4: launch_v_decode<SPLITZIP_FP8_E4M3, 3>(grid, st, l.mode, l.chunk_shift, a); break;
    default: launch_v_decode<SPLITZIP_FP8_E4M3, 4>(grid, st, l.mode, l.chunk_shift, a); break;
  }
  if (v->escape_mode == SPLITZIP_ESC_ABS32 && n_elems) {
    // M is known to the device only: a grid that strides over whatever the header says
    const uint64_t most = (comp_bytes - a.off_pos) / 5;
    uint64_t g = (most + kThreads - 1) / kThreads;
    const uint64_t cap = (uint64_t)cu_count() * 8;
    if (g > cap) g = cap;
    if (g) SPLITZIP_V_DISPATCH1(v_scatter_kernel, l.dtype, dim3((unsigned)g), dim3(kThreads), st, a);
  }
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

const char* splitzip_strerror(int err) {
  switch (err) {
    case SPLITZIP_OK: return "ok";
    case SPLITZIP_ERR_INVALID_ARG: return "invalid argument";
    case SPLITZIP_ERR_UNSUPPORTED: return "unsupported size or format";
    case SPLITZIP_ERR_CAPACITY: return "buffer too small";
    case SPLITZIP_ERR_HIP: return "HIP runtime error";
    default: return "unknown error";
  }
}

int splitzip_codebook_from_dec(const uint8_t dec[16], int dtype, splitzip_codebook* out) {
  if (!dec || !out || !dtype_ok(dtype)) return SPLITZIP_ERR_INVALID_ARG;
  splitzip_codebook cb;
  memset(&cb, 0, sizeof cb);
  cb.dtype = (uint32_t)dtype;
  for (unsigned k = 0; k < 16; ++k) {
    const unsigned v = dec[k];
    if (v >= exp_values(dtype) || cb.member[v]) return SPLITZIP_ERR_INVALID_ARG;
    cb.dec[k] = (uint8_t)v;
    cb.enc[v] = (uint8_t)k;
    cb.member[v] = 1;
  }
  *out = cb;
  return SPLITZIP_OK;
}

int splitzip_calibrate(const void* h_sample, uint64_t n_elems, int dtype, splitzip_codebook* out,
                       uint64_t* hist_out) {
  if (!out || !dtype_ok(dtype) || (n_elems && !h_sample)) return SPLITZIP_ERR_INVALID_ARG;
  uint64_t hist[256] = {0};
  if (dtype == SPLITZIP_BF16) {
    const uint16_t* p = static_cast<const uint16_t*>(h_sample);
    for (uint64_t i = 0; i < n_elems; ++i) hist[(p[i] >> 7) & 0xff]++;
  } else {
    const uint8_t* p = static_cast<const uint8_t*>(h_sample);
    for (uint64_t i = 0; i < n_elems; ++i) hist[(p[i] >> 2) & 0x1f]++;
  }
  if (hist_out) memcpy(hist_out, hist, sizeof hist);
  return splitzip_codebook_from_hist(hist, dtype, out);
}

int splitzip_codebook_from_hist(const uint64_t hist[256], int dtype, splitzip_codebook* out) {
  if (!hist || !out || !dtype_ok(dtype)) return SPLITZIP_ERR_INVALID_ARG;
  // rank exponents by (count descending, value ascending): insertion into a sorted top-16 list
  const unsigned nv = exp_values(dtype);
  uint8_t top[16];
  unsigned filled = 0;
  for (unsigned v = 0; v < nv; ++v) {
    unsigned at = filled;
    while (at > 0 && hist[top[at - 1]] < hist[v]) --at;   // strict: equal counts keep the smaller value first
    if (at >= 16) continue;
    const unsigned last = filled < 16 ? filled : 15;
    for (unsigned i = last; i > at; --i) top[i] = top[i - 1];
    top[at] = (uint8_t)v;
    if (filled < 16) ++filled;
  }
  return splitzip_codebook_from_dec(top, dtype, out);
}

int splitzip_histogram(const void* d_sample, uint64_t n_elems, int dtype, uint64_t* d_hist, void* stream) {
  if (!dtype_ok(dtype) || !d_hist || (n_elems && !d_sample) || !aligned16(d_sample) ||
      (reinterpret_cast<uintptr_t>(d_hist) & 7u))
    return SPLITZIP_ERR_INVALID_ARG;
  if (n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
  if (n_elems == 0) return SPLITZIP_OK;
  const uint64_t nvec = (n_elems * (dtype == SPLITZIP_BF16 ? 2 : 1) + 15) / 16;
  uint64_t grid = (nvec + 4 * 1024 - 1) / (4 * 1024);   // at least four vectors per thread
  const uint64_t most = (uint64_t)cu_count();   // one workgroup per CU: with two, their 512 final adds per bin cost more than the extra waves bring
  if (grid > most) grid = most;
  if (grid < 1) grid = 1;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == SPLITZIP_BF16)
    hipLaunchKernelGGL(histogram_kernel<true>, dim3((unsigned)grid), dim3(1024), 0, st, static_cast<const uint8_t*>(d_sample), n_elems, d_hist);
  else
    hipLaunchKernelGGL(histogram_kernel<false>, dim3((unsigned)grid), dim3(1024), 0, st, static_cast<const uint8_t*>(d_sample), n_elems, d_hist);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

size_t splitzip_total_bytes(uint64_t n_elems, uint64_t n_escapes, int dtype) {
  if (!dtype_ok(dtype) || n_elems >> 32) return 0;
  const Layout L = make_layout(n_elems, dtype);
  return (size_t)(L.off_pos + a256(2 * n_escapes) + n_escapes);
}
size_t splitzip_fixed_bytes(uint64_t n_elems, int dtype) { return splitzip_total_bytes(n_elems, 0, dtype); }
size_t splitzip_compress_bound(uint64_t n_elems, int dtype) { return splitzip_total_bytes(n_elems, n_elems, dtype); }

size_t splitzip_workspace_bytes(uint64_t n_elems, int dtype) {
  if (!dtype_ok(dtype) || n_elems >> 32) return 0;
  return (size_t)(kWsHeaderBytes + kStatusBytes + kStageFloor + a256(n_elems));
}

int splitzip_workspace_init(void* d_workspace, size_t workspace_bytes, void* stream) {
  if (!d_workspace || !aligned16(d_workspace) || workspace_bytes < kWsHeaderBytes + kStatusBytes + kStageFloor)
    return SPLITZIP_ERR_INVALID_ARG;
  // No word of a workspace needs a defined value before a call; the header is cleared all the same, so that what
  // a later version of the library may keep there starts from zero.
  hipLaunchKernelGGL(workspace_init_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                     static_cast<uint32_t*>(d_workspace), (uint32_t)(kWsHeaderBytes / 4));
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

void splitzip_internal_test_hooks(uint64_t stage_bytes, uint64_t status_bytes, uint32_t finish_groups, uint64_t direct_bytes) {
  g_hooks.direct_bytes = direct_bytes;
  g_hooks.stage_bytes = stage_bytes;
  g_hooks.status_bytes = status_bytes;
  g_hooks.finish_groups = finish_groups == 1 || finish_groups == 2 || finish_groups == 4 ? finish_groups : 0;
}

void splitzip_internal_test_short(uint32_t looks, uint32_t anywhere) {
  g_hooks.short_looks = looks;
  g_hooks.short_anywhere = anywhere != 0;
}

void splitzip_internal_test_launch(uint32_t cpt, uint32_t cpw, uint32_t xcd) {
  const auto size_or_0 = [](uint32_t v) { return v == 1 || v == 2 || v == 4 || v == 8 ? v : 0u; };
  g_hooks.cpt = size_or_0(cpt);
  g_hooks.cpw = size_or_0(cpw);
  g_hooks.xcd = xcd <= 2 ? xcd : 0u;
}

}  // extern "C"

namespace {

// table and page geometry of a splitzip_paged as the kernels see them (base left null); false if unusable for
// words of dtype
bool paging_geometry(const splitzip_paged* pg, int dtype, Words* w) {
  if (!pg || !pg->d_block_table || (reinterpret_cast<uintptr_t>(pg->d_block_table) & 3u)) return false;
  const uint64_t es = dtype == SPLITZIP_BF16 ? 2 : 1;
  const uint32_t be = pg->block_elems;
  if (be < kChunk || (be & (be - 1u)) || pg->n_pool_blocks == 0) return false;
  if ((pg->page_stride_bytes & 15u) || (pg->offset_bytes & 15u)) return false;
  if (pg->offset_bytes + (uint64_t)be * es > pg->page_stride_bytes) return false;       // the tensor's part of a page fits the page
  w->base = nullptr;
  w->table = pg->d_block_table;
  w->page_stride = pg->page_stride_bytes;
  w->page_shift = (uint32_t)__builtin_ctz(be);
  w->n_pages = pg->n_pool_blocks;
  return true;
}

// a splitzip_paged as the kernels see it; false if the description is not usable for n_elems words of dtype
bool paged_words(const splitzip_paged* pg, uint64_t n_elems, int dtype, Words* w) {
  if (!paging_geometry(pg, dtype, w) || !pg->d_pool || !aligned16(pg->d_pool)) return false;
  if ((uint64_t)pg->n_blocks * pg->block_elems < n_elems) return false;                   // the table covers the tensor
  w->base = static_cast<uint8_t*>(pg->d_pool) + pg->offset_bytes;
  return true;
}

// ---- the workspace of splitzip_compress_noalloc: one copy per GPU, alive until the process ends ----
// Header, status area and staging area as in a caller's workspace, only smaller.
constexpr uint64_t kScratchStatusBytes = 256u << 10, kScratchStageBytes = 768u << 10;
static __device__ __align__(256) uint32_t scratch[(kWsHeaderBytes + kScratchStatusBytes + kScratchStageBytes) / 4];

// The array's address on the current device (each GPU holds its own copy at its own address), looked up once per
// device with that device current; null if the runtime refuses.  `scratch` itself is a host-side stand-in and is
// never handed to a kernel.
void* scratch_on_current_device() {
  static std::mutex lock;
  static void* ptr[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> hold(lock);
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    ptr[dev] = p;
  }
  return ptr[dev];
}

// a workspace as the compress calls see it: header, then the status words, then the staging of escape values
struct WsView {
  uint8_t* base;
  uint64_t status_bytes, stage_bytes;
};

// the view of a workspace: a caller's (d_workspace non-null: sized by splitzip_workspace_bytes for its largest tensor,
// n_max elements) or the library's own array on the current device; an error code if it is too small or not to be had
int workspace_view(void* d_workspace, size_t workspace_bytes, uint64_t n_max, int dtype, WsView* v) {
  if (d_workspace) {
    if (workspace_bytes < splitzip_workspace_bytes(n_max, dtype)) return SPLITZIP_ERR_CAPACITY;
    v->base = static_cast<uint8_t*>(d_workspace);
    v->status_bytes = kStatusBytes;
    v->stage_bytes = (workspace_bytes - kWsHeaderBytes - kStatusBytes) & ~(uint64_t)255u;
  } else {
    v->base = static_cast<uint8_t*>(scratch_on_current_device());
    if (!v->base) return SPLITZIP_ERR_HIP;
    v->status_bytes = kScratchStatusBytes;
    v->stage_bytes = kScratchStageBytes;
  }
  // tests of the paths that small areas force
  const uint64_t hs = g_hooks.status_bytes, hg = g_hooks.stage_bytes;
  if (hs && hs < v->status_bytes) v->status_bytes = hs;
  if (hg && hg < v->stage_bytes) v->stage_bytes = hg;
  return SPLITZIP_OK;
}

uint64_t tiles_of(uint64_t chunks, uint32_t cpt) { return (chunks + 4ull * cpt - 1) >> (2 + __builtin_ctz(cpt)); }   // cpt: a power of two
// bytes of the status area a tensor of `tiles` tiles takes: a count per tile, a sum per group of tiles
uint64_t status_need(uint64_t tiles) { return a256(4 * tiles + 4 * ((tiles + kSumGroup - 1) / kSumGroup)); }

// chunks per wave and tile for a tensor of `chunks` chunks: `at_least`, doubled until the tensor's counts fit
// `status_bytes`; 0 if nothing fits
uint32_t pick_cpt(uint64_t chunks, uint32_t at_least, uint64_t status_bytes) {
  for (uint32_t cpt = at_least; cpt <= kMaxRange / 4; cpt *= 2)
    if (status_need(tiles_of(chunks, cpt)) <= status_bytes) return cpt;
  return 0;
}

// Chunks per wave and tile to begin with, by the chunks of a launch.  A tile's time is mostly the latency of one wave's
// work, so short launches are split finer, down to where the tiles no longer fill whole rounds of the chip, and long
// ones are bound by how 16 KB runs stream.  us per call (device), by chunks per wave:
//   BF16  one / two: 6.3 / 6.9 (100 chunks), 7.3 / 7.8 (2048), 9.4 / 9.9 (6000), 10.6 / 10.5 (8192), 15.8 / 15.9
//         (16 384), 18.2 / 18.6 (19 200), 27.7 / 25.2 (32 768)
//   E5M2  one / two / four: 6.4 / 6.9 / 8.0 (100), 8.0 / 8.2 / 9.6 (4096), 9.3 / 9.1 / 10.9 (8192), 12.9 / 12.0 / 14.3
//         (16 384), two / four: 17.6 / 18.8 (32 768), 167.6 / 170.1 (524 288), 338.3 / 336.3 (1 Mi), 666 / 661 (2 Mi)
// Tensors that differ in length: the launch has a row of workgroups per tensor, as long as the longest (chunks_padded in
// all), and passes by a workgroup without a tile at about four in a nanosecond.  From 48 of them per CU on the next size
// is better: us by chunks per wave, BF16 one / two: 8.6 / 8.9 (600 chunks beside 63 tensors of 5: 9371 without a tile),
// 12.7 / 10.9 (1500 beside 63 of 50: 22 837), 26.1 / 21.4 (20 000 beside seven of two), 59.1 / 35.2 (13 000 beside 63 of
// two); E5M2 two / four: 10.8 / 11.4 (1500 beside 63 of 50: 11 418), 57.9 / 56.7 (32 of 4096 beside 32 of 512: 14 336),
// 17.4 / 16.7 (20 000 beside seven of two: 17 498), 33.7 / 21.3 (13 000 beside 63 of two).
uint32_t pick_base_cpt(uint64_t chunks, uint64_t chunks_padded, int dtype, uint64_t cus) {
  const uint32_t most = dtype == SPLITZIP_BF16 ? Bf16::kCpt : E5m2::kCpt;
  uint32_t cpt = dtype == SPLITZIP_BF16 ? (chunks <= 20480 ? 1u : 2u) : chunks <= 6144 ? 1u : chunks <= 786432 ? 2u : 4u;
  while (cpt < most && (chunks_padded - chunks) / (4 * cpt) > cus * 48) cpt *= 2;
  return cpt;
}

// the launches of k tensors: dense pass (one workgroup per tile, started by the hardware in the tiles' order), sums if
// the finishing pass wants them, finishing pass
template <typename F, uint32_t N>
void launch_compress(unsigned tiles, unsigned finish_wgs, unsigned sums, unsigned k, bool is_long, unsigned lds_pad, hipStream_t st, const TileArgs<N>& args) {
  if (tiles) {
    const dim3 grid(tiles, k), block(kTileThreads);
    const uint32_t cpt = args.shared.cpt;
    if (cpt == 1) launch(compress_tile_kernel<F, 1, N, kTileOnce>, grid, block, lds_pad, st, args);
    else if (cpt == 2) launch(is_long ? compress_tile_kernel<F, 2, N, kTileLong> : compress_tile_kernel<F, 2, N, kTileOnce>, grid, block, lds_pad, st, args);
    else if (cpt == F::kCpt && (is_long || N > kBatchFew)) launch(compress_tile_kernel<F, F::kCpt, N, kTileLong>, grid, block, lds_pad, st, args);   // four chunks: many tensors are many tiles
    else if constexpr (N <= kBatchFew) launch(cpt == F::kCpt ? compress_tile_kernel<F, F::kCpt, N, kTileOnce> : compress_tile_kernel<F, F::kCpt, N, kTileLoop>, grid, block, lds_pad, st, args);
    if (args.shared.use_group_sums) launch(tile_group_sum_kernel<F, N>, dim3(sums, k), dim3(64), 0, st, args);
  }
  const dim3 grid(finish_wgs ? finish_wgs : 1u, k);
  if (args.shared.finish_groups == 1) launch(compress_finish_kernel<F, N, 1>, grid, dim3(kTileThreads), 0, st, args);
  else if (args.shared.finish_groups == 2) launch(compress_finish_kernel<F, N, 2>, grid, dim3(kTileThreads), 0, st, args);
  else launch(compress_finish_kernel<F, N, 4>, grid, dim3(kTileThreads), 0, st, args);
}

template <typename F>
void launch_small(unsigned k, hipStream_t st, const TileArgs<kBatchMax>& args) {
  if (k == 1) {
    const TileArgs<1> one = {args.shared, {args.item[0]}};
    launch(compress_small_kernel<F, 1>, dim3(1), dim3(kSmallThreads), 0, st, one);
  } else if (k <= kBatchFew) {
    launch(compress_small_kernel<F, kBatchFew>, dim3(k), dim3(kSmallThreads), 0, st, few(args));
  } else {
    launch(compress_small_kernel<F, kBatchMax>, dim3(k), dim3(kSmallThreads), 0, st, args);
  }
}

template <typename F, int CPT>
void launch_short(unsigned tiles, unsigned k, hipStream_t st, const TileArgs<kBatchMax>& args) {
  const dim3 grid(tiles ? tiles : 1u, k), block(kTileThreads);
  if (k == 1) {
    const TileArgs<1> one = {args.shared, {args.item[0]}};
    launch(compress_short_kernel<F, 1, CPT>, grid, block, 0, st, one);
  } else if (k <= kBatchFew) {
    launch(compress_short_kernel<F, kBatchFew, CPT>, grid, block, 0, st, few(args));
  } else if constexpr (CPT == 1) {   // (two chunks per wave: pick_short)
    launch(compress_short_kernel<F, kBatchMax, CPT>, grid, block, 0, st, args);
  }
}

// How the next tensors of a compress call are launched: a function of their lengths, the word type and the status area.
struct CompressPlan {
  uint32_t k;               // tensors of this launch; 0 if not even one fits
  uint32_t cpt;             // chunks per wave and tile
  uint64_t tiles_max;       // of the longest tensor: the dense pass has k rows of so many workgroups
  bool small;               // one launch of compress_small_kernel
  bool is_short;            // one launch of compress_short_kernel
  bool by_xcd;              // the dense pass takes its tiles in xcd_order
  uint32_t lds_pad;         // unused LDS asked for at the launch of the dense pass: fewer workgroups per CU
  bool is_long;             // the dense pass stores through the L2 (kTileLong)
  uint32_t finish_groups;   // groups of kGroup tiles per workgroup of the finishing pass
  uint32_t finish_wgs;      // workgroups of the finishing pass per tensor
  bool group_sums;          // the finishing pass is given sums of kSumGroup tile counts
  uint32_t launches() const { return small || is_short ? 1u : group_sums ? 3u : tiles_max ? 2u : 1u; }
};

constexpr uint32_t kSmallestShort = 16;   // shorter tensors are one workgroup's work
uint64_t short_status_need(uint64_t tiles) { return kShortCopies * short_copy_bytes(tiles); }
// Chunks per wave of compress_short_kernel if it takes these tensors, else 0; wgs: its workgroups with a tile, tiles_max: of the
// longest tensor.
// us per call, one behind the other, of two launches (of one workgroup per tensor up to 40 chunks) and this way: BF16 16 chunks 4.1
// and 4.1, 24 4.6 and 4.0, 40 5.7 and 4.0, 100 6.9 and 4.1, 512 7.0 and 4.2, 1024 7.1 and 4.6, and with two chunks per wave 1025 7.2 and 5.5, 2048 7.3 and
// 5.6; E5M2 100 7.3 and 4.0, 1024 7.0 and 4.2, 2048 7.2 and 5.2; 64 BF16 tensors of 16 chunks 4.85 and 5.0, of 32 6.3 and 5.4, 16 of 100 7.1 and 5.0.
// The line is what calls on several streams leave one another: five workgroups fit a CU (four with two chunks per wave), a
// process has four hardware queues, and where the launches of all are not resident together they wait for workgroups that wait for the
// chip.  us per call of four streams side by side, two launches and this way: BF16 1024 chunks (256 workgroups) 2.0 and 1.6, 1280 2.1 and 1.9, but 1536 2.3
// and 2.3-3.8, 1792 2.4 and 4.4, 2048 2.5 and 5.4, 2816 2.8 and 75; with two chunks per wave 1536 2.3 and 2.0, 2048 2.5 and 2.1.  Of a batch the tensors
// wait only for themselves: 16 of 100 (400 workgroups) 2.4 and 2.0, 64 of 32 (512) 2.4 and 2.3, four of 500 2.6 and 2.5, but two of 1024 2.5 and 2.8, 64 of 60
// 3.5 and 4.3, four of 1000 3.4 and 8.2, and with two chunks per wave 64 of 60 (512) 3.5 and 3.7, four of 1000 3.4 and 4.3.
// On a stream of 32 CUs 2048 chunks take 10 us in two launches and took 360 this way.  Beside elementwise kernels that fill the chip
// 1000 chunks 20.2 and 16.0, 2048 20.2 and 17.6, four of 500 20.8 and 15.8, 64 of 32 21.1 and 14.7; beside matrix products 166 and 109, 165 and 110, 163
// and 103, 103 and 102.
// Tensors that differ in length, as in pick_base_cpt, only that workgroups without a tile ask for more of a CU here; on 1 / 3 / 4 streams,
// two launches and this: one of 500 chunks beside 40 of 12 (4800 workgroups without a tile) 7.6 / 3.5 / 3.0 and 6.2 / 3.0 / 2.8, 1000 beside 40 of 4 (9900) 8.8 / 4.3 /
// 3.4 and 7.2 / 4.0 / 3.7, 1024 beside 20 of 8 (5080) 8.0 / 3.4 / 3.0 and 6.8 / 3.4 / 3.2; two chunks per wave 1500 beside 20 of 8 (3740) 8.3 / 4.0 / 3.6 and 6.9 / 3.0 / 2.8, 1024
// beside 30 of 8 (3810) 9.1 / 4.0 / 3.5 and 8.5 / 4.3 / 4.0, beside 50 of 8 (6350) 10.6 / 7.6 / 3.5 and 11.9 / 8.6 / 4.4.
// What bounds calls of up to 500 chunks now is the host: a launch takes it 2.3 us.
uint32_t pick_short(const splitzip_item* items, uint32_t k, uint64_t status_bytes, uint64_t cus, uint64_t* wgs, uint64_t* tiles_max) {
  uint64_t chunks_max = 0;
  for (uint32_t q = 0; q < k; ++q) {
    const uint64_t c = chunks_of(items[q].n_elems);
    if (c > chunks_max) chunks_max = c;
  }
  if (chunks_max <= kSmallestShort) return 0;
  for (uint32_t cpt = 1; cpt <= kShortMostCpt; cpt *= 2) {
    const uint64_t longest = tiles_of(chunks_max, cpt);
    if (longest > kShortTiles || longest > cus) continue;
    if (cpt > 1 && k > kBatchFew) break;   // so many rows that one would have two chunks per wave for leave more without a tile than the limit below
    uint64_t tiles = 0, need = 0;
    for (uint32_t q = 0; q < k; ++q) {
      const uint64_t t = tiles_of(chunks_of(items[q].n_elems), cpt);
      tiles += t;
      need += short_status_need(t);
    }
    const bool fit = cpt > 1 ? tiles <= cus : longest <= cus / 2 ? tiles <= 2 * cus : tiles <= cus + cus / 4;
    if (fit && longest * k - tiles <= (cpt > 1 ? 3000u : 5000u) && need <= status_bytes) {
      *wgs = tiles;
      *tiles_max = longest;
      return cpt;
    }
  }
  return 0;
}

// items[0, n_items): what is left of the call; n_max: its longest tensor; once(wgs): how many CUs so many workgroups can have, 0 if what
// is enqueued may run more than once
template <typename Once>
CompressPlan plan_compress(const splitzip_item* items, uint32_t n_items, uint64_t n_max, int dtype, uint64_t status_bytes, uint64_t stage_bytes, const Once& once) {
  CompressPlan p;
  memset(&p, 0, sizeof p);
  const uint32_t k_most = tensors_of_compress(items, n_items, status_bytes, stage_bytes);
  uint64_t wgs;
  if (!g_hooks.any() && g_hooks.short_looks.load() != kNoShort && pick_short(items, k_most, status_bytes, kMostCus, &wgs, &p.tiles_max)) {
    p.cpt = pick_short(items, k_most, status_bytes, once(wgs), &wgs, &p.tiles_max);
    if (p.cpt) {
      p.is_short = true;
      p.k = k_most;
      return p;
    }
    p.tiles_max = 0;
  }
  // as many of the next tensors as find room for their counts in the status area; all of them share
  // the tile size of the one that needs the largest
  const uint64_t cus = (uint64_t)cu_count();   // asks the runtime: once per call
  uint64_t chunks_all = 0, chunks_max = 0;
  for (uint32_t q = 0; q < k_most; ++q) {
    const uint64_t c = chunks_of(items[q].n_elems);
    chunks_all += c;
    if (c > chunks_max) chunks_max = c;
  }
  const uint32_t forced_cpt = g_hooks.cpt.load();
  p.cpt = forced_cpt ? forced_cpt : pick_base_cpt(chunks_all, chunks_max * k_most, dtype, cus);
  uint64_t taken = 0;   // of the status area, by the tensors so far
  for (; p.k < k_most; ++p.k) {
    const uint32_t need = pick_cpt(chunks_of(items[p.k].n_elems), p.cpt, status_bytes);
    if (!need || (p.k >= kBatchFew && need > (dtype == SPLITZIP_BF16 ? Bf16::kCpt : E5m2::kCpt))) break;   // there is no kTileLoop for more
    uint64_t total = need == p.cpt ? taken : 0;
    for (uint32_t q = need == p.cpt ? p.k : 0; q <= p.k; ++q) total += status_need(tiles_of(chunks_of(items[q].n_elems), need));
    if (total > status_bytes) break;
    taken = total;
    p.cpt = need;
  }
  uint64_t tiles_all = 0;
  for (uint32_t q = 0; q < p.k; ++q) {
    const uint64_t tiles = tiles_of(chunks_of(items[q].n_elems), p.cpt);
    tiles_all += tiles;
    if (tiles > p.tiles_max) p.tiles_max = tiles;
  }
  p.small = chunks_of(n_max) <= (dtype == SPLITZIP_BF16 ? Bf16::kSmallChunks : E5m2::kSmallChunks) && !g_hooks.any();
  // Launches of 2048 tiles and more take them in xcd_order, BF16 where a wave has two chunks, and from 6144 on with fewer workgroups per CU (Bf16::kTileLdsPad).  us per call,
  // in the order of the tiles, in xcd_order and, BF16, in it with fewer workgroups: BF16, one chunk per wave, 10.93 / 10.78 / 11.40 (2048 tiles: 16 tensors of 512
  // chunks), but 11.84 / 12.18 (one tensor of 9500 chunks), 12.28 / 12.43 (9983), 12.38 / 12.59 (two of 5000), 13.61 / 13.82 (three of 4000), 15.70 / 15.68 / 16.14 (4096 tiles); two
  // 25.46 / 25.27 / 25.53 (4095), 25.07 / 25.02 / 25.28 (4096: one tensor), 34.31 / 34.33 / 34.13 (6144), 43.16 / 42.96 / 42.48 (8192), 78.1 / - / 76.4 (16 000), 1241 / - / 1201 (262 144); E5M2 11.70 / 11.66 (2048), 17.62 / 17.39 and
  // 17.14 / 17.01 (4096), 27.42 / 26.95 (8192), 46.4 / 45.0 (16 000), 690 / 665 (131 072 of 16 KB).  What counts are
  // the tiles that there are: where the tensors differ in length, most of a launch's workgroups may have none, and they
  // take longer to pass by that way (BF16, one tensor of 13 000 chunks beside 63 of two: 35.1 and 40.6; 16 of 8192
  // beside 48 of 16: 91.5 and 95.6; but 32 of 16 384 beside 32 of 16: 328 and 321).
  p.by_xcd = tiles_all >= 2048 && p.tiles_max * p.k <= 2 * tiles_all && (dtype != SPLITZIP_BF16 || p.cpt > 1);
  if (const uint32_t forced = g_hooks.xcd.load()) p.by_xcd = forced == 2;
  p.lds_pad = p.by_xcd && dtype == SPLITZIP_BF16 && (tiles_all >= 6144 || g_hooks.xcd.load() == 2) ? Bf16::kTileLdsPad : 0u;
  // Launches that memory alone bounds store through the L2 (kTileLong).  us per call, without and with:
  // BF16 21.0 and 21.2 (3072 tiles), 25.6 and 25.7 (4096), 35.05 and 34.98 (6144), 82.2 and 80.9 (16 384), 158.2 and
  // 155.8 (32 768), 563 and 561 (122 880); E5M2 11.9 and 12.3 (2048), 17.6 and 17.7 (4096), 23.19 and 23.06 (6144),
  // 28.2 and 27.9 (8192), 89.2 and 88.5 (32 768).
  p.is_long = tiles_all >= 6144;
  const uint32_t groups_max = (uint32_t)((p.tiles_max + kGroup - 1) / kGroup);
  // many groups in the launch: several per workgroup, as long as the chip still gets a few workgroups per CU
  p.finish_groups = 1;
  while (p.finish_groups < kFinishMost && (uint64_t)groups_max * p.k / (2 * p.finish_groups) >= cus * 8) p.finish_groups *= 2;
  if (const uint32_t forced = g_hooks.finish_groups.load()) p.finish_groups = forced;
  p.finish_wgs = (groups_max + p.finish_groups - 1) / p.finish_groups;
  // A finishing workgroup that sums all tile counts of its tensor itself reads 4 bytes per tile: fine while all
  // workgroups of the launch together read no more than kDirectBytes that way, mostly from the L2, and one launch fewer;
  // beyond that they read sums of kSumGroup counts instead (tile_group_sum_kernel).  us per call, with the sums and
  // without, and the MB of counts read without: one BF16 tensor 18.4 and 16.9 (16 385 chunks, 4), 27.6 and 26.1 (32 769,
  // 4), 65.6 and 65.1 (100 000, 39); one E5M2 tensor 20.1 and 18.6 (32 769, 4), 30.2 and 29.1 (65 537, 17), 49.2 and
  // 48.9 (131 072, 67); 64 BF16 tensors of 64 MiB 1262-1292 and 1259 (67).
  const uint64_t direct_budget = g_hooks.direct_bytes.load() ? g_hooks.direct_bytes.load() : kDirectBytes;
  p.group_sums = (uint64_t)p.finish_wgs * p.k * p.tiles_max * 4 > direct_budget;
  return p;
}

// The compress calls, all of them: n_items tensors (a host list), each under its own codebook -- the items' own (host)
// or d_cbs[k] (device memory).  paging: table and page geometry shared by all items, or contiguous tensors (table null).
// d_workspace: the caller's workspace, or null with own_scratch for the library's own array.
int compress_launch(const splitzip_item* items, uint32_t n_items, int dtype, const Words& paging, uint64_t paged_room,
                   const splitzip_codebook* d_cbs, void* d_workspace, size_t workspace_bytes, bool own_scratch,
                   splitzip_sizes* d_sizes, void* stream) {
  if (!dtype_ok(dtype) || (n_items && (!items || !d_sizes)) || (own_scratch ? d_workspace != nullptr : !d_workspace) ||
      !aligned16(d_workspace) || (reinterpret_cast<uintptr_t>(d_sizes) & 7u) || (reinterpret_cast<uintptr_t>(d_cbs) & 3u))
    return SPLITZIP_ERR_INVALID_ARG;
  uint64_t n_max = 0;
  CallCodebooks books;
  for (uint32_t i = 0; i < n_items; ++i) {
    const splitzip_item& it = items[i];
    if (!it.d_out || (it.n_elems && !it.d_in) || !aligned16(it.d_in) || !aligned16(it.d_out) || (!d_cbs && !books.ok(it.cb, dtype)))
      return SPLITZIP_ERR_INVALID_ARG;
    if (it.n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
    if (paging.table && it.n_elems > paged_room) return SPLITZIP_ERR_INVALID_ARG;   // the table does not cover the tensor
    if (it.out_capacity < splitzip_fixed_bytes(it.n_elems, dtype)) return SPLITZIP_ERR_CAPACITY;
    if (it.n_elems > n_max) n_max = it.n_elems;
  }
  WsView ws;
  const int rc = workspace_view(d_workspace, workspace_bytes, n_max, dtype, &ws);
  if (rc != SPLITZIP_OK) return rc;
  if (n_items == 0) return SPLITZIP_OK;
  if (!pick_cpt(chunks_of(n_max), 1, ws.status_bytes)) return SPLITZIP_ERR_CAPACITY;
  const hipStream_t st = static_cast<hipStream_t>(stream);

  uint32_t i = 0;
  while (i < n_items) {
    const CompressPlan p = plan_compress(items + i, n_items - i, n_max, dtype, ws.status_bytes, ws.stage_bytes, [st](uint64_t wgs) { return cus_once(st, wgs); });
    const uint32_t k = p.k;
    if (k == 0) return SPLITZIP_ERR_CAPACITY;   // cannot happen: every tensor fits alone
    TileArgs<kBatchMax> args;   // the first k items are filled in, and no other is looked at
    TileShared& a = args.shared;
    uint64_t off = 0;
    for (uint32_t q = 0; q < k; ++q) {
      const splitzip_item& it = items[i + q];
      TileItem& to = args.item[q];
      if (!d_cbs) memcpy(to.dec, it.cb->dec, 16);   // codebook_ok has shown that dec and the encode table describe the same bijection
      else memset(to.dec, 0, 16);
      to.in = static_cast<const uint8_t*>(it.d_in);
      to.out = static_cast<uint8_t*>(it.d_out);
      to.n = (uint32_t)it.n_elems;
      to.capacity = it.out_capacity;
      to.status_off = (uint32_t)off;
      const uint64_t tiles = tiles_of(chunks_of(it.n_elems), p.cpt);
      off += p.is_short ? short_status_need(tiles) : status_need(tiles);
    }
    a.sizes = d_sizes + i;
    a.d_cbs = d_cbs ? d_cbs + i : nullptr;
    a.status = ws.base + kWsHeaderBytes;
    // The tiles' slots begin behind the words of this launch: what it leaves of the status area is as good for records.  (From the
    // staging area alone a launch of 64 tensors gave a tile of four chunks 16 records, and outliers leave 27 there, so that nearly
    // all tiles were encoded twice.  us per call, BF16 with 0.66 % escapes, then and now: 64 tensors of 100 chunks 31.1 and 11.0, 64 of 1000 95.2
    // and 45.2, 48 of 2000 115 and 62, 64 of 4000 269 and 189.)
    a.stage = a.status + off;
    a.stage_cap = ((g_hooks.stage_bytes ? ws.stage_bytes : ws.status_bytes - off + ws.stage_bytes) / k) & ~(uint64_t)255u;
    a.cpt = p.cpt;
    a.tile_shift = 2u + (uint32_t)__builtin_ctz(p.cpt);
    {
      const uint64_t per_tile = p.tiles_max ? a.stage_cap / 4 / p.tiles_max : 0;
      a.slot_cap = (uint32_t)(per_tile < kSlotCapMost ? per_tile : kSlotCapMost);
    }
    a.paging = paging;
    a.finish_groups = p.finish_groups;
    a.use_group_sums = p.group_sums ? 1u : 0u;
    a.by_xcd = p.by_xcd ? 1u : 0u;
    const unsigned tiles_max = (unsigned)p.tiles_max, sums_max = (tiles_max + kSumGroup - 1) / kSumGroup;
    if (p.is_short) {
      a.tag = next_call_tag();
      a.looks = short_looks();
      if (dtype == SPLITZIP_BF16) (p.cpt == 1 ? launch_short<Bf16, 1> : launch_short<Bf16, 2>)(tiles_max, k, st, args);
      else (p.cpt == 1 ? launch_short<E5m2, 1> : launch_short<E5m2, 2>)(tiles_max, k, st, args);
    } else if (p.small) {
      if (dtype == SPLITZIP_BF16) launch_small<Bf16>(k, st, args);
      else launch_small<E5m2>(k, st, args);
    } else if (k == 1) {
      const TileArgs<1> one = {args.shared, {args.item[0]}};
      if (dtype == SPLITZIP_BF16) launch_compress<Bf16>(tiles_max, p.finish_wgs, sums_max, 1, p.is_long, p.lds_pad, st, one);
      else launch_compress<E5m2>(tiles_max, p.finish_wgs, sums_max, 1, p.is_long, p.lds_pad, st, one);
    } else if (k <= kBatchFew) {
      if (dtype == SPLITZIP_BF16) launch_compress<Bf16>(tiles_max, p.finish_wgs, sums_max, k, p.is_long, p.lds_pad, st, few(args));
      else launch_compress<E5m2>(tiles_max, p.finish_wgs, sums_max, k, p.is_long, p.lds_pad, st, few(args));
    } else {
      if (dtype == SPLITZIP_BF16) launch_compress<Bf16>(tiles_max, p.finish_wgs, sums_max, k, p.is_long, p.lds_pad, st, args);
      else launch_compress<E5m2>(tiles_max, p.finish_wgs, sums_max, k, p.is_long, p.lds_pad, st, args);
    }
    if (hipGetLastError() != hipSuccess) return SPLITZIP_ERR_HIP;
    i += k;
  }
  return SPLITZIP_OK;
}

// one tensor through compress_launch: the codebook on the host (cb) or in device memory (d_cb)
int compress_one(const Words& in, uint64_t n_elems, int dtype, const splitzip_codebook* cb, const splitzip_codebook* d_cb,
                 void* d_out, size_t out_capacity, void* d_workspace, size_t workspace_bytes, bool own_scratch,
                 splitzip_sizes* d_sizes, void* stream) {
  if (!d_sizes || (!cb && !d_cb)) return SPLITZIP_ERR_INVALID_ARG;
  splitzip_item it;
  it.d_in = in.base;
  it.n_elems = n_elems;
  it.d_out = d_out;
  it.out_capacity = out_capacity;
  it.cb = cb;
  return compress_launch(&it, 1, dtype, in, in.table ? n_elems : 0, d_cb, d_workspace, workspace_bytes, own_scratch, d_sizes, stream);
}

constexpr unsigned kDecodeLdsPad = 22800;   // five workgroups of the decoder per CU

// cpw: most_cpw at most
template <typename F, uint32_t N>
void launch_decompress(uint32_t cpw, dim3 grid, unsigned lds_pad, hipStream_t st, const DArgs<N>& args) {
  constexpr uint32_t most = most_cpw(F::DT, N > 1);
  if (cpw == 1) launch(decompress_kernel<F, 1, N>, grid, dim3(kThreads), lds_pad, st, args);
  else if (cpw == 2 || most == 2) launch(decompress_kernel<F, 2, N>, grid, dim3(kThreads), lds_pad, st, args);
  else if (cpw == 4 || most == 4) launch(decompress_kernel<F, most < 4 ? 2 : 4, N>, grid, dim3(kThreads), lds_pad, st, args);
  else launch(decompress_kernel<F, most, N>, grid, dim3(kThreads), lds_pad, st, args);
}

// how up to kBatchMax streams of a decompress call are launched, by the lengths of what they decode to
struct DecompressPlan {
  uint32_t cpw;        // chunks per wave
  uint32_t wgs;        // workgroups per stream: what the longest needs
  uint32_t by_xcd;     // they take their tiles in xcd_order
  uint32_t lds_pad;    // unused LDS asked for at the launch: fewer workgroups per CU
};
DecompressPlan plan_decompress(const splitzip_ditem* items, uint32_t k, int dtype) {
  uint64_t chunks_all = 0, chunks_max = 0, n_all = 0, beyond = 0;
  for (uint32_t q = 0; q < k; ++q) {
    const uint64_t c = chunks_of(items[q].n_elems), fixed = splitzip_fixed_bytes(items[q].n_elems, dtype);
    chunks_all += c;
    if (c > chunks_max) chunks_max = c;
    n_all += items[q].n_elems;
    if (items[q].comp_bytes > fixed) beyond += items[q].comp_bytes - fixed;
  }
  DecompressPlan p;
  const uint64_t cus = (uint64_t)cu_count();   // asks the runtime: once per call
  p.cpw = pick_decompress_cpw(chunks_all, k > 1, many_escapes(beyond, n_all), dtype, cus);
  // Streams that differ in length, as in pick_base_cpt: more chunks per wave where many of the launch's workgroups have
  // none.  Device us by chunks per wave, BF16 one / two: 4.4 / 4.0 (600 chunks beside 63 streams of 5: 9371 without a tile), 12.8
  // / 7.8 (3000 beside 63 of two), 18.2 / 14.2 (20 000 beside seven of two), two / four, where the streams are a small part of it:
  // 26.3 / 14.1 (13 000 beside 63 of two), 69.9 / 39.8 (32 768 beside 63 of two), 32.8 / 34.2 (four of 8192 beside 60 of 200:
  // 60 000), 18.4 / 18.8 (8192 beside 63 of 100); E5M2 one / two / four: 4.4 / 3.9 / 4.3 (600 beside 63 of 5: 4686), 7.7 / 6.0 / 5.9
  // (1500 beside 63 of 50: 11 418), four / eight: 14.3 / 8.9 (13 000 beside 63 of two: 51 184), 36.9 / 22.5 (32 768 beside 63 of
  // two), 14.3 / 18.7 (8192 beside 63 of 100: 31 862), 28.6 / 31.1 (two of 9000 beside 62 of 1000: 31 000).  The limits were set
  // with an earlier decoder; where they are off with this one (the last two calls of BF16, the last of E5M2) it is by 2 to 9 %.
  const uint64_t none = chunks_max * k - chunks_all;   // chunks that the padded grid has room for and the streams do not have
  if (!g_hooks.cpw.load()) {
    const uint32_t most = dtype == SPLITZIP_BF16 && none <= 8 * chunks_all ? 2u : most_cpw(dtype, k > 1);
    const auto limit = [&](uint32_t cpw) { return dtype == SPLITZIP_BF16 ? (cpw < 2 ? 32u : 224u) : cpw < 4 ? 32u : chunks_all < 256 * cus ? 160u : 96u; };
    while (p.cpw < most && none / (kWaves * p.cpw) > cus * limit(p.cpw)) p.cpw *= 2;
  }
  p.wgs = (uint32_t)((chunks_max + (uint64_t)kWaves * p.cpw - 1) / (kWaves * p.cpw));
  if (p.wgs < 1) p.wgs = 1;
  // Launches of 4096 workgroups and more take their tiles in xcd_order.  us per call, in the order of the tiles and that way: BF16
  // 21.3 and 20.9 (4096 workgroups of two chunks per wave), 21.0 and 20.6 (8192 of one: a stream of 32 768 chunks), 38.8 and 38.1 (65 536 chunks), 39.2
  // and 38.4 (64 streams of 1024), 74.0 and 72.9 (64 of 1999), 606.6 and 599.2 (262 144), but 11.8 and 12.0 (2048: one stream of 16 384 chunks); E5M2,
  // without the fewer workgroups below, 18.66 and 18.67 (6144), 23.2 and 23.1 (8192), 663 and 641 (131 072), but 13.52 and 13.56 (2048).  As in
  // plan_compress, by the workgroups that have a tile (BF16, one stream of 32 768 chunks beside 63 of two, with another
  // decoder: 97.3 and 111.1).
  uint64_t wgs_all = 0;
  const uint32_t shift = (uint32_t)__builtin_ctz(kWaves * p.cpw);
  for (uint32_t q = 0; q < k; ++q) wgs_all += (chunks_of(items[q].n_elems) + kWaves * p.cpw - 1) >> shift;
  p.by_xcd = wgs_all >= 4096u && (uint64_t)p.wgs * k <= 2 * wgs_all ? 1u : 0u;
  if (const uint32_t forced = g_hooks.xcd.load()) p.by_xcd = forced == 2 ? 1u : 0u;
  // Fewer workgroups per CU, five instead of eight, where a launch is long and its waves have much on their way.  us per call
  // with eight / six / five / four: BF16, two chunks per wave, 1240 / 1184 / 1172 / 1170 (2 Mi chunks), 300.9 / 295.5 / 292.8 /
  // 293.1 (524 288), 75.9 / 75.2 / 74.1 / 74.1 (131 072 with seven escapes each), with one chunk 1224 / 1198 / 1231 / 1231; E5M2,
  // four chunks, 648 / 637 / 619 / 632 (2 Mi), 158.8 / 157.7 / 156.7 / 158.1 (524 288), with two 635 / 638 / 678 / 751.
  // Not where a wave's records outgrow the 128 that it asks for beside its planes: it then waits for memory once more, and the
  // other workgroups of the CU are what fills that wait.  By the records per chunk, as the streams' lengths tell, with five / eight:
  // BF16 150.2 / 152.4 (262 144 chunks in 64 streams, 58 records), 156.0 / 154.9 (67), 183.8 / 161.9 (144), 141.3 / 121.7 (200 000
  // in one stream, 144), 508 / 400 (524 288, 384); E5M2 313.1 / 315.1 (1 Mi, 26), 327.9 / 317.8 (31), 366.7 / 341.8 (51), 514 /
  // 432 (205).
  const bool within = beyond * kChunk <= 3 * n_all * (dtype == SPLITZIP_BF16 ? 64u : 28u);   // three bytes per record
  // E5M2 from 16 384 workgroups on: 13.5 and 14.3 (2048 workgroups), 23.4 and 23.9 (4096), 28.98 and 28.93 (5513).
  const bool enough = dtype == SPLITZIP_BF16 ? p.cpw == 2 : p.cpw == 4 && (wgs_all >= 16384u || g_hooks.xcd.load() == 2);
  p.lds_pad = p.by_xcd && within && enough ? kDecodeLdsPad : 0u;
  return p;
}

// splitzip_decompress with the codebook either on the host (cb) or in device memory (d_cb); the words contiguous or paged
int decompress_impl(const void* d_comp, size_t comp_bytes, uint64_t n_elems, int dtype, const splitzip_codebook* cb,
                    const splitzip_codebook* d_cb, const Words& out, splitzip_sizes* d_sizes, void* stream) {
  const void* d_out = out.base;
  if (!dtype_ok(dtype) || !d_comp || (n_elems && !d_out)) return SPLITZIP_ERR_INVALID_ARG;
  if (!aligned16(d_comp) || !aligned16(d_out) || (reinterpret_cast<uintptr_t>(d_sizes) & 7u))
    return SPLITZIP_ERR_INVALID_ARG;
  if (d_cb ? (reinterpret_cast<uintptr_t>(d_cb) & 3u) != 0 : !codebook_ok(cb, dtype)) return SPLITZIP_ERR_INVALID_ARG;
  if (n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
  if (comp_bytes < splitzip_fixed_bytes(n_elems, dtype)) return SPLITZIP_ERR_CAPACITY;

  DArgs<1> args;
  DShared& a = args.shared;
  DItem& to = args.item[0];
  describe_stream(d_comp, comp_bytes, out.base, n_elems, dtype, &to);
  if (!d_cb) memcpy(to.dec, cb->dec, 16);
  else memset(to.dec, 0, 16);
  a.sizes = d_sizes;
  a.d_cbs = d_cb;   // an address in device memory, not read here
  a.paging = out;
  a.reserved[0] = a.reserved[1] = 0;
  a.own_dec = 0;
  const splitzip_ditem item = {d_comp, comp_bytes, n_elems, out.base, nullptr};
  const DecompressPlan p = plan_decompress(&item, 1, dtype);
  a.by_xcd = p.by_xcd;
  if (dtype == SPLITZIP_BF16) launch_decompress<DBf16>(p.cpw, dim3(p.wgs), p.lds_pad, static_cast<hipStream_t>(stream), args);
  else launch_decompress<DE5m2>(p.cpw, dim3(p.wgs), p.lds_pad, static_cast<hipStream_t>(stream), args);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

}  // namespace

extern "C" {

int splitzip_compress(const void* d_in, uint64_t n_elems, int dtype, const splitzip_codebook* cb,
                      void* d_out, size_t out_capacity, void* d_workspace, size_t workspace_bytes,
                      splitzip_sizes* d_sizes, void* stream) {
  return compress_one(contiguous_words(d_in), n_elems, dtype, cb, nullptr, d_out, out_capacity, d_workspace, workspace_bytes, false, d_sizes, stream);
}

uint64_t splitzip_noalloc_max_elems(void) { return 1ull << 30; }

int splitzip_compress_noalloc(const void* d_in, uint64_t n_elems, int dtype, const splitzip_codebook* cb, void* d_out,
                              size_t out_capacity, splitzip_sizes* d_sizes, void* stream) {
  if (n_elems > splitzip_noalloc_max_elems()) return SPLITZIP_ERR_UNSUPPORTED;
  return compress_one(contiguous_words(d_in), n_elems, dtype, cb, nullptr, d_out, out_capacity, nullptr, 0, true, d_sizes, stream);
}

int splitzip_decompress(const void* d_comp, size_t comp_bytes, uint64_t n_elems, int dtype,
                        const splitzip_codebook* cb, void* d_out, splitzip_sizes* d_sizes, void* stream) {
  return decompress_impl(d_comp, comp_bytes, n_elems, dtype, cb, nullptr, contiguous_words(d_out), d_sizes, stream);
}

int splitzip_codebook_device(const uint64_t* d_hist, int dtype, splitzip_codebook* d_cb, void* stream) {
  if (!dtype_ok(dtype) || !d_hist || !d_cb || (reinterpret_cast<uintptr_t>(d_hist) & 7u) || (reinterpret_cast<uintptr_t>(d_cb) & 3u))
    return SPLITZIP_ERR_INVALID_ARG;
  hipLaunchKernelGGL(codebook_kernel, dim3(1), dim3(1024), 0, static_cast<hipStream_t>(stream), d_hist, exp_values(dtype),
                     (uint32_t)dtype, d_cb);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

int splitzip_compress_paged(const splitzip_paged* src, uint64_t n_elems, int dtype, const splitzip_codebook* cb,
                            void* d_out, size_t out_capacity, void* d_workspace, size_t workspace_bytes,
                            splitzip_sizes* d_sizes, void* stream) {
  Words w;
  if (!dtype_ok(dtype) || !paged_words(src, n_elems, dtype, &w)) return SPLITZIP_ERR_INVALID_ARG;
  return compress_one(w, n_elems, dtype, cb, nullptr, d_out, out_capacity, d_workspace, workspace_bytes, false, d_sizes, stream);
}

int splitzip_decompress_paged(const void* d_comp, size_t comp_bytes, uint64_t n_elems, int dtype,
                              const splitzip_codebook* cb, const splitzip_paged* dst, splitzip_sizes* d_sizes,
                              void* stream) {
  Words w;
  if (!dtype_ok(dtype) || !paged_words(dst, n_elems, dtype, &w)) return SPLITZIP_ERR_INVALID_ARG;
  return decompress_impl(d_comp, comp_bytes, n_elems, dtype, cb, nullptr, w, d_sizes, stream);
}

int splitzip_compress_dcb(const void* d_in, uint64_t n_elems, int dtype, const splitzip_codebook* d_cb,
                          void* d_out, size_t out_capacity, void* d_workspace, size_t workspace_bytes,
                          splitzip_sizes* d_sizes, void* stream) {
  if (!d_cb) return SPLITZIP_ERR_INVALID_ARG;
  return compress_one(contiguous_words(d_in), n_elems, dtype, nullptr, d_cb, d_out, out_capacity, d_workspace, workspace_bytes, false, d_sizes, stream);
}

int splitzip_decompress_dcb(const void* d_comp, size_t comp_bytes, uint64_t n_elems, int dtype,
                            const splitzip_codebook* d_cb, void* d_out, splitzip_sizes* d_sizes, void* stream) {
  if (!d_cb) return SPLITZIP_ERR_INVALID_ARG;
  return decompress_impl(d_comp, comp_bytes, n_elems, dtype, nullptr, d_cb, contiguous_words(d_out), d_sizes, stream);
}

int splitzip_decompress_own(const void* d_comp, size_t comp_bytes, uint64_t n_elems, int dtype, void* d_out,
                            splitzip_sizes* d_sizes, void* stream) {
  if (!d_comp) return SPLITZIP_ERR_INVALID_ARG;
  // the header's 16 decode entries are where a splitzip_codebook keeps its own: the stream serves as one
  static_assert(offsetof(splitzip_codebook, dec) == 0, "dec first");
  const splitzip_codebook* own = reinterpret_cast<const splitzip_codebook*>(static_cast<const uint8_t*>(d_comp) + kHeaderDecOffset);
  return decompress_impl(d_comp, comp_bytes, n_elems, dtype, nullptr, own, contiguous_words(d_out), d_sizes, stream);
}

}  // extern "C"

namespace {

// the batch decompress calls; paging: table and page geometry shared by all items, or contiguous tensors (table null)
// d_cbs (nullable): n_items codebooks in device memory, used instead of the items' own
int decompress_batch_impl(const splitzip_ditem* items, uint32_t n_items, int dtype, const Words& paging, uint64_t paged_room,
                          const splitzip_codebook* d_cbs, bool own_dec, splitzip_sizes* d_sizes, void* stream) {
  if (!dtype_ok(dtype) || (n_items && !items) || (reinterpret_cast<uintptr_t>(d_sizes) & 7u) || (reinterpret_cast<uintptr_t>(d_cbs) & 3u))
    return SPLITZIP_ERR_INVALID_ARG;
  CallCodebooks books;
  for (uint32_t i = 0; i < n_items; ++i) {
    const splitzip_ditem& it = items[i];
    if (!it.d_comp || (it.n_elems && !it.d_out) || !aligned16(it.d_comp) || !aligned16(it.d_out) ||
        (!d_cbs && !own_dec && !books.ok(it.cb, dtype)))
      return SPLITZIP_ERR_INVALID_ARG;
    if (it.n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
    if (paging.table && it.n_elems > paged_room) return SPLITZIP_ERR_INVALID_ARG;
    if (it.comp_bytes < splitzip_fixed_bytes(it.n_elems, dtype)) return SPLITZIP_ERR_CAPACITY;
  }
  uint32_t i = 0;
  while (i < n_items) {
    DArgs<kBatchMax> args;   // the first k items are filled in, and no other is looked at
    DShared& a = args.shared;
    const uint32_t k = tensors_of_launch(items + i, n_items - i);
    for (uint32_t q = 0; q < k; ++q) {
      const splitzip_ditem& it = items[i + q];
      DItem& to = args.item[q];
      if (!d_cbs && !own_dec) memcpy(to.dec, it.cb->dec, 16);
      else memset(to.dec, 0, 16);
      describe_stream(it.d_comp, it.comp_bytes, it.d_out, it.n_elems, dtype, &to);
    }
    a.sizes = d_sizes;
    a.d_cbs = d_cbs ? d_cbs + i : nullptr;
    a.own_dec = own_dec ? 1u : 0u;
    a.paging = paging;
    const DecompressPlan p = plan_decompress(items + i, k, dtype);
    a.reserved[0] = a.reserved[1] = 0;
    a.by_xcd = p.by_xcd;
    const dim3 grid(p.wgs, k);
    const hipStream_t st = static_cast<hipStream_t>(stream);
    if (dtype == SPLITZIP_BF16) k <= kBatchFew ? launch_decompress<DBf16>(p.cpw, grid, p.lds_pad, st, few(args)) : launch_decompress<DBf16>(p.cpw, grid, p.lds_pad, st, args);
    else k <= kBatchFew ? launch_decompress<DE5m2>(p.cpw, grid, p.lds_pad, st, few(args)) : launch_decompress<DE5m2>(p.cpw, grid, p.lds_pad, st, args);
    if (hipGetLastError() != hipSuccess) return SPLITZIP_ERR_HIP;
    i += k;
  }
  return SPLITZIP_OK;
}

// workgroups that leave every thread four vectors of a sample of n words; one at least
uint64_t most_wgs(uint64_t n, int dtype) {
  const uint64_t w = (n * (dtype == SPLITZIP_BF16 ? 2 : 1) + 16 * 4096 - 1) / (16 * 4096);
  return w ? w : 1;
}
// a sample's workgroups: its share of one per CU (all: words of all samples of the launch), but no more than most_wgs
uint32_t wgs_of_sample(uint64_t n, uint64_t all, int dtype, uint64_t cus) {
  const uint64_t share = all ? cus * n / all : 0, most = most_wgs(n, dtype);
  return (uint32_t)(share > most ? most : share ? share : 1);
}
constexpr uint32_t kCalibrateAtOnce = 72;
struct CalibratePlan {
  uint32_t step;   // samples per launch
  bool at_once;    // a launch clears, counts and ranks; or clearing and ranking are launches of their own
  uint32_t launches(uint32_t n_items) const { return (n_items + step - 1) / step + (at_once ? 0 : 2); }
};
CalibratePlan plan_calibrate(const splitzip_item* items, uint32_t n_items, int dtype, uint64_t cus) {
  // Short samples go up to kHistMostShort to a launch, and others kHistMost: their workgroups are dealt out whole, and 256 CUs divide the better
  // among the fewer.
  uint64_t wgs_short = 0, all = 0;
  for (uint32_t i = 0; i < n_items; ++i) {
    wgs_short += most_wgs(items[i].n_elems, dtype);
    all += items[i].n_elems;
  }
  const bool are_short = wgs_short <= cus;
  // One launch does it all where no sample has more than kCalibrateAtOnce workgroups; more of them, all at the one word, take longer than
  // two more launches.  Device us per call with one and with three: BF16 9.73 and 10.09 (2048 chunks: 64 workgroups), 10.12 and 10.22 (2300: 72),
  // 10.90 and 10.37 (2600: 82), 12.84 and 11.12 (4096: 128), 20.6 and 13.7 (8192: 256), two of 2600 11.64 and 10.79, of 4096 14.6 and 12.2, four of 4096 (64 each) 13.6 and 13.4; E5M2 8.56 and 9.40
  // (4096: 64), 9.55 and 9.59 (5000: 79), 10.22 and 9.86 (6000: 94), 11.55 and 10.46 (8192: 128), 19.6 and 12.8 (16 384: 256).
  // And not where a call takes several launches with a codebook's tail each (100 of 1000 chunks 45.4 and 48.0).
  CalibratePlan p;
  p.at_once = are_short || n_items <= kHistMost;
  for (uint32_t i = 0; p.at_once && i < n_items; ++i) p.at_once = wgs_of_sample(items[i].n_elems, all, dtype, cus) <= kCalibrateAtOnce;
  p.step = p.at_once && are_short && n_items > kHistMost ? kHistMostShort : kHistMost;
  return p;
}
// the arguments of a calibration launch over k samples; its workgroups
template <uint32_t N>
uint32_t deal_samples(const splitzip_item* items, uint32_t k, int dtype, uint64_t cus, uint64_t tag, HistBatchArgs<N>* a) {
  uint64_t all = 0;
  for (uint32_t q = 0; q < k; ++q) all += items[q].n_elems;
  uint32_t wgs = 0;
  a->tag = tag;
  for (uint32_t q = 0; q < k; ++q) {
    const uint64_t n = items[q].n_elems;
    a->first[q] = wgs;
    a->in[q] = static_cast<const uint8_t*>(items[q].d_in);
    a->n[q] = n;
    a->start[q] = histogram_start(a->in[0], a->in[q], q, n * (dtype == SPLITZIP_BF16 ? 2 : 1) / 16);
    wgs += wgs_of_sample(n, all, dtype, cus);
  }
  for (uint32_t q = k; q <= N; ++q) a->first[q] = wgs;   // (what else there is of samples that are not there is not looked at)
  return wgs;
}
template <uint32_t N>
void launch_calibrate(const HistBatchArgs<N>& a, uint32_t wgs, int dtype, uint64_t* hists, splitzip_codebook* d_cbs, hipStream_t st) {
  if (dtype == SPLITZIP_BF16) hipLaunchKernelGGL((calibrate_batch_kernel<true, N>), dim3(wgs), dim3(1024), 0, st, a, hists, d_cbs);
  else hipLaunchKernelGGL((calibrate_batch_kernel<false, N>), dim3(wgs), dim3(1024), 0, st, a, hists, d_cbs);
}

}  // namespace

extern "C" {

int splitzip_compress_batch(const splitzip_item* items, uint32_t n_items, int dtype, void* d_workspace,
                            size_t workspace_bytes, splitzip_sizes* d_sizes, void* stream) {
  return compress_launch(items, n_items, dtype, contiguous_words(nullptr), 0, nullptr, d_workspace, workspace_bytes, false, d_sizes, stream);
}

int splitzip_decompress_batch(const splitzip_ditem* items, uint32_t n_items, int dtype, splitzip_sizes* d_sizes,
                              void* stream) {
  return decompress_batch_impl(items, n_items, dtype, contiguous_words(nullptr), 0, nullptr, false, d_sizes, stream);
}

int splitzip_calibrate_batch_device(const splitzip_item* items, uint32_t n_items, int dtype, uint64_t* d_hists,
                                    splitzip_codebook* d_cbs, void* stream) {
  if (!dtype_ok(dtype) || (n_items && (!items || !d_hists || !d_cbs)) || (reinterpret_cast<uintptr_t>(d_hists) & 7u) ||
      (reinterpret_cast<uintptr_t>(d_cbs) & 3u))
    return SPLITZIP_ERR_INVALID_ARG;
  for (uint32_t i = 0; i < n_items; ++i) {
    if ((items[i].n_elems && !items[i].d_in) || !aligned16(items[i].d_in)) return SPLITZIP_ERR_INVALID_ARG;
    if (items[i].n_elems >> 32) return SPLITZIP_ERR_UNSUPPORTED;
  }
  if (n_items == 0) return SPLITZIP_OK;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  const uint64_t cus = (uint64_t)cu_count();   // asks the runtime: once per call
  const CalibratePlan p = plan_calibrate(items, n_items, dtype, cus);
  const uint64_t tag = next_call_tag() << (kCtlTagShift - kShortTagShift) | kCtlTag;
  if (!p.at_once) hipLaunchKernelGGL(zero_words_kernel, dim3(64), dim3(256), 0, st, d_hists, 256ull * n_items);
  for (uint32_t i = 0; i < n_items; i += p.step) {
    const uint32_t k = n_items - i < p.step ? n_items - i : p.step;
    uint64_t* hists = d_hists + 256ull * i;
    if (p.step == kHistMost) {
      HistBatchArgs<kHistMost> a;
      const uint32_t wgs = deal_samples(items + i, k, dtype, cus, tag, &a);
      if (p.at_once) launch_calibrate(a, wgs, dtype, hists, d_cbs + i, st);
      else if (dtype == SPLITZIP_BF16) hipLaunchKernelGGL(histogram_batch_kernel<true>, dim3(wgs), dim3(1024), 0, st, a, hists);
      else hipLaunchKernelGGL(histogram_batch_kernel<false>, dim3(wgs), dim3(1024), 0, st, a, hists);
    } else {
      HistBatchArgs<kHistMostShort> a;
      const uint32_t wgs = deal_samples(items + i, k, dtype, cus, tag, &a);
      launch_calibrate(a, wgs, dtype, hists, d_cbs + i, st);
    }
  }
  if (!p.at_once) hipLaunchKernelGGL(codebook_kernel, dim3(n_items), dim3(1024), 0, st, d_hists, exp_values(dtype), (uint32_t)dtype, d_cbs);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

int splitzip_compress_batch_dcb(const splitzip_item* items, uint32_t n_items, int dtype, const splitzip_codebook* d_cbs,
                                void* d_workspace, size_t workspace_bytes, splitzip_sizes* d_sizes, void* stream) {
  if (n_items && !d_cbs) return SPLITZIP_ERR_INVALID_ARG;
  return compress_launch(items, n_items, dtype, contiguous_words(nullptr), 0, d_cbs, d_workspace, workspace_bytes, false, d_sizes, stream);
}

int splitzip_decompress_batch_dcb(const splitzip_ditem* items, uint32_t n_items, int dtype, const splitzip_codebook* d_cbs,
                                  splitzip_sizes* d_sizes, void* stream) {
  if (n_items && !d_cbs) return SPLITZIP_ERR_INVALID_ARG;
  return decompress_batch_impl(items, n_items, dtype, contiguous_words(nullptr), 0, d_cbs, false, d_sizes, stream);
}

int splitzip_decompress_batch_own(const splitzip_ditem* items, uint32_t n_items, int dtype, splitzip_sizes* d_sizes,
                                  void* stream) {
  return decompress_batch_impl(items, n_items, dtype, contiguous_words(nullptr), 0, nullptr, true, d_sizes, stream);
}

int splitzip_compress_batch_paged(const splitzip_item* items, uint32_t n_items, int dtype, const splitzip_paged* paging,
                                  void* d_workspace, size_t workspace_bytes, splitzip_sizes* d_sizes, void* stream) {
  Words w;
  if (!dtype_ok(dtype) || !paging_geometry(paging, dtype, &w)) return SPLITZIP_ERR_INVALID_ARG;
  return compress_launch(items, n_items, dtype, w, (uint64_t)paging->n_blocks * paging->block_elems, nullptr, d_workspace,
                        workspace_bytes, false, d_sizes, stream);
}

int splitzip_decompress_batch_paged(const splitzip_ditem* items, uint32_t n_items, int dtype, const splitzip_paged* paging,
                                    splitzip_sizes* d_sizes, void* stream) {
  Words w;
  if (!dtype_ok(dtype) || !paging_geometry(paging, dtype, &w)) return SPLITZIP_ERR_INVALID_ARG;
  return decompress_batch_impl(items, n_items, dtype, w, (uint64_t)paging->n_blocks * paging->block_elems, nullptr, false, d_sizes, stream);
}

// the plan of a call's first launch, for tests of the rules (exported, not declared in splitzip.h): only the items' n_elems are read
void splitzip_internal_compress_plan(const splitzip_item* items, uint32_t n_items, int dtype, uint32_t cus, uint32_t out[9]) {
  uint64_t n_max = 0;
  for (uint32_t q = 0; q < n_items; ++q)
    if (items[q].n_elems > n_max) n_max = items[q].n_elems;
  const uint64_t stage = splitzip_workspace_bytes(n_max, dtype) - kWsHeaderBytes - kStatusBytes;
  const CompressPlan p = plan_compress(items, n_items, n_max, dtype, kStatusBytes, stage, [](uint64_t) { return 0ull; });   // the plan under capture
  const CompressPlan o = plan_compress(items, n_items, n_max, dtype, kStatusBytes, stage, [cus](uint64_t) { return (uint64_t)cus; });   // otherwise, where a stream has so many CUs
  const uint32_t v[9] = {p.k, p.cpt, (uint32_t)p.tiles_max, p.launches(), p.by_xcd, p.finish_groups, p.group_sums, p.small, o.is_short ? o.cpt : 0u};
  memcpy(out, v, sizeof v);
}
// the launches of a calibration call on a chip of 256 CUs
uint32_t splitzip_internal_calibrate_launches(const splitzip_item* items, uint32_t n_items, int dtype) {
  return plan_calibrate(items, n_items, dtype, 256).launches(n_items);
}
// whether a workgroup of the calibration call `tag` waits at a control word
int splitzip_internal_calibrate_waits(uint64_t word, uint64_t tag) { return ctl_waits(word, tag); }
// the tile that workgroup b of a tensor of n tiles takes in a launch by XCDs
uint32_t splitzip_internal_xcd_tile(uint32_t b, uint32_t n) { return xcd_order(b, n - 1); }
// how many escapes a stream of comp_bytes bytes has room for, as the decoder is told
uint32_t splitzip_internal_stream_room(uint64_t comp_bytes, uint64_t n_elems, int dtype) {
  DItem it;
  describe_stream(nullptr, comp_bytes, nullptr, n_elems, dtype, &it);
  return it.most;
}
void splitzip_internal_decompress_plan(const splitzip_ditem* items, uint32_t n_items, int dtype, uint32_t out[4]) {
  const DecompressPlan p = plan_decompress(items, tensors_of_launch(items, n_items), dtype);
  out[0] = p.cpw; out[1] = p.wgs; out[2] = p.by_xcd; out[3] = p.lds_pad;
}

int splitzip_traffic_probe(const void* d_src, size_t read_bytes, void* d_dst, size_t write_bytes, void* stream) {
  if (!d_src || !d_dst || !aligned16(d_src) || !aligned16(d_dst) || write_bytes > read_bytes)
    return SPLITZIP_ERR_INVALID_ARG;
  const uint64_t nread = read_bytes / 16, nwrite = write_bytes / 16;
  if (!nread) return SPLITZIP_OK;
  uint64_t grid = (uint64_t)cu_count() * 8;
  const uint64_t need = (nread + 4 * kThreads - 1) / (4 * kThreads);
  if (grid > need) grid = need;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(traffic_probe_kernel, dim3((unsigned)grid), dim3(kThreads), 0, static_cast<hipStream_t>(stream),
                     static_cast<const u32x4*>(d_src), nread, static_cast<u32x4*>(d_dst), nwrite);
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}


int splitzip_traffic_probe_shape(const void* d_src, size_t read_bytes, void* d_dst, size_t write_bytes, uint32_t reads_per_step,
                                 uint32_t writes_per_step, uint32_t wgs_per_cu, uint32_t flags, void* stream) {
  if (!d_src || !d_dst || !aligned16(d_src) || !aligned16(d_dst) || wgs_per_cu > 32 || flags > 63u || (flags & 12u) == 8u || ((flags & 16u) && (flags & 12u)))
    return SPLITZIP_ERR_INVALID_ARG;
  const uint32_t R = reads_per_step, W = writes_per_step;
  const uint64_t nread = R ? read_bytes / 16 : 0, nwrite = W ? write_bytes / 16 : 0;
  const uint64_t rs = R ? (nread + (uint64_t)R * kThreads - 1) / ((uint64_t)R * kThreads) : 0;
  const uint64_t wsteps = W ? (nwrite + (uint64_t)W * kThreads - 1) / ((uint64_t)W * kThreads) : 0;
  const uint64_t steps = rs > wsteps ? rs : wsteps;
  if (!steps) return R || W ? SPLITZIP_OK : SPLITZIP_ERR_INVALID_ARG;
  uint64_t grid = wgs_per_cu ? (uint64_t)cu_count() * wgs_per_cu : steps;   // 0: one step per workgroup
  if (grid > steps) grid = steps;
  if (grid >> 31) return SPLITZIP_ERR_UNSUPPORTED;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  const u32x4* src = static_cast<const u32x4*>(d_src);
  u32x4* dst = static_cast<u32x4*>(d_dst);
  const uint32_t blocked = ((flags & 16u) ? 3u : (flags & 4u) ? ((flags & 8u) ? 2u : 1u) : 0u) | ((flags & 32u) ? 4u : 0u);
  bool found = false;
#define SPLITZIP_SHAPE(RR, WW)                                                                                              \
  if (R == RR && W == WW) {                                                                                                 \
    found = true;                                                                                                           \
    switch (flags & 3u) {                                                                                                   \
      case 0: hipLaunchKernelGGL((traffic_shape_kernel<RR, WW, false, false>), dim3((unsigned)grid), dim3(kThreads), 0, st, src, nread, dst, nwrite, steps, blocked); break; \
      case 1: hipLaunchKernelGGL((traffic_shape_kernel<RR, WW, true, false>), dim3((unsigned)grid), dim3(kThreads), 0, st, src, nread, dst, nwrite, steps, blocked); break;  \
      case 2: hipLaunchKernelGGL((traffic_shape_kernel<RR, WW, false, true>), dim3((unsigned)grid), dim3(kThreads), 0, st, src, nread, dst, nwrite, steps, blocked); break;  \
      default: hipLaunchKernelGGL((traffic_shape_kernel<RR, WW, true, true>), dim3((unsigned)grid), dim3(kThreads), 0, st, src, nread, dst, nwrite, steps, blocked); break;  \
    }                                                                                                                       \
  }
  SPLITZIP_SHAPE(1, 0) SPLITZIP_SHAPE(2, 0) SPLITZIP_SHAPE(4, 0) SPLITZIP_SHAPE(8, 0)
  SPLITZIP_SHAPE(0, 1) SPLITZIP_SHAPE(0, 2) SPLITZIP_SHAPE(0, 4) SPLITZIP_SHAPE(0, 8)
  SPLITZIP_SHAPE(4, 3) SPLITZIP_SHAPE(8, 6) SPLITZIP_SHAPE(16, 12) SPLITZIP_SHAPE(3, 4) SPLITZIP_SHAPE(6, 8) SPLITZIP_SHAPE(12, 16)
  SPLITZIP_SHAPE(1, 1) SPLITZIP_SHAPE(2, 2) SPLITZIP_SHAPE(4, 4)
#undef SPLITZIP_SHAPE
  if (!found) return SPLITZIP_ERR_INVALID_ARG;
  return hipGetLastError() == hipSuccess ? SPLITZIP_OK : SPLITZIP_ERR_HIP;
}

}  // extern "C"
