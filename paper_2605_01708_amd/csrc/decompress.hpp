// SplitZip for MI355X: the decompress kernel (dense decode of both formats, scatter correction in LDS; one stream or a batch).
// Part of the single translation unit splitzip.hip (included inside its anonymous namespace).
#ifndef SPLITZIP_DECOMPRESS_HPP
#define SPLITZIP_DECOMPRESS_HPP

// ---------------------------------------------------------------------------
// decompress
// ---------------------------------------------------------------------------

// The arguments of a launch: what all its streams share, then the streams (N: room for kBatchMax or kBatchFew of them, or for the one
// of a single call).  blockIdx.y picks the stream, blockIdx.x the tile.  What a wave needs of the layout before its first
// load comes ready: with a tile per workgroup, a scalar instruction of the beginning is one per wave.
struct DItem {
  const uint8_t* comp;
  uint8_t* out;
  uint32_t n;
  uint32_t most;           // escapes that the stream has room for, n at most
  uint32_t code256, pos256;   // where the code plane and the positions start, in units of 256 bytes
  uint8_t dec[16];         // its codebook
};
struct DShared {
  splitzip_sizes* sizes;   // nullable; one record, status bits sticky
  const splitzip_codebook* d_cbs;   // nullable: codebooks in device memory, one per stream, used instead of dec
  Words paging;            // table and page geometry shared by all tensors (table null: contiguous tensors); base unused
  uint32_t by_xcd;         // the workgroups take their tiles in xcd_order
  uint32_t own_dec;        // 1: every stream is decoded with the 16 decode entries of its own header
  uint32_t reserved[2];
};
template <uint32_t N>
struct alignas(N == 1 ? 16 : 64) DArgs {
  DShared shared;
  DItem item[N];
};
static_assert(sizeof(DShared) == 64 && sizeof(DItem) == 48, "whole 16-byte words for the copies of decompress_kernel");

// a stream of comp_bytes bytes (at least what it takes without escapes) as the kernel is told of it; dec left alone
inline void describe_stream(const void* comp, uint64_t comp_bytes, void* out, uint64_t n, int dtype, DItem* it) {
  const Layout L = make_layout(n, dtype);
  it->comp = static_cast<const uint8_t*>(comp);
  it->out = static_cast<uint8_t*>(out);
  it->n = (uint32_t)n;
  it->code256 = (uint32_t)(L.off_code >> 8);
  it->pos256 = (uint32_t)(L.off_pos >> 8);
  // the largest m with off_pos + a256(2 m) + m <= comp_bytes: 128 records take 384 bytes, in all or in part
  const uint64_t room = comp_bytes - L.off_pos, whole = room / 384, rest = room - 384 * whole;
  const uint64_t m = 128 * whole + (rest > 256 ? rest - 256 : 0);
  it->most = (uint32_t)(m < n ? m : n);
}

// header checks, by one wave of the stream's first tile: lane i < 16 holds word i of the header in hw
// dec: the 16 decode entries the caller's codebook has, four to a word; M: as the table states it
__device__ inline bool decompress_check_header(const DItem& it, uint32_t dtype, uint32_t hw, const u32x4& dec, uint32_t M, splitzip_sizes* sizes, int lane) {
  uint32_t h[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) h[i] = __builtin_amdgcn_readlane(hw, i);
  const uint64_t m = h[6] | ((uint64_t)h[7] << 32), total = h[8] | ((uint64_t)h[9] << 32);
  if (sizes && lane == 0) {
    sizes->total_bytes = total;
    sizes->n_escapes = m;
  }
  // (that total lies inside the stream follows from M <= most)
  return h[0] == 0x31505a53u && h[1] == (1u | (dtype << 16) | (4u << 24)) && h[2] == kChunk && h[3] == 0 && h[4] == it.n && h[5] == 0 &&
         m == M && M <= it.most && total == ((uint64_t)it.pos256 << 8) + a256(2 * m) + m && h[14] == 0 && h[15] == 0 &&
         h[10] == dec.x && h[11] == dec.y && h[12] == dec.z && h[13] == dec.w;   // the 16 entries, four to a word
}

// BF16: the plane words of one chunk as a wave holds them, two half-chunks of 8 elements per lane each
struct PlanesBf16 {
  u32x2 sm[2];
  uint32_t cd[2];
};
// The planes of a wave's j-th chunk, out of the runs that hold those of all its chunks (a load that reaches beyond gives
// zeros, so no load stands behind a condition, and the compiler knows how many are on their way).
__device__ inline void load_planes(__amdgpu_buffer_rsrc_t sm, __amdgpu_buffer_rsrc_t cd, int j, int lane, PlanesBf16& in) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    in.sm[h] = ld_run8(sm, 8u * (uint32_t)lane + (uint32_t)(j * kChunk + h * kHalf));
    in.cd[h] = ld_run4(cd, 4u * (uint32_t)lane + (uint32_t)(j * kChunk + h * kHalf) / 2);
  }
}
// dense decode into registers: o[4 h + d] holds elements 2 d and 2 d + 1 of the lane's group in half h
__device__ inline u32x8 decode_chunk_bf16(const PlanesBf16& in, const uint32_t* tbl) {
  u32x8 o;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t smw[2] = {in.sm[h].x, in.sm[h].y};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      // code byte b -> both exponents already in place (bits 7..14 and 23..30)
      const uint32_t cb = (in.cd[h] >> (8 * b)) & 0xffu;
      // [a0, a0, a1, a1], then keep mantissa in the low and sign in the high byte of each half-word (eq. (2))
      const uint32_t p = byte_perm(0u, smw[b >> 1], (b & 1) ? 0x03030202u : 0x01010000u);
      o[4 * h + b] = (p & 0x807f807fu) | tbl[cb];
    }
  }
  return o;
}

// E5M2: the plane words of one chunk as a wave holds them, 16 elements per lane.  Lanes 2p and 2p+1 share 12
// bytes of the 3-bit plane: the even lane loads bytes 0..7 of them, the odd lane bytes 4..11 -- the same
// instruction for every lane (no branch, no register written from two places), the overlap costs nothing.
struct PlanesE5m2 {
  u32x2 sm, cd;
};
__device__ inline void load_planes(__amdgpu_buffer_rsrc_t sm, __amdgpu_buffer_rsrc_t cd, int j, int lane, PlanesE5m2& in) {
  in.sm = ld_run8(sm, (uint32_t)(lane >> 1) * 12u + (uint32_t)(lane & 1) * 4u + (uint32_t)(j * 384));
  in.cd = ld_run8(cd, 8u * (uint32_t)lane + (uint32_t)(j * kHalf));
}
// dense decode into registers: o[d] holds elements 4 d .. 4 d + 3
__device__ inline u32x4 decode_chunk_e5m2(const PlanesE5m2& in, const uint32_t* tbl, int lane) {
  u32x4 o;
  // the lane's 48 plane bits: the even lane's start at its first byte, the odd lane's two bytes further on
  const uint32_t lo = (lane & 1) ? (in.sm.x >> 16) | (in.sm.y << 16) : in.sm.x;
  const uint32_t hi = (lane & 1) ? in.sm.y >> 16 : in.sm.y & 0xffffu;
  const uint32_t r[4] = {lo & 0xfffu, (lo >> 12) & 0xfffu, (lo >> 24) | ((hi & 0xfu) << 8), (hi >> 4) & 0xfffu};
  const uint32_t cdw[2] = {in.cd.x, in.cd.y};
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    // two code bytes -> four exponents already in place (bits 2..6 of each byte)
    const uint32_t c01 = (cdw[d >> 1] >> (16 * (d & 1))) & 0xffu, c23 = (cdw[d >> 1] >> (16 * (d & 1) + 8)) & 0xffu;
    o[d] = unpack3_e5m2(r[d]) | tbl[c01] | (tbl[c23] << 16);
  }
  return o;
}

// one dword of an LDS tile gets bits in the places of mask
__device__ inline void patch_dword(uint32_t* d, uint32_t mask, uint32_t bits) {
  __hip_atomic_fetch_and(d, ~mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  __hip_atomic_fetch_or(d, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// the two formats as seen by the decompress kernel
struct DBf16 {
  static constexpr int DT = SPLITZIP_BF16;
  static constexpr int ES = 2;   // bytes per word
  static constexpr uint32_t kSmBytes = kChunk;   // bytes of a chunk's sign+mantissa plane
  // bytes of it, CPW chunks at most, that a section of so many times 256 holds from chunk c on
  template <int CPW>
  __device__ static inline uint32_t sm_left(uint32_t section256, uint32_t c) {
    const int32_t left = (int32_t)section256 - (int32_t)(4 * c);
    return (uint32_t)(left < 0 ? 0 : left > 4 * CPW ? 4 * CPW : left) << 8;
  }
  typedef PlanesBf16 In;
  typedef u32x8 Out;
  // table entry for a code byte: both exponents in place for one dword of output
  __device__ static inline uint32_t table(int cb, const u32x4& dec) { return (dec16_at(dec, cb & 15) << 7) | (dec16_at(dec, cb >> 4) << 23); }
  __device__ static inline Out decode(const In& in, const uint32_t* tbl, int) { return decode_chunk_bf16(in, tbl); }
  __device__ static inline void store(uint8_t* cptr, int lane, Out o) {
    st_stream(reinterpret_cast<u32x4*>(cptr) + (uint32_t)lane, u32x4{o[0], o[1], o[2], o[3]});
    st_stream(reinterpret_cast<u32x4*>(cptr) + (uint32_t)(64 + lane), u32x4{o[4], o[5], o[6], o[7]});
  }
  // The chunk as an LDS tile in element order (2 KB), for chunks with escapes: registers -> tile, the
  // correction of one element by one lane, tile -> registers.
  static constexpr uint32_t kTileDwords = 512;
  __device__ static inline void to_tile(Out o, uint32_t* tile, int lane) {
    reinterpret_cast<u32x4*>(tile)[lane] = u32x4{o[0], o[1], o[2], o[3]};
    reinterpret_cast<u32x4*>(tile)[64 + lane] = u32x4{o[4], o[5], o[6], o[7]};
  }
  __device__ static inline Out from_tile(const uint32_t* tile, int lane) {
    const u32x4 a = reinterpret_cast<const u32x4*>(tile)[lane], b = reinterpret_cast<const u32x4*>(tile)[64 + lane];
    return Out{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  }
  __device__ static inline bool patch_tile(uint32_t* tile, uint32_t pos, uint32_t val) {
    const uint32_t sh = 16 * (pos & 1u);
    patch_dword(tile + (pos >> 1), 0x7f80u << sh, val << (7 + sh));
    return true;
  }
};
struct DE5m2 {
  static constexpr int DT = SPLITZIP_FP8_E5M2;
  static constexpr int ES = 1;
  static constexpr uint32_t kSmBytes = 3 * kChunk / 8;
  template <int CPW>
  __device__ static inline uint32_t sm_left(uint32_t section256, uint32_t c) {
    const int32_t left = (int32_t)(section256 << 8) - (int32_t)(384 * c);   // below 2^31: three bits per element
    // a lane's eight bytes may reach over the section's end: into the code plane behind it, not out of the run
    return (uint32_t)(left <= 0 ? 0 : left + 8 > 384 * CPW ? 384 * CPW : left + 8);
  }
  typedef PlanesE5m2 In;
  typedef u32x4 Out;
  __device__ static inline uint32_t table(int cb, const u32x4& dec) { return (dec16_at(dec, cb & 15) << 2) | (dec16_at(dec, cb >> 4) << 10); }
  __device__ static inline Out decode(const In& in, const uint32_t* tbl, int lane) { return decode_chunk_e5m2(in, tbl, lane); }
  __device__ static inline void store(uint8_t* cptr, int lane, Out o) { st_stream(reinterpret_cast<u32x4*>(cptr) + (uint32_t)lane, o); }
  static constexpr uint32_t kTileDwords = 256;
  __device__ static inline void to_tile(Out o, uint32_t* tile, int lane) { reinterpret_cast<u32x4*>(tile)[lane] = o; }
  __device__ static inline Out from_tile(const uint32_t* tile, int lane) { return reinterpret_cast<const u32x4*>(tile)[lane]; }
  __device__ static inline bool patch_tile(uint32_t* tile, uint32_t pos, uint32_t val) {
    if (val > 31u) return false;
    const uint32_t sh = 8 * (pos & 3u);
    patch_dword(tile + (pos >> 2), 0x7cu << sh, val << (2 + sh));
    return true;
  }
};

// A wave's LDS accesses are carried out in program order; this keeps the compiler from reordering accesses it takes for
// unrelated because they go through different types.
__device__ inline void lds_in_order() { asm volatile("" ::: "memory"); }

// One workgroup: a tile of 4 waves x CPW chunks of one stream.
// What bounds it: long launches the memory (64 BF16 tensors of 64 MiB 1191 us, 6.3 TB/s; 64 E5M2 tensors of 32 MiB 620 us, 6.5
// TB/s); short ones the trips to memory that a wave makes one after the other, and the instructions of its beginning.  Until
// a wave asked for everything at once -- it waited for M before its first plane, and for memory once per chunk -- they took
// 1236 and 675 us, one tensor of 64 MiB 22.1 (20.2 now), 64 of 2 MiB 42.1 (38.9), 100 chunks 3.4 (2.2).
// A wave asks for everything it can name before it waits for anything: the slice of the offset table, then the planes of
// its CPW chunks; the decode table is built meanwhile.  The table entries arrive first, and the escape records of all those
// chunks, which follow one another in the stream, are one run: two loads of it travel while the planes do.
template <typename F, int CPW, uint32_t N>
__global__ __launch_bounds__(kThreads) void decompress_kernel(const DArgs<N> args) {
  __shared__ uint32_t tbl[256];
  __shared__ __attribute__((aligned(16))) uint32_t lds_chunk[kWaves * F::kTileDwords];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  DShared b;
  DItem it;
  {
    // whole and once, as in args_arrived
    u32x4 x[4], y[3];
    __builtin_memcpy(x, &args.shared, 64);
    __builtin_memcpy(y, &args.item[blockIdx.y], 48);
    asm volatile("" : "+s"(x[0]), "+s"(x[1]), "+s"(x[2]), "+s"(x[3]), "+s"(y[0]), "+s"(y[1]), "+s"(y[2]));
    __builtin_memcpy(&b, x, 64);
    __builtin_memcpy(&it, y, 48);
  }
  const uint32_t n_chunks = (uint32_t)(((uint64_t)it.n + kChunk - 1) / kChunk);
  constexpr uint32_t kTileShift = CPW == 1 ? 2 : CPW == 2 ? 3 : CPW == 4 ? 4 : 5;
  const uint32_t n_tiles = (n_chunks + (1u << kTileShift) - 1u) >> kTileShift;
  const uint32_t tile = b.by_xcd ? xcd_order(blockIdx.x, n_tiles - 1) : blockIdx.x;
  if (tile >= (n_tiles ? n_tiles : 1u)) return;
  const uint8_t* comp = as_global(it.comp);
  Words w = item_words(b.paging, as_global(it.out));
  w.table = as_global(b.paging.table);
  splitzip_sizes* const sizes = as_global(b.sizes);
  const u32x4 dec = b.own_dec ? load_dec16(it.comp + kHeaderDecOffset) : b.d_cbs ? load_dec16(b.d_cbs[blockIdx.y].dec) : dec16_from(it.dec);

  // The stream's first wave also looks at the header: lane i holds its word i, asked for before anything else.
  const uint32_t c0 = (tile * kWaves + wave) * CPW;   // the wave's first chunk
  const bool checks = c0 == 0;
  uint32_t hw = 0;
  if (checks) hw = reinterpret_cast<const uint32_t*>(comp)[lane & 15];
  // This wave's slice of the offset table, lane c <-> its chunk c, one entry more for the end, and M as the table states
  // it (its last entry) in the lanes behind.  One load without a condition: M as a load of its own, the same for all
  // lanes, was waited for on the spot, before any of the planes had been asked for.
  const uint32_t entry = c0 + lane < n_chunks ? c0 + lane : n_chunks;
  const uint32_t my_tab = *reinterpret_cast<const uint32_t*>(comp + (kHeaderBytes + 4u * (lane <= CPW ? entry : n_chunks)));
  // the runs of both planes, up to the padded end of their sections: of no length for a wave without chunks
  const uint32_t sm256 = (kHeaderBytes + 4u * (n_chunks + 1) + 255u) >> 8;
  const auto sm = run_of(comp + ((uint64_t)sm256 << 8) + (uint64_t)c0 * F::kSmBytes, F::template sm_left<CPW>(it.code256 - sm256, c0));
  const int32_t cd_left = (int32_t)(it.pos256 - it.code256) - (int32_t)(2 * c0);
  const auto cd = run_of(comp + ((uint64_t)it.code256 << 8) + (uint64_t)c0 * (kChunk / 2), (uint32_t)(cd_left < 0 ? 0 : cd_left > 2 * CPW ? 2 * CPW : cd_left) << 8);
  typename F::In in[CPW];
#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    load_planes(sm, cd, j, lane, in[j]);
    // Chunk by chunk, where the compiler would ask for one plane of both first: a stream of 12 288 chunks 8.7 us instead of
    // 9.3.  (Launches of many rounds, mostly of several streams, are 1 to 2 % slower that way, E5M2 4 to 5 %.)
    if (F::ES == 2 && CPW == 2 && N == 1) __builtin_amdgcn_sched_barrier(0);
  }
  tbl[tid] = F::table(tid, dec);
  lds_barrier();

  const uint32_t stated = __builtin_amdgcn_readlane(my_tab, 63);   // a wave has fewer than 63 chunks
  // escapes are only trusted if their sections lie inside the stream
  const uint32_t M = stated <= it.most ? stated : 0u;
  const uint16_t* pos_arr = reinterpret_cast<const uint16_t*>(comp + ((uint64_t)it.pos256 << 8));
  const uint8_t* val_arr = reinterpret_cast<const uint8_t*>(pos_arr) + a256(2ull * stated);
  // The records of these chunks: the first 128 of the run that they are if the table is in order (it ends with M for the lanes behind).
  const uint32_t run0 = __builtin_amdgcn_readlane(my_tab, 0), run1 = __builtin_amdgcn_readlane(my_tab, CPW);
  const uint32_t run = run1 >= run0 && run1 <= M ? (run1 - run0 < 128u ? run1 - run0 : 128u) : 0u;
  uint16_t pos[2];
  uint8_t val[2];
  {
    const auto pr = run_of(reinterpret_cast<const uint8_t*>(pos_arr + run0), 2u * run), vr = run_of(val_arr + run0, run);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      pos[q] = ld_run2(pr, 2u * (uint32_t)lane + 128u * q);
      val[q] = ld_run1(vr, (uint32_t)lane + 64u * q);
    }
  }
  // paged tensor: the pool pages of the wave's chunks, lane c <-> its chunk c (entries beyond the pool are clamped where they are used)
  uint32_t my_pages = 0;
  if (w.table && n_chunks) my_pages = w.table[(c0 + lane < n_chunks ? c0 + lane : 0u) >> (w.page_shift - 10)];
  bool bad = checks && !decompress_check_header(it, F::DT, hw, dec, stated, sizes, lane);   // an inconsistent header or record

  // lane c <-> chunk c: its records, none if its entries are inconsistent; where they start in the run; how many of them the
  // run holds.  Once for all chunks: the scalar unit, which the four SIMDs share, is what short chunks keep busiest.
  const bool has = lane < CPW && c0 + lane < n_chunks;
  const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)my_tab, 0x101, 0xf, 0xf, false);   // row_shl:1, the entry behind
  const uint32_t my_left = it.n - (c0 + lane) * kChunk, my_len = my_left < kChunk ? my_left : kChunk;
  const bool valid = next >= my_tab && next - my_tab <= my_len && next <= M;
  bad = bad || (has && !valid);
  const uint32_t my_cnt = has && valid ? next - my_tab : 0u, my_at = my_tab - run0;
  const uint32_t my_here = my_at < run ? (my_cnt < run - my_at ? my_cnt : run - my_at) : 0u;
  const uint32_t n_full = it.n / kChunk;   // complete chunks
  uint8_t* const out0 = w.base + (uint64_t)F::ES * c0 * kChunk;   // (contiguous words)

#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    if (c0 + j >= n_chunks) break;
    const bool full = c0 + j < n_full;
    typename F::Out r = F::decode(in[j], tbl, lane);
    uint32_t* t = lds_chunk + (uint32_t)wave * F::kTileDwords;
    const uint32_t cnt = __builtin_amdgcn_readlane(my_cnt, j);
    if (cnt > 0) {
      // The chunk laid out in LDS, its records applied to it by a lane each, and back: every word is stored once.  (One
      // after the other in registers, which of them by its number, an escape is 22 instructions of the scalar unit.)
      const uint32_t at = __builtin_amdgcn_readlane(my_at, j), here = __builtin_amdgcn_readlane(my_here, j);
      const uint32_t clen = full ? kChunk : it.n - (c0 + j) * kChunk;
      F::to_tile(r, t, lane);
      lds_in_order();
      // a chunk's positions ascend: each must lie above the one before it
      auto apply = [&](uint32_t k, uint32_t limit, uint32_t p, uint32_t before, uint32_t v) {
        if (k < limit && (p >= clen || (k > 0 && p <= before) || !F::patch_tile(t, p, v))) bad = true;
      };
      // lane and register <-> record of the run
      apply(lane - at, here, pos[0], lane_before(pos[0], 0u), val[0]);
      if (at + here > 64) apply(64 + lane - at, here, pos[1], lane_before(pos[1], (uint32_t)__builtin_amdgcn_readlane((uint32_t)pos[0], 63)), val[1]);
      // the others, four times 64 on their way at a time
      if (here < cnt) {
        const uint32_t lo = run0 + at;
#pragma unroll 1
        for (uint32_t k0 = here; k0 < cnt; k0 += 256) {
          const auto pr = run_of(reinterpret_cast<const uint8_t*>(pos_arr + lo + k0), 2u * (cnt - k0)), vr = run_of(val_arr + lo + k0, cnt - k0);
          uint16_t p[4];
          uint8_t v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            p[q] = ld_run2(pr, 2u * (uint32_t)lane + 128u * q);
            v[q] = ld_run1(vr, (uint32_t)lane + 64u * q);
          }
          uint32_t carry = k0 ? pos_arr[lo + k0 - 1] : 0u;   // the position in front of these
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q) {
            apply(k0 + 64 * q + lane, cnt, p[q], lane_before(p[q], carry), v[q]);
            carry = (uint32_t)__builtin_amdgcn_readlane((uint32_t)p[q], 63);
          }
        }
      }
      lds_in_order();
      r = F::from_tile(t, lane);
      lds_in_order();
    }
    uint8_t* cptr = out0 + F::ES * j * kChunk;
    if (w.table) {
      uint32_t page = __builtin_amdgcn_readlane(my_pages, j);
      page = page < w.n_pages ? page : w.n_pages - 1;   // a bad table entry never leaves the pool
      cptr = chunk_at<F::ES>(w, (uint64_t)(c0 + j) * kChunk, page);
    }
    if (full) {
      F::store(cptr, lane, r);
    } else {
      // the tensor's ragged end, word by word out of the LDS tile
      const uint32_t clen = it.n - (c0 + j) * kChunk;
      F::to_tile(r, t, lane);
      lds_in_order();
#pragma unroll 1
      for (uint32_t i = lane; i < clen; i += 64) {
        if (F::ES == 2) reinterpret_cast<uint16_t*>(cptr)[i] = reinterpret_cast<const uint16_t*>(t)[i];
        else cptr[i] = reinterpret_cast<const uint8_t*>(t)[i];
      }
    }
  }
  if (bad && sizes) atomicOr(&sizes->status, SPLITZIP_STATUS_BAD_STREAM);
}

#endif  // SPLITZIP_DECOMPRESS_HPP
