// SplitZip for MI355X: the format variants of the paper's ablations (sections "Ablation on Top-k
// Exponent Coding" and "Ablation on Escape-Position Metadata", appendices "Ablation on Chunk Size"
// and "SplitZip on FP8") through one generic set of kernels.  Part of the single translation unit
// splitzip.hip (included inside its anonymous namespace).
//
// These kernels follow the structure of the tuned path: a dense pass that also counts the escapes of every chunk
// and stages the escape records of every block of 1024 elements in a slot of the workspace, and a short finishing
// pass that ranks the records and moves them to their final place (the paper's own structure, appendix "Quad64
// Vectorized Encoding", counts in the dense pass and reads the input a second time to write the records).  One set
// of templates serves all formats, the main one included, so that they can be compared with one another on equal
// terms: a block of 1024 elements per wave, eight elements per lane and step, both planes packed as LSB-first bit
// streams of 3, 4 or 8 bits in registers (a quad of lanes exchanges the bytes of a 3-bit group by DPP, so every
// global access is a whole dword).  The tuned path for the main format is compress.hpp / decompress.hpp.
#ifndef SPLITZIP_VARIANTS_HPP
#define SPLITZIP_VARIANTS_HPP

constexpr uint32_t kVBlock = 1024;   // elements a wave handles at a time
constexpr uint32_t kVStep = 512;     // ... in two steps of 8 elements per lane
constexpr uint32_t kVSlotCap = 128;  // escape records a block's slot holds (one in eight elements: a block with more is encoded again by the finishing pass)

// Per-format field arithmetic: e, a and the inverse (eq. (1) and (2); FP8 by analogy), element by element and for
// a lane's eight elements (NW dwords of words) at a time:
//   pack    the eight sign+mantissa fields, LSB first: 8 SB bits in sm (sm[1] for BF16 only)
//   unpack  their inverse, exponent fields zero
//   pair    two exponents in place, as an entry of the decode table; VPair dwords of them make the words
template <int DT>
struct VFmt;
template <>
struct VFmt<SPLITZIP_BF16> {
  static constexpr int ES = 2, SB = 8, EXPS = 256, NW = 4, LO = 7;
  __device__ static inline uint32_t exponent(uint32_t x) { return (x >> 7) & 0xffu; }
  __device__ static inline uint32_t signmant(uint32_t x) { return ((x >> 8) & 0x80u) | (x & 0x7fu); }
  __device__ static inline uint32_t combine(uint32_t a, uint32_t e) { return ((a & 0x80u) << 8) | (e << 7) | (a & 0x7fu); }
  __device__ static inline void pack(const uint32_t (&w)[4], uint32_t (&sm)[2]) {
    uint32_t t[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) t[d] = (w[d] & 0x007f007fu) | ((w[d] >> 8) & 0x00800080u);
    sm[0] = byte_perm(t[1], t[0], 0x06040200u);
    sm[1] = byte_perm(t[3], t[2], 0x06040200u);
  }
  __device__ static inline void unpack(const uint32_t (&sm)[2], uint32_t (&w)[4]) {
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] = byte_perm(0u, sm[d >> 1], (d & 1) ? 0x03030202u : 0x01010000u) & 0x807f807fu;
  }
  __device__ static inline uint32_t pair(uint32_t e0, uint32_t e1) { return (e0 << 7) | (e1 << 23); }
};
template <>
struct VFmt<SPLITZIP_FP8_E5M2> {
  static constexpr int ES = 1, SB = 3, EXPS = 32, NW = 2, LO = 2;
  __device__ static inline uint32_t exponent(uint32_t x) { return (x >> 2) & 0x1fu; }
  __device__ static inline uint32_t signmant(uint32_t x) { return ((x >> 5) & 0x4u) | (x & 0x3u); }
  __device__ static inline uint32_t combine(uint32_t a, uint32_t e) { return ((a & 0x4u) << 5) | (e << 2) | (a & 0x3u); }
  __device__ static inline void pack(const uint32_t (&w)[2], uint32_t (&sm)[2]) {
    sm[0] = pack3_e5m2(w[0]) | (pack3_e5m2(w[1]) << 12);
    sm[1] = 0;
  }
  __device__ static inline void unpack(const uint32_t (&sm)[2], uint32_t (&w)[2]) {
    w[0] = unpack3_e5m2(sm[0] & 0xfffu);
    w[1] = unpack3_e5m2((sm[0] >> 12) & 0xfffu);
  }
  __device__ static inline uint32_t pair(uint32_t e0, uint32_t e1) { return (e0 << 2) | (e1 << 10); }
};
template <>
struct VFmt<SPLITZIP_FP8_E4M3> {
  static constexpr int ES = 1, SB = 4, EXPS = 16, NW = 2, LO = 3;
  __device__ static inline uint32_t exponent(uint32_t x) { return (x >> 3) & 0xfu; }
  __device__ static inline uint32_t signmant(uint32_t x) { return ((x >> 4) & 0x8u) | (x & 0x7u); }
  __device__ static inline uint32_t combine(uint32_t a, uint32_t e) { return ((a & 0x8u) << 4) | (e << 3) | (a & 0x7u); }
  // the fields of four bytes in their low nibbles <-> 16 bits
  __device__ static inline uint32_t pack4(uint32_t w) {
    const uint32_t t = ((w >> 4) & 0x08080808u) | (w & 0x07070707u);
    const uint32_t u = t | (t >> 4);            // bytes 0 and 2 hold a pair each
    return byte_perm(0u, u, 0x0c0c0200u);
  }
  __device__ static inline uint32_t unpack4(uint32_t r) {
    const uint32_t u = byte_perm(0u, r, 0x0c010c00u);
    const uint32_t t = (u | (u << 4)) & 0x0f0f0f0fu;
    return ((t & 0x08080808u) << 4) | (t & 0x07070707u);
  }
  __device__ static inline void pack(const uint32_t (&w)[2], uint32_t (&sm)[2]) {
    sm[0] = pack4(w[0]) | (pack4(w[1]) << 16);
    sm[1] = 0;
  }
  __device__ static inline void unpack(const uint32_t (&sm)[2], uint32_t (&w)[2]) {
    w[0] = unpack4(sm[0] & 0xffffu);
    w[1] = unpack4(sm[0] >> 16);
  }
  __device__ static inline uint32_t pair(uint32_t e0, uint32_t e1) { return (e0 << 3) | (e1 << 11); }
};

__host__ __device__ inline uint32_t v_sm_bits(uint32_t dtype) { return dtype == SPLITZIP_BF16 ? 8u : dtype == SPLITZIP_FP8_E5M2 ? 3u : 4u; }
__host__ __device__ inline uint32_t v_exp_values(uint32_t dtype) { return dtype == SPLITZIP_BF16 ? 256u : dtype == SPLITZIP_FP8_E5M2 ? 32u : 16u; }
__host__ __device__ inline uint32_t v_exp_bits(uint32_t dtype) { return dtype == SPLITZIP_BF16 ? 8u : dtype == SPLITZIP_FP8_E5M2 ? 5u : 4u; }
// bytes of the value section for m escapes of vb bits each
__host__ __device__ inline uint64_t v_val_bytes(uint64_t m, uint32_t vb) { return (m * vb + 7) / 8; }
__host__ __device__ inline uint32_t v_pos_bytes(uint32_t mode, uint32_t chunk) {
  return mode == SPLITZIP_ESC_SENTINEL ? 0u : mode == SPLITZIP_ESC_ABS32 ? 4u : chunk > 256u ? 2u : 1u;
}

// what every variant kernel needs to know about a call
struct VArgs {
  const uint8_t* in;     // compress: the words; decompress: the stream
  uint8_t* out;          // compress: the stream; decompress: the words
  uint64_t capacity;     // bytes of the stream buffer (compress: room, decompress: what the caller holds)
  uint64_t n;
  uint32_t dtype, code_bits, k, mode;
  uint32_t chunk_shift;  // log2 of the chunk the counts are kept for (10 in the absolute mode: the wave's block)
  uint32_t pos_bytes;
  uint32_t val_bits;     // bits per escape value: 8, or the exponent field's own width
  uint8_t* val_stage;    // compress, val_bits < 8: workspace for the values as whole bytes, until v_pack_kernel packs them
  uint64_t n_chunks;     // of that chunk size
  uint64_t sm_bytes, code_bytes;
  uint64_t off_tab, off_sm, off_code, off_pos;
  uint32_t* counts;      // workspace: escapes per chunk
  uint32_t* offs;        // exclusive offsets, n_chunks + 1: in the stream, or in the workspace in the absolute mode
  uint32_t* wg_sums;     // workspace: escapes per workgroup of the dense pass (kWaves blocks)
  uint32_t* tile_sums;   // workspace: escapes per tile of kVScanTile chunks
  uint32_t n_tiles;
  const uint32_t* sums;  // what the finishing pass sums up: wg_sums, or tile_sums for tensors of many workgroups
  uint32_t n_sums;
  uint32_t sum_shift;    // log2 of the chunks per sum
  uint32_t ahead;        // records per block that the finishing pass fetches before it knows the counts
  uint32_t* slots;       // workspace: per block of 1024 elements kVSlotCap records, position in the block | exponent << 16

  splitzip_sizes* sizes;
  uint32_t hdr[16];      // the header of a stream of this call, words 6..9 (M, total) left 0
  uint8_t dec[16];
  uint32_t escape_code;  // the code of an escaped element: 0, or all ones in the sentinel mode
};

// The 16 decode entries of the kernel's arguments as opaque scalars: a choice between the four words by a lane's own
// index (dec16_at) must stay a choice between registers.  Left to itself the compiler turns it into one load from a
// chosen address of the argument block and makes that a scalar load, with the first lane's address for all lanes.
// (The tuned kernels choose between arguments and device memory first, which keeps the words in registers.)
__device__ inline u32x4 v_dec16(const VArgs& a) {
  u32x4 d = dec16_from(a.dec);
  uint32_t w[4] = {d.x, d.y, d.z, d.w};
  asm("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[2]), "+s"(w[3]));
  return u32x4{w[0], w[1], w[2], w[3]};
}

// The finishing pass's own copy of the arguments, those it needs fetched at once (as in args_arrived): the compiler would
// fetch each where it is used first, half a dozen trips one after the other in a kernel of a few microseconds.
__device__ inline VArgs v_args_arrived(const VArgs& args) {
  VArgs a = args;
  asm volatile("" : "+s"(a.in), "+s"(a.out), "+s"(a.capacity), "+s"(a.n), "+s"(a.k), "+s"(a.mode), "+s"(a.chunk_shift), "+s"(a.val_bits), "+s"(a.val_stage),
               "+s"(a.n_chunks), "+s"(a.off_sm), "+s"(a.off_code), "+s"(a.off_pos), "+s"(a.counts), "+s"(a.offs), "+s"(a.slots));
  asm volatile("" : "+s"(a.wg_sums), "+s"(a.sums), "+s"(a.n_sums), "+s"(a.sum_shift), "+s"(a.ahead), "+s"(a.escape_code));
  a.in = as_global(a.in);
  a.out = as_global(a.out);
  a.val_stage = as_global(a.val_stage);
  a.counts = as_global(a.counts);
  a.offs = as_global(a.offs);
  a.slots = as_global(a.slots);
  a.wg_sums = as_global(a.wg_sums);
  a.sums = as_global(a.sums);
  return a;
}

// how many of the eight elements starting at g0 exist (the valid ones are always a prefix of the group)
__device__ inline uint32_t v_nvalid(const VArgs& a, uint64_t g0) {
  return g0 >= a.n ? 0u : (a.n - g0 < 8 ? (uint32_t)(a.n - g0) : 8u);
}

// the words of a lane's eight elements from g0 on; words beyond N read as zero
template <int DT, bool FULL>
__device__ inline void v_load8(const VArgs& a, uint64_t g0, uint32_t (&w)[VFmt<DT>::NW]) {
  using F = VFmt<DT>;
  const uint32_t nv = FULL ? 8u : v_nvalid(a, g0);
  if (nv == 8) {
    if (F::ES == 2) {
      const u32x4 v = ld_stream(reinterpret_cast<const u32x4*>(a.in + 2 * g0));
      w[0] = v.x; w[1] = v.y; w[F::NW - 2] = v.z; w[F::NW - 1] = v.w;
    } else {
      const u32x2 v = ld_stream(reinterpret_cast<const u32x2*>(a.in + g0));
      w[0] = v.x; w[1] = v.y;
    }
  } else {
#pragma unroll
    for (int d = 0; d < F::NW; ++d) w[d] = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if ((uint32_t)j < nv) {
        if (F::ES == 2) w[j >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(a.in)[g0 + j] << (16 * (j & 1));
        else w[j >> 2] |= (uint32_t)a.in[g0 + j] << (8 * (j & 3));
      }
  }
}
// exponent of element j of a lane's eight
template <int DT>
__device__ inline uint32_t v_exponent_of(const uint32_t (&w)[VFmt<DT>::NW], int j) {
  using F = VFmt<DT>;
  return F::ES == 2 ? (w[j >> 1] >> (F::LO + 16 * (j & 1))) & (F::EXPS - 1) : (w[(j >> 2) & (F::NW - 1)] >> (F::LO + 8 * (j & 3))) & (F::EXPS - 1);
}

// A wave's LDS accesses are carried out in program order; this keeps the compiler from reordering
// accesses it takes for unrelated because they go through different types, and waits for the data.
__device__ inline void v_lds_settle() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Groups of eight 3-bit fields are 24 bits: a quad of lanes shares 12 bytes.  v_pack24: the dword of them that lane
// q < 3 of the quad stores (lane 3 stores none); v_unpack24: a lane's 24 bits back, dword q held by lane q < 3 of the
// quad and any value by lane 3 (bits 24..31 of the result are not defined).
__device__ inline uint32_t v_pack24(uint32_t c, uint32_t q) {
  const uint32_t next = __builtin_amdgcn_mov_dpp(c, 0xF9, 0xf, 0xf, false);   // quad_perm [1,2,3,3]
  return (c >> (8 * q)) | (next << (24 - 8 * q));
}
__device__ inline uint32_t v_unpack24(uint32_t d, uint32_t q) {
  const uint32_t prev = __builtin_amdgcn_mov_dpp(d, 0x90, 0xf, 0xf, false);   // quad_perm [0,0,1,2]
  return __builtin_amdgcn_alignbit(d, prev, 32 - 8 * q);                      // lane 0: a shift by 0 of its own dword
}

// A step's 512 fields of NB bits, one lane's eight in v: global accesses of whole dwords at byte offset off of the
// plane (off = 64 NB per step); bytes at or beyond end, the padded end of the section, are left alone.
template <int NB, bool FULL>
__device__ inline void v_store_plane(uint8_t* plane, uint64_t off, uint64_t end, uint32_t lane, const uint32_t (&v)[2]) {
  if (NB == 8) {
    if (FULL || off + 8 * lane < end) st_stream(reinterpret_cast<u32x2*>(plane + off) + lane, u32x2{v[0], v[1]});
  } else if (NB == 4) {
    if (FULL || off + 4 * lane < end) st_stream(reinterpret_cast<uint32_t*>(plane + off) + lane, v[0]);
  } else {
    const uint32_t q = lane & 3u, at = (lane >> 2) * 12 + 4 * q, d = v_pack24(v[0], q);
    if (q < 3 && (FULL || off + at < end)) st_stream(reinterpret_cast<uint32_t*>(plane + off + at), d);
  }
}
// What v_store_plane wrote, as it comes from memory; v_plane_fields makes a lane's eight fields of it.  No load stands
// behind a condition: a lane beyond the section's end reads its last bytes (last: where the last load may start).
template <int NB>
__device__ inline void v_load_plane(const uint8_t* plane, uint32_t off, uint32_t last, uint32_t lane, uint32_t (&v)[2]) {
  const uint32_t q = lane & 3u;   // of 3-bit fields lane 3 of a quad reads its neighbour's dword
  const uint32_t want = off + (NB == 8 ? 8u * lane : NB == 4 ? 4u * lane : (lane >> 2) * 12u + 4u * (q < 3 ? q : 2u)), at = want < last ? want : last;
  v[1] = 0;
  if (NB == 8) {
    const u32x2 x = ld_stream(reinterpret_cast<const u32x2*>(plane + at));
    v[0] = x.x; v[1] = x.y;
  } else {
    v[0] = ld_stream(reinterpret_cast<const uint32_t*>(plane + at));
  }
}
template <int NB>
__device__ inline void v_plane_fields(uint32_t (&v)[2], uint32_t lane) {
  if (NB == 3) v[0] = v_unpack24(v[0], lane & 3u) & 0xffffffu;
}

// Split + encode of a lane's eight elements: packed a, packed codes, and an escape mask with the codes' stride (bit
// CB j = element j).  lut: exponent -> code, | 0x10000 for an escape: shifted by CB bits per element, four entries
// add up to 4 CB bits of codes and, from bit 16 on, the flags in the same places.
template <int DT, int CB>
__device__ inline void v_encode8(const uint32_t* lut, uint32_t nv, const uint32_t (&w)[VFmt<DT>::NW], uint32_t (&sm)[2],
                                 uint32_t (&code)[2], uint32_t& esc) {
  VFmt<DT>::pack(w, sm);
  uint32_t u[2];
#pragma unroll
  for (int q = 0; q < 2; ++q)
    u[q] = lut[v_exponent_of<DT>(w, 4 * q)] + (lut[v_exponent_of<DT>(w, 4 * q + 1)] << CB) +
           ((lut[v_exponent_of<DT>(w, 4 * q + 2)] + (lut[v_exponent_of<DT>(w, 4 * q + 3)] << CB)) << (2 * CB));
  code[1] = 0;
  if (CB == 4) {
    code[0] = byte_perm(u[1], u[0], 0x05040100u);
    esc = byte_perm(u[1], u[0], 0x07060302u);
  } else {
    code[0] = (u[0] & 0xfffu) | ((u[1] & 0xfffu) << 12);
    esc = (u[0] >> 16) | ((u[1] >> 16) << 12);
  }
  if (nv < 8) {   // words beyond N were loaded as zero: their codes and escape bits go
    code[0] &= (1u << (CB * nv)) - 1u;
    esc &= (1u << (CB * nv)) - 1u;
  }
}

// wave_sparse_excl with the total of the lower 32 lanes beside that of all
__device__ inline uint32_t v_sparse_excl(uint32_t c, uint32_t& excl, uint32_t& low_total) {
  uint32_t total = 0;
  excl = 0;
  low_total = 0;
  for (uint32_t k = 1;; ++k) {
    const uint64_t m = __ballot(c >= k);
    if (!m) break;
    excl = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, excl));
    total += (uint32_t)__popcll(m);
    low_total += (uint32_t)__popc((uint32_t)m);
  }
  return total;
}

// the encode table of v_encode8, by the first wave of the workgroup: escapes everywhere, the k codes on top
__device__ inline void v_build_encode_table(const VArgs& a, uint32_t* lut, uint32_t tid) {
  if (tid < 64) {
#pragma unroll
    for (int q = 0; q < 4; ++q) lut[q * 64 + tid] = 0x10000u | a.escape_code;
    const uint32_t e = dec16_at(v_dec16(a), tid & 15u);
    if (tid < a.k) lut[e] = tid;
  }
}

// The positions of the block's first `cap` escapes into s_pos, its words into s_words.  (The steps' arrays one by one: out
// of a struct the dense pass's code came another way, 26.6 us instead of 26.5 for 64 MiB.)
template <int DT, int CB>
__device__ inline void v_stage_block(uint32_t* s_words, uint16_t* s_pos, uint32_t cap, uint32_t lane, const uint32_t (&w)[2][VFmt<DT>::NW],
                                     const uint32_t (&esc)[2], const uint32_t (&excl)[2], const uint32_t (&tot)[2]) {
  using F = VFmt<DT>;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    // the lane's words in its own bytes of the block's LDS copy
    if (F::ES == 2) reinterpret_cast<u32x4*>(s_words)[s * 64 + lane] = u32x4{w[s][0], w[s][1], w[s][F::NW - 2], w[s][F::NW - 1]};
    else reinterpret_cast<u32x2*>(s_words)[s * 64 + lane] = u32x2{w[s][0], w[s][1]};
    uint32_t m = esc[s], r = (s ? tot[0] : 0u) + excl[s];
    while (m) {
      const uint32_t bit = (uint32_t)__ffs(m) - 1u, j = CB == 4 ? bit >> 2 : (bit * 11u) >> 5;   // bit / CB
      m &= m - 1;
      if (r < cap) s_pos[r] = (uint16_t)(s * kVStep + lane * 8 + j);
      ++r;
    }
  }
  v_lds_settle();
}
// One block of 1024 elements by one wave, its words in w: planes out, the positions of its first `cap` escapes in s_pos, its words in
// s_words if it has any.  tot: the escapes of its two steps, low: those of the lower 32 lanes.
template <int DT, int CB, bool FULL>
__device__ inline uint32_t v_encode_block(const VArgs& a, const uint32_t* lut, uint32_t* s_words, uint16_t* s_pos, uint32_t cap, uint64_t blk,
                                          uint32_t lane, const uint32_t (&w)[2][VFmt<DT>::NW], uint32_t (&tot)[2], uint32_t (&low)[2]) {
  using F = VFmt<DT>;
  const uint64_t sm_end = a256(a.sm_bytes), code_end = a256(a.code_bytes);
  uint32_t esc[2], excl[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const uint64_t g = blk * kVBlock + s * kVStep;
    uint32_t sm[2], code[2];
    v_encode8<DT, CB>(lut, FULL ? 8u : v_nvalid(a, g + lane * 8), w[s], sm, code, esc[s]);
    v_store_plane<F::SB, FULL>(a.out + a.off_sm, g / 8 * F::SB, sm_end, lane, sm);
    v_store_plane<CB, FULL>(a.out + a.off_code, g / 8 * CB, code_end, lane, code);
    tot[s] = v_sparse_excl(__popc(esc[s]), excl[s], low[s]);
  }
  const uint32_t total = tot[0] + tot[1];
  if (total) v_stage_block<DT, CB>(s_words, s_pos, cap, lane, w, esc, excl, tot);
  return total;
}
// exponent of the block's element p, out of its words
template <int DT>
__device__ inline uint32_t v_staged_exponent(const uint32_t* s_words, uint32_t p) {
  using F = VFmt<DT>;
  return F::exponent(F::ES == 2 ? (uint32_t)reinterpret_cast<const uint16_t*>(s_words)[p] : (uint32_t)reinterpret_cast<const uint8_t*>(s_words)[p]);
}

// The same for the dense pass: the escape counts of its chunks, its escape
// records (position in the block | exponent << 16, in element order) into its slot.  Returns the block's count.
// The positions are ranked and collected in LDS first; the records then leave 64 at a time (with 6 % escapes a
// block has 60, and a store per element and lane was half of the kernel's time).
template <int DT, int CB, bool FULL>
__device__ inline uint32_t v_dense_block(const VArgs& a, const uint32_t* lut, uint32_t* s_words, uint16_t* s_pos, uint64_t blk,
                                         uint32_t lane, const uint32_t (&w)[2][VFmt<DT>::NW]) {
  uint32_t tot[2], low[2];
  const uint32_t total = v_encode_block<DT, CB, FULL>(a, lut, s_words, s_pos, kVSlotCap, blk, lane, w, tot, low);
  if (total) {
    uint32_t* slot = a.slots + blk * kVSlotCap;
    for (uint32_t i = lane; i < (total < kVSlotCap ? total : kVSlotCap); i += 64) {
      const uint32_t p = s_pos[i];
      slot[i] = p | (v_staged_exponent<DT>(s_words, p) << 16);
    }
  }
  if (a.chunk_shift == 10) {
    if (lane == 0) a.counts[blk] = total;
  } else if (lane < 4) {   // two 256-element chunks per step
    const uint64_t c = blk * 4 + lane;
    const uint32_t s_low = lane < 2 ? low[0] : low[1], s_tot = lane < 2 ? tot[0] : tot[1];
    if (c < a.n_chunks) a.counts[c] = lane & 1u ? s_tot - s_low : s_low;
  }
  return total;
}

// Compress pass 1: both planes, the escape count of every chunk and of every workgroup, the escape records.
// Bound by memory like the tuned dense pass: one 64 MiB BF16 tensor takes 24.0 us under 3-bit codes (29.8 us with the
// planes staged through LDS in two dependent steps and a store per escape and lane) and 21.5 us in the main format.
template <int DT, int CB>
__global__ __launch_bounds__(kThreads) void v_dense_kernel(const VArgs a) {
  using F = VFmt<DT>;
  __shared__ uint32_t lut[256];
  __shared__ __attribute__((aligned(16))) uint32_t s_words[kWaves][kVBlock * F::ES / 4];
  __shared__ uint16_t s_pos[kWaves][kVSlotCap];
  __shared__ uint32_t s_cnt[kWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint64_t blk = (uint64_t)blockIdx.x * kWaves + wave;
  const bool live = blk * kVBlock < a.n, full = (blk + 1) * kVBlock <= a.n;
  uint32_t w[2][F::NW], cnt = 0;
  // the block's words first, all of them: the table is built while they are on their way
  if (full) {
#pragma unroll
    for (int s = 0; s < 2; ++s) v_load8<DT, true>(a, blk * kVBlock + s * kVStep + lane * 8, w[s]);
    v_build_encode_table(a, lut, tid);
    lds_barrier();
    cnt = v_dense_block<DT, CB, true>(a, lut, s_words[wave], s_pos[wave], blk, lane, w);
  } else {
    if (live) {
#pragma unroll
      for (int s = 0; s < 2; ++s) v_load8<DT, false>(a, blk * kVBlock + s * kVStep + lane * 8, w[s]);
    }
    v_build_encode_table(a, lut, tid);
    lds_barrier();
    if (live) cnt = v_dense_block<DT, CB, false>(a, lut, s_words[wave], s_pos[wave], blk, lane, w);
  }
  if (lane == 0) s_cnt[wave] = cnt;
  lds_barrier();
  if (tid == 0) {
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) sum += s_cnt[q];
    a.wg_sums[blockIdx.x] = sum;
  }
  // the finishing pass reads whole vectors of four sums
  if (blockIdx.x == gridDim.x - 1 && tid > 0 && tid < 4 && (blockIdx.x & 3u) + tid < 4) a.wg_sums[blockIdx.x + tid] = 0;
}

constexpr uint32_t kVScanTile = 1024;   // counts per workgroup of the summing kernel

// compress pass 2, for tensors of more than kVDirectSums workgroups: the escapes of every tile of 1024 chunks
__global__ __launch_bounds__(1024) void v_tile_sum_kernel(const VArgs a) {
  __shared__ uint32_t s_wave[16];
  const uint64_t c = (uint64_t)blockIdx.x * kVScanTile + threadIdx.x;
  const uint32_t sum = wave_last(wave_incl_scan(c < a.n_chunks ? a.counts[c] : 0u));
  if ((threadIdx.x & 63u) == 0) s_wave[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t all = 0;
#pragma unroll
    for (uint32_t w = 0; w < 16; ++w) all += s_wave[w];
    a.tile_sums[blockIdx.x] = all;
  }
  // the finishing pass reads whole vectors of four sums
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x > 0 && threadIdx.x < 4 && (blockIdx.x & 3u) + threadIdx.x < 4) a.tile_sums[blockIdx.x + threadIdx.x] = 0;
}

constexpr uint32_t kVFinishBlocks = 32;   // blocks of 1024 elements per workgroup of the finishing pass
// Up to this many workgroups of the dense pass (64 Mi elements) the finishing pass sums their counts itself; beyond
// that its workgroups would together read more than 128 MB of them, and it is given sums of kVScanTile chunks.
constexpr uint32_t kVDirectSums = 16384;

constexpr int kVAnyPos = -1;
// where the records of a stream go: positions of PB bytes (none in the sentinel mode; kVAnyPos: as the call says), and exponents, as bytes of the
// stream or, if values are narrower than a byte, of the workspace (v_pack_kernel); the rooms are in records
template <int PB>
struct VSink {
  uint8_t* pos;
  uint8_t* val;
  uint32_t pos_room, val_room;
  uint32_t pos_mask;   // of the element index: relative to the chunk, or (absolute mode) all of it
  uint32_t pb;
  __device__ inline VSink(const VArgs& a, uint32_t M) {
    pb = PB == kVAnyPos ? a.pos_bytes : PB;
    const uint64_t off_val = a.off_pos + a256((uint64_t)pb * M);
    pos = a.out + a.off_pos;
    pos_room = pb == 0 ? 0 : room32(a.capacity, a.off_pos, pb == 4 ? 2 : pb == 2 ? 1 : 0);
    val = a.val_bits == 8 ? a.out + off_val : a.val_stage;
    val_room = a.val_bits != 8 ? ~0u : room32(a.capacity, off_val, 0);
    pos_mask = pb == 4 ? ~0u : (1u << a.chunk_shift) - 1u;
  }
  __device__ inline void put(uint32_t rank, uint32_t elem, uint32_t e) const {
    const uint32_t p = elem & pos_mask;
    if (pb != 0 && rank < pos_room) {
      if (pb == 1) pos[rank] = (uint8_t)p;
      if (pb == 2) reinterpret_cast<uint16_t*>(pos)[rank] = (uint16_t)p;
      if (pb == 4) reinterpret_cast<uint32_t*>(pos)[rank] = p;
    }
    if (rank < val_room) val[rank] = (uint8_t)e;
  }
};

// The header, the sizes record, the table's last entry and the zero padding, by one workgroup, once M is known.
__device__ inline void v_write_trailer(const VArgs& a, const uint32_t (&hdr)[16], uint32_t M, uint32_t tid) {
  const uint64_t n_blocks = (a.n + kVBlock - 1) / kVBlock;
  if (tid == 0) a.offs[a.n_chunks] = M;   // the table's last entry; in the absolute mode a word of the workspace, for v_pack_kernel
  const uint64_t pos_sec = a256((uint64_t)a.pos_bytes * M), total = a.off_pos + pos_sec + v_val_bytes(M, a.val_bits);
  // zero padding: behind the table, behind what the dense pass covered of each plane, behind the positions
  const uint64_t tab_end = a.mode == SPLITZIP_ESC_ABS32 ? kHeaderBytes : a.off_tab + 4 * (a.n_chunks + 1);
  for (uint64_t i = tab_end + tid; i < a.off_sm; i += kThreads) a.out[i] = 0;
  const uint64_t sm_cov = n_blocks * (kVBlock / 8) * v_sm_bits(a.dtype), code_cov = n_blocks * (kVBlock / 8) * a.code_bits;
  for (uint64_t i = sm_cov + tid; i < a256(a.sm_bytes); i += kThreads) a.out[a.off_sm + i] = 0;
  for (uint64_t i = code_cov + tid; i < a256(a.code_bytes); i += kThreads) a.out[a.off_code + i] = 0;
  for (uint64_t i = (uint64_t)a.pos_bytes * M + tid; i < pos_sec; i += kThreads)
    if (a.off_pos + i < a.capacity) a.out[a.off_pos + i] = 0;
  if (tid < 16) {
    uint32_t w = hdr[tid];
    if (tid == 6) w = M;
    if (tid == 8) w = (uint32_t)total;
    if (tid == 9) w = (uint32_t)(total >> 32);
    reinterpret_cast<uint32_t*>(a.out)[tid] = w;
  }
  if (tid == 0) {
    a.sizes->total_bytes = total;
    a.sizes->n_escapes = M;
    a.sizes->status = total > a.capacity ? SPLITZIP_STATUS_OVERFLOW : 0u;
    a.sizes->reserved = 0;
  }
}

// Compress pass 3: one workgroup per kVFinishBlocks blocks.  It sums the counts (the whole tensor's: M; those before
// its blocks: its first rank), writes its chunks' entries of the offset table, and moves its blocks' records from
// their slots to their ranks, a wave per block and eight blocks per wave: nothing but trips to memory, so the arguments, the
// counts of the wave's blocks, the first a.ahead records of every block and the sums are asked for at once; the others as
// soon as the wave's own counts are there, all before the one barrier.
// A block with more records than its slot holds is encoded once more from the words.  (For the two million records of a
// 64 MiB tensor under a top-8 codebook 9.2 us when the counts went through LDS and every load stood behind a condition --
// each was waited for before the next was asked for -- and 7.0 now; 6.4 and 5.3 with 0.1 % escapes.)
// Workgroup 0 also writes the header, the sizes record and the zero padding.
template <int DT, int PB>
__global__ __launch_bounds__(kThreads) void v_finish_kernel(const VArgs args) {
  using F = VFmt<DT>;
  const VArgs a = v_args_arrived(args);
  constexpr uint32_t kPerWave = kVFinishBlocks / kWaves;
  __shared__ uint32_t lut[256];
  __shared__ uint32_t s_part[3][kWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63, g = blockIdx.x;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t cpb_shift = 10u - a.chunk_shift;   // log2 of the chunks per block: 0 or 2
  const uint32_t n_blocks = (uint32_t)((a.n + kVBlock - 1) / kVBlock);
  const uint32_t blk0 = g * kVFinishBlocks + wave * kPerWave;   // the wave's first block
  const uint32_t blocks_here = n_blocks > blk0 ? (n_blocks - blk0 < kPerWave ? n_blocks - blk0 : kPerWave) : 0;
  const uint64_t c0 = (uint64_t)g * kVFinishBlocks << cpb_shift;   // the group's first chunk
  // Every load is one of a bounded run, at an offset beyond its end where a lane wants none: behind conditions, the first
  // use of each was waited for before the next was asked for.
  constexpr uint32_t kNone = 0xfffffff0u;
  // the wave's chunks, one per lane (8 or 32 of them), then the first records of its blocks
  const uint64_t my_c = ((uint64_t)blk0 << cpb_shift) + lane;
  const bool have = lane < (kPerWave << cpb_shift) && my_c < a.n_chunks;
  const uint32_t mine = ld_run4<0>(run_of(reinterpret_cast<const uint8_t*>(a.counts), 4u * (uint32_t)a.n_chunks), have ? 4u * (uint32_t)my_c : kNone);
  uint32_t rec[kPerWave], rec2[kPerWave] = {};
  const uint32_t* const slots = a.slots + (uint64_t)blk0 * kVSlotCap;
  const auto slot_run = run_of(reinterpret_cast<const uint8_t*>(slots), 4u * kVSlotCap * blocks_here);
  const uint32_t first_off = lane < a.ahead ? 4u * lane : kNone;
#pragma unroll
  for (uint32_t q = 0; q < kPerWave; ++q) rec[q] = ld_run4<0>(slot_run, first_off == kNone ? kNone : first_off + 4u * kVSlotCap * q);
  // escapes before the group's first chunk and in the whole tensor: by the sums that lie before it entirely, the rest by chunk
  uint32_t before = 0, all = 0;
  const uint64_t whole = c0 >> a.sum_shift;
  // 16-byte aligned; what the last vector holds behind the sums is zero
  const uint32_t nvec = (a.n_sums + 3) / 4, v_first = (uint32_t)(whole / 4);
  const auto sum_run = run_of(reinterpret_cast<const uint8_t*>(a.sums), 16u * nvec);
  u32x4 v[4];
  auto fetch = [&](uint32_t v0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = ld_run16<0>(sum_run, 16u * (v0 + q * kThreads + tid));
    }
  };
  fetch(0);
  v_build_encode_table(a, lut, tid);
  // what the wave's chunks hold before each lane's, and with it where each of its blocks starts: the rest of their records
  // is asked for at once as well (top-8: a block in three has more than 64)
  const uint32_t incl = wave_incl_scan(mine), wave_total = wave_last(incl), my_excl = incl - mine;
  auto starts = [&](uint32_t q) { return q < kPerWave ? (uint32_t)__builtin_amdgcn_readlane(my_excl, q << cpb_shift) : wave_total; };
  uint32_t bp[kPerWave + 1];   // wave-uniform: escapes of the wave's blocks before each block
#pragma unroll
  for (uint32_t q = 0; q <= kPerWave; ++q) bp[q] = starts(q);
  // (none, as a rule, where a codebook of 16 leaves one or two per block: 13 000 blocks 15.1 us a call, 14.7 without these loads)
  if (a.ahead >= 64u || wave_total > a.ahead) {
#pragma unroll
    for (uint32_t q = 0; q < kPerWave; ++q) {
      const uint32_t n_b = bp[q + 1] - bp[q], i = a.ahead + lane;
      rec2[q] = ld_run4<0>(slot_run, n_b <= kVSlotCap && i < n_b ? 4u * (kVSlotCap * q + i) : kNone);
    }
  }
  for (uint32_t v0 = 0;;) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t sum = v[q].x + v[q].y + v[q].z + v[q].w;
      all += sum;
      before += v0 + q * kThreads + tid < v_first ? sum : 0u;
    }
    v0 += 4 * kThreads;
    if (v0 >= nvec) break;
    fetch(v0);
  }
  if (tid < (whole & 3u)) before += a.sums[4 * v_first + tid];   // sums of the vector that the group starts in
  for (uint64_t c = (whole << a.sum_shift) + tid; c < c0 && c < a.n_chunks; c += kThreads) before += a.counts[c];
  before = wave_last(wave_incl_scan(before));
  all = wave_last(wave_incl_scan(all));
  if (lane == 63) {
    s_part[0][wave] = wave_total;
    s_part[1][wave] = before;
    s_part[2][wave] = all;
  }
  __syncthreads();
  uint32_t first = 0, M = 0;   // the rank of the wave's first record; all records of the tensor
#pragma unroll
  for (uint32_t w = 0; w < kWaves; ++w) {
    first += s_part[1][w] + (w < wave ? s_part[0][w] : 0u);
    M += s_part[2][w];
  }
  first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
  M = (uint32_t)__builtin_amdgcn_readfirstlane((int)M);
  if (have && a.mode != SPLITZIP_ESC_ABS32) a.offs[my_c] = first + my_excl;
  const VSink<PB> sink(a, M);

  const uint32_t elem0 = blk0 * kVBlock;   // fewer than 2^32 elements
  uint32_t many = 0;   // a block with more records than the two fetches took, or more than its slot holds
#pragma unroll
  for (uint32_t q = 0; q < kPerWave; ++q) {
    const uint32_t n_b = bp[q + 1] - bp[q];
    if (n_b <= kVSlotCap) {
      if (lane < a.ahead && lane < n_b) sink.put(first + bp[q] + lane, elem0 + q * kVBlock + (rec[q] & 0xffffu), rec[q] >> 16);
      if (a.ahead + lane < n_b) sink.put(first + bp[q] + a.ahead + lane, elem0 + q * kVBlock + (rec2[q] & 0xffffu), rec2[q] >> 16);
    }
    many |= n_b > a.ahead + 64 ? 1u : 0u;
  }
  if (many) {
#pragma unroll 1
    for (uint32_t q = 0; q < kPerWave; ++q) {
      const uint32_t from = starts(q), n_b = starts(q + 1) - from;
      if (n_b > kVSlotCap) continue;
#pragma unroll 1
      for (uint32_t i = a.ahead + 64 + lane; i < n_b; i += 64) {
        const uint32_t r = slots[q * kVSlotCap + i];
        sink.put(first + from + i, elem0 + q * kVBlock + (r & 0xffffu), r >> 16);
      }
    }
    // blocks whose records did not fit their slots
#pragma unroll 1
    for (uint32_t q = 0; q < blocks_here; ++q) {
      const uint32_t from = starts(q);
      if (starts(q + 1) - from <= kVSlotCap) continue;
      uint32_t rank = first + from;
#pragma unroll 1
      for (uint32_t s = 0; s < 2; ++s) {
        const uint64_t g0 = (uint64_t)(blk0 + q) * kVBlock + s * kVStep + lane * 8;
        uint32_t w[F::NW];
        v_load8<DT, false>(a, g0, w);
        uint32_t esc = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) esc |= (lut[v_exponent_of<DT>(w, j)] >> 16) << j;
        esc &= (1u << v_nvalid(a, g0)) - 1u;
        const uint32_t cnt = __popc(esc), sc = wave_incl_scan(cnt);
        uint32_t r = rank + sc - cnt;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (!((esc >> j) & 1u)) continue;
          sink.put(r, (uint32_t)g0 + j, v_exponent_of<DT>(w, j));
          ++r;
        }
        rank += __builtin_amdgcn_readlane(sc, 63);
      }
    }
  }
  if (g == 0) v_write_trailer(a, args.hdr, M, tid);
}

// Short calls (splitzip_variant_compress): the passes above in one launch, as in compress_short_kernel, a block per wave or two.
// short_words: where the workgroups' words lie (the blocks' slots, which nothing is staged in here); tag, looks: as there; tiles: the
// launch's workgroups (asked for as gridDim, a launch has 256 bytes more of arguments).
// us per call, two launches and this: BF16 top-8 7.8 and 4.4 (4 blocks), 8.0 and 5.1 (100), 8.2 and 5.3 (1000), sentinels 7.8 and 4.3, 8.1 and 5.1
// (100); E5M2 7.8 and 4.4, 7.9 and 5.1; with the planes stored and the records staged before the count is told, BF16 top-8 5.5 (100), 6.1
// (1000).  Narrow values are still packed by v_pack_kernel.  Up to 256 workgroups, as in pick_short: on 1 / 2 / 3 / 4 streams side by side 2000 blocks in
// two launches, with a block per wave and this way, with two, BF16 top-8 8.7 / 4.8 / 3.6 / 2.9, 6.2 / 3.5 / 3.2 / 5.2, 8.3 / 4.3 / 3.2 / 2.5, sentinels 7.7 / 4.1 / 3.1 / 2.6, 5.3 / 3.1 /
// 2.7 / 2.9, 6.2 / 3.4 / 2.6 / 2.1.
struct VShortArgs {
  VArgs a;
  uint64_t* short_words;
  uint64_t tag;
  uint32_t looks, tiles;
};
// BPW: blocks per wave.
template <int DT, int CB, int BPW>
__global__ __launch_bounds__(kThreads, BPW == 1 ? 1 : 4) void v_short_kernel(const VShortArgs args) {
  using F = VFmt<DT>;
  static_assert(kThreads == kTileThreads, "ShortCounts");
  __shared__ uint32_t lut[256];
  __shared__ __attribute__((aligned(16))) uint32_t s_words[kWaves][BPW][kVBlock * F::ES / 4];
  __shared__ uint16_t s_pos[kWaves][BPW][kVBlock];   // room for all of a wave's records
  __shared__ uint32_t s_cnt[kWaves];
  __shared__ ShortShared s_short;
  const VArgs a = v_args_arrived(args.a);
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  ShortCounts counts(args.short_words, args.tag, args.tiles, blockIdx.x);
  uint32_t blk = 0, count[BPW];                  // the wave's first block, the escapes of its blocks
  bool live[BPW], full[BPW];
  uint32_t w[BPW][2][F::NW];
  uint32_t sm[BPW][2][2], code[BPW][2][2], esc[BPW][2], excl[BPW][2], tot[BPW][2], low[BPW][2];   // of the blocks' steps
  uint32_t in_tile = 0, total = 0;               // escapes of the tile before the wave's blocks; all of them
  auto encode = [&](uint32_t tile, bool build) {
    blk = (tile * kWaves + wave) * BPW;
    // the blocks' words first, all of them: the table is built while they are on their way
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      const uint64_t e0 = (uint64_t)(blk + b) * kVBlock;
      live[b] = e0 < a.n, full[b] = e0 + kVBlock <= a.n;
      if (full[b]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) v_load8<DT, true>(a, e0 + s * kVStep + lane * 8, w[b][s]);
      } else if (live[b]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) v_load8<DT, false>(a, e0 + s * kVStep + lane * 8, w[b][s]);
      }
    }
    if (build) {
      v_build_encode_table(args.a, lut, tid);
      lds_barrier();
    }
    uint32_t mine = 0;
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      count[b] = tot[b][0] = tot[b][1] = low[b][0] = low[b][1] = 0;
      if (live[b]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          v_encode8<DT, CB>(lut, full[b] ? 8u : v_nvalid(a, (uint64_t)(blk + b) * kVBlock + s * kVStep + lane * 8), w[b][s], sm[b][s], code[b][s], esc[b][s]);
          tot[b][s] = v_sparse_excl(__popc(esc[b][s]), excl[b][s], low[b][s]);
        }
        count[b] = tot[b][0] + tot[b][1];
        mine += count[b];
      }
    }
    if (lane == 0) s_cnt[wave] = mine;
    lds_barrier();
    in_tile = total = 0;
#pragma unroll
    for (uint32_t q = 0; q < kWaves; ++q) {
      const uint32_t x = s_cnt[q];
      in_tile += q < wave ? x : 0u;
      total += x;
    }
  };
  auto deliver = [&] {
    const uint64_t sm_end = a256(a.sm_bytes), code_end = a256(a.code_bytes);
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint64_t step = ((uint64_t)(blk + b) * kVBlock + s * kVStep) / 8, sm_at = step * F::SB, code_at = step * CB;
        if (full[b]) {
          v_store_plane<F::SB, true>(a.out + a.off_sm, sm_at, sm_end, lane, sm[b][s]);
          v_store_plane<CB, true>(a.out + a.off_code, code_at, code_end, lane, code[b][s]);
        } else if (live[b]) {
          v_store_plane<F::SB, false>(a.out + a.off_sm, sm_at, sm_end, lane, sm[b][s]);
          v_store_plane<CB, false>(a.out + a.off_code, code_at, code_end, lane, code[b][s]);
        }
      }
      if (count[b]) v_stage_block<DT, CB>(s_words[wave][b], s_pos[wave][b], kVBlock, lane, w[b], esc[b], excl[b], tot[b]);
    }
  };
  auto place = [&](uint32_t tile) {
    const VSink<kVAnyPos> sink(a, counts.M);
    uint32_t base = counts.first + in_tile;
    const uint32_t cpb_shift = 10u - a.chunk_shift;   // log2 of the chunks per block: 0 or 2
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      const uint64_t c = ((uint64_t)(blk + b) << cpb_shift) + lane;
      if (a.mode != SPLITZIP_ESC_ABS32 && lane < (1u << cpb_shift) && c < a.n_chunks)
        a.offs[c] = base + (lane == 0 ? 0u : lane == 1 ? low[b][0] : lane == 2 ? tot[b][0] : tot[b][0] + low[b][1]);
      for (uint32_t i = lane; i < count[b]; i += 64) {
        const uint32_t p = s_pos[wave][b][i];
        sink.put(base + i, (blk + b) * kVBlock + p, v_staged_exponent<DT>(s_words[wave][b], p));
      }
      base += count[b];
    }
    if (tile == 0) v_write_trailer(a, args.a.hdr, counts.M, tid);
  };
  counts.run(s_short, args.looks, total, tid, wave, encode, deliver, place);
}

// compress pass 4, for values narrower than a byte: the value section as an LSB-first bit stream of val_bits per
// value, from the whole-byte values of the workspace.  Every thread makes whole bytes of the section from the
// values that overlap them, so no two threads write the same byte.
__global__ __launch_bounds__(kThreads) void v_pack_kernel(const VArgs a) {
  const uint32_t M = a.offs[a.n_chunks], vb = a.val_bits;
  const uint64_t off_val = a.off_pos + a256((uint64_t)a.pos_bytes * M), bytes = v_val_bytes(M, vb);
  for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < bytes; b += (uint64_t)gridDim.x * kThreads) {
    uint32_t byte = 0;
    for (uint64_t r = 8 * b / vb; r < M && r * vb < 8 * b + 8; ++r) {
      const int64_t shift = (int64_t)(r * vb) - (int64_t)(8 * b);   // where value r starts, relative to this byte
      const uint32_t v = a.val_stage[r];
      byte |= shift >= 0 ? v << shift : v >> -shift;
    }
    if (off_val + b < a.capacity) a.out[off_val + b] = (uint8_t)byte;
  }
}

// ---- decompress -----------------------------------------------------------------------------

// What the decode kernel is told, ready to be used: with a block of 1024 elements per wave, a scalar instruction of the
// beginning is one per block, and the four SIMDs share the scalar unit.
struct VDecodeArgs {
  const uint8_t* in;
  uint8_t* out;
  const uint8_t* sm;       // the stream's sections (of an empty tensor: the stream)
  const uint8_t* code;
  const uint32_t* tab;     // unused in the absolute mode
  const uint8_t* pos;
  splitzip_sizes* sizes;   // nullable
  uint64_t capacity, off_pos;
  uint32_t n, n_chunks, sm_last, code_last;   // see v_load_plane
  uint32_t k, val_bits;
  uint32_t hdr[16];        // as in VArgs
  uint8_t dec[16];
};
static_assert(sizeof(VDecodeArgs) == 176, "whole 16-byte words for the copy of v_decode_kernel");

// escape value idx of a stream whose value section starts at val (the section is known to lie inside the stream)
__device__ inline uint32_t v_value(const uint8_t* val, uint32_t bits, uint64_t idx) {
  if (bits == 8) return val[idx];
  const uint64_t bit = idx * bits;
  const uint32_t sh = (uint32_t)(bit & 7u);
  uint32_t v = val[bit >> 3] >> sh;
  if (sh + bits > 8) v |= (uint32_t)val[(bit >> 3) + 1] << (8 - sh);
  return v & ((1u << bits) - 1u);
}

// The values of the count records from lo on, all of them inside the section, as a run: value i, or nothing in particular
// from count on.  Narrow values (FP8, as wide as the exponent field) take two loads, the second of which fetches nothing
// for values that are bytes; what was loaded is made a value where it is used (of), so that nothing waits for it.
template <int DT>
struct VValues {
  __amdgpu_buffer_rsrc_t run, next;
  uint32_t bit0, bits;   // of the run's first byte, where value 0 starts
  struct Loaded { uint32_t low, high; };
  __device__ inline VValues(const uint8_t* val, uint32_t val_bits, uint32_t lo, uint32_t count) {
    bits = VFmt<DT>::ES == 2 ? 8u : val_bits;
    const uint64_t first = (uint64_t)lo * bits;
    bit0 = VFmt<DT>::ES == 2 ? 0u : (uint32_t)first & 7u;
    const uint32_t bytes = VFmt<DT>::ES == 2 || !count ? count : (bit0 + count * bits + 7u) >> 3;
    run = run_of(val + (first >> 3), bytes);
    if (VFmt<DT>::ES == 1) next = run_of(val + (first >> 3) + 1, bits == 8 || !bytes ? 0u : bytes - 1);
  }
  __device__ inline Loaded at(uint32_t i) const {
    const uint32_t byte = VFmt<DT>::ES == 2 ? i : (bit0 + i * bits) >> 3;
    return Loaded{ld_run1(run, byte), VFmt<DT>::ES == 2 ? 0u : (uint32_t)ld_run1(next, byte)};
  }
  __device__ inline uint32_t of(const Loaded& x, uint32_t i) const {
    if (VFmt<DT>::ES == 2) return x.low;
    return ((x.low | (x.high << 8)) >> ((bit0 + i * bits) & 7u)) & ((1u << bits) - 1u);
  }
};

// an inconsistent header or record: sticky bit in the caller's sizes record (nullable)
__device__ inline void v_flag_bad(splitzip_sizes* sizes) {
  if (sizes) atomicOr(&sizes->status, SPLITZIP_STATUS_BAD_STREAM);
}

// The header as every wave reads it: lane i holds word i & 15.  Compared with what the call expects and, words 6 to 9 (M,
// total), with what follows from M; all words at once, the expected ones put into lanes (one after the other in the scalar
// unit they were 60 instructions of a wave).  Wave-uniform result; M through m_out.
template <uint32_t PB>
__device__ inline bool v_check_header(const VDecodeArgs& a, uint32_t hw, uint32_t* m_out) {
  const uint32_t M = (uint32_t)__builtin_amdgcn_readlane((int)hw, 6);
  const uint64_t total = a.off_pos + a256((uint64_t)PB * M) + v_val_bytes(M, a.val_bits);
  uint32_t want = hw;
  const uint32_t word = threadIdx.x & 15u;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (i != 6) want = word == (uint32_t)i ? (i == 7 ? 0u : i == 8 ? (uint32_t)total : i == 9 ? (uint32_t)(total >> 32) : a.hdr[i]) : want;
  *m_out = M;
  return (__ballot(want != hw) == 0) & (M <= a.n) & (total <= a.capacity);
}

// One block of 1024 elements per wave.  Everything that depends on nothing -- the header, the offsets of the
// block's chunks, the block's slices of both planes -- is fetched at once; the escape records of the chunks
// follow as soon as the offsets are known and travel while the planes are decoded in registers, two elements per
// table entry.  A block with records goes through an LDS tile, where they are applied a lane each (in the sentinel
// mode by the lane that holds the sentinel, its exponent from the chunk's first 64 values in LDS); a block without
// is stored from the registers.  In the absolute mode the correction is left to v_scatter_kernel.
// Bound by the trips to memory of a wave that has one block, and before that by the scalar unit: 300 scalar instructions a
// wave, 128 waves a CU.  With the sections' addresses in the arguments, offsets kept in lanes and all of the header compared
// at once it takes, us before and now: a 64 MiB BF16 tensor top-8 22.9 and 20.6 (records ahead: 128 instead of 64, a third of
// the blocks have more), with chunks of 256 31.6 and 21.2, 4 Mi elements 5.1 and 3.9; 32 Mi elements of E4M3 top-8 with 4-bit
// values 21.6 and 15.5.  Loads that are given as bounded runs instead took 24.4: a run is five scalar instructions.
// MANY (sentinel mode): more than a quarter of the elements escaped.  4 Mi random words of BF16, top-15: 9.0 us, against
// 11.1 one sentinel after the other; 32 Mi of them 40 and 52; but 27.5 and 23.7 with 1 % escapes.
template <int DT, int CB, int MODE, int CS, bool MANY = false>
__global__ __launch_bounds__(kThreads) void v_decode_kernel(const VDecodeArgs args) {
  using F = VFmt<DT>;
  // escape mode, chunk size and position width are compile-time here: none of the format's choices costs a branch
  constexpr uint32_t PB = MODE == SPLITZIP_ESC_POS ? (CS == 10 ? 2u : 1u) : MODE == SPLITZIP_ESC_ABS32 ? 4u : 0u;
  constexpr uint32_t kPairs = 1u << (2 * CB), kPairMask = kPairs - 1u, per_blk = kVBlock >> CS, chunk = 1u << CS;
  constexpr uint32_t kAhead = MODE == SPLITZIP_ESC_POS && CS == 10 ? 128 : 64;   // records of a chunk that are asked for before they are counted on
  __shared__ uint32_t tbl[kPairs];
  __shared__ __attribute__((aligned(16))) uint32_t s_tile[kWaves][kVBlock * F::ES / 4];
  __shared__ uint8_t s_val[kWaves][MODE == SPLITZIP_ESC_SENTINEL ? 64 * per_blk : 1];
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  VDecodeArgs a;
  {
    // whole and once, as in args_arrived
    u32x4 x[11];
    __builtin_memcpy(x, &args, sizeof args);
    asm volatile("" : "+s"(x[0]), "+s"(x[1]), "+s"(x[2]), "+s"(x[3]), "+s"(x[4]), "+s"(x[5]), "+s"(x[6]), "+s"(x[7]), "+s"(x[8]), "+s"(x[9]), "+s"(x[10]));
    __builtin_memcpy(&a, x, sizeof args);
  }
  const uint8_t* const in = as_global(a.in);
  uint8_t* const out = as_global(a.out);
  splitzip_sizes* const sizes = as_global(a.sizes);
  const uint32_t blk = blockIdx.x * kWaves + wave, n_full = a.n / kVBlock, rest = a.n % kVBlock;
  const bool full = blk < n_full, live = full || (blk == n_full && rest);
  const uint32_t in_block = full ? kVBlock : live ? rest : 0u;   // elements of the block
  const uint32_t c_first = blk * per_blk;

  const uint32_t hw = reinterpret_cast<const uint32_t*>(in)[lane & 15u];
  uint32_t my_off = 0;   // lane q holds the offset of chunk c_first + q, of the last entry at most
  if (MODE != SPLITZIP_ESC_ABS32) {
    const uint32_t c = c_first + (lane <= per_blk ? lane : per_blk);
    my_off = as_global(a.tab)[c < a.n_chunks ? c : a.n_chunks];
  }
  // the block's slices of both planes
  uint32_t sm[2][2], cd[2][2];
#pragma unroll
  for (uint32_t s = 0; s < 2; ++s) {
    v_load_plane<F::SB>(as_global(a.sm), blk * (kVBlock / 8 * F::SB) + s * (kVStep / 8 * F::SB), a.sm_last, lane, sm[s]);
    v_load_plane<CB>(as_global(a.code), blk * (kVBlock / 8 * CB) + s * (kVStep / 8 * CB), a.code_last, lane, cd[s]);
  }
  // the decode table: both exponents of a pair of codes in place (entries beyond k are zero)
  if (tid < kPairs) {
    const u32x4 d = dec16_from(a.dec);
    tbl[tid] = F::pair(dec16_at(d, tid & ((1u << CB) - 1u)), dec16_at(d, tid >> CB));
  }
  uint32_t M;
  const bool ok = v_check_header<PB>(a, hw, &M);
  if (blockIdx.x == 0 && tid == 0) {
    if (sizes) {
      sizes->total_bytes = (uint32_t)__builtin_amdgcn_readlane(hw, 8) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hw, 9) << 32);
      sizes->n_escapes = M;
    }
    if (!ok) v_flag_bad(sizes);
  }
  lds_barrier();            // the table (an LDS-only barrier: the planes stay on their way)
  if (!ok || !live) return;   // nothing of a stream with a bad header is followed
  const uint8_t* const pos_sec = as_global(a.pos);
  const uint8_t* const val = pos_sec + a256((uint64_t)PB * M);
  constexpr uint32_t sentinel = (1u << CB) - 1u;
  // codes the codebook does not have can only occur if it leaves some unused (wave-uniform: no per-element work otherwise)
  const bool check_codes = a.k + (MODE == SPLITZIP_ESC_SENTINEL ? 1u : 0u) < (1u << CB);
  bool bad = false;

  // lane q <-> the block's chunk q: how many elements and how many records it has, no records if its entries are inconsistent
  // (sentinels are looked at one by one)
  uint32_t my_n = 0;
  if (MODE != SPLITZIP_ESC_ABS32) {
    const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)my_off, 0x101, 0xf, 0xf, false);   // row_shl:1, the entry behind
    const uint32_t left = in_block - (lane << CS), len = left < chunk ? left : chunk;
    const bool has = lane < per_blk && (lane << CS) < in_block, valid = next >= my_off && next - my_off <= len && next <= M;
    if (MODE == SPLITZIP_ESC_POS) bad = has && !valid;
    my_n = has && (valid || MODE == SPLITZIP_ESC_SENTINEL) ? next - my_off : 0u;
    my_off = has ? my_off : 0u;
  }
  // the first kAhead records of every chunk of the block are asked for now (in the sentinel mode: values without positions)
  typename VValues<DT>::Loaded rec_e[per_blk][kAhead / 64];
  uint32_t rec_p[per_blk][kAhead / 64], rec_lo[per_blk], rec_n[per_blk], any = 0;
#pragma unroll
  for (uint32_t q = 0; q < per_blk; ++q) {
    rec_lo[q] = __builtin_amdgcn_readlane(my_off, q);
    rec_n[q] = __builtin_amdgcn_readlane(my_n, q);
    if (MODE == SPLITZIP_ESC_ABS32) continue;
    any |= rec_n[q];
    uint32_t here = rec_n[q] < kAhead ? rec_n[q] : kAhead;
    if (MODE == SPLITZIP_ESC_SENTINEL) {   // records beyond M are no part of the stream, and an entry may lie behind the next
      const uint32_t hi = rec_lo[q] + rec_n[q], to = hi < M ? hi : M;
      here = to <= rec_lo[q] ? 0u : to - rec_lo[q] < kAhead ? to - rec_lo[q] : kAhead;
    }
    const auto pr = run_of(pos_sec + (uint64_t)PB * rec_lo[q], PB * here);
    const VValues<DT> vals(val, a.val_bits, rec_lo[q], here);
#pragma unroll
    for (uint32_t r = 0; r < kAhead / 64; ++r) {
      rec_p[q][r] = PB == 2 ? ld_run2(pr, 2u * lane + 128u * r) : PB == 1 ? ld_run1(pr, lane + 64u * r) : 0u;
      rec_e[q][r] = vals.at(lane + 64u * r);
    }
  }

  // dense decode; the codes all ones are the sentinels
  uint32_t o[2][F::NW], sent[2] = {0, 0};
#pragma unroll
  for (uint32_t s = 0; s < 2; ++s) {
    v_plane_fields<F::SB>(sm[s], lane);
    v_plane_fields<CB>(cd[s], lane);
    const uint32_t c = cd[s][0], from = s * kVStep + lane * 8, nv = in_block <= from ? 0u : in_block - from < 8 ? in_block - from : 8u;   // of the lane's elements
    F::unpack(sm[s], o[s]);
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b) {
      const uint32_t t = tbl[(c >> (2 * CB * b)) & kPairMask];
      if (F::ES == 2) o[s][b & (F::NW - 1)] |= t;
      else o[s][b >> 1] |= t << (16 * (b & 1));
    }
    if (MODE == SPLITZIP_ESC_SENTINEL) {
      sent[s] = CB == 4 ? c & (c >> 1) & (c >> 2) & (c >> 3) & 0x11111111u : c & (c >> 1) & (c >> 2) & 0x249249u;
      if (nv < 8) sent[s] &= (1u << (CB * nv)) - 1u;
    }
    if (check_codes) {
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) {
        const uint32_t code = (c >> (CB * j)) & sentinel;
        if (j < nv && code >= a.k && !(MODE == SPLITZIP_ESC_SENTINEL && code == sentinel)) bad = true;
      }
    }
  }
  if (MODE == SPLITZIP_ESC_SENTINEL) any = __ballot((sent[0] | sent[1]) != 0) != 0;

  // Sentinels in many places: a lane's eight at a time, in registers -- the exponent goes where the decode table left none,
  // no code all ones being in the codebook -- and every exponent asked for before the first is used: those beyond a
  // chunk's first 64 come from memory.
  if constexpr (MANY) {
#pragma unroll
    for (uint32_t q = 0; q < per_blk; ++q) s_val[wave][64 * q + lane] = (uint8_t)VValues<DT>(val, a.val_bits, rec_lo[q], 0).of(rec_e[q][0], lane);
    v_lds_settle();
    uint32_t carry = 0;
#pragma unroll
    for (uint32_t s = 0; s < 2; ++s) {
      // rank of every sentinel inside its chunk, then its exponent from the chunk's values
      uint32_t excl, low;
      const uint32_t tot = v_sparse_excl(__popc(sent[s]), excl, low);
      const uint32_t q = CS == 10 ? 0u : 2 * s + (lane >> 5);   // the lane's chunk inside the block
      uint32_t lo = rec_lo[0], n_q = rec_n[0], rank = excl + carry;
      if (CS == 8) {
        const uint32_t q0 = (2 * s) & (per_blk - 1), q1 = (2 * s + 1) & (per_blk - 1);
        lo = lane < 32 ? rec_lo[q0] : rec_lo[q1];
        n_q = lane < 32 ? rec_n[q0] : rec_n[q1];
        rank = lane < 32 ? excl : excl - low;
      } else {
        carry = tot;
      }
      const uint64_t hi = c_first + q < a.n_chunks ? lo + n_q : 0u;   // the offset behind the chunk's
      uint32_t e[8];
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) {
        e[j] = 0;
        if ((sent[s] >> (CB * j)) & 1u) {
          const uint64_t r = (uint64_t)(uint32_t)(lo + rank);
          if (r < hi && r < M) e[j] = rank < 64 && r >= lo ? (uint32_t)s_val[wave][64 * q + rank] : v_value(val, a.val_bits, r);
          else bad = true;
          ++rank;
        }
      }
#pragma unroll
      for (uint32_t j = 0; j < 8; ++j) {
        if (e[j] >= (uint32_t)F::EXPS) { bad = true; e[j] = 0; }
        if (F::ES == 2) o[s][j >> 1] |= e[j] << (F::LO + 16 * (j & 1));
        else o[s][(j >> 2) & (F::NW - 1)] |= e[j] << (F::LO + 8 * (j & 3));
      }
    }
    any = 0;
  }

  uint32_t* tile = s_tile[wave];
  if (any || !full) {
#pragma unroll
    for (uint32_t s = 0; s < 2; ++s) {
      if (F::ES == 2) reinterpret_cast<u32x4*>(tile)[s * 64 + lane] = u32x4{o[s][0], o[s][1], o[s][F::NW - 2], o[s][F::NW - 1]};
      else reinterpret_cast<u32x2*>(tile)[s * 64 + lane] = u32x2{o[s][0], o[s][1]};
    }
    // one element of the tile gets the exponent e
    auto patch = [&](uint32_t at, uint32_t e) {
      if (F::ES == 2) {
        uint16_t* t = reinterpret_cast<uint16_t*>(tile) + at;
        *t = (uint16_t)F::combine(F::signmant(*t), e);
      } else {
        uint8_t* t = reinterpret_cast<uint8_t*>(tile) + at;
        *t = (uint8_t)F::combine(F::signmant(*t), e);
      }
    };
    if (MODE == SPLITZIP_ESC_SENTINEL && !MANY) {
#pragma unroll
      for (uint32_t q = 0; q < per_blk; ++q) s_val[wave][64 * q + lane] = (uint8_t)VValues<DT>(val, a.val_bits, rec_lo[q], 0).of(rec_e[q][0], lane);
    }
    v_lds_settle();
    if (MODE == SPLITZIP_ESC_SENTINEL && !MANY) {
      uint32_t carry = 0;
#pragma unroll
      for (uint32_t s = 0; s < 2; ++s) {
        // rank of every sentinel inside its chunk, then its exponent from the chunk's values
        uint32_t excl, low;
        const uint32_t tot = v_sparse_excl(__popc(sent[s]), excl, low);
        const uint32_t q = CS == 10 ? 0u : 2 * s + (lane >> 5);   // the lane's chunk inside the block
        uint32_t lo = rec_lo[0], n_q = rec_n[0], rank = excl + carry;
        if (CS == 8) {
          const uint32_t q0 = (2 * s) & (per_blk - 1), q1 = (2 * s + 1) & (per_blk - 1);
          lo = lane < 32 ? rec_lo[q0] : rec_lo[q1];
          n_q = lane < 32 ? rec_n[q0] : rec_n[q1];
          rank = lane < 32 ? excl : excl - low;
        } else {
          carry = tot;
        }
        const uint64_t hi = c_first + q < a.n_chunks ? lo + n_q : 0u;   // the offset behind the chunk's
        uint32_t m = sent[s];
        while (m) {
          const uint32_t bit = (uint32_t)__ffs(m) - 1u, j = CB == 4 ? bit >> 2 : (bit * 11u) >> 5;   // bit / CB
          m &= m - 1;
          const uint64_t r = (uint64_t)(uint32_t)(lo + rank);
          uint32_t e = 0;
          if (r < hi && r < M) e = rank < 64 && r >= lo ? (uint32_t)s_val[wave][64 * q + rank] : v_value(val, a.val_bits, r);
          else bad = true;
          if (e >= (uint32_t)F::EXPS) { bad = true; e = 0; }
          patch(s * kVStep + lane * 8 + j, e);
          ++rank;
        }
      }
    }
    if (MODE == SPLITZIP_ESC_POS) {
      // the records of the block's chunks, one lane each, straight into the tile
#pragma unroll
      for (uint32_t q = 0; q < per_blk; ++q) {
        if (rec_n[q] == 0) continue;
        const uint32_t left = in_block - (q << CS), len = left < chunk ? left : chunk;
        // a chunk's positions ascend: each must lie above the one before it
        auto apply = [&](uint32_t i, uint32_t p, uint32_t before, uint32_t e) {
          if (i >= rec_n[q]) return;
          if (p >= len || (i > 0 && p <= before) || e >= (uint32_t)F::EXPS) bad = true;
          else patch(q * chunk + p, e);
        };
        uint32_t carry = 0;   // the position in front of a round's first
        const VValues<DT> ahead(val, a.val_bits, rec_lo[q], 0);
#pragma unroll
        for (uint32_t r = 0; r < kAhead / 64; ++r) {
          if (r > 0 && rec_n[q] <= 64 * r) break;
          apply(64 * r + lane, rec_p[q][r], lane_before(rec_p[q][r], carry), ahead.of(rec_e[q][r], 64 * r + lane));
          carry = (uint32_t)__builtin_amdgcn_readlane(rec_p[q][r], 63);
        }
        // the others, four times 64 on their way at a time
#pragma unroll 1
        for (uint32_t i0 = kAhead; i0 < rec_n[q]; i0 += 256) {
          const uint32_t lo = rec_lo[q] + i0, left = rec_n[q] - i0;
          const auto pr = run_of(pos_sec + (uint64_t)PB * lo, PB * left);
          const VValues<DT> vals(val, a.val_bits, lo, left);
          uint32_t p[4];
          typename VValues<DT>::Loaded e[4];
#pragma unroll
          for (uint32_t r = 0; r < 4; ++r) {
            p[r] = PB == 2 ? ld_run2(pr, 2u * lane + 128u * r) : ld_run1(pr, lane + 64u * r);
            e[r] = vals.at(lane + 64u * r);
          }
#pragma unroll
          for (uint32_t r = 0; r < 4; ++r) {
            apply(i0 + 64 * r + lane, p[r], lane_before(p[r], carry), vals.of(e[r], 64 * r + lane));
            carry = (uint32_t)__builtin_amdgcn_readlane(p[r], 63);
          }
        }
      }
    }
    v_lds_settle();
#pragma unroll
    for (uint32_t s = 0; s < 2; ++s) {
      if (F::ES == 2) {
        const u32x4 v = reinterpret_cast<const u32x4*>(tile)[s * 64 + lane];
        o[s][0] = v.x; o[s][1] = v.y; o[s][F::NW - 2] = v.z; o[s][F::NW - 1] = v.w;
      } else {
        const u32x2 v = reinterpret_cast<const u32x2*>(tile)[s * 64 + lane];
        o[s][0] = v.x; o[s][1] = v.y;
      }
    }
  }

  uint8_t* const dst = out + (uint64_t)F::ES * kVBlock * blk;
  if (full) {
#pragma unroll
    for (uint32_t s = 0; s < 2; ++s) {
      if (F::ES == 2) st_stream(reinterpret_cast<u32x4*>(dst) + s * 64 + lane, u32x4{o[s][0], o[s][1], o[s][F::NW - 2], o[s][F::NW - 1]});
      else st_stream(reinterpret_cast<u32x2*>(dst) + s * 64 + lane, u32x2{o[s][0], o[s][1]});
    }
  } else {
#pragma unroll 1
    for (uint32_t i = lane; i < rest; i += 64) {
      if (F::ES == 2) reinterpret_cast<uint16_t*>(dst)[i] = reinterpret_cast<const uint16_t*>(tile)[i];
      else dst[i] = reinterpret_cast<const uint8_t*>(tile)[i];
    }
  }
  if (bad) v_flag_bad(sizes);
}

// absolute mode: every record overwrites the exponent field of its element (runs after v_decode_kernel)
template <int DT>
__global__ __launch_bounds__(kThreads) void v_scatter_kernel(const VDecodeArgs a) {
  using F = VFmt<DT>;
  uint32_t M;
  if (!v_check_header<4>(a, reinterpret_cast<const uint32_t*>(a.in)[threadIdx.x & 15], &M)) return;
  const uint32_t* pos = reinterpret_cast<const uint32_t*>(a.pos);
  const uint8_t* val = a.pos + a256(4ull * M);
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < M; i += (uint64_t)gridDim.x * kThreads) {
    const uint32_t p = pos[i], e = v_value(val, a.val_bits, i);
    // the element indices ascend
    if (p >= a.n || e >= (uint32_t)F::EXPS || (i > 0 && p <= pos[i - 1])) { bad = true; continue; }
    if (F::ES == 2) {
      uint16_t* t = reinterpret_cast<uint16_t*>(a.out) + p;
      *t = (uint16_t)F::combine(F::signmant(*t), e);
    } else {
      a.out[p] = (uint8_t)F::combine(F::signmant(a.out[p]), e);
    }
  }
  if (bad) v_flag_bad(a.sizes);
}

#endif  // SPLITZIP_VARIANTS_HPP
