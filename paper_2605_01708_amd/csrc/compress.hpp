// SplitZip for MI355X: the compress kernels (dense transform of both formats with escape staging, one tile per workgroup; the finishing pass that ranks and places the escape records; the trailer; the one-launch kernel for small tensors).
// Part of the single translation unit splitzip.hip (included inside its anonymous namespace).
#ifndef SPLITZIP_COMPRESS_HPP
#define SPLITZIP_COMPRESS_HPP

// ---------------------------------------------------------------------------
// compress
// ---------------------------------------------------------------------------

// what the dense pass and the trailer need to know of one tensor and its stream
struct Planes {
  Words w;        // the tensor's words (read only here)
  uint8_t* out;
  uint64_t n, capacity;
  uint64_t off_tab, off_sm, off_code, off_pos, sm_bytes, code_bytes;
  uint32_t n_chunks, dtype;
};

__host__ __device__ inline Planes make_planes(const Words& in, void* out, uint64_t n, uint64_t capacity, int dtype) {
  const Layout L = make_layout(n, dtype);
  Planes p;
  p.w = in;
  p.out = static_cast<uint8_t*>(out);
  p.n = n;
  p.capacity = capacity;
  p.off_tab = L.off_tab; p.off_sm = L.off_sm; p.off_code = L.off_code; p.off_pos = L.off_pos;
  p.sm_bytes = L.sm_bytes; p.code_bytes = L.code_bytes;
  p.n_chunks = (uint32_t)L.n_chunks;
  p.dtype = (uint32_t)dtype;
  return p;
}

// where a chunk's escape records go: LDS staging (first pass) or their final place
struct LdsSink {
  uint16_t* pos;
  uint8_t* val;
  uint32_t tag;   // OR-ed into the position: which of the wave's chunks the record belongs to
  uint32_t cap;   // records the staging holds
  __device__ inline void put(uint32_t r, uint32_t p, uint32_t e) const {
    if (r < cap) {
      pos[r] = (uint16_t)(p | tag);
      val[r] = (uint8_t)e;
    }
  }
};
// a tile's slot in the staging area: records in the order of the tile's elements, position | exponent << 16
struct SlotSink {
  uint32_t* slot;
  uint32_t cap;   // records the slot holds
  __device__ inline void put(uint32_t r, uint32_t p, uint32_t e) const {
    if (r < cap) slot[r] = p | (e << 16);
  }
};
// records of 2^shift bytes between `from` and `capacity`, 2^32 - 1 at most (ranks are compared in 32 bits)
__device__ inline uint32_t room32(uint64_t capacity, uint64_t from, int shift) {
  const uint64_t room = capacity > from ? (capacity - from) >> shift : 0;
  return room < 0xffffffffull ? (uint32_t)room : 0xffffffffu;
}
// the final place of the records of a tensor: positions and, behind them, values
struct FinalSink {
  uint16_t* pos;
  uint8_t* val;
  uint32_t pos_room, val_room;   // records that fit below the capacity (a tensor has fewer than 2^32)
  __device__ inline void put(uint32_t r, uint32_t p, uint32_t e) const {
    if (r < pos_room) pos[r] = (uint16_t)p;
    if (r < val_room) val[r] = (uint8_t)e;
  }
};
// counting only
struct NullSink {
  __device__ inline void put(uint32_t, uint32_t, uint32_t) const {}
};

// Dense transform of 8 BF16 elements held in four dwords.
//   sm   : 8 sign+mantissa bytes, a = ((x >> 8) & 0x80) | (x & 0x7f)        (eq. (1))
//   code : 8 nibbles, element j in nibble j
//   F    : 8 nibbles, nibble j = 1 if element j is an escape
__device__ inline void encode8_bf16(const uint32_t (&w)[4], const uint16_t* lut, u32x2& sm,
                                    uint32_t& code, uint32_t& F) {
  uint32_t t[4], u[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    // bytes 0 and 2 of t hold a of the low / high half-word
    t[d] = (w[d] & 0x007f007fu) | ((w[d] >> 8) & 0x00800080u);
    const uint32_t e0 = (w[d] >> 7) & 0xffu, e1 = (w[d] >> 23) & 0xffu;
    // low byte: code pair; high byte: flag pair in the same nibble layout
    u[d] = (uint32_t)lut[e0] + ((uint32_t)lut[e1] << 4);
  }
  sm.x = byte_perm(t[1], t[0], 0x06040200u);
  sm.y = byte_perm(t[3], t[2], 0x06040200u);
  // x = [code(u_lo), code(u_hi), flag(u_lo), flag(u_hi)]
  const uint32_t x01 = byte_perm(u[1], u[0], 0x05010400u), x23 = byte_perm(u[3], u[2], 0x05010400u);
  code = byte_perm(x23, x01, 0x05040100u);
  F = byte_perm(x23, x01, 0x07060302u);
}

// escape records of one lane's 8 elements (flag nibbles in m), ranks r, r+1, ...
// The lane parks its four dwords in its own 16 bytes of LDS so that the escaping element can be
// picked with a run-time index (registers cannot be indexed that way).
template <typename Sink>
__device__ inline void emit_half_bf16(uint32_t* park, const uint32_t (&w)[4], uint32_t m, uint32_t r,
                                      uint32_t pos0, const Sink& sink) {
  if (m) {
    *reinterpret_cast<u32x4*>(park) = u32x4{w[0], w[1], w[2], w[3]};
    const uint16_t* x = reinterpret_cast<const uint16_t*>(park);
    do {
      const uint32_t jj = (uint32_t)(__ffs(m) - 1) >> 2;
      m &= m - 1;
      sink.put(r, pos0 + jj, ((uint32_t)x[jj] >> 7) & 0xffu);
      ++r;
    } while (m);
  }
}

// One chunk's words into registers: lane l holds elements [8 l, 8 l + 8) of each half-chunk.
// Elements past N read as zero.  LONG: kTileLong.
template <bool FULL, bool LONG>
__device__ inline void load_chunk_bf16(const Planes& a, const uint8_t* cptr, uint64_t cbase, int lane, uint32_t (&w)[2][4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t g0 = cbase + h * kHalf + lane * 8;   // first element of this lane's group
    uint32_t nvalid = 8;
    if (!FULL) nvalid = g0 >= a.n ? 0u : (uint32_t)(a.n - g0 < 8 ? a.n - g0 : 8);
    if (FULL) {
      // chunk pointer (wave-uniform) + a 32-bit lane offset: no 64-bit vector arithmetic
      const u32x4 v = LONG ? ld_run16(run_of(cptr, 2 * kChunk), 16u * (uint32_t)(h * 64 + lane)) : ld_stream(reinterpret_cast<const u32x4*>(cptr) + (uint32_t)(h * 64 + lane));
      w[h][0] = v.x; w[h][1] = v.y; w[h][2] = v.z; w[h][3] = v.w;
    } else if (nvalid == 8) {
      const u32x4 v = ld_stream(reinterpret_cast<const u32x4*>(cptr + 2 * (g0 - cbase)));
      w[h][0] = v.x; w[h][1] = v.y; w[h][2] = v.z; w[h][3] = v.w;
    } else {
      const uint16_t* p = reinterpret_cast<const uint16_t*>(cptr + 2 * (g0 - cbase));
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t lo = (uint32_t)(2 * d) < nvalid ? p[2 * d] : 0u;
        const uint32_t hi = (uint32_t)(2 * d + 1) < nvalid ? p[2 * d + 1] : 0u;
        w[h][d] = lo | (hi << 16);
      }
    }
  }
}

// One chunk's planes and escapes, as a wave holds them: the lane's 8 elements of each half-chunk
struct CodedBf16 {
  u32x2 sm[2];
  uint32_t code[2], F[2];     // nibbles; F: 1 for an escape
  uint32_t excl[2], tot0;     // escapes of the lanes below, per half; all of the first half
};
// One chunk by one wave, its words in w, in four steps: dense transform; planes out; escapes per lane and half, ranked over the
// wave (the chunk's count, wave-uniform, is returned); escape records into `sink` from rank `base` on, in element order:
// half, lane, element.
template <bool FULL>
__device__ inline void encode_chunk_bf16(const Planes& a, const uint16_t* lut, uint64_t cbase, int lane, const uint32_t (&w)[2][4], CodedBf16& c) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    encode8_bf16(w[h], lut, c.sm[h], c.code[h], c.F[h]);
    if (!FULL) {
      const uint64_t g0 = cbase + h * kHalf + lane * 8;
      const uint32_t nvalid = g0 >= a.n ? 0u : (uint32_t)(a.n - g0 < 8 ? a.n - g0 : 8);
      // elements past N contribute zero nibbles (their sm bytes are already 0)
      const uint32_t keep = nvalid == 8 ? ~0u : ((1u << (4 * nvalid)) - 1u);
      c.code[h] &= keep;
      c.F[h] &= keep;
    }
  }
}
__device__ inline uint32_t count_chunk_bf16(CodedBf16& c) {
  c.tot0 = wave_sparse_excl(__popc(c.F[0]), c.excl[0]);
  return c.tot0 + wave_sparse_excl(__popc(c.F[1]), c.excl[1]);
}
template <bool FULL, bool LONG>
__device__ inline void store_chunk_bf16(const Planes& a, uint64_t cbase, int lane, const CodedBf16& c) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t g0 = cbase + h * kHalf + lane * 8;
    // Sections are padded to 256 bytes and a lane's group never straddles the padded end, so
    // whole-group stores also write the zero padding.
    if (FULL && LONG) {
      st_run(run_of(a.out + a.off_sm + cbase, kChunk), 8u * (uint32_t)(h * 64 + lane), c.sm[h]);
      st_run(run_of(a.out + a.off_code + (cbase >> 1), kChunk / 2), 4u * (uint32_t)(h * 64 + lane), c.code[h]);
    } else if (FULL) {
      st_stream(reinterpret_cast<u32x2*>(a.out + a.off_sm + cbase) + (uint32_t)(h * 64 + lane), c.sm[h]);
      st_stream(reinterpret_cast<uint32_t*>(a.out + a.off_code + (cbase >> 1)) + (uint32_t)(h * 64 + lane), c.code[h]);
    } else {
      if (g0 < a256(a.sm_bytes)) st_stream(reinterpret_cast<u32x2*>(a.out + a.off_sm + g0), c.sm[h]);
      if ((g0 >> 1) < a256(a.code_bytes)) st_stream(reinterpret_cast<uint32_t*>(a.out + a.off_code + (g0 >> 1)), c.code[h]);
    }
  }
}
template <typename Sink>
__device__ inline void emit_chunk_bf16(uint32_t* park, int lane, const uint32_t (&w)[2][4], const CodedBf16& c, uint32_t total, uint32_t base, const Sink& sink) {
  if (!total) return;
  emit_half_bf16(park, w[0], c.F[0], base + c.excl[0], lane * 8, sink);
  emit_half_bf16(park, w[1], c.F[1], base + c.tot0 + c.excl[1], kHalf + lane * 8, sink);
}

// ---- FP8 E5M2 (appendix "SplitZip on FP8"): byte = s eeeee mm, e = (x >> 2) & 31, a = s m1 m0 ----
// One chunk by one wave; lane l owns the 16 consecutive elements [16 l, 16 l + 16): one 16-byte
// load, 8 bytes of codes, 6 bytes of the 3-bit plane (lanes 2p and 2p+1 share 12 bytes: the even
// lane stores 8 of them, the odd lane 4).

// a of the four bytes of w, packed LSB first into 12 bits
__device__ inline uint32_t pack3_e5m2(uint32_t w) {
  const uint32_t t = ((w >> 5) & 0x04040404u) | (w & 0x03030303u);
  const uint32_t x = t + (t << 5);   // bytes 0|1 meet in bits 5..10, bytes 2|3 in bits 21..26; no field overlaps another
  return ((x >> 5) & 0x3fu) | ((x >> 15) & 0xfc0u);
}
// inverse: 12 bits -> the sign and mantissa bits of four bytes, exponent field zero
__device__ inline uint32_t unpack3_e5m2(uint32_t r) {
  const uint32_t u = (r | (r << 10)) & 0x003f003fu;
  const uint32_t t = (u | (u << 5)) & 0x07070707u;
  return ((t & 0x04040404u) << 5) | (t & 0x03030303u);
}

template <bool FULL, bool LONG>
__device__ inline void load_chunk_e5m2(const Planes& a, const uint8_t* cptr, uint64_t cbase, int lane, uint32_t (&w)[4]) {
  const uint64_t g0 = cbase + lane * 16;
  uint32_t nvalid = 16;
  if (!FULL) nvalid = g0 >= a.n ? 0u : (uint32_t)(a.n - g0 < 16 ? a.n - g0 : 16);
  if (FULL) {
    const u32x4 v = LONG ? ld_run16(run_of(cptr, kChunk), 16u * (uint32_t)lane) : ld_stream(reinterpret_cast<const u32x4*>(cptr) + (uint32_t)lane);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else if (nvalid == 16) {
    const u32x4 v = ld_stream(reinterpret_cast<const u32x4*>(cptr + (g0 - cbase)));
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else {
    const uint8_t* p = cptr + (g0 - cbase);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      uint32_t x = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((uint32_t)(4 * d + j) < nvalid) x |= (uint32_t)p[4 * d + j] << (8 * j);
      w[d] = x;
    }
  }
}

struct CodedE5m2 {
  uint32_t lo, hi;            // the lane's 48 plane bits: lo holds bits 0..31, hi bits 32..47
  uint32_t code[2], F[2];
  uint32_t mine, excl;        // escapes of the lane, of the lanes below
};
// the four steps of a chunk, as for BF16; element order inside the chunk: lane, element
template <bool FULL>
__device__ inline void encode_chunk_e5m2(const Planes& a, const uint16_t* lut, uint64_t cbase, int lane, const uint32_t (&w)[4], CodedE5m2& c) {
  uint32_t r[4], u[8];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    r[d] = pack3_e5m2(w[d]);
    // entry of a byte: at byte offset (byte & 0x7c) of the table (see kLutShift)
    const uint8_t* lb = reinterpret_cast<const uint8_t*>(lut);
    const uint32_t t0 = *reinterpret_cast<const uint16_t*>(lb + (w[d] & 0x7cu));
    const uint32_t t1 = *reinterpret_cast<const uint16_t*>(lb + ((w[d] >> 8) & 0x7cu));
    const uint32_t t2 = *reinterpret_cast<const uint16_t*>(lb + ((w[d] >> 16) & 0x7cu));
    const uint32_t t3 = *reinterpret_cast<const uint16_t*>(lb + ((w[d] >> 24) & 0x7cu));
    // low byte: code pair; high byte: flag pair in the same nibble layout
    u[2 * d] = t0 + (t1 << 4);
    u[2 * d + 1] = t2 + (t3 << 4);
  }
  c.lo = r[0] | (r[1] << 12) | (r[2] << 24);
  c.hi = (r[2] >> 8) | (r[3] << 4);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t x01 = byte_perm(u[4 * q + 1], u[4 * q], 0x05010400u), x23 = byte_perm(u[4 * q + 3], u[4 * q + 2], 0x05010400u);
    c.code[q] = byte_perm(x23, x01, 0x05040100u);
    c.F[q] = byte_perm(x23, x01, 0x07060302u);
    asm volatile("" : "+v"(c.F[q]));   // made once: the compiler would make it again where it is counted and where it is used (1 to 2 % of a call)
  }
  if (!FULL) {
    // elements past N contribute zero nibbles (their plane bits are already 0)
    const uint64_t g0 = cbase + lane * 16;
    const uint32_t nvalid = g0 >= a.n ? 0u : (uint32_t)(a.n - g0 < 16 ? a.n - g0 : 16);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t nv = nvalid > (uint32_t)(8 * q) ? nvalid - 8 * q : 0u;
      const uint32_t keep = nv >= 8 ? ~0u : ((1u << (4 * nv)) - 1u);
      c.code[q] &= keep;
      c.F[q] &= keep;
    }
  }
}
__device__ inline uint32_t count_chunk_e5m2(CodedE5m2& c) {
  c.mine = __popc(c.F[0]) + __popc(c.F[1]);
  return wave_sparse_excl(c.mine, c.excl);
}
template <bool FULL, bool LONG>
__device__ inline void store_chunk_e5m2(const Planes& a, uint64_t cbase, int lane, const CodedE5m2& c) {
  const uint64_t g0 = cbase + lane * 16;
  // plane bytes of this lane pair: [12 p, 12 p + 12) of the chunk's 384
  // quad_perm [1,1,3,3]: the odd neighbour's bits
  // (a quad permute reads lanes of its own quad only: every lane gets a value, the old one is never kept)
  const uint32_t lo_up = __builtin_amdgcn_mov_dpp(c.lo, 0xF5, 0xf, 0xf, false);
  const uint32_t hi_up = __builtin_amdgcn_mov_dpp(c.hi, 0xF5, 0xf, 0xf, false);
  const uint64_t sm_chunk = (uint64_t)(uint32_t)(cbase >> 10) * 384u;   // the chunk's plane bytes start here: a scalar product
  const uint64_t sm_off = sm_chunk + (uint32_t)(lane >> 1) * 12;
  uint8_t* sm_chunk_ptr = a.out + a.off_sm + sm_chunk;
  uint8_t* sm_dst = sm_chunk_ptr + (uint32_t)(lane >> 1) * 12;
  // the pair's 12 bytes, all in the even lane
  uint32_t d0 = c.lo, d1 = (c.hi & 0xffffu) | (lo_up << 16), d2 = (lo_up >> 16) | (hi_up << 16);
  if (FULL) {
    // Both lanes of a pair write the pair's 12 bytes (quad_perm [0,0,2,2]: the even neighbour's bits): one
    // instruction writes the chunk's 384 bytes back to back, and it is issued whatever the lane -- so the
    // compiler can count on it when it works out how long a wave must wait for the loads issued before it.
    const uint32_t lo_dn = __builtin_amdgcn_mov_dpp(c.lo, 0xA0, 0xf, 0xf, false);
    const uint32_t hi_dn = __builtin_amdgcn_mov_dpp(c.hi, 0xA0, 0xf, 0xf, false);
    d0 = lo_dn; d1 = (hi_dn & 0xffffu) | (lo_up << 16);
    if (LONG) {
      st_run(run_of(sm_chunk_ptr, 3 * kChunk / 8), (uint32_t)(lane >> 1) * 12u, u32x3{d0, d1, d2});
      st_run(run_of(a.out + a.off_code + (cbase >> 1), kChunk / 2), 8u * (uint32_t)lane, u32x2{c.code[0], c.code[1]});
    } else {
      st_stream(reinterpret_cast<u32x3*>(sm_dst), u32x3{d0, d1, d2});
      st_stream(reinterpret_cast<u32x2*>(a.out + a.off_code + (cbase >> 1)) + (uint32_t)lane, u32x2{c.code[0], c.code[1]});
    }
  } else {
    // dword by dword up to the padded end of each plane; the pad can reach 128 bytes past the
    // chunk's own 384 plane bytes
    const uint64_t sm_end = a256(a.sm_bytes);
    if (!(lane & 1)) {
      if (sm_off < sm_end) *reinterpret_cast<uint32_t*>(sm_dst) = d0;
      if (sm_off + 4 < sm_end) *reinterpret_cast<uint32_t*>(sm_dst + 4) = d1;
      if (sm_off + 8 < sm_end) *reinterpret_cast<uint32_t*>(sm_dst + 8) = d2;
    }
    const uint64_t past = sm_chunk + 384 + 4 * (uint32_t)lane;
    if (lane < 32 && past < sm_end) *reinterpret_cast<uint32_t*>(a.out + a.off_sm + past) = 0;
    if ((g0 >> 1) < a256(a.code_bytes))
      *reinterpret_cast<u32x2*>(a.out + a.off_code + (g0 >> 1)) = u32x2{c.code[0], c.code[1]};
  }
}
template <typename Sink>
__device__ inline void emit_chunk_e5m2(uint32_t* park, int lane, const uint32_t (&w)[4], const CodedE5m2& c, uint32_t total, uint32_t base, const Sink& sink) {
  if (total && c.mine) {
    *reinterpret_cast<u32x4*>(park) = u32x4{w[0], w[1], w[2], w[3]};
    const uint8_t* x = reinterpret_cast<const uint8_t*>(park);
    uint32_t rr = base + c.excl;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      uint32_t m = c.F[q];
      while (m) {
        const uint32_t jj = 8 * q + ((uint32_t)(__ffs(m) - 1) >> 2);
        m &= m - 1;
        sink.put(rr, lane * 16 + jj, ((uint32_t)x[jj] >> 2) & 0x1fu);
        ++rr;
      }
    }
  }
}

// the two formats as seen by the compress kernel
struct Bf16 {
  static constexpr int DT = SPLITZIP_BF16;
  static constexpr int ES = 2;   // bytes per word
  struct Regs { uint32_t w[2][4]; };
  __device__ static inline void arrived(Regs& r) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int d = 0; d < 4; ++d) asm volatile("" : "+v"(r.w[h][d]));
  }
  // A workgroup of four waves takes a tile of 4 cpt chunks (pick_base_cpt: 16 KB of words, less for short launches), at
  // most kCpt of a wave's chunks at a time.  Eight workgroups per CU, what the
  // registers allow, serve launches of few tiles best and five those of many: us per call with eight / five / four,
  // 1219 / 1199 / 1203 (262 144 tiles), 309 / 306 / 307 (65 536), 26.5 / 26.9 / 27.1 (4096: one tensor), 17.4 / 18.1 / 18.0
  // (2048), and 43.0 / 42.5 (8192), 34.3 / 34.1 (6144) by a later kernel; unused LDS asked for at the launch sets the number
  // (plan_compress).
  static constexpr uint32_t kCpt = 2;
  static constexpr uint32_t kTileLdsPad = 22000;   // five workgroups per CU
  static constexpr uint32_t kSmallChunks = 40;
  static constexpr int kLutShift = 0;       // the LDS encode table holds the entry of exponent e in slot e
  // a chunk goes the fast way if it is complete (then nothing of a pad is its business: N is a multiple of 1024 there)
  __device__ static inline bool full(const Planes& a, uint64_t cbase) { return cbase + kChunk <= a.n; }
  template <bool FULL, bool LONG = false>
  __device__ static inline void load(const Planes& a, const uint8_t* cptr, uint64_t cbase, int lane, Regs& r) { load_chunk_bf16<FULL, LONG>(a, cptr, cbase, lane, r.w); }
  typedef CodedBf16 Coded;
  template <bool FULL>
  __device__ static inline void encode(const Planes& a, const uint16_t* lut, uint64_t cbase, int lane, const Regs& r, Coded& c) { encode_chunk_bf16<FULL>(a, lut, cbase, lane, r.w, c); }
  __device__ static inline uint32_t count(Coded& c) { return count_chunk_bf16(c); }
  template <bool FULL, bool LONG = false>
  __device__ static inline void store(const Planes& a, uint64_t cbase, int lane, const Coded& c) { store_chunk_bf16<FULL, LONG>(a, cbase, lane, c); }
  template <typename Sink>
  __device__ static inline void emit(uint32_t* park, int lane, const Regs& r, const Coded& c, uint32_t total, uint32_t base, const Sink& sink) { emit_chunk_bf16(park, lane, r.w, c, total, base, sink); }
};
struct E5m2 {
  static constexpr int DT = SPLITZIP_FP8_E5M2;
  static constexpr int ES = 1;
  struct Regs { uint32_t w[4]; };
  __device__ static inline void arrived(Regs& r) {
#pragma unroll
    for (int d = 0; d < 4; ++d) asm volatile("" : "+v"(r.w[d]));
  }
  // a tile of 4 cpt chunks: 16 KB of words in the longest launches and in padded ones, 4 or 8 KB below (pick_base_cpt); eight workgroups per CU (730 us for 64 tensors of 32 MiB against 750 us with six and
  // 790 us with five)
  static constexpr uint32_t kCpt = 4;
  static constexpr uint32_t kSmallChunks = 48;
  // The LDS encode table holds the entry of exponent e in slots 2 e and 2 e + 1: its byte offset is then
  // the word's byte with the sign and mantissa bits masked off, one instruction per element.
  static constexpr int kLutShift = 1;
  // the tensor's last chunk always goes the careful way: 384 plane bytes per chunk leave a pad behind an odd chunk count
  __device__ static inline bool full(const Planes& a, uint64_t cbase) { return cbase + kChunk < a.n; }
  template <bool FULL, bool LONG = false>
  __device__ static inline void load(const Planes& a, const uint8_t* cptr, uint64_t cbase, int lane, Regs& r) { load_chunk_e5m2<FULL, LONG>(a, cptr, cbase, lane, r.w); }
  typedef CodedE5m2 Coded;
  template <bool FULL>
  __device__ static inline void encode(const Planes& a, const uint16_t* lut, uint64_t cbase, int lane, const Regs& r, Coded& c) { encode_chunk_e5m2<FULL>(a, lut, cbase, lane, r.w, c); }
  __device__ static inline uint32_t count(Coded& c) { return count_chunk_e5m2(c); }
  template <bool FULL, bool LONG = false>
  __device__ static inline void store(const Planes& a, uint64_t cbase, int lane, const Coded& c) { store_chunk_e5m2<FULL, LONG>(a, cbase, lane, c); }
  template <typename Sink>
  __device__ static inline void emit(uint32_t* park, int lane, const Regs& r, const Coded& c, uint32_t total, uint32_t base, const Sink& sink) { emit_chunk_e5m2(park, lane, r.w, c, total, base, sink); }
};

// The steps of a chunk one after the other (planes out only if STORE): its escape count, wave-uniform.
template <typename F, bool FULL, bool STORE, bool LONG = false, typename Sink>
__device__ inline uint32_t process_chunk(const Planes& a, const uint16_t* lut, uint32_t* park, uint64_t cbase, int lane,
                                         const typename F::Regs& r, uint32_t base, const Sink& sink) {
  typename F::Coded c;
  F::template encode<FULL>(a, lut, cbase, lane, r, c);
  if (STORE) F::template store<FULL, LONG>(a, cbase, lane, c);
  const uint32_t total = F::count(c);
  F::emit(park, lane, r, c, total, base, sink);
  return total;
}

// header, sizes record and the zero padding behind the positions: one wave, once M is known
__device__ void compress_write_trailer(const Planes& a, const u32x4& dec, splitzip_sizes* sizes, uint32_t M,
                                       uint32_t err_flags, int lane) {
  const uint64_t off_val = a.off_pos + a256(2ull * M);
  const uint64_t total = off_val + M;
  for (uint64_t i = 2ull * M + lane; i < a256(2ull * M); i += 64)
    if (a.off_pos + i < a.capacity) a.out[a.off_pos + i] = 0;
  // chunk_off[C] = M, then zero padding up to the sign+mantissa plane
  uint32_t* tab = reinterpret_cast<uint32_t*>(a.out + a.off_tab);
  for (uint64_t i = (uint64_t)a.n_chunks + lane; a.off_tab + 4 * i < a.off_sm; i += 64) tab[i] = i == a.n_chunks ? M : 0u;
  if (lane == 0) {
    uint32_t h[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) h[i] = 0;
    h[0] = 0x31505a53u;                           // "SZP1"
    h[1] = 1u | (a.dtype << 16) | (4u << 24);      // version, dtype, code bits
    h[2] = kChunk;
    h[4] = (uint32_t)a.n; h[5] = (uint32_t)(a.n >> 32);
    h[6] = M;
    h[8] = (uint32_t)total; h[9] = (uint32_t)(total >> 32);
    h[10] = dec.x; h[11] = dec.y; h[12] = dec.z; h[13] = dec.w;
    uint4* ho = reinterpret_cast<uint4*>(a.out);
#pragma unroll
    for (int i = 0; i < 4; ++i) ho[i] = make_uint4(h[4 * i], h[4 * i + 1], h[4 * i + 2], h[4 * i + 3]);
    sizes->total_bytes = total;
    sizes->n_escapes = M;
    sizes->status = (total > a.capacity ? SPLITZIP_STATUS_OVERFLOW : 0u) | err_flags;
    sizes->reserved = 0;
  }
}

// ---- the two passes of a compress call ----
// Pass 1, compress_tile_kernel: one workgroup of four waves per tile of 4 x cpt chunks (16 KB of words in long
// launches, less in short ones: pick_base_cpt), started by the hardware in the order of the tiles -- the access
// pattern the memory system likes best, see traffic_shape_kernel -- or, in long launches, in xcd_order.  A workgroup waits for nobody: planes out; escapes of the tile staged in LDS, then written
// as (position | exponent << 16) records, in element order, to the tile's slot of the staging area; the tile's
// entries of the offset table as offsets inside the tile; the tile's escape count to the status area.
// Pass 2, compress_finish_kernel: one workgroup per group of 16 tiles.  It sums the counts (all of the tensor's:
// M; those before the group: its first rank), adds what lies before each tile to the tile's table entries and
// moves the records from the slots to their ranks in the position and value arrays.  A tile with more escapes
// than its slot (or its LDS staging) holds is encoded once more from the words, straight to the final place.
// (Launches that are few chunks, and not captured, do both in one: compress_short_kernel.)
// Between the passes lies a kernel boundary: no workgroup ever waits for another, nothing needs to be resident
// together, and no word of the workspace needs a defined value before a call.
constexpr uint32_t kTileThreads = 256;
constexpr uint32_t kGroup = 16;             // tiles per group of the finishing pass
constexpr uint32_t kFinishMost = 4;         // groups per workgroup of the finishing pass, at most
constexpr uint32_t kSlotAhead = 16;         // threads per tile that fetch records before the finishing pass knows the counts, two records each
constexpr uint32_t kTileStageCap = 256;     // escapes a wave can stage in LDS
constexpr uint32_t kSlotCapMost = 1024;     // records per tile slot, at most
constexpr uint64_t kDirectBytes = 128ull << 20;   // the finishing pass sums the tile counts itself if all its workgroups together read no more than this many bytes of them
constexpr uint32_t kSumGroup = 64;          // beyond: sums of this many tile counts, by tile_group_sum_kernel
// Tensors per launch: their descriptors travel as kernel arguments, in a block with room for kBatchFew of them (3.2 KB) or for kBatchMax
// (7.8 KB, which take the host 0.1 us more).  us per call in launches of 64 and this way: compress BF16 160 tensors of 20 chunks 16.1 and 6.2, 147 of
// 108 25.8 and 16.1, 100 of 1000 69.8 and 62.6, 90 of 5900 306.6 and 304.2, E5M2 143 of 537 45.2 and 30.7; decompress 147 of 108 15.2 and 12.3, 100 of
// 1000 61.8 and 58.4, E5M2 143 of 537 34.5 and 26.9.
constexpr uint32_t kBatchFew = 64, kBatchMax = 160;
constexpr uint32_t kRedo = 0x80000000u;     // in a tile's count: its records are not in its slot
constexpr uint32_t kMore = 1u;              // in a group's mark of the finishing pass, beside kRedo
static_assert(kGroup * kSlotAhead == kTileThreads, "every thread fetches records of one tile ahead");

// The arguments of a launch: what all its tensors share, then the tensors (N: room for kBatchMax or kBatchFew of them, or for the
// one of a single call, whose two launches then carry 144 bytes instead of 3.2 KB each).  A workgroup needs the first part and one
// tensor's, 144 bytes; both are fetched whole before anything is done with them (args_arrived).
struct TileItem {
  const uint8_t* in;
  uint8_t* out;
  uint64_t capacity;
  uint32_t n;
  uint32_t status_off;            // where the tensor's counts start in `status`
  uint8_t dec[16];                // its codebook, as its 16 decode entries: the kernels build the encode table from them
};
struct TileShared {
  splitzip_sizes* sizes;          // one record per tensor
  uint8_t* status;                // per tensor: u32 count of every tile, then u32 sum of every kSumGroup tiles
  uint8_t* stage;                 // per tensor stage_cap bytes: the tiles' slots
  union {
    uint64_t stage_cap;
    uint64_t tag;                 // compress_short_kernel, which stages nothing there: the call's
  };
  const splitzip_codebook* d_cbs; // nullable: codebooks in device memory, one per tensor, used instead of dec
  Words paging;                   // table and page geometry shared by all tensors (table null: contiguous tensors); base unused
  uint32_t cpt;                   // chunks per wave and tile, a power of two
  uint32_t tile_shift;            // log2 of the chunks per tile (4 cpt)
  union {
    uint32_t slot_cap;            // records per tile slot, the same for all tensors of the launch
    uint32_t looks;               // compress_short_kernel, which has no slots: how often a workgroup looks for the others' counts
  };
  uint32_t finish_groups;         // groups of kGroup tiles per workgroup of the finishing pass, 1 to kFinishMost
  uint32_t use_group_sums;        // the finishing pass reads sums of kSumGroup tile counts (tile_group_sum_kernel) instead of all tile counts
  uint32_t by_xcd;                // the dense pass takes its tiles in xcd_order
  __device__ inline u32x4 dec16_of(const TileItem& it, uint32_t k) const { return d_cbs ? load_dec16(d_cbs[k].dec) : dec16_from(it.dec); }
};
template <uint32_t N>
struct alignas(N == 1 ? 16 : 64) TileArgs {
  TileShared shared;
  TileItem item[N];
};
static_assert(sizeof(TileShared) == 96 && sizeof(TileItem) == 48, "whole 16-byte words for args_arrived");

// Copies of both parts, all of them waited for here and once.  Left to itself the compiler fetches an argument where
// it is used first, which for these kernels meant four or five trips to the argument block one after the other --
// and every launch has a new block that no cache holds -- before the first load of data was on its way.  With this,
// and a group's counts asked for beside everything else, one tensor's finishing pass went from 3.8 to 3.1 us.
template <uint32_t N>
__device__ inline void args_arrived(const TileArgs<N>& args, uint32_t item, TileShared& a, TileItem& it) {
  u32x4 x[6], y[3];
  __builtin_memcpy(x, &args.shared, 96);
  __builtin_memcpy(y, &args.item[item], 48);
  asm volatile("" : "+s"(x[0]), "+s"(x[1]), "+s"(x[2]), "+s"(x[3]), "+s"(x[4]), "+s"(x[5]), "+s"(y[0]), "+s"(y[1]), "+s"(y[2]));
  __builtin_memcpy(&a, x, 96);
  __builtin_memcpy(&it, y, 48);
  a.sizes = as_global(a.sizes);
  a.status = as_global(a.status);
  a.stage = as_global(a.stage);
  a.d_cbs = as_global(a.d_cbs);
  a.paging.table = as_global(a.paging.table);
  it.in = as_global(it.in);
  it.out = as_global(it.out);
}

// what both passes derive from the arguments for one tensor
struct TileGeom {
  Planes P;
  uint32_t tile_chunks, n_tiles;
  uint32_t* counts;      // n_tiles
  uint32_t* group_sums;  // ceil(n_tiles / kSumGroup)
  uint32_t* slots;       // n_tiles x slot_cap records
};
__device__ inline TileGeom tile_geom(const TileShared& a, const TileItem& it, uint32_t item, int dtype) {
  TileGeom g;
  g.P = make_planes(item_words(a.paging, it.in), it.out, it.n, it.capacity, dtype);
  g.tile_chunks = 1u << a.tile_shift;
  g.n_tiles = (g.P.n_chunks + g.tile_chunks - 1) >> a.tile_shift;
  g.counts = reinterpret_cast<uint32_t*>(a.status + it.status_off);
  g.group_sums = g.counts + g.n_tiles;
  g.slots = reinterpret_cast<uint32_t*>(a.stage + (uint64_t)item * a.stage_cap);
  return g;
}

// The LDS encode table (exponent e in slots e << shift ... : its code, or the escape mark 0x100) from the 16 decode
// entries of the codebook, by the first wave of the workgroup alone: escape marks everywhere, then the 16 codes on
// top (the LDS takes a wave's writes in order); the caller's barrier makes it visible to the others.  Entries that
// are no exponent of the format (a codebook in device memory is not the host's to check) are left out.
__device__ inline void build_encode_table(uint16_t* lut, const u32x4& d, int tid, int shift) {
  if (tid < 64) {
#pragma unroll
    for (int q = 0; q < 4; ++q) lut[q * 64 + tid] = 0x100u;
    const uint32_t k = (uint32_t)tid >> shift, sub = (uint32_t)tid & ((1u << shift) - 1u);
    const uint32_t e = dec16_at(d, k & 15u);
    if (k < 16 && e < (256u >> shift)) lut[(e << shift) + sub] = (uint16_t)k;
  }
}

// a barrier for LDS traffic only: global loads that are on their way stay on their way
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// What the dense pass is built for.  kTileOnce: a wave has CPT chunks, so that no loop over the chunks is left (its
// constants and copies of registers were 2 to 5 % of a call; us, with a loop and without: E5M2, 16 384 chunks 12.6 and
// 11.7, 64 tensors of 100 chunks 9.6 and 9.0; BF16, 128 chunks 6.0 and 5.8).  kTileLong: that in a launch that memory
// alone bounds: addresses are a scalar and an offset, and stores go through the L2 as they are written; short launches
// lose by it.  kTileLoop: a wave has more chunks, CPT of them at a time (very large tensors, whose counts would not fit).
constexpr int kTileOnce = 0, kTileLong = 1, kTileLoop = 2;

// CPT: chunks of a wave whose loads are issued together, before anything else happens in the workgroup.  Wave w of
// the tile owns the chunks [w cpt, w cpt + cpt) of the tile.
template <typename F, int CPT, uint32_t N, int KIND>
__global__ __launch_bounds__(kTileThreads) void compress_tile_kernel(const TileArgs<N> args) {
  constexpr bool LONG = KIND == kTileLong;
  constexpr int NW = kTileThreads / 64;
  __shared__ uint16_t lut[256];
  __shared__ uint16_t stage_pk[NW][kTileStageCap];
  __shared__ uint8_t stage_val[NW][kTileStageCap];
  __shared__ u32x4 s_park[kTileThreads];
  __shared__ uint32_t s_cnt[NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t item = blockIdx.y;
  TileShared a;
  TileItem it;
  args_arrived(args, item, a, it);
  if (KIND != kTileLoop) {
    a.cpt = CPT;
    a.tile_shift = CPT == 1 ? 2 : CPT == 2 ? 3 : 4;
  }
  const TileGeom G = tile_geom(a, it, item, F::DT);
  const Planes& P = G.P;
  // xcd_order, written out as one condition with the last tile straight from the length: as a call under by_xcd, or with
  // G.n_tiles - 1, the registers of what follows are laid out differently and it comes out slower (us per call: BF16, 3
  // tensors of 5937 chunks 17.1 and 16.7, 4 of 1999 paged 11.1 and 10.9; E5M2, 3 of 5937 13.3 and 13.2).  Without
  // elements there is no last tile, and no tile either.
  const uint32_t t = a.by_xcd && ((it.n - 1u) >> (10 + a.tile_shift)) >= (blockIdx.x | (kXcdWindow - 1u))
                         ? xcd_place(blockIdx.x) : blockIdx.x;
  if (t >= G.n_tiles) return;
  const uint32_t r0 = t << a.tile_shift, nb = P.n_chunks - r0 < G.tile_chunks ? P.n_chunks - r0 : G.tile_chunks;
  const uint32_t w0 = (uint32_t)wave * a.cpt;                                   // the wave's first chunk inside the tile
  const uint32_t mine = nb > w0 ? (nb - w0 < a.cpt ? nb - w0 : a.cpt) : 0u;     // and how many it has
  uint32_t* park = reinterpret_cast<uint32_t*>(&s_park[tid]);

  uint32_t wave_count = 0, my_start = 0;   // lane c: escapes of the wave before its c-th chunk
  const LdsSink lds{stage_pk[wave], stage_val[wave], 0u, kTileStageCap};
  typename F::Regs w[CPT];
  // A tile all of whose chunks are complete (every tile but a tensor's last, as a rule) takes a path without a
  // condition per chunk: nothing stands between the loads, and the compiler need not merge the registers of two
  // ways of loading a chunk.
  const uint32_t r_last = r0 + G.tile_chunks - 1;
  if (nb == G.tile_chunks && F::full(P, (uint64_t)r_last * kChunk)) {
    auto fetch = [&](uint32_t it0) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const uint64_t cbase = (uint64_t)(r0 + w0 + it0 + j) * kChunk;
        const uint8_t* cptr = chunk_at<F::ES>(P.w, cbase, P.w.table ? page_of_wave_chunk(P.w, r0 + w0 + it0 + j) : 0u);
        F::template load<true, LONG>(P, cptr, cbase, lane, w[j]);
      }
    };
    // the words first: the table is built while they are on their way
    fetch(0);
    build_encode_table(lut, a.dec16_of(it, item), tid, F::kLutShift);
    lds_barrier();
    for (uint32_t it0 = 0; it0 < a.cpt; it0 += CPT) {
      if (it0 > 0) fetch(it0);   // tiles of more than CPT chunks per wave (very large tensors)
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        if ((uint32_t)lane == it0 + j) my_start = wave_count;
        wave_count += process_chunk<F, true, true, LONG>(P, lut, park, (uint64_t)(r0 + w0 + it0 + j) * kChunk, lane, w[j], wave_count, lds);
      }
    }
  } else {
    // the wave's chunks [it0, it0 + CPT) into w (nothing for chunks it does not have)
    auto fetch = [&](uint32_t it0) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const uint32_t c = it0 + j;
        if (c < mine) {
          const uint64_t cbase = (uint64_t)(r0 + w0 + c) * kChunk;
          const uint8_t* cptr = chunk_at<F::ES>(P.w, cbase, P.w.table ? page_of_chunk(P.w, r0 + w0 + c) : 0u);
          if (F::full(P, cbase)) F::template load<true>(P, cptr, cbase, lane, w[j]);
          else F::template load<false>(P, cptr, cbase, lane, w[j]);
        }
      }
    };
    fetch(0);
    build_encode_table(lut, a.dec16_of(it, item), tid, F::kLutShift);
    lds_barrier();
    // dense pass; the wave's escape records into its LDS staging in element order, the chunks' counts kept in lanes
    for (uint32_t it0 = 0; it0 < mine; it0 += CPT) {
      if (it0 > 0) fetch(it0);
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const uint32_t c = it0 + j;
        if (c >= mine) break;
        const uint64_t cbase = (uint64_t)(r0 + w0 + c) * kChunk;
        if ((uint32_t)lane == c) my_start = wave_count;
        wave_count += F::full(P, cbase) ? process_chunk<F, true, true>(P, lut, park, cbase, lane, w[j], wave_count, lds)
                                        : process_chunk<F, false, true>(P, lut, park, cbase, lane, w[j], wave_count, lds);
      }
    }
  }
  if (lane == 0) s_cnt[wave] = wave_count;
  lds_barrier();
  uint32_t before = 0, total = 0;
  bool redo = false;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const uint32_t c = s_cnt[q];
    before += q < wave ? c : 0u;
    total += c;
    redo = redo || c > kTileStageCap;
  }
  redo = redo || total > a.slot_cap;
  // the tile's entries of the offset table, for now as offsets inside the tile
  uint32_t* tab = reinterpret_cast<uint32_t*>(P.out + P.off_tab);
  if ((uint32_t)lane < mine) tab[r0 + w0 + lane] = before + my_start;
  if (!redo) {
    uint32_t* slot = G.slots + (uint64_t)t * a.slot_cap + before;   // staged record i of this wave is the (before + i)-th of the tile
    for (uint32_t i = lane; i < wave_count; i += 64) slot[i] = (uint32_t)stage_pk[wave][i] | ((uint32_t)stage_val[wave][i] << 16);
  }
  if (tid == 0) G.counts[t] = total | (redo ? kRedo : 0u);
  // the finishing pass reads whole vectors of four counts: the tensor's last tile clears what its vector holds behind it
  if (t == G.n_tiles - 1 && tid > 0 && tid < 4 && (t & 3u) + tid < 4) G.counts[t + tid] = 0;
}

// sums of kSumGroup tile counts each, for launches beyond kDirectBytes (one wave per sum)
template <typename F, uint32_t N>
__global__ __launch_bounds__(64) void tile_group_sum_kernel(const TileArgs<N> args) {
  TileShared a;
  TileItem it;
  args_arrived(args, blockIdx.y, a, it);
  const TileGeom G = tile_geom(a, it, blockIdx.y, F::DT);
  const uint32_t g = blockIdx.x, t = g * kSumGroup + threadIdx.x;
  if (g * kSumGroup >= G.n_tiles) return;
  const uint32_t sum = wave_last(wave_incl_scan(t < G.n_tiles ? G.counts[t] & ~kRedo : 0u));
  if (threadIdx.x == 0) G.group_sums[g] = sum;
}

template <typename F, uint32_t N, uint32_t GROUPS>
__global__ __launch_bounds__(kTileThreads) void compress_finish_kernel(const TileArgs<N> args) {
  constexpr int NW = kTileThreads / 64;
  static_assert(GROUPS <= kFinishMost && kFinishMost <= NW, "one wave scans the counts of one group");
  __shared__ uint16_t lut[256];
  __shared__ u32x4 s_park[kTileThreads];
  __shared__ uint32_t s_cnt[GROUPS][kGroup];       // the counts of the groups' tiles, redo mark included
  __shared__ uint32_t s_tp[GROUPS][kGroup + 1];    // escapes of a group's tiles before each tile
  __shared__ uint32_t s_red[2 * NW];
  __shared__ uint32_t s_mark[GROUPS];              // kMore: a group has a tile with more records than were fetched ahead; kRedo: one that is encoded again
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t item = blockIdx.y;
  TileShared a;
  TileItem it;
  args_arrived(args, item, a, it);
  const TileGeom G = tile_geom(a, it, item, F::DT);
  const Planes& P = G.P;
  const uint32_t n_groups = (G.n_tiles + kGroup - 1) / kGroup;
  // the workgroup's groups: [g0, g0 + ng) -- GROUPS of them in a row (1 to kFinishMost: a launch of many
  // groups gives every workgroup several, so that fewer rounds of workgroups pass through the chip; each round
  // costs the same few trips to memory whatever it carries)
  const uint32_t g0 = blockIdx.x * GROUPS;
  if (g0 >= (n_groups ? n_groups : 1u)) return;   // a tensor without elements still gets its header
  const uint32_t ng = n_groups - g0 < GROUPS ? (n_groups > g0 ? n_groups - g0 : 1u) : GROUPS;
  uint32_t* park = reinterpret_cast<uint32_t*>(&s_park[tid]);
  uint32_t* tab = reinterpret_cast<uint32_t*>(P.out + P.off_tab);
  const uint32_t group_entries = kGroup << a.tile_shift;

  // Everything whose address does not depend on the counts is fetched at once: the counts themselves, the
  // groups' table entries (one per thread and group, or a few) and the first 2 kSlotAhead records of every tile's slot
  // (two per thread: hardly a tile has more, so hardly a workgroup has to go to memory once more after the barrier).
  // No load stands behind a condition: each is one of a bounded run, at an offset beyond its end where a thread wants none
  // (guarded one by one, each by a few scalar instructions and a branch, and with a condition per group where the groups
  // are the kernel's own now, a call took 0.4 us more: BF16, 128 chunks 5.83 and 5.44, 16 384 16.3 and 15.7; E5M2, 4096
  // chunks 7.56 and 7.14).
  constexpr uint32_t kNone = 0xfffffff0u;
  const uint32_t t_first = g0 * kGroup, c_first = t_first << a.tile_shift;   // the workgroup's first tile and chunk
  const uint32_t tiles_here = G.n_tiles > t_first ? (G.n_tiles - t_first < GROUPS * kGroup ? G.n_tiles - t_first : GROUPS * kGroup) : 0u;
  const uint32_t chunks_here = P.n_chunks > c_first ? (P.n_chunks - c_first < GROUPS * group_entries ? P.n_chunks - c_first : GROUPS * group_entries) : 0u;
  // wave q: the counts of the tiles of group q
  const auto count_run = run_of(reinterpret_cast<const uint8_t*>(G.counts + t_first), 4u * tiles_here);
  const uint32_t c_mine = ld_run4<0>(count_run, (uint32_t)wave < GROUPS && (uint32_t)lane < kGroup ? 4u * ((uint32_t)wave * kGroup + lane) : kNone);
  // All counts, four per load, four loads per thread on their way at a time (they start 256-byte aligned, the dense pass has
  // cleared what the last vector holds behind them, and the first group's tiles start with a vector); none if there are
  // sums of them.
  const uint32_t nvec = a.use_group_sums ? 0u : (G.n_tiles + 3) / 4, v_first = t_first / 4;
  const auto vec_run = run_of(reinterpret_cast<const uint8_t*>(G.counts), 16u * nvec);
  u32x4 v[4];
  auto fetch = [&](uint32_t v0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = ld_run16<0>(vec_run, 16u * (v0 + q * kTileThreads + tid));
  };
  fetch(0);
  const uint32_t sl = (uint32_t)tid / kSlotAhead, sj = (uint32_t)tid % kSlotAhead;   // tile of a group, record of the tile
  uint32_t my_entry[GROUPS], rec_ahead[GROUPS], rec_ahead2[GROUPS];
  {
    const auto tab_run = run_of(reinterpret_cast<const uint8_t*>(tab + c_first), 4u * chunks_here);
    const auto slot_run = run_of(reinterpret_cast<const uint8_t*>(G.slots + (uint64_t)t_first * a.slot_cap), 4u * a.slot_cap * tiles_here);
#pragma unroll
    for (uint32_t q = 0; q < GROUPS; ++q) {
      const uint32_t rec = 4u * ((q * kGroup + sl) * a.slot_cap + sj);
      my_entry[q] = ld_run4<0>(tab_run, (uint32_t)tid < group_entries ? 4u * (q * group_entries + tid) : kNone);
      rec_ahead[q] = ld_run4<0>(slot_run, sj < a.slot_cap ? rec : kNone);
      rec_ahead2[q] = ld_run4<0>(slot_run, sj + kSlotAhead < a.slot_cap ? rec + 4u * kSlotAhead : kNone);
    }
  }
  uint32_t before = 0, all = 0;
  for (uint32_t v0 = 0;;) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t sum = (v[q].x & ~kRedo) + (v[q].y & ~kRedo) + (v[q].z & ~kRedo) + (v[q].w & ~kRedo);
      all += sum;
      before += v0 + q * kTileThreads + tid < v_first ? sum : 0u;
    }
    v0 += 4 * kTileThreads;
    if (v0 >= nvec) break;
    fetch(v0);
  }
  if (a.use_group_sums) {
    const uint32_t n_sums = (G.n_tiles + kSumGroup - 1) / kSumGroup, whole = t_first / kSumGroup;   // sums that lie before the first group entirely
    for (uint32_t i = tid; i < n_sums; i += kTileThreads) {
      const uint32_t c = G.group_sums[i];
      all += c;
      before += i < whole ? c : 0u;
    }
    for (uint32_t i = whole * kSumGroup + tid; i < t_first; i += kTileThreads) before += G.counts[i] & ~kRedo;
  }
  before = wave_last(wave_incl_scan(before));
  all = wave_last(wave_incl_scan(all));
  if (lane == 0) {
    s_red[wave] = before;
    s_red[NW + wave] = all;
  }
  if ((uint32_t)wave < ng) {
    // what lies before each tile inside the group
    const uint32_t c = c_mine;
    const uint32_t incl = wave_incl_scan(c & ~kRedo);
    if ((uint32_t)lane < kGroup) {
      s_cnt[wave][lane] = c;
      s_tp[wave][lane] = incl - (c & ~kRedo);
    }
    if (lane == 63) s_tp[wave][kGroup] = incl;
    const uint64_t more = __ballot((c & ~kRedo) > 2 * kSlotAhead && !(c & kRedo)), again = __ballot((c & kRedo) != 0);
    if (lane == 0) s_mark[wave] = (more ? kMore : 0u) | (again ? kRedo : 0u);
  } else if ((uint32_t)wave < GROUPS && lane == 0) {
    s_mark[wave] = 0;
  }
  lds_barrier();   // the records and entries stay on their way
  uint32_t first = 0, M = 0;   // the rank of the first record of the group at hand; all records of the tensor
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    first += s_red[q];
    M += s_red[NW + q];
  }
  const uint64_t off_val = P.off_pos + a256(2ull * M);
  FinalSink fin;
  fin.pos = reinterpret_cast<uint16_t*>(P.out + P.off_pos);
  fin.pos_room = room32(P.capacity, P.off_pos, 1);
  fin.val = P.out + off_val;
  fin.val_room = room32(P.capacity, off_val, 0);

  // header, pads and sizes by one wave of the first workgroup, which does it while the others place the records
  if (g0 == 0 && wave == NW - 1) compress_write_trailer(P, a.dec16_of(it, item), a.sizes + item, M, 0u, lane);

  // Tiles whose records are not in their slots: once more from the words, by the offsets inside the tile that the
  // first pass left in the table.  Rare, and kept out of the way of the groups that have none: looking at every
  // tile's count for the mark, one LDS read after the other, was half of this kernel's time.
  uint32_t marks = 0;
#pragma unroll
  for (uint32_t q = 0; q < GROUPS; ++q) marks |= s_mark[q];
  if (marks & kRedo) {
    build_encode_table(lut, a.dec16_of(it, item), tid, F::kLutShift);
    __syncthreads();
    uint32_t group_first = first;
#pragma unroll 1
    for (uint32_t q = 0; q < ng; ++q) {
#pragma unroll 1
      for (uint32_t l = 0; l < kGroup; ++l) {
        if (!(s_cnt[q][l] & kRedo)) continue;   // uniform: the counts are the same for every thread
        const uint32_t r0 = ((g0 + q) * kGroup + l) << a.tile_shift;
        const uint32_t nb = P.n_chunks - r0 < G.tile_chunks ? P.n_chunks - r0 : G.tile_chunks;
        typename F::Regs w;
#pragma unroll 1
        for (uint32_t k = wave; k < nb; k += NW) {
          const uint64_t cbase = (uint64_t)(r0 + k) * kChunk;
          const uint32_t base = group_first + s_tp[q][l] + tab[r0 + k];
          const uint8_t* cptr = chunk_at<F::ES>(P.w, cbase, P.w.table ? page_of_chunk(P.w, r0 + k) : 0u);
          if (F::full(P, cbase)) {
            F::template load<true>(P, cptr, cbase, lane, w);
            process_chunk<F, true, false>(P, lut, park, cbase, lane, w, base, fin);
          } else {
            F::template load<false>(P, cptr, cbase, lane, w);
            process_chunk<F, false, false>(P, lut, park, cbase, lane, w, base, fin);
          }
        }
      }
      group_first += s_tp[q][kGroup];
    }
    __syncthreads();   // the table has been read by whoever needed its entries as offsets inside a tile
  }

#pragma unroll
  for (uint32_t q = 0; q < GROUPS; ++q) {
    if (q >= ng) break;
    const uint32_t t0 = (g0 + q) * kGroup, c0 = t0 << a.tile_shift;
    const uint32_t entries = P.n_chunks > c0 ? (P.n_chunks - c0 < group_entries ? P.n_chunks - c0 : group_entries) : 0u;
    const uint32_t* cnt = s_cnt[q];
    const uint32_t* tp = s_tp[q];
    // the table entries: what lies before the tile added to the offsets inside the tile
    if ((uint32_t)tid < entries) tab[c0 + tid] = my_entry[q] + first + tp[(uint32_t)tid >> a.tile_shift];
    for (uint32_t e = tid + kTileThreads; e < entries; e += kTileThreads) tab[c0 + e] += first + tp[e >> a.tile_shift];
    // the records fetched ahead
    const uint32_t cl = cnt[sl];
    if (!(cl & kRedo) && sj < cl) fin.put(first + tp[sl] + sj, rec_ahead[q] & 0xffffu, rec_ahead[q] >> 16);
    if (!(cl & kRedo) && sj + kSlotAhead < cl) fin.put(first + tp[sl] + sj + kSlotAhead, rec_ahead2[q] & 0xffffu, rec_ahead2[q] >> 16);
    // The rest of the slots of tiles with more records than that: rank r of the group belongs to the last tile that
    // starts at or before r.  Two records per thread are on their way at a time.
    const uint32_t group_total = tp[kGroup];
    if (s_mark[q] & kMore) {   // a tile of the group has more records than were fetched ahead
      auto locate = [&](uint32_t r, uint32_t& l, uint32_t& j) -> bool {
        l = 0;
#pragma unroll
        for (uint32_t step = kGroup / 2; step; step >>= 1)
          if (tp[l + step] <= r) l += step;
        j = r - tp[l];
        return r < group_total && j >= 2 * kSlotAhead && !(cnt[l] & kRedo);
      };
      for (uint32_t r = tid; r < group_total; r += 2 * kTileThreads) {
        uint32_t l0, j0, l1, j1, rec0 = 0, rec1 = 0;
        const bool take0 = locate(r, l0, j0), take1 = locate(r + kTileThreads, l1, j1);
        if (take0) rec0 = G.slots[(uint64_t)(t0 + l0) * a.slot_cap + j0];
        if (take1) rec1 = G.slots[(uint64_t)(t0 + l1) * a.slot_cap + j1];
        if (take0) fin.put(first + r, rec0 & 0xffffu, rec0 >> 16);
        if (take1) fin.put(first + r + kTileThreads, rec1 & 0xffffu, rec1 >> 16);
      }
    }
    first += group_total;
  }
}

// ---- small tensors: one launch, one workgroup per tensor ----
// Up to F::kSmallChunks chunks a tensor is one workgroup's work in a captured call and in a batch that is too much for the short launch below
// (pick_short), and up to kSmallestShort in every call: 16 waves own consecutive runs of its chunks, so the
// counts meet in LDS, every rank is known behind one barrier and nothing is staged outside the workgroup.  What bounds
// such a call is the launch: the second one takes the host 2.7 us and the device 3.1 us.  Device us per call, this
// kernel / two launches: BF16 5.2 / 6.8 (17 chunks), 6.4 / 6.7 (33), 7.3 / 6.6 (49), 10.6 / 6.6 (97); E5M2 5.6 / 7.6
// (17), 6.8 / 7.9 (33), 7.6 / 7.8 (49), 8.8 / 7.8 (65); with the host's part, one call after the other, BF16 5.1 / 9.3
// (17 chunks), 6.1 / 9.3 (33).
constexpr uint32_t kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr uint32_t kSmallStageCap = 384;   // escapes a wave stages in LDS; a wave with more goes over its chunks again

template <typename F, uint32_t N>
__global__ __launch_bounds__(kSmallThreads) void compress_small_kernel(const TileArgs<N> args) {
  __shared__ uint16_t lut[256];
  __shared__ uint16_t stage_pos[kSmallWaves][kSmallStageCap];
  __shared__ uint8_t stage_val[kSmallWaves][kSmallStageCap];
  __shared__ u32x4 s_park[kSmallThreads];
  __shared__ uint32_t s_cnt[kSmallWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t item = blockIdx.x;
  TileShared a;
  TileItem it;
  args_arrived(args, item, a, it);
  const Planes P = make_planes(item_words(a.paging, it.in), it.out, it.n, it.capacity, F::DT);
  const uint32_t per = (P.n_chunks + kSmallWaves - 1) / kSmallWaves, c0 = (uint32_t)wave * per;   // the wave's chunks: [c0, c0 + mine)
  const uint32_t mine = P.n_chunks > c0 ? (P.n_chunks - c0 < per ? P.n_chunks - c0 : per) : 0u;
  uint32_t* park = reinterpret_cast<uint32_t*>(&s_park[tid]);

  auto fetch = [&](uint32_t c, typename F::Regs& w) {
    const uint64_t cbase = (uint64_t)(c0 + c) * kChunk;
    const uint8_t* cptr = chunk_at<F::ES>(P.w, cbase, P.w.table ? page_of_chunk(P.w, c0 + c) : 0u);
    if (F::full(P, cbase)) F::template load<true>(P, cptr, cbase, lane, w);
    else F::template load<false>(P, cptr, cbase, lane, w);
  };
  typename F::Regs cur, nxt;
  if (mine > 0) fetch(0, cur);
  const u32x4 dec = a.dec16_of(it, item);
  build_encode_table(lut, dec, tid, F::kLutShift);
  lds_barrier();
  const LdsSink lds{stage_pos[wave], stage_val[wave], 0u, kSmallStageCap};
  uint32_t count = 0, my_start = 0;   // lane c: escapes of the wave before its c-th chunk
  for (uint32_t c = 0; c < mine; ++c) {
    if (c + 1 < mine) fetch(c + 1, nxt);   // the next chunk's words travel while this one is worked on
    const uint64_t cbase = (uint64_t)(c0 + c) * kChunk;
    if ((uint32_t)lane == c) my_start = count;
    count += F::full(P, cbase) ? process_chunk<F, true, true>(P, lut, park, cbase, lane, cur, count, lds)
                               : process_chunk<F, false, true>(P, lut, park, cbase, lane, cur, count, lds);
    cur = nxt;
  }
  if (lane == 0) s_cnt[wave] = count;
  lds_barrier();
  const uint32_t c_lane = (uint32_t)lane < kSmallWaves ? s_cnt[lane] : 0u, incl = wave_incl_scan(c_lane);
  const uint32_t M = wave_last(incl), first = (uint32_t)__builtin_amdgcn_readlane(incl - c_lane, wave);
  const uint64_t off_val = P.off_pos + a256(2ull * M);
  FinalSink fin;
  fin.pos = reinterpret_cast<uint16_t*>(P.out + P.off_pos);
  fin.pos_room = room32(P.capacity, P.off_pos, 1);
  fin.val = P.out + off_val;
  fin.val_room = room32(P.capacity, off_val, 0);
  uint32_t* tab = reinterpret_cast<uint32_t*>(P.out + P.off_tab);
  if ((uint32_t)lane < mine) tab[c0 + lane] = first + my_start;
  if (count <= kSmallStageCap) {
    for (uint32_t i = lane; i < count; i += 64) fin.put(first + i, stage_pos[wave][i], stage_val[wave][i]);
  } else {
#pragma unroll 1
    for (uint32_t c = 0; c < mine; ++c) {
      const uint64_t cbase = (uint64_t)(c0 + c) * kChunk;
      const uint32_t base = first + (uint32_t)__builtin_amdgcn_readlane(my_start, c);
      fetch(c, cur);
      if (F::full(P, cbase)) process_chunk<F, true, false>(P, lut, park, cbase, lane, cur, base, fin);
      else process_chunk<F, false, false>(P, lut, park, cbase, lane, cur, base, fin);
    }
  }
  if (wave == kSmallWaves - 1) compress_write_trailer(P, dec, a.sizes + item, M, 0u, lane);   // the wave with the fewest chunks
}

// ---- short launches: one kernel, whose workgroups tell one another their counts ----
// What bounds a short call is its launches: the finishing pass takes the host 2.3 us, and the device 3 us and the gap in
// front of it.  Here a workgroup takes a tile of four chunks, one per wave, as in the dense pass, tells its count to the others
// of its tensor, waits until all counts are there, and places its own records, which have not left its LDS.
//   A tile's word in the status area: the call's tag (47 bits, another one for every call, so that no word needs a defined
//   value before a call), kShortLeft, kShortTaken and the count.  One atomic word says all there is to say: nothing else that
//   a workgroup writes is read by another.  There are kShortCopies copies of a tensor's words and a workgroup reads one of
//   them: all workgroups reading the same few lines from the device's point of coherence took longer than the work.
//   No wait is without an end.  A workgroup that has looked a.looks times (50 us, in which the rest of the launch has not got onto
//   the chip) marks its tile as left, looks once more and, if counts are missing still, ends.  The mark and the count are
//   each written, and the write waited for, before the writer looks at the other words: so whoever publishes last of all
//   sees all counts the first time it looks, and with them the mark of every workgroup that looked for the last time
//   before that.  Tiles left are encoded again by whichever workgroup takes them first (kShortTaken, in the first copy).
constexpr uint32_t kShortCopies = 8;
constexpr uint32_t kShortMostCpt = 2;   // chunks per wave
constexpr int kShortTagShift = 17;
constexpr uint32_t kShortCount = 0x7fffu, kShortLeft = 0x8000u, kShortTaken = 0x10000u;
static_assert(kTileThreads / 64 * kShortMostCpt * kChunk <= kShortCount && (kShortLeft | kShortTaken | kShortCount) >> kShortTagShift == 0, "a tile's count and its marks below the tag");
// bytes of one copy of a tensor's words; a tensor without elements has one, too
__host__ __device__ inline uint64_t short_copy_bytes(uint64_t tiles) { return a256(8 * (tiles ? tiles : 1)); }

// LDS of it; a thread looks at one word, so a tensor has no more tiles than that
constexpr uint32_t kShortTiles = kTileThreads;
struct ShortShared {
  static constexpr int NW = kTileThreads / 64;
  uint32_t all[NW], before[NW], state[NW], won;
  uint32_t tile[kShortTiles];   // only where tiles were left
};
// What the workgroups of a tensor tell one another.
struct ShortCounts {
  static constexpr int NW = kTileThreads / 64;
  uint64_t* words;     // the first copy of the tensor's
  uint64_t tag;
  uint32_t n_tiles, copy, own;   // copy: words from one copy to the next; own: the workgroup's tile
  uint64_t v;          // the word of tile `tid`
  uint32_t state;      // bit 0: all counts are there; bit 1: a tile was left
  uint32_t first, M;   // escapes of the tensor before a tile; all of them

  __device__ inline ShortCounts(uint64_t* at, uint64_t call, uint32_t tiles, uint32_t tile)
      : words(at), tag(call), n_tiles(tiles), copy((uint32_t)(short_copy_bytes(tiles) / 8)), own(tile), v(call), state(0), first(0), M(0) {}
  // The own word, written at the device's point of coherence before anyone of this workgroup looks at the others', as
  // often as `times` at most; meanwhile() while it is on its way.  rank() and overall() follow.
  template <typename Meanwhile>
  __device__ inline void tell_and_look(ShortShared& s, uint32_t total, uint32_t mark, uint32_t times, uint32_t tid, uint32_t wave, const Meanwhile& meanwhile) {
    if (tid < kShortCopies) st_agent(words + tid * copy + own, tag | mark | total);
    meanwhile();
    if (wave == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    bool here;
    for (;;) {
      if (tid < n_tiles) v = ld_agent(words + (own % kShortCopies) * copy + tid);
      here = __all(((v ^ tag) >> kShortTagShift) == 0);
      if (here || --times == 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    const bool left = __any((uint32_t)v & kShortLeft);
    if ((tid & 63u) == 0) s.state[wave] = (here ? 1u : 0u) | (left ? 2u : 0u);
  }
  // with a barrier
  __device__ inline void rank(ShortShared& s, uint32_t tile, uint32_t tid, uint32_t wave) {
    const uint32_t x = (uint32_t)v & kShortCount;
    const uint32_t all = wave_last(wave_incl_scan(x)), before = wave_last(wave_incl_scan(tid < tile ? x : 0u));
    if ((tid & 63u) == 0) {
      s.before[wave] = before;
      s.all[wave] = all;
    }
    lds_barrier();
    first = M = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      first += s.before[q];
      M += s.all[q];
    }
  }
  __device__ inline void overall(const ShortShared& s) {
    state = 1u;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const uint32_t x = s.state[q];
      state = (state & (x | 2u)) | (x & 2u);
    }
  }
  // whether a tile that was marked as left is this workgroup's now
  __device__ inline bool take(ShortShared& s, uint32_t tile, uint32_t told, uint32_t tid) {
    __syncthreads();
    if (tid == 0) {
      uint64_t seen = tag | kShortLeft | told;
      s.won = __hip_atomic_compare_exchange_strong(words + tile, &seen, seen | kShortTaken, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
    }
    __syncthreads();
    return s.won != 0;
  }
  // A workgroup's way through a launch: encode(tile, first) makes a tile and leaves its count in total, deliver() writes its
  // planes and stages its records, place(tile) puts those where first and M say.
  template <typename Encode, typename Deliver, typename Place>
  __device__ inline void run(ShortShared& s, uint32_t looks, const uint32_t& total, uint32_t tid, uint32_t wave, const Encode& encode, const Deliver& deliver, const Place& place) {
    encode(own, true);
    if (n_tiles > 1) {
      tell_and_look(s, total, 0u, looks, tid, wave, deliver);
    } else {   // nobody to tell
      deliver();
      if (tid == 0) v |= total;
      if ((tid & 63u) == 0) s.state[wave] = 1u;
    }
    rank(s, own, tid, wave);
    overall(s);
    if (state == 1u) {
      place(own);
      return;
    }
    bool keep = (state & 1u) != 0;
    if (!keep) {
      __syncthreads();
      tell_and_look(s, total, kShortLeft, 1u, tid, wave, [] {});
      rank(s, own, tid, wave);
      overall(s);
      if (!(state & 1u)) return;
      keep = take(s, own, total, tid);
    }
    if (keep) place(own);
    // tiles that their workgroups have left (the loop is not one with what is above: that cost 0.3 us, in registers)
    s.tile[tid] = (uint32_t)v & (kShortLeft | kShortTaken | kShortCount);
    __syncthreads();
#pragma unroll 1
    for (uint32_t tile = 0; tile < n_tiles; ++tile) {
      const uint32_t told = s.tile[tile];
      if (tile == own || !(told & kShortLeft) || (told & kShortTaken) || !take(s, tile, told & kShortCount, tid)) continue;
      encode(tile, false);
      deliver();
      rank(s, tile, tid, wave);
      place(tile);
    }
  }
};

// CPT: chunks per wave.  What a launch may not do is fill the chip: calls on other streams have theirs there (pick_short).  So one of
// more than 256 workgroups with a chunk per wave has two, at most 128 registers each: 2048 chunks 5.2 us a call with one, 5.6 with two, and
// on four streams side by side 5.4 and 2.1.
// The count is told before the planes are on
// their way: us per call with them in front of it and behind, BF16 4.87 and 4.59 (1024 chunks), E5M2 4.64 and 4.17.
// Workgroups of eight waves get onto a busy chip late, and everyone waits for them (beside
// elementwise kernels that fill it 22 to 27 us a call, 16.9 with four, two launches 20.2).  It gains most where chunks escape whole: the finishing pass encodes tiles whose
// records outgrow their slots once more, a workgroup 16 of them (2048 chunks of random words 62 us a call, 14 this way).
template <typename F, uint32_t N, int CPT>
__global__ __launch_bounds__(kTileThreads, CPT == 1 ? 1 : 4) void compress_short_kernel(const TileArgs<N> args) {
  constexpr int NW = kTileThreads / 64;
  __shared__ uint16_t lut[256];
  __shared__ uint16_t stage_pos[NW][CPT * kChunk];   // room for all of a wave's records
  __shared__ uint8_t stage_val[NW][CPT * kChunk];
  __shared__ u32x4 s_park[kTileThreads];
  __shared__ uint32_t s_cnt[NW];
  __shared__ ShortShared s_short;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t item = blockIdx.y, own = blockIdx.x;
  TileShared a;
  TileItem it;
  args_arrived(args, item, a, it);
  const Planes P = make_planes(item_words(a.paging, it.in), it.out, it.n, it.capacity, F::DT);
  const uint32_t n_tiles = (P.n_chunks + NW * CPT - 1) / (NW * CPT);
  if (own >= (n_tiles ? n_tiles : 1u)) return;   // a tensor without elements still gets its header
  ShortCounts counts(reinterpret_cast<uint64_t*>(a.status + it.status_off), a.tag, n_tiles, own);
  uint32_t* park = reinterpret_cast<uint32_t*>(&s_park[tid]);
  const LdsSink lds{stage_pos[wave], stage_val[wave], 0u, CPT * kChunk};

  uint32_t c = 0, count[CPT] = {}, mine = 0;   // the wave's first chunk, the escapes of its chunks, all of them
  uint32_t in_tile = 0, total = 0;             // escapes of the tile before the wave's chunks; all of them
  // A tile's words and counts, then, with the count told, its planes out and its records staged: the others need the one,
  // and the stores need not be over when they are looked for.
  typename F::Regs w[CPT];
  typename F::Coded coded[CPT];
  bool whole = false;                          // all chunks of the tile are complete
  auto encode = [&](uint32_t tile, bool build) {
    c = CPT * (NW * tile + wave);
    auto table = [&]() {   // while the words are on their way
      if (!build) return;
      build_encode_table(lut, a.dec16_of(it, item), tid, F::kLutShift);
      lds_barrier();
    };
    auto words_of = [&](int j) { return chunk_at<F::ES>(P.w, (uint64_t)(c + j) * kChunk, P.w.table ? page_of_wave_chunk(P.w, c + j) : 0u); };
    whole = F::full(P, (uint64_t)(CPT * NW * (tile + 1) - 1) * kChunk);
    if (whole) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) F::template load<true>(P, words_of(j), (uint64_t)(c + j) * kChunk, lane, w[j]);
      table();
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        F::template encode<true>(P, lut, (uint64_t)(c + j) * kChunk, lane, w[j], coded[j]);
        count[j] = F::count(coded[j]);
      }
    } else {
      bool full[CPT];
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const uint64_t cbase = (uint64_t)(c + j) * kChunk;
        full[j] = F::full(P, cbase);
        if (c + j < P.n_chunks) {
          const uint8_t* cptr = words_of(j);
          if (full[j]) F::template load<true>(P, cptr, cbase, lane, w[j]);
          else F::template load<false>(P, cptr, cbase, lane, w[j]);
        }
      }
      table();
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const uint64_t cbase = (uint64_t)(c + j) * kChunk;
        count[j] = 0;
        if (c + j < P.n_chunks) {
          if (full[j]) F::template encode<true>(P, lut, cbase, lane, w[j], coded[j]);
          else F::template encode<false>(P, lut, cbase, lane, w[j], coded[j]);
          count[j] = F::count(coded[j]);
        }
      }
    }
    mine = 0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) mine += count[j];
    if (lane == 0) s_cnt[wave] = mine;
    lds_barrier();
    in_tile = total = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const uint32_t x = s_cnt[q];
      in_tile += q < wave ? x : 0u;
      total += x;
    }
  };
  auto deliver = [&]() {
    uint32_t first = 0;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const uint64_t cbase = (uint64_t)(c + j) * kChunk;
      if (whole || (c + j < P.n_chunks && F::full(P, cbase))) F::template store<true>(P, cbase, lane, coded[j]);
      else if (c + j < P.n_chunks) F::template store<false>(P, cbase, lane, coded[j]);
      F::emit(park, lane, w[j], coded[j], count[j], first, lds);
      first += count[j];
    }
  };

  // the tile's records and table entries where they belong; the stream's header and pads with the first tile
  auto place = [&](uint32_t tile) {
    const uint64_t off_val = P.off_pos + a256(2ull * counts.M);
    FinalSink fin;
    fin.pos = reinterpret_cast<uint16_t*>(P.out + P.off_pos);
    fin.pos_room = room32(P.capacity, P.off_pos, 1);
    fin.val = P.out + off_val;
    fin.val_room = room32(P.capacity, off_val, 0);
    const uint32_t base = counts.first + in_tile;
    if (lane < CPT && c + lane < P.n_chunks) reinterpret_cast<uint32_t*>(P.out + P.off_tab)[c + lane] = base + (CPT > 1 && lane ? count[0] : 0u);
    for (uint32_t i = lane; i < mine; i += 64) fin.put(base + i, stage_pos[wave][i], stage_val[wave][i]);
    if (tile == 0 && wave == NW - 1) compress_write_trailer(P, a.dec16_of(it, item), a.sizes + item, counts.M, 0u, lane);
  };
  static_assert(CPT <= (int)kShortMostCpt, "the second chunk's entry is what the first holds");
  counts.run(s_short, a.looks, total, (uint32_t)tid, (uint32_t)wave, encode, deliver, place);
}

#endif  // SPLITZIP_COMPRESS_HPP
