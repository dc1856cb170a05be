// SplitZip for MI355X: calibration histogram, workspace initialisation and the plain streaming kernel used as a measurement aid.
// Part of the single translation unit splitzip.hip (included inside its anonymous namespace).
#ifndef SPLITZIP_AUX_KERNELS_HPP
#define SPLITZIP_AUX_KERNELS_HPP

// ---------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------

// Calibration histogram (section 3.3) of a device sample: exponent counts, added to hist[256].
// Every workgroup counts into 64 copies of the bins in LDS, one per lane, interleaved: the count of bin b in
// the copy of lane l is word 64 b + l, so a lane only ever touches its own bank and no two lanes of a wave an
// address in common, whatever they count.  (Eight copies in rows of 256 words, the first version, sent all
// lanes that count the same exponent -- most of them, the distribution being what it is -- to one bank: 39 % of
// the LDS cycles were conflict cycles.)  The waves of a workgroup share the copies, hence atomic adds.
// Workgroup wg of the n_wgs that share the sample; they begin at its vector `start` (below their number) and go round.
// began(): when the bins are clear; counted(): when a wave has counted what it has; sum(bin, c): the workgroup's count of every bin
// of the format, by one thread each.
template <bool BF16, typename Began, typename Counted, typename Sum>
__device__ inline void histogram_body(const uint8_t* in, uint64_t n, uint32_t wg, uint32_t n_wgs, uint32_t start, const Began& began, const Counted& counted, const Sum& sum) {
  constexpr int BINS = BF16 ? 256 : 32;
  __shared__ __attribute__((aligned(16))) uint32_t bins[BINS * 64];
  const int tid = threadIdx.x;
  for (int i = tid; i < BINS * 16; i += 1024) reinterpret_cast<u32x4*>(bins)[i] = u32x4{0u, 0u, 0u, 0u};
  lds_barrier();
  began();
  uint32_t* mine = bins + (tid & 63);
  const uint64_t bytes = n * (BF16 ? 2 : 1), nvec = bytes / 16;
  const u32x4* v = reinterpret_cast<const u32x4*>(in);
  auto count = [&](const u32x4& q) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (BF16) {
        atomicAdd(&mine[((w[d] >> 7) & 0xffu) * 64], 1u);
        atomicAdd(&mine[((w[d] >> 23) & 0xffu) * 64], 1u);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) atomicAdd(&mine[((w[d] >> (8 * j + 2)) & 31u) * 64], 1u);
      }
    }
  };
  // four vectors per thread in flight: the loads of a step are all issued before the first is counted
  const uint64_t step = (uint64_t)n_wgs * 1024;
  const auto from_to_end = [&](const auto& at) {
    uint64_t i = wg * 1024ull + tid;
    for (; i + 3 * step < nvec; i += 4 * step) {
      u32x4 q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = ld_stream(at(i + u * step));
#pragma unroll
      for (int u = 0; u < 4; ++u) count(q[u]);
    }
    for (; i < nvec; i += step) count(ld_stream(at(i)));
  };
  if (start) {
    from_to_end([&](uint64_t i) {
      const uint32_t p = (uint32_t)i + start;   // a sample has fewer than 2^30 vectors
      return v + (p < (uint32_t)nvec ? p : p - (uint32_t)nvec);
    });
  } else {
    from_to_end([&](uint64_t i) { return v + i; });
  }
  // the words behind the last whole vector, by workgroup 0
  if (wg == 0) {
    for (uint64_t i = nvec * 16 + (uint64_t)tid * (BF16 ? 2 : 1); i < bytes; i += 1024 * (BF16 ? 2 : 1)) {
      const uint32_t e = BF16 ? ((uint32_t)(in[i] | (in[i + 1] << 8)) >> 7) & 0xffu : ((uint32_t)in[i] >> 2) & 31u;
      atomicAdd(&mine[e * 64], 1u);
    }
  }
  counted();
  __syncthreads();
  // four threads per bin, sixteen copies each
  if (tid < 4 * BINS) {
    const uint32_t bin = (uint32_t)tid >> 2, q = (uint32_t)tid & 3u;
    uint32_t c = 0;   // a workgroup counts fewer than 2^32 words
#pragma unroll
    for (uint32_t r = 0; r < 16; ++r) c += bins[bin * 64 + ((16 * q + r + bin) & 63u)];   // bin b starts at copy b: the lanes' reads spread over the banks
    c += (uint32_t)__shfl_xor((int)c, 1);
    c += (uint32_t)__shfl_xor((int)c, 2);
    if (q == 0) sum(bin, c);
  }
}

template <bool BF16>
__global__ __launch_bounds__(1024) void histogram_kernel(const uint8_t* in, uint64_t n, uint64_t* hist) {
  histogram_body<BF16>(in, n, blockIdx.x, gridDim.x, 0, [] {}, [] {}, [=](uint32_t bin, uint32_t c) {
    if (c) atomicAdd(reinterpret_cast<unsigned long long*>(&hist[bin]), (unsigned long long)c);   // non-zero totals go to the global bins
  });
}

// Section 3.3 on the device: the three tables from 256 exponent counts, one thread of a workgroup of 1024 with each (count: of
// exponent threadIdx.x, for the first 256); four threads rank exponent v by (count descending,
// exponent ascending) among the format's exponents, a quarter of them each, the 16 first ranks form the codebook.
// Bound by the compares of one CU: with counts below 2^31, as good as always, they are 32 bits wide (9.5 us a launch
// with 64-bit ones, 5 with these).  The tables leave as whole words.
constexpr uint32_t kBookWords = sizeof(splitzip_codebook) / 4;
__device__ inline void write_codebook(uint64_t count, uint32_t n_values, uint32_t dtype, splitzip_codebook* cb) {
  __shared__ uint64_t h[256];
  __shared__ __attribute__((aligned(16))) uint32_t h2[256];   // twice the count, and one
  __shared__ uint32_t s_tab[kBookWords];
  static_assert(sizeof(splitzip_codebook) == 532 && offsetof(splitzip_codebook, enc) == 16 && offsetof(splitzip_codebook, member) == 272, "tables as words");
  const uint32_t tid = threadIdx.x;
  bool wide = false;
  if (tid < 256) {
    const uint64_t c = tid < n_values ? count : 0;
    h[tid] = c;
    h2[tid] = ((uint32_t)c << 1) + 1u;
    wide = c >> 31;
  }
  if (tid < kBookWords) s_tab[tid] = tid == 132 ? dtype : 0u;
  const bool any_wide = __syncthreads_or(wide) != 0;
  const uint32_t v = tid >> 2, part = tid & 3u, each = n_values / 4;   // n_values is 256 or 32
  uint32_t rank = 0;
  if (!any_wide) {
    // another exponent comes first if its count is larger (2 c + 1 > 2 mine + 1), or equal and it is smaller (2 c + 1 > 2 mine for
    // those below): two instructions each; those of v's own four that are below v and equal are added behind the loop
    const uint32_t mine = h2[v];
#pragma unroll 4
    for (uint32_t i = 0; i < each / 4; ++i) {
      const uint32_t u = 4 * (4 * i + part);   // the four threads read 16 bytes each side by side
      const u32x4 c = *reinterpret_cast<const u32x4*>(&h2[u]);
      const uint32_t limit = mine - (u + 4 <= v ? 1u : 0u);
      rank += (c.x > limit ? 1u : 0u) + (c.y > limit ? 1u : 0u) + (c.z > limit ? 1u : 0u) + (c.w > limit ? 1u : 0u);
    }
    if (part == ((v >> 2) & 3u)) {
#pragma unroll
      for (uint32_t j = 0; j < 3; ++j) rank += j < (v & 3u) && h2[(v & ~3u) + j] == mine ? 1u : 0u;
    }
  } else {
    const uint64_t mine = h[v];
    for (uint32_t i = 0; i < each; ++i) {
      const uint32_t u = 4 * i + part;
      rank += (h[u] > mine || (h[u] == mine && u < v)) ? 1u : 0u;
    }
  }
  rank += (uint32_t)__shfl_xor((int)rank, 1);
  rank += (uint32_t)__shfl_xor((int)rank, 2);
  uint8_t* tab = reinterpret_cast<uint8_t*>(s_tab);
  if (part == 0 && v < n_values && rank < 16) {
    tab[rank] = (uint8_t)v;
    tab[16 + v] = (uint8_t)rank;
    tab[272 + v] = 1;
  }
  __syncthreads();
  if (tid < kBookWords) reinterpret_cast<uint32_t*>(cb)[tid] = s_tab[tid];
}

// one workgroup per codebook (workgroup b: counts hist + 256 b, tables cb + b)
__global__ __launch_bounds__(1024) void codebook_kernel(const uint64_t* hist, uint32_t n_values, uint32_t dtype, splitzip_codebook* cb) {
  write_codebook(threadIdx.x < 256 ? hist[256 * blockIdx.x + threadIdx.x] : 0, n_values, dtype, cb + blockIdx.x);
}

__global__ void zero_words_kernel(uint64_t* p, uint64_t nwords) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < nwords; i += (uint64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// Calibration of several samples in one launch: the workgroups [first[k], first[k + 1]) count sample k.
// As many workgroups as the chip has CUs, dealt out by the samples' lengths: a workgroup has 64 KB of bins to clear and
// to add up, and a CU that streams for one workgroup reads faster than for two (64 BF16 tensors of 8 MiB: 82 us with
// one workgroup per CU, 103-107 us with two, in one round or in two).
constexpr uint32_t kHistMost = 64;          // samples of a launch
constexpr uint32_t kHistMostShort = 160;    // the same where they are short
template <uint32_t N>
struct HistBatchArgs {
  uint64_t tag;                    // of this call, see calibrate_batch_kernel
  const uint8_t* in[N];
  uint64_t n[N];
  uint32_t start[N];       // see histogram_start
  uint32_t first[N + 1];   // behind the last sample: its end, up to the last entry
  // the last sample that starts at or before workgroup wg
  __device__ inline uint32_t sample_of(uint32_t wg) const {
    uint32_t k = 0;
#pragma unroll
    for (uint32_t step = N <= 64 ? 32 : 128; step; step >>= 1)
      if (k + step <= N && first[k + step] <= wg) k += step;
    return k;
  }
};
// The vector that the workgroups of sample k (of nvec vectors) begin at.  Samples that begin a multiple of 1 MiB apart
// (equal lengths that are powers of two, allocations of their own) would be read in step, all of them at the same place of
// their MiB: each of those starts 17 KB further in than the one before it, up to 256 KB.  us per call from the start and
// this way: E5M2 8 of 16 MiB 31.4-34.7 and 30.5, 64 of 4 MiB 55.6 and 51.3; BF16 16 of 16 MiB 57.0 and 52.8.  (Others gain
// nothing by it: 100 of 1999 KiB read that way and then compressed and decompressed 197 us, 195 without.)
inline uint32_t histogram_start(const void* first, const void* in, uint32_t k, uint64_t nvec) {
  const bool in_step = ((reinterpret_cast<uintptr_t>(in) - reinterpret_cast<uintptr_t>(first)) & ((1u << 20) - 1u)) == 0;
  return in_step && nvec >= 4096 ? (k * 1088u) & (nvec < 16384 ? 4095u : 16383u) : 0u;
}
// Samples with many workgroups each: the counts alone, added to bins that a launch in front has cleared.
template <bool BF16>
__global__ __launch_bounds__(1024) void histogram_batch_kernel(const HistBatchArgs<kHistMost> a, uint64_t* hists) {
  const uint32_t k = a.sample_of(blockIdx.x);
  uint64_t* hist = hists + 256 * k;
  histogram_body<BF16>(a.in[k], a.n[k], blockIdx.x - a.first[k], a.first[k + 1] - a.first[k], a.start[k], [] {}, [] {}, [=](uint32_t bin, uint32_t c) {
    if (c) atomicAdd(reinterpret_cast<unsigned long long*>(&hist[bin]), (unsigned long long)c);
  });
}

// Counts, hists + 256 k, and codebook of sample k from its workgroups.  One alone writes its sums and ranks them.  Several add
// theirs to the global bins, which one of them clears, and the last to have added ranks them.  Who does what is settled in a word
// among the membership flags of the codebook to be, kCtlReady and the workgroups that have added under the call's tag:
// whoever first sees no tag of this call there puts it there, clears the bins and says so when it has counted, and nobody
// adds before that.  (It is running and waits for nobody, so the wait for it ends.)  In the end the word is overwritten with
// flags, bytes of 0 and 1, which are no tag: its first bit is set.  Calls that overlap on the same outputs leave nothing of
// use in them, but they end: a workgroup waits only while the word bears its own call's tag without kCtlReady, and whoever puts
// a tag there has yet to look whether it is to add kCtlReady to it.  (By compare and exchange, as the tag: where the codebooks
// are host memory, that is what the bus can do.)
// Clearing by a launch in front, and ranking by one behind, made a call three launches.  us per call, BF16, then and now: 64
// chunks 10.6 and 8.3, 1024 10.8 and 8.8, 64 samples of two 10.9 and 6.1, 64 of 100 12.0 and 10.4, 64 of 4096 88.5 and 86.5; E5M2 64 of 20 10.8 and
// 5.1, 64 of 4096 50.2 and 48.7.
constexpr int kCtlTagShift = 17;
constexpr uint64_t kCtlReady = 1u << 16, kCtlTag = 1ull << 63;
__host__ __device__ inline bool ctl_waits(uint64_t word, uint64_t tag) { return ((word ^ tag) >> kCtlTagShift) == 0 && !(word & kCtlReady); }
template <bool BF16, uint32_t N>
__global__ __launch_bounds__(1024) void calibrate_batch_kernel(const HistBatchArgs<N> a, uint64_t* hists, splitzip_codebook* cbs) {
  __shared__ uint64_t s_count[256];
  __shared__ uint32_t s_last;
  const uint32_t k = a.sample_of(blockIdx.x);
  const uint32_t n_wgs = a.first[k + 1] - a.first[k];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  uint64_t* hist = hists + 256 * k;
  splitzip_codebook* cb = cbs + k;
  uint64_t* ctl = reinterpret_cast<uint64_t*>((reinterpret_cast<uintptr_t>(cb) + offsetof(splitzip_codebook, member) + 7) & ~(uintptr_t)7);
  const bool several = n_wgs > 1, minds = several && tid >= 960;   // the last wave minds the word
  bool clears = false;
  if (tid < 256) s_count[tid] = 0;
  histogram_body<BF16>(
      a.in[k], a.n[k], blockIdx.x - a.first[k], n_wgs, a.start[k],
      [&] {
        if (!minds) return;
        if (lane == 0) {
          uint64_t seen = ld_agent(ctl);
          clears = ((seen ^ a.tag) >> kCtlTagShift) != 0 &&
                   __hip_atomic_compare_exchange_strong(ctl, &seen, a.tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        clears = __any(clears);
        if (clears) {
#pragma unroll
          for (uint32_t q = 0; q < 4; ++q) st_agent(hist + 64 * q + lane, (uint64_t)0);
        }
      },
      [&] {
        if (!minds) return;
        if (clears) {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the bins are clear
          if (lane == 0) {
            uint64_t seen = a.tag;   // what it has put there
            while (!__hip_atomic_compare_exchange_strong(ctl, &seen, seen | kCtlReady, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &&
                   ctl_waits(seen, a.tag)) {}
          }
        }
        while (ctl_waits(ld_agent(ctl), a.tag)) __builtin_amdgcn_s_sleep(1);
      },
      [&](uint32_t bin, uint32_t c) {
        if (!several) s_count[bin] = c;
        else if (c) atomicAdd(reinterpret_cast<unsigned long long*>(&hist[bin]), (unsigned long long)c);
      });
  if (several) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what this wave has added
    __syncthreads();
    if (tid == 0) s_last = (__hip_atomic_fetch_add(ctl, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kCtlReady - 1)) == n_wgs - 1 ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
  } else {
    __syncthreads();
    if (tid < 256) hist[tid] = s_count[tid];
  }
  write_codebook(tid < 256 ? several ? ld_agent(hist + tid) : s_count[tid] : 0, BF16 ? 256u : 32u, BF16 ? SPLITZIP_BF16 : SPLITZIP_FP8_E5M2, cb);
}

__global__ void workspace_init_kernel(uint32_t* p, uint32_t nwords) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += gridDim.x * blockDim.x) p[i] = i == 0 ? 1u : 0u;
}

// Per step a workgroup reads four coalesced 4 KB runs and writes three: the codec's 4:3 traffic
// without its arithmetic.
__global__ __launch_bounds__(kThreads) void traffic_probe_kernel(const u32x4* src, uint64_t nread,
                                                                  u32x4* dst, uint64_t nwrite) {
  const uint64_t steps = (nread + 4 * kThreads - 1) / (4 * kThreads);
  for (uint64_t s = blockIdx.x; s < steps; s += gridDim.x) {
    u32x4 v[4];
    // a step inside both buffers runs without a condition per access: all its loads are on their way before the
    // first is waited for, and its stores follow one another without a wait in between
    const bool whole = (4 * (s + 1)) * kThreads <= nread && (3 * (s + 1)) * kThreads <= nwrite;
    if (whole) {
      const u32x4* sp = src + 4 * s * kThreads + threadIdx.x;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = ld_stream(sp + i * kThreads);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t idx = (4 * s + i) * kThreads + threadIdx.x;
        v[i] = idx < nread ? ld_stream(src + idx) : u32x4{0u, 0u, 0u, 0u};
      }
    }
    v[0].x ^= v[3].x; v[1].y ^= v[3].y; v[2].z ^= v[3].z; v[0].w ^= v[3].w;
    if (whole) {
      u32x4* dp = dst + 3 * s * kThreads + threadIdx.x;
#pragma unroll
      for (int i = 0; i < 3; ++i) st_stream(dp + i * kThreads, v[i]);
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const uint64_t idx = (3 * s + i) * kThreads + threadIdx.x;
        if (idx < nwrite) st_stream(dst + idx, v[i]);
      }
    }
  }
}

// The same with its shape as arguments, for finding out what the memory system gives a streaming kernel at best:
// per step a workgroup reads R coalesced 4 KB runs and writes W (either may be 0: write only, read only), with
// temporal or non-temporal accesses; the steps are dealt to the workgroups round robin (neighbouring workgroups
// work on neighbouring runs) or in one contiguous block each (the way the codec's kernels own their chunks).
template <int R, int W, bool NTL, bool NTS>
__global__ __launch_bounds__(kThreads) void traffic_shape_kernel(const u32x4* src, uint64_t nread, u32x4* dst, uint64_t nwrite,
                                                                  uint64_t steps, uint32_t blocked_in) {
  const uint32_t blocked = blocked_in & 3u;
  const bool blocked_narrow = (blocked_in & 4u) != 0;
  const uint64_t per = (steps + gridDim.x - 1) / gridDim.x;
  const uint64_t s0 = blocked ? blockIdx.x * per : blockIdx.x;
  const uint64_t s_end = blocked ? (s0 + per < steps ? s0 + per : steps) : steps, stride = blocked ? 1 : gridDim.x;
  // blocked == 2: every workgroup starts somewhere else inside its block and wraps around, so that the workgroups
  // are not all at the same distance from the start of their blocks at the same time
  const uint64_t len = s_end > s0 ? s_end - s0 : 0, rot = blocked == 2 && len ? (blockIdx.x * 37ull) % len : 0;
  u32x4 acc = u32x4{0u, 0u, 0u, 0u};
  // blocked == 3: the steps are handed out in order through a counter (the word behind the written bytes, zeroed
  // by the caller): the next step's number is fetched while this step's runs are on their way
  __shared__ uint32_t s_ticket[2];
  uint32_t* counter = reinterpret_cast<uint32_t*>(dst + nwrite);
  uint64_t tk = 0;
  if (blocked == 3) {
    if (threadIdx.x == 0) s_ticket[0] = atomicAdd(counter, 1u);
    __syncthreads();
    tk = s_ticket[0];
  }
  for (uint64_t q = 0; blocked == 3 ? tk < steps : s0 + q * stride < s_end; ++q) {
    const uint64_t s = blocked == 3 ? tk : blocked == 2 ? s0 + (q + rot) % len : s0 + q * stride;
    if (blocked == 3) {
      if (threadIdx.x == 0) s_ticket[(q + 1) & 1] = atomicAdd(counter, 1u);
      __syncthreads();
      tk = s_ticket[(q + 1) & 1];
    }
    u32x4 v[R > 0 ? R : 1];
    v[0] = u32x4{(uint32_t)s, threadIdx.x, 0u, 0u};
    // A step that lies inside both buffers entirely (all but the last, as a rule) runs without a condition per
    // access: every load of the step is on its way before the first is waited for, and so is every store.
    const bool whole = (R == 0 || ((uint64_t)R * (s + 1)) * kThreads <= nread) && (W == 0 || ((uint64_t)W * (s + 1)) * kThreads <= nwrite);
    if (whole) {
      const u32x4* sp = src + (uint64_t)R * s * kThreads + threadIdx.x;
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = NTL ? ld_stream(sp + i * kThreads) : sp[i * kThreads];
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const uint64_t idx = ((uint64_t)R * s + i) * kThreads + threadIdx.x;
        v[i] = u32x4{0u, 0u, 0u, 0u};
        if (idx < nread) v[i] = NTL ? ld_stream(src + idx) : src[idx];
      }
    }
    if (W == 0) {
#pragma unroll
      for (int i = 0; i < R; ++i) acc ^= v[i];
    }
    if (blocked_narrow) {
      // the codec's store shapes: two thirds of the step's bytes as 8-byte stores, one third as 4-byte stores
      if (W == 3 && whole) {
        uint8_t* base = reinterpret_cast<uint8_t*>(dst + (uint64_t)W * s * kThreads);
#pragma unroll
        for (int i = 0; i < 4; ++i) st_stream(reinterpret_cast<u32x2*>(base) + i * kThreads + threadIdx.x, u32x2{v[i % (R > 0 ? R : 1)].x, v[i % (R > 0 ? R : 1)].y});
#pragma unroll
        for (int i = 0; i < 4; ++i) st_stream(reinterpret_cast<uint32_t*>(base + 8192) + i * kThreads + threadIdx.x, v[i % (R > 0 ? R : 1)].z);
      }
      continue;
    }
    if (whole) {
      u32x4* dp = dst + (uint64_t)W * s * kThreads + threadIdx.x;
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const u32x4 o = v[R > 0 ? i % R : 0];
        if (NTS) st_stream(dp + i * kThreads, o);
        else dp[i * kThreads] = o;
      }
    } else {
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const uint64_t idx = ((uint64_t)W * s + i) * kThreads + threadIdx.x;
        const u32x4 o = v[R > 0 ? i % R : 0];
        if (idx < nwrite) {
          if (NTS) st_stream(dst + idx, o);
          else dst[idx] = o;
        }
      }
    }
  }
  // read only: the words must be used; no tensor holds this pattern in every lane
  if (W == 0 && acc.x == 0x5a17c0deu && acc.y == 0x5a17c0deu && acc.z == 0x5a17c0deu && acc.w == 0x5a17c0deu) dst[0] = acc;
}

#endif  // SPLITZIP_AUX_KERNELS_HPP
