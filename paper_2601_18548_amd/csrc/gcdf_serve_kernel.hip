// Persistent serving kernel (continuous batching of gcdf_request) for gfx950.
#include "gcdf_tile.h"

namespace gcdf {
// ----------------------------------------------------------------------------
// Persistent serving kernel.  Requests are published by the host in sequence
// order into ServeCtl (pinned host memory); every workgroup walks the sequence
// with its own cursor and claims tiles from the slot's (seq, count) word (a
// compare-and-swap re-tags it for a new request, a fetch_add hands out the
// rest), so a late workgroup can never run tiles of a request that has since
// been replaced in its slot under the wrong descriptor (descriptors are read
// seqlock-style, see desc_ntiles).  The first workgroup
// that stays idle ends the launch for all (the drain word); tiles not yet
// claimed then wait in the claim words for the next launch.
//
// Memory ordering is paid per request, not per tile: claims are relaxed; a
// workgroup acquires (system scope) once when it sees new publications; when it
// leaves a request (its next claim finds no tile left) it releases its output
// stores at agent scope once and adds the number of tiles it ran to the slot's
// done counter.  The workgroup whose addition completes the request acquires,
// decodes the per-knot minimum, restores the key scratch and publishes
// completion with a system-scope release store.  (Acquire and release at agent
// or system scope invalidate or write back the L2, which per tile would evict
// the packed weights.)
// ----------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ T sys_relaxed(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A value that is the same for the whole workgroup (read from LDS), as a scalar.
template <class T>
__device__ __forceinline__ T uniform(T v) {
  static_assert(sizeof(T) == 8, "64-bit values");
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
}

template <class T>
__device__ __forceinline__ T dev_relaxed(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A request's descriptor, field by field, with relaxed loads of the given kind.
template <class L>
__device__ __forceinline__ void load_desc(ServeDesc& o, const ServeDesc* d, uint64_t seq, L&& ld) {
  o.knots = ld(&d->knots);
  o.points = ld(&d->points);
  o.K = ld(&d->K);
  o.Np = ld(&d->Np);
  o.nblk = ld(&d->nblk);
  o.ntiles = ld(&d->ntiles);
  o.done_target = ld(&d->done_target);
  o.d = ld(&d->d);
  o.J = ld(&d->J);
  o.minkey = ld(&d->minkey);
  o.dmin = ld(&d->dmin);
  o.argmin = ld(&d->argmin);
  o.Jmin = ld(&d->Jmin);
  o.want_grad = ld(&d->want_grad);
  o.seq = seq;
}

// Device copies of the descriptors.  Every workgroup reading a request's fields from
// host memory cost a few hundred microseconds per request (256-512 workgroups times
// 18 reads over the host link, all at once), so the workgroup that claims a request's
// first tile reads them, stores this copy and then the request's number; the others
// read the copy.  A copy has one writer at a time: the next request in the slot is
// claimed only after this one has completed, which needs the writer's own tile.
// Readers check the number before and after, as with the host's descriptors.
__device__ __forceinline__ void store_copy(ServeDev* dev, uint32_t s, const ServeDesc& o) {
  __hip_atomic_store(&dev->ready[s], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // the marker before the fields
  ServeDesc* d = &dev->desc[s];
  auto put = [](auto* p, auto v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  put(&d->knots, o.knots);
  put(&d->points, o.points);
  put(&d->K, o.K);
  put(&d->Np, o.Np);
  put(&d->nblk, o.nblk);
  put(&d->ntiles, o.ntiles);
  put(&d->done_target, o.done_target);
  put(&d->d, o.d);
  put(&d->J, o.J);
  put(&d->minkey, o.minkey);
  put(&d->dmin, o.dmin);
  put(&d->argmin, o.argmin);
  put(&d->Jmin, o.Jmin);
  put(&d->want_grad, o.want_grad);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // the fields before the number
  __hip_atomic_store(&dev->ready[s], (unsigned long long)(o.seq + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool load_copy(const ServeDev* dev, uint32_t s, uint64_t want, ServeDesc& o) {
  if (dev_relaxed(&dev->ready[s]) != want + 1) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  load_desc(o, &dev->desc[s], want, [](auto* p) { return dev_relaxed(p); });
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the fields precede the re-check
  return dev_relaxed(&dev->ready[s]) == want + 1;
}

// Tile count of request `want` from its slot's descriptor, read seqlock-style:
// the descriptor's seq before and after the read must both be `want`.  Returns
// false if the slot no longer holds `want` (it has completed and the host is
// rewriting or has rewritten the slot for a later request).
__device__ __forceinline__ bool desc_ntiles(const ServeDesc* d, uint64_t want, int64_t& nt) {
  const uint64_t a = sys_relaxed(&d->seq);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // system scope: the field read follows
  nt = sys_relaxed(&d->ntiles);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // the field read precedes the re-check
  const uint64_t b = sys_relaxed(&d->seq);
  return a == want && b == want;
}

template <int W, int MODE, bool SPH>
__global__ __launch_bounds__((Geo<W, MODE>::THREADS), (Geo<W, MODE>::WGS)) void serve_loop(const DevNet net, ServeCtl* ctl, ServeDev* dev,
                                                          uint64_t first_seq, uint64_t idle_ticks, uint32_t epoch) {
  __shared__ __attribute__((aligned(16))) char lds[Geo<W, MODE>::LDS_BYTES];
  __shared__ int64_t claim_info[3];  // claimed seq (or -1: exit, -2: none), tile, seq to finalize (or -1)
  __shared__ ServeDesc cur;          // the request this workgroup is working on
  __shared__ ServeDesc nxt;          // the request it claims next, once read
  __shared__ ServeDesc fin;          // a request this workgroup completes
  __shared__ uint32_t ovf;
  TileCtx<W, MODE> tc(lds, &ovf, net, threadIdx.x);
  const int tid = threadIdx.x;
  // thread 0's view of the queue, kept in LDS between its claims: held in registers it
  // would take them from every lane of the tiles
  struct Cursor {
    uint64_t seq;         // this workgroup's place in the request sequence
    uint64_t cur_seq;     // the request in cur
    uint64_t nxt_seq;     // the request in nxt
    uint64_t pub, nt_seq;
    int64_t ntiles;
    uint64_t open_count;  // tiles of request cur_seq run here and not yet reported
    uint64_t idle_since;
    uint32_t slots;
  };
  __shared__ Cursor kept;
  if (tid == 0)
    kept = Cursor{first_seq, ~0ull, ~0ull, 0, ~0ull, 0, 0, __builtin_amdgcn_s_memrealtime(), sys_relaxed(&ctl->slots)};
  while (true) {
    if (tid == 0) {
      uint64_t nxt_seq = kept.nxt_seq;
      uint64_t seq = kept.seq, cur_seq = kept.cur_seq, pub = kept.pub, nt_seq = kept.nt_seq, open_count = kept.open_count;
      int64_t ntiles = kept.ntiles;
      const uint64_t idle_since = kept.idle_since;
      const uint32_t slots = kept.slots;
      int backoff = 1;
      // One workgroup in 64 reads the host's words each time round and passes what it
      // finds on through device memory; the others do so only now and then (all of them
      // polling host memory kept the link busy for the reads that matter).
      const bool leader = (blockIdx.x & 63) == 0;
      uint32_t idle_rounds = 0;
      int64_t got_seq = -1, got_tile = 0, fin_seq = -1;
      bool leave = false;
      // Report the tiles of request cur_seq run here (the caller has established that
      // no further tile of it will be claimed here); the report that completes the
      // request makes this workgroup its finalizer.
      auto report = [&]() {
        const uint32_t s = (uint32_t)(cur_seq % slots);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // this workgroup's stores and atomics
        const unsigned long long done =
            __hip_atomic_fetch_add(&dev->done[s], open_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + open_count;
        open_count = 0;
        if (done == cur.done_target) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // every contributor's results
          fin = cur;
          fin_seq = (int64_t)cur_seq;
        }
      };
      while (true) {
        if (__hip_atomic_load(&dev->drain, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) {
          // another workgroup ended this launch: claim nothing more
          if (open_count) report();
          leave = true;
          break;
        }
        if (seq >= pub) {
          uint64_t p = dev_relaxed(&dev->pub);
          if (p <= pub && (leader || (idle_rounds & 7) == 7)) {
            p = sys_relaxed(&ctl->published);
            if (p > pub) __hip_atomic_fetch_max(&dev->pub, (unsigned long long)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (p > pub) {
            pub = p;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // system scope: the new descriptors
          }
        }
        if (seq < pub) {
          const uint32_t s = (uint32_t)(seq % slots);
          const uint64_t s32 = seq & 0xffffffffull;
          // Claim word of the slot: (request tag << 32) | tiles handed out.  While it has
          // an older tag nobody has claimed a tile of seq, so seq cannot have completed:
          // the workgroup whose compare-and-swap re-tags the word has its tile 0 and
          // reads the host's descriptor; the others wait for its copy, and read the
          // host's themselves should it be long in coming.  (Request 0 finds its own tag,
          // and no copy.)  A swap that fails is tried again while the tag is older: an
          // add that comes late for the slot's last request changes the count alone.
          // Each failure is another workgroup's add or re-tagging, so the tries end.
          unsigned long long v = dev_relaxed(&dev->claim[s]);
          bool tagged = false;
          while (!tagged && (v >> 32) < s32)
            tagged = __hip_atomic_compare_exchange_strong(&dev->claim[s], &v, (s32 << 32) | 1ull, __ATOMIC_RELAXED,
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (tagged) {
            load_desc(nxt, &ctl->desc[s], seq, [](auto* p) { return sys_relaxed(p); });
            store_copy(dev, s, nxt);
            nt_seq = nxt_seq = seq;
            ntiles = nxt.ntiles;
            got_seq = (int64_t)seq;
            got_tile = 0;
            break;
          }
          // from here on the word's tag is s32 or newer (tags only grow)
          if (nt_seq != seq) {
            for (int tries = 0; seq != 0 && tries < 64; ++tries) {
              if (load_copy(dev, s, seq, nxt)) {
                nt_seq = nxt_seq = seq;
                ntiles = nxt.ntiles;
                break;
              }
              if ((dev_relaxed(&dev->claim[s]) >> 32) > s32) break;  // the slot has moved on
              __builtin_amdgcn_s_sleep(8);
            }
            if (nt_seq != seq) {
              // A cursor behind the others can reach a request that has completed and
              // whose slot the host has already given to a later request: the
              // descriptor then describes that later request, and its tile count must
              // not be taken for seq's.
              if (!desc_ntiles(&ctl->desc[s], seq, ntiles)) {
                if (open_count && cur_seq == seq) report();  // (none: seq is complete)
                ++seq;
                if (fin_seq >= 0) break;
                continue;
              }
              nt_seq = seq;
            }
            v = dev_relaxed(&dev->claim[s]);
          }
          // Every claim but a request's first is a fetch_add, which never has to be retried.
          bool moved_on = false;
          do {
            const uint64_t vs = v >> 32, vc = v & 0xffffffffull;
            if (vs > s32) { moved_on = true; break; }  // slot already reused: seq is complete
            if ((int64_t)vc >= ntiles) { moved_on = true; break; }
            const unsigned long long w =
                __hip_atomic_fetch_add(&dev->claim[s], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t ws = w >> 32, wc = w & 0xffffffffull;
            if (ws == s32) {
              if ((int64_t)wc < ntiles) { got_seq = (int64_t)seq; got_tile = (int64_t)wc; }
              else moved_on = true;
              break;
            }
            // Between the load and the add, request seq finished and a later request
            // took the slot: the add handed out tile wc of that request, which must be
            // run here.  Its tag is the low half of its sequence number.
            const uint64_t later = seq + ((ws - s32) & 0xffffffffull);
            // (no tiles of seq can be unreported here: seq could not have completed)
            seq = later;
            if (pub < later + 1) pub = later + 1;
            int64_t lnt = 0;
            bool held = false;
            // The request that tagged the word was published before its first claim,
            // so its descriptor is in place; a read that misses it is a visibility
            // delay, re-read (bounded).  A slot holding a newer request means `later`
            // has completed, so all its tiles were handed out: wc is past them.
            for (int tries = 0; tries < (1 << 20); ++tries) {
              const uint64_t ds = sys_relaxed(&ctl->desc[s].seq);
              if (ds != kDescWriting && ds < later) {
                __builtin_amdgcn_s_sleep(2);
                continue;
              }
              held = desc_ntiles(&ctl->desc[s], later, lnt);
              if (held || ds != later) break;
            }
            if (!held && sys_relaxed(&ctl->desc[s].seq) < later) {
              // never seen: report it to the host, which stops serving with an error
              __hip_atomic_store(&ctl->fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
              if (open_count) report();
              leave = true;
              break;
            }
            nt_seq = held ? later : ~0ull;
            ntiles = held ? lnt : 0;
            if (held && (int64_t)wc < lnt) { got_seq = (int64_t)later; got_tile = (int64_t)wc; }
            else moved_on = true;
          } while (false);
          if (got_seq >= 0 || leave) break;
          if (moved_on) {
            if (open_count && cur_seq == seq) report();  // leaving request seq
            ++seq;
            if (fin_seq >= 0) break;
          }
        } else {
          if ((leader || (idle_rounds & 7) == 7) && sys_relaxed(&ctl->stop)) {
            __hip_atomic_store(&dev->drain, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (open_count) report();  // (none expected)
            leave = true;
            break;
          }
          if (__builtin_amdgcn_s_memrealtime() - idle_since > idle_ticks) {
            // idle: end the launch for every workgroup
            __hip_atomic_store(&dev->drain, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (open_count) report();  // (none expected: every published request has been left)
            leave = true;
            break;
          }
          // idle: back off up to ~4 us between polls of host memory
          ++idle_rounds;
          for (int i = 0; i < backoff; ++i) __builtin_amdgcn_s_sleep(16);
          backoff = backoff < 8 ? 2 * backoff : 8;
        }
      }
      // -1: exit (after finalizing, if fin_seq is set), -2: nothing claimed but a request to finalize
      claim_info[0] = got_seq >= 0 ? got_seq : (fin_seq >= 0 && !leave ? -2 : -1);
      claim_info[1] = got_tile;
      claim_info[2] = fin_seq;
      if (got_seq >= 0 && (uint64_t)got_seq != cur_seq) {
        if (nxt_seq == (uint64_t)got_seq) cur = nxt;
        else load_desc(cur, &ctl->desc[got_seq % slots], (uint64_t)got_seq, [](auto* p) { return sys_relaxed(p); });
        cur_seq = (uint64_t)got_seq;
      }
      if (got_seq >= 0) ++open_count;
      kept.seq = seq;
      kept.cur_seq = cur_seq;
      kept.nxt_seq = nxt_seq;
      kept.pub = pub;
      kept.nt_seq = nt_seq;
      kept.ntiles = ntiles;
      kept.open_count = open_count;
    }
    __syncthreads();
    const int64_t gs = claim_info[0];
    if (claim_info[2] >= 0) {
      // this workgroup completed request fin.seq: per-knot minimum, key scratch restored
      if (fin.dmin) {
        for (int64_t k = tid; k < fin.K; k += Geo<W, MODE>::THREADS) {
          float dm;
          int32_t am;
          minkey_decode(__hip_atomic_load(fin.minkey + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), dm, am);
          fin.dmin[k] = dm;
          fin.argmin[k] = am;
          fin.minkey[k] = 0ull;
        }
      }
      if (fin.Jmin) {
        // J at the argmin pairs (knot k, point argmin[k]): the pair-list tiles of
        // gcdf_query's Jmin pass, run by this workgroup
        __threadfence();
        __syncthreads();  // every argmin written above is visible to the workgroup
        Job pj{};
        pj.knots = uniform(fin.knots);
        pj.points = uniform(fin.points);
        pj.K = uniform(fin.K);
        pj.Np = uniform(fin.Np);
        pj.pidx32 = uniform(fin.argmin);
        pj.npairs = pj.K;
        pj.J = uniform(fin.Jmin);
        for (int64_t q0 = 0; q0 < pj.K; q0 += kTileQ) {
          // (an opaque tile start: as an induction variable, a lane's offset into J was
          // spilled at the end of the tile's prologue while only wave 0 was active, and
          // the other waves reloaded what had never been stored)
          int64_t q = q0;
          asm volatile("" : "+s"(q));
          process_tile<W, MODE, 2, true, true, false, false, SPH>(net, pj, 0, q, tc);
        }
      }
      __threadfence_system();
      __syncthreads();
      if (tid == 0)
        __hip_atomic_store(&ctl->complete[fin.seq % kept.slots], fin.seq + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (gs == -1) break;
    if (gs < 0) continue;
    const int64_t t = uniform(claim_info[1]), nblk = uniform(cur.nblk);
    Job job{};
    job.knots = uniform(cur.knots);
    job.points = uniform(cur.points);
    job.K = uniform(cur.K);
    job.Np = uniform(cur.Np);
    job.d = uniform(cur.d);
    job.J = uniform(cur.J);
    job.minkey = uniform(cur.minkey);
    const int64_t kk = t / nblk;
    const int64_t q0 = (t - kk * nblk) * kTileQ;
    if (cur.want_grad) process_tile<W, MODE, 2, true, false, false, false, SPH, true>(net, job, kk, q0, tc);
    else process_tile<W, MODE, 2, false, false, false, false, SPH, true>(net, job, kk, q0, tc);
    __syncthreads();  // every wave's stores are done before thread 0 may report the tile
    if (tid == 0) kept.idle_since = __builtin_amdgcn_s_memrealtime();
  }
  report_overflow<W, MODE, 2>(net, tc);
}

template <int W, int MODE, bool SPH>
static hipError_t launch_serve_t(const DevNet& net, ServeCtl* ctl, ServeDev* dev, uint64_t first_seq,
                                 uint64_t idle_ticks, uint32_t epoch, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL((serve_loop<W, MODE, SPH>), dim3(num_cu * Geo<W, MODE>::WGS), dim3((Geo<W, MODE>::THREADS)), 0, s, net, ctl, dev, first_seq, idle_ticks,
                     epoch);
  return hipGetLastError();
}

template <bool SPH>
static hipError_t launch_serve_k(const DevNet& net, ServeCtl* ctl, ServeDev* dev, uint64_t first_seq,
                                 uint64_t idle_ticks, uint32_t epoch, int num_cu, hipStream_t s) {
  if (net.width == 256) {
    switch (net.mode) {
      case kFP32: return launch_serve_t<256, kFP32, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
      case kBF16: return launch_serve_t<256, kBF16, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
      case kBF16X2F16: return launch_serve_t<256, kBF16X2F16, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
      default: return launch_serve_t<256, kBF16X2, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
    }
  }
  switch (net.mode) {
    case kFP32: return launch_serve_t<512, kFP32, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
    case kBF16: return launch_serve_t<512, kBF16, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
    case kBF16X2F16: return launch_serve_t<512, kBF16X2F16, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
    default: return launch_serve_t<512, kBF16X2, SPH>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
  }
}

hipError_t launch_serve(const DevNet& net, ServeCtl* ctl, ServeDev* dev, uint64_t first_seq, uint64_t idle_ticks,
                        uint32_t epoch, int num_cu, hipStream_t s) {
  return net.in_dim == kInDimSphere ? launch_serve_k<true>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s)
                                    : launch_serve_k<false>(net, ctl, dev, first_seq, idle_ticks, epoch, num_cu, s);
}


}  // namespace gcdf
