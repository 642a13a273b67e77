// Keypoint bookkeeping after tracking (Sec. III-B/III-D): cell mask, global
// cap, new identifiers, stable compaction of the surviving tracks, acceptance
// of stereo matches and the output records TR_t / DET_t, written straight
// into mapped pinned host memory (the host reads them after the frame's wait,
// with no copy).
//
// One 1024-thread workgroup per camera group (a mono camera, a stereo pair, a
// star rig). A selection is a chain of memory round trips and barriers, so what
// does not depend on earlier steps (keys, the previous keypoints and their
// results) is loaded at the start. Identifiers are assigned in (group, cell)
// order: a stream's groups hand the next free one on as soon as they know how
// many detections they take. Every ordering decision is a prefix count over
// flags (wave ballots plus a scan of the 16 wave totals), so the result does not
// depend on thread timing. Mono 320x240 (200 keypoints, 300 cells) 5.9 -> 5.1
// us, a pair of 300 8.9 -> 8.5, a four-camera rig of 6,000 (two pairs, one after
// the other before) 40 -> 24. What is left is the chain: records laid out in LDS
// and stored in whole lines took 5.6, 9.3 and 25.
//
// Rules (all on integers):
//  * a cell is masked when it holds at least k surviving tracks of the camera;
//  * the candidates are the (up to k) winners of the unmasked cells, in key
//    slots cell * k + rank; the best (score desc, cell asc, rank asc) up to
//    cap - live are kept, found with a 256-bin score histogram instead of a
//    sort (equal scores are taken in slot order);
//  * the kept ones get consecutive identifiers in slot (cell, rank) order;
//  * a stereo match is accepted while the right camera has room.
//
// Phases: kSelectAll reads the speculative stereo match of every selected
// winner (indexed by key slot). With deferred stereo matching the work splits in
// two launches around the stereo tracking launch: kSelectLeft does
// everything except the right cameras' matches and leaves the new detections'
// place in the left state in sel_base / n_sel; kSelectRight accepts the
// matches (indexed by selection rank) into the right cameras.
#include "fe_common.h"
#include "group_order.h"
#include "wave_ops.h"

namespace vio {

constexpr int kMaxCells = 8192;

namespace {

constexpr int kWaves = kSelectThreads / 64;

// group_order.h's memory: device-scope atomics (only the values themselves are
// passed on), and a wave that waits.
struct AgentMem {
  static __device__ __forceinline__ int32_t add(int32_t* p, int32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  template <class T>
  static __device__ __forceinline__ T load(T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  template <class T>
  static __device__ __forceinline__ void store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
};

struct ScanScratch {
  int wave_tot[2][kWaves];
};

// A thread's handle on the block's scan scratch. Every thread makes the same
// sequence of scan calls, so `tog` agrees across the block.
struct Scan {
  ScanScratch* sh;
  int tog;
};

// Exclusive prefix count of `flag` over the block's threads in thread order;
// returns the thread's offset and sets `total`. All threads must call it.
// One barrier per call: the wave totals alternate between two buffers, and a
// buffer is rewritten two calls later, which a thread reaches only after the
// next call's barrier, i.e. after every thread has read this call's totals.
// Two flags with one barrier: the prefix count of `flag` and both totals (a
// wave's two counts share one word).
__device__ __forceinline__ int block_scan_flag2(bool flag, bool flag2, Scan& sc, int& total, int& total2) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long m = __ballot(flag), m2 = __ballot(flag2);
  const int below = __popcll(m & ((1ull << lane) - 1ull));
  int* tot = sc.sh->wave_tot[sc.tog];
  sc.tog ^= 1;
  if (lane == 0) tot[wave] = __popcll(m) | (__popcll(m2) << 16);
  __syncthreads();
  int off = 0, all = 0, all2 = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = tot[w];
    off += w < wave ? (t & 0xFFFF) : 0;
    all += t & 0xFFFF;
    all2 += t >> 16;
  }
  total = all;
  total2 = all2;
  return off + below;
}

__device__ __forceinline__ int block_scan_flag(bool flag, Scan& sc, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long m = __ballot(flag);
  const int below = __popcll(m & ((1ull << lane) - 1ull));
  int* tot = sc.sh->wave_tot[sc.tog];
  sc.tog ^= 1;
  if (lane == 0) tot[wave] = __popcll(m);
  __syncthreads();
  int off = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = tot[w];
    off += w < wave ? t : 0;
    all += t;
  }
  total = all;
  return off + below;
}



__device__ __forceinline__ vio_track make_rec(int64_t id, int cam, int status, float x, float y, float th, float fb,
                                              float res, int age, int score) {
  vio_track t;
  t.id = id;
  t.x = x;
  t.y = y;
  t.theta = th;
  t.fb_err = fb;
  t.resid_rms = res;
  t.age = age;
  t.camera = (int16_t)cam;
  t.status = (int16_t)status;
  t.score = score;
  return t;
}

__device__ __forceinline__ Kp make_kp(int64_t id, float x, float y, float px, float py, int age) {
  Kp k;
  k.id = id;
  k.x = x;
  k.y = y;
  k.px = px;
  k.py = py;
  k.age = age;
  k.reserved = 0;
  return k;
}

// A live keypoint's id and position, kept in LDS for the neighbour stereo
// start's pair table while the selection writes the state.
struct PairRow {
  int64_t id;
  float x, y;
};
constexpr int kPairLds = 1024;  // rows per camera kept in LDS (cameras of larger caps read global memory)

// A camera's previous keypoint and its tracking result.
struct PrevRow {
  Kp kp;
  TrackRes r;
};
// Row j of `cd` (j < cap; garbage past the camera's live rows).
__device__ __forceinline__ PrevRow load_row(const CamDesc& cd, const FrameCam& fc, int j) {
  PrevRow p{};
  if (j < cd.cap) {
    p.kp = cd.state[fc.parity ^ 1][j];
    if (fc.has_prev) {
      // a short attempt that was not kept: its fallback, computed beside it
      // (both results loaded at once, so the choice costs no second round
      // trip; the fallback slot of a kept track is not used)
      p.r = cd.res[j];
      if (cd.res_fb) {
        const TrackRes rf = cd.res_fb[j];
        if (p.r.pad[0] != 0) p.r = rf;
      }
    } else {
      p.r.x = p.kp.x;
      p.r.y = p.kp.y;
    }
  }
  return p;
}

// Carries camera c's previous keypoints into its current state: the survivors
// of temporal tracking (all of them when there was no previous frame) in their
// old order, with their records. Adds the survivors to `occ` when given, and
// their ids and positions to `tab` when given. `row`: this thread's first row.
// Returns the survivor count; *n_rec receives the number of records written.
__device__ __forceinline__ int carry_survivors(const CamDesc& cd, const FrameCam& fc, int n_prev, PrevRow row,
                                               unsigned* occ, Scan& sc, int* n_rec, bool count_fallback,
                                               PairRow* tab = nullptr, int64_t* tab_ids = nullptr) {
  const int P = fc.parity;
  int base = 0, n_fb = 0;
  for (int j0 = 0; j0 < n_prev; j0 += kSelectThreads) {
    const int j = j0 + (int)threadIdx.x;
    if (j0 > 0) row = load_row(cd, fc, j);
    const Kp kp = row.kp;
    const TrackRes r = row.r;
    const bool alive = j < n_prev && (!fc.has_prev || r.status == VIO_TRACKED);
    int total, fb_tot;
    const int pos = base + (count_fallback ? block_scan_flag2(alive, j < n_prev && fc.has_prev && r.pad[0] != 0, sc,
                                                              total, fb_tot)
                                           : block_scan_flag(alive, sc, total));
    if (count_fallback) n_fb += fb_tot;
    if (j < n_prev) {
      if (alive) {
        if (occ) {
          const int cx = (int)floorf(r.x / (float)cd.cell), cy = (int)floorf(r.y / (float)cd.cell);
          if (cx >= 0 && cx < cd.ncx && cy >= 0 && cy < cd.ncy) atomicAdd(&occ[cy * cd.ncx + cx], 1u);
        }
        cd.state[P][pos] = fc.has_prev ? make_kp(kp.id, r.x, r.y, kp.x, kp.y, kp.age + 1) : kp;
        if (tab) tab[pos] = PairRow{kp.id, fc.has_prev ? r.x : kp.x, fc.has_prev ? r.y : kp.y};
        if (tab_ids) tab_ids[pos] = kp.id;
      }
      if (fc.has_prev)
        cd.rec[fc.rec_slot][j] = make_rec(kp.id, cd.local, r.status, r.x, r.y, r.theta, r.fb, r.resid,
                             alive ? kp.age + 1 : kp.age, -1);
    }
    base += total;
  }
  *n_rec = fc.has_prev ? n_prev : 0;
  if (threadIdx.x == 0) {
    int32_t* st = cd.stats_out[fc.rec_slot];
    st[kStatFallback] = n_fb;
    st[kStatTracked] = fc.has_prev ? base : 0;
    st[kStatLost] = fc.has_prev ? n_prev - base : 0;
    st[kStatDetected] = 0;
    st[kStatMatched] = 0;
  }
  return base;
}

// Appends the accepted stereo matches of the n_new detections of a detecting
// camera to right camera R, after its n_surv_r survivors and n_rec_r temporal
// records. id(i), sres(i): detection i's identifier and match; `sr`: the match
// of detection threadIdx.x.
template <class IdOf, class SresOf>
__device__ __forceinline__ int accept_matches(const CamDesc& R, const FrameCam& fr, int rc, int n_new, int n_surv_r,
                                              int n_rec_r, IdOf id_of, SresOf sres, TrackRes sr, Counters* cnt,
                                              Scan& sc, PairRow* tab = nullptr) {
  const int PR = fr.parity;
  int m_base = 0;
  for (int i0 = 0; i0 < n_new; i0 += kSelectThreads) {
    const int i = i0 + (int)threadIdx.x;
    const bool valid = i < n_new;
    int64_t id = 0;
    if (valid) {
      if (i0 > 0) sr = sres(i);
      id = id_of(i);
    }
    const bool matched = valid && sr.status == VIO_TRACKED;
    int m_tot;
    const int mrank = m_base + block_scan_flag(matched, sc, m_tot);
    if (valid) {
      const bool accepted = matched && n_surv_r + mrank < R.cap;
      const int st = matched ? (accepted ? VIO_MATCHED : VIO_LOST_CAP) : sr.status;
      R.rec[fr.rec_slot][n_rec_r + i] = make_rec(id, R.local, st, sr.x, sr.y, sr.theta, sr.fb, sr.resid, 0, -1);
      if (accepted) {
        R.state[PR][n_surv_r + mrank] = make_kp(id, sr.x, sr.y, sr.x, sr.y, 0);
        if (tab) tab[n_surv_r + mrank] = PairRow{id, sr.x, sr.y};
      }
    }
    m_base += m_tot;
  }
  const int accepted = min(m_base, max(0, R.cap - n_surv_r));
  if (threadIdx.x == 0) {
    cnt->n_live[PR][rc] = n_surv_r + accepted;
    cnt->rec_count[rc] = n_rec_r + n_new;
    *R.rec_count_out[fr.rec_slot] = n_rec_r + n_new;
    R.stats_out[fr.rec_slot][kStatMatched] = accepted;
  }
  return n_surv_r + accepted;
}

// The neighbour stereo start's table of target camera R (parity PR): its
// n_right keypoints, in id order, that also live among detecting camera L's
// n_left keypoints (parity P; both states are sorted by id), as L's position
// and the offset from L to R. The next frame's stereo matches into R read it.
// tl / tr: both cameras' ids and positions as the selection wrote them to
// LDS (when they fit; tl_ids: the left ids again, contiguous, for the
// search), else the states in memory, with the left ids staged in s_ids (LDS
// room for kPairIdsLds ids) when they fit there.
constexpr int kPairIdsLds = kMaxCells / 2;  // int64 ids in the occupancy array's bytes

__device__ void build_pairs(const CamDesc& L, int P, int n_left, const CamDesc& R, int PR, int rc, int n_right,
                            Counters* cnt, Scan& sc, const PairRow* tl, const int64_t* tl_ids, const PairRow* tr,
                            int64_t* s_ids) {
  const bool staged = !tl && n_left <= kPairIdsLds;
  if (staged) {
    __syncthreads();  // the LDS array's previous use is over
    for (int k = (int)threadIdx.x; k < n_left; k += kSelectThreads) s_ids[k] = L.state[P][k].id;
    __syncthreads();
  }
  int base = 0;
  for (int i0 = 0; i0 < n_right; i0 += kSelectThreads) {
    const int i = i0 + (int)threadIdx.x;
    bool found = false;
    float4 e = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < n_right) {
      int64_t qid;
      float qx, qy;
      if (tr) {
        const PairRow q = tr[i];
        qid = q.id;
        qx = q.x;
        qy = q.y;
      } else {
        const Kp q = R.state[PR][i];
        qid = q.id;
        qx = q.x;
        qy = q.y;
      }
      int at = -1;
      if (tl_ids) {
        // lower bound over the contiguous LDS ids, branch-free: every lane
        // takes the same floor(log2(n_left)) + 1 steps of halving size
        if (n_left > 0) {
          int pos = 0;  // ids below qid so far
          for (int step = 1 << (31 - __clz(n_left)); step > 0; step >>= 1) {
            const int probe = pos + step;
            const int64_t v = tl_ids[min(probe, n_left) - 1];
            pos = probe <= n_left && v < qid ? probe : pos;
          }
          at = pos < n_left && tl_ids[pos] == qid ? pos : -1;
        }
      } else {
        int lo = 0, hi = n_left - 1;
        while (lo <= hi) {
          const int mid = (lo + hi) >> 1;
          const int64_t id = staged ? s_ids[mid] : L.state[P][mid].id;
          if (id == qid) {
            at = mid;
            break;
          }
          if (id < qid) lo = mid + 1;
          else hi = mid - 1;
        }
      }
      if (at >= 0) {
        float lx, ly;
        if (tl) {
          lx = tl[at].x;
          ly = tl[at].y;
        } else {
          const Kp l = L.state[P][at];
          lx = l.x;
          ly = l.y;
        }
        e = make_float4(lx, ly, qx - lx, qy - ly);
        found = true;
      }
    }
    int total;
    const int pos = base + block_scan_flag(found, sc, total);
    if (found) R.pairs[PR][pos] = e;
    base += total;
  }
  if (threadIdx.x == 0) cnt->n_pairs[PR][rc] = base;
}

__global__ __launch_bounds__(kSelectThreads) void k_select(const CamDesc* __restrict__ cams,
                                                          const FrameTable* __restrict__ frame, Counters* cnt,
                                                          SelectGroups groups, int phase, Tuning tune) {
  __shared__ ScanScratch s_scan;
  __shared__ int s_hsum[4];
  Scan sc{&s_scan, 0};
  __shared__ __align__(8) unsigned s_occ[kMaxCells];  // cell occupancy; later the pair search's left ids
  __shared__ uint16_t s_sel[kMaxCells];  // key slot of selection rank i (rank < cap <= kMaxCells, slot < 2^16)
  __shared__ int s_hist[256];
  __shared__ int s_thr[2];
  __shared__ int64_t s_id0;
  // the detecting and the target camera's rows for the neighbour stereo start's pair table
  __shared__ PairRow s_pl[kPairLds], s_pr[kPairLds];
  __shared__ int64_t s_plid[kPairLds];  // s_pl's ids, contiguous for the pair search
  // the launch's groups in camera order, or in ticket order where some wait for others
  int gi = (int)blockIdx.x;
  if (groups.chained && phase != kSelectRight) {
    __shared__ int s_group;
    if (threadIdx.x == 0) s_group = take_group<AgentMem>(&cnt->select_ticket, groups.n);
    __syncthreads();
    gi = __builtin_amdgcn_readfirstlane(s_group);
  }
  const auto grp = groups.g[gi];
  const int lc = grp.cam;
  const CamDesc& L = cams[lc];
  const FrameCam& fl = frame->cam[lc];
  if (!fl.active) return;
  const int P = fl.parity, Q = P ^ 1;
  const int tid = (int)threadIdx.x;
  if (phase == kSelectRight) {
    const int n_new = cnt->n_sel[lc], sel_base = cnt->sel_base[lc];
    for (int t = 0; t < L.n_targets; ++t) {
      const int rc = lc + 1 + t;
      const FrameCam& fr = frame->cam[rc];
      const int PR = fr.parity;
      const int n_rec_r = fr.has_prev ? cnt->n_live[PR ^ 1][rc] : 0;
      const TrackRes* sres = L.sres + (size_t)t * L.nslots;
      TrackRes sr{};
      if (tid < n_new) sr = sres[tid];
      const int n_r = accept_matches(cams[rc], fr, rc, n_new, cnt->n_live[PR][rc], n_rec_r,
                                     [&](int i) { return L.state[P][sel_base + i].id; },
                                     [&](int i) { return sres[i]; }, sr, cnt, sc);
      __syncthreads();
      if (tune.stereo_nb) {
        build_pairs(L, P, sel_base + n_new, cams[rc], PR, rc, n_r, cnt, sc, nullptr, nullptr, nullptr,
                    reinterpret_cast<int64_t*>(s_occ));
        __syncthreads();
      }
    }
    return;
  }
  // what depends on no earlier step: the thread's first key slot and rows
  const int ncells = L.ncells, kc = L.kcell, nslots = L.nslots;
  const uint32_t* keys = L.keys[fl.pyr];
  const uint32_t key0 = tid < nslots ? keys[tid] : 0u;
  const PrevRow row_l = load_row(L, fl, tid);
  PrevRow row_r{};
  if (L.n_targets > 0) row_r = load_row(cams[lc + 1], frame->cam[lc + 1], tid);
  const auto key_of = [&](int slot) { return slot < kSelectThreads ? key0 : slot < nslots ? keys[slot] : 0u; };
  const auto cell_of = [kc](int slot) { return kc == 1 ? slot : slot / kc; };
  {
    for (int i = tid; i < ncells; i += kSelectThreads) s_occ[i] = 0;
    for (int i = tid; i < 256; i += kSelectThreads) s_hist[i] = 0;
    __syncthreads();

    // ---- left / mono camera: survivors and occupancy ----------------------
    int n_rec = 0;
    const bool count_fb = tune.learned != 0 || tune.plevels > 0;
    // pair rows in LDS (all-in-one selection with the neighbour stereo start)
    const bool pairs_lds = phase == kSelectAll && tune.stereo_nb && L.cap <= kPairLds;
    const int n_surv = carry_survivors(L, fl, cnt->n_live[Q][lc], row_l, s_occ, sc, &n_rec, count_fb,
                                       pairs_lds ? s_pl : nullptr, pairs_lds ? s_plid : nullptr);
    __syncthreads();

    // ---- candidates of unmasked cells, score histogram --------------------
    for (int i = tid; i < nslots; i += kSelectThreads) {
      const uint32_t key = key_of(i);
      if (key && (int)s_occ[cell_of(i)] < kc) atomicAdd(&s_hist[key >> 24], 1);
    }
    __syncthreads();
    // Score threshold of the best `room` candidates: thread t < 256 holds bin
    // v = 255 - t, so a scan in thread order gives cum(v) = #candidates
    // scoring >= v. With more candidates than room, thr is the bin where cum
    // first reaches room and rem the number taken from it; thr = 256 takes
    // none (no room), thr = -1 takes all.
    {
      const int room = max(0, L.cap - n_surv);
      int hv = 0, incl = 0;
      if (tid < 256) {
        hv = s_hist[255 - tid];
        incl = wave_incl_scan(hv);
        if ((tid & 63) == 63) s_hsum[tid >> 6] = incl;
      }
      __syncthreads();
      if (tid < 256) {
        const int w = tid >> 6;
        int before = 0, total = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int t = s_hsum[k];
          before += k < w ? t : 0;
          total += t;
        }
        const int cum = before + incl;
        if (room > 0 && total > room && cum >= room && cum - hv < room) {
          s_thr[0] = 255 - tid;
          s_thr[1] = room - (cum - hv);
        }
        if (tid == 0 && (room == 0 || total <= room)) {
          s_thr[0] = room == 0 ? 256 : -1;
          s_thr[1] = 0;
        }
        if (tid == 0) {
          // the group's identifiers follow those of the stream's earlier groups
          const int64_t id0 = grp.first ? cnt->next_id[L.stream] : take_id<AgentMem>(&cnt->id_chain[grp.prev]);
          s_id0 = id0;
          const int64_t next = id0 + min(room, total);
          if (grp.last) cnt->next_id[L.stream] = next;
          else hand_on_id<AgentMem>(&cnt->id_chain[lc], next);
        }
      }
      __syncthreads();
    }
    const int thr = s_thr[0], rem = s_thr[1];
    const int64_t next_id = s_id0;

    // ---- selection in slot order, identifiers, DET_t records --------------
    int n_new = 0, eq_base = 0;
    for (int i0 = 0; i0 < nslots; i0 += kSelectThreads) {
      const int slot = i0 + (int)threadIdx.x;
      const uint32_t key = key_of(slot);
      const bool cand = key && (int)s_occ[slot < nslots ? cell_of(slot) : 0] < kc;
      const int score = (int)(key >> 24);
      const bool is_eq = cand && score == thr;
      int eq_tot, sel_tot;
      const int eq_rank = eq_base + block_scan_flag(is_eq, sc, eq_tot);
      const bool sel = cand && (score > thr || (is_eq && eq_rank < rem));
      const int rank = n_new + block_scan_flag(sel, sc, sel_tot);
      if (sel) {
        const int idx = 0xFFFFFF - (int)(key & 0xFFFFFFu);
        const float x = (float)(idx % L.w), y = (float)(idx / L.w);
        const int64_t id = next_id + rank;
        L.state[P][n_surv + rank] = make_kp(id, x, y, x, y, 0);
        if (pairs_lds) {
          s_pl[n_surv + rank] = PairRow{id, x, y};
          s_plid[n_surv + rank] = id;
        }
        L.rec[fl.rec_slot][n_rec + rank] = make_rec(id, L.local, VIO_DETECTED, x, y, 0.f, 0.f, 0.f, 0, score);
        s_sel[rank] = (uint16_t)slot;
      }
      eq_base += eq_tot;
      n_new += sel_tot;
    }
    if (threadIdx.x == 0) {
      cnt->n_live[P][lc] = n_surv + n_new;
      cnt->rec_count[lc] = n_rec + n_new;
      *L.rec_count_out[fl.rec_slot] = n_rec + n_new;
      L.stats_out[fl.rec_slot][kStatDetected] = n_new;
    }
    // the key buffer of the frame kPyrSlots - 1 frames ahead: the frames in
    // between may already run their detectors beside this selection (their
    // buffers were cleared by earlier selections), and that frame cannot be
    // submitted before this one has completed
    uint32_t* next_keys = L.keys[(fl.pyr + kPyrSlots - 1) % kPyrSlots];
    for (int i = threadIdx.x; i < nslots; i += kSelectThreads) next_keys[i] = 0u;
    __syncthreads();

    // ---- target cameras (a pair's right camera, a star's other three):
    //      survivors, then accepted stereo matches
    for (int t = 0; t < L.n_targets; ++t) {
      const int rc = lc + 1 + t;
      const CamDesc& R = cams[rc];
      const FrameCam& fr = frame->cam[rc];
      const int PR = fr.parity;
      int n_rec_r = 0;
      const bool pairs_lds_r = pairs_lds && R.cap <= kPairLds;
      const TrackRes* sres = L.sres + (size_t)t * nslots;
      TrackRes sr{};
      if (phase == kSelectAll && tid < n_new) sr = sres[s_sel[tid]];
      const PrevRow row = row_r;
      if (t + 1 < L.n_targets) row_r = load_row(cams[rc + 1], frame->cam[rc + 1], tid);
      const int n_surv_r = carry_survivors(R, fr, cnt->n_live[PR ^ 1][rc], row, nullptr, sc, &n_rec_r, count_fb,
                                           pairs_lds_r ? s_pr : nullptr);
      if (phase == kSelectAll) {
        const int n_r = accept_matches(R, fr, rc, n_new, n_surv_r, n_rec_r, [&](int i) { return next_id + i; },
                                       [&](int i) { return sres[s_sel[i]]; }, sr, cnt, sc,
                                       pairs_lds_r ? s_pr : nullptr);
        if (tune.stereo_nb) {
          __syncthreads();
          build_pairs(L, P, n_surv + n_new, R, PR, rc, n_r, cnt, sc, pairs_lds ? s_pl : nullptr,
                      pairs_lds ? s_plid : nullptr, pairs_lds_r ? s_pr : nullptr, reinterpret_cast<int64_t*>(s_occ));
        }
      } else if (tid == 0) {
        // the matches come from the stereo tracking launch; kSelectRight appends them
        cnt->sel_base[lc] = n_surv;
        cnt->n_sel[lc] = n_new;
        cnt->n_live[PR][rc] = n_surv_r;
      }
      __syncthreads();
    }
  }
}

}  // namespace

hipError_t launch_select(const CamDesc* d_cams, const FrameTable* d_frame, Counters* d_cnt, const SelectGroups& groups,
                         int phase, Tuning tune, hipStream_t s) {
  if (groups.n <= 0) return hipSuccess;
  launch_kernel(k_select, dim3(groups.n), dim3(kSelectThreads), 0, s, d_cams, d_frame, d_cnt, groups, phase, tune);
  return hipGetLastError();
}

}  // namespace vio
