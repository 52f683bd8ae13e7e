// gv_pool.h -- the batched driver's pool kernel: stage baskets in LDS.
//
// Every wavefront keeps a pool of tracks in LDS and follows them, and the
// secondaries they make, until none is left or its share of the launch is
// done.  Each track carries a tag, the stage it waits for: the next step of a
// photon, of a charged track, of a charged track in vacuum, or one of the
// discrete interactions (Sec. 3.5) that its last step selected.  The wavefront
// takes up to 64 tracks of one tag through that stage in registers and puts
// them back with their next tag; secondaries go into free slots.  These are the
// stage baskets of Sec. 2.1.1 at the scale of a wavefront: it runs one stage
// at a time with its lanes full, while the step kernel (k_step_batched), whose
// lanes follow one track each through whole steps, runs the interaction code of
// each process for the few lanes that need it.
//
// What bounded the step kernel, and what this split is for:
//   * divergence: about one photon step in six ends in an interaction, so
//     nearly every iteration of a wavefront executed Compton and pair code for
//     a few lanes;
//   * the launch as a barrier: a launch lasted as long as its slowest track
//     (up to 256 steps while the population is low), and a shower needs as many
//     launches as it has generations.  Here a wavefront follows secondaries
//     itself, so a small batch ends in a few launches.
// Below the population that fills the GPU (2 x 256 tracks per CU) this kernel
// is the faster one, above it the step kernel: of 1000 x 10 GeV e- in 50 layers
// the part below took 8.1 ms in the step kernel and takes 2.5 ms here, while at
// 2 to 3 million tracks the step kernel makes 1.6e10 steps/s and this one
// 1.0e10 (its round trips through LDS, and spilled secondaries).  Against the step
// kernel alone, as it was then: one 1 GeV e- 3.05 -> 1.31 ms; 100 of them 4.68 -> 2.14
// ms; 1,000 of 10 GeV 21.6 -> 15.1 ms (with the smaller step kernel).  What bounds it is the latency of single histories: a
// photon step is ~1.2 us of dependent instructions for a lone track.
//
// Nothing observable depends on the schedule: a track's random numbers are
// keyed by (event, track id, step), and each stage is the step kernel's own
// function on the same state.  The state between a step and its interaction
// is the track alone (the tag says which process; the step count is advanced
// after the interaction), so an interaction may be taken any time later.
//
// A pool belongs to one wavefront, so nothing in the loop waits for another.  A
// wavefront whose input is used up begins no step `budget` ticks of the wall clock
// after its own start, one stage apart; it makes the interactions that wait, which no
// step follows, and leaves.
#pragma once
#include "gv_kernels.h"

namespace gv {

constexpr int kPoolBlock = 256;             // four wavefronts, each with a pool of its own
constexpr int kPoolWaves = kPoolBlock / 64;
constexpr int kPoolDep = 64;               // deposit cache entries per wavefront
// slots of a pool (at most four tags per lane, a multiple of 64) and workgroups
// per CU, whose pools together fill its LDS
template <class P> struct PoolSize {
    static constexpr int kSlots = 192;
    static constexpr int wgs(bool integ) { return P::kMixed && !integ ? 3 : 2; }
};

enum : int {
    kTagFree = 0,
    kTagBusy = 1,       // in a stage, or reserved for a secondary
    kTagPhoton = 2,     // waits for its next step
    kTagCharged = 3,
    kTagVacuum = 4,     // charged, in a volume without material in a uniform field (helix)
    kTagCompton = 5,    // waits for the interaction that its last step ended with
    kTagPair = 6,
    kTagDelta = 7,
    kTagBrems = 8,
    kTagAnnih = 9,      // e+ at rest
    kNTag = 10
};

template <class P> struct PoolMem {
    using R = typename P::R;
    static constexpr int kSlots = PoolSize<P>::kSlots;
    double x[kSlots], y[kSlots], z[kSlots];
    uint64_t tid[kSlots];
    R ux[kSlots], uy[kSlots], uz[kSlots], T[kSlots];
    int vt[kSlots];                         // volume * 4 + type
    uint32_t ev[kSlots], nstep[kSlots];
    uint32_t tag[64];                       // lane l: tags of slots 4 l .. 4 l + 3, one byte each
    uint32_t list[64];                      // slots picked for the stage in hand
};

struct PoolDep {
    uint32_t key[kPoolDep];
    double val[kPoolDep];
};

template <class P> struct PoolArgs {
    Soa<P> in[3];
    Soa<P> out[3];
    Ctrl* ctrl;
    CtrlMirror* mirror;    // what the host reads between launches
    uint32_t cap;
    int parity;
    long long budget;      // wall-clock ticks from its start after which a wavefront with no input left puts its tracks back
    int inner;             // steps a track takes in registers per stage, at most
    Sinks S;
    TabView<typename P::R> tv;
};

__device__ __forceinline__ int mbcnt64(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Tags and lists pass between the lanes of a wavefront through LDS: relaxed
// atomics through LDS pointers, which the wavefront's DS instructions take in
// order (a generic pointer would make them flat instructions, which are not
// ordered against those).
template <class T> struct LdsPtr {
    typedef __attribute__((address_space(3))) T type;
};
template <class T> __device__ __forceinline__ T lds_get(const T* p)
{
    return __hip_atomic_load((const typename LdsPtr<T>::type*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T> __device__ __forceinline__ void lds_put(T* p, T v)
{
    __hip_atomic_store((typename LdsPtr<T>::type*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// keeps the compiler from moving LDS accesses of one stage across the next
__device__ __forceinline__ void pool_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// What a wavefront knows of its pool, the same in all its lanes but `ready`.
struct PoolState {
    int ready;   // lane t: tracks that wait with tag t
    int live;    // slots that are not free
};

// Picks up to `want` slots whose tag is `tag` and marks them busy; lane l gets
// the l-th of them (-1 beyond the last).  Returns how many.
template <class P> __device__ __forceinline__ int pool_pick(PoolMem<P>& M, int lane, int tag, int want, int& slot)
{
    pool_fence();
    uint32_t tags = lds_get(&M.tag[lane]);
    const int n_lanes = PoolSize<P>::kSlots / 4;
    int found = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool m = lane < n_lanes && (int)((tags >> (8 * k)) & 255u) == tag;
        const uint64_t mask = __ballot(m);
        const int r = found + mbcnt64(mask);
        if (m && r < want) {
            lds_put(&M.list[r], (uint32_t)(lane * 4 + k));
            tags = (tags & ~(255u << (8 * k))) | ((uint32_t)kTagBusy << (8 * k));
        }
        found += __popcll(mask);
    }
    lds_put(&M.tag[lane], tags);
    pool_fence();
    const int n = min(found, want);
    slot = lane < n ? (int)lds_get(&M.list[lane]) : -1;
    return n;
}

// a free slot for each lane that wants one (-1: the pool is full)
template <class P> __device__ __forceinline__ int pool_alloc(PoolMem<P>& M, PoolState& st, int lane, bool want)
{
    const uint64_t mask = __ballot(want);
    const int need = __popcll(mask);
    if (need == 0) return -1;
    int slot;
    const int got = pool_pick(M, lane, kTagFree, need, slot);
    st.live += got;
    const int rank = mbcnt64(mask);
    return want && rank < got ? (int)lds_get(&M.list[rank]) : -1;
}

// Hands slots back with their next tag (kTagFree: the track is gone).  Every
// lane of the wavefront calls it; slot < 0: nothing.
// TAGS: bit t set if tag t can come up (kTagFree always can).
template <uint32_t TAGS, class P>
__device__ __forceinline__ void pool_put(PoolMem<P>& M, PoolState& st, int lane, int slot, int tag)
{
    pool_fence();
    const bool has = slot >= 0;
    if (has) lds_put(reinterpret_cast<uint8_t*>(&M.tag[0]) + slot, (uint8_t)tag);
#pragma unroll
    for (int s = kTagPhoton; s < kNTag; ++s) {
        if (!((TAGS >> s) & 1u)) continue;
        const int k = __popcll(__ballot(has && tag == s));
        st.ready += lane == s ? k : 0;
    }
    st.live -= __popcll(__ballot(has && tag == kTagFree));
    pool_fence();
}

template <class P> __device__ __forceinline__ void pool_load(const PoolMem<P>& M, int s, Track<P>& t)
{
    t.x[0] = M.x[s];
    t.x[1] = M.y[s];
    t.x[2] = M.z[s];
    t.u[0] = M.ux[s];
    t.u[1] = M.uy[s];
    t.u[2] = M.uz[s];
    t.T = M.T[s];
    const int vt = M.vt[s];
    t.vol = vt >> 2;
    t.type = vt & 3;
    t.ev = M.ev[s];
    t.tid = M.tid[s];
    t.nstep = M.nstep[s];
}

template <class P> __device__ __forceinline__ void pool_store(PoolMem<P>& M, int s, const Track<P>& t)
{
    M.x[s] = t.x[0];
    M.y[s] = t.x[1];
    M.z[s] = t.x[2];
    M.ux[s] = t.u[0];
    M.uy[s] = t.u[1];
    M.uz[s] = t.u[2];
    M.T[s] = t.T;
    M.vt[s] = t.vol * 4 + t.type;
    M.ev[s] = t.ev;
    M.tid[s] = t.tid;
    M.nstep[s] = t.nstep;
}

template <class P, class R = typename P::R>
__device__ __forceinline__ void pool_store_child(PoolMem<P>& M, int s, const Track<P>& parent, const Child<R>& c)
{
    M.x[s] = parent.x[0];
    M.y[s] = parent.x[1];
    M.z[s] = parent.x[2];
    M.ux[s] = c.u[0];
    M.uy[s] = c.u[1];
    M.uz[s] = c.u[2];
    M.T[s] = c.T;
    M.vt[s] = parent.vol * 4 + c.type;
    M.ev[s] = parent.ev;
    M.tid[s] = c.tid;
    M.nstep[s] = 0;
}

// Deposits of a wavefront's stages, summed per (event, cell) in a table of its
// own (as dep_add, whose table a workgroup shares between barriers).  Returns
// false if the deposit found no entry and went to HBM.
__device__ __forceinline__ bool pool_deposit(PoolDep& dc, const Sinks& S, uint32_t ev, int vol, const DepAcc& a)
{
    if (a.e == 0.0 && a.x == 0ull) return true;
    const int cell = vol_cell(c_geom, vol);
    if (cell < 0) {
        sink_add_acc(S, &S.ledger[(size_t)ev * 4 + 1], a);
        return true;
    }
    const uint64_t k64 = (uint64_t)ev * (uint64_t)c_geom.n_cells + (uint64_t)cell;
    if (k64 < kDepEmpty) {
        const uint32_t k = (uint32_t)k64;
        uint32_t h = (k * 2654435761u) >> 26;   // 6 bits: kPoolDep = 64
        for (int probe = 0; probe < 4; ++probe) {
            const uint32_t old = atomicCAS(&dc.key[h], kDepEmpty, k);
            if (old == kDepEmpty || old == k) {
                if (S.fixed) {
                    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
                    __hip_atomic_fetch_add((lds_u64*)&dc.val[h], a.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                } else {
                    typedef __attribute__((address_space(3))) double lds_double;
                    __hip_atomic_fetch_add((lds_double*)&dc.val[h], a.e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                return true;
            }
            h = (h + 1) & (kPoolDep - 1);
        }
    }
    sink_add_acc(S, &S.edep[k64], a);
    return false;
}

// write the wavefront's cached sums to HBM and empty the table
__device__ __forceinline__ void pool_dep_flush(PoolDep& dc, const Sinks& S, int lane)
{
    pool_fence();
#pragma unroll
    for (int i = lane; i < kPoolDep; i += 64) {
        const uint32_t k = dc.key[i];
        if (k != kDepEmpty) {
            if (S.fixed)
                atomicAdd(reinterpret_cast<unsigned long long*>(&S.edep[k]),
                          (unsigned long long)__double_as_longlong(dc.val[i]));
            else
                unsafeAtomicAdd(&S.edep[k], dc.val[i]);
            dc.key[i] = kDepEmpty;
            dc.val[i] = 0.0;
        }
    }
    pool_fence();
}

// per-wavefront sums of one launch
struct PoolCount {
    uint32_t steps[3];
    uint32_t loads, stores;
    uint32_t lane_iters;   // iterations of the wavefront's step loops
    RkSum rk;
};

// Steps of a stage go on while at least 5/8 of its tracks still step: with ~0.8
// of the photons going on per step and a round trip through LDS worth half a
// step, fewer lanes cost more than the round trip.
__device__ __forceinline__ int pool_min_active(int n) { return max(1, (5 * n) >> 3); }

template <class P, class R = typename P::R>
__device__ __forceinline__ void pool_end_track(const Sinks& S, const Track<P>& t, const StepOut<R>& o, unsigned* cnt)
{
    account_rare(S, t.ev, o, cnt);
    if (o.status == kEscaped) escape_count(S, t.type, t.T, t.u[2]);
}

// steps of up to 64 photons; returns this lane's next tag
template <class P, class R = typename P::R>
__device__ __forceinline__ int pool_photons(const PoolArgs<P>& A, const Ctx<P>& c, Track<P>& t, bool act, int n,
                                            unsigned* cnt, PoolCount& pc)
{
    int tag = kTagPhoton;
    const int min_act = pool_min_active(n);
    t.type = kGamma;
    for (int it = 0;;) {
        if (act) {
            StepOut<R> o;
            init_out(t, o);
            if (!stage_prestep(c, t, o)) {
                pool_end_track(A.S, t, o, cnt);
                tag = kTagFree;
                act = false;
            } else {
                Limits<R> L;
                stage_limit(c, t, L);
                Geo G;
                stage_geom(c, t, G);
                Prop<R> pr;
                stage_move<P, false>(c, t, L, G, pr);
                pc.steps[kGamma] += 1;
                if (pr.lim == kLimPhys && !pr.crossed) {
                    tag = L.usel * L.stot < L.sa ? kTagCompton : kTagPair;
                    act = false;
                } else {
                    if (t.vol == kOutside) {
                        o.e_escaped += (double)t.T;
                        o.status = kEscaped;
                        pool_end_track(A.S, t, o, cnt);
                        tag = kTagFree;
                        act = false;
                    }
                    t.nstep += 1;
                }
            }
        }
        it += 1;
        if (it >= A.inner || __popcll(__ballot(act)) < min_act) {
            pc.lane_iters += it;
            break;
        }
    }
    return tag;
}

// steps of up to 64 charged tracks; returns this lane's next tag
template <class P, bool INTEG, class R = typename P::R>
__device__ __forceinline__ int pool_charged(const PoolArgs<P>& A, const Ctx<P>& c, Track<P>& t, bool act, int n,
                                            bool vac_ok, unsigned* cnt, PoolCount& pc, PoolDep& dc, int lane)
{
    int tag = kTagCharged;
    const int min_act = pool_min_active(n);
    DepAcc acc{0.0, 0ull};
    int acc_vol = t.vol;
    const bool had = act;
    bool fit = true;
    for (int it = 0;;) {
        if (act) {
            StepOut<R> o;
            init_out(t, o);
            if (t.vol != kOutside && t.T < (R)c.ph->t_track) {
                // PreStep below the tracking cut; an e+ annihilates in a stage of its own
                o.edep += (double)t.T;
                t.T = (R)0;
                tag = t.type == kPositron ? kTagAnnih : kTagFree;
                act = false;
            } else if (!stage_prestep(c, t, o)) {
                pool_end_track(A.S, t, o, cnt);
                tag = kTagFree;
                act = false;
            } else {
                Limits<R> L;
                stage_limit(c, t, L);
                Geo G;
                stage_geom(c, t, G);
                Prop<R> pr;
                stage_move<P, INTEG>(c, t, L, G, pr);
                if (INTEG) {
                    pc.rk.acc += (uint32_t)pr.rk.acc;
                    pc.rk.rej += (uint32_t)pr.rk.rej;
                    pc.rk.slots += (uint32_t)pr.rk.iters;
                }
                stage_msc(c, t, L, pr);
                const bool stopped = stage_eloss(c, t, L, pr, o);
                pc.steps[kElectron] += t.type == kElectron ? 1u : 0u;
                pc.steps[kPositron] += t.type == kPositron ? 1u : 0u;
                if (stopped) {
                    tag = t.type == kPositron ? kTagAnnih : kTagFree;
                    act = false;
                } else if (pr.lim == kLimPhys && !pr.crossed) {
                    tag = L.usel * L.stot < L.sa ? kTagDelta : kTagBrems;
                    act = false;
                } else {
                    if (t.vol == kOutside) {
                        o.e_escaped += (double)t.T;
                        o.status = kEscaped;
                        pool_end_track(A.S, t, o, cnt);
                        tag = kTagFree;
                        act = false;
                    } else if (!INTEG && vac_ok && vol_material(c_geom, t.vol) < 0 && !(t.T < (R)c.ph->t_track)) {
                        tag = kTagVacuum;
                        act = false;
                    }
                    t.nstep += 1;
                }
            }
            if (o.vol_pre != acc_vol) {
                fit &= pool_deposit(dc, A.S, t.ev, acc_vol, acc);
                acc.e = 0.0;
                acc.x = 0ull;
                acc_vol = o.vol_pre;
            }
            acc_add(A.S, acc, o.edep);
        }
        it += 1;
        if (it >= A.inner || __popcll(__ballot(act)) < min_act) {
            pc.lane_iters += it;
            break;
        }
    }
    if (had) fit &= pool_deposit(dc, A.S, t.ev, acc_vol, acc);
    if (__any(!fit)) pool_dep_flush(dc, A.S, lane);
    return tag;
}

// vacuum steps (helix, uniform field) of up to 64 charged tracks above the
// tracking cut: the step kernel's vacuum forms
template <class P, class R = typename P::R>
__device__ __forceinline__ int pool_vacuum(const PoolArgs<P>& A, const Ctx<P>& c, Track<P>& t, bool act, int n,
                                           int max_iter, unsigned* cnt, PoolCount& pc)
{
    int tag = kTagVacuum;
    const int min_act = pool_min_active(n);
    WorldRun<P> run;
    if (act) run = world_run(c, t);
    for (int it = 0;;) {
        if (act) {
            StepOut<R> o;
            if (t.vol == 0) step_world(c, run, t, o);
            else step_track<P, false, true>(c, t, o);
            pc.steps[kElectron] += (t.type == kElectron && o.did_step) ? 1u : 0u;
            pc.steps[kPositron] += (t.type == kPositron && o.did_step) ? 1u : 0u;
            if (o.status != kAlive) {
                pool_end_track(A.S, t, o, cnt);
                tag = kTagFree;
                act = false;
            } else if (vol_material(c_geom, t.vol) >= 0) {
                tag = kTagCharged;
                act = false;
            }
        }
        it += 1;
        if (it >= max_iter || __popcll(__ballot(act)) < min_act) {
            pc.lane_iters += it;
            break;
        }
    }
    return tag;
}

// the kernel's own arguments (its first and only one; see opaque_ptr)
template <class P> __device__ __forceinline__ const PoolArgs<P>& pool_args()
{
    return *opaque_ptr((const PoolArgs<P>*)__builtin_amdgcn_kernarg_segment_ptr());
}
template <class P> __device__ __forceinline__ Ctx<P> pool_ctx(const PoolArgs<P>& A, uint64_t seed)
{
    return stage_ctx<P>(A.tv, seed);
}

// the tag of a track that waits for its next step
template <class P> __device__ __forceinline__ int pool_step_tag(const Track<P>& t, bool vac_ok)
{
    using R = typename P::R;
    if (t.type == kGamma) return kTagPhoton;
    const bool vac = vac_ok && t.vol != kOutside && vol_material(c_geom, t.vol) < 0 && !(t.T < (R)c_phys.t_track);
    return vac ? kTagVacuum : kTagCharged;
}

// One discrete interaction per lane (TAG at compile time), its deposit, and
// the slots of its secondaries.  A secondary takes its parent's slot if the
// parent ends, else a free one; with none free it goes to the output queue.
template <class P, int TAG, class R = typename P::R>
__device__ __forceinline__ void pool_interact(PoolMem<P>& M, PoolState& st, uint64_t seed, int slot, int lane, unsigned* cnt, PoolCount& pc, PoolDep& dc)
{
    const bool act = slot >= 0;
    const PoolArgs<P>& A = pool_args<P>();
    const Ctx<P> c = pool_ctx(A, seed);
    Track<P> t;
    StepOut<R> o;
    o.status = kDead;
    o.nchild = 0;
    o.ch[0].type = o.ch[1].type = kGamma;
    bool fit = true;
    if (act) {
        pool_load(M, slot, t);
        if (TAG == kTagCompton || TAG == kTagPair) t.type = kGamma;
        if (TAG == kTagAnnih) t.type = kPositron;
        init_out(t, o);
        if (TAG == kTagAnnih) {
            annihilate(c, t, o);
            o.status = kDead;
        } else {
            interact(c, t, TAG == kTagCompton || TAG == kTagDelta, o);
            t.nstep += 1;
        }
        if (TAG == kTagCompton || TAG == kTagPair) {
            DepAcc acc{0.0, 0ull};
            acc_add(A.S, acc, o.edep);
            fit = pool_deposit(dc, A.S, t.ev, t.vol, acc);
        }
        account_rare(A.S, t.ev, o, cnt);
    }
    const bool alive = act && o.status == kAlive;
    // secondaries beyond the parent's own slot: at most one
    const bool extra = act && o.nchild > (alive ? 0 : 1);
    const int slot2 = pool_alloc(M, st, lane, extra);
    int tag1 = kTagFree, tag2 = kTagFree;
    if (alive) {
        pool_store(M, slot, t);
        tag1 = t.type == kGamma ? kTagPhoton : kTagCharged;
    } else if (act && o.nchild > 0) {
        pool_store_child(M, slot, t, o.ch[0]);
        tag1 = o.ch[0].type == kGamma ? kTagPhoton : kTagCharged;
    }
    const int qt = alive ? o.ch[0].type : o.ch[1].type;
    if (slot2 >= 0) {
        if (alive) pool_store_child(M, slot2, t, o.ch[0]);
        else pool_store_child(M, slot2, t, o.ch[1]);
        tag2 = qt == kGamma ? kTagPhoton : kTagCharged;
    }
    const bool spill = extra && slot2 < 0;
    if (__any(spill)) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint64_t m = __ballot(spill && qt == q);
            if (!m) continue;
            const int leader = __ffsll((unsigned long long)m) - 1;
            uint32_t base = 0;
            if (lane == leader) {
                base = atomicAdd(&A.ctrl->count[A.parity ^ 1][q], (uint32_t)__popcll(m));
                atomicAdd(&cnt[kCPoolSpills], (unsigned)__popcll(m));
            }
            base = (uint32_t)__shfl((int)base, leader, 64);
            if (spill && qt == q) {
                const uint32_t pos = base + (uint32_t)mbcnt64(m);
                if (pos < A.cap && pos >= base) {
                    if (alive) store_child(A.out[q], pos, t, o.ch[0]);
                    else store_child(A.out[q], pos, t, o.ch[1]);
                    pc.stores += 1;
                } else {
                    atomicOr(&A.ctrl->overflow, 1u);
                }
            }
        }
    }
    constexpr uint32_t kBack = (1u << kTagPhoton) | (1u << kTagCharged);
    pool_put<kBack>(M, st, lane, slot, tag1);
    if (__any(slot2 >= 0)) pool_put<kBack>(M, st, lane, slot2, tag2);
    if (TAG == kTagCompton || TAG == kTagPair)
        if (__any(!fit)) pool_dep_flush(dc, A.S, lane);
}

// What a wavefront does next (uniform).
enum : int { kTakeNone = 0, kTakeStage = 1, kTakeInput = 2 };

// The fullest stage; but if that would leave lanes empty and input tracks are
// left, room is made for a chunk of those instead.  n: tracks picked, or input
// slots reserved.
template <class P>
__device__ __forceinline__ int pool_take(PoolMem<P>& M, PoolState& st, int lane, bool drain, bool input, int chunk,
                                         int& tag, int& n, int& slot)
{
    int best = -1, bn = 0;
#pragma unroll
    for (int s = kTagPhoton; s < kNTag; ++s) {
        const int v = __builtin_amdgcn_readlane(st.ready, s);
        if (v > bn && (!drain || s >= kTagCompton)) {
            bn = v;
            best = s;
        }
    }
    tag = best;
    if (input && bn < 64 && st.live + chunk <= PoolSize<P>::kSlots) {
        n = pool_pick(M, lane, kTagFree, chunk, slot);
        st.live += n;
        return kTakeInput;
    }
    if (best < 0) return kTakeNone;
    n = pool_pick(M, lane, best, 64, slot);
    st.ready -= lane == best ? n : 0;
    return kTakeStage;
}

// INTEG: field integrators compiled in (RK4 / RK45), as in the step kernel.
template <class P, bool INTEG>
__global__ void __launch_bounds__(kPoolBlock, PoolSize<P>::wgs(INTEG)) k_pool(PoolArgs<P>)
{
    const PoolArgs<P>& A0 = pool_args<P>();
    constexpr int kSlots = PoolSize<P>::kSlots;
    __shared__ PoolMem<P> pools[kPoolWaves];
    __shared__ PoolDep dep[kPoolWaves];
    __shared__ unsigned cnt[kNCount];
    __shared__ unsigned long long rk_lds[4];
    __shared__ uint32_t n_vac_lds;

    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    PoolMem<P>& M = pools[wid];
    const uint32_t n0 = min(A0.ctrl->count[A0.parity][0], A0.cap);
    const uint32_t n1 = min(A0.ctrl->count[A0.parity][1], A0.cap);
    const uint32_t n2 = min(A0.ctrl->count[A0.parity][2], A0.cap);
    // input in chunks of one type: a full wavefront each, or fewer tracks when
    // that spreads a small population over all wavefronts
    const uint32_t waves = gridDim.x * kPoolWaves, wave = blockIdx.x * kPoolWaves + (uint32_t)wid;
    const uint32_t chunk = max(1u, min(64u, (n0 + n1 + n2 + waves - 1) / waves));
    const uint32_t c0 = (n0 + chunk - 1) / chunk, c1 = (n1 + chunk - 1) / chunk, c2 = (n2 + chunk - 1) / chunk;
    const uint32_t n_chunks = c0 + c1 + c2;
    const bool vac_ok = !INTEG && c_geom.field_map == kMapUniform && c_geom.Bmag != 0.0;

    lds_put(&M.tag[lane], 0u);   // all free
    for (int i = lane; i < kPoolDep; i += 64) {
        dep[wid].key[i] = kDepEmpty;
        dep[wid].val[i] = 0.0;
    }
    for (int i = threadIdx.x; i < kNCount; i += kPoolBlock) cnt[i] = 0;
    if (threadIdx.x < 4) rk_lds[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) n_vac_lds = 0;
    const uint64_t seed = A0.ctrl->seed;
    PoolCount pc{{0u, 0u, 0u}, 0u, 0u, 0u, {0u, 0u, 0u}};
    PoolState st{0, 0};
    __syncthreads();

    uint32_t next_chunk = wave;   // this wavefront's own chunk first, then whichever is left
    bool drain = false, staged = false;
    const long long t0 = (long long)wall_clock64();
    for (;;) {
        int tag, n, slot;
        // with no input left, the launch's share is done `budget` ticks after its
        // start, and one stage at least: interactions that wait are taken (no step
        // follows them), then the tracks go to the output queues, to be shared out
        // evenly again.  By the clock and not by a count, because a stage may be one
        // photon step or a hundred integration attempts, and the launch lasts as
        // long as its slowest wavefront.
        drain |= staged && next_chunk >= n_chunks && (long long)wall_clock64() - t0 >= pool_args<P>().budget;
        const bool input = !drain && next_chunk < n_chunks;
        const int what = pool_take(M, st, lane, drain, input, (int)chunk, tag, n, slot);
        if (what == kTakeNone) break;
        if (n == 0) {   // tags and counts disagree: report it instead of going round for ever
            if (lane == 0) atomicOr(&pool_args<P>().ctrl->overflow, 4u);
            break;
        }
        if (what == kTakeInput) {
            const PoolArgs<P>& A = pool_args<P>();
            const uint32_t k = next_chunk;
            const int ty = k < c0 ? kGamma : k < c0 + c1 ? kElectron : kPositron;
            const uint32_t first = (k - (ty == kGamma ? 0u : ty == kElectron ? c0 : c0 + c1)) * chunk;
            const uint32_t nt = ty == kGamma ? n0 : ty == kElectron ? n1 : n2;
            const uint32_t i = first + (uint32_t)lane;
            int tag1 = kTagFree;
            if (slot >= 0 && i < nt) {
                Track<P> t;
                if (ty == kGamma) load_track(A.in[kGamma], i, kGamma, t);
                else if (ty == kElectron) load_track(A.in[kElectron], i, kElectron, t);
                else load_track(A.in[kPositron], i, kPositron, t);
                pc.loads += 1;
                pool_store(M, slot, t);
                tag1 = pool_step_tag(t, vac_ok);
            }
            pool_put<(1u << kTagPhoton) | (1u << kTagCharged) | (1u << kTagVacuum)>(M, st, lane, slot, tag1);
            next_chunk = n_chunks;
            if (n_chunks > waves) {
                uint32_t k2 = 0;
                if (lane == 0) k2 = waves + atomicAdd(&A.ctrl->ticket, 1u);
                next_chunk = (uint32_t)__builtin_amdgcn_readfirstlane((int)k2);
            }
            continue;
        }
        const PoolArgs<P>& A = pool_args<P>();
        staged = true;
        if (tag == kTagPhoton || tag == kTagCharged || tag == kTagVacuum) {
            Track<P> t;
            if (slot >= 0) pool_load(M, slot, t);
            const Ctx<P> c = pool_ctx(A, seed);
            const bool act = slot >= 0;
            if (tag == kTagPhoton) {
                const int next = pool_photons<P>(A, c, t, act, n, cnt, pc);
                if (act && next != kTagFree) pool_store(M, slot, t);
                pool_put<(1u << kTagPhoton) | (1u << kTagCompton) | (1u << kTagPair)>(M, st, lane, slot, next);
            } else if (INTEG || tag == kTagCharged) {
                const int next = pool_charged<P, INTEG>(A, c, t, act, n, vac_ok, cnt, pc, dep[wid], lane);
                if (act && next != kTagFree) pool_store(M, slot, t);
                pool_put<(1u << kTagCharged) | (1u << kTagVacuum) | (1u << kTagDelta) | (1u << kTagBrems) |
                         (1u << kTagAnnih)>(M, st, lane, slot, next);
            } else {
                const int next = pool_vacuum<P>(A, c, t, act, n, 32, cnt, pc);
                if (act && next != kTagFree) pool_store(M, slot, t);
                pool_put<(1u << kTagCharged) | (1u << kTagVacuum)>(M, st, lane, slot, next);
            }
        } else if (tag == kTagCompton) {
            pool_interact<P, kTagCompton>(M, st, seed, slot, lane, cnt, pc, dep[wid]);
        } else if (tag == kTagPair) {
            pool_interact<P, kTagPair>(M, st, seed, slot, lane, cnt, pc, dep[wid]);
        } else if (tag == kTagDelta) {
            pool_interact<P, kTagDelta>(M, st, seed, slot, lane, cnt, pc, dep[wid]);
        } else if (tag == kTagBrems) {
            pool_interact<P, kTagBrems>(M, st, seed, slot, lane, cnt, pc, dep[wid]);
        } else {
            pool_interact<P, kTagAnnih>(M, st, seed, slot, lane, cnt, pc, dep[wid]);
        }
    }
    const PoolArgs<P>& A = pool_args<P>();
    // tracks left in the pool to the output queues: counted by type, reserved
    // at once, written
    uint32_t n_vac = 0;
    if (st.live > 0) {
        pool_fence();
        int left[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < kSlots / 64; ++k) {
            const int s = k * 64 + lane;
            const bool has = lds_get(reinterpret_cast<const uint8_t*>(&M.tag[0]) + s) != kTagFree;
            const int ty = has ? (M.vt[s] & 3) : 3;
#pragma unroll
            for (int q = 0; q < 3; ++q) left[q] += __popcll(__ballot(ty == q));
        }
        uint32_t base[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            uint32_t b = 0;
            if (lane == 0 && left[q]) b = atomicAdd(&A.ctrl->count[A.parity ^ 1][q], (uint32_t)left[q]);
            base[q] = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
        }
#pragma unroll 1
        for (int k = 0; k < kSlots / 64; ++k) {
            const int s = k * 64 + lane;
            const bool has = lds_get(reinterpret_cast<const uint8_t*>(&M.tag[0]) + s) != kTagFree;
            Track<P> t;
            t.type = 3;
            if (has) pool_load(M, s, t);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const uint64_t m = __ballot(t.type == q);
                if (t.type == q) {
                    const uint32_t pos = base[q] + (uint32_t)mbcnt64(m);
                    if (pos < A.cap && pos >= base[q]) {
                        store_track(A.out[q], pos, t);
                        pc.stores += 1;
                        n_vac += (q != kGamma && t.vol != kOutside && vol_material(c_geom, t.vol) < 0) ? 1u : 0u;
                    } else {
                        atomicOr(&A.ctrl->overflow, 1u);
                    }
                }
                base[q] += (uint32_t)__popcll(m);
            }
        }
    }
    pool_dep_flush(dep[wid], A.S, lane);
    if (n_vac) atomicAdd(&n_vac_lds, n_vac);
    if (pc.steps[0]) atomicAdd(&cnt[kCSteps + 0], pc.steps[0]);
    if (pc.steps[1]) atomicAdd(&cnt[kCSteps + 1], pc.steps[1]);
    if (pc.steps[2]) atomicAdd(&cnt[kCSteps + 2], pc.steps[2]);
    if (pc.loads) atomicAdd(&cnt[kCLoads], pc.loads);
    if (pc.stores) atomicAdd(&cnt[kCStores], pc.stores);
    if (lane == 0 && pc.lane_iters) atomicAdd(&rk_lds[3], 64ull * pc.lane_iters);
    if (INTEG && (pc.rk.acc | pc.rk.rej | pc.rk.slots)) {
        atomicAdd(&rk_lds[0], (unsigned long long)pc.rk.acc);
        atomicAdd(&rk_lds[1], (unsigned long long)pc.rk.rej);
        atomicAdd(&rk_lds[2], (unsigned long long)pc.rk.slots);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kNCount; i += kPoolBlock)
        if (cnt[i]) atomicAdd(&A.S.counters[i], (unsigned long long)cnt[i]);
    if (threadIdx.x < 4 && rk_lds[threadIdx.x]) atomicAdd(&A.S.counters[kCRkSub + threadIdx.x], rk_lds[threadIdx.x]);
    if (threadIdx.x == 0 && n_vac_lds) atomicAdd(&A.ctrl->n_vac, n_vac_lds);
    finish_launch(A.ctrl, A.parity, gridDim.x, A.mirror, A.S.counters);
}

}  // namespace gv
