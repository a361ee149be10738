// Several blocks of one launch that work together round after round, on one die of the part.
//
// The part has eight dies of 32 compute units, each with an L2 of its own.  Blocks that depend on each other once or twice
// a round pay 2.5 us per launch and as much again until a launch's first loads are back; inside a launch a dependency
// is a store, a flag and a load.  Across dies those have to reach memory and the flags of 32 blocks cost 1.3 to 1.5 us (256
// blocks 3.4); on one die they meet in its L2: 0.77 us for 2 to 32 blocks, 1.13 us with 4 KB a block written before and
// read behind it.
//
// What makes it sound:
//  - Nobody waits without end for a block that may not have started.  A launch has `want` blocks for every die; each block
//    adds itself to the count of the die that it finds itself on, the first die whose blocks are complete is the one, and all
//    others end.  Launches that begin together can each hold a part of every die: so after kPickTicks a launch picks the die
//    where it has most blocks and gives up the others.  Where that one is not complete for `patience` either, because other
//    work holds its compute units, it is closed with the blocks it has by then.  The members are running when the rounds begin,
//    so whatever they wait for does happen; where they are fewer than wanted they share the work.
//  - A word a die, beside the library's code, says that a launch has picked it: others pick another one.  (Two with the same die would
//    wait for each other, and neither be complete: four streams with calls of eight rounds took 25 to 35 us for a round of
//    each, the same as launches 14.3, like this 14.4.)  The first member gives the die back.  A launch that finds all taken for
//    `patience` picks one all the same; launches of several processes do not see each other's words: those that hold equal
//    parts pick by lot, and those that picked the same one all the same lose patience at different times, by lot again.
//  - Within a die the vector L1 caches write through to the die's L2: a store that has been waited for (vmcnt) is in L2, and
//    a load with the sc1 bit, which does not look into L1, reads it there.  Data that one block leaves for another are
//    read with load_fresh*, never with an ordinary load.  (Device-scope stores would go on to memory: 1.0 to 1.5 us.)
//  - While the members are at work their compute units may have no room for other blocks, so a launch is kept to some milliseconds.
//  - The members' waits for each other are bounded all the same: after kPolls polls, seconds, they give up and set bit 31 of the
//    status word.  (Before that a block waits for times that it sees pass itself, and for one that is between two stores.)
#pragma once

#include "dq_common.h"

namespace dq {

constexpr long long kPickTicks = 1000;           // of the 100 MHz clock: 10 us (each call waits so long where several launches begin together)
constexpr int kPolls = 1 << 23;
constexpr uint32_t kGaveUp = 0x80000000u;        // in the status word

// In device memory; all zero before the launch.
struct DieControl {
    uint32_t home;                               // 1 + the die, whether the launch owns it; with kPicked and a lot: not complete yet
    uint32_t members;
    uint32_t joined[kDies];                      // top bit: closed
    uint32_t pad[34];                            // (the flags on cache lines that other dies' blocks do not touch)
    uint64_t flag[2][kDieUnits];                 // phase << 32 | value, by the parity of the phase
};

struct DieMember {
    DieControl *ctl;
    int me, count;                               // me < 0: not a member
};

__device__ __forceinline__ uint32_t load_fresh(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_fresh(const float *p)
{
    return __uint_as_float(load_fresh(reinterpret_cast<const uint32_t *>(p)));
}
// Sixteen bytes at byte `at` (a multiple of sixteen) behind p, zeros from byte `size` on.
__device__ __forceinline__ uint4 load_fresh16(const void *p, uint32_t size, uint32_t at)
{
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    constexpr int kSc1 = 16;
    const v4u t = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, size, 0x00020000),
                                                        static_cast<int>(at), 0, kSc1);
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ float4 load_fresh_f4(const float *p, uint32_t size, uint32_t at)
{
    const uint4 t = load_fresh16(p, size, at);
    return make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
}
// What this wavefront has stored is in L2 (and what it has loaded is there) when it goes on.
__device__ __forceinline__ void wait_for_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ uint32_t die_number()
{
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v & (kDies - 1);
}

// All threads of the block call it; sh: three words of LDS, kept until die_leave; taken: a word a die, zero where no launch has picked it.  The die is
// closed after `patience` ticks (up to twice that, by lot), where not even half of the blocks are there only after four times as many.
__device__ __forceinline__ DieMember die_join(DieControl *ctl, uint32_t *taken, uint32_t want, long long patience, int *sh)
{
    constexpr uint32_t kClosed = 0x80000000u, kDieBits = 0xffu, kPicked = 0x100u, kOwned = 0x200u, kLotShift = 10, kLots = 8;
    if (threadIdx.x == 0) {
        const uint32_t die = die_number();
        int me = -1, count = 0, owner = 0;
        const auto swap = [&](uint32_t *p, uint32_t from, uint32_t to) {
            return __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const auto picked_here = [&](uint32_t home) { return (home & (kDieBits | kPicked)) == ((die + 1) | kPicked); };
        // home = a die, if there is none yet; the first of the launches that want a die owns it
        const auto claim = [&](uint32_t which, uint32_t more, bool owned_only) {
            const bool own = swap(taken + which, 0u, 1u);
            if (!own && owned_only) return false;
            if (swap(&ctl->home, 0u, (which + 1) | more | (own ? kOwned : 0u))) return true;
            if (own) __hip_atomic_store(taken + which, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        };
        const uint32_t ticket = __hip_atomic_fetch_add(&ctl->joined[die], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ticket < want) {                             // (not closed, and not more than are wanted)
            // (a die whose blocks may have been told to end cannot become the one: `home` says another's number by then)
            const auto settle = [&] {
                if (!claim(die, 0u, false)) {
                    const uint32_t home = load_fresh(&ctl->home);
                    if (!picked_here(home) || !swap(&ctl->home, home, (die + 1) | (home & kOwned))) return;
                }
                const uint32_t c = __hip_atomic_fetch_or(&ctl->joined[die], kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&ctl->members, min(c, want), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            if (ticket == want - 1) settle();
            const long long start = wall_clock64();
            uint32_t home;
            while ((home = load_fresh(&ctl->home)) == 0 || picked_here(home)) {
                const long long now = wall_clock64(), waited = now - start;
                if (home == 0 && waited > kPickTicks) {
                    const uint32_t lot = static_cast<uint32_t>(now);
                    const uint32_t best = die_pick([&](uint32_t i) { return load_fresh(taken + i) ? 0u : load_fresh(&ctl->joined[i]); }, die, lot);
                    claim(best, kPicked | ((lot >> 3) % kLots) << kLotShift, waited < patience);
                }
                if (home != 0) {
                    const long long limit = patience + (home >> kLotShift) * (patience / kLots);
                    if (waited > limit && (load_fresh(&ctl->joined[die]) >= (want + 1) / 2 || waited > 4 * limit)) settle();
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if ((home & (kDieBits | kPicked)) == die + 1) {          // (its members are counted by a block that is running)
                uint32_t n;
                while ((n = load_fresh(&ctl->members)) == 0) __builtin_amdgcn_s_sleep(1);
                me = static_cast<int>(ticket);           // (< n: it was counted, or home had been another die's)
                count = static_cast<int>(n);
                owner = ticket == 0 && (home & kOwned) != 0;
            }
        }
        sh[0] = me;
        sh[1] = count;
        sh[2] = owner;
    }
    __syncthreads();
    // (the same for all: said so, or every loop over members is one whose lanes may part)
    return DieMember{ctl, __builtin_amdgcn_readfirstlane(sh[0]), __builtin_amdgcn_readfirstlane(sh[1])};
}

// At the end of a member, by one thread: the die is given back.
__device__ __forceinline__ void die_leave(uint32_t *taken, const int *sh)
{
    if (sh[2]) __hip_atomic_store(taken + die_number(), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every member has come this far, and what its wavefronts had stored and waited for (wait_for_memory) before this one's call can
// be read with load_fresh.  One wavefront of every member calls it, with the same phase, one more each time (from 1); the
// fewer loads it has under way the better: it waits for them too.  Returns member i's value in lane i (0 past the last
// member); sets *dead if the wait was given up.
__device__ __forceinline__ uint32_t die_wait(const DieMember &d, uint32_t phase, uint32_t value, int *dead)
{
    if (d.count == 1) return threadIdx.x % kWave == 0 ? value : 0u;
    uint64_t *flag = d.ctl->flag[phase & 1];             // (two sets: no one is two phases ahead)
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == 0)
        __hip_atomic_store(flag + d.me, static_cast<uint64_t>(phase) << 32 | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    uint64_t t;
    for (int polls = 0;; ++polls) {
        t = lane < d.count ? __hip_atomic_load(flag + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                           : static_cast<uint64_t>(phase) << 32;
        if (__all(static_cast<uint32_t>(t >> 32) == phase)) break;
        if (polls == kPolls) {
            *dead = 1;
            break;
        }
    }
    asm volatile("" ::: "memory");
    return static_cast<uint32_t>(t);
}

}  // namespace dq
