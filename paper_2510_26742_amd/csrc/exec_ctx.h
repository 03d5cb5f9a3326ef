// Execution contexts of the action expert's kernel bodies.
//
// Every operation of the expert (Table 2, rows of the action expert) is written once as a device
// function ("body") templated on a context that answers three questions:
//   - which work item am I?                       cx.bx / cx.by / cx.bz  (blockIdx of a per-operation launch)
//   - how do I read what OTHER blocks produced in the operation before, and how do I publish what I produce?
//                                                  cx.ld(ptr) / cx.st(ptr, v)
//   - when may I start reading it?                 cx.wait_inputs()
// LaunchCtx is the per-operation launch (one graph node per operation, Section 3.1 of the paper): the kernel
// boundary orders and publishes everything, loads and stores are ordinary, the wait is empty.
// PersistCtx is one persistent kernel for the whole denoise loop (Section 5.2: software barriers instead of
// kernel boundaries, weights requested before the wait).  The chip has eight dies with an L2 each that
// ordinary accesses do not keep coherent inside a kernel, so data that crosses blocks is stored write-through
// and loaded past the L2 (device-scope bits of the buffer instructions), so a barrier writes nothing back: it
// waits for stores to be acknowledged and exchanges flags; see grid barrier below.  Weights, tables and the prefix key/value cache are constant
// during the kernel and are read with ordinary loads before the wait.
// Both contexts run the same arithmetic in the same order, so the two paths agree bit for bit.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

// A pointer read from memory could point anywhere, so accesses through it are FLAT: they count towards both wait counters
// and are waited for with everything else in flight.  This says that it points to global memory (kernel arguments need
// no such help).
template <class T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)p;
}

// the same for a uniform pointer, and it is in scalar registers from here on: its arithmetic does not move behind a wait
__device__ __forceinline__ const char* computed_global(const char* p) {
  typedef const __attribute__((address_space(1))) char* Global;
  Global g = (Global)p;
  asm volatile("" : "+s"(g));
  return (const char*)g;
}

// Exchange between lanes l and l ^ 32 / l ^ 16 in one vector instruction (v_permlane32_swap_b32 and v_permlane16_swap_b32:
// the upper half (odd rows of 16) of the first operand changes places with the lower half (even rows) of the second), where
// a shuffle is a round trip through the LDS crossbar in the tail of a kernel body.
// swap_halves(a, b): lanes 0 .. 31 get (a, a of lane + 32), lanes 32 .. 63 get (b of lane - 32, b)
__device__ __forceinline__ u32x2_t swap_halves(unsigned a, unsigned b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); }
__device__ __forceinline__ float add_xor32(float v) {
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor16(float v) {
  const u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_xor32(float v) {
  const u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor16(float v) {
  const u32x2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

struct LaunchCtx {
  static constexpr bool kPersistent = false, kLean = false;
  int bx, by, bz;
  __device__ __forceinline__ static LaunchCtx from_block_idx() { return LaunchCtx{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z}; }
  template <class T>
  __device__ __forceinline__ T ld(const T* p) const { return *p; }
  template <class T>
  __device__ __forceinline__ T ld_bulk(const T* p) const { return *p; }
  template <class T>
  __device__ __forceinline__ void st(T* p, const T& v) const { *p = v; }
  __device__ __forceinline__ unsigned off(const void*) const { return 0; }
  template <class T>
  __device__ __forceinline__ void st_off(unsigned, const T&) const {}
  __device__ __forceinline__ void wait_inputs() const {}
  __device__ __forceinline__ void mark(int) const {}
  __device__ __forceinline__ int tid() const { return (int)threadIdx.x; }
  static constexpr bool staged = false;
};

// Requests 1 KiB of a wave straight into LDS: lane l's 16 bytes at base + off land at byte address lds + 16 l.  Assembly,
// because behind the builtin the compiler makes every LDS read wait for all loads in flight; whoever reads the data waits
// for vmcnt(0) first.  base, lds: uniform
__device__ __forceinline__ void request_to_lds(const char* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const unsigned char* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

// ------------------------------------------------------------------------------------------------
// Grid barrier of the persistent kernel.  A block arrives by storing the epoch into its own word of its die's flag line
// (hardware register XCC_ID names the die a wave runs on): an ordinary store, which stays in the die's L2, where the
// other blocks of the die see it with an L1-bypassing load.  One block per die, the leader, polls those words - one
// 128-byte line for 32 blocks - and then tells every die, in a word of that die's own cache line, that its die has
// completed the epoch; a block polls its die's line (one 32-byte load) until all dies that hold blocks have.  Two
// store-to-poll hops, one inside the die and one between dies, and no read-modify-write: a counter per die instead of
// the flags serialises 32 atomics in the L2 (probe of 256 blocks, per barrier: 1.56 us with counters, 1.05 us with
// flags; with a store before and a load after it 2.27 against 1.86).  There is no cache write-back in the barrier:
// everything another block will read is stored write-through (PersistCtxT::st) and each wave waits until its own stores
// are acknowledged.  The leader requests its own prefetch only after that (loads return in order per compute unit: its
// polls would queue behind it), so it is chosen among the blocks that the attention leaves idle.  Arrive and wait are separate calls, so a block requests the next operation's constant
// operands between them.  Every wait is bounded: when the bound runs out the error word is raised,
// every wait that is not complete by then or starts later gives up within 64 polls (give_up), so the kernel drains, and the
// host reports the failure.
// Words (unsigned; groups 128 bytes apart so that no two are in one cache line):
enum {
  GB_ERR = 0,          // != 0: a bounded wait ran out
  GB_START = 32,       // start-up counter: blocks registered
  GB_TICKETS = 33,     // init_some: blocks that asked to take part, + GB_BACK for each that did in the turn before, | GB_CLOSED once it goes on without the others
  GB_TAKEN = 34,       // init_some: blocks that take part, once that is decided, | GB_REST if they do all that is left
  GB_MEMBERS = 64,     // + 32 x: blocks resident on die x
  GB_LEADER = 320,     // + 32 x: 1 + index of the block that leads die x (+ 2^16 if it asked to)
  GB_DONE = 576,       // + 32 y + x: last epoch that die x completed, as told to die y (one cache line per reading die)
  GB_SINK = 832,       // never read: where a read-ahead block would store its folded loads (keeps the loads alive)
  GB_FLAGS = 864,      // + GB_MAX_BLOCKS x + r: last epoch that block r of die x arrived at
  GB_MAX_BLOCKS = 256, // largest grid
  GB_WORDS = GB_FLAGS + 8 * GB_MAX_BLOCKS
};
constexpr unsigned GB_CLOSED = 1u << 16, GB_BACK = 1u << 20, GB_REST = 1u << 16;   // (more than any grid)
constexpr long long GB_WINDOW = 2500;   // of the 100 MHz counter: 25 us, within which the blocks of a launch on an otherwise idle device have long come (10)
// A loop that goes on with the blocks that have come does so in turns of GB_LAYERS, with barrier words for each; the blocks that have come meanwhile join in
// between.  With all of the grid a turn does all layers that are left, and so does the last one.  So a moment in which other work holds the chip costs no
// more than that and a turn on the few units that were free.  ms of pi0_prefill, the blocks of the start throughout / turns of 1 / 2 / 4 layers:
// 27 / 3 layers (1.8 alone) beside a loop on 224 units for 3 ms  8.8 / 4.6 / 4.8 / 5.25,
// 27 / 18 layers beside a loop that stays, on 64 units 7.43 / 7.93 / 7.61 / 7.46, 128 7.94 / 8.38 / 8.22 / 8.04, 160 10.43 / 10.75 / 10.68 / 10.52.
// (A kernel that ends after 1, 2, 4, 8 layers and is launched again: 6.3 in the first case, and the launches that find nothing left cost 1.7 us each,
// 222 -> 236 us over two layers, where turns cost 0 .. 3.  Over eighteen, alone, 1 view 2562 -> 2551, 2 views + 21 tokens 4035 -> 4054: the layers' code
// lies in another loop and is another one.)
constexpr int GB_LAYERS = 4, GB_TURNS = 8;
inline int gb_turns(int layers) { return layers >= GB_LAYERS * GB_TURNS ? GB_TURNS : (layers + GB_LAYERS - 1) / GB_LAYERS; }

// Barrier words to zero, in a launch ahead of the kernel's
__device__ __forceinline__ void gb_clear(unsigned* sync, int turns, unsigned i) {   // piece i of the words of that many turns; the error words stay as they are
  constexpr unsigned PIECES = (GB_WORDS - GB_START) / 4;
  if (i < PIECES * (unsigned)turns) reinterpret_cast<uint4*>(sync + i / PIECES * GB_WORDS + GB_START)[i % PIECES] = uint4{0u, 0u, 0u, 0u};
}

// TRACE: a timeline is recorded (a kernel of its own: the code for it in every operation costs instruction cache).  LEAN: no address of the
// barrier's words stays in registers from one barrier to the next, for kernels with an operation that takes all there are (a spilled
// address is a round trip in every barrier)
template <bool TRACE, bool LEAN = false>
struct GridBarrierT {
  unsigned* w;          // GB_WORDS words, zeroed before the launch
  unsigned xcc;         // die of this block
  unsigned members;     // blocks on this die
  unsigned rank;        // this block's place among them
  bool leader;          // this block tells the other dies when this one is complete
  unsigned present;     // bit x set: die x holds at least one block
  unsigned spin_limit;
  unsigned epoch;       // barriers this block has arrived at
  long long* trace;     // optional: where thread 0 notes the wall clock (100 MHz) when a wait ends

  __device__ __forceinline__ static unsigned ld_dev(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ static void st_dev(unsigned* p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

  // (opaque: the compiler knows these values as the same in all lanes, drops the builtin and then has addresses in vector registers.  Not
  // the instruction itself as assembly, in front of which the compiler leaves no wait state for the register that it reads)
  __device__ __forceinline__ static unsigned scalar(unsigned v) {
    asm volatile("" : "+v"(v));
    return (unsigned)__builtin_amdgcn_readfirstlane((int)v);
  }

  // a constant, made here each time: ahead of a loop that this code is in, it would hold a register throughout
  __device__ __forceinline__ static unsigned here(unsigned v) {
    asm volatile("" : "+s"(v));
    return v;
  }

  // all threads of the block; one counter barrier, after which every block knows who shares its die
  // may_lead: the block is one of those that should lead their die (if a die has none, another one does)
  __device__ __forceinline__ void init(unsigned* words, unsigned limit, bool may_lead) {
    w = as_global(words);
    spin_limit = limit;
    epoch = 0;
    trace = nullptr;
    xcc = (unsigned)__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7u;   // XCC_ID, bits 3:0
    unsigned r = 0;
    if (threadIdx.x == 0) {
      __hip_atomic_fetch_max(&w[GB_LEADER + 32 * xcc], here(blockIdx.x + 1u + (may_lead ? 1u << 16 : 0u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      r = __hip_atomic_fetch_add(&w[GB_MEMBERS + 32 * xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // both are in place before this block counts as registered
      __hip_atomic_fetch_add(&w[GB_START], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned spins = 0;
      while (ld_dev(&w[GB_START]) < gridDim.x) {
        __builtin_amdgcn_s_sleep(2);
        if (++spins > spin_limit || ld_dev(&w[GB_ERR]) != 0u) { st_dev(&w[GB_ERR], 1u); break; }
      }
    }
    __syncthreads();
    rank = (unsigned)__builtin_amdgcn_readfirstlane((int)r);   // of the first wave, which alone uses it (no shared memory: a kernel may want all of it)
    members = ld_dev(&w[GB_MEMBERS + 32 * xcc]);
    leader = (ld_dev(&w[GB_LEADER + 32 * xcc]) & 0xffffu) == (unsigned)blockIdx.x + 1u;
    present = 0;
    for (unsigned k = 0; k < 8u; k++) present |= ld_dev(&w[GB_MEMBERS + 32 * k]) != 0u ? 1u << k : 0u;
  }

  // As init, for kernels whose operations any number of blocks can share out: goes on as soon as all blocks of the grid have come, or with fewer once
  // none has come for GB_WINDOW x grid / n with n there, half of what a layer then takes them at most, so that no wait depends on compute units that other work holds.
  // A block that comes later waits for the next turn, in front of which the blocks of the one before come here again; one for which none is
  // left ends (false), and so does one whose wait ran out here, and any once a wait has (the error words stay raised).
  // most: no more than this many at once; 0: init, all of the grid (a round trip less).  first, stride: this block's items are first, first + stride, ..
  // (all of the grid: blockIdx.x, gridDim.x).  begin, end: the layers to do.  first, stride, end: before, those of the turn before, 0 at the
  // start.  shared: four words of shared memory that nothing else uses.
  // pi0_prefill, which promises its caller no resident grid, runs its loops so: 2 views + 21 tokens and two denoises, as launches -> so, 12.16 -> 11.87 ms.
  __device__ __forceinline__ bool init_some(unsigned* words, unsigned limit, bool may_lead, unsigned most, unsigned* shared, int layers, int& first, int& stride, int& begin,
                                            int& end) {
    if (scalar(most) == 0u) {
      init(words, limit, may_lead);
      if (LEAN) {
        members = scalar(members);
        present = scalar(present);
      }
      first = (int)scalar(blockIdx.x);
      stride = (int)scalar(gridDim.x);
      begin = 0;
      end = layers;
      return true;
    }
    spin_limit = limit;
    epoch = 0;
    trace = nullptr;
    xcc = (unsigned)__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7u;   // XCC_ID, bits 3:0
    if (thread() == 0u) {
      const unsigned grid = gridDim.x;
      if (most > grid) most = grid;
      unsigned ticket = 0, r = 0, taken = 0, k = (unsigned)end / GB_LAYERS;
      bool in = false;
      for (bool back = k != 0u;; back = false, k++) {
        unsigned* const v = as_global(words) + k * GB_WORDS;
        const unsigned before = __hip_atomic_fetch_add(&v[GB_TICKETS], back ? here(GB_BACK + 1u) : here(1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ticket = before & (GB_CLOSED - 1u);
        in = (before & GB_CLOSED) == 0u && ticket < most;
        const unsigned last = k == GB_TURNS - 1 || ((int)k + 1) * GB_LAYERS >= layers ? GB_REST : 0u;
        if (in) {
          if (k == 0u && ticket + 1u == most) st_dev(&v[GB_TAKEN], most | (most == grid ? GB_REST : last));
          __hip_atomic_fetch_max(&v[GB_LEADER + 32 * xcc], here(blockIdx.x + 1u + (may_lead ? 1u << 16 : 0u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          r = __hip_atomic_fetch_add(&v[GB_MEMBERS + 32 * xcc], here(1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // both are in place before this block counts as registered
          __hip_atomic_fetch_add(&v[GB_START], here(1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // who closes the count: in the first turn any block that is tired of waiting, later the first one of the turn before, once all of that one are back
        const bool closes = k == 0u ? in : back && first == 0;
        long long since = (long long)wall_clock64();
        unsigned seen = ticket, spins = 0;
        while (true) {
          taken = ld_dev(&v[GB_TAKEN]);   // (all loads of a poll at once)
          const unsigned started = ld_dev(&v[GB_START]), tickets = ld_dev(&v[GB_TICKETS]), error = ld_dev(&v[GB_ERR]) | (k != 0u ? ld_dev(&v[GB_ERR] - GB_WORDS) : 0u);
          if (++spins > spin_limit || error != 0u) {
            st_dev(&v[GB_ERR], here(1u));
            taken = 0;   // takes no part (a stride of one in its place would have every block do all of the work)
            break;
          }
          if (taken != 0u && (!in || started >= (taken & (GB_REST - 1u)))) break;
          if (closes && taken == 0u) {
            bool close = k != 0u && tickets / GB_BACK == (unsigned)stride;
            if (k == 0u) {
              if (tickets != seen) {
                seen = tickets;
                since = (long long)wall_clock64();
              } else {
                close = ((long long)wall_clock64() - since) * (tickets & (GB_CLOSED - 1u)) > GB_WINDOW * grid;
              }
            }
            if (close) {
              const unsigned came = __hip_atomic_fetch_or(&v[GB_TICKETS], here(GB_CLOSED), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              const unsigned n = (came & (GB_CLOSED - 1u)) < most ? came & (GB_CLOSED - 1u) : most;
              if ((came & GB_CLOSED) == 0u) st_dev(&v[GB_TAKEN], n | (n == grid ? GB_REST : last));
            }
          }
          if (in) __builtin_amdgcn_s_sleep(2);
          else __builtin_amdgcn_s_sleep(32);   // waits for a turn's end
        }
        if (in || taken == 0u || taken >= GB_REST) break;
      }
      shared[0] = in ? taken : 0u;
      shared[1] = ticket;
      shared[2] = r;
      shared[3] = k;
    }
    __syncthreads();
    const unsigned taken = scalar(shared[0]), ticket = scalar(shared[1]), n = taken & (GB_REST - 1u);
    first = (int)scalar(n == gridDim.x ? blockIdx.x : ticket);
    stride = (int)n;
    rank = scalar(shared[2]);
    const int turn = (int)scalar(shared[3]);
    __syncthreads();
    if (n == 0u) return false;
    w = as_global(words) + turn * GB_WORDS;
    begin = turn * GB_LAYERS;
    end = taken < GB_REST ? begin + GB_LAYERS : layers;
    members = ld_dev(&w[GB_MEMBERS + 32 * xcc]);
    leader = (ld_dev(&w[GB_LEADER + 32 * xcc]) & 0xffffu) == (unsigned)blockIdx.x + 1u;
    present = 0;
    for (unsigned k = 0; k < 8u; k++) present |= ld_dev(&w[GB_MEMBERS + 32 * k]) != 0u ? 1u << k : 0u;
    if (LEAN) {
      members = scalar(members);
      present = scalar(present);
    }
    return true;
  }

  // the error word is looked at on every 64th poll: behind each poll it would double the time between two polls
  __device__ __forceinline__ bool give_up(unsigned spins) const {
    return spins > spin_limit || ((spins & 63u) == 0u && ld_dev(&w[GB_ERR]) != 0u);
  }

  __device__ __forceinline__ static unsigned thread() {
    unsigned t = threadIdx.x;
    if (LEAN) asm volatile("" : "+v"(t));
    return t;
  }

  __device__ __forceinline__ void fail() {
    unsigned one = 1u;
    if (LEAN) asm volatile("" : "+v"(one));
    st_dev(&w[GB_ERR], one);
  }

  // all threads of the block, after the block's last store of the operation
  __device__ __forceinline__ void arrive() {
    // A block without a work item in an operation arrives without having waited for the operation before (flags and epochs
    // only grow, so a later epoch stands for the earlier ones too), and goes on to prefetch for the one after.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores have been acknowledged (a workgroup-scope
                                                        // fence does not wait for them)
    __syncthreads();
    epoch++;
    const unsigned t = thread();
    unsigned* const flags = w + GB_FLAGS + GB_MAX_BLOCKS * xcc;
    if (t == 0) __hip_atomic_store(flags + rank, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (leader) {
      if (t < 64) {
        unsigned spins = 0;
        while (true) {
          bool behind = false;
          for (unsigned r = t; r < members; r += 64) behind |= ld_dev(flags + r) < epoch;
          if (__builtin_amdgcn_ballot_w64(behind) == 0ull) break;
          if (give_up(++spins)) {
            if (t == 0) fail();
            break;
          }
        }
        if (t < 8) st_dev(&w[GB_DONE + 32 * t + xcc], epoch);
      }
      __syncthreads();   // loads return in order per compute unit: no prefetch of the leader's other waves in front of its polls
    }
  }

  // all threads of the block: returns once every block has arrived at the barrier this block arrived at last
  __device__ __forceinline__ void wait() {
    const unsigned t = thread();
    if (t < 8) {   // lane x reads what die x has told this die
      const unsigned lane = t;
      const bool counts = ((present >> lane) & 1u) != 0u;
      unsigned spins = 0;
      while (true) {
        const bool behind = counts && ld_dev(&w[GB_DONE + 32 * xcc + lane]) < epoch;
        if (__builtin_amdgcn_ballot_w64(behind) == 0ull) break;
        if (give_up(++spins)) {
          if (lane == 0) fail();
          break;
        }
      }
    }
    __syncthreads();
    if (TRACE && trace != nullptr && threadIdx.x == 0) *trace = (long long)wall_clock64();
  }
};

// cache-policy bit of gfx950 buffer instructions: device scope (stores write through to memory, loads do
// not hit in the die's L2 or the compute unit's L1)
#define PI0_AUX_DEVICE_SCOPE 16

// BULK_CACHED: the operation's large inputs (activation matrices, statistic partials, attention operands) are read
// with ordinary cached loads, so that the 32 blocks of a die fetch them from memory once instead of 32 times (read
// past the L2 by every block, an operation's inputs cross the fabric 256 times: measured 2 - 3.5 us per operation).
// That is only coherent if no cache of the reading die can hold an older copy of those addresses, which the caller
// guarantees by giving every operation instance of the loop its own never-read buffers whose cache lines are each
// written by one block only ("fresh" data path of the barrier experiment).
template <bool BULK_CACHED, bool TRACE, bool LEAN = false>
struct PersistCtxT {
  static constexpr bool kPersistent = true;
  static constexpr bool kLean = LEAN;
  int bx, by, bz;                  // work item of the current operation
  __amdgpu_buffer_rsrc_t arena;    // buffer resource over the activation arena
  const char* arena_base;
  GridBarrierT<TRACE, LEAN>* bar;
  bool staged = false;             // weights of the item's first feature tile are in the body's shared memory already
  int thread;                      // threadIdx.x, made opaque per operation: per-lane address arithmetic of one operation
                                   // is then not hoisted out of the layer loop, where it would hold registers throughout

  __device__ __forceinline__ int tid() const { return thread; }
  __device__ __forceinline__ unsigned off(const void* p) const { return (unsigned)(reinterpret_cast<const char*>(p) - arena_base); }

  template <class T>
  __device__ __forceinline__ T ld(const T* p) const {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8 || sizeof(T) == 4 || sizeof(T) == 2, "access size");
    if constexpr (sizeof(T) == 16) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(arena, off(p), 0, PI0_AUX_DEVICE_SCOPE));
    else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(arena, off(p), 0, PI0_AUX_DEVICE_SCOPE));
    else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(arena, off(p), 0, PI0_AUX_DEVICE_SCOPE));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(arena, off(p), 0, PI0_AUX_DEVICE_SCOPE));
  }
  // store at an arena offset that was computed ahead of the wait, plus a constant
  template <class T>
  __device__ __forceinline__ void st_off(unsigned o, const T& v) const {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8 || sizeof(T) == 4 || sizeof(T) == 2, "access size");
    if constexpr (sizeof(T) == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), arena, o, 0, PI0_AUX_DEVICE_SCOPE);
    else if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), arena, o, 0, PI0_AUX_DEVICE_SCOPE);
    else if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), arena, o, 0, PI0_AUX_DEVICE_SCOPE);
    else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), arena, o, 0, PI0_AUX_DEVICE_SCOPE);
  }
  template <class T>
  __device__ __forceinline__ void st(T* p, const T& v) const {
    st_off(off(p), v);
  }
  template <class T>
  __device__ __forceinline__ T ld_bulk(const T* p) const {
    if constexpr (BULK_CACHED) return *p;
    else return ld(p);
  }
  __device__ __forceinline__ void wait_inputs() const { bar->wait(); }
  // timeline sample k (1 .. 4) of the current operation, by thread 0, when a timeline is being recorded
  __device__ __forceinline__ void mark(int k) const {
    if (TRACE && bar->trace != nullptr && thread == 0) bar->trace[2 + k] = (long long)wall_clock64();
  }
  template <bool B>
  __device__ __forceinline__ PersistCtxT<B, TRACE> as() const {
    PersistCtxT<B, TRACE> c;
    c.bx = bx; c.by = by; c.bz = bz; c.arena = arena; c.arena_base = arena_base; c.bar = bar; c.staged = staged; c.thread = thread;
    return c;
  }
};
