// Shared device-side definitions of the TABX kernels: launch arguments, per-lane registers,
// the LDS exchange area, the float32 helpers whose rounding both sides of the parity tests
// agree on, zone lookup, state load / store and the lane-to-unit mapping.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "tabx.h"

#pragma clang fp contract(off)

namespace tabx {

constexpr int kTileFloats = 1280;  // a tile of rows is about 4 KB, at least one row
constexpr int kMaxPasses = 10;     // most store passes of one flush of the packed form
constexpr int kMaxHalfPasses = 5;  // ... of half a row of two wavefronts: 268 chunks at most
constexpr int kPassBatch = 5;      // ... fetched from LDS together

struct PolicyArgs {
    TabxPolicy       pol;
    TabxPolicyMemory mem;          // mem_valid == nullptr: no policy in this launch
    const uint8_t   *controlled;
    uint8_t         *actions_out;
    uint8_t         *next_action;  // scripted tick: decided at the end of one call, applied by the next
};

// What the kernels read of TabxParams: all of it but the planner's last field, with which every pointer behind would
// lie eight bytes further in its cache line (stand-alone observe 13v13 x 68 8.28 us, then 8.49; step x 263 5.70, 5.83).
struct KParams {
    int32_t  num_envs, num_units, grid_w, grid_h, max_zones, max_steps;
    float    map_w, map_h, cell_size, dt, turn_rate, lava_dps, swamp_mult, reveal_time, boundary_frac;
    float    collision_alpha, collision_slop;
    int32_t  zone_shapes, num_levels;
    uint32_t level_seed;
    int32_t  hurtbox_cone, hit_all, env_id_offset, dynamics;
    float    move_gain, restitution;
};
static_assert(sizeof(KParams) == offsetof(TabxParams, shared_machine) && sizeof(TabxParams) == sizeof(KParams) + 4 &&
              offsetof(KParams, zone_shapes) == offsetof(TabxParams, zone_shapes) &&
              offsetof(KParams, level_seed) == offsetof(TabxParams, level_seed) &&
              offsetof(KParams, move_gain) == offsetof(TabxParams, move_gain), "the same fields, but for the last");

struct KArgs {
    KParams      p;
    TabxScenario sc;
    TabxState    st;
    const uint8_t *actions;
    const uint8_t *env_mask;
    float    *rewards;
    uint8_t  *dones;
    float    *obs;
    uint64_t *vis_mask;
    uint8_t  *action_mask;
    int       obs_dim;             // D
    int       envs_per_block;      // G
    int       rows_per_pass;       // S: consecutive rows the lanes of a wavefront work on at a time
    int       rows_per_tile;       // T: consecutive rows a wavefront assembles and stores together
    int       tiles;               // tiles of a full env group: ceil(G * N / T)
    int       passes_per_tile;     // T / S
    uint32_t  line;                // a tile's image starts where its first row does in memory, modulo line + 1 floats
                                   //     (of an `obs` on a 128-byte line: elsewhere more lines are shared)
    int       lines;               // enum Lines
    int       stage_floats;        // a wavefront's staging area in dynamic LDS (they come first)
    int       zone_chunks;         // ZC: 16-byte chunks of the zone part of a row
    unsigned  magic_n, magic_zc, magic_s, magic_tc;   // x / N, / ZC, / S, / (4 + ZC) as multiplications (see quotient)
    int       num_groups;          // workgroups that have envs to process
    int       zone_offset;         // the envs' zone descriptors (ZoneLds) in dynamic LDS, floats
    int       zones_in_lds;        // ... which sit there for elliptical zones, for deciding units and
                                   //     for the zone part of the rows
    int       script_offset;       // scripted units deciding in the observe stage: their LDS, floats
    int       groups_per_xcd;      // ceil(num_groups / 8)
    int       twin;                // 2, 3, 4 or 8: a workgroup has that many times the wavefronts that hold
                                   //    an env's units (one, or two from 65 units on); those step the
                                   //    envs, all of them make tiles
    int       obs_chunks;          // workgroups that share the tiles of one env group (>= 1)
    int       tiles_per_chunk;     // tiles per such workgroup
    int       packed;              // 1: rows with the units in registers (tabx_observe_packed.h)
    int       even;                // ... 64 < N: by the kernel that keeps three wavefronts per SIMD
    int       copy_passes;         // ... store passes of one flush, <= kMaxPasses
    int       rows_per_flush;      // ... R: consecutive rows of an env staged before they are stored
    int       obs_per_chunk;       // ... observers per workgroup that shares an env group
    unsigned  pace;                // a wavefront begins its flush n (from 0) no sooner than n times this after its
                                   //     first, in 1/16 of a tick of the constant clock (10 ns); 0: at will
    float     inv_cell;            // 1 / cell_size, used only when that is exact (power of two)
    uint32_t  cells;               // FAST_CELL: cells of one row's grid
    uint32_t  flags;               // Flag bits
    int       in_turn;             // the tiles are dealt to the wavefronts one by one, not in runs
    int       shared_machine;      // TabxParams.shared_machine (for plan_pace)
    PolicyArgs pa;
    float *global_stream;          // where the global state goes if it is streamed (st.global_state is null then)
};

// How the tiles of a group lie in the 128-byte lines of the rows: each starts on one; neighbours share one, which each
// writes its part of; a wavefront hands a shared one on to its next tile.
template <int V> struct Constant { static constexpr int value = V; };
enum Lines : int { LINES_OWN, LINES_SHARED, LINES_CARRIED };

// What a launch has to do besides the plain tick, one bit each.
enum Flag : uint32_t {
    DYNAMIC = 1,                   // persistent velocities
    COLLIDE = 2,                   // body collisions
    ELLIPSES = 4,                  // elliptical zones
    CONE_BOUND = 8, HIT_ALL = 16,  // the two other readings of the hurtbox
    KILLS = 32, RETURNS = 64,      // running episode metrics
    LEVELS = 128,                  // level bank
    FAST_CELL = 256,               // a cell grid; cell size a power of two, offsets by 24-bit products
    EARLY_CELL = 512,              // a cell grid, and nothing but its own motion decides where a unit is
};

// A paced wavefront (see plan_pace, tabx_kernels.hip): the low word of the constant clock (10 ns) when it starts
// its rows, and the wait until `due` ticks after that; nothing where `pace` / `due` is 0.  One block of scalar
// instructions each: as a loop of the compiler's, the branches cost launches without a pace up to 5 %.
__device__ __forceinline__ unsigned pace_start(unsigned pace)
{
    unsigned now;
    asm volatile("s_mov_b32 %0, 0\n\t"
                 "s_cmp_eq_u32 %1, 0\n\t"
                 "s_cbranch_scc1 .Lstarted%=\n\t"
                 "s_memrealtime vcc\n\t"
                 "s_waitcnt lgkmcnt(0)\n\t"
                 "s_mov_b32 %0, vcc_lo\n"
                 ".Lstarted%=:"
                 : "=&s"(now) : "s"(__builtin_amdgcn_readfirstlane((int)pace)) : "vcc", "scc");
    return now;
}

__device__ __forceinline__ void pace_wait(unsigned since, unsigned due)
{
    asm volatile("s_cmp_eq_u32 %1, 0\n\t"
                 "s_cbranch_scc1 .Lheld%=\n"
                 ".Lhold%=:\n\t"
                 "s_memrealtime vcc\n\t"
                 "s_waitcnt lgkmcnt(0)\n\t"
                 "s_sub_u32 vcc_lo, vcc_lo, %0\n\t"
                 "s_cmp_ge_u32 vcc_lo, %1\n\t"
                 "s_cbranch_scc1 .Lheld%=\n\t"
                 "s_sleep 1\n\t"
                 "s_branch .Lhold%=\n"
                 ".Lheld%=:"
                 : : "s"(__builtin_amdgcn_readfirstlane((int)since)), "s"(__builtin_amdgcn_readfirstlane((int)due)) : "vcc", "scc");
}

// Per-wavefront time stamps of an instrumented build (-DTABX_TRACE; compiled out of the product), eight
// per wavefront, for up to eight wavefronts per workgroup: slot 0 kernel entry, 6 before the step stage,
// 1 after it, 2 / 4 start and end of the rows, 5 kernel end, 7 hardware ids (3 is free).
#ifdef TABX_TRACE
constexpr int kTraceWaves = 8;
__device__ unsigned long long g_trace[1 << 21];
#define TABX_STAMP(slot)                                                                          \
    do {                                                                                          \
        if ((threadIdx.x & 63) == 0)                                                              \
            g_trace[(((size_t)blockIdx.x * kTraceWaves + (threadIdx.x >> 6)) * 8 + (slot)) & ((1 << 21) - 1)] = \
                wall_clock64();                                                                   \
    } while (0)
#else
#define TABX_STAMP(slot) do { } while (0)
#endif

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte store, 4-byte aligned
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));   // 8-byte store, 4-byte aligned

constexpr float kTwoPi = 6.28318530717958647692f;
// Sine and cosine of a heading in [0, 2*pi]: quadrant index n = trunc(theta *
// 2/pi + 1/2), remainder through a two-term split of pi/2, degree-9 / degree-8
// Taylor polynomials in Horner form with explicit fused multiply-adds.
__device__ __forceinline__ void heading_sincos(float theta, float &s, float &c)
{
    float q = theta * 0.63661977236758134308f;
    q = q + 0.5f;
    const int   n  = (int)q;
    const float fn = (float)n;
    float r = __builtin_fmaf(-fn, 1.57079637050628662109375f, theta);
    r       = __builtin_fmaf(-fn, -4.37113882867379435e-8f, r);
    const float r2 = r * r;
    float ps = __builtin_fmaf(r2, 1.0f / 362880.0f, -1.0f / 5040.0f);
    ps       = __builtin_fmaf(r2, ps, 1.0f / 120.0f);
    ps       = __builtin_fmaf(r2, ps, -1.0f / 6.0f);
    const float r3 = r * r2;
    const float sr = __builtin_fmaf(r3, ps, r);
    float pc = __builtin_fmaf(r2, 1.0f / 40320.0f, -1.0f / 720.0f);
    pc       = __builtin_fmaf(r2, pc, 1.0f / 24.0f);
    pc       = __builtin_fmaf(r2, pc, -0.5f);
    const float cr = __builtin_fmaf(r2, pc, 1.0f);
    const int quad = n & 3;
    const float a = (quad & 1) ? cr : sr;          // |sin| source
    const float b = (quad & 1) ? sr : cr;          // |cos| source
    s = (quad & 2) ? -a : a;
    c = (quad == 1 || quad == 2) ? -b : b;
}

__device__ __forceinline__ float clamp_between(float v, float lo, float hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Same value as clamp_between for finite inputs with lo <= hi (the sign of a zero
// result may differ, which the callers square away); one instruction.
__device__ __forceinline__ float median3(float v, float lo, float hi)
{
    return __builtin_amdgcn_fmed3f(v, lo, hi);
}

// What the step stage already knows about a unit and the observe stage needs again.
struct Carry {
    float cu, su;      // cosine / sine of the heading
    float ratio;       // hp / hmax
    int   tick;        // the env's tick counter after the step
    bool  restarted;   // the env's episode ended in this step
    int   warm;        // a byte loaded only to bring its cache line in (see step_env)
    // scripted units: the remembered target position as it was at the start of the call
    // (loaded with the state: at the end of the wavefront a load would queue behind its stores)
    int   mem_valid;
    float mem_x, mem_y;
};

// Registers of one unit: mutable state, then read-only specification.
struct Unit {
    float x, y, vx, vy, theta, hp, cd, reveal, cur_speed;
    int   alive;
    float hmax, radius, mass, speed, dmg, range, cooldown;
    float sight_angle, cos_half, sight_range, hurt_hw;
    int   team, enabled;
};

// Where a lane sits: env slot g of the workgroup, unit u of that env, `base` =
// workgroup lane of the env's unit 0, e = env index, k = e * N + u.  A lane without a unit of its own
// (`has` is false) stands at the group's first unit, so that every lane may load.
struct Place {
    int grp;           // which run of G envs this workgroup owns
    int chunk;         // which share of the rows of these envs it writes (stand-alone observe)
    int l, g, u, base, e;
    bool has;
    uint32_t k;        // (at most 2^30 units)
    int row;           // row of the scenario arrays that configures env e (its level, or e itself)
    uint32_t ks;       // row * N + u
};

// What the observe stage needs of every unit, left in LDS by the wavefront that holds it.
template <int L>
struct Records {
    float4 own[4][L];             // the four chunks of the unit's block in its own row:
                                  //   health, health / maximum, x, y
                                  //   heading, attack range, damage, cooldown left
                                  //   cooldown ratio, body radius, mass, sight angle
                                  //   alive, current speed, zone type, team
    float4 view[L];               // cos(heading), sin(heading), sight range^2, cos(cone / 2)
    float2 mark[L];               // hurtbox half-width, flags (an int): alive | team<<1 | heals<<2 |
                                  //   enabled<<3 | assassin<<4 | decides<<5 | hidden in its bush<<6 |
                                  //   bush key<<8 | zone code<<20
};

// Policy stage: what a deciding unit needs of itself and of the others.
template <int L>
struct Scan {
    float4 pose[L];               // x, y, cos(theta), sin(theta)
    float4 body[L];               // radius, max health, health, -
    int    seer[L];               // alive | team<<1 | concealable<<2 | bush key<<8
    float2 bound[L];              // beyond these squared distances, and behind this cone, nobody is seen (policy_env)
    int    who[L];                // the n-th deciding unit: its lane
};

struct NoRecords {};

// TILES: the observe stage reads records (tabx_observe.h).  POLICY: the policy stage runs (a single-
// wavefront workgroup without it keeps the 1.3 KB, which decide how many fit a CU: 10v10 x 8192 with
// body collisions 63.5 us with 11, 72.9 with 10).  PAIR: the two wavefronts that step an env
// are not the whole workgroup (group_barrier).
template <int WAVES, bool TILES, bool POLICY, bool PAIR_ = false>
struct __attribute__((aligned(64))) Shared {
    static constexpr int L = 64 * WAVES;
    static constexpr bool PAIR = PAIR_;
    union {
        struct {                  // step stage
            union {
                float4 pj[L];     // collision partners: x, y, radius, mass
                float4 aim0[L];   // combat, a striker's pose: x, y, cos(theta), sin(theta)
                float2 share[L];  // afterwards: this unit's term in the team-0 / team-1 ratio sums
            };
            float4 aim1[L];       // ... its hurtbox: range | target team in the sign bit,
                                  //     half-width, damage, cos(cone / 2)
            unsigned long long best[L];   // ... the closest body in it: (distance^2 bits, index)
        } st;
        std::conditional_t<POLICY, Scan<L>, NoRecords> po;      // policy stage
        std::conditional_t<TILES, Records<L>, NoRecords> rec;   // observe stage, rows in tiles
        struct {                  // observe stage, units in registers: what an observer's row needs
            float4 pose[L];       // x, y, cos(theta), sin(theta)
            float4 reach[L];      // attack range, hurtbox half-width, sight range^2, cos(cone / 2)
            int    seer[L];       // alive | team<<1 | heals<<2 | enabled<<3 | bush key<<8
        } ob;
    };
    uint64_t ballots[WAVES][4];
    int      level_rows[64];      // level bank: the row an env slot has just switched to, or -1
    unsigned arrivals;            // PAIR: arrivals of the two wavefronts at their barriers so far
};

// Orders LDS traffic between the lanes of a workgroup without waiting for global
// stores in flight (a full __syncthreads would drain them).  One wavefront executes
// its LDS operations in order, so a single-wave workgroup only pins the code order.
template <int WAVES>
__device__ __forceinline__ void lds_barrier()
{
    if (WAVES == 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
}

// The barrier of the wavefronts that hold the units of an env (the stages up to the rows).  Where they
// are two of more wavefronts of the workgroup, the others wait at the workgroup's own barrier
// meanwhile, so the two count each other's arrivals in LDS: the n-th barrier is passed once 2 n
// arrivals are in.  Both execute the same sequence of barriers (every condition around one is uniform
// over the env), and both are resident, so the wait ends.
template <int WAVES, class Sh>
__device__ __forceinline__ void group_barrier(Sh &sh)
{
    if constexpr (Sh::PAIR) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        unsigned before = 0;
        if ((threadIdx.x & 63) == 0)
            before = __hip_atomic_fetch_add(&sh.arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const unsigned goal = ((unsigned)__builtin_amdgcn_readfirstlane((int)before) | 1u) + 1u;
        while (__hip_atomic_load(&sh.arrivals, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < goal)
            __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    } else {
        lds_barrier<WAVES>();
    }
}

// The launch arguments where the kernel-argument segment holds them.  The kernels have more
// argument words than scalar registers; fields that are needed once, late or rarely (episode
// metrics, level bank, masks written at the end) are read through this pointer at the point of
// use instead of sitting in registers, or spilled, from the first instruction on.
typedef const __attribute__((address_space(4))) KArgs *LateArgs;
__device__ __forceinline__ LateArgs late_args()
{
    return (LateArgs)__builtin_amdgcn_kernarg_segment_ptr();
}

// The launch arguments, fetched anew for the stage that follows.  A wavefront has too few scalar registers
// for what all stages need between them, and what the compiler fetches once at the top it spills.
__device__ __forceinline__ const KArgs &again()
{
    LateArgs p = late_args();
    asm volatile("" : "+s"(p));
    return *(const KArgs *)p;
}

// Brings all lines of the launch arguments into the scalar cache at once.  The stages read them where they need
// them, and a lone wavefront would wait for each line in turn.
__device__ __forceinline__ void warm_args()
{
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    const Words w = (Words)late_args();
    uint32_t any = 0;
#pragma unroll
    for (int line = 0; line < (int)(sizeof(KArgs) / 64); ++line) any |= w[16 * line];
    asm volatile("" ::"s"(any));
}

// Element k of a per-unit array (at most 2^30 elements: its byte offset fits 32 bits, so the
// access is "uniform base + 32-bit lane offset" and needs no 64-bit address arithmetic per lane).
template <class T>
__device__ __forceinline__ T &at32(T *base, uint32_t k)
{
    char *const bytes = reinterpret_cast<char *>(const_cast<std::remove_const_t<T> *>(base));
    return *reinterpret_cast<T *>(bytes + (uint32_t)(k * (uint32_t)sizeof(T)));
}

// The same index, made anew where it is used.  (An index that reaches the accesses from another basic block
// is widened there, and each access then adds 64-bit addresses lane by lane.)
__device__ __forceinline__ uint32_t here(uint32_t k)
{
    asm volatile("" : "+v"(k));
    return k;
}

// Whether the launch has any of the bits.  (Tested where it is asked: kept from one place to the next, every
// answer takes two scalar registers, of which there are too few.)
__device__ __forceinline__ bool flagged(const KArgs &a, uint32_t bits)
{
    uint32_t f = a.flags;
    asm volatile("" : "+s"(f));
    return (f & bits) != 0;
}

// The zone code stored in the cell under a position (0 without a cell grid).
__device__ __forceinline__ int grid_cell(const KArgs &a, int row, float x, float y)
{
    if (flagged(a, FAST_CELL)) {
        // dividing by a power of two and multiplying by its reciprocal round identically
        int cx = (int)(x * a.inv_cell), cy = (int)(y * a.inv_cell);
        cx = cx > a.p.grid_w - 1 ? a.p.grid_w - 1 : cx;
        cy = cy > a.p.grid_h - 1 ? a.p.grid_h - 1 : cy;
        cx = cx < 0 ? 0 : cx;
        cy = cy < 0 ? 0 : cy;
        return (int)at32(a.sc.terrain, __umul24((uint32_t)row, a.cells) +
                                           __umul24((uint32_t)cy, (uint32_t)a.p.grid_w) + (uint32_t)cx);
    }
    const LateArgs late = late_args();
    const int8_t *const terrain = late->sc.terrain;
    if (terrain == nullptr) return 0;
    const int w = late->p.grid_w, h = late->p.grid_h;
    int cx = (int)(x / late->p.cell_size), cy = (int)(y / late->p.cell_size);
    cx = cx > w - 1 ? w - 1 : cx;
    cy = cy > h - 1 ? h - 1 : cy;
    cx = cx < 0 ? 0 : cx;
    cy = cy < 0 ? 0 : cy;
    return (int)terrain[((size_t)row * h + cy) * w + cx];
}

// Zone code under a position: low two bits = zone type, upper bits = zone identity; 0 = open.
// Cell-grid zones: the code stored in the cell.  Elliptical zones (App. A "Zones"): the last
// listed active zone whose ellipse holds the point, tested without division as
// (dx^2)*hy^2 + (dy^2)*hx^2 <= hx^2*hy^2; identity = slot index + 1, and `own_effect` returns
// that zone's effect magnitude.  `zd` = the env's zone descriptors (LDS or global), `row` = its
// row of the scenario arrays.
__device__ __forceinline__ int zone_at(const KArgs &a, const float *zd, int row, float x, float y,
                                       float &own_effect)
{
    if (flagged(a, ELLIPSES)) {
        int code = 0;
        // four slots per round, their descriptors fetched together (a slot beyond the last one
        // re-reads the last and is masked out), so that the fetch latency is paid once per round
        const int Z = a.p.max_zones;
        for (int z0 = 0; z0 < Z; z0 += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int z = z0 + k;
                const float *d = zd + 6 * (z < Z ? z : Z - 1);
                const float kind = d[0];
                const float dx = x - d[1];
                const float dy = y - d[2];
                const float hx2 = d[3] * d[3];
                const float hy2 = d[4] * d[4];
                const bool inside = (z < Z) && (kind != 0.0f) &&
                                    (((dx * dx) * hy2) + ((dy * dy) * hx2) <= hx2 * hy2);
                code = inside ? (((int)kind & 3) | ((z + 1) << 2)) : code;
                own_effect = inside ? d[5] : own_effect;
            }
        }
        return code;
    }
    return grid_cell(a, row, x, y);
}
// Effect magnitude that applies in the zone just found: its own (elliptical zones) or the
// global parameter (cell grid).
__device__ __forceinline__ float zone_magnitude(const KArgs &a, float own_effect, float global_value)
{
    return flagged(a, ELLIPSES) ? +own_effect : +global_value;
}

// x / n for the small values that occur inside a workgroup, magic = ceil(65536 / n) from the host: exact
// as long as x * (magic * n - 65536) < 65536, so for every x < 1024 with n <= 64, and for the zone chunks
// of a group, x < 64 * 24 with n <= 24.
__device__ __forceinline__ int quotient(int x, unsigned magic)
{
    return (int)(__umul24((unsigned)x, magic) >> 16);
}

// Product of small non-negative values: one full-rate instruction.
__device__ __forceinline__ int mul24(int x, int y) { return (int)__umul24((unsigned)x, (unsigned)y); }

// The lanes of the wavefront for which `v` holds.
__device__ __forceinline__ uint64_t lanes_where(bool v) { return __builtin_amdgcn_ballot_w64(v); }

// Row of the scenario arrays that configures env `env`.
__device__ __forceinline__ int row_of(const KArgs &a, int env)
{
    if (a.p.num_levels <= 0) return env;
    const int lv = a.st.level[env];
    return lv < 0 ? 0 : (lv >= a.p.num_levels ? a.p.num_levels - 1 : lv);
}

// How many envs the group holds (the last one may be partial, surplus workgroups have none).
__device__ __forceinline__ int envs_of_group(const KArgs &a, int grp)
{
    const int left = grp < a.num_groups ? a.p.num_envs - grp * a.envs_per_block : 0;
    return left < a.envs_per_block ? left : a.envs_per_block;
}

// The zone descriptors of the workgroup's envs in LDS, ZC 16-byte chunks per env, laid out as the
// zone part of the rows (so they can be read as 6 floats per slot, and an inactive slot is zero).  A slot is (type, centre x, centre y, three more), so three chunks
// hold two slots and a chunk has the centre of one slot at most: chunk 0 of three has x and y of the
// first slot in its floats 1 and 2, chunk 1 the second slot's x in float 3, chunk 2 its y in float 0.
// `rel` is -1 if that slot is active (its centre is relative to the observer), else 0.
struct ZoneLds {
    float4 *val;      // [G][ZC]
    int    *rel;      // [G][ZC]
};

__device__ __forceinline__ ZoneLds zone_lds(const KArgs &a, float *dyn)
{
    float4 *v = reinterpret_cast<float4 *>(dyn + a.zone_offset);
    return {v, reinterpret_cast<int *>(v + a.envs_per_block * a.zone_chunks)};
}

// x / 3 for x < 100
__device__ __forceinline__ int third(int x) { return mul24(x, 171) >> 9; }

// Chunk zc of env slot g, whose zones are row `row` of the descriptors.  Its four floats and the types of
// the two slots they can belong to are fetched together: asking for the floats of active slots only is a
// second round trip, which a small batch waits for (step of 30v33 x 252, four ellipses: 9.9 -> 9.1 us).
// LATE: the arguments are read where they are needed.  The kernels of two wavefronts per env have no scalar
// registers left for them (they would reserve scratch memory); in the others it costs (5v5 x 4096 11.3 ->
// 12.1 us).
template <bool LATE>
__device__ __forceinline__ void put_zone_chunk(const KArgs &a, const ZoneLds &Z, int g, int zc, int row)
{
    const LateArgs late = late_args();
    const int zlen = 6 * (LATE ? late->p.max_zones : a.p.max_zones);
    const int ZC = LATE ? late->zone_chunks : a.zone_chunks;
    const float *d = (LATE ? late->sc.zone_desc : a.sc.zone_desc) + (size_t)row * zlen;
    const int first_slot = 3 * (third(4 * zc) & ~1);         // first float of the slot of float 4 zc
    const int last_slot = first_slot + (4 * zc + 3 >= first_slot + 6 ? 6 : 0);
    const float kind[2] = {d[first_slot], d[last_slot < zlen ? last_slot : 0]};
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = d[4 * zc + k < zlen ? 4 * zc + k : 0];
    int rel = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int zz = 4 * zc + k;
        const bool second = zz >= first_slot + 6;
        const bool active = zz < zlen && (second ? kind[1] : kind[0]) != 0.0f;
        const int comp = zz - (second ? last_slot : first_slot);
        v[k] = active ? v[k] : 0.0f;
        if (active && (comp == 1 || comp == 2)) rel = -1;
    }
    Z.val[g * ZC + zc] = make_float4(v[0], v[1], v[2], v[3]);
    Z.rel[g * ZC + zc] = rel;
}

// All zone chunks of the workgroup's envs, by the LANES lanes that call it (`l`: index among them).
template <int LANES, bool LATE>
__device__ __forceinline__ void put_zones(const KArgs &a, const ZoneLds &Z, int grp, int l)
{
    const LateArgs late = late_args();
    const int envs_here = envs_of_group(a, grp);
    const int ZC = LATE ? late->zone_chunks : a.zone_chunks;
    for (int q = l; q < envs_here * ZC; q += LANES) {
        const int g = quotient(q, LATE ? late->magic_zc : a.magic_zc);
        put_zone_chunk<LATE>(a, Z, g, q - g * ZC, row_of(a, grp * a.envs_per_block + g));
    }
}

__device__ __forceinline__ void load_spec(const KArgs &a, uint32_t k, Unit &U)
{
    U.enabled = at32(a.sc.enabled, k);
    U.team = at32(a.sc.team, k);
    U.hmax = at32(a.sc.hmax, k);
    U.radius = at32(a.sc.radius, k);
    U.speed = at32(a.sc.speed, k);
    U.dmg = at32(a.sc.dmg, k);
    U.range = at32(a.sc.range, k);
    U.cooldown = at32(a.sc.cooldown, k);
    U.cos_half = at32(a.sc.sight_cos_half, k);
    U.hurt_hw = at32(a.sc.hurt_halfwidth, k);
    U.mass = at32(a.sc.mass, k);
    U.sight_angle = at32(a.sc.sight_angle, k);
    U.sight_range = at32(a.sc.sight_range, k);
}

// The unit's state and specification; first what decides where the unit is after its move.  STEP_ONLY: no
// rows follow, which alone need the mass (but for body collisions), the cone (but where it bounds the hurtbox)
// and the sight; load_more has the exceptions.
template <bool STEP_ONLY>
__device__ __forceinline__ void load_unit(const KArgs &a, uint32_t k, uint32_t ks, Unit &U)
{
    U.alive = at32(a.st.alive, k);
    U.enabled = at32(a.sc.enabled, ks);
    U.x = at32(a.st.x, k);
    U.y = at32(a.st.y, k);
    U.vx = at32(a.st.vx, k);
    U.vy = at32(a.st.vy, k);
    __builtin_amdgcn_sched_barrier(0x78f);     // (no load crosses)
    U.cur_speed = at32(a.st.cur_speed, k);
    U.theta = at32(a.st.theta, k);
    U.cd = at32(a.st.cd, k);
    U.hp = at32(a.st.hp, k);
    U.reveal = at32(a.st.reveal, k);
    U.team = at32(a.sc.team, ks);
    U.hmax = at32(a.sc.hmax, ks);
    U.dmg = at32(a.sc.dmg, ks);
    U.range = at32(a.sc.range, ks);
    U.hurt_hw = at32(a.sc.hurt_halfwidth, ks);
    U.radius = at32(a.sc.radius, ks);
    U.cooldown = at32(a.sc.cooldown, ks);
    U.speed = at32(a.sc.speed, ks);
    if (!STEP_ONLY) {
        U.mass = at32(a.sc.mass, ks);
        U.cos_half = at32(a.sc.sight_cos_half, ks);
        U.sight_angle = at32(a.sc.sight_angle, ks);
        U.sight_range = at32(a.sc.sight_range, ks);
    }
}

__device__ __forceinline__ void load_more(const KArgs &a, uint32_t ks, Unit &U)
{
    if (flagged(a, COLLIDE)) U.mass = at32(late_args()->sc.mass, here(ks));
    if (flagged(a, CONE_BOUND)) U.cos_half = at32(late_args()->sc.sight_cos_half, here(ks));
}

// The bytes as 0 or 1: any non-zero one means the adversaries, or alive.  Apart from the loads, since
// folding a byte waits for it: what is asked for after that is a round trip later.  (The empty
// instruction keeps the compiler from moving the folding, and with it the wait, up to the loads.)
__device__ __forceinline__ void fold_byte(int &byte)
{
    asm volatile("" : "+v"(byte));
    byte = (byte + 255) >> 8;
}

__device__ __forceinline__ void store_state(const KArgs &a, uint32_t k, const Unit &U)
{
    k = here(k);
    at32(a.st.x, k) = U.x;
    at32(a.st.y, k) = U.y;
    at32(a.st.vx, k) = U.vx;
    at32(a.st.vy, k) = U.vy;
    at32(a.st.theta, k) = U.theta;
    at32(a.st.hp, k) = U.hp;
    at32(a.st.cd, k) = U.cd;
    at32(a.st.reveal, k) = U.reveal;
    at32(a.st.cur_speed, k) = U.cur_speed;
    at32(a.st.alive, k) = (uint8_t)U.alive;
}

// Episode start for one unit: spawn pose, full health, timers cleared.  Returns
// the terrain cell code under the spawn point.
__device__ __forceinline__ int spawn_unit(const KArgs &a, const float *zd, int row, uint32_t ks,
                                          Unit &U, float &zeff)
{
    U.x = at32(a.sc.init_x, ks);
    U.y = at32(a.sc.init_y, ks);
    U.theta = at32(a.sc.init_theta, ks);
    U.vx = 0.0f;
    U.vy = 0.0f;
    U.hp = U.enabled ? U.hmax : 0.0f;
    U.cd = 0.0f;
    U.reveal = 0.0f;
    U.alive = U.enabled ? 1 : 0;
    const int code = zone_at(a, zd, row, U.x, U.y, zeff);
    U.cur_speed = (code & 3) == TABX_ZONE_SWAMP
                      ? U.speed * zone_magnitude(a, zeff, a.p.swamp_mult) : U.speed;
    return code;
}

// SHARED_GROUPS: several workgroups may share the rows of an env group (stand-alone observe).
template <int WAVES, bool SHARED_GROUPS = false>
__device__ __forceinline__ Place locate(const KArgs &a)
{
    Place P;
    const int N = a.p.num_units;
    P.l = (int)threadIdx.x;           // (only the wavefronts that step or publish hold units)
    // Workgroups are dealt to the 8 XCDs round robin; give each XCD one contiguous eighth of
    // the env range, so that neighbouring env groups, which share the cache lines at the ends
    // of their SoA segments, meet in the same L2.
    const int slot = (int)(blockIdx.x >> 3);
    const int in_xcd = SHARED_GROUPS && a.obs_chunks > 1 ? slot / a.obs_chunks : slot;
    P.chunk = SHARED_GROUPS ? slot - in_xcd * a.obs_chunks : 0;
    P.grp = in_xcd < a.groups_per_xcd ? (int)(blockIdx.x & 7) * a.groups_per_xcd + in_xcd : a.num_groups;
    P.has = P.l < envs_of_group(a, P.grp) * N;
    const int lane = P.has ? P.l : 0;
    P.g = WAVES == 1 ? quotient(lane, a.magic_n) : 0;
    P.base = WAVES == 1 ? mul24(P.g, N) : 0;
    P.u = lane - P.base;
    P.e = P.grp * a.envs_per_block + P.g;
    P.k = (uint32_t)(P.grp * a.envs_per_block) * (uint32_t)N + (uint32_t)lane;
    P.row = P.e;
    P.ks = P.k;
    if (a.p.num_levels > 0 && P.grp < a.num_groups) {      // folded into the bank whatever the array holds
        const int lv = at32(a.st.level, (uint32_t)P.e);
        P.row = lv < 0 ? 0 : (lv >= a.p.num_levels ? a.p.num_levels - 1 : lv);
        P.ks = (uint32_t)P.row * (uint32_t)N + (uint32_t)P.u;
    }
    return P;
}

// The lanes of the caller's env (envs of one wavefront).
__device__ __forceinline__ uint64_t lanes_of_env(const Place &P, int N)
{
    return (N >= 64 ? ~0ull : ((1ull << N) - 1ull)) << P.base;
}

// How many lanes of the caller's env satisfy each of K predicates.
template <int WAVES, int K, class Sh>
__device__ __forceinline__ void env_counts(Sh &sh, const Place &P, int N,
                                           const bool (&pred)[K], int (&cnt)[K])
{
    if (WAVES == 1) {
        const uint64_t range = lanes_of_env(P, N);
#pragma unroll
        for (int q = 0; q < K; ++q) cnt[q] = __popcll(lanes_where(pred[q]) & range);
    } else {
        const int wv = P.l >> 6;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const uint64_t b = lanes_where(pred[q]);
            if ((P.l & 63) == 0) sh.ballots[wv][q] = b;
        }
        group_barrier<WAVES>(sh);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            cnt[q] = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) cnt[q] += __popcll(sh.ballots[w][q]);
        }
        group_barrier<WAVES>(sh);
    }
}

// Mean health ratio of both teams over their enabled units (the bracketed means of
// Eq. 1): the terms published in sh.share are added in ascending unit index; a term
// of +0.0f (unit of the other team, or disabled) leaves a finite sum unchanged.  Eight terms are
// fetched together, also the last few (what lies behind the env's terms is fetched with them and not
// added): one by one, each is a trip to LDS that a small batch waits for.
template <class Sh>
__device__ __forceinline__ void team_means(const Sh &sh, const Place &P, int N,
                                           int c0, int c1, float &m0, float &m1)
{
    static_assert(sizeof(sh.st.aim0) >= sizeof(sh.st.share) + 8 * sizeof(float2), "terms behind the last");
    float s0 = 0.0f, s1 = 0.0f;
    const float2 *term = sh.st.share + P.base;
    int left = N;
    for (; left >= 8; left -= 8, term += 8) {
        float2 q[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) q[k] = term[k];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s0 = s0 + q[k].x;
            s1 = s1 + q[k].y;
        }
    }
    if (left > 0) {
        float2 q[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) q[k] = term[k];
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            if (k >= left) break;
            s0 = s0 + q[k].x;
            s1 = s1 + q[k].y;
        }
    }
    const float r0 = s0 / (float)(c0 > 0 ? c0 : 1), r1 = s1 / (float)(c1 > 0 ? c1 : 1);
    m0 = c0 > 0 ? r0 : 0.0f;
    m1 = c1 > 0 ? r1 : 0.0f;
}

// Squared gap between attacker i's forward rectangle [0, L] x [-hw, hw] and the
// centre of j (closest point of the rectangle), from j's offset (dx, dy);
// `along` returns the offset's component along i's heading.
__device__ __forceinline__ float hurtbox_gap2(float dx, float dy, float ci, float si, float L,
                                              float hw, float neg_hw, float &along)
{
    const float lx = (dx * ci) + (dy * si);
    const float ly = (dy * ci) - (dx * si);
    const float ex = lx - median3(lx, 0.0f, L);
    const float ey = ly - median3(ly, neg_hw, hw);
    along = lx;
    return (ex * ex) + (ey * ey);
}

} // namespace tabx
