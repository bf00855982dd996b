// TABX batched battle-environment step and observation for MI355X (gfx950).
//
// Work layout.  A 64-lane wavefront advances G = floor(64 / N) whole environments
// at once (N = units per env): lane l owns unit l % N of env slot l / N, so the
// struct-of-arrays state of the G envs is one contiguous, coalesced run of G*N
// elements per field.  For 64 < N <= 128 a workgroup of two wavefronts owns one
// env.  The per-unit stages run in registers; what other lanes need is published
// in LDS and read back as broadcasts inside the all-pairs loops.
//
// The observation tensor is almost all of the HBM traffic, and HBM only takes it
// at full rate when every cache line is completed by consecutive stores.  The
// observe stage therefore assembles rows in LDS, as exact images, and streams them to
// HBM front to back, 16 bytes per lane and 1 KB per store instruction: either in tiles
// of consecutive rows that any wavefront of the workgroup makes from unit records in
// LDS (tabx_observe.h), or, where no further wavefront shares the work, observer by
// observer with the units in registers (tabx_observe_packed.h).
//
// Files: tabx_device.h (launch arguments, registers, LDS exchange area, zones, helpers),
// tabx_policy.h (heuristic policy: scan stage and rule cascade), tabx_step.h (step
// stage), tabx_observe.h and tabx_observe_packed.h (observe stage, where scripted units
// also decide), this file (kernels, argument checks, launches, the C entry points).
//
// The rules follow the paper's App. A ("Interaction Dynamics", "Reward",
// "Observation and Global State", "Zones").  All arithmetic is float32 with one
// rounding per written operation: the file is compiled with -ffp-contract=off
// and uses fmaf only where it is spelled out.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "tabx.h"

#pragma clang fp contract(off)

#include "tabx_device.h"
#include "tabx_policy.h"
#include "tabx_step.h"
#include "tabx_observe.h"
#include "tabx_observe_packed.h"

namespace tabx {

template <int WAVES, bool DO_POLICY, bool DO_STEP, bool DO_OBS, bool SCRIPT = false,
          int TWIN = 0, bool EVEN = false>
__global__ __launch_bounds__(64 * WAVES * (TWIN ? TWIN : 1))
__attribute__((amdgpu_waves_per_eu(1, EVEN ? 3 : 8))) void tabx_tick_kernel(const KArgs args)
{
    // without further wavefronts to share the rows with, the units stay in registers
    constexpr bool PACKED = DO_OBS && TWIN == 0;
    // TWIN: the workgroup has TWIN times the wavefronts that hold an env's units
    constexpr bool PAIR = WAVES == 2 && TWIN != 0;
    __shared__ Shared<WAVES, DO_OBS && !PACKED, DO_POLICY, PAIR> sh;
    extern __shared__ __attribute__((aligned(16))) float dyn[];
    // all wavefronts of the workgroup write rows; with TWIN only the first of them steps the envs
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool lead = !TWIN || wave < WAVES;
    if (PAIR) {
        if (threadIdx.x == 0) sh.arrivals = 0;
        lds_barrier<2>();
    }
    TABX_STAMP(0);
#ifdef TABX_TRACE
    if ((threadIdx.x & 63) == 0) {
        unsigned hw = 0, xcc = 0;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        g_trace[(((size_t)blockIdx.x * kTraceWaves + (threadIdx.x >> 6)) * 8 + 7) & ((1 << 21) - 1)] =
            ((unsigned long long)xcc << 32) | hw;
    }
#endif
    const KArgs &a = args;
    // (The register that is named here keeps a SIMD at three of these wavefronts, or four: more of them stream
    // slower.  One wavefront, three and four per SIMD: 5v5 x 65536 83.4 and 84.6 us; two, four and five: 64v64 x
    // 4000 776 and 809; EVEN: see plan_shape.)
    if constexpr (PACKED && (EVEN || (WAVES == 1 && DO_STEP))) asm volatile("" ::: "v135");
    else if constexpr (PACKED && WAVES == 2) asm volatile("" ::: "v103");
    warm_args();
    Place P = locate<WAVES, DO_OBS && !DO_STEP>(a);
    if (P.grp >= a.num_groups) return;           // (the grid is rounded up to the eight XCDs)
    const ZoneLds Z = zone_lds(a, dyn);
    ScriptLds<WAVES> *script = reinterpret_cast<ScriptLds<WAVES> *>(dyn + a.script_offset);
    const float *zd = reinterpret_cast<const float *>(Z.val + P.g * a.zone_chunks);
    Carry C = {1.0f, 0.0f, 0.0f, 0, false, 0, 0, 0.0f, 0.0f};
    float speed = 0.0f;
    // a wavefront that waits for the step fetches the zones meanwhile, unless the wavefronts that step
    // read them first (a policy's bush search, elliptical zones: nothing but the workgroup's barrier
    // before the rows orders the two) or may move an env to another level, whose zones they then write
    const bool zones_elsewhere = TWIN && !DO_POLICY && a.p.num_levels == 0 && a.p.zone_shapes == 0;
    if (DO_OBS && TWIN && wave == WAVES && zones_elsewhere) {
        put_zones<64, WAVES == 2>(a, Z, P.grp, (int)(threadIdx.x & 63));
        lds_barrier<1>();
        if (P.chunk == 0) global_state_zones<64>(a, Z, P.grp, (int)(threadIdx.x & 63));
    }
    if (lead) {
        const KArgs &a = again();
        Unit U = {};
        int code_u = 0;                              // the zone code under the unit
        StepIn in = {0, -1, 0.0f, 0, 0.0f, 0.0f, 0.0f};
        load_unit<!DO_OBS && !DO_POLICY>(a, P.k, P.ks, U);
        PolicyIn pin = {};
        if (DO_POLICY) load_policy(a, P, pin);
        if (DO_STEP) load_step(a, P, in);
        if (DO_STEP && !DO_OBS) load_more(a, P.ks, U);
        if (DO_STEP) load_more_step(a, P, in);
        // scripted units: the action decided on at the end of the previous call and the memory, asked for
        // with the state (whether the unit is the policy's to move or not: one round trip for all)
        int told = 0, waiting = 0;
        if (SCRIPT) {
            const LateArgs late = late_args();
            const uint8_t *const controlled = late->pa.controlled;
            told = controlled ? at32(controlled, P.k) : 1;
            waiting = at32(late->pa.next_action, P.k);
            C.mem_valid = at32(late->pa.mem.mem_valid, P.k);
            C.mem_x = at32(late->pa.mem.mem_x, P.k);
            C.mem_y = at32(late->pa.mem.mem_y, P.k);
        }
        // (a lane without a unit of its own has loaded the group's first one)
        fold_byte(U.alive);
        U.alive = P.has ? U.alive : 0;
        U.enabled = P.has ? U.enabled : 0;
        // the unit's move and the grid cell under it, which is asked for while the rest is on its way
        float zeff = 0.0f;
        int code = 0;
        bool oob = false;
        if (DO_STEP && !DO_POLICY) oob = move_unit(a, U, in);
        if (!flagged(a, ELLIPSES) && (!DO_STEP || DO_POLICY || flagged(a, EARLY_CELL))) code = grid_cell(a, P.row, U.x, U.y);
        ZoneRegs Zr = {};
        if (PACKED) Zr = load_zone_regs(a, P);
        if (a.zones_in_lds && !zones_elsewhere) {
            put_zones<64 * WAVES, WAVES == 2>(a, Z, P.grp, P.l);
            group_barrier<WAVES>(sh);
        }
        if ((!DO_STEP || DO_POLICY) && flagged(a, ELLIPSES)) code = zone_at(a, zd, P.row, U.x, U.y, zeff);
        fold_byte(U.team);
        int forced = -1;
        if (SCRIPT && told && U.enabled && U.alive) {
            forced = waiting;
            at32(late_args()->pa.actions_out, here(P.k)) = (uint8_t)forced;
        }
        if constexpr (DO_POLICY) {
            float cu, su;
            heading_sincos(U.theta, su, cu);
            forced = policy_env<WAVES>(a, sh, P, U, pin, code, cu, su, zd);
        }
        TABX_STAMP(6);
        if (DO_STEP) {
            const KArgs &a = again();
            const int stood = DO_POLICY ? code : 0;
            if (DO_POLICY) oob = move_unit(a, U, in);
            if (flagged(a, COLLIDE)) collide_env<WAVES>(a, sh, P, U);
            if (DO_POLICY || !flagged(a, EARLY_CELL)) code = zone_at(a, zd, P.row, U.x, U.y, zeff);
            code_u = U.enabled ? code : stood;
            const bool restarted = step_env<WAVES>(a, sh, Z, zd, P, U, code_u, zeff, oob, C, in, forced);
            if (PACKED && a.p.num_levels > 0 && restarted) {
                // zone slots of the envs that changed level
                const int row = Zr.lane ? sh.level_rows[Zr.zg] : -1;
                if (row >= 0) Zr = load_zone_regs(a, P, row);
            }
        } else if (DO_OBS) {
            code_u = code;
            heading_sincos(U.theta, C.su, C.cu);
            C.ratio = U.hp / U.hmax;       // (disabled units: masked in the rows)
        }
        TABX_STAMP(1);
        if constexpr (PACKED) {
            const KArgs &a = again();
            observe_packed<WAVES, SCRIPT, SCRIPT || DO_POLICY, EVEN>(a, sh, dyn, P, U, code_u, C, Zr, told, script, zd);
        } else if constexpr (DO_OBS) {
            group_barrier<WAVES>(sh);          // the step stage is done with the LDS union
            publish_units<WAVES, SCRIPT>(a, sh, P, U, code_u, C.ratio, C.cu, C.su, told, script);
            if (!zones_elsewhere && P.chunk == 0) {
                group_barrier<WAVES>(sh);
                global_state_zones<64 * WAVES>(a, Z, P.grp, P.l);
            }
            speed = U.speed;
        }
    }
    if constexpr (DO_OBS && !PACKED) {
        lds_barrier<2>();                  // the whole workgroup
        TABX_STAMP(2);
        float *stg = dyn + wave * a.stage_floats;
        {
            const KArgs &a = again();
            if constexpr (WAVES == 1) {
                float *const global_state = late_args()->global_stream;
                if (global_state && P.chunk == 0)
                    stream_global_state<64 * TWIN>(a, sh.rec, Z, global_state, P.grp, (int)threadIdx.x);
            }
            const int first = P.chunk * a.tiles_per_chunk;
            const int end = first + a.tiles_per_chunk < a.tiles ? first + a.tiles_per_chunk : a.tiles;
            // (see plan_shape)
            const bool in_turn = WAVES == 1 && DO_STEP && a.in_turn;
            const int share = (end - first + WAVES * TWIN - 1) / (WAVES * TWIN);
            const int begin = first + (in_turn ? wave : wave * share), step = in_turn ? WAVES * TWIN : 1;
            const int stop = !in_turn && begin + share < end ? begin + share : end;
            const auto rows = [&](auto fold, auto lines) {
                write_rows<WAVES, SCRIPT, fold.value, lines.value, WAVES == 1 && !DO_STEP>(a, sh.rec, Z, stg, P.grp, begin, step, stop, script);
            };
            const auto rows_by_lines = [&](auto fold) {
                if (a.lines == LINES_OWN) rows(fold, Constant<LINES_OWN>{});
                else if (a.lines == LINES_SHARED) rows(fold, Constant<LINES_SHARED>{});
                else rows(fold, Constant<LINES_CARRIED>{});
            };
            if (a.zone_chunks == 0) rows_by_lines(Constant<1>{});
            else rows_by_lines(Constant<0>{});
        }
        TABX_STAMP(4);
        if (SCRIPT) {
            lds_barrier<2>();              // all bids are in
            if (lead) decide_units<WAVES>(a, sh.rec, script, P, speed, C, zd);
        }
    }
    if (DO_STEP) asm volatile("" ::"v"(C.warm));    // keeps the cache-warming load of step_env
    TABX_STAMP(5);
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void tabx_reset_kernel(const KArgs a)
{
    __shared__ Shared<WAVES, false, false> sh;
    Place P = locate<WAVES>(a);
    if (P.grp >= a.num_groups) return;
    const int N = a.p.num_units;
    const bool go = P.has && !(a.env_mask && a.env_mask[P.e] == 0);
    if (a.p.num_levels > 0) {
        const int row = advance_level<WAVES>(a, sh, P, go);
        if (row >= 0) {
            P.row = row;
            P.ks = (uint32_t)row * (uint32_t)N + (uint32_t)P.u;
        }
    }
    Unit U = {};
    float ratio = 0.0f;
    if (go) {
        load_spec(a, P.ks, U);
        fold_byte(U.team);
        float zeff = 0.0f;
        spawn_unit(a, a.sc.zone_desc + (size_t)P.row * 6 * a.p.max_zones, P.row, P.ks, U, zeff);
        ratio = U.enabled ? U.hp / U.hmax : 0.0f;
        store_state(a, P.k, U);
        if (a.p.dynamics == 1) {
            a.st.ax[P.k] = 0.0f;
            a.st.ay[P.k] = 0.0f;
        }
    }
    const bool en = go && U.enabled;
    sh.st.share[P.l] = make_float2((en && U.team == 0) ? ratio : 0.0f,
                                   (en && U.team != 0) ? ratio : 0.0f);
    const bool pred[2] = {en && U.team == 0, en && U.team != 0};
    int cnt[2];
    env_counts<WAVES>(sh, P, N, pred, cnt);
    lds_barrier<WAVES>();
    float m0, m1;
    team_means(sh, P, N, cnt[0], cnt[1], m0, m1);
    if (go && P.u == 0) {
        a.st.t[P.e] = 0;
        a.st.phi_prev[P.e] = m0 - m1;
        if (a.st.ret_run) a.st.ret_run[P.e] = 0.0f;
        if (a.st.kill_run) a.st.kill_run[P.e] = 0;
    }
}

// Global state: every enabled unit's own block, then the zone slots with absolute centres.
// One thread per unit (16 floats, four 16-byte stores) or per zone chunk.
__global__ __launch_bounds__(256) void tabx_global_state_kernel(const KArgs a, float *out)
{
    const int N = a.p.num_units;
    const int zlen = 6 * a.p.max_zones;
    const int Dg = 16 * N + zlen;
    const size_t units = (size_t)a.p.num_envs * N;
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid < units) {
        const int e = (int)(tid / N);
        const int u = (int)(tid - (size_t)e * N);
        const int row = row_of(a, e);
        Unit U = {};
        const uint32_t k = (uint32_t)tid, ks = (uint32_t)row * (uint32_t)N + (uint32_t)u;
        load_unit<false>(a, k, ks, U);
        fold_byte(U.team);
        fold_byte(U.alive);
        float4 q[4];
        if (U.enabled) {
            float zeff = 0.0f;
            const int code = zone_at(a, a.sc.zone_desc + (size_t)row * zlen, row, U.x, U.y, zeff);
            q[0] = make_float4(U.hp, U.hp / U.hmax, U.x, U.y);
            q[1] = make_float4(U.theta, U.range, U.dmg, U.cd);
            q[2] = make_float4(U.cooldown != 0.0f ? U.cd / U.cooldown : 0.0f, U.radius, U.mass,
                               U.sight_angle);
            q[3] = make_float4(U.alive ? 1.0f : 0.0f, U.cur_speed, (float)(code & 3), (float)U.team);
        } else {
            q[0] = q[1] = q[2] = q[3] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        float *d = out + (size_t)e * Dg + 16 * u;       // Dg may be 2 mod 4: 8-byte aligned rows
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f4u o = {q[k].x, q[k].y, q[k].z, q[k].w};
            *reinterpret_cast<f4u *>(d + 4 * k) = o;
        }
    }
    // zone floats: one thread per float, after the unit threads
    const size_t zt = tid;
    const size_t zones = (size_t)a.p.num_envs * zlen;
    if (zlen > 0 && zt < zones) {
        const int e = (int)(zt / zlen);
        const int zz = (int)(zt - (size_t)e * zlen);
        const float *d = a.sc.zone_desc + (size_t)row_of(a, e) * zlen;
        const int comp = zz % 6;
        out[(size_t)e * Dg + 16 * N + zz] = d[zz - comp] != 0.0f ? d[zz] : 0.0f;
    }
}

// ------------------------------------------------------------------ host side

// The machine the launch shapes below are tuned for (MI355X, gfx950).  tabx_launch_info reports
// them, so that a caller, or a test that runs on the device, can hold them against the
// properties the device itself reports.
constexpr int kComputeUnits = 256;
constexpr int kLdsPerCuBytes = 160 * 1024;          // a CU's LDS, shared by its resident workgroups
constexpr int kLdsPerWorkgroupBytes = 64 * 1024;    // the most one workgroup may take
constexpr int kWavefrontLanes = 64;
constexpr size_t kLdsGranuleBytes = 1280;           // LDS is given out in these
constexpr size_t kL2Bytes = (size_t)32 << 20;                // the L2s of all XCDs
constexpr size_t kLastLevelCacheBytes = (size_t)256 << 20;   // the cache in front of HBM, all XCDs

static size_t lds_granules(size_t bytes) { return (bytes + kLdsGranuleBytes - 1) / kLdsGranuleBytes * kLdsGranuleBytes; }

enum Mode { MODE_RESET, MODE_STEP, MODE_OBSERVE, MODE_STEP_OBSERVE, MODE_POLICY,
            MODE_POLICY_STEP_OBSERVE, MODE_SCRIPTED_STEP_OBSERVE };

// The calls that write observation rows.
static bool has_rows(Mode mode)
{
    return mode == MODE_OBSERVE || mode == MODE_STEP_OBSERVE || mode == MODE_POLICY_STEP_OBSERVE ||
           mode == MODE_SCRIPTED_STEP_OBSERVE;
}

static bool aligned(const void *p, size_t n) { return ((uintptr_t)p % n) == 0; }

static int check_params(const TabxParams *p)
{
    if (!p) return TABX_ERR_NULL;
    if (p->num_envs < 0 || p->num_units < 1 || p->num_units > TABX_N_MAX) return TABX_ERR_SHAPE;
    if (p->max_zones < 0 || p->max_zones > TABX_Z_MAX) return TABX_ERR_SHAPE;
    if (p->grid_w < 0 || p->grid_h < 0 || ((p->grid_w == 0) != (p->grid_h == 0)))
        return TABX_ERR_SHAPE;
    if (p->max_steps < 1) return TABX_ERR_SHAPE;
    if (p->zone_shapes != 0 && p->zone_shapes != 1) return TABX_ERR_SHAPE;
    if (p->zone_shapes == 1 && (p->grid_w != 0 || p->max_zones < 1)) return TABX_ERR_SHAPE;
    if (p->num_levels < 0) return TABX_ERR_SHAPE;
    if ((p->hurtbox_cone | p->hit_all | p->dynamics) & ~1) return TABX_ERR_SHAPE;
    if (p->env_id_offset < 0 || (int64_t)p->env_id_offset + p->num_envs > INT32_MAX)
        return TABX_ERR_SHAPE;
    if ((int64_t)p->num_levels * p->num_units > (int64_t)1 << 30) return TABX_ERR_SHAPE;
    if ((int64_t)p->num_envs * p->num_units > (int64_t)1 << 30) return TABX_ERR_SHAPE;
    const float pos[] = {p->map_w, p->map_h, p->cell_size, p->dt};
    for (float v : pos)
        if (!(v > 0.0f) || !(v < 3.0e38f)) return TABX_ERR_PARAM;
    const float fin[] = {p->turn_rate, p->lava_dps, p->swamp_mult, p->reveal_time,
                         p->boundary_frac, p->collision_alpha, p->collision_slop,
                         p->move_gain, p->restitution};
    for (float v : fin)
        if (!(v > -3.0e38f && v < 3.0e38f)) return TABX_ERR_PARAM;
    return TABX_OK;
}

static int check_scenario(const TabxParams *p, const TabxScenario *s)
{
    if (!s) return TABX_ERR_NULL;
    const float *f[] = {s->init_x, s->init_y, s->init_theta, s->hmax, s->radius, s->mass,
                        s->speed, s->dmg, s->range, s->cooldown, s->sight_angle,
                        s->sight_cos_half, s->sight_range, s->hurt_halfwidth};
    for (const float *q : f) {
        if (!q) return TABX_ERR_NULL;
        if (!aligned(q, 4)) return TABX_ERR_ALIGN;
    }
    if (!s->team || !s->enabled) return TABX_ERR_NULL;
    if ((p->grid_w > 0) != (s->terrain != nullptr)) return TABX_ERR_NULL;
    if ((p->max_zones > 0) != (s->zone_desc != nullptr)) return TABX_ERR_NULL;
    if (s->zone_desc && !aligned(s->zone_desc, 4)) return TABX_ERR_ALIGN;
    return TABX_OK;
}

static int check_state(const TabxParams *p, const TabxState *s)
{
    if (!s) return TABX_ERR_NULL;
    if (p->num_levels > 0) {
        const void *lv[] = {s->level, s->next_level, s->level_draws};
        for (const void *q : lv) {
            if (!q) return TABX_ERR_NULL;
            if (!aligned(q, 4)) return TABX_ERR_ALIGN;
        }
    }
    const float *f[] = {s->x, s->y, s->vx, s->vy, s->theta, s->hp, s->cd, s->reveal,
                        s->cur_speed, s->phi_prev};
    for (const float *q : f) {
        if (!q) return TABX_ERR_NULL;
        if (!aligned(q, 4)) return TABX_ERR_ALIGN;
    }
    if (!s->alive || !s->t) return TABX_ERR_NULL;
    if (!aligned(s->t, 4)) return TABX_ERR_ALIGN;
    if (p->dynamics == 1 && (!s->ax || !s->ay)) return TABX_ERR_NULL;
    const void *m4[] = {s->ret_run, s->ep_count, s->ep_len, s->ep_return, s->global_state,
                        s->ax, s->ay};
    for (const void *q : m4)
        if (q && !aligned(q, 4)) return TABX_ERR_ALIGN;
    return TABX_OK;
}

// Whether v is a power of two whose reciprocal (`inv`) is exact.
static bool power_of_two(float v, float *inv)
{
    int ex = 0;
    *inv = 1.0f / v;
    return frexpf(v, &ex) == 0.5f && ex > -100 && ex < 100;
}

static void take_params(const TabxParams *p, KArgs &a)
{
    memcpy(&a.p, p, sizeof a.p);
    a.shared_machine = p->shared_machine;
}

// What the launch has to do besides the plain tick, and how it finds a unit's cell.
static void set_flags(const TabxParams *p, const TabxState *st, KArgs &a)
{
    const uint64_t rows = p->num_levels > 0 ? p->num_levels : p->num_envs;
    const uint64_t cells = (uint64_t)p->grid_w * (uint64_t)p->grid_h;
    a.cells = (uint32_t)cells;
    a.flags = (p->dynamics == 1 ? DYNAMIC : 0) | (p->collision_alpha > 0.0f ? COLLIDE : 0) |
              (p->zone_shapes == 1 ? ELLIPSES : 0) | (p->hurtbox_cone ? CONE_BOUND : 0) |
              (p->hit_all ? HIT_ALL : 0) | (st->kill_run ? KILLS : 0) | (st->ret_run ? RETURNS : 0) |
              (p->num_levels > 0 ? LEVELS : 0) |
              (cells > 0 && !(p->collision_alpha > 0.0f) ? EARLY_CELL : 0);
    if (cells > 0 && power_of_two(p->cell_size, &a.inv_cell) && rows < (1u << 24) && cells < (1u << 24) &&
        rows * cells <= 1ull << 32)
        a.flags |= FAST_CELL;
}

// A wavefront's staging area for `floats` floats: whole store passes (64 lanes of 16 bytes).
static size_t whole_passes(size_t floats) { return (floats + 255) / 256 * 256; }

// The staging area of a tile of `rows` rows of `dim` floats, which starts anywhere within `line` + 1 floats.
static size_t tile_floats(int rows, int dim, int line)
{
    return whole_passes((size_t)rows * dim + (dim % 32 ? line - 1 : 0));
}

// The zone descriptors of a workgroup's envs: 16-byte chunks with a mask each.
static size_t zone_floats(const KArgs &a) { return ((size_t)a.envs_per_block * a.zone_chunks * 5 + 3) / 4 * 4; }

// Dynamic LDS of a launch and where its parts lie (fills the offsets in `a`).
static size_t plan_lds(Mode mode, KArgs &a, int waves)
{
    const bool observing = has_rows(mode);
    if (mode == MODE_RESET) return 0;
    size_t floats = 0;
    if (observing) {
        if (a.packed && waves == 2) {
            // two alternating areas of one row; the second half's store passes read whole passes
            const int row_chunks = ((a.obs_dim + 3) / 4 + 3) & ~3, half = ((a.obs_dim / 4 >> 1) + 3) & ~3;
            floats = 4 * ((size_t)row_chunks + half + 64 * a.copy_passes);
        } else {
            // one staging area per wavefront
            a.stage_floats = (int)(a.packed ? whole_passes((size_t)a.envs_per_block * a.rows_per_flush * a.obs_dim)
                                            : tile_floats(a.rows_per_tile, a.obs_dim, a.line));
            floats = (size_t)a.stage_floats * waves * (a.twin ? a.twin : 1);
        }
    }
    // zones: elliptical ones; the bush search of deciding units; the copied part of the rows of a tile
    a.zones_in_lds = a.zone_chunks > 0 &&
                     (a.p.zone_shapes == 1 || mode == MODE_POLICY || mode == MODE_POLICY_STEP_OBSERVE ||
                      mode == MODE_SCRIPTED_STEP_OBSERVE || (observing && !a.packed));
    a.zone_offset = (int)floats;
    if (a.zones_in_lds) floats += zone_floats(a);
    // the bidding area of scripted units that decide in the observe stage
    floats = (floats + 3) / 4 * 4;
    a.script_offset = (int)floats;
    if (mode == MODE_SCRIPTED_STEP_OBSERVE)
        floats += (waves == 1 ? sizeof(ScriptLds<1>) : sizeof(ScriptLds<2>)) / sizeof(float);
    return floats * sizeof(float);
}

// How many wavefronts of the rows' kernels a SIMD holds (by their vector registers).  (Of the scripted tiles of envs of
// two wavefronts there are never more than the four per SIMD that 98 registers leave: four workgroups of four in a CU's
// LDS, or six wavefronts in batches of two envs per CU.)
static int wavefronts_per_simd(Mode mode, const KArgs &a, int waves)
{
    if (a.packed) return waves == 1 || a.even ? 3 : 4;
    return mode == MODE_SCRIPTED_STEP_OBSERVE ? 4 : 5;
}

// Whether all workgroups of a launch with rows are resident from its start.
static bool one_generation(Mode mode, const KArgs &a, int waves, size_t lds)
{
    const int w = waves * (a.twin ? a.twin : 1);
    const bool policy = mode == MODE_POLICY_STEP_OBSERVE;
    const size_t fixed = !a.packed    ? (waves == 1 ? sizeof(Shared<1, true, true>) : sizeof(Shared<2, true, true, true>))
                         : waves == 1 ? (policy ? sizeof(Shared<1, false, true>) : sizeof(Shared<1, false, false>))
                                      : (policy ? sizeof(Shared<2, false, true>) : sizeof(Shared<2, false, false>));
    const int by_simd = 4 * wavefronts_per_simd(mode, a, waves) / w, by_lds = kLdsPerCuBytes / (int)lds_granules(fixed + lds);
    return a.num_groups <= kComputeUnits * (by_simd < by_lds ? by_simd : by_lds);
}

// Flushes of a wavefront, and how long HBM takes, at 6 TB/s, for one of each wavefront of the launch.
static int flushes_per_wavefront(const KArgs &a, int waves)
{
    const int w = waves * (a.twin ? a.twin : 1);
    return a.packed ? (a.p.num_units + a.rows_per_flush - 1) / a.rows_per_flush : (a.tiles + w - 1) / w;
}

static double hbm_us_per_flush(const KArgs &a, int waves)
{
    return 4.0 * a.obs_dim * a.p.num_units * a.p.num_envs / 6e6 / flushes_per_wavefront(a, waves);
}

// Holds the wavefronts of a launch to the pace at which HBM takes all their rows together (a.pace).
// Where all workgroups are resident from the start and live as long as the launch, some of them write faster
// than others: the even XCDs get more of HBM than the odd ones while both ask for all they can, and so do
// wavefronts that share their SIMD with fewer others.  The launch then ends with the slow ones alone, which
// cannot use what has become free (64v64 x 1024: workgroups of even XCDs end at 158 ... 173 us, of odd ones at
// 184 ... 203).  A flush that is not due yet waits, and what it would have taken goes to those behind.
// Measured, without / with: 64v64 x 1024 211.5 / 198.5 us, x 1300 278 / 247.5, 40v40 x 1500 135 / 122, 64v64 x 400
// 100 / 89, 10v10 x 8192 with collisions and ellipses 60.5 / 54.5, 10v10 x 4000 with zones 35 / 28.5, 32v32 x 700
// 44 / 36.5.  (The wait is between flushes only: with one after the last as well the masks, the decisions of
// scripted units and the workgroup's end came later, 57, 29.2 and 37.4 in the last three.)  With several generations, workgroups of all ages side by side even each other out, and a pace
// only costs (10v10 x 16384 102 / 108 ... 124 us).
static void plan_pace(Mode mode, KArgs &a, int waves, size_t lds)
{
    a.pace = 0;
    if (!has_rows(mode) || (mode == MODE_OBSERVE && waves == 1)) return;     // (several workgroups share a group there)
    // Beside other work (unpaced / paced): a workgroup that had to wait for its place cannot see that it is late and
    // would take all of the launch's time once more (10v10 with collisions and ellipses, 2 x 8192 on two streams
    // 91 / 95.5 us, x 8192 beside a product of 2048 x 2048 matrices 74 / 88; scripted 10v10 with zones 2 x 4000
    // 43.6 / 46).  Envs of two wavefronts take about that time per row by themselves and keep the gain (64v64 2 x
    // 512 233 / 222, x 1024 beside the product 218 / 208).
    if (a.shared_machine && waves == 1) return;
    // Few rows: such a launch is mostly its start (5v5 x 6000, 38 MB: 13.4 us, 14.0 paced; x 8000 17.8 and 17.1).
    const double bytes = 4.0 * a.obs_dim * a.p.num_units * a.p.num_envs;
    if (bytes < 50e6) return;
    if (!one_generation(mode, a, waves, lds)) return;
    // Tiles of envs of two wavefronts that share lines go out at 3.9 to 4.4 TB/s at most, and looking at the clock
    // costs them 1 % (33v33 with 7 zones x 1000 77.8 us, 78.8 paced, 64v64 with 3 x 400 120.0 and 121.1); rows of
    // whole chunks whose lines are handed on reach the pace (64v64 with 2 x 400 96.5, 92.6 paced).
    if (waves == 2 && !a.packed && (a.lines == LINES_SHARED || a.obs_dim % 4 != 0)) return;
    // Few flushes per wavefront: no time to fall behind in (tiles, 4v4 x 14000, four each: 18.4 us, 19.0 paced; units
    // in registers, 5v5 x 16384, five each: 30.7 and 30.6 ... 33).
    const int flushes = flushes_per_wavefront(a, waves);
    if (flushes < (a.packed ? 8 : 5)) return;
    // ... nor where a wavefront needs longer for a tile than HBM for one of each (by the microseconds that is, unpaced
    // and paced: tiles that start on lines, 0.67 ... 1.0 level to 2 % slower, 1.0 ... 1.3 2 % faster, then 7; others
    // 0.9 ... 1.2 1 % slower, 1.2 ... 1.3 level, then 1 to 7 % faster).
    if (waves == 1 && !a.packed && hbm_us_per_flush(a, waves) < (a.lines == LINES_OWN ? 1.0 : 1.2)) return;
    // The rate, in TB/s of rows, at which a launch is shortest; up to 4 % to either side cost little, 10 % too slow
    // costs that much and 10 % too fast leaves little of the gain.  Tiles: 6.0 (64v64 x 400, 27v28 x 1200); rows of
    // whole 128-byte lines that the last-level cache takes all of 7.0 (6.5 ... 7.8: 32v32 x 700, 8v8 x 5000, 16v16 x
    // 1300); rows that leave lines partly written, beyond that cache, 5.6 (32v32 with 8 zones x 1000); rows that end
    // on half a chunk 6.5 where shared lines are handed on (24v24 with 5 zones x 1200 50.9 at 5.2, 48.0 at 6.5, 32v32
    // with 3 x 1000 65.5 and 60.4), else 5.2 (10v10 with 3 x 4000 32.4, 36.8 at 5.6).  Units in registers: 5.85, rows of whole lines of two
    // wavefronts 6.1.
    const bool lines = a.obs_dim % 32 == 0, cached = bytes <= (double)kLastLevelCacheBytes;
    double rate = lines ? (cached ? 7.0 : 6.0) : (cached ? 6.0 : 5.6);
    if (a.obs_dim % 4 != 0) rate = a.lines == LINES_CARRIED ? 6.5 : 5.2;
    if (a.packed) rate = waves == 2 && lines ? 6.1 : 5.85;
    const double ticks = bytes / (rate * 1e12) * 100e6 / flushes;
    // Two wavefronts with the units in registers take 0.9 us per row by themselves, and looking at the clock
    // costs them 2 % (64v64 x 600 135.5 us and 138; x 700 145 and 140).
    if (a.packed && waves == 2 && ticks < 90.0) return;
    a.pace = (unsigned)(16.0 * ticks);
}

// Enqueues one kernel and returns the status of THIS launch (the runtime's sticky "last error"
// is neither read nor cleared: an error the caller's own earlier work left pending stays theirs).
template <class Kernel, class Arg0>
static hipError_t enqueue(Kernel kernel, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream,
                          Arg0 &a0)
{
    void *args[] = {(void *)&a0};
    return hipLaunchKernel((const void *)kernel, grid, block, args, lds_bytes, stream);
}

template <int WAVES>
static hipError_t launch_mode(Mode mode, KArgs a, hipStream_t stream)
{
    const dim3 grid((unsigned)(8 * a.groups_per_xcd * a.obs_chunks));
    const dim3 block(64 * WAVES * (a.twin ? a.twin : 1));
    const size_t lds = plan_lds(mode, a, WAVES);
    plan_pace(mode, a, WAVES, lds);
    switch (mode) {
    case MODE_RESET:
        return enqueue(tabx_reset_kernel<WAVES>, grid, block, lds, stream, a);
    case MODE_STEP:
        return enqueue(tabx_tick_kernel<WAVES, false, true, false>, grid, block, lds, stream, a);
    case MODE_OBSERVE:
        if (WAVES == 1 && a.twin)
            return enqueue(tabx_tick_kernel<1, false, false, true, false, 2>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.twin > 2)
            return enqueue(tabx_tick_kernel<2, false, false, true, false, 3>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.twin)
            return enqueue(tabx_tick_kernel<2, false, false, true, false, 2>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.even)
            return enqueue(tabx_tick_kernel<2, false, false, true, false, 0, true>, grid, block, lds, stream, a);
        return enqueue(tabx_tick_kernel<WAVES, false, false, true>, grid, block, lds, stream, a);
    case MODE_STEP_OBSERVE:
        if (WAVES == 1 && a.twin > 4)
            return enqueue(tabx_tick_kernel<1, false, true, true, false, 8>, grid, block, lds, stream, a);
        if (WAVES == 1 && a.twin > 2)
            return enqueue(tabx_tick_kernel<1, false, true, true, false, 4>, grid, block, lds, stream, a);
        if (WAVES == 1 && a.twin)
            return enqueue(tabx_tick_kernel<1, false, true, true, false, 2>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.twin > 2)
            return enqueue(tabx_tick_kernel<2, false, true, true, false, 3>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.twin)
            return enqueue(tabx_tick_kernel<2, false, true, true, false, 2>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.even)
            return enqueue(tabx_tick_kernel<2, false, true, true, false, 0, true>, grid, block, lds, stream, a);
        return enqueue(tabx_tick_kernel<WAVES, false, true, true>, grid, block, lds, stream, a);
    case MODE_POLICY:
        return enqueue(tabx_tick_kernel<WAVES, true, false, false>, grid, block, lds, stream, a);
    case MODE_POLICY_STEP_OBSERVE:
        if (a.twin)
            return enqueue(tabx_tick_kernel<WAVES, true, true, true, false, 2>, grid, block, lds, stream, a);
        if (WAVES == 2 && a.even)
            return enqueue(tabx_tick_kernel<2, true, true, true, false, 0, true>, grid, block, lds, stream, a);
        return enqueue(tabx_tick_kernel<WAVES, true, true, true>, grid, block, lds, stream, a);
    case MODE_SCRIPTED_STEP_OBSERVE:
        if (WAVES == 1 && a.twin > 4)
            return enqueue(tabx_tick_kernel<1, false, true, true, true, 8>, grid, block, lds, stream, a);
        if (WAVES == 1 && a.twin > 2)
            return enqueue(tabx_tick_kernel<1, false, true, true, true, 4>, grid, block, lds, stream, a);
        if (WAVES == 1)
            return enqueue(tabx_tick_kernel<1, false, true, true, true, 2>, grid, block, lds, stream, a);
        if (a.twin > 2)
            return enqueue(tabx_tick_kernel<2, false, true, true, true, 3>, grid, block, lds, stream, a);
        if (a.twin)
            return enqueue(tabx_tick_kernel<2, false, true, true, true, 2>, grid, block, lds, stream, a);
        if (a.even)
            return enqueue(tabx_tick_kernel<2, false, true, true, true, 0, true>, grid, block, lds, stream, a);
        return enqueue(tabx_tick_kernel<2, false, true, true, true>, grid, block, lds, stream, a);
    }
    return hipErrorInvalidValue;
}

// How a call is laid out on the machine: envs per workgroup, rows per tile, wavefronts per env
// group (all written into `a`; needs a.obs_dim and a.p).  Returns the wavefronts an env takes
// (1 or 2).
static int plan_shape(Mode mode, const TabxParams *p, KArgs &a)
{
    // N <= 64: one wavefront steps G = floor(64 / N) whole envs.  64 < N <= 128: two wavefronts
    // per env.
    const int N = p->num_units;
    const int waves = N <= 64 ? 1 : 2;
    int G = waves == 1 ? 64 / N : 1;
    a.zone_chunks = (6 * p->max_zones + 3) / 4;
    if (a.zone_chunks > 0 && G > 64 / a.zone_chunks) {
        // More zone chunks than lanes (few units per env, many zone slots).  Full wavefronts count where the
        // machine is full (2v2 with 16 slots x 16384 33 us with two envs per wavefront, 17 with sixteen); a
        // small batch is one chain, which grows with the envs of a wavefront (x 64 8.9 and 13 us, x 4096
        // 10.9 and 14.4; 4v5 with 12 slots, three and seven: x 2048 12.5 and 13.7, x 4096 17.4 and 14.8).
        const int few = a.zone_chunks > 64 ? 1 : 64 / a.zone_chunks;
        const int most = (p->num_envs + 8 * kComputeUnits - 1) / (8 * kComputeUnits);   // eight groups per CU
        if ((p->num_envs + few - 1) / few <= 3 * kComputeUnits) G = few;
        else if ((p->num_envs + G - 1) / G <= kComputeUnits) G = few > most ? few : most;
    }
    a.envs_per_block = G;
    a.magic_n = (65536u + N - 1) / N;
    a.magic_zc = a.zone_chunks ? (65536u + a.zone_chunks - 1) / a.zone_chunks : 0;
    // rows per tile: one observer per row that the 64 lanes hold all units of, about 4 KB
    int S = G;
    if (S > kTileFloats / a.obs_dim) S = kTileFloats / a.obs_dim;
    if (S < 1) S = 1;
    a.rows_per_pass = S;
    a.magic_tc = (65536u + 4 + a.zone_chunks - 1) / (4 + a.zone_chunks);
    a.magic_s = (65536u + S - 1) / S;
    a.tiles = (G * N + S - 1) / S;
    a.num_groups = (p->num_envs + G - 1) / G;
    a.groups_per_xcd = (a.num_groups + 7) / 8;
    // Long-lived wavefronts make a long tail at the end of the launch, and a wavefront's chain of
    // rows is the latency floor of a small batch, so the rows of an env group are split:
    //  - a stand-alone observe uses several workgroups per group (each loads the group's units and
    //    writes its share of the rows);
    //  - a launch that also steps cannot (the second workgroup would need the state after the first
    //    one's step), but the wavefronts of ONE workgroup can: the first one steps the envs and
    //    leaves the units in LDS, then all of them write rows.
    a.obs_chunks = 1;
    a.obs_per_chunk = N;
    a.twin = 0;
    a.packed = 0;
    a.even = 0;
    int K = 1;                                   // passes per tile
    // The form with the units in registers (tabx_observe_packed.h) needs, for envs of one wavefront, whole
    // 16-byte chunks per row, a zone chunk per lane at most and R rows of G envs in kMaxPasses store passes.
    const int cpr = a.obs_dim / 4;
    const int R = waves == 1 && N % 2 == 0 && 2 * G * cpr <= 64 * kMaxPasses ? 2 : 1;
    const bool packs = waves == 2 || (a.obs_dim % 4 == 0 && G * a.zone_chunks <= 64 &&
                                      R * G * cpr <= 64 * kMaxPasses);
    const bool rows = has_rows(mode);
    a.rows_per_flush = R;
    if (waves == 1) {
        a.copy_passes = (R * G * cpr + 63) / 64;
        // under one residency round (eight single-wavefront workgroups per CU)
        const bool small_batch = a.num_groups <= 8 * kComputeUnits;
        // eight or more flushes of two rows (10v10 x 16384: 120 us with one wavefront per group, 101.5 with
        // two; 5v5 x 65536 84 and 82); with body collisions the step stage is longer, and the two are level
        // or either ahead (one / two: 10v10 x 8192 62.3 / 62.4, 9v9 x 15000 with ellipses 81 / 89, without
        // 71 / 68, 12v12 x 10000 85 / 81, 16v16 x 4400 with ellipses 83 / 77)
        const bool long_chain = N >= 16 && !(p->collision_alpha > 0.0f);
        // a batch of at most three env groups per CU is one chain from the first load to the last store
        const bool tiny_batch = a.num_groups <= 3 * kComputeUnits && N > 4;
        // ... and one group per CU with many tiles, or two with a tile per row (32v32 x 200: 24.4 us with four
        // wavefronts, 18 with eight; scripted 42 and 20; 15v15 x 120 15.4 and 12.5, 12v12 x 500 13.4 and 11.4;
        // 22v22 x 300 20.5 and 17.0, x 512 20.8 and 20.0; three groups per CU: 20v20 x 600 20.6 and 24.1)
        const bool lone_groups = a.num_groups <= kComputeUnits, few_groups = a.num_groups <= 2 * kComputeUnits;
        if (mode == MODE_OBSERVE) {
            // about four flushes per workgroup (10v10, two rows a flush: 3 workgroups per group 94.7 us, 2 96.8,
            // 4 99; 19 units, one row a flush, x 850: 5 8.6 us, 3 10.1), at most two where each fetches
            // elliptical zones
            const int flushes = packs ? (N + R - 1) / R : (N + 1) / 2;
            int share = N < 4 ? 1 : (flushes + 3) / 4 + (flushes < 8 ? 1 : 0);
            if (share > 8) share = 8;
            if (share > 2 && p->zone_shapes == 1) share = 2;
            a.twin = packs ? 0 : 2;
            a.obs_per_chunk = ((N + share - 1) / share + R - 1) / R * R;
            a.obs_chunks = packs ? (N + a.obs_per_chunk - 1) / a.obs_per_chunk : share;
        } else if (mode == MODE_STEP_OBSERVE) {
            a.twin = packs && !small_batch && !long_chain ? 0 : 2;
            // (16v16 x 6144: 90 us with two wavefronts, 88 with four; 5v5 x 4096 14 and 12.5)
            if ((N >= 32 || tiny_batch) && (N > 20 || p->zone_shapes == 0)) a.twin = 4;
            if (lone_groups && N > 20 && p->zone_shapes == 0) a.twin = 8;
            if (few_groups && N > 32) a.twin = 8;
        } else if (rows) {
            // scripted: 10v10 x 16384 139 us with one wavefront per group, 121 with two; the policy as a
            // scan stage keeps them all waiting, so it has one unless the rows ask for tiles
            a.twin = mode == MODE_POLICY_STEP_OBSERVE && packs ? 0 : 2;
            // ... and four from 32 units on where there is more than one generation: with four tiles' passes in
            // flight 16v16 with zones x 6144 105.5 -> 96 us, 20v20 x 5000 113 -> 109.5, 24v24 with zones x 3000
            // 137 -> 123, 32v32 x 3000 172 -> 160; a single generation is paced, and two are better there
            // (16v16 x 4000 54 us and 58, 32v32 x 1536 82 and 88).
            if (mode == MODE_SCRIPTED_STEP_OBSERVE && (tiny_batch || (N >= 32 && !small_batch)))
                a.twin = lone_groups && N > 32 ? 8 : 4;
        }
        // Tiles that share lines (see write_rows) are longer chains, and up to four groups per CU two wavefronts
        // each are too few to hide them (two / four: 11v12 with 7 zones x 2000 27.9 / 23.5 us, 15v16 with 7 x 1800
        // 38 / 34.5, scripted 28v28 with 2 x 800 56 / 40.5, 24v24 with 4 x 1000 49 / 37.5).
        if (a.twin == 2 && (mode == MODE_STEP_OBSERVE || mode == MODE_SCRIPTED_STEP_OBSERVE) && N > 20 &&
            a.num_groups <= 4 * kComputeUnits && a.obs_dim % 32 != 0 && p->zone_shapes == 0)
            a.twin = 4;
        // On a full machine a plain tick stores two passes' rows at a time: 10v10 x 16384 107 -> 101.5 us,
        // 16v16 x 6144 93.8 -> 88; with a generation or less, shorter chains count (9v8 x 5003 39 and 48).  A
        // scripted tick, whose passes also bid, only where four wavefronts share (10v10 x 16384 122 and 131).
        const bool wide_scripted = mode == MODE_SCRIPTED_STEP_OBSERVE && a.twin == 4;
        if ((mode == MODE_STEP_OBSERVE || wide_scripted) && a.twin && !small_batch && a.tiles >= 8 * a.twin &&
            2 * S * a.obs_dim <= 2 * kTileFloats)
            K = 2;
        // Likewise where four wavefronts have six or more tiles each and there are at most two groups per CU
        // (15v15 x 800 17.1 -> 16.7 us, 12v12 with zones 15.8 -> 14.7; with fewer tiles, or three groups, one
        // pass per tile is better: 10v10 x 1200 14.9 and 15.4, 12v12 x 1400 16.9 and 17.4).
        if (mode == MODE_STEP_OBSERVE && a.twin == 4 && few_groups && a.tiles >= 6 * a.twin) K = 2;
        // A scripted tick likewise, if there are at most three groups per two CUs or the tiles stay under 6.4 KB
        // (15v15 x 799 21.2 -> 19.3 us, 20v20 x 500 20.9 -> 18.9; 16v16 with 8 KB x 799 18.5 -> 17.8, x 997 19.0
        // and 20.2; 32v32 x 400 29.1 -> 27.7, x 500 29.9 and 30.1).
        if (wide_scripted && few_groups && a.tiles >= 6 * a.twin &&
            (2 * a.num_groups <= 3 * kComputeUnits || 2 * S * a.obs_dim <= 1600))
            K = 2;
        // ... and where they have eight or more each beyond five groups per CU, short of a full machine (32v32
        // with zones x 1536 98 -> 92 us, 24v24 61.5 -> 57.4; x 1200 without zones 68.6 and 70.7).
        if (mode == MODE_STEP_OBSERVE && a.twin == 4 && a.num_groups > 5 * kComputeUnits && a.tiles >= 8 * a.twin) K = 2;
        // And with elliptical zones, whose lookups leave the other wavefronts waiting: where two share in
        // up to four groups per CU (12v12 x 500 23.0 -> 20.8 us, 4v4 x 2000 14.3 -> 13.5; beyond, x 12000 20
        // and 26), and where four do (30v30 x 1500 98 -> 84).
        if (mode == MODE_STEP_OBSERVE && (a.twin == 2 || a.twin == 4) && p->zone_shapes == 1 && a.tiles >= 2 * a.twin &&
            (N > 20 || a.num_groups <= 4 * kComputeUnits))
            K = 2;
    } else if (rows) {
        const int row_chunks = ((a.obs_dim + 3) / 4 + 3) & ~3, half = ((cpr >> 1) + 3) & ~3;
        a.copy_passes = ((half > row_chunks - half ? half : row_chunks - half) + 63) / 64;
        // What a workgroup with `w` wavefronts that make tiles takes of a CU's LDS.
        const auto tile_lds = [&](int w) {
            return sizeof(Shared<2, true, true, true>) + sizeof(float) * (w * tile_floats(1, a.obs_dim, 3) + zone_floats(a)) +
                   (mode == MODE_SCRIPTED_STEP_OBSERVE ? sizeof(ScriptLds<2>) : 0);
        };
        const int E = p->num_envs;
        const size_t row_bytes = sizeof(float) * (size_t)E * N * a.obs_dim;
        if (E <= 2 * kComputeUnits) {
            // At most two envs per CU: the chain of N rows is what such a launch waits for, so more
            // wavefronts write rows as well.  Four more with one env per CU, or while the last-level cache
            // takes all rows; beyond that HBM takes what two more write (64v64, two / four / six in all:
            // x 64 140 / 68 / 53 us, x 256 142 / 70 / 62, x 300 147 / 76 / 87, x 512 150 / 115 / 124;
            // 33v33 x 512 82 / 42 / 37; 50v50 x 300 118 / 61 / 55, x 400 - / 62 / 68).
            const bool six = (E <= kComputeUnits || row_bytes <= kLastLevelCacheBytes / 4 * 3) &&
                             tile_lds(6) <= kLdsPerWorkgroupBytes;
            a.twin = six && mode != MODE_POLICY_STEP_OBSERVE ? 3 : 2;
        } else if (a.obs_dim % 4 != 0) {
            // Rows that end on half a chunk go out in whole ones from tiles only: worth it for one
            // generation of workgroups that is not yet bound by HBM (33v33, 7 zone slots: x 600 64 us, 83
            // with the units in registers, x 1000 77 and 87, x 1280 109 and 96; 50v50 x 768 121 and 124,
            // x 1000 161 and 139; 63v64 x 768 191 and 165).
            const int held = kLdsPerCuBytes / (int)lds_granules(tile_lds(4));
            if (E <= held * kComputeUnits && row_bytes <= 2 * kLastLevelCacheBytes) a.twin = 2;
        }
        // Units in registers, from six envs per CU on: the kernel that keeps three wavefronts per SIMD, if
        // it needs no more rounds over the machine than the one that lets the CU hold eight envs, which
        // leaves some SIMDs with four wavefronts and some with two.  (33v33, three / four: x 1200 91 / 86
        // us, x 1500 93 / 98, x 2048 162 / 127, x 2500 176 / 189, x 3000 185 / 202, x 4000 258 / 240.)
        // It also takes the rows that end on half a chunk: their code would cost the other kernel 2 us.  The
        // tick with the policy as a scan stage likewise (x 1500 8 % between the two), and the scripted tick, both
        // of whose kernels have that code (three / four: x 1300 94.8 / 101.7 us, x 1500 97.2 / 105.0, x 2048
        // 170 / 121, x 3000 199.5 / 209, x 4000 271 / 253, with 7 zones x 1500 103.5 / 111, 40v40 x 1800 218 / 153).
        if (!a.twin) {
            const size_t fixed = mode == MODE_POLICY_STEP_OBSERVE ? sizeof(Shared<2, false, true>)
                                                                  : sizeof(Shared<2, false, false>);
            const bool scripted = mode == MODE_SCRIPTED_STEP_OBSERVE;
            const size_t lds = fixed + 16 * (size_t)(row_chunks + half + 64 * a.copy_passes) +
                               (scripted ? sizeof(ScriptLds<2>) : 0);
            const int held = kLdsPerCuBytes / (int)lds_granules(lds);
            const auto rounds = [&](int envs) {
                const int at_once = (envs < held ? envs : held) * kComputeUnits;
                return (E + at_once - 1) / at_once;
            };
            a.even = (!scripted && a.obs_dim % 4 != 0) || (E > 5 * kComputeUnits && rounds(6) == rounds(8));
        }
    }
    a.packed = rows && a.twin == 0;
    a.passes_per_tile = K;
    a.rows_per_tile = K * S;
    a.tiles = (G * N + a.rows_per_tile - 1) / a.rows_per_tile;
    a.tiles_per_chunk = (a.tiles + a.obs_chunks - 1) / a.obs_chunks;
    // A tile's image starts where the tile does within a line, unless that takes one more store instruction (and
    // its share of the LDS) while the last-level cache takes all rows (7 units with 5 zones, 9 rows of 568 bytes, x
    // 20000, observed: 22.5 us, 24.3 with the sixth; beyond, 10v10 with 3 zones x 16384 115 without, 103 with;
    // rows of envs of two wavefronts fill their areas, which are planned for already).
    const double bytes = 4.0 * a.obs_dim * N * p->num_envs;
    const size_t tile = (size_t)a.rows_per_tile * a.obs_dim;
    a.line = whole_passes(tile + 30) == whole_passes(tile + 2) ||
                     (waves == 1 && bytes > (double)kLastLevelCacheBytes) ? 31 : 3;
    // Each wavefront writes one contiguous run of the group's tiles.  Taken in turn, tile by tile,
    // batches whose rows are a power of two bytes long lost a tenth of the store rate (16v16 without
    // zones x 12000 155 us in turn, 137 like this; 32v32 x 6000 319 and 295).
    // Ticks of odd numbers of units up to 20 go in turn: runs cost 9v8 with zones (x 4000 29.1 us in turn, 30.0 in
    // runs; x 5003 32.7 and 34.4; x 20000 94.6 and 96.6; all with tiles that share lines and hand none on); 5, 7, 13
    // and 21 units are level, and wider odd rows are better in runs (30v29 x 5000 232 us in turn, 229 in runs).
    a.in_turn = rows && waves == 1 && a.twin && mode != MODE_OBSERVE && (N & 1) && N < 21;
    // Shared lines are handed on where a wavefront has neighbouring tiles, from where the launch is mostly rows (see
    // plan_pace), and beyond that cache from four tiles per wavefront on (5v5 with 3 zones x 65536, observed, two or
    // three: 129 us, 134 handed on; 8v7 with one x 20000, four: 67 and 62.5).  Where none can be, the code that hands
    // them on costs 1 % (9v8 with 7 ellipses x 5003 34.0 us, 33.5 without;
    // scripted 8v7 with 5 x 10000 52.2 and 51.6).
    const int per_wavefront = a.twin ? a.tiles_per_chunk / (waves * a.twin) : 0;
    const bool neighbours = !a.in_turn && a.tiles_per_chunk > waves * a.twin;
    // Envs of two wavefronts wait for their chain of rows until HBM takes no more, and the moves of a handed-on line
    // are part of it: rows of whole chunks, which gain less than those that end within one, hand on where four
    // wavefronts write them and HBM takes 2.1 us for a row of each (shared / handed on and paced: 50v50 with 2 zones x
    // 480, 2.06 us, 7 % slower, x 512, 2.2, 81.5 / 77.5; 64v64 with 2 x 330, 1.81, 83 / 86.5, x 400, 2.2, 101 / 93; 55v55
    // with 6 x 440, 2.07, 8 % faster; with six wavefronts, 1.1 ... 2.5 us, 4 to 7 % slower in all of 53; half a chunk at
    // the end: 40v40 with one x 300, 123 MB, 60.2 / 58.1, 50v50 with 3 x 700 114 / 110).
    const auto chain_of_two = [&] {
        return waves == 2 && a.obs_dim % 4 == 0 && !(a.twin == 2 && hbm_us_per_flush(a, waves) >= 2.1);
    };
    // Likewise a tick of one generation in which HBM has taken a tile of every wavefront before the next ones are made;
    // rows of whole chunks gain more, the more so the more lines a wavefront hands on (shared / handed on, in order of
    // the microseconds that is per tile; whole chunks, up to eight tiles: 13v13 with 4 zones x 1267, 1.38, 18.6 / 19.5,
    // scripted 63 units x 314, 1.66, 4 % slower, 59 or 60 with 4 x 465, 2.29, 13 % faster; more: scripted 35 x 1275,
    // 0.93, 32.6 / 35.3, 20v20 with 4 x 583, 1.03, 23.2 / 24.9, 10v10 with 4 x 2906, 1.33, 24.9 / 23.0, 15v15 with 2 x
    // 2710, 1.78, 49.7 / 37.8; half a chunk at the end: 13v13 with 7 x 1070, 1.21, 20.4 / 21.8, scripted 18v18 with
    // 7 x 1573, 1.30, 48.3 / 50.1, 15v14 with one x 2567, 1.56, 45.6 / 43.3, 53 with 7 x 741, 1.66, 41.2 / 39.4).
    const auto chain_bound = [&] {
        return waves == 1 && a.obs_chunks == 1 &&
               hbm_us_per_flush(a, waves) < (a.obs_dim % 4 == 0 && flushes_per_wavefront(a, waves) > 8 ? 1.25 : 1.5) &&
               one_generation(mode, a, waves, plan_lds(mode, a, waves));
    };
    if (a.obs_dim % 4 == 0 && tile % 32 == 0 && G * N * a.obs_dim % 32 == 0) a.lines = LINES_OWN;
    else if (neighbours && a.line == 31 && bytes > 50e6 &&
             (per_wavefront >= 4 || bytes <= (double)kLastLevelCacheBytes) && !chain_of_two() && !chain_bound()) a.lines = LINES_CARRIED;
    else a.lines = LINES_SHARED;
    return waves;
}

// Where the global state is streamed to, or null: the lanes that hold the units write their blocks then.  Those
// stores stay in the L2s and are overwritten there by the next tick, which is the better way as long as they fit
// beside the rows that pass through: at five eighths of the L2s the two meet (stored / streamed: 12v12 x 12000, 18 MB,
// 96 / 99 us, 16v16 x 9000, 18 MB, 107.5 / 110, 10v10 with zones x 14000, 21 MB, 96.5 / 95, x 15000, 22 MB, 106 / 100,
// x 16384 115 / 108.5, scripted 122 / 116.5, 16v16 x 12000, 25 MB, 153 / 145, 9v8 with zones x 18000, 23 MB,
// 107 / 104.5).  These are three batches ticked in turn, whose states together do not fit.  One batch that is ticked
// over and over, with nothing in between, leaves its state in the L2s: stored it is 4 to 5 % faster up to twice their
// size (10v10 with zones x 16384 98.9 us, 104.3 streamed, scripted 106.4 and 110.5, x 30000 171 and 182).  Launches with the units in registers, and envs of two wavefronts, have no use for it (a row of theirs
// is as long as the state of its env, and there are as many as units).
static float *plan_global(const KArgs &a)
{
    const size_t bytes = sizeof(float) * (size_t)a.p.num_envs * a.obs_dim;
    return !a.packed && bytes > kL2Bytes / 8 * 5 ? a.st.global_state : nullptr;
}

// The plan of an entry point's call (enum TabxCall), for the queries that enqueue nothing.
static int plan_call(const TabxParams *p, int call, const void *out, KArgs &a, Mode &mode, int &waves, size_t &lds)
{
    const int rc = check_params(p);
    if (rc) return rc;
    if (!out) return TABX_ERR_NULL;
    if (call < TABX_CALL_RESET || call > TABX_CALL_SCRIPTED_STEP_OBSERVE) return TABX_ERR_SHAPE;
    static const Mode modes[] = {MODE_RESET, MODE_STEP, MODE_OBSERVE, MODE_STEP_OBSERVE, MODE_POLICY,
                                 MODE_POLICY_STEP_OBSERVE, MODE_SCRIPTED_STEP_OBSERVE};
    mode = modes[call];
    take_params(p, a);
    a.obs_dim = 16 * p->num_units + 6 * p->max_zones;
    waves = plan_shape(mode, p, a);
    lds = plan_lds(mode, a, waves);
    plan_pace(mode, a, waves, lds);
    return TABX_OK;
}

static int run(Mode mode, const TabxParams *p, const TabxScenario *sc, const TabxState *st,
               const uint8_t *actions, const uint8_t *env_mask, float *rewards,
               uint8_t *dones, float *obs, uint64_t *vis_mask, uint8_t *action_mask,
               void *stream, const TabxPolicy *policy = nullptr,
               const TabxPolicyMemory *memory = nullptr, const uint8_t *controlled = nullptr,
               uint8_t *actions_out = nullptr)
{
    int rc = check_params(p);
    if (rc) return rc;
    if (p->num_envs == 0) return TABX_OK;          // empty batch: nothing to validate or do
    if ((rc = check_scenario(p, sc))) return rc;
    if ((rc = check_state(p, st))) return rc;
    const bool deciding = mode == MODE_POLICY || mode == MODE_POLICY_STEP_OBSERVE ||
                          mode == MODE_SCRIPTED_STEP_OBSERVE;
    const bool stepping = mode == MODE_STEP || mode == MODE_STEP_OBSERVE ||
                          mode == MODE_POLICY_STEP_OBSERVE || mode == MODE_SCRIPTED_STEP_OBSERVE;
    const bool observing = has_rows(mode);
    if (deciding) {
        if (!policy || !memory || !actions_out) return TABX_ERR_NULL;
        if (!memory->mem_x || !memory->mem_y || !memory->mem_valid) return TABX_ERR_NULL;
        if (!aligned(memory->mem_x, 4) || !aligned(memory->mem_y, 4)) return TABX_ERR_ALIGN;
        if (mode == MODE_SCRIPTED_STEP_OBSERVE && !memory->next_action) return TABX_ERR_NULL;
        const float fin[] = {policy->epsilon, policy->xi, policy->assassin_speed, policy->ranger_range};
        for (float v : fin)
            if (!(v > -3.0e38f && v < 3.0e38f)) return TABX_ERR_PARAM;
    }
    if (stepping) {
        if (!actions || !rewards || !dones) return TABX_ERR_NULL;
        if (!aligned(rewards, 4)) return TABX_ERR_ALIGN;
    }
    if (observing) {
        if (!obs) return TABX_ERR_NULL;
        if (!aligned(obs, 16) || (vis_mask && !aligned(vis_mask, 16))) return TABX_ERR_ALIGN;
    }
    KArgs a;
    take_params(p, a);
    a.sc = *sc;
    a.st = *st;
    a.actions = actions;
    a.env_mask = env_mask;
    a.rewards = rewards;
    a.dones = dones;
    a.obs = obs;
    a.vis_mask = vis_mask;
    a.action_mask = action_mask;
    a.obs_dim = 16 * p->num_units + 6 * p->max_zones;
    set_flags(p, st, a);
    a.pa = {};
    if (deciding) {
        a.pa.pol = *policy;
        a.pa.mem = *memory;
        a.pa.controlled = controlled;
        a.pa.actions_out = actions_out;
        a.pa.next_action = memory->next_action;
    }

    hipStream_t s = (hipStream_t)stream;
    const int waves = plan_shape(mode, p, a);
    a.global_stream = observing && waves == 1 ? plan_global(a) : nullptr;
    if (a.global_stream) a.st.global_state = nullptr;
    const hipError_t err = waves == 1 ? launch_mode<1>(mode, a, s) : launch_mode<2>(mode, a, s);
    return err == hipSuccess ? TABX_OK : TABX_ERR_LAUNCH;
}

} // namespace tabx

#ifdef TABX_TRACE
// Instrumented builds only: copies the first n time stamps to the host / clears them.
extern "C" int tabx_dbg_read(void *dst, int n)
{
    if (hipDeviceSynchronize() != hipSuccess) return -1;
    return hipMemcpyFromSymbol(dst, HIP_SYMBOL(tabx::g_trace), (size_t)n * 8) == hipSuccess ? 0 : -1;
}
extern "C" int tabx_dbg_clear(void)
{
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(tabx::g_trace)) != hipSuccess) return -1;
    return hipMemset(p, 0, sizeof(tabx::g_trace)) == hipSuccess ? 0 : -1;
}
#endif

extern "C" {

int tabx_obs_dim(const TabxParams *p)
{
    const int rc = tabx::check_params(p);
    if (rc) return rc;
    return 16 * p->num_units + 6 * p->max_zones;
}

int tabx_num_actions(void) { return TABX_NUM_ACTIONS; }

int tabx_reset(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
               const uint8_t *env_mask, void *stream)
{
    return tabx::run(tabx::MODE_RESET, p, sc, st, nullptr, env_mask, nullptr, nullptr, nullptr,
                     nullptr, nullptr, stream);
}

int tabx_step(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
              const uint8_t *actions, float *rewards, uint8_t *dones, void *stream)
{
    return tabx::run(tabx::MODE_STEP, p, sc, st, actions, nullptr, rewards, dones, nullptr,
                     nullptr, nullptr, stream);
}

int tabx_observe(const TabxParams *p, const TabxScenario *sc, const TabxState *st, float *obs,
                 uint64_t *vis_mask, uint8_t *action_mask, void *stream)
{
    return tabx::run(tabx::MODE_OBSERVE, p, sc, st, nullptr, nullptr, nullptr, nullptr, obs,
                     vis_mask, action_mask, stream);
}

int tabx_step_observe(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
                      const uint8_t *actions, float *rewards, uint8_t *dones, float *obs,
                      uint64_t *vis_mask, uint8_t *action_mask, void *stream)
{
    return tabx::run(tabx::MODE_STEP_OBSERVE, p, sc, st, actions, nullptr, rewards, dones, obs,
                     vis_mask, action_mask, stream);
}

int tabx_global_state(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
                      float *out, void *stream)
{
    int rc = tabx::check_params(p);
    if (rc) return rc;
    if (p->num_envs == 0) return TABX_OK;
    if ((rc = tabx::check_scenario(p, sc))) return rc;
    if ((rc = tabx::check_state(p, st))) return rc;
    if (!out) return TABX_ERR_NULL;
    if (!tabx::aligned(out, 16)) return TABX_ERR_ALIGN;
    tabx::KArgs a = {};
    tabx::take_params(p, a);
    a.sc = *sc;
    a.st = *st;
    tabx::set_flags(p, st, a);
    const size_t units = (size_t)p->num_envs * p->num_units;
    const size_t zones = (size_t)p->num_envs * 6 * p->max_zones;
    const size_t threads = units > zones ? units : zones;
    void *args[] = {(void *)&a, (void *)&out};
    const hipError_t err = hipLaunchKernel((const void *)tabx::tabx_global_state_kernel,
                                           dim3((unsigned)((threads + 255) / 256)), dim3(256), args,
                                           0, (hipStream_t)stream);
    return err == hipSuccess ? TABX_OK : TABX_ERR_LAUNCH;
}

int tabx_heuristic_actions(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
                           const TabxPolicy *policy, const TabxPolicyMemory *memory,
                           const uint8_t *controlled, uint8_t *actions, void *stream)
{
    return tabx::run(tabx::MODE_POLICY, p, sc, st, nullptr, nullptr, nullptr, nullptr, nullptr,
                     nullptr, nullptr, stream, policy, memory, controlled, actions);
}

int tabx_policy_step_observe(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
                             const TabxPolicy *policy, const TabxPolicyMemory *memory,
                             const uint8_t *controlled, uint8_t *actions, float *rewards,
                             uint8_t *dones, float *obs, uint64_t *vis_mask,
                             uint8_t *action_mask, void *stream)
{
    return tabx::run(tabx::MODE_POLICY_STEP_OBSERVE, p, sc, st, actions, nullptr, rewards, dones,
                     obs, vis_mask, action_mask, stream, policy, memory, controlled, actions);
}

int tabx_scripted_step_observe(const TabxParams *p, const TabxScenario *sc, const TabxState *st,
                               const TabxPolicy *policy, const TabxPolicyMemory *memory,
                               const uint8_t *controlled, uint8_t *actions, float *rewards,
                               uint8_t *dones, float *obs, uint64_t *vis_mask,
                               uint8_t *action_mask, void *stream)
{
    return tabx::run(tabx::MODE_SCRIPTED_STEP_OBSERVE, p, sc, st, actions, nullptr, rewards,
                     dones, obs, vis_mask, action_mask, stream, policy, memory, controlled,
                     actions);
}

int tabx_part(const TabxParams *p, const TabxScenario *sc, const TabxState *st, int32_t first_env,
              int32_t count, TabxParams *pp, TabxScenario *psc, TabxState *pst)
{
    int rc = tabx::check_params(p);
    if (rc) return rc;
    if (!sc || !st || !pp || !psc || !pst) return TABX_ERR_NULL;
    if (first_env < 0 || count < 0 || (int64_t)first_env + count > p->num_envs) return TABX_ERR_SHAPE;
    const size_t N = (size_t)p->num_units;
    const size_t e0 = (size_t)first_env, u0 = e0 * N;
    *pp = *p;
    pp->num_envs = count;
    pp->env_id_offset = p->env_id_offset + first_env;
    if (count < p->num_envs) pp->shared_machine = 1;
    *psc = *sc;
    if (p->num_levels == 0) {          // one scenario row per env: the part starts at its own
        const float **f[] = {&psc->init_x, &psc->init_y, &psc->init_theta, &psc->hmax, &psc->radius,
                             &psc->mass, &psc->speed, &psc->dmg, &psc->range, &psc->cooldown,
                             &psc->sight_angle, &psc->sight_cos_half, &psc->sight_range,
                             &psc->hurt_halfwidth};
        for (const float **q : f)
            if (*q) *q += u0;
        if (psc->team) psc->team += u0;
        if (psc->enabled) psc->enabled += u0;
        if (psc->terrain) psc->terrain += e0 * (size_t)p->grid_h * (size_t)p->grid_w;
        if (psc->zone_desc) psc->zone_desc += e0 * 6 * (size_t)p->max_zones;
    }
    *pst = *st;
    float **uf[] = {&pst->x, &pst->y, &pst->vx, &pst->vy, &pst->theta, &pst->hp, &pst->cd,
                    &pst->reveal, &pst->cur_speed};
    for (float **q : uf)
        if (*q) *q += u0;
    if (pst->alive) pst->alive += u0;
    if (pst->t) pst->t += e0;
    if (pst->phi_prev) pst->phi_prev += e0;
    if (pst->ret_run) pst->ret_run += e0;
    if (pst->kill_run) pst->kill_run += e0;
    if (pst->ep_count) pst->ep_count += e0;
    if (pst->ep_len) pst->ep_len += e0;
    if (pst->ep_return) pst->ep_return += e0;
    if (pst->ep_win) pst->ep_win += e0;
    if (pst->ep_first_kill) pst->ep_first_kill += e0;
    if (pst->level) pst->level += e0;
    if (pst->next_level) pst->next_level += e0;
    if (pst->level_draws) pst->level_draws += e0;
    if (pst->global_state)
        pst->global_state += e0 * (16 * N + 6 * (size_t)p->max_zones);
    if (pst->ax) pst->ax += u0;
    if (pst->ay) pst->ay += u0;
    return TABX_OK;
}

int tabx_launch_info(const TabxParams *p, int call, TabxLaunchInfo *info)
{
    using namespace tabx;
    KArgs a = {};
    Mode mode;
    int waves;
    size_t lds;
    const int rc = plan_call(p, call, info, a, mode, waves, lds);
    if (rc) return rc;
    info->workgroups = 8 * a.groups_per_xcd * a.obs_chunks;
    info->threads_per_workgroup = 64 * waves * (a.twin ? a.twin : 1);
    info->envs_per_workgroup = a.envs_per_block;
    info->wavefronts_per_env_group = waves * (a.twin ? a.twin : 1);
    info->rows_per_flush = a.packed ? a.rows_per_flush : a.rows_per_tile;
    info->dynamic_lds_bytes = (int32_t)lds;
    info->assumed_compute_units = kComputeUnits;
    info->assumed_lds_per_cu_bytes = kLdsPerCuBytes;
    info->assumed_lds_per_workgroup_bytes = kLdsPerWorkgroupBytes;
    info->assumed_wavefront_lanes = kWavefrontLanes;
    return TABX_OK;
}

int tabx_row_form(const TabxParams *p, int call, TabxRowForm *form)
{
    using namespace tabx;
    KArgs a = {};
    Mode mode;
    int waves;
    size_t lds;
    const int rc = plan_call(p, call, form, a, mode, waves, lds);
    if (rc) return rc;
    float any;
    a.st.global_state = &any;
    form->lines = has_rows(mode) && !a.packed ? a.lines : -1;
    form->pace = (int32_t)a.pace;
    form->wavefronts_per_simd = has_rows(mode) ? wavefronts_per_simd(mode, a, waves) : -1;
    form->streams_global_state = has_rows(mode) && waves == 1 && plan_global(a) != nullptr;
    return TABX_OK;
}

const char *tabx_strerror(int code)
{
    switch (code) {
    case TABX_OK: return "ok";
    case TABX_ERR_NULL: return "a required pointer is NULL (or an optional one does not match the shape)";
    case TABX_ERR_SHAPE: return "unsupported shape (num_units, max_zones, grid, max_steps or num_envs)";
    case TABX_ERR_ALIGN: return "a pointer is not aligned as required";
    case TABX_ERR_LAUNCH: return "the HIP runtime refused the kernel launch";
    case TABX_ERR_PARAM: return "a physics constant is not finite or not positive";
    default: return "unknown error code";
    }
}

} // extern "C"
