// Step stage of the TABX tick (App. A "Interaction Dynamics", "Reward", "Zones"): timers,
// kinematics, actions, hurtbox combat, zone effects, rewards, termination and auto-reset.
#pragma once
#include "tabx_device.h"
#include "tabx_policy.h"   // policy_hash draws the levels

#pragma clang fp contract(off)

namespace tabx {

// Level bank: an episode of the lane's env is about to start (`take`, uniform over the env's
// lanes).  Unit 0 takes the queued level (folded into [0, num_levels)), refills the queue with
// a uniform draw, the hash of (level_seed, env, draws so far), and tells the env's other lanes
// through LDS (one slot per env of the workgroup).  Returns the env's new row, or -1
// if it keeps its level.  All lanes call it.
template <int WAVES, class Sh>
__device__ __forceinline__ int advance_level(const KArgs &a, Sh &sh, const Place &P,
                                             bool take)
{
    if (P.has && P.u == 0) {
        int row = -1;
        if (take) {
            const LateArgs late = late_args();
            int32_t *const level = late->st.level, *const next_level = late->st.next_level;
            int32_t *const level_draws = late->st.level_draws;
            const uint32_t L = (uint32_t)a.p.num_levels;
            row = (int)((uint32_t)next_level[P.e] % L);
            const uint32_t n = (uint32_t)level_draws[P.e];
            level[P.e] = row;
            next_level[P.e] = (int)(policy_hash(a.p.level_seed, (uint32_t)(P.e + a.p.env_id_offset), 0u, n, 3u) % L);
            level_draws[P.e] = (int)(n + 1u);
        }
        sh.level_rows[P.g] = row;
    }
    group_barrier<WAVES>(sh);
    return P.has ? sh.level_rows[P.g] : -1;
}

// What the step stage reads besides the unit's state and specification.
struct StepIn {
    int   act;                     // the unit's entry of the action array
    int   t;                       // the env's tick counter, potential and running metrics
    float phi_prev;
    int   kills_run;
    float ret_run;
    float acx, acy;                // persistent velocities: the acceleration the last action stage set
};

// Issued with the state at the top of the kernel: whatever the wavefront waits for first (zones on
// their way to LDS, a policy's memory), these are not a second round trip after it.
__device__ __forceinline__ void load_step(const KArgs &a, const Place &P, StepIn &in)
{
    const uint32_t e = (uint32_t)P.e;
    in.act = at32(a.actions, P.k);
    in.t = at32(a.st.t, e);
    in.phi_prev = at32(a.st.phi_prev, e);
}

// ... where the launch asks for them.
__device__ __forceinline__ void load_more_step(const KArgs &a, const Place &P, StepIn &in)
{
    if (flagged(a, DYNAMIC | KILLS | RETURNS)) {
        const LateArgs late = late_args();
        const uint32_t e = here((uint32_t)P.e), k = here(P.k);
        if (flagged(a, DYNAMIC)) {
            in.acx = at32(late->st.ax, k);
            in.acy = at32(late->st.ay, k);
        }
        if (flagged(a, KILLS)) in.kills_run = at32(late->st.kill_run, e);
        if (flagged(a, RETURNS)) in.ret_run = at32(late->st.ret_run, e);
    }
}

// Stage 1: explicit Euler move, arena penalty + clip.  Returns whether the move took the unit out of the
// arena.  (Of the unit's loads it needs the first six only.)
__device__ __forceinline__ bool move_unit(const KArgs &a, Unit &U, const StepIn &in)
{
    const float dt = a.p.dt;
    const bool moves = U.enabled && U.alive;
    if (flagged(a, DYNAMIC)) {         // the velocity from the acceleration first, then the position
        U.vx = moves ? U.vx + in.acx * dt : U.vx;
        U.vy = moves ? U.vy + in.acy * dt : U.vy;
    }
    const float nx = U.x + U.vx * dt;
    const float ny = U.y + U.vy * dt;
    const bool oob = (nx < 0.0f) | (nx > a.p.map_w) | (ny < 0.0f) | (ny > a.p.map_h);
    U.x = moves ? clamp_between(nx, 0.0f, a.p.map_w) : U.x;
    U.y = moves ? clamp_between(ny, 0.0f, a.p.map_h) : U.y;
    return moves & oob;
}

// Stage 1b: overlapping bodies are pushed apart.  Every unit sums, over its partners in
// ascending index, the share of each overlap it has to give way for; all pairs are taken
// on the positions after the kinematic update; then the unit is clipped again.
template <int WAVES, class Sh>
__device__ __forceinline__ void collide_env(const KArgs &a, Sh &sh, const Place &P, Unit &U)
{
    const int N = a.p.num_units;
    const LateArgs late = late_args();
    const bool dynamic = late->p.dynamics == 1;
    const bool on = U.enabled != 0;
    {
        // partner record: x, y, radius, mass (negative mass: not a body)
        sh.st.pj[P.l] = make_float4(U.x, U.y, U.radius, on ? U.mass : -1.0f);
        // (with persistent velocities the partners' velocities travel in the next array, which
        // the combat stage rewrites only after the barrier that ends this stage)
        if (dynamic) sh.st.aim1[P.l] = make_float4(U.vx, U.vy, 0.0f, 0.0f);
        group_barrier<WAVES>(sh);
        float ax = 0.0f, ay = 0.0f;
        float dvx = 0.0f, dvy = 0.0f;
        const float inv_i = 1.0f / U.mass;             // 0 for a kinematic body, which takes no impulse
        const bool bounces = dynamic && inv_i != 0.0f;
        // Few bodies touch, and a pair's square root and divisions cost several times the test whether it
        // can: each lane first marks the partners that are near enough, without a branch, and then
        // works its own ones off in ascending index, as many rounds as the busiest lane has contacts.
        // (10v10, ellipses, impulses: step stage 15.5 -> 6 us.)  A pair counts if pen > slop (push)
        // or pen > 0 (impulse), pen = (r_i + r_j) - dist; beyond reach^2 * (1 + 2^-16), reach =
        // r_i + r_j + max(-slop, 0), the rounded pen is below both, and a pair that does not count
        // adds a zero product, which leaves the finite sums unchanged.
        const float rebound = 1.0f + late->p.restitution;
        const float margin = a.p.collision_slop < 0.0f ? -a.p.collision_slop : 0.0f;
        uint64_t close[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            uint32_t half[2] = {0u, 0u};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int first = 64 * w + 32 * h;
                const int count = N - first < 32 ? N - first : 32;
#pragma unroll 4
                for (int b = 0; b < count; ++b) {
                    const float4 J = sh.st.pj[P.base + first + b];
                    const float dx = J.x - U.x;
                    const float dy = J.y - U.y;
                    const float reach = (U.radius + J.z) + margin;
                    const bool apart = (dx * dx) + (dy * dy) > (reach * reach) * (1.0f + 0x1p-16f);
                    half[h] |= apart || !(J.w >= 0.0f) ? 0u : 1u << b;
                }
            }
            close[w] = ((uint64_t)half[1] << 32) | half[0];
            // (not with itself, and only bodies)
            if (P.u >= 64 * w && P.u < 64 * w + 64) close[w] &= ~(1ull << (P.u & 63));
            if (!on) close[w] = 0ull;
        }
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            while (close[w] != 0ull) {
                const int jj = 64 * w + __builtin_ctzll(close[w]);
                close[w] &= close[w] - 1ull;
                const float4 J = sh.st.pj[P.base + jj];
                const float dx = J.x - U.x;
                const float dy = J.y - U.y;
                const float dist = __builtin_sqrtf((dx * dx) + (dy * dy));
                const float pen = (U.radius + J.z) - dist;
                const bool apart = dist > 0.0f;
                // coincident centres separate along x, the lower index to the left
                const float nx = apart ? dx / dist : (P.u < jj ? 1.0f : -1.0f);
                const float ny = apart ? dy / dist : 0.0f;
                if (dynamic) {
                    // impulse along the normal from the relative velocity, unless the pair is
                    // already separating; split by inverse mass (the slop gates the correction only)
                    const float4 V = sh.st.aim1[P.base + jj];
                    const float rvx = V.x - U.vx;
                    const float rvy = V.y - U.vy;
                    const float vn = (rvx * nx) + (rvy * ny);
                    const float inv_j = 1.0f / J.w;
                    const float jimp = (rebound * (0.0f - vn)) / (inv_i + inv_j);
                    const bool hit = bounces && (pen > 0.0f) && !(vn > 0.0f);
                    // (subtracting a zero product leaves the finite sum unchanged)
                    const float je = hit ? jimp * inv_i : 0.0f;
                    dvx = dvx - (je * nx);
                    dvy = dvy - (je * ny);
                }
                // a kinematic body (infinite mass) gives way to nobody; a body of finite mass
                // gives way to it for the whole corrected depth
                const float inf = __builtin_inff();
                const float share = U.mass == inf ? 0.0f : (J.w == inf ? 1.0f : J.w / (U.mass + J.w));
                const float c = ((pen - a.p.collision_slop) * a.p.collision_alpha) * share;
                const float ce = pen > a.p.collision_slop ? c : 0.0f;
                ax = ax - (ce * nx);
                ay = ay - (ce * ny);
            }
        }
        U.x = on ? clamp_between(U.x + ax, 0.0f, a.p.map_w) : U.x;
        U.y = on ? clamp_between(U.y + ay, 0.0f, a.p.map_h) : U.y;
        if (dynamic) {
            U.vx = on ? U.vx + dvx : U.vx;
            U.vy = on ? U.vy + dvy : U.vy;
        }
        group_barrier<WAVES>(sh);          // the partner records are rewritten for the combat stage
    }
}

// The rest of the tick, from the actions on.
// `forced` >= 0 replaces the unit's entry of the action array (the policy stage chose it).
// `Z`: the zone descriptors of the group's envs in LDS, rewritten for envs that change level; `zd`
// those of the lane's env; `oob`: the move took the unit out of the arena; `code_u`, `zeff`: the zone under it
// and, for elliptical ones, its effect magnitude.  Returns whether any env of the workgroup restarted.
//
// A small batch is one chain of instructions, a lone wavefront issues one in about four cycles, and on a full
// machine the wavefronts of a SIMD issue this stage in turn: so it is selects instead of branches, and what a
// striker needs is looked up by its rank.
template <int WAVES, class Sh>
__device__ __forceinline__ bool step_env(const KArgs &a, Sh &sh,
                                         const ZoneLds &Z, const float *zd,
                                         Place &P, Unit &U, int &code_u, float &zeff, bool oob,
                                         Carry &C, const StepIn &in, int forced)
{
    const int N = a.p.num_units;
    const float dt = a.p.dt;
    const bool has = P.has;
    const int alive0 = U.alive;
    const bool on = U.enabled != 0;
    const int act = alive0 ? (forced >= 0 ? forced : in.act) : TABX_ACT_NOOP;
    const int t_new = in.t + 1;
    const float phi_prev = in.phi_prev;
    const LateArgs late = late_args();
    float acx = 0.0f, acy = 0.0f;

    // The action array is the one input that is new in every tick, so its lines come from HBM,
    // where a read queues behind the observation stores for microseconds once those are
    // flowing, and every wavefront's step stage waits for its action bytes.  The first
    // wavefronts of each XCD, which start while HBM is still idle, therefore touch every line of
    // their XCD's share of the array (lane l of the j-th wavefront: line 64 j + l); the later
    // generations find them in the cache.  Measured with a fresh action batch per tick:
    // c3 108.6 -> 102.5 us, c4 95.4 -> 89.7 us (101 / 88 us with actions that are cached anyway).
    {
        const uint32_t span = (uint32_t)(a.groups_per_xcd * a.envs_per_block) * (uint32_t)N;   // units per XCD
        if ((blockIdx.x >> 3) <= span / 8192u) {
            const uint32_t off = ((blockIdx.x >> 3) * 64u + (threadIdx.x & 63u)) * 128u;
            const uint64_t at = (uint64_t)(blockIdx.x & 7u) * span + off;
            if (off < span && at < (uint32_t)a.p.num_envs * (uint32_t)N) C.warm = at32(a.actions, (uint32_t)at);
        }
    }

    // stage 1, the timers
    {
        const float c = U.cd - dt, r = U.reveal - dt;
        U.cd = on ? (c > 0.0f ? c : 0.0f) : U.cd;
        U.reveal = on ? (r > 0.0f ? r : 0.0f) : U.reveal;
    }

    // stage 2a: movement sets next tick's velocity, rotation turns the heading now
    float cu, su;
    {
        // the velocity the unit wants: its current speed along a move action, else none
        const float sp = U.cur_speed;
        const float wx = act == TABX_ACT_MOVE_XP ? sp : (act == TABX_ACT_MOVE_XM ? -sp : 0.0f);
        const float wy = act == TABX_ACT_MOVE_YP ? sp : (act == TABX_ACT_MOVE_YM ? -sp : 0.0f);
        if (flagged(a, DYNAMIC)) {
            // the acceleration for the next tick's physics stage; what is not alive holds neither
            acx = alive0 ? (wx - U.vx) * late->p.move_gain : 0.0f;
            acy = alive0 ? (wy - U.vy) * late->p.move_gain : 0.0f;
            if (!alive0) U.vx = U.vy = 0.0f;
        } else {
            U.vx = wx;
            U.vy = wy;
        }
        float left = U.theta + (a.p.turn_rate * dt);
        if (left >= kTwoPi) left = left - kTwoPi;
        float right = U.theta - (a.p.turn_rate * dt);
        if (right < 0.0f) right = right + kTwoPi;
        if (act == TABX_ACT_ROT_LEFT) U.theta = left;
        if (act == TABX_ACT_ROT_RIGHT) U.theta = right;
        heading_sincos(U.theta, su, cu);
    }
    // stage 2b: combat, seen from the victims.  Few units strike in a tick (the cooldowns see to
    // that), so instead of every unit scanning its env for targets, every unit tests itself
    // against the strikers of its env only.  The n-th striker of an env (of those a wavefront holds) publishes
    // its pose and hurtbox in the n-th place of the env; each unit
    // in that hurtbox (body circle against the forward rectangle, role filter, optionally the
    // sight cone's angle) bids for "closest" with an LDS atomic minimum over the 64-bit key
    // (squared distance bits, unit index): the smallest key is the closest valid body, the
    // lowest index among equally distant ones.
    const bool eligible = act == TABX_ACT_ATTACK && U.cd <= 0.0f;
    int my_rank = -1;              // the unit's place if it strikes
    // how many the env has, per wavefront that holds its units (two hold one env: the count is uniform, and known
    // to be, or a round of the loops below takes 40 ns more, 64v64 x 200 0.7 us of the step stage's 6.3)
    int strikers[WAVES];
    {
        const uint64_t b = lanes_where(eligible);
        const uint64_t mine = WAVES == 1 ? b & lanes_of_env(P, N) : b;
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
        strikers[0] = __popcll(mine);
        if (WAVES == 2 && (P.l & 63) == 0) sh.ballots[P.l >> 6][0] = b;
        if (eligible) {
            U.cd = U.cooldown;
            my_rank = (WAVES == 1 ? P.base : P.l & 64) + rank;
            const int want = (U.dmg < 0.0f) ? U.team : 1 - U.team;   // healers reach allies only
            // the attack range is never negative: its sign bit carries the team the strike is for
            const float range_want = __int_as_float(__float_as_int(U.range) | (want << 31));
            sh.st.aim0[my_rank] = make_float4(U.x, U.y, cu, su);
            sh.st.aim1[my_rank] = make_float4(range_want, U.hurt_hw, U.dmg, U.cos_half);
            sh.st.best[my_rank] = ~0ull;
        }
    }
    group_barrier<WAVES>(sh);
    if (WAVES == 2) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) strikers[w] = __builtin_amdgcn_readfirstlane(__popcll(sh.ballots[w][0]));
    }

    float acc = 0.0f;              // what lands on this unit, strikers in ascending index
    bool struck = false;           // ... and whether any of it was damage
    {
        const float r2 = U.radius * U.radius;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int first = WAVES == 1 ? P.base : 64 * w;
            for (int n = 0; WAVES == 1 ? lanes_where(n < strikers[w]) != 0ull : n < strikers[w]; ++n) {
                const float4 A0 = sh.st.aim0[first + n];
                const float4 A1 = sh.st.aim1[first + n];
                const int rb = __float_as_int(A1.x);
                const float range = __int_as_float(rb & 0x7fffffff);
                const int want = (rb >> 31) & 1;
                const float dx = U.x - A0.x;
                const float dy = U.y - A0.y;
                float along;
                const float g2 = hurtbox_gap2(dx, dy, A0.z, A0.w, range, A1.y, -A1.y, along);
                const float d2 = (dx * dx) + (dy * dy);
                bool ok = alive0 && n < strikers[w] && U.team == want && first + n != my_rank && g2 <= r2;
                if (flagged(a, CONE_BOUND)) ok = ok && ((d2 == 0.0f) || (along >= A1.w * __builtin_sqrtf(d2)));
                if (ok) {
                    const unsigned long long key =
                        ((unsigned long long)(unsigned)__float_as_int(d2) << 32) | (unsigned)P.u;
                    atomicMin(&sh.st.best[first + n], key);
                }
                if (flagged(a, HIT_ALL)) {                 // a strike lands on everybody in the hurtbox
                    acc = ok ? acc + A1.z : acc;
                    struck = struck || (ok && A1.z > 0.0f);
                }
            }
        }
    }
    group_barrier<WAVES>(sh);

    // stage 2c: a strike has landed if anybody bid; unless everybody in the hurtbox is struck,
    // the victims now look up which striker designated them
    bool landed = false;
    if (eligible) landed = sh.st.best[my_rank] != ~0ull;
    if (!flagged(a, HIT_ALL)) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int first = WAVES == 1 ? P.base : 64 * w;
            for (int n = 0; WAVES == 1 ? lanes_where(n < strikers[w]) != 0ull : n < strikers[w]; ++n) {
                const bool mine = n < strikers[w] && (unsigned)sh.st.best[first + n] == (unsigned)P.u;
                const float d = sh.st.aim1[first + n].z;
                acc = acc + (mine ? d : 0.0f);
                struck = struck || (mine && d > 0.0f);
            }
        }
    }
    struck = struck || (landed && U.dmg > 0.0f);
    {
        // subtract once, together with the arena penalty; clamp
        const float bdmg = oob ? (a.p.boundary_frac * U.hmax) * dt : 0.0f;
        const float h = (U.hp - acc) - bdmg;
        U.hp = alive0 ? clamp_between(h, 0.0f, U.hmax) : U.hp;
        if (alive0 && struck) U.reveal = a.p.reveal_time;
    }
    // (the ratio terms written next share LDS with the strikers' poses, which nobody reads any
    // more: the bids above were the last use, and a barrier has passed since)

    // stage 3: zone effects at the new position, alive flag
    float ratio;
    {
        const int zone = code_u & 3;
        const float h = U.hp - (zone_magnitude(a, zeff, a.p.lava_dps) * dt);
        U.hp = on && alive0 && zone == TABX_ZONE_LAVA ? (h > 0.0f ? h : 0.0f) : U.hp;
        const float slowed = U.speed * zone_magnitude(a, zeff, a.p.swamp_mult);
        if (on) U.cur_speed = zone == TABX_ZONE_SWAMP ? +slowed : +U.speed;
        U.alive = on && U.hp > 0.0f ? 1 : 0;
        ratio = U.hp / U.hmax;
        ratio = on ? ratio : 0.0f;
    }
    const bool first_team = on && U.team == 0, second_team = on && U.team != 0;
    sh.st.share[P.l] = make_float2(first_team ? ratio : 0.0f, second_team ? ratio : 0.0f);
    const bool pred[4] = {first_team, second_team, U.alive && U.team == 0, U.alive && U.team != 0};
    int cnt[4];
    env_counts<WAVES>(sh, P, N, pred, cnt);
    // episode metrics need the alive counts at entry as well (first loss of a unit)
    int before[2] = {0, 0};
    if (flagged(a, KILLS)) {
        const bool pred0[2] = {alive0 && U.team == 0, alive0 && U.team != 0};
        env_counts<WAVES>(sh, P, N, pred0, before);
    }
    group_barrier<WAVES>(sh);

    // reward (Eq. 1), termination, terminal bonus
    float m0, m1;
    team_means(sh, P, N, cnt[0], cnt[1], m0, m1);
    const float phi = m0 - m1;
    const float dense = phi - phi_prev;
    const bool done = has && (cnt[2] == 0 || cnt[3] == 0 || t_new >= a.p.max_steps);
    // does any env of this workgroup restart?  (one env per workgroup when WAVES == 2:
    // the flag is already uniform there, up to the idle lanes)
    bool any_done;
    if (WAVES == 1) {
        any_done = lanes_where(done) != 0ull;
    } else {
        const uint64_t b = lanes_where(done);
        if ((P.l & 63) == 0) sh.ballots[P.l >> 6][0] = b;
        group_barrier<WAVES>(sh);
        any_done = (sh.ballots[0][0] | sh.ballots[WAVES - 1][0]) != 0ull;
    }
    const float bonus = m0 > m1 ? 1.0f : -1.0f;
    const float r0 = done ? dense + bonus : +dense;
    const float r1 = done ? -dense - bonus : -dense;
    if (has) at32(a.rewards, here(P.k)) = on ? (U.team ? +r1 : +r0) : 0.0f;

    // auto-reset of finished envs; the potential of the fresh state seeds phi_prev
    float phi_next = phi;
    group_barrier<WAVES>(sh);          // everyone has read the ratio terms of the finished tick
    if (any_done) {
        bool on_next = on;
        if (flagged(a, LEVELS)) {
            // the finished envs move to their queued level: new specifications, new zones
            const int row = advance_level<WAVES>(a, sh, P, done);
            if (row >= 0) {
                P.row = row;
                P.ks = (uint32_t)row * (uint32_t)N + (uint32_t)P.u;
                load_spec(a, P.ks, U);
                fold_byte(U.team);
                on_next = U.enabled != 0;
            }
            if (a.zones_in_lds) {
                // (level_rows holds an entry for every env of the group, and only for those)
                constexpr bool LATE = WAVES == 2;
                const int ZC = LATE ? late->zone_chunks : a.zone_chunks;
                const int chunks = envs_of_group(a, P.grp) * ZC;
                for (int q = P.l; q < chunks; q += 64 * WAVES) {
                    const int g = quotient(q, LATE ? late->magic_zc : a.magic_zc);
                    const int moved = sh.level_rows[g];
                    if (moved >= 0) put_zone_chunk<LATE>(a, Z, g, q - g * ZC, moved);
                }
                group_barrier<WAVES>(sh);
            }
        }
        if (done) {
            // a new episode remembers nothing
            uint8_t *const mem_valid = late->pa.mem.mem_valid;
            if (mem_valid) at32(mem_valid, P.k) = 0;
            code_u = spawn_unit(a, zd, P.row, P.ks, U, zeff);
            acx = 0.0f;
            acy = 0.0f;
            ratio = U.enabled ? U.hp / U.hmax : 0.0f;
            heading_sincos(U.theta, su, cu);
        }
        int c0 = cnt[0], c1 = cnt[1];
        if (flagged(a, LEVELS)) {
            // teams and placeholders may differ in the new level
            const bool pred1[2] = {on_next && U.team == 0, on_next && U.team != 0};
            int fresh[2];
            env_counts<WAVES>(sh, P, N, pred1, fresh);
            c0 = fresh[0];
            c1 = fresh[1];
        }
        sh.st.share[P.l] = make_float2((on_next && U.team == 0) ? ratio : 0.0f,
                                    (on_next && U.team != 0) ? ratio : 0.0f);
        group_barrier<WAVES>(sh);
        float f0, f1;
        team_means(sh, P, N, c0, c1, f0, f1);
        if (done) phi_next = f0 - f1;
    }
    if (has && P.u == 0) {
        const uint32_t e = here((uint32_t)P.e);
        at32(a.st.t, e) = done ? 0 : t_new;
        at32(a.st.phi_prev, e) = phi_next;
        at32(a.dones, e) = done ? 1 : 0;
        // episode metrics: first loss of a unit, running allied return, summary at the end
        int kills = 0;
        if (flagged(a, KILLS)) {
            kills = in.kills_run;
            if (kills == 0) kills = (cnt[3] < before[1] ? 1 : 0) | (cnt[2] < before[0] ? 2 : 0);
            at32(late->st.kill_run, e) = (int8_t)(done ? 0 : kills);
        }
        float ret = 0.0f;
        if (flagged(a, RETURNS)) {
            ret = in.ret_run + r0;
            at32(late->st.ret_run, e) = done ? 0.0f : +ret;
        }
        if (done) {
            if (late->st.ep_count) late->st.ep_count[P.e] += 1;
            if (late->st.ep_len) late->st.ep_len[P.e] = t_new;
            if (late->st.ep_return && late->st.ret_run) late->st.ep_return[P.e] = ret;
            if (late->st.ep_win) late->st.ep_win[P.e] = (m0 > m1) ? 1 : 0;
            if (late->st.ep_first_kill && late->st.kill_run) late->st.ep_first_kill[P.e] = (int8_t)kills;
        }
    }
    if (has) {
        store_state(a, P.k, U);
        if (flagged(a, DYNAMIC)) {
            const uint32_t k = here(P.k);
            at32(late->st.ax, k) = acx;
            at32(late->st.ay, k) = acy;
        }
    }
    C.cu = cu;
    C.su = su;
    C.ratio = ratio;
    C.tick = done ? 0 : t_new;
    C.restarted = done;
    return any_done;
}

} // namespace tabx
