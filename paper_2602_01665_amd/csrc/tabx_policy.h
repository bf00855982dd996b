// Heuristic policy stage of the TABX tick (Sec. 4.2; App. A "Role-Appropriate Heuristic
// Policy Mechanism").
#pragma once
#include "tabx_device.h"

#pragma clang fp contract(off)

namespace tabx {

// Role-appropriate heuristic policy (Sec. 4.2; App. A "Role-Appropriate Heuristic Policy
// Mechanism" and the table of tier parameters).  Lane = deciding unit; the units of its env
// are scanned through records in LDS.  Visibility and reach are the tests of the observation
// (fan-shaped field of view, bush rule, hurtbox, role filter), from the observer's side.

// Counter-based random numbers: two multiply / xor-shift rounds over the draw's coordinates.
__device__ __forceinline__ uint32_t policy_hash(uint32_t seed, uint32_t env, uint32_t unit,
                                                uint32_t tick, uint32_t draw)
{
    uint32_t x = seed;
    x ^= env * 0x9E3779B9u;
    x ^= unit * 0x85EBCA6Bu;
    x ^= tick * 0xC2B2AE35u;
    x ^= draw * 0x27D4EB2Fu;
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}

// The cardinal move that closes most of the offset (gx, gy); idle if there is none.
__device__ __forceinline__ int move_along(float gx, float gy)
{
    const float ax = __builtin_fabsf(gx), ay = __builtin_fabsf(gy);
    const int along_x = gx > 0.0f ? TABX_ACT_MOVE_XP : (gx < 0.0f ? TABX_ACT_MOVE_XM : TABX_ACT_NOOP);
    const int along_y = gy > 0.0f ? TABX_ACT_MOVE_YP : TABX_ACT_MOVE_YM;
    return ax >= ay ? along_x : along_y;
}

// What a deciding unit has made out of the units it sees.
struct Sighting {
    int    tgt;            // selected target (unit index in the env) or -1
    float  tgt_d2;         // its squared distance
    bool   tgt_in_box;     // ... and whether the unit's combat action would reach it
    float4 T;              // its x, y, cos(theta), sin(theta)
    float  tr;             // its body radius
    bool   any_enemy;      // nearest visible enemy: exists,
    float  near_d2, near_dx, near_dy;   // squared distance and offset
    bool   can_hit;        // something worth a strike is in the hurtbox
};

// The rule cascade of the policy for one deciding unit (state in U, heading cosine / sine
// cu, su): first rule that applies, then the epsilon-greedy override.  Updates the unit's
// remembered target position and writes the action to out[k].
__device__ __forceinline__ int policy_cascade(const KArgs &a, const Place &P, const Unit &U,
                                              float cu, float su, bool in_bush, const Sighting &S,
                                              uint32_t tick, int remembered, float mx, float my,
                                              const float *zd, uint8_t *out)
{
    const PolicyArgs &pa = a.pa;
    const bool healer = U.dmg < 0.0f;
    const bool assassin = U.speed >= pa.pol.assassin_speed;
    const bool ranger = U.range >= pa.pol.ranger_range;
    int act;
    const uint32_t env_id = (uint32_t)(P.e + a.p.env_id_offset);     // the env's index in the whole batch
    const uint32_t coin = policy_hash(pa.pol.seed, env_id, (uint32_t)P.u, tick, 2u) & 1u;
    const int search_turn = coin ? TABX_ACT_ROT_LEFT : TABX_ACT_ROT_RIGHT;
    if (S.tgt >= 0) {
        const float4 T = S.T;
        pa.mem.mem_x[P.k] = T.x;
        pa.mem.mem_y[P.k] = T.y;
        if (!remembered) pa.mem.mem_valid[P.k] = 1;
        const float tdx = T.x - U.x;
        const float tdy = T.y - U.y;
        const float reach = U.range + S.tr;
        const bool within = S.tgt_d2 <= reach * reach;
        const float kite = pa.pol.xi * U.range;
        // turning towards the side the target is on
        const float lx = (tdx * cu) + (tdy * su);
        const float ly = (tdy * cu) - (tdx * su);
        const int turn = ly > 0.0f ? TABX_ACT_ROT_LEFT
                                   : (ly < 0.0f ? TABX_ACT_ROT_RIGHT
                                                : (lx < 0.0f ? TABX_ACT_ROT_LEFT : TABX_ACT_NOOP));
        // Assassins go behind the target, Healers to it, the rest in front of it
        const float standoff = 0.5f * U.range;
        const float ox = T.z * standoff, oy = T.w * standoff;
        const float gx = healer ? T.x : (assassin ? T.x - ox : T.x + ox);
        const float gy = healer ? T.y : (assassin ? T.y - oy : T.y + oy);
        const int approach = move_along(gx - U.x, gy - U.y);
        const int retreat = move_along(-S.near_dx, -S.near_dy);
        act = (S.can_hit && U.cd <= 0.0f) ? (int)TABX_ACT_ATTACK
              : (within && !S.tgt_in_box) ? turn
              : (ranger && S.any_enemy && S.near_d2 < kite * kite) ? retreat
              : S.tgt_in_box ? (int)TABX_ACT_NOOP            // aligned, waiting for the cooldown
                             : approach;
    } else if (remembered) {
        const float gx = mx - U.x;
        const float gy = my - U.y;
        const bool arrived = (gx * gx) + (gy * gy) <= 1.0f;
        if (arrived) pa.mem.mem_valid[P.k] = 0;
        act = arrived ? search_turn : move_along(gx, gy);
    } else {
        // Rangers outside a bush walk to the nearest bush zone they know of, then search
        // (`zd`: the env's zone descriptors in LDS)
        bool found = false;
        float bush_d2 = 0.0f, bx = 0.0f, by = 0.0f;
        if (ranger && !in_bush) {
            for (int z = 0; z < a.p.max_zones; ++z) {
                const float *d = zd + 6 * z;
                const float zx = d[1] - U.x;
                const float zy = d[2] - U.y;
                const float d2 = (zx * zx) + (zy * zy);
                const bool take = ((int)d[0] == TABX_ZONE_BUSH) && (!found || d2 < bush_d2);
                found = found || take;
                bush_d2 = take ? d2 : bush_d2;
                bx = take ? zx : bx;
                by = take ? zy : by;
            }
        }
        act = found ? move_along(bx, by) : search_turn;
    }
    // epsilon-greedy override
    const uint32_t h0 = policy_hash(pa.pol.seed, env_id, (uint32_t)P.u, tick, 0u);
    const float u0 = (float)(h0 >> 8) * (1.0f / 16777216.0f);
    if (u0 < pa.pol.epsilon)
        act = (int)(policy_hash(pa.pol.seed, env_id, (uint32_t)P.u, tick, 1u) & 7u);
    out[P.k] = (uint8_t)act;
    return act;
}

// What the policy stage reads besides the unit's state and specification; issued with them at the top of
// the kernel, for every unit: whether it decides is known only a round trip later (6v9 x 227, GPU time of
// the heuristic call 8.3 -> 7.8 us).
struct PolicyIn {
    int   told;                    // the policy moves it, if it lives
    int   tick;                    // the env's tick counter
    int   remembered;              // the unit's memory
    float mx, my;
};

__device__ __forceinline__ void load_policy(const KArgs &a, const Place &P, PolicyIn &in)
{
    // (no branch: the loads of one block leave together)
    const uint8_t *const controlled = a.pa.controlled;
    const int byte = at32(controlled ? controlled : a.st.alive, P.k);
    in.told = controlled ? byte : 1;
    in.tick = at32(a.st.t, (size_t)P.e);
    in.remembered = at32(a.pa.mem.mem_valid, P.k);
    in.mx = at32(a.pa.mem.mem_x, P.k);
    in.my = at32(a.pa.mem.mem_y, P.k);
}

// Marks the partners first ... first + count - 1 (at most 32) of an env, records from `base` on, that the unit
// at (x, y), heading (cu, su), may see: bit b for partner first + b.  A mark costs eleven instructions, a root
// and two products less than the test itself, and few partners are in sight (64 x 64 arena, one in fifteen).
// `bound` is taken wide enough (see policy_env) that a pair left out fails the test.
template <class Sh>
__device__ __forceinline__ uint32_t mark_near(const Sh &sh, int base, int first, int count, float x, float y,
                                              float cu, float su, float2 bound)
{
    const float4 *pose = sh.po.pose + base + first;
    uint32_t bits = 0;
#pragma unroll 4
    for (int b = 0; b < count; ++b) {
        const float dx = pose[b].x - x;
        const float dy = pose[b].y - y;
        const float d2 = __builtin_fmaf(dy, dy, dx * dx);
        const float dot = __builtin_fmaf(dy, su, dx * cu);
        const bool far = d2 > bound.x;
        const bool behind = dot * __builtin_fabsf(dot) < __builtin_fmaf(bound.y, d2, -1e-30f);
        bits = bits + bits + ((far | behind) ? 0u : 1u);
    }
    return count > 0 ? __builtin_bitreverse32(bits) >> (32 - count) : 0u;
}

// Decides for the lane's unit from the state in U (heading cosine / sine cu, su, zone code
// code_u under it); returns the action, or -1 if the unit is not the policy's to move.  Writes
// the action and the remembered target position.  All lanes of the workgroup call it.
template <int WAVES, class Sh>
__device__ __forceinline__ int policy_env(const KArgs &a, Sh &sh, const Place &P,
                                          const Unit &U, const PolicyIn &in, int code_u, float cu,
                                          float su, const float *zd)
{
    const int N = a.p.num_units;
    const bool in_bush = (code_u & 3) == TABX_ZONE_BUSH;
    const int my_key = in_bush ? (code_u & 0xff) : 0x100;          // 0x100 matches no cell code
    const bool concealable = in_bush && !(U.reveal > 0.0f);
    sh.po.pose[P.l] = make_float4(U.x, U.y, cu, su);
    sh.po.body[P.l] = make_float4(U.radius, U.hmax, U.hp, 0.0f);
    sh.po.seer[P.l] = U.alive | (U.team << 1) | (concealable ? 4 : 0) | (my_key << 8);
    const bool decide = U.enabled && U.alive && in.told;
    // What mark_near compares with.  A pair is seen if d2 <= sight^2 and dot >= c sqrt(d2), each product and sum
    // rounded.  Marks round otherwise, by a few 2^-24 of sqrt(d2) in dot and of d2; c less 2^-18 leaves eight times
    // that, and with z |z| growing in z the root needs no taking: dot |dot| >= c' |c'| d2.  What underflows is
    // below 1e-30, and comparisons that meet a NaN mark.
    const float cone = U.cos_half - 0x1p-18f;
    const float sight2 = U.sight_range * U.sight_range;
    const bool unit_heading = __builtin_fabsf(cu) + __builtin_fabsf(su) < 4.0f;      // (or theta is no heading)
    const float2 bound = make_float2(__builtin_fmaf(sight2, 1.0f + 0x1p-20f, 1e-30f),
                                     unit_heading ? cone * __builtin_fabsf(cone) : -__builtin_inff());

    // Which lane marks for whom.  Usually half of the units decide (the adversaries), so as many lanes
    // as there are to spare, `parts` in all, share the partners of each deciding unit, a run of them each.  Two
    // wavefronts (N > 64): every lane marks for its own unit.  (Heuristic call, adversaries, testing every pair and
    // marking first: 10v10 x 16384 18.4 and 14.9 us, 32v32 x 1536 15.9 and 9.7, 64v64 x 1024 42.7 and 17.2.)
    int parts = 1, rank = 0;
    if (WAVES == 1) {
        const uint64_t deciding = lanes_where(decide);
        const int count = __popcll(deciding);
        rank = __popcll(deciding & ((1ull << P.l) - 1ull));
        if (count > 0) {
            // 64 / count, eight at most
            parts = 1 + (count <= 32) + (count <= 21) + (count <= 16) + (count <= 12) + (count <= 10) + (count <= 9) +
                    (count <= 8);
            while (parts * parts > 2 * N) --parts;
        }
        if (parts > 1) {
            sh.po.bound[P.l] = bound;
            if (decide) sh.po.who[rank] = P.l | (P.base << 8);
        }
    }
    // the living units of the lane's env but the lane's own
    uint64_t others[WAVES];
    {
        const uint64_t b = lanes_where(U.alive);
        if (WAVES == 1) others[0] = (b >> P.base) & (N >= 64 ? ~0ull : (1ull << N) - 1ull);
        else if ((P.l & 63) == 0) sh.ballots[P.l >> 6][0] = b;
    }
    group_barrier<WAVES>(sh);
    if (WAVES == 2) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) others[w] = sh.ballots[w][0];
    }
    uint64_t near[WAVES];
    if (WAVES == 1 && parts > 1) {
        // (quotients of integers below 128 by one of at most eight: half a step keeps them off the borders)
        const float per = __builtin_amdgcn_rcpf((float)parts);
        const int span = (int)(((float)(N + parts) - 0.5f) * per);                 // N / parts, rounded up: at most 32
        const int mine = (int)(((float)P.l + 0.5f) * per), part = P.l - mul24(mine, parts);
        const int w = sh.po.who[mine < 64 ? mine : 0];
        const int me = w & 63, base = (w >> 8) & 63;               // (lanes to spare: whatever stands there)
        const float4 O = sh.po.pose[me];
        const int first = mul24(part, span), left = N - first;
        const uint32_t bits = mark_near(sh, base, first, left < span ? left : span, O.x, O.y, O.z, O.w, sh.po.bound[me]);
        near[0] = 0ull;
        for (int p = 0; p < parts; ++p)
            near[0] |= (uint64_t)(uint32_t)__shfl((int)bits, mul24(rank, parts) + p) << mul24(p, span);
    } else {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            uint32_t half[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int first = 64 * w + 32 * h, left = N - first;
                half[h] = mark_near(sh, P.base, first, left < 32 ? left : 32, U.x, U.y, cu, su, bound);
            }
            near[w] = ((uint64_t)half[1] << 32) | half[0];
        }
    }

    // The target by role (Healer: injured allies first, then nearest; Assassin: lowest maximum health, then
    // nearest; others: nearest enemy; the lower index on ties), the nearest visible enemy, and whether anything
    // worth a strike is in the hurtbox: the marked units in ascending index.
    const bool healer = U.dmg < 0.0f;
    const bool assassin = U.speed >= a.pa.pol.assassin_speed;
    int tgt = -1, nearest = -1;
    bool can_hit = false, tgt_in_box = false;
    float tgt_d2 = 0.0f, tgt_key = 0.0f, near_d2 = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        uint64_t m = decide ? near[w] & others[w] : 0ull;
        if (P.u >= 64 * w && P.u < 64 * w + 64) m &= ~(1ull << (P.u & 63));
        while (m != 0ull) {
            const int j = 64 * w + __builtin_ctzll(m);
            m &= m - 1ull;
            const int fj = sh.po.seer[P.base + j];
            const float4 A = sh.po.pose[P.base + j];
            const float4 B = sh.po.body[P.base + j];
            const float dx = A.x - U.x;
            const float dy = A.y - U.y;
            float dot;
            const float g2 = hurtbox_gap2(dx, dy, cu, su, U.range, U.hurt_hw, -U.hurt_hw, dot);
            const float d2 = (dx * dx) + (dy * dy);
            const bool in_cone = (d2 == 0.0f) | (dot >= U.cos_half * __builtin_sqrtf(d2));
            const bool same_team = ((fj >> 1) & 1) == U.team;
            const bool same_bush = (fj >> 8) == my_key;
            const bool concealed = (fj & 4) && !same_team && !same_bush;
            const bool seen = (d2 <= sight2) & in_cone & !concealed;
            // (a seen unit is inside the cone, so a cone-bounded hurtbox needs no further test)
            const bool candidate = seen & (healer == same_team);
            const bool attackable = candidate & (g2 <= B.x * B.x);
            const bool injured = B.z < B.y;
            can_hit = can_hit | (attackable & (!healer | injured));
            const bool nearer = seen & !same_team & ((nearest < 0) | (d2 < near_d2));
            nearest = nearer ? j : nearest;
            near_d2 = nearer ? d2 : near_d2;
            const float key = healer ? (injured ? 0.0f : 1.0f) : (assassin ? +B.y : 0.0f);
            const bool better = candidate & ((tgt < 0) | (key < tgt_key) | ((key == tgt_key) & (d2 < tgt_d2)));
            tgt = better ? j : tgt;
            tgt_d2 = better ? d2 : tgt_d2;
            tgt_key = better ? key : tgt_key;
            tgt_in_box = better ? attackable : tgt_in_box;
        }
    }

    int act = -1;
    if (decide) {
        Sighting S;
        S.tgt = tgt;
        S.tgt_d2 = tgt_d2;
        S.tgt_in_box = tgt_in_box;
        S.T = sh.po.pose[P.base + (tgt >= 0 ? tgt : 0)];
        S.tr = sh.po.body[P.base + (tgt >= 0 ? tgt : 0)].x;
        S.any_enemy = nearest >= 0;
        S.near_d2 = near_d2;
        const float4 E = sh.po.pose[P.base + (nearest >= 0 ? nearest : 0)];
        S.near_dx = E.x - U.x;
        S.near_dy = E.y - U.y;
        S.can_hit = can_hit;
        act = policy_cascade(a, P, U, cu, su, in_bush, S, (uint32_t)in.tick, in.remembered, in.mx, in.my, zd,
                             a.pa.actions_out);
    }
    group_barrier<WAVES>(sh);          // the records may be overwritten by the next stage
    return act;
}

} // namespace tabx
