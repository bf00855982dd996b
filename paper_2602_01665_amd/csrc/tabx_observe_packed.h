// Observe stage of the TABX tick with the units in registers: the wavefronts that hold the units of an
// env group also write all of its rows.
#pragma once
#include "tabx_device.h"
#include "tabx_observe.h"

#pragma clang fp contract(off)

namespace tabx {

// Lane l keeps unit l % N of env slot l / N for the whole launch, and pass i writes the rows of observer
// i of all G envs (64 < N: two wavefronts hold the one env and make every row together).  Compared with
// the tiles of tabx_observe.h nothing but the observer is read from LDS per pass, at the price of G
// short runs per flush and of an address register per store pass; where further wavefronts share a
// group the tiles win (no copy of the units per wavefront).  Measured, same box, here / with tiles:
// 10v10 x 16384 stand-alone observe 94.7 / 97.0 us, 5v5 x 65536 fused tick 84.9 / 87.6 us, 64v64 x 768
// fused tick 153 / 169 us (but 64v64 x 512 150 / 115 us with four wavefronts).  Envs of one wavefront: rows
// of whole 16-byte chunks only.
//
// Zone slots of the rows: lane (env slot zg, 16-byte chunk zc of the zone part) keeps its four zone
// floats in registers for the whole launch: the value (zero if the slot is inactive) and which
// observer coordinate to subtract (centre x / y of an active slot).
struct ZoneRegs {
    bool  lane;
    int   zg, zc;
    float val[4];
    int   sx[4], sy[4];
};

// Issued at the top of the kernel so that the descriptor loads are long done when the observe stage
// needs them.
__device__ __forceinline__ ZoneRegs load_zone_regs(const KArgs &a, const Place &P, int row_override = -1)
{
    ZoneRegs Z = {};
    const int zlen = 6 * a.p.max_zones;
    const int ZC = a.zone_chunks;
    Z.zg = ZC > 0 ? P.l / ZC : 0;
    Z.zc = P.l - Z.zg * ZC;
    Z.lane = ZC > 0 && Z.zg < envs_of_group(a, P.grp);
    if (Z.lane) {
        const int row = row_override >= 0 ? row_override : row_of(a, P.grp * a.envs_per_block + Z.zg);
        const float *d = a.sc.zone_desc + (size_t)row * zlen;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int zz = 4 * Z.zc + k;
            if (zz < zlen) {
                const int comp = zz % 6;
                const bool active = d[zz - comp] != 0.0f;
                Z.val[k] = active ? d[zz] : 0.0f;
                Z.sx[k] = (active && comp == 1) ? -1 : 0;
                Z.sy[k] = (active && comp == 2) ? -1 : 0;
            }
        }
    }
    return Z;
}

// DECIDING: a launch with a policy.  EVEN: see plan_shape (tabx_kernels.hip), at most three wavefronts per SIMD.
// `stg`: the staging area, G * R rows (WAVES == 2: two alternating areas of one row); `C`: what the step
// stage left (heading, health ratio); `told`: the policy moves the unit (SCRIPT, see tabx_observe.h).
template <int WAVES, bool SCRIPT, bool DECIDING, bool EVEN, class Sh>
__device__ __forceinline__ void observe_packed(const KArgs &a, Sh &sh, float *stg, const Place &P,
                                               const Unit &U, int code_u, const Carry &C,
                                               const ZoneRegs &Zr, int told,
                                               ScriptLds<WAVES> *script, const float *zd)
{
    typedef float v4 __attribute__((ext_vector_type(4)));
    const int N = a.p.num_units;
    const int G = a.envs_per_block;
    const int D = a.obs_dim;                     // (WAVES == 1: a multiple of 4)
    const int CPR = D >> 2;                      // whole 16-byte chunks per row
    // whether a row may end on half a chunk besides (the plain launches have it in the EVEN kernels only)
    constexpr bool HALF_CHUNK = WAVES == 2 && (EVEN || DECIDING);
    const int zlen = 6 * a.p.max_zones;
    const bool has = P.has;
    const bool want_vis = late_args()->vis_mask != nullptr;
    const int envs_here = envs_of_group(a, P.grp);
    const int lane = P.l & 63;
    const int wv = P.l >> 6;
    v4 *const stage = reinterpret_cast<v4 *>(stg);
    const bool blocks_aligned = (D & 15) == 0;   // every block is then one aligned 64-byte group

    lds_barrier<WAVES>();                        // the step stage is done with the LDS union

    // ---- publish this unit as an observer
    const float cu = C.cu, su = C.su, ratio = C.ratio;
    const int alive = has ? U.alive : 0;
    const bool enabled = has && U.enabled;
    const bool in_bush = (code_u & 3) == TABX_ZONE_BUSH;
    const int my_code = code_u & 0xff;
    const bool hidden = in_bush && !(U.reveal > 0.0f);
    const float cd_ratio = U.cooldown != 0.0f ? U.cd / U.cooldown : 0.0f;
    const float r2_me = U.radius * U.radius;
    const bool decides = SCRIPT && enabled && alive && told;
    {
        const int key = in_bush ? my_code : 0x100;         // 0x100 matches no cell code
        sh.ob.pose[P.l] = make_float4(U.x, U.y, cu, su);
        sh.ob.reach[P.l] = make_float4(U.range, U.hurt_hw, U.sight_range * U.sight_range, U.cos_half);
        int role = 0;
        if (SCRIPT) {
            role = (U.speed >= late_args()->pa.pol.assassin_speed ? 16 : 0) | (decides ? 32 : 0);
            script->tkey[P.l] = ~0ull;
            script->nkey[P.l] = ~0ull;
            script->canhit[P.l] = 0;
            script->hmax[P.l] = has ? U.hmax : 0.0f;
            script->order[P.l] = __float_as_int(U.radius);
        }
        sh.ob.seer[P.l] = alive | (U.team << 1) | (U.dmg < 0.0f ? 4 : 0) | (enabled ? 8 : 0) | role | (key << 8);
        uint8_t *const action_mask = late_args()->action_mask;
        if (has && action_mask && P.chunk == 0)
            action_mask[P.k] = (alive && U.cd <= 0.0f) ? 1 : 0;
    }
    // what differs between a unit's block in its own row and in another unit's row
    const int own_mask = enabled ? -1 : 0;
    const float own_alive = alive ? 1.0f : 0.0f;
    const float own_zone = (float)(code_u & 3);
    const float own_team = (float)U.team;
    float *const global_state = late_args()->st.global_state;
    if (global_state && P.chunk == 0) {
        // the own block with its absolute position is the unit's block of the global state, the zone slots
        // with absolute centres are its tail
        if (has) {
            f4u *gs = reinterpret_cast<f4u *>(global_state + (size_t)P.e * D + 16 * P.u);
            auto masked = [own_mask](float v) { return __int_as_float(__float_as_int(v) & own_mask); };
            gs[0] = f4u{masked(U.hp), masked(ratio), masked(U.x), masked(U.y)};
            gs[1] = f4u{masked(U.theta), masked(U.range), masked(U.dmg), masked(U.cd)};
            gs[2] = f4u{masked(cd_ratio), masked(U.radius), masked(U.mass), masked(U.sight_angle)};
            gs[3] = f4u{masked(own_alive), masked(U.cur_speed), masked(own_zone), masked(own_team)};
        }
        if (Zr.lane) {
            float *gz = global_state + (size_t)(P.grp * G + Zr.zg) * D + 16 * N + 4 * Zr.zc;
            if (!HALF_CHUNK || zlen - 4 * Zr.zc >= 4) {
                *reinterpret_cast<f4u *>(gz) = f4u{Zr.val[0], Zr.val[1], Zr.val[2], Zr.val[3]};
            } else {
                gz[0] = Zr.val[0];
                gz[1] = Zr.val[1];
            }
        }
    }

    const int zg = Zr.zg, zc = Zr.zc;
    const int zone_seer0 = WAVES == 1 ? zg * N : 0;        // lane of observer 0 of the zone lane's env
    const bool cone_free = a.p.hurtbox_cone == 0;          // the hurtbox is the plain rectangle
    const int R = WAVES == 2 ? 1 : a.rows_per_flush;
    int copy_passes = a.copy_passes;
    const int zone_dst0 = (WAVES == 1 ? zg * R * D : 0) + 16 * N + 4 * zc;

    // ---- store passes: chunk t = 64 p + l of the staged rows -> (env slot, chunk in its R rows)
    constexpr int PASSES = WAVES == 2 ? kMaxHalfPasses : kMaxPasses;
    unsigned dst_off[PASSES];
    bool valid[PASSES];
    // (WAVES == 2: each wavefront streams one contiguous half of the row, both whole 64-byte groups)
    const int half_row = ((CPR >> 1) + 3) & ~3;
    const int row_chunks = ((HALF_CHUNK ? (D + 3) >> 2 : CPR) + 3) & ~3;   // pitch of the two alternating row areas
    // the PHYSICAL chunk the lane reads in pass 0; it holds logical chunk staged_chunk(first_chunk)
    const int first_chunk = WAVES == 2 ? wv * half_row + lane : P.l;
    if (WAVES == 2) {
        const int end = wv == 0 ? half_row : row_chunks;
        int phys = first_chunk;
        int q = staged_chunk(first_chunk);
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            valid[p] = phys < end && q < CPR && envs_here > 0;
            dst_off[p] = (unsigned)(4 * q);
            q += 64;
            phys += 64;
        }
    } else {
        const int RC = R * CPR;                  // chunks per env slot and flush
        int tg = 0;                              // env slot of chunk t
        int q = staged_chunk(P.l);               // chunk within the env's R staged rows
        while (q >= RC) {                        // (RC >= 64 for all but tiny rows)
            q -= RC;
            tg += 1;
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            // (a pass beyond copy_passes holds only chunks of env slots >= G >= envs_here)
            valid[p] = tg < envs_here;
            dst_off[p] = (unsigned)(tg * N * D + 4 * q);
            q += 64;                             // chunk t + 64 of the next pass
            if (RC >= 64) {                      // at most one env slot further
                const bool next_slot = q >= RC;
                q = next_slot ? q - RC : q;
                tg = next_slot ? tg + 1 : tg;
            } else {
                while (q >= RC) {
                    q -= RC;
                    tg += 1;
                }
            }
        }
    }

    lds_barrier<WAVES>();

    // scripted deciders: what this unit contributes to a bid, whoever the observer is
    bool injured_me = false;
    unsigned rank_me = 0;          // how many units of the env have a smaller maximum health
    if (SCRIPT) {
        injured_me = U.hp < U.hmax;
        for (int jj = 0; jj < N; ++jj) rank_me += script->hmax[P.base + jj] < U.hmax ? 1u : 0u;
    }

    // ---- one pass per observer index i: every lane's unit seen from observer i of its env
    float *out = a.obs + (size_t)P.grp * G * N * D;
    uint64_t my_row = 0;
    const int blk_row0 = WAVES == 1 ? P.g * R * D : 0;
    // the observers this workgroup writes the rows of: all of them, or its share when the rows
    // of an env group are spread over several short-lived workgroups
    const int i_begin = P.chunk * a.obs_per_chunk;
    const int i_end = (i_begin + a.obs_per_chunk < N) ? i_begin + a.obs_per_chunk : N;
    TABX_STAMP(2);
    const unsigned pace = a.pace;
    const unsigned first_row = pace_start(pace);
    unsigned due = 0;
    float4 A = sh.ob.pose[0], B = sh.ob.reach[0];        // the observer
    int fi = sh.ob.seer[0];
    for (int i0 = i_begin; i0 < i_end; i0 += R) {
        // (no faster than HBM takes all workgroups' rows together: plan_pace, tabx_kernels.hip)
        pace_wait(first_row, due >> 4);
        due += pace;
        v4 *const area = stage + (WAVES == 1 ? 0 : (i0 & 1) * row_chunks);
        for (int rr = 0; rr < R; ++rr) {
            const int i = i0 + rr;
            const int oi = P.base + i;
            if (WAVES == 1) {
                A = sh.ob.pose[oi];
                B = sh.ob.reach[oi];
                fi = sh.ob.seer[oi];
            }
            const int buf = rr * D;
            // offset of this unit from the observer; `dot` is its component along the heading
            const float dx = U.x - A.x;
            const float dy = U.y - A.y;
            float dot;
            const float g2 = hurtbox_gap2(dx, dy, A.z, A.w, B.x, B.y, -B.y, dot);
            const float d2 = (dx * dx) + (dy * dy);
            const bool in_range = d2 <= B.z;
            const bool in_cone = (d2 == 0.0f) || (dot >= B.w * __builtin_sqrtf(d2));
            const bool same_team = ((fi >> 1) & 1) == U.team;
            const bool same_bush = (fi >> 8) == my_code;
            const bool concealed = hidden && !same_team && !same_bush;
            const bool self = i == P.u;
            const bool pair = alive && (fi & 1) && !self;
            const bool seen = pair && in_range && in_cone && !concealed;
            const bool hit = pair && ((((fi >> 2) & 1) != 0) == same_team) && (g2 <= r2_me) &&
                             (in_cone || cone_free);
            if (SCRIPT) {
                // observer i decides its next action: this unit bids if i sees it (nothing to do
                // in a pass whose observers decide nothing or see nobody)
                const bool vis = seen && (fi & 32);
                if (__ballot(vis) != 0ull) {
                    const bool i_heals = (fi & 4) != 0;
                    const unsigned d2b = (unsigned)__float_as_int(d2);
                    if (vis && hit && (!i_heals || injured_me)) atomicOr(&script->canhit[oi], 1);
                    if (vis && !same_team)
                        atomicMin(&script->nkey[oi], ((unsigned long long)d2b << 32) | (unsigned)P.u);
                    if (vis && (i_heals == same_team)) {
                        // Healer: injured allies first; Assassin: lowest maximum health first
                        const unsigned order = i_heals ? (injured_me ? 0u : 1u) : ((fi & 16) ? rank_me : 0u);
                        const unsigned hi = (order << 8) | (d2b >> 24);
                        const unsigned lo = (d2b << 8) | ((unsigned)P.u << 1) | (hit ? 1u : 0u);
                        atomicMin(&script->tkey[oi], ((unsigned long long)hi << 32) | lo);
                    }
                }
            }
            if (want_vis) {
                // the ballot over the lanes is observer i's row: its own lane keeps it (WAVES == 2:
                // one word per wavefront, lane i % 64 keeps it and 64 rows go out together)
                const uint64_t b = __ballot(seen);
                my_row = (WAVES == 1 ? self : lane == (i & 63)) ? b : my_row;
                if (WAVES == 2 && ((i & 63) == 63 || i + 1 == N)) {
                    const int row = (i & ~63) + lane;
                    if (row <= i && envs_here > 0)         // (N > 64: two words)
                        late_args()->vis_mask[2 * ((size_t)P.grp * N + row) + wv] = my_row;
                }
            }
            if (has) {
                // block position in the row: own block first, then the others in index order
                const int blk = self ? 0 : (P.u < i ? P.u + 1 : P.u);
                const int m = self ? own_mask : (seen ? -1 : 0);
                auto masked = [m](float v) { return __int_as_float(__float_as_int(v) & m); };
                // (128-bit vector values: as four-member structs the last chunk has been seen to go
                // out as four separate dwords, each a many-way bank conflict)
                const v4 w0 = {masked(U.hp), masked(ratio), masked(self ? U.x : dx), masked(self ? U.y : dy)};
                const v4 w1 = {masked(U.theta), masked(U.range), masked(U.dmg), masked(U.cd)};
                const v4 w2 = {masked(cd_ratio), masked(U.radius), masked(U.mass), masked(U.sight_angle)};
                const v4 w3 = {masked(self ? own_alive : 1.0f),
                               masked(self ? U.cur_speed : (same_team ? 1.0f : 0.0f)),
                               masked(self ? own_zone : (hit ? 1.0f : 0.0f)),
                               masked(self ? own_team : U.cur_speed)};
                const int cb = (buf + blk_row0 + 16 * blk) >> 2;       // first 16-byte chunk of the block
                if (blocks_aligned) {
                    // (cb is a multiple of 4: the block's chunks are permuted among themselves)
                    v4 *d = area + cb;
                    const int sw = (cb >> 3) & 3;
                    d[sw] = w0;
                    d[1 ^ sw] = w1;
                    d[2 ^ sw] = w2;
                    d[3 ^ sw] = w3;
                } else {
                    area[staged_chunk(cb)] = w0;
                    area[staged_chunk(cb + 1)] = w1;
                    area[staged_chunk(cb + 2)] = w2;
                    area[staged_chunk(cb + 3)] = w3;
                }
            }
            if (Zr.lane) {
                const float4 O = WAVES == 2 ? A : sh.ob.pose[zone_seer0 + i];
                const int en = ((WAVES == 2 ? fi : sh.ob.seer[zone_seer0 + i]) & 8) ? -1 : 0;
                const int xb = __float_as_int(O.x), yb = __float_as_int(O.y);
                float zo[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float shift = __int_as_float((xb & Zr.sx[k]) | (yb & Zr.sy[k]));
                    zo[k] = __int_as_float(__float_as_int(Zr.val[k] - shift) & en);
                }
                area[staged_chunk((buf + zone_dst0) >> 2)] = v4{zo[0], zo[1], zo[2], zo[3]};
            }
        }
        if (WAVES == 2) {
            // the next observer, on its way while the row goes out
            const int next = i0 + 1 < N ? i0 + 1 : i0;
            A = sh.ob.pose[next];
            B = sh.ob.reach[next];
            fi = sh.ob.seer[next];
        }
        lds_barrier<WAVES>();

        // stream the finished rows: LDS chunk -> one 16-byte store, row order, 1 KB per instruction
        float *row = out + i0 * D;
        // the lane reads physical chunk first_chunk + 64 p in pass p: whole runs, in lane order; all
        // passes are fetched from LDS first, then the stores are issued
        const v4 *src = area + first_chunk;
        // (counted anew: as ten answers kept from row to row they take twenty scalar registers)
        asm volatile("" : "+s"(copy_passes));
        v4 v[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (p < copy_passes) v[p] = src[p * 64];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            int store = valid[p] ? 1 : 0;
            // (made opaque, the masks stay in vector registers and the stores of a row are tested one by
            // one: 33v33 x 1500 98 -> 93 us; with fewer envs per CU it costs, x 1000 77 -> 83)
            if (EVEN) asm volatile("" : "+v"(store));
            if (p < copy_passes && store) {
                // (single-wavefront rows go out non-temporal: they are never read back by the kernel, and
                // the hint measurably raises the store rate there; it lowers it for 8 KB rows)
                f4u o = v[p];
                f4u *dp = reinterpret_cast<f4u *>(row + dst_off[p]);
                if (WAVES == 1) __builtin_nontemporal_store(o, dp);
                else *dp = o;
            }
        }
        if (HALF_CHUNK && (D & 3) != 0 && P.l == 64 && envs_here > 0) {
            const v4 t = area[staged_chunk(D >> 2)];
            *reinterpret_cast<f2u *>(row + (D & ~3)) = f2u{t.x, t.y};
        }
        if (WAVES == 1) lds_barrier<1>();        // (two wavefronts alternate between two areas)
        // Two-wavefront envs (a full machine of workgroups that live as long as the launch): the wavefront
        // lets its row stores land before it goes on.  Without this the XCDs drain at different
        // rates and the launch lasts as long as the slowest (64v64 x 1024: 217 us against 208).
        if (WAVES == 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }

    TABX_STAMP(4);
    if (want_vis && WAVES == 1) {
        uint64_t *const vis_mask = late_args()->vis_mask;
        if (has && P.u >= i_begin && P.u < i_end) {
            const uint64_t range = N >= 64 ? ~0ull : ((1ull << N) - 1ull);
            vis_mask[P.k] = (my_row >> P.base) & range;
        }
    }

    if (SCRIPT) {
        lds_barrier<WAVES>();                    // all bids are in
        if (decides) {
            auto T = [&](int l) { return sh.ob.pose[P.base + l]; };
            decide_unit(a, P, U, cu, su, in_bush, script->tkey[P.l], script->nkey[P.l], script->canhit[P.l] != 0,
                        T, [&](int l) { return __int_as_float(script->order[P.base + l]); }, C, zd);
        }
    }
}

} // namespace tabx
