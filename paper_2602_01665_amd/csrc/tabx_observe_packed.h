// Observe stage of the TABX tick with the units in registers: one wavefront per env group.
#pragma once
#include "tabx_device.h"
#include "tabx_observe.h"

#pragma clang fp contract(off)

namespace tabx {

// The form of the observe stage for a wavefront that does all the rows of its group (or, stand-alone,
// every third of them) and already holds the units: lane l keeps unit l % N of env slot l / N for the
// whole launch, and pass i writes the rows of observer i of all G envs.  Compared with the tiles of
// tabx_observe.h nothing but the observer is read from LDS per pass, at the price of G short runs per
// flush and of an address register per store pass.  Measured (10v10 x 16384 stand-alone observe, 5v5 x
// 65536 fused tick, same box): 94.7 and 84.9 us here, 97.0 and 87.6 us with tiles; where several
// wavefronts share a group the tiles win (they need no copy of the units per wavefront).  Rows of
// whole 16-byte chunks only.
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

// `stg`: the staging area, G * R rows; `C`: what the step stage left (heading, health ratio).
__device__ __forceinline__ void observe_packed(const KArgs &a, Shared<1, false> &sh, float *stg,
                                               const Place &P, const Unit &U, int code_u,
                                               const Carry &C, const ZoneRegs &Zr)
{
    typedef float v4 __attribute__((ext_vector_type(4)));
    const int N = a.p.num_units;
    const int G = a.envs_per_block;
    const int D = a.obs_dim;                     // a multiple of 4
    const int CPR = D >> 2;                      // 16-byte chunks per row
    const int zlen = 6 * a.p.max_zones;
    const bool has = P.has;
    const bool want_vis = late_args()->vis_mask != nullptr;
    const bool want_gs = late_args()->st.global_state != nullptr;
    const int envs_here = envs_of_group(a, P.grp);
    v4 *const stage = reinterpret_cast<v4 *>(stg);
    const bool blocks_aligned = (D & 15) == 0;   // every block is then one aligned 64-byte group

    lds_barrier<1>();                            // the step stage is done with the LDS union

    // ---- publish this unit as an observer
    const float cu = C.cu, su = C.su, ratio = C.ratio;
    const int alive = has ? U.alive : 0;
    const bool enabled = has && U.enabled;
    const bool in_bush = (code_u & 3) == TABX_ZONE_BUSH;
    const int my_code = code_u & 0xff;
    const bool hidden = in_bush && !(U.reveal > 0.0f);
    const float cd_ratio = U.cooldown != 0.0f ? U.cd / U.cooldown : 0.0f;
    const float r2_me = U.radius * U.radius;
    {
        const int key = in_bush ? my_code : 0x100;         // 0x100 matches no cell code
        sh.ob.pose[P.l] = make_float4(U.x, U.y, cu, su);
        sh.ob.reach[P.l] = make_float4(U.range, U.hurt_hw, U.sight_range * U.sight_range, U.cos_half);
        sh.ob.seer[P.l] = alive | (U.team << 1) | (U.dmg < 0.0f ? 4 : 0) | (enabled ? 8 : 0) | (key << 8);
        uint8_t *const action_mask = late_args()->action_mask;
        if (has && action_mask && P.chunk == 0)
            action_mask[P.k] = (alive && U.cd <= 0.0f) ? 1 : 0;
    }
    // what differs between a unit's block in its own row and in another unit's row
    const int own_mask = enabled ? -1 : 0;
    const float own_alive = alive ? 1.0f : 0.0f;
    const float own_zone = (float)(code_u & 3);
    const float own_team = (float)U.team;

    const int zg = Zr.zg, zc = Zr.zc;
    const int zone_seer0 = zg * N;               // lane of observer 0 of the zone lane's env
    const bool cone_free = a.p.hurtbox_cone == 0;          // the hurtbox is the plain rectangle
    const int R = a.rows_per_flush;
    const int zone_dst0 = zg * R * D + 16 * N + 4 * zc;

    // ---- store passes: chunk t = 64 p + l of the staged rows -> (env slot, chunk in its R rows)
    unsigned dst_off[kMaxPasses];
    bool valid[kMaxPasses];
    {
        const int RC = R * CPR;                  // chunks per env slot and flush
        int tg = 0;                              // env slot of chunk t
        int q = staged_chunk(P.l);               // chunk within the env's R staged rows
        while (q >= RC) {                        // (RC >= 64 for all but tiny rows)
            q -= RC;
            tg += 1;
        }
#pragma unroll
        for (int p = 0; p < kMaxPasses; ++p) {
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

    lds_barrier<1>();

    // ---- one pass per observer index i: every lane's unit seen from observer i of its env
    float *out = a.obs + (size_t)P.grp * G * N * D;
    uint64_t my_row = 0;
    const int blk_row0 = P.g * R * D;
    // the observers this workgroup writes the rows of: all of them, or its share when the rows
    // of an env group are spread over several short-lived workgroups
    const int i_begin = P.chunk * a.obs_per_chunk;
    const int i_end = (i_begin + a.obs_per_chunk < N) ? i_begin + a.obs_per_chunk : N;
    for (int i0 = i_begin; i0 < i_end; i0 += R) {
        for (int rr = 0; rr < R; ++rr) {
            const int i = i0 + rr;
            const int oi = P.base + i;
            const float4 A = sh.ob.pose[oi];
            const float4 B = sh.ob.reach[oi];
            const int fi = sh.ob.seer[oi];
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
            if (want_vis) {
                // the ballot over the lanes is observer i's row; its own lane keeps it
                const uint64_t b = __ballot(seen);
                my_row = self ? b : my_row;
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
                if (self && want_gs) {
                    // the own block with its absolute position is the unit's block of the global state
                    f4u *gs = reinterpret_cast<f4u *>(late_args()->st.global_state + (size_t)P.e * D + 16 * P.u);
                    gs[0] = w0;
                    gs[1] = w1;
                    gs[2] = w2;
                    gs[3] = w3;
                }
                const int cb = (buf + blk_row0 + 16 * blk) >> 2;       // first 16-byte chunk of the block
                if (blocks_aligned) {
                    // (cb is a multiple of 4: the block's chunks are permuted among themselves)
                    v4 *d = stage + cb;
                    const int sw = (cb >> 3) & 3;
                    d[sw] = w0;
                    d[1 ^ sw] = w1;
                    d[2 ^ sw] = w2;
                    d[3 ^ sw] = w3;
                } else {
                    stage[staged_chunk(cb)] = w0;
                    stage[staged_chunk(cb + 1)] = w1;
                    stage[staged_chunk(cb + 2)] = w2;
                    stage[staged_chunk(cb + 3)] = w3;
                }
            }
            if (Zr.lane) {
                const float4 O = sh.ob.pose[zone_seer0 + i];
                const int en = (sh.ob.seer[zone_seer0 + i] & 8) ? -1 : 0;
                const int xb = __float_as_int(O.x), yb = __float_as_int(O.y);
                float zo[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float shift = __int_as_float((xb & Zr.sx[k]) | (yb & Zr.sy[k]));
                    zo[k] = __int_as_float(__float_as_int(Zr.val[k] - shift) & en);
                }
                stage[staged_chunk((buf + zone_dst0) >> 2)] = v4{zo[0], zo[1], zo[2], zo[3]};
                if (want_gs && i == 0) {
                    // ... and the zone slots with absolute centres are its tail
                    float *gz = late_args()->st.global_state + (size_t)(P.grp * G + zg) * D + 16 * N + 4 * zc;
                    if (zlen - 4 * zc >= 4)      // (always: the row is whole chunks)
                        *reinterpret_cast<f4u *>(gz) = f4u{Zr.val[0], Zr.val[1], Zr.val[2], Zr.val[3]};
                }
            }
        }
        lds_barrier<1>();

        // stream the finished rows: LDS chunk -> one 16-byte store, row order, 1 KB per instruction
        float *row = out + i0 * D;
        // the lane reads physical chunk l + 64 p in pass p: whole runs, in lane order; all passes are
        // fetched from LDS first, then the stores are issued
        const float4 *src = reinterpret_cast<const float4 *>(stg) + P.l;
        float4 v[kMaxPasses];
#pragma unroll
        for (int p = 0; p < kMaxPasses; ++p)
            if (p < a.copy_passes) v[p] = src[p * 64];
#pragma unroll
        for (int p = 0; p < kMaxPasses; ++p) {
            if (p < a.copy_passes && valid[p]) {
                // (non-temporal: the rows are never read back by the kernel, and the hint measurably
                // raises the store rate)
                f4u o = {v[p].x, v[p].y, v[p].z, v[p].w};
                __builtin_nontemporal_store(o, reinterpret_cast<f4u *>(row + dst_off[p]));
            }
        }
        lds_barrier<1>();
    }

    if (want_vis) {
        uint64_t *const vis_mask = late_args()->vis_mask;
        if (has && P.u >= i_begin && P.u < i_end) {
            const uint64_t range = N >= 64 ? ~0ull : ((1ull << N) - 1ull);
            vis_mask[P.k] = (my_row >> P.base) & range;
        }
    }
}

} // namespace tabx
