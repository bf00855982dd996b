// Observe stage of the TABX tick (App. A "Observation and Global State").
#pragma once
#include "tabx_device.h"
#include "tabx_policy.h"   // the scripted units' rule cascade

#pragma clang fp contract(off)

namespace tabx {

// Observation rows of every unit of the workgroup's envs, visibility masks, action masks.
//
// A row is N blocks of 16 floats (the observer's own block first, then the other units in
// ascending index) followed by the zone slots.  The envs of a workgroup are consecutive, so all
// their rows, in the order (env, observer), are ONE contiguous run of HBM.  It is produced in
// tiles of S = floor(64 / N) consecutive rows: lane l holds unit l % N of the env that row
// l / N of the tile belongs to and tests itself against that row's observer.  What a lane needs
// of its unit and of the observer comes from records that the wavefront which stepped the envs
// has left in LDS, so any wavefront of the workgroup can take any tile and no unit state stays
// in registers from tile to tile.  The rows of a tile (about 4 KB) are assembled in LDS, in the
// wavefront's own staging area, as an exact image of the run and go out in 16-byte chunks.

// LDS of the scripted units that decide their next action inside the observe stage: per
// deciding unit the smallest bids for "target" and "nearest enemy" and the "something to
// strike" flag, per unit what a bidder or a decider needs beyond the observe-stage records.
template <int WAVES>
struct ScriptLds {
    static constexpr int L = 64 * WAVES;
    unsigned long long tkey[L];   // role key << 40 | bits(distance^2) << 8 | index << 1 | in hurtbox
    unsigned long long nkey[L];   // bits(distance^2) << 32 | index
    int                canhit[L];
    int                order[L];  // injured | units of the env with a smaller maximum health << 1
    float              hmax[L];
};

// Leaves the lane's unit in LDS as the observe stage needs it (state in U, heading cosine / sine
// cu, su, zone code code_u; `told`: the policy moves it); also the action mask and the units' part of the global state.
template <int WAVES, bool SCRIPT, class Sh>
__device__ __forceinline__ void publish_units(const KArgs &a, Sh &sh, const Place &P,
                                              const Unit U, int code_u, float ratio, float cu,
                                              float su, int told, ScriptLds<WAVES> *script)
{
    const bool has = P.has;
    const int alive = has ? U.alive : 0;
    const bool enabled = has && U.enabled;
    const bool in_bush = (code_u & 3) == TABX_ZONE_BUSH;
    const int code = code_u & 0xff;
    const float cd_ratio = U.cooldown != 0.0f ? U.cd / U.cooldown : 0.0f;
    int flags = alive | (U.team << 1) | (U.dmg < 0.0f ? 4 : 0) | (enabled ? 8 : 0) |
                (in_bush && !(U.reveal > 0.0f) ? 64 : 0) |
                ((in_bush ? code : 0x100) << 8) |          // 0x100 matches no cell code
                (code << 20);
    if (SCRIPT) {
        const bool decides = enabled && alive && told;
        flags |= (U.speed >= late_args()->pa.pol.assassin_speed ? 16 : 0) | (decides ? 32 : 0);
        script->tkey[P.l] = ~0ull;
        script->nkey[P.l] = ~0ull;
        script->canhit[P.l] = 0;
        script->hmax[P.l] = has ? U.hmax : 0.0f;
    }
    const float4 own[4] = {make_float4(U.hp, ratio, U.x, U.y),
                           make_float4(U.theta, U.range, U.dmg, U.cd),
                           make_float4(cd_ratio, U.radius, U.mass, U.sight_angle),
                           make_float4(alive ? 1.0f : 0.0f, U.cur_speed, (float)(code_u & 3),
                                       (float)U.team)};
#pragma unroll
    for (int k = 0; k < 4; ++k) sh.rec.own[k][P.l] = own[k];
    sh.rec.view[P.l] = make_float4(cu, su, U.sight_range * U.sight_range, U.cos_half);
    sh.rec.mark[P.l] = make_float2(U.hurt_hw, __int_as_float(flags));
    if (has && P.chunk == 0) {
        uint8_t *const action_mask = late_args()->action_mask;
        if (action_mask) action_mask[P.k] = (alive && U.cd <= 0.0f) ? 1 : 0;
        float *const global_state = late_args()->st.global_state;
        if (global_state) {
            // the own block with its absolute position is the unit's block of the global state
            f4u *gs = reinterpret_cast<f4u *>(global_state + (size_t)P.e * a.obs_dim + 16 * P.u);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f4u q = {own[k].x, own[k].y, own[k].z, own[k].w}, none = {};
                gs[k] = enabled ? q : none;
            }
        }
    }
    if (SCRIPT) {
        group_barrier<WAVES>(sh);
        int rank = 0;
        for (int jj = 0; jj < a.p.num_units; ++jj)
            rank += script->hmax[P.base + jj] < U.hmax ? 1 : 0;
        script->order[P.l] = (rank << 1) | (U.hp < U.hmax ? 1 : 0);
    }
}

// The zone slots with absolute centres are the tail of the global state (from the chunks in LDS).
template <int LANES>
__device__ __forceinline__ void global_state_zones(const KArgs &a, const ZoneLds &Z, int grp, int l)
{
    float *const out = late_args()->st.global_state;
    if (!out) return;
    const int zlen = 6 * a.p.max_zones, ZC = a.zone_chunks;
    const int envs_here = envs_of_group(a, grp);
    for (int q = l; q < envs_here * ZC; q += LANES) {
        const int g = quotient(q, a.magic_zc);
        const int zc = q - g * ZC;
        const float4 v = Z.val[q];
        float *d = out + (size_t)(grp * a.envs_per_block + g) * a.obs_dim + 16 * a.p.num_units + 4 * zc;
        const int left = zlen - 4 * zc;
        if (left >= 4) {
            *reinterpret_cast<f4u *>(d) = f4u{v.x, v.y, v.z, v.w};
        } else {                                   // (zlen is even: half a chunk)
            d[0] = v.x;
            d[1] = v.y;
        }
    }
}

// The global state of the workgroup's envs, from the records: every unit's own block, whose position is absolute,
// then the zone slots with absolute centres, past the caches (see plan_global).  An env's part is one run of HBM, a
// lane per 16-byte chunk, by LANES lanes (`l`: index among them): what goes past the caches has to be whole lines
// (from the lanes that hold the units, 64 bytes apart, 10v10 x 16384 116 -> 126 us).
template <int LANES>
__device__ __forceinline__ void stream_global_state(const KArgs &a, const Records<64> &rec, const ZoneLds &Z,
                                                    float *out, int grp, int l)
{
    const int N = a.p.num_units, D = a.obs_dim, ZC = a.zone_chunks, zlen = 6 * a.p.max_zones;
    const int chunks = 4 * N + ZC, all = envs_of_group(a, grp) * chunks;
    // (quotients below 64 of dividends below 2048: half a step keeps them off the borders)
    const float per = __builtin_amdgcn_rcpf((float)chunks);
    out += (size_t)grp * a.envs_per_block * D;
    for (int q = l; q < all; q += LANES) {
        const int g = (int)(((float)q + 0.5f) * per);
        const int c = q - mul24(g, chunks), zc = c - 4 * N;
        const int unit = mul24(g, N) + (zc < 0 ? c >> 2 : 0);
        const float4 v = zc < 0 ? rec.own[0][64 * (c & 3) + unit] : Z.val[mul24(g, ZC) + zc];
        const bool on = zc >= 0 || (__float_as_int(rec.mark[unit].y) & 8);
        const f4u w = {on ? v.x : 0.0f, on ? v.y : 0.0f, on ? v.z : 0.0f, on ? v.w : 0.0f};
        float *const d = out + (mul24(g, D) + 4 * c);
        if (zc < 0 || zlen - 4 * zc >= 4) {
            __builtin_nontemporal_store(w, reinterpret_cast<f4u *>(d));
        } else {                                   // (zlen is even: half a chunk)
            d[0] = w.x;
            d[1] = w.y;
        }
    }
}

// Where 16-byte chunk c of a staged tile lives in LDS: the four chunks of every aligned 64-byte
// group are permuted by the group's index (XOR with bits 3..4 of c).  Measured on gfx950
// (SQ_LDS_BANK_CONFLICT / SQ_LDS_IDX_ACTIVE of one-pattern kernels): a 16-byte write of 64 lanes
// takes 8 cycles when every 8 consecutive lanes hit 8 different 16-byte slots modulo 128 bytes;
// the unit blocks that neighbouring lanes write are 64 bytes apart, which unpermuted puts every
// other lane on the same slot (32 cycles; 16 with one spare chunk per 16; 8 with this
// permutation).  A 16-byte read takes 4 cycles only if lane t reads chunk base + t, 8 as soon as
// a spare chunk interrupts the run and 12 if the lanes of a group read it in permuted order.  So
// the store passes read the physical chunks in lane order and undo the permutation on the way
// out: lane t's chunk goes to the place of logical chunk staged_chunk(t) in HBM, which is in the
// same 64-byte group, so every store instruction still writes whole lines.  The map is its own
// inverse, and staged_chunk(c + 32 k) = staged_chunk(c) + 32 k.
__device__ __forceinline__ int staged_chunk(int c) { return c ^ ((c >> 3) & 3); }

// Writes the rows of the tiles tile, tile + tile_step, ... < tile_end of env group `grp`
// (wavefront-uniform values).  `stg` is the calling wavefront's staging area.
//
// A tile is the business of one wavefront.  WAVES == 1: the records of the next pass are fetched
// before the tile goes out, so that their latency passes behind the stores.
// WAVES == 2 (one env, a tile is one row): the wavefront goes over the units in two halves.
// FOLD: there are no zone slots.
// LINES (KArgs::lines): how the tiles lie in the 128-byte lines of the rows.  A line that is written in two parts,
// by two store instructions or for two tiles, costs HBM far more than its bytes (24v24 with 4 zones x 986: WRITE_SIZE
// 156 MB and 152, write requests under 64 bytes 2.4 % and none, 47 us and 36).  So a tile's image starts at the place within a line
// at which the tile does in memory, every store instruction then writes whole lines, and the line that two tiles of a
// wavefront share goes out with the second one.  With tiles that start on a chunk / on a line / and that hand the
// shared line on: 32v32 with 3 zones x 2000 135 / 123 / 115 us, 20v20 with one x 3000 85 / 80 / 74, 15v15 with 5 x
// 8000 133 / 124 / 113, 27v28 with 4 x 1200 67.5 / 66 / 53, scripted 10v10 with 5 x 16384 123 / 116.5 / 110.  The
// forms are code of their own: what the third one does costs small launches 2 to 4 % (10v11 with one zone x 64 11.4
// and 11.8 us), and the second one's 1 % where no tile needs it (10v10 with 8 x 16384).
//
// UNPACED: a launch that is never paced (stand-alone observe of envs of one wavefront).
//
// SCRIPT: the units the heuristic policy moves decide their next action from the very pair
// tests the observation rows are made of (App. A "Role-Appropriate Heuristic Policy Mechanism":
// a unit acts on what it sees and can reach).  Every unit that a deciding observer sees bids
// with LDS atomic minima for "its target" (key: the role's order, then distance, then index,
// with "in its hurtbox" riding in the lowest bit) and for "its nearest enemy"; afterwards the
// deciding units read their winners (decide_units).
template <int WAVES, bool SCRIPT, bool FOLD, int LINES, bool UNPACED>
__device__ __forceinline__ void write_rows(const KArgs &a, const Records<64 * WAVES> &rec,
                                           const ZoneLds &Z, float *stg, int grp, int tile,
                                           int tile_step, int tile_end, ScriptLds<WAVES> *script)
{
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef float v2 __attribute__((ext_vector_type(2)));
    typedef float v4h __attribute__((ext_vector_type(4), aligned(8)));
    const int N = a.p.num_units;
    const int D = a.obs_dim;
    const int T = a.rows_per_tile, S = a.rows_per_pass;
    const int ZC = a.zone_chunks, zlen = 6 * a.p.max_zones;
    const unsigned magic_n = a.magic_n, magic_tc = a.magic_tc;
    const int passes_per_tile = a.passes_per_tile;
    float *const obs = a.obs;
    const int lane = (int)(threadIdx.x & 63);
    constexpr int HALVES = WAVES;
    const int rows = envs_of_group(a, grp) * N;
    const size_t row0 = (size_t)grp * a.envs_per_block * N;       // the group's first row
    uint64_t *const vis_mask = late_args()->vis_mask;
    const bool whole = LINES == LINES_OWN || (D & 3) == 0;             // rows are whole 16-byte chunks
    const bool grouped = (D & 15) == 0;          // ... and whole 64-byte groups
    // the lane's place in a pass: row slot s, unit u
    const int s = WAVES == 1 ? quotient(lane, magic_n) : 0;
    int u = WAVES == 1 ? lane - s * N : lane;
    const bool holds = s < S && (HALVES == 2 || u < N);
    // the rest of a row, copied chunk by chunk: the own block (four chunks) and the zone slots; without
    // zone slots the observer's own lane puts its block where the others put theirs, which saves the
    // extra trip through LDS
    const int TC = FOLD ? 0 : 4 + ZC;
    const int ts0 = WAVES == 1 ? quotient(lane, magic_tc) : 0;
    int vis_lo = 0, vis_hi = 0;
    uint64_t passes_done = 0;
    const int lane_chunk = whole ? staged_chunk(lane) : lane;

    // what a pass works on: the lane's row f (observer i of the env whose units start at record gN)
    // and what it reads of the observer and of its unit
    int f = 0, i = 0, gN = 0, fi = 0, fu = 0;
    v2 opos = {};
    float4 V = {}, Ub = {}, Ug = {}, Uk = {}, Us = {};
    float orange = 0.0f, ohw = 0.0f;
    auto fetch = [&](int f0, int r0, int rows_here) {
        f = f0 + (r0 + s < rows_here ? r0 + s : 0);
        gN = WAVES == 1 ? mul24(quotient(f, magic_n), N) : 0;
        i = f - gN;
        opos = *reinterpret_cast<const v2 *>(&rec.own[0][f].z);
        V = rec.view[f];
        orange = rec.own[1][f].y;
        const float2 M = rec.mark[f];
        ohw = M.x;
        fi = __float_as_int(M.y);
        const int uk = gN + (u < N ? u : 0);
        Ub = rec.own[0][uk];
        Ug = rec.own[1][uk];
        Uk = rec.own[2][uk];
        Us = rec.own[3][uk];
        fu = __float_as_int(rec.mark[uk].y);
    };
    // the copied part of the rows of a tile, into its staging area
    auto copy_tail = [&](int f0, int rows_here, int pad, float *buf) {
                for (int q = lane, ts = ts0; q < rows_here * TC;
                     q += 64, ts = WAVES == 1 ? quotient(q, magic_tc) : 0) {
                    const int c = q - mul24(ts, TC);
                    const int tf = f0 + ts;
                    const int zc = c - 4;
                    const bool zone = zc >= 0;
                    const int zi = WAVES == 1 ? mul24(quotient(tf, magic_n), ZC) + zc : zc;
                    const float4 v = zone ? Z.val[zi] : rec.own[0][c * (64 * WAVES) + tf];
                    const int rel = zone ? Z.rel[zi] : 0;
                    const v2 pos = *reinterpret_cast<const v2 *>(&rec.own[0][tf].z);
                    const int en = (__float_as_int(rec.mark[tf].y) << 28) >> 31;         // enabled: bit 3
                    const int kind = zc - 3 * third(zc);
                    const float x = __int_as_float(__float_as_int(pos.x) & rel);
                    const float y = __int_as_float(__float_as_int(pos.y) & rel);
                    const float tv[4] = {v.x - (kind == 2 ? y : 0.0f), v.y - (kind == 0 ? x : 0.0f),
                                         v.z - (kind == 0 ? y : 0.0f), v.w - (kind == 1 ? x : 0.0f)};
                    float to[4];
        #pragma unroll
                    for (int k = 0; k < 4; ++k) to[k] = __int_as_float(__float_as_int(tv[k]) & en);
                    const int at = pad + mul24(ts, D) + 4 * c + (zone ? 16 * N - 16 : 0);
                    if (whole) {
                        const v4 w = {to[0], to[1], to[2], to[3]};
                        reinterpret_cast<v4 *>(buf)[staged_chunk(at >> 2)] = w;
                    } else {
                        // (a row ends on half a chunk: its second half belongs to the next row)
                        v2 *d = reinterpret_cast<v2 *>(buf + at);
                        d[0] = v2{to[0], to[1]};
                        if (!zone || 4 * zc + 2 < zlen) d[1] = v2{to[2], to[3]};
                    }
                }
    };
    auto rows_of = [&](int t) { const int left = rows - t * T; return left < T ? left : T; };
    auto pad_of = [&](int t) { return LINES == LINES_OWN ? 0 : (int)(((uint32_t)row0 + (uint32_t)(t * T)) * (uint32_t)D & a.line); };
    if (tile < tile_end && tile * T < rows) {
        fetch(tile * T, 0, rows_of(tile));
    }

    // (stand-alone observe of envs of one wavefront, and tiles of two that share lines, are never paced, and the test
    // for it cost them 1 to 3 %: 15v15 with 5 zones x 8000, observed, 98.7 us, 95.4 without, 32v32 with 7 x 15 8.55 and
    // 8.44, the tick of 50v50 with 2 x 400 67.6 and 65.9)
    constexpr bool PACED = !UNPACED && (WAVES == 1 || LINES != LINES_SHARED);
    const unsigned pace = a.pace;
    const unsigned first_row = PACED ? pace_start(pace) : 0u;
    unsigned due = 0;
    bool carried = false;                        // the head of the tile's first line is there already
    for (; tile < tile_end && tile * T < rows; tile += tile_step) {
        // (a launch that is one generation of workgroups: see plan_pace, tabx_kernels.hip.  Here, with nothing due
        // before the first tile, and not behind a branch after all but the last: small batches 1 to 2 % shorter, 30v29
        // with 12 zones x 79 19.6 us and 19.2)
        if (PACED) pace_wait(first_row, due >> 4);
        due += pace;
        const int f0 = tile * T;                 // the tile's first row within the group
        const int rows_here = rows_of(tile);
        // where the tile starts within a 128-byte line (or a 16-byte chunk: KArgs::line)
        const int pad = pad_of(tile);
        float *const buf = stg;
        v4 *const vstage = reinterpret_cast<v4 *>(buf);
        int pass = tile * passes_per_tile;
        for (int r0 = 0; r0 < rows_here; r0 += S, ++pass) {
#pragma unroll 1
        for (int h = 0; h < HALVES; ++h) {
            if (HALVES == 2 && h) {
                u = lane + 64;
                fetch(f0, r0, rows_here);
            }
            const int sr = r0 + s;               // the lane's row of the tile
            const bool has = holds && sr < rows_here && (HALVES == 1 || u < N);
            // offset of this unit from the observer; `dot` is its component along the heading
            const float dx = Ub.z - opos.x;
            const float dy = Ub.w - opos.y;
            float dot;
            const float g2 = hurtbox_gap2(dx, dy, V.x, V.y, orange, ohw, -ohw, dot);
            const float d2 = (dx * dx) + (dy * dy);
            const bool same_team = ((fi ^ fu) & 2) == 0;
            const bool same_bush = ((fi >> 8) & 0x1ff) == (fu >> 20);
            const bool concealed = (fu & 64) && !same_team && !same_bush;
            const bool self = i == u;
            const bool pair = has && (fi & fu & 1) && !self && d2 <= V.z && !concealed;
            const bool seen = pair && (d2 == 0.0f || dot >= V.w * __builtin_sqrtf(d2));
            // (only ever asked of a unit that is seen, so a cone-bounded hurtbox adds no test)
            const bool hit = (((fi & 4) != 0) == same_team) && (g2 <= Uk.y * Uk.y);
            if (SCRIPT) {
                // the observer decides its next action: this unit bids if it is seen (nothing to
                // do in a pass whose observers decide nothing or see nobody)
                const bool vis = seen && (fi & 32);
                if (__ballot(vis) != 0ull) {
                    const int uk = gN + (u < N ? u : 0);
                    const bool i_heals = (fi & 4) != 0;
                    const unsigned d2b = (unsigned)__float_as_int(d2);
                    const int ord = script->order[uk];
                    const bool injured = (ord & 1) != 0;
                    if (vis && hit && (!i_heals || injured)) atomicOr(&script->canhit[f], 1);
                    if (vis && !same_team)
                        atomicMin(&script->nkey[f], ((unsigned long long)d2b << 32) | (unsigned)u);
                    if (vis && (i_heals == same_team)) {
                        // Healer: injured allies first; Assassin: lowest maximum health first
                        const unsigned order = i_heals ? (injured ? 0u : 1u)
                                                       : ((fi & 16) ? (unsigned)(ord >> 1) : 0u);
                        const unsigned hi = (order << 8) | (d2b >> 24);
                        const unsigned lo = (d2b << 8) | ((unsigned)u << 1) | (hit ? 1u : 0u);
                        atomicMin(&script->tkey[f], ((unsigned long long)hi << 32) | lo);
                    }
                }
            }
            if (vis_mask) {
                // the ballot over the lanes holds the rows of the pass's observers: lane p keeps
                // the ballot of pass p of the group (WAVES == 2: one word of the one row)
                const uint64_t b = __ballot(seen);
                if (HALVES == 2) {
                    if (lane == 0) vis_mask[2 * (row0 + f) + h] = b;
                } else {
                    vis_lo = lane == pass ? (int)(uint32_t)b : vis_lo;
                    vis_hi = lane == pass ? (int)(uint32_t)(b >> 32) : vis_hi;
                    passes_done |= 1ull << pass;
                }
            }
            if (has && (FOLD || !self)) {
                // block position in the row: behind the own block, in index order
                const int at = pad + mul24(sr, D) + 16 * (FOLD && self ? 0 : u < i ? u + 1 : u);
                const int m = seen || (FOLD && self && (fi & 8)) ? -1 : 0;
                auto masked = [m](float v) { return __int_as_float(__float_as_int(v) & m); };
                // (written as 128-bit vector values: as four-member structs the last chunk has been
                // seen to go out as four separate dwords, each a many-way bank conflict)
                v4 w0 = {masked(Ub.x), masked(Ub.y), masked(dx), masked(dy)};
                const v4 w1 = {masked(Ug.x), masked(Ug.y), masked(Ug.z), masked(Ug.w)};
                const v4 w2 = {masked(Uk.x), masked(Uk.y), masked(Uk.z), masked(Uk.w)};
                v4 w3 = {masked(1.0f), seen && same_team ? 1.0f : 0.0f, seen && hit ? 1.0f : 0.0f,
                         masked(Us.y)};
                if (FOLD && self) {
                    w0.z = masked(Ub.z);
                    w0.w = masked(Ub.w);
                    w3 = v4{masked(Us.x), masked(Us.y), masked(Us.z), masked(Us.w)};
                }
                if (grouped) {
                    // (the block is one 64-byte group: its chunks are permuted among themselves)
                    char *const d = reinterpret_cast<char *>(buf);
                    const int at0 = 4 * at | ((at >> 1) & 48);
                    *reinterpret_cast<v4 *>(d + at0) = w0;
                    *reinterpret_cast<v4 *>(d + (at0 ^ 16)) = w1;
                    *reinterpret_cast<v4 *>(d + (at0 ^ 32)) = w2;
                    *reinterpret_cast<v4 *>(d + (at0 ^ 48)) = w3;
                } else if (whole) {
                    const int cb = at >> 2;
                    vstage[staged_chunk(cb)] = w0;
                    vstage[staged_chunk(cb + 1)] = w1;
                    vstage[staged_chunk(cb + 2)] = w2;
                    vstage[staged_chunk(cb + 3)] = w3;
                } else {
                    // (8-byte aligned: two 8-byte halves per instruction)
                    v4h *d = reinterpret_cast<v4h *>(buf + at);
                    d[0] = w0;
                    d[1] = w1;
                    d[2] = w2;
                    d[3] = w3;
                }
            }
            if (HALVES == 1 && r0 + S < rows_here) fetch(f0, r0 + S, rows_here);
        }
        }
        if (HALVES == 2) u = lane;
        copy_tail(f0, rows_here, pad, buf);
        {
            const int next = tile + tile_step;
            if (next < tile_end && next * T < rows) fetch(next * T, 0, rows_of(next));
        }
        lds_barrier<1>();

        // stream the finished rows: LDS chunk -> one 16-byte store, 1 KB per instruction
        float *const out = obs + (row0 + f0) * D - pad;
        const int floats = pad + rows_here * D;
        // LINES_CARRIED: a line that two tiles share goes out with the second one, if both are this wavefront's
        // (whose tiles are neighbours: plan_shape).
        const bool carry = LINES == LINES_CARRIED && tile + 1 < tile_end && (tile + 1) * T < rows && floats >= 32;
        const int chunks = carry ? (floats & ~31) >> 2 : floats >> 2;
        const int first = carried ? 0 : (pad + 3) >> 2;        // the first chunk that is the tile's alone
        const float4 *src = reinterpret_cast<const float4 *>(buf) + lane;
        char *dst = reinterpret_cast<char *>(out);
        for (int left = chunks, skip = first; left > 0; left -= 64 * kPassBatch, skip = 0) {
            float4 v[kPassBatch];
#pragma unroll
            for (int p = 0; p < kPassBatch; ++p)
                if (64 * p < left) v[p] = src[64 * p];
#pragma unroll
            for (int p = 0; p < kPassBatch; ++p) {
                const int c = lane_chunk + 64 * p;
                if (c < left && (p > 0 || c >= skip)) {
                    f4u o = {v[p].x, v[p].y, v[p].z, v[p].w};
                    f4u *dp = reinterpret_cast<f4u *>(dst + 1024 * p + (uint32_t)(16 * lane_chunk));
                    // single-wave envs stream with the non-temporal hint: the rows are never
                    // read back by the kernel, and the hint measurably raises the store rate there
                    // (it lowers it for the two-wave, 8 KB-row case)
                    if (WAVES == 1) __builtin_nontemporal_store(o, dp);
                    else *dp = o;
                }
            }
            src += 64 * kPassBatch;
            dst += 1024 * kPassBatch;
        }
        if (!whole) {
            // the half chunks at the two ends: lane 0 the first, lane 1 the last
            const bool head = lane == 0 && (pad & 2) && !carried, tail = lane == 1 && (floats & 2) != 0 && !carry;
            if (head || tail) {
                const int at = head ? pad : floats - 2;
                *reinterpret_cast<v2 *>(out + at) = *reinterpret_cast<const v2 *>(buf + at);
            }
        }
        lds_barrier<1>();
        carried = carry;
        if (carry) {
            const int rest = floats & 31, from = (floats - rest) >> 2;      // (the shared line, its first chunk)
            if (whole) {
                if (4 * lane < rest) vstage[staged_chunk(lane)] = vstage[staged_chunk(from + lane)];
            } else if (2 * lane < rest) {
                reinterpret_cast<v2 *>(buf)[lane] = reinterpret_cast<const v2 *>(buf)[2 * from + lane];
            }
        }
        // (8 KB rows: the wavefront lets its row land before it goes on, which keeps the XCDs together,
        // as in tabx_observe_packed.h: 64v64 x 512 125 us without, 117 with)
        if (WAVES == 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (WAVES == 1 && vis_mask) {
        // lane l writes row l of the group, if it was this wavefront's: row l % S of pass l / S
        const int p = quotient(lane, a.magic_s);
        const uint32_t lo = (uint32_t)__shfl(vis_lo, p), hi = (uint32_t)__shfl(vis_hi, p);
        const uint64_t range = N >= 64 ? ~0ull : ((1ull << N) - 1ull);
        if (lane < rows && ((passes_done >> p) & 1))
            vis_mask[row0 + lane] = ((((uint64_t)hi << 32) | lo) >> mul24(lane - mul24(p, S), N)) & range;
    }
}

// A scripted unit with the winning bids `tk`, `nk`: what it has made out of the units it sees, and the
// rule cascade.  pose_of(j): x, y, cos, sin of unit j of its env; radius_of(j): its body radius.
template <class PoseOf, class RadiusOf>
__device__ __forceinline__ void decide_unit(const KArgs &a, const Place &P, const Unit &U, float cu,
                                            float su, bool in_bush, unsigned long long tk,
                                            unsigned long long nk, bool can_hit, PoseOf pose_of,
                                            RadiusOf radius_of, const Carry &C, const float *zd)
{
    Sighting S;
    S.tgt = tk == ~0ull ? -1 : (int)((tk >> 1) & 0x7f);
    S.tgt_d2 = __int_as_float((int)(unsigned)(tk >> 8));
    S.tgt_in_box = (tk & 1ull) != 0ull;
    const int tl = S.tgt >= 0 ? S.tgt : 0;
    S.T = pose_of(tl);
    S.tr = radius_of(tl);
    S.any_enemy = nk != ~0ull;
    S.near_d2 = __int_as_float((int)(unsigned)(nk >> 32));
    const float4 E = pose_of(S.any_enemy ? (int)(nk & 0x7f) : 0);
    S.near_dx = E.x - U.x;
    S.near_dy = E.y - U.y;
    S.can_hit = can_hit;
    const int remembered = C.restarted ? 0 : C.mem_valid;
    policy_cascade(a, P, U, cu, su, in_bush, S, (uint32_t)C.tick, remembered, C.mem_x, C.mem_y, zd,
                   late_args()->pa.next_action);
}

// Scripted units: everybody has bid (all rows of the group are written); the lane's unit reads
// its winners and runs the rule cascade.
template <int WAVES>
__device__ __forceinline__ void decide_units(const KArgs &a, const Records<64 * WAVES> &rec,
                                             const ScriptLds<WAVES> *script, const Place &P,
                                             float speed, const Carry &C, const float *zd)
{
    const float4 B = rec.own[0][P.l], G = rec.own[1][P.l], V = rec.view[P.l];
    const int fu = __float_as_int(rec.mark[P.l].y);
    if (!(fu & 32)) return;
    Unit U = {};
    U.x = B.z;
    U.y = B.w;
    U.range = G.y;
    U.dmg = G.z;
    U.cd = G.w;
    U.speed = speed;
    auto pose_of = [&](int j) {
        const float4 b = rec.own[0][P.base + j], v = rec.view[P.base + j];
        return make_float4(b.z, b.w, v.x, v.y);
    };
    decide_unit(a, P, U, V.x, V.y, ((fu >> 20) & 3) == TABX_ZONE_BUSH, script->tkey[P.l], script->nkey[P.l],
                script->canhit[P.l] != 0, pose_of, [&](int j) { return rec.own[2][P.base + j].y; }, C, zd);
}

} // namespace tabx
