// composer_model.h -- the composer's kernels on the CPU, one scenario lane after the other.
//
// TEST INFRASTRUCTURE, included by hip_host_stub.cpp: reads the walk lists, segments and
// overlap ranges exactly as the device code does (register slots, folds, linked collectives,
// LDS channels, member slots, counted arrivals, segment durations in the finish rows), so that
// a loader that lays them out wrongly shows on the CPU, under AddressSanitizer, against the
// oracle.  Walkers run in turn until they wait; when all of them wait the launch fails.
// Collective costs are the caller's (echo_stub_set_costs).  Tree ensembles are not modelled.
#pragma once

#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

#include "echo_internal.h"

namespace echo_model {

using namespace echo;

inline uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
inline int64_t q16(int64_t d, uint64_t f) { return (int64_t)(((uint64_t)d * f + 32768u) >> 16); }
inline int64_t jittered(int64_t d, int32_t op, const echo_scenario &sc) {
    const uint64_t k = ((uint64_t)sc.jitter_stream << 36) + (uint64_t)op + 1;
    const uint64_t u = mix64(sc.jitter_seed + k * 0x9E3779B97F4A7C15ull) >> 32;
    const uint64_t amp = (uint64_t)sc.jitter_amp_q16;
    return q16(d, 65536 - amp + ((u * (2 * amp + 1)) >> 32));
}
inline uint32_t factor(uint32_t m, const echo_scenario &sc, uint32_t cls) {
    uint32_t F = 65536u;
    for (int t = 0; t < kTypes; ++t)
        if ((m >> t) & 1u) F = std::max(F, sc.slowdown_q16[cls][t]);
    return F;
}

// the tile draws jitter: its durations come from the finish rows from the first sweep on
inline bool tile_jitter(const WalkArgs &a, int32_t tile) {
    for (int32_t s = tile * kLanes; s < std::min(a.n_scen, (tile + 1) * kLanes); ++s)
        if (a.scen[s].jitter_amp_q16 != 0) return true;
    return false;
}

inline void sums(const WalkArgs &a, int32_t tile) {
    const int64_t n = a.chunks[a.n_chunks].rec0;
    for (int32_t s = tile * kLanes; s < std::min(a.n_scen, (tile + 1) * kLanes); ++s) {
        int64_t sum = 0;
        for (int64_t i = 0; i < n; ++i) {
            const SegRec &r = a.recs[i];
            sum += jittered(r.dur, r.op, a.scen[s]);
            if (!(r.meta & kRecLast)) continue;
            a.finish[(int64_t)r.op * a.n_scen + s] = sum;
            sum = 0;
        }
    }
}

// false: the lists are inconsistent, or every walker waits
inline bool sweep(const WalkArgs &a, int32_t tile) {
    struct Walker {
        int64_t slot[kStreams][kLanes] = {}, none[kLanes] = {};
        int64_t item, end;
        bool launched = false;
    };
    struct Channel {
        unsigned count = 0;
        int64_t latest[kLanes] = {};
    };
    const int64_t ns = a.n_scen, s0 = (int64_t)tile * kLanes;
    const int lanes = (int)std::min<int64_t>(kLanes, ns - s0);
    const bool ops = a.in == kInOps, refined = a.in != kInNone && !ops;
    const bool load_d = refined || (!ops && tile_jitter(a, tile));
    const bool keep = !a.final_pass || a.digest || a.timelines;
    auto at = [&](int64_t *base, int64_t row) { return base + row * ns + s0; };
    std::vector<Walker> ws(a.n_walkers);
    std::vector<Channel> ch((size_t)((a.n_walkers + kBlockWalkers - 1) / kBlockWalkers) * kChannels * 2);
    for (int32_t w = 0; w < a.n_walkers; ++w) {
        ws[w].item = a.round_off[w] * kBlock;
        ws[w].end = a.round_off[w + 1] * kBlock;
    }
    bool moved = true, done = false;
    while (moved && !done) {
        moved = false;
        done = true;
        for (int32_t w = 0; w < a.n_walkers; ++w) {
            Walker &k = ws[w];
            for (; k.item < k.end; ++k.item, moved = true) {
                const WalkItem &it = a.items[k.item];
                if (it.meta & kEmpty) continue;
                const int64_t in_round = k.item % kBlock;
                if (in_round > 0 && (a.items[k.item - 1].meta & kEmpty)) return false;   // padding inside a round
                const int kind = item_kind(it.meta);
                const int sq = (it.meta & kNoReg) ? -1 : item_stream(it.meta);
                const uint32_t aux = (uint32_t)it.aux;
                const bool comm = kind == ECHO_COMM || kind == kResolve;
                Channel *c = comm && (aux & kAuxLocal) ? &ch[(size_t)(w / kBlockWalkers) * kChannels * 2 + aux_barrier(aux)] : nullptr;
                auto arrive = [&](const int64_t *v) {
                    for (int l = 0; l < lanes; ++l) c->latest[l] = std::max(c->latest[l], v[l]);
                    ++c->count;
                };
                if (kind == kResolve) {
                    int64_t b[kLanes] = {}, own[kLanes] = {};
                    if (c) {
                        if ((it.meta & kLaunch) && !k.launched) {
                            if (keep) std::copy_n(k.slot[0], lanes, at(a.start, it.op));
                            arrive(k.slot[0]);
                            k.launched = moved = true;
                        }
                        if (c->count < aux_expected(aux)) break;
                        std::copy_n(c->latest, lanes, b);
                    } else if (aux & kAuxSlots) {
                        bool all = true;
                        for (unsigned m = 0; m < aux_expected(aux); ++m)
                            for (int l = 0; l < lanes; ++l) {
                                const int64_t v = a.slots[(it.far_off + (int64_t)m) * ns + s0 + l];
                                all = all && v >= 0;
                                b[l] = std::max(b[l], v);
                            }
                        if (!all) break;
                    } else {
                        if (a.count[(int64_t)it.coll * a.n_tiles + tile] < (unsigned)a.c_N[it.coll]) break;
                        for (int l = 0; l < lanes; ++l) b[l] = (int64_t)a.arrive[(int64_t)it.coll * ns + s0 + l];
                    }
                    k.launched = false;
                    const int sl = aux_slot(aux);
                    if (sl < kClassSlots && a.block_class[(int64_t)(w / kBlockWalkers) * kClassSlots + sl] != it.dur) return false;
                    if (it.meta & kLinked) {
                        if (keep) std::copy_n(at(a.start, it.op), lanes, own);
                        for (int l = 0; l < lanes; ++l) {
                            const int64_t p = sq >= 0 ? k.slot[sq][l] : at(a.finish, it.nfar)[l];
                            b[l] = std::max(b[l], p);
                            own[l] = std::max(own[l], p);
                        }
                        if (keep) std::copy_n(own, lanes, at(a.start, it.op));
                    }
                    for (int l = 0; l < lanes; ++l) {
                        const int64_t f = b[l] + a.class_cost[it.dur * ns + s0 + l];
                        if (keep || (it.meta & kNeedF)) at(a.finish, it.op)[l] = f;
                        if (a.digest && a.final_pass)
                            a.digest[s0 + l] += mix64(mix64((uint64_t)it.op ^ (uint64_t)at(a.start, it.op)[l]) ^ (uint64_t)f);
                        if (sq >= 0) k.slot[sq][l] = f;
                        else k.none[l] = std::max(k.none[l], f);
                        if (it.meta & kFold) k.slot[0][l] = std::max(k.slot[0][l], f);
                    }
                    continue;
                }
                int64_t ready[kLanes] = {};
                for (int q = 0; q < kStreams; ++q)
                    if ((item_regmask(it.meta) >> q) & 1u)
                        for (int l = 0; l < lanes; ++l) ready[l] = std::max(ready[l], k.slot[q][l]);
                for (int32_t q = 0; (it.meta & kHasFar) && q < it.nfar; ++q) {
                    const RowPair u = a.far[it.far_off + q];
                    for (int l = 0; l < lanes; ++l) {
                        int64_t f = at(a.finish, u.last)[l];
                        if (!a.final_pass && u.first >= 0) f += at(a.start, u.first)[l];
                        ready[l] = std::max(ready[l], f);
                    }
                }
                if (keep) std::copy_n(ready, lanes, at(a.start, it.op));
                if (kind == ECHO_COMM) {
                    if (c) {
                        arrive(ready);
                    } else if (aux & kAuxSlots) {
                        std::copy_n(ready, lanes, a.slots + it.dur * ns + s0);
                    } else {
                        for (int l = 0; l < lanes; ++l) {
                            unsigned long long &x = a.arrive[(int64_t)it.coll * ns + s0 + l];
                            x = std::max(x, (unsigned long long)ready[l]);
                        }
                        ++a.count[(int64_t)it.coll * a.n_tiles + tile];
                    }
                    continue;
                }
                // the segment's place among the round's: where its duration is fetched from
                int64_t q = 0;
                for (int64_t x = k.item - in_round; x < k.item; ++x) q += (a.items[x].meta & 1u) == 0;
                if (q >= kDurs || a.rows[k.item / kBlock * kDurs + q] != it.coll) return false;
                const int64_t r0 = a.rec_rows[k.item / kBlock * kDurs + q], r1 = r0 + it.aux;
                if (r0 < 0 || r1 > a.n_recs || a.recs[r0].op != it.op || a.recs[r1 - 1].op != it.coll) return false;
                for (int l = 0; l < lanes; ++l) {
                    int64_t &row = at(a.finish, it.coll)[l];
                    if (ops) {
                        int64_t t = ready[l];
                        for (int64_t i = r0; i < r1; ++i) {
                            const SegRec &r = a.recs[i];
                            at(a.start, r.op)[l] = t;
                            t += jittered(r.dur, r.op, a.scen[s0 + l]);
                            at(a.finish, r.op)[l] = t;
                        }
                        if (sq >= 0) k.slot[sq][l] = t;
                        else k.none[l] = std::max(k.none[l], t);
                        continue;
                    }
                    const int64_t d = load_d ? row : it.dur, f = ready[l] + d;
                    if (!a.final_pass) row = d;
                    else if (keep || (it.meta & kNeedF)) row = f;
                    if (sq >= 0) k.slot[sq][l] = f;
                    else k.none[l] = std::max(k.none[l], f);
                }
            }
            done = done && k.item == k.end;
        }
    }
    if (done && a.final_pass)
        for (const Walker &k : ws)
            for (int l = 0; l < lanes; ++l) {
                int64_t &step = a.step[s0 + l];
                step = std::max(step, k.none[l]);
                for (int q = 0; q < kStreams; ++q) step = std::max(step, k.slot[q][l]);
            }
    return done;
}

// the ops' own times; unflagged segments keep their base durations
inline void expand(const WalkArgs &a, int32_t tile) {
    const int64_t n = a.chunks[a.n_chunks].rec0, ns = a.n_scen;
    for (int32_t s = tile * kLanes; s < std::min(a.n_scen, (tile + 1) * kLanes); ++s) {
        int64_t t = 0, oseg = 0;
        bool on = false;
        for (int64_t i = 0; i < n; ++i) {
            const SegRec &r = a.recs[i];
            if (r.meta & kRecFirst) {
                t = a.start[(int64_t)r.op * ns + s];
                on = a.in != kInNone && (r.meta & kRecCand) && a.xflag[oseg++ * a.n_tiles + tile];
            }
            int64_t d = jittered(r.dur, r.op, a.scen[s]);
            if (on && (r.meta & kRecCompute)) {
                if (a.ext) d += a.ext[i * a.mstride + s];
                else d = q16(d, factor(a.tmask[i * a.mstride + s], a.scen[s], r.meta & 7u));
            }
            if (a.digest) a.digest[s] += mix64(mix64((uint64_t)r.op ^ (uint64_t)t) ^ (uint64_t)(t + d));
            if (a.timelines) {
                a.start[(int64_t)r.op * ns + s] = t;
                a.finish[(int64_t)r.op * ns + s] = t + d;
            }
            t += d;
        }
    }
}

// every comm op of a segment's ranges against every op of the segment
inline void overlaps(const OverlapArgs &a) {
    const int64_t ns = a.n_scen;
    for (int64_t o = 0; o < a.n_osegs; ++o) {
        const OverlapSeg &os = a.osegs[o];
        for (int32_t tile = 0; tile < a.n_tiles; ++tile) {
            uint8_t &flag = a.xflag[o * a.n_tiles + tile];
            const bool was = a.prev_refined && flag;
            bool now = false;
            for (int64_t s = (int64_t)tile * kLanes; s < std::min<int64_t>(ns, (tile + 1) * (int64_t)kLanes); ++s) {
                const echo_scenario &sc = a.scen[s];
                int64_t t = a.start[(int64_t)os.first * ns + s], total = 0;
                for (int32_t i = os.rec0; i < os.rec0 + os.n; ++i) {
                    const SegRec &r = a.recs[i];
                    const int64_t D = jittered(r.dur, r.op, sc), at = (int64_t)i * a.mstride + s;
                    const uint32_t cls = r.meta & 7u, before = !was ? 0 : a.ext ? a.ext[at] : a.tmask[at];
                    const int64_t d = !was ? D : a.ext ? D + before : q16(D, factor(before, sc, cls));
                    uint32_t m = 0, e = 0;
                    int64_t covered = 0, dn = D;
                    if (r.meta & kRecCompute) {
                        std::vector<std::pair<int64_t, int64_t>> in;
                        for (int32_t k = os.cand0; k < os.cand0 + os.ncand; ++k)
                            for (int32_t x = a.ranges[k].lo; x < a.ranges[k].hi; ++x) {
                                const int64_t lo = std::max(t, a.start[(int64_t)a.cl[x] * ns + s]);
                                const int64_t up = std::min(t + d, a.finish[(int64_t)a.cl[x] * ns + s]);
                                if (lo >= up) continue;
                                m |= 1u << a.cl_type[x];
                                in.emplace_back(lo, up);
                            }
                        std::sort(in.begin(), in.end());
                        int64_t end = t;
                        for (const auto &iv : in)
                            if (iv.second > end) {
                                covered += iv.second - std::max(end, iv.first);
                                end = iv.second;
                            }
                        if (a.ext) {
                            const int64_t oc = std::min(covered, D);
                            e = (uint32_t)(q16(oc, factor(m, sc, cls)) - oc);
                            dn = D + e;
                        } else {
                            dn = q16(D, factor(m, sc, cls));
                        }
                        if (a.chg && dn != d) a.chg[s] = 1;
                    }
                    if (a.ext) a.ext[at] = e;
                    else a.tmask[at] = (uint8_t)m;
                    now = now || (a.ext ? e != 0 : m != 0);
                    t += d;
                    total += dn;
                }
                a.finish[(int64_t)os.last * ns + s] = total;
            }
            flag = now;
        }
    }
}

}  // namespace echo_model
