// cf_inst.hpp -- the single-filter kernel instantiations behind
// cfl::Launchers.  Included only by the cf_inst_f*.hip (query, delete,
// recount) and cf_insi_f*.hip (insert) translation units, each of which
// instantiates one fingerprint width; the insert units are built at -O1
// (see the build script).
#pragma once

#include <type_traits>

#include "cf_launch.hpp"

namespace cfl {
namespace inst {

using cfk::Counters;
using cfk::kBlock;

// Query, delete and recount: independent of the eviction policy.
template <int F, int B, int HASH, int POL>
struct InstQD {
    using G = cfk::Geom<F, B>;
    using W = typename G::W;
    static void query(const void *t, const cfk::Place &pl, const uint64_t *k, uint64_t n,
                      uint8_t *o, int grid, hipStream_t s) {
        cfk::query_kernel<G, HASH, POL>
            <<<grid, kBlock, 0, s>>>(static_cast<const W *>(t), pl, k, n, o);
    }
    static void del(void *t, const cfk::Place &pl, const uint64_t *k, uint64_t n, uint8_t *o,
                    Counters *c, int grid, hipStream_t s) {
        cfk::delete_kernel<G, HASH, POL>
            <<<grid, kBlock, 0, s>>>(static_cast<W *>(t), pl, k, n, o, c);
    }
    static void recount(const void *t, uint64_t nw, Counters *c, int grid, hipStream_t s) {
        cfk::recount_kernel<G><<<grid, kBlock, 0, s>>>(static_cast<const W *>(t), nw, c);
    }
    static void fill(Launchers &L) {
        L.query = &query;
        L.del = &del;
        L.recount = &recount;
        L.words_per_bucket = uint64_t(G::WPB);
        L.word_bytes = uint64_t(sizeof(W));
    }
};

// Insert, per eviction policy and breadth-first probe width.
template <int F, int B, int HASH, int EVICT, int POL>
struct InstI {
    using G = cfk::Geom<F, B>;
    static constexpr int PW = EVICT == 0 ? cfk::probe_width<G>() : 1;
    using W = typename G::W;
    template <class R>
    static void run(void *t, const cfk::Place &pl, const uint64_t *k, uint64_t n, uint8_t *o,
                    uint32_t *kk, Counters *c, uint32_t *q, uint64_t seg, cfk::LostLog log,
                    uint32_t me, uint64_t seed, const R &rest, bool grouped, int grid,
                    hipStream_t s) {
        if (PW > 1 && grouped)
            cfk::insert_kernel<G, HASH, EVICT, POL, PW, R><<<grid, kBlock, 0, s>>>(
                static_cast<W *>(t), pl, k, n, o, kk, c, q, seg, log, me, seed, rest);
        else
            cfk::insert_kernel<G, HASH, EVICT, POL, 1, R><<<grid, kBlock, 0, s>>>(
                static_cast<W *>(t), pl, k, n, o, kk, c, q, seg, log, me, seed, rest);
    }
    static void ins(void *t, const cfk::Place &pl, const uint64_t *k, uint64_t n, uint8_t *o,
                    uint32_t *kk, Counters *c, uint32_t *q, uint64_t seg, cfk::LostLog log,
                    uint32_t me, uint64_t seed, const cfk::Rest *rest, bool grouped, int grid,
                    hipStream_t s) {
        if (rest) run(t, pl, k, n, o, kk, c, q, seg, log, me, seed, *rest, grouped, grid, s);
        else run(t, pl, k, n, o, kk, c, q, seg, log, me, seed, cfk::NoRest{}, grouped, grid, s);
    }
};

// The partitioned insert: the splits and the move know nothing of the bucket
// size, the placement of entries in a part nothing of hash and policy.
template <int F, int HASH, int POL>
void split(const uint64_t *k, uint32_t n, const cfk::Place &pl, uint32_t shift, uint32_t nbins,
           uint32_t *cur, cfk::Ents out, uint32_t cap, uint8_t *o, uint32_t *kk, uint32_t *ovl,
           uint32_t *ovl_n, hipStream_t s) {
    const uint32_t grid = (n + cfk::kSplitTile - 1) / cfk::kSplitTile;
    cfk::bulk_split_kernel<F, HASH, POL><<<grid, cfk::kSplitBlock, cfk::split_lds(F, nbins), s>>>(
        k, n, pl, shift, nbins, cur, out, cap, o, kk, ovl, ovl_n);
}
template <int F>
void resplit(cfk::Ents in, const uint32_t *in_n, uint32_t nbins, uint32_t cap_in, uint32_t shift,
             uint32_t fine, uint32_t *cur, cfk::Ents out, uint32_t cap, uint32_t *ovl,
             uint32_t *ovl_n, hipStream_t s) {
    const uint32_t tiles = (cap_in + cfk::kSplitTile - 1) / cfk::kSplitTile;
    cfk::bulk_resplit_kernel<F>
        <<<nbins * cfk::kBulkSegs * tiles, cfk::kSplitBlock, cfk::split_lds(F, 1u << fine), s>>>(
            in, in_n, nbins, cap_in, tiles, shift, fine, cur, out, cap, ovl, ovl_n);
}
template <int F, int HASH, int POL>
void move(cfk::Ents list, const uint32_t *list_n, uint32_t list_cap, const cfk::Place &pl,
          uint32_t part_shift, uint32_t shift, uint32_t nbins, uint32_t *cur, cfk::Ents out,
          uint32_t cap, uint32_t *ovl, uint32_t *ovl_n, int parts, hipStream_t s) {
    cfk::bulk_move_kernel<F, HASH, POL>
        <<<parts, cfk::kSplitBlock, cfk::split_lds(F, nbins), s>>>(
            list, list_n, list_cap, pl, part_shift, shift, nbins, cur, out, cap, ovl, ovl_n);
}
template <int F, int B>
void place(void *t, uint64_t m, uint32_t shift, cfk::Ents in, const uint32_t *in_n, uint32_t runs,
           uint32_t stride, uint32_t cap, cfk::Ents list, uint32_t *list_n, uint32_t list_cap,
           const uint32_t *ovl_n, Counters *c, int parts, hipStream_t s) {
    using G = cfk::Geom<F, B>;
    cfk::bulk_insert_kernel<G>
        <<<parts, cfk::kPlaceBlock, (size_t(B) * F / 8) << shift, s>>>(
            static_cast<typename G::W *>(t), m, shift, in, in_n, runs, stride, cap, list, list_n,
            list_cap, ovl_n, c);
}

template <int F, int B, int POL>
void fill_qd(int hash, Launchers &L) {
    if (hash == 0) InstQD<F, B, 0, POL>::fill(L);
    else InstQD<F, B, 1, POL>::fill(L);
}

template <int F, int B, int POL>
void fill_ins(int hash, int evict, Launchers &L) {
    L.split = hash == 0 ? &split<F, 0, POL> : &split<F, 1, POL>;
    L.resplit = &resplit<F>;
    L.move = hash == 0 ? &move<F, 0, POL> : &move<F, 1, POL>;
    L.place = &place<F, B>;
    L.ins = hash == 0 ? (evict == 0 ? &InstI<F, B, 0, 0, POL>::ins : &InstI<F, B, 0, 1, POL>::ins)
                      : (evict == 0 ? &InstI<F, B, 1, 0, POL>::ins : &InstI<F, B, 1, 1, POL>::ins);
}

// Fills the query/delete/recount part (INSERT = false) or the insert part
// (INSERT = true) of L for p's bucket size; false if unsupported.
template <int F, bool INSERT>
bool pick_b(const cf_params &p, Launchers &L) {
    auto one = [&](auto bconst) {
        constexpr int B = decltype(bconst)::value;
        const bool off = p.placement == CF_PLACE_OFFSET;
        if constexpr (INSERT) {
            if (off) fill_ins<F, B, 1>(p.hash, p.evict, L);
            else fill_ins<F, B, 0>(p.hash, p.evict, L);
        } else {
            if (off) fill_qd<F, B, 1>(p.hash, L);
            else fill_qd<F, B, 0>(p.hash, L);
        }
        return true;
    };
    switch (p.slots_per_bucket) {
        case 4: return one(std::integral_constant<int, 4>{});
        case 8: return one(std::integral_constant<int, 8>{});
        case 16: return one(std::integral_constant<int, 16>{});
        case 32: return one(std::integral_constant<int, 32>{});
        default: return false;
    }
}

}  // namespace inst
}  // namespace cfl
