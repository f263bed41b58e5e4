// The partitioned insert's host arithmetic for tests/test_bulk_plan.py.
#include "cf_bulk_plan.hpp"

namespace {

template <int F>
bool round_trip(uint32_t tag, uint32_t idx, uint32_t bucket) {
    const cfk::Ent e = cfk::unpack_ent<F>(cfk::pack_ent<F>(cfk::Ent{tag, idx, bucket}), idx);
    return e.tag == tag && e.idx == idx && e.bucket == bucket;
}

}  // namespace

extern "C" {

int wanted(uint64_t m, uint32_t b, uint32_t f, int walk, uint64_t n) {
    return cfl::bulk_wanted(cfl::BulkTable{m, b, f, walk != 0}, n);
}

int fits(uint64_t m, uint32_t b, uint32_t f, int walk, uint64_t n) {
    const cfl::BulkTable t{m, b, f, walk != 0};
    return cfl::bulk_fits(t, cfl::bulk_plan(t, n));
}

uint64_t most(uint64_t m, uint32_t b, uint32_t f, int walk, uint64_t n) {
    return cfl::bulk_most(cfl::BulkTable{m, b, f, walk != 0}, n);
}

uint64_t least(uint64_t m, uint32_t b, uint32_t f, int walk, uint64_t most) {
    return cfl::bulk_least(cfl::BulkTable{m, b, f, walk != 0}, most);
}

void plan(uint64_t m, uint32_t b, uint32_t f, uint64_t len, uint64_t *out) {
    const cfl::BulkPlan p = cfl::bulk_plan(cfl::BulkTable{m, b, f, false}, len);
    const uint64_t v[] = {p.shift, p.parts, p.bins,  p.fine,  p.cap1, p.cap2, p.list_cap, p.cursors,
                          p.o_cur, p.o_listn, p.o_a, p.o_a32, p.o_b,  p.o_b32, p.o_list,
                          p.o_list32, p.o_ovl, p.bytes};
    for (uint64_t x : v) *out++ = x;
}

int entry_survives(uint32_t f, uint32_t tag, uint32_t idx, uint32_t bucket) {
    return f == 8 ? round_trip<8>(tag, idx, bucket)
           : f == 16 ? round_trip<16>(tag, idx, bucket) : round_trip<32>(tag, idx, bucket);
}

uint64_t lds_bytes(uint32_t f, uint32_t bins) { return cfk::split_lds(int(f), bins); }
}
