// Numbering of the workgroups of the K-loop split-fp16 engine.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace knm {

constexpr int kPatch = 64;  // workgroups per patch = resident workgroups per XCD (32 CUs x 2)
constexpr int kPatchF = 8;  // fixed blocks per patch (measured: 2..8 within 4 % of each other, 64 is 25 % slower)

// Workgroup -> (fixed block, stream chunk).  Workgroups are dealt round-robin to the 8 XCDs
// (each with its own L2) in launch order, and the ones resident together on an XCD are
// consecutive in that order.  They are therefore numbered so that each XCD works through
// "patches" of pf fixed blocks x pc chunks: the pf fixed-block images, which every
// workgroup re-reads for each of its stream tiles, stay in that XCD's L2, and a stream tile
// fetched by one workgroup is reused by the pf - 1 others on the same chunk.  The chunks are taken in groups of pc (the last one
// narrower).  In each, 8 patches at a time go to the 8 XCDs, and the fixed blocks that are left when fewer
// than 8 whole patches remain are split over them in equal shares, rounded up: no XCD gets more than one
// workgroup per group above the even share (whole patches dealt out left some XCDs with a fifth more than others at 235 fixed blocks x 5 chunks).
struct PatchMap {
    int pc;                  // chunks of a group
    int64_t n_fblocks;       // fixed blocks of this launch
    int64_t full_groups;     // groups of pc chunks; slots_full places per XCD each
    int64_t slots_full, slots_last;
    int pc_last;             // chunks of the last group (0: none)
    int pf, pf_last;         // fixed blocks of a patch
    static PatchMap make(int64_t f_blocks, int64_t chunks)
    {
        PatchMap pm;
        pm.pc = kPatch / kPatchF;
        pm.pf = kPatchF;
        pm.n_fblocks = f_blocks;
        pm.full_groups = chunks / pm.pc;
        pm.pc_last = (int)(chunks % pm.pc);
        pm.pf_last = pm.pc_last > 0 ? kPatch / pm.pc_last : 1; // as many workgroups per patch
        pm.slots_full = slots(f_blocks, pm.pf, pm.pc);
        pm.slots_last = pm.pc_last > 0 ? slots(f_blocks, pm.pf_last, pm.pc_last) : 0;
        return pm;
    }
    int64_t workgroups() const { return 8 * (full_groups * slots_full + slots_last); }
    static int64_t slots(int64_t n_f, int pf, int pc)
    {
        const int64_t whole = n_f / (8 * pf);
        return whole * pf * pc + ((n_f - whole * 8 * pf) * pc + 7) / 8;
    }
    // false: no work for this workgroup
    __host__ __device__ bool find(int64_t block, int64_t &f, int64_t &c) const
    {
        const int xcd = (int)(block & 7);
        int64_t slot = block >> 3;
        int64_t group = full_groups;
        int gc = pc_last, gf = pf_last;
        if (slot < full_groups * slots_full) {
            group = slot / slots_full;
            slot -= group * slots_full;
            gc = pc;
            gf = pf;
        } else {
            slot -= full_groups * slots_full;
            if (slot >= slots_last) return false;
        }
        const int per_patch = gf * gc;
        const int64_t whole = n_fblocks / (8 * gf);
        if (slot < whole * per_patch) {
            const int within = (int)(slot % per_patch);
            f = ((slot / per_patch) * 8 + xcd) * gf + within % gf;
            c = group * pc + within / gf;
            return true;
        }
        slot -= whole * per_patch;
        const int64_t rest = (n_fblocks - whole * 8 * gf) * gc, share = (rest + 7) / 8;
        const int64_t i = xcd * share + slot;
        if (i >= rest) return false;
        f = whole * 8 * gf + i / gc;
        c = group * pc + i % gc;
        return true;
    }
};

} // namespace knm
