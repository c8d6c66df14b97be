// Fused execution of a plan's small steps: every maximal subtree of small
// steps becomes one program that a single work-group runs out of LDS
// (fused.hip), and one launch runs all of a plan's programs in every residue
// plane. What is left of the plan is a list of larger steps over the
// programs' results.
#pragma once

#include <cstdint>
#include <vector>

#include "internal.hpp"

namespace tn {

// A step of a program: offsets are LDS entries, masks as in StepArgs.
// sr: shared bonds | output rank << 8 | kFuseRoot for the program's last
// step, whose output goes to global memory.
struct FuseStep {
    uint32_t offA, offB, offC;
    uint16_t maskA, sr;
};
constexpr uint32_t kFuseRoot = 0x8000u;

// A program's header. The blob holds the headers, then the programs (each
// n_steps FuseSteps, n_items words (step | chunk of 64 outputs << 16) sorted by
// level and n_levels + 1 item offsets, padded to 16 bytes), then the entries
// of the programs' initial tensors, laid out as in LDS, one byte or (wide)
// one 32-bit word each.
struct FuseProg {
    uint32_t prog, prog_bytes;             // byte offset in the blob
    uint32_t init, n_init;                 // first entry and entries of its initial tensors
    uint32_t n_steps, n_items, n_levels;
    uint32_t final;                        // 1: the root is the whole network's scalar
    int64_t root_off;                      // global output offset (entries), unless final
    uint32_t lds_elems;                    // its LDS entries (the program follows them)
    int32_t root_rank;
};
static_assert(sizeof(FuseStep) == 16 && sizeof(FuseProg) == 48, "device layout");

// How a contraction executes a plan: programs first, then steps in order.
// The offsets of its steps replace the plan's. Without programs it is the
// plan step by step.
struct Exec {
    std::vector<FuseProg> progs;
    std::vector<FuseStep> psteps;       // all programs' steps
    std::vector<uint32_t> pitems, plevels;
    std::vector<int32_t> pinit;         // initial tensors of the programs, in program order
    std::vector<int32_t> pinit_first;   // first of them per program (one more at the end)
    std::vector<uint32_t> pinit_off;    // their LDS entries
    std::vector<int32_t> prog_out;      // the tensor each program ends in
    uint32_t prog_end = 0;              // bytes of headers and programs
    uint32_t n_entries = 0;             // initial entries of all programs
    uint32_t lds_bytes = 0;             // LDS of the largest program
    std::vector<Step> steps;            // steps outside the programs
    std::vector<int32_t> init_ids;      // initial tensors those read
    std::vector<int64_t> init_off;      // and their offsets (entries)
    int64_t init_elems = 0, arena_elems = 0;
    double prog_entries = 0, prog_macs = 0;  // algorithmic totals of the programs, one plane
};

// LDS of a program for es-byte entries: its tensors, then the program; at most
// what a work-group may ask for on gfx950.
constexpr int64_t kMaxProgramLds = int64_t(160) << 10;
inline uint32_t lds_of(const FuseProg& pg, int es) {
    return (pg.lds_elems * uint32_t(es) + 15) / 16 * 16 + pg.prog_bytes;
}
// Bytes of the blob.
int64_t blob_bytes(const Exec& ex, bool wide);
// Writes the blob (zeroed by the caller) for a network's initial entries.
void fill_blob(const Network& net, const Plan& plan, const Exec& ex, bool wide, uint8_t* blob);

// The fused execution of a plan for an element size of es bytes.
void build_exec(const Plan& plan, int es, Exec& ex);
// Keeps the plan's execution for its default arithmetic with it; once the plan
// has its steps, and again when its count bound changes.
void keep_exec(Plan& plan);
// The plan step by step.
void plain_exec(const Plan& plan, Exec& ex);
// Checks an execution's layout against the liveness of its tensors: no tensor
// may overlap another one that is alive at the same time. Programs' results are
// written first and stay until they are read, where they are read; a program's
// LDS accesses stay within what it asks for.
tn_status verify_exec(const Plan& plan, const Exec& ex, int es);
// Kept with the plan for its default arithmetic (keep_exec); nullptr when the
// plan holds none for this element size.
const Exec* plan_exec(const Plan& plan, int es);

}  // namespace tn
