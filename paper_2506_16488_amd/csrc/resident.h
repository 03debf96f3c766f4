// Arguments of the resident search kernel (resident.hip): one workgroup runs
// a whole query.
#pragma once

#include "ppsp_dev.h"

namespace ppsp {

constexpr uint32_t RES_MAXDEG = 64;   // graphs with a vertex above this degree use the round kernels
constexpr uint32_t RES_ID_BITS = 27;  // and those with more vertices than this many bits count

// What a workgroup reports for its query.
enum ResidentStatus : uint32_t {
    RES_DONE = 0,       // answered
    RES_SPILL = 1,      // its frontier outgrew the queue: run it with the round kernels
    RES_TIMEOUT = 2,    // the time limit passed
    RES_OVERFLOW = 4,   // a tentative distance reached 2^32 - 1: whether any does in order, the round kernels say
};
enum ResidentStat { RS_ROUNDS = 0, RS_ENTRIES = 1, RS_SCANV = 2, RS_SCANE = 3, RS_SUCC = 4, RS_CARRY = 5, RS_STATUS = 6, RS_N = 8 };

struct ResidentArgs {
    const uint32_t *row_ptr;
    const uint2 *arcs;
    const uint32_t *in_row_ptr; // transpose (a directed graph's backward searches)
    const uint2 *in_arcs;
    const int2 *xy;
    uint64_t ws2;
    uint32_t fb;
    uint32_t n;
    const SearchDesc *sd;       // searches 2q, 2q + 1 of query q (pair), or search q
    const Partner *partners;
    const uint64_t *delta;      // threshold increment per search (key units)
    uint32_t nquery;
    uint32_t *D;                // distances, cleared to infinity: [nquery][n][2] (pair) or [nquery][n]
    uint4 *spill;               // [nquery][4][spcap] frontier entries beyond the two LDS queues, two far lists
    uint32_t spcap;
    uint64_t *mu;               // [npair] (distance, meeting vertex), written for every query with a partner
    unsigned long long *qstat;  // [nquery][RS_N]
    uint32_t theta_mode;
    unsigned long long ticks;   // time limit in wall-clock ticks from the launch's start (0: none)
    unsigned long long *t_begin;   // its start (~0 before)
};

}  // namespace ppsp
