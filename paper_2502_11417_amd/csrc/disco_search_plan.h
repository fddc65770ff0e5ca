// Passes of a wait or slope search, from sizes alone: plain host code, which a host compiler takes without the GPU's headers.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "disco.h"

constexpr int SB_DEPTH = 10;                      // bisection steps per pass, at most
// The list: up to this many requests one workgroup takes all remaining steps (1 us per 1000 of them and round, where all of them
// change between the same two candidates); longer ones take further passes (empty ones are two launches each, 4 to 5 us).
// The workgroups of several searches walk their lists side by side, where further passes cost every search its own.  10^6
// requests, 32 steps, with a limit of 8192 and of 32 768: one search 85 / 86 us, server TTFTs of whole milliseconds (thousands
// at one value) 87 / 105; four searches 142 / 117, 16 276 / 215, 64 791 / 698.
constexpr unsigned LIST_MAX = 32768, LIST_MAX_FEW = 8192;
constexpr int LIST_FEW = 2;
// An entry holds the request's index in 32 bits: a trace of more requests has no list and takes every step by passes.
constexpr int64_t LIST_REQ = (int64_t)1 << 32;

struct SearchPlan {
    int depth[DISCO_MAX_STEPS + 1];               // steps of each pass, 0 behind the last one
    int npass;
    bool list;                                    // the second pass lists the requests that still change
    unsigned cap;                                 // entries of a search's list
};

// room: entries that the scratch has for a search.  One pass, two passes that share the steps out evenly, or two full ones and the
// rest from the list of the second; passes behind those for searches whose list is too long.
inline SearchPlan search_plan(int64_t n_req, int n_search, int n_steps, size_t room)
{
    SearchPlan s{};
    const size_t limit = n_search <= LIST_FEW ? LIST_MAX_FEW : LIST_MAX;
    s.cap = (unsigned)(room < limit ? room : limit);
    if (n_steps <= SB_DEPTH) {
        s.depth[s.npass++] = n_steps;
    } else if (n_steps <= 2 * SB_DEPTH) {
        s.depth[s.npass++] = (n_steps + 1) / 2;
        s.depth[s.npass++] = n_steps / 2;
    } else {
        s.list = n_req <= LIST_REQ;
        for (int left = n_steps; left > 0; left -= SB_DEPTH) s.depth[s.npass++] = left < SB_DEPTH ? left : SB_DEPTH;
    }
    return s;
}
