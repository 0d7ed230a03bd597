// How many iterations a solve launches between two looks at its columns, and
// which of a batch's kept graphs holds them.  Host code without HIP types.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

namespace fs {

// The chunks between two looks at the column states.  A solve used to launch
// check_every iterations at a time, whatever was left to do: a solve of 35
// iterations launched 64, refinement steps of 9 launched 32 each (an idle
// iteration of three empty launches takes 5-7 us).  Now the columns' rate
// of convergence says how many are left; a look never comes later than
// every check_every iterations, and at each multiple of it, as before.
// Chunks are multiples of kChunk iterations, replayed as graphs of kChunk
// and kLongChunk, which the batch keeps.
constexpr int32_t kChunk = 4, kLongChunk = 16;

// Place of the graph of `iters` iterations among a batch's kept graphs: the
// two chunk lengths have their own, which no other length takes, since
// chunks of both are launched without a wait in between and a graph may
// only be destroyed when nothing of it runs.  All other lengths (check_every
// not a multiple of kChunk) share the third: they are launched once between
// two looks, so the one that a new length replaces has ended.
constexpr int kGraphs = 3;
inline int graph_place(int32_t iters)
{
    return iters == kChunk ? 0 : iters == kLongChunk ? 1 : 2;
}

struct Pace {
    int32_t every = 32;
    int32_t since = 0;                    // iterations since the start
    std::vector<double> rr, rate;         // per column: |r|^2 at the last
    std::vector<int32_t> iter;            //   look, its fall per iteration
    // iterations of the next chunk, from the nc states of the last look
    // (status `running`: the column iterates)
    template <class State>
    int32_t next(const State *states, size_t nc, int32_t running)
    {
        if (rr.size() != nc) {
            rr.assign(nc, 0.0);
            rate.assign(nc, 0.0);
            iter.assign(nc, 0);
        }
        double want = kChunk;
        for (size_t c = 0; c < nc; ++c) {
            const State &s = states[c];
            if (s.status == running && s.rr > 0.0) {
                // a tolerance that underflows (rtol |b| below 1e-162, the
                // way to ask for maxit iterations) is never met: infinity
                const double left = s.tol2 > 0.0 ? std::log(s.rr / s.tol2)
                                                 : HUGE_VAL;
                if (s.iter > iter[c] && rr[c] > s.rr && since > 0)
                    rate[c] = std::log(rr[c] / s.rr) / (s.iter - iter[c]);
                // unknown rate: two iterations per digit of |r|
                const double it = rate[c] > 0.0 ? left / rate[c]
                                                : 0.434 * left;
                if (it > want) want = it;
            }
            rr[c] = s.rr;
            iter[c] = s.iter;
        }
        const int32_t room = every - since % every;
        int32_t n = room;
        if (every % kChunk == 0 && want < room)
            n = std::min(room, (int32_t(std::ceil(want)) + kChunk - 1) /
                                   kChunk * kChunk);
        since += n;
        return n;
    }
};

}  // namespace fs
