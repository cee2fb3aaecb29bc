// What the Picard loop's host does next (host code, no device types).
//
// The host queues iterations in batches and reads the loop's progress (window
// start t, iterations done k) while the last one of a batch still runs, so that
// the GPU never waits for it.  t and k come from one store and one load; even so
// nothing is concluded from a read that may be older than the queue: only a read
// after the stream was synchronised, with nothing queued since, can say that the
// loop is stuck.
#pragma once

#include <cmath>
#include <cstdint>

namespace pd {

// t and k as one 64-bit word, as the kernels publish and the host reads them.
inline uint64_t pack_progress(int32_t t, int32_t k) { return (uint64_t)(uint32_t)t | (uint64_t)(uint32_t)k << 32; }
inline int32_t progress_t(uint64_t w) { return (int32_t)(uint32_t)w; }
inline int32_t progress_k(uint64_t w) { return (int32_t)(uint32_t)(w >> 32); }

enum class PicardNext {
    QUEUE,    // queue n more iterations
    DRAIN,    // the queued ones may finish the loop: synchronise and read again
    STUCK,    // all T iterations have run and t < T
};
struct PicardPlan {
    PicardNext next;
    int n;
};

// T steps, windows of p, `issued` iterations queued so far; drained: the stream
// has been synchronised since the last one was.
inline PicardPlan picard_plan(int T, int p, int issued, int t, int k, int first_stride, bool drained) {
    // every iteration advances t by at most p, so at least this many
    // more are needed.  Beyond that, queue as many as the mean stride
    // after the first predicts (the first window holds copies of x_0 and
    // in practice slides by one), but at most as many as are already
    // done: strides grow as the trajectory converges, so early means
    // overestimate what is left, and iterations queued past the end
    // (they find p_eff = 0 on the device and return at once) still cost
    // a dispatch each.  Iterations still queued count against it.
    // The first batch adds one iteration more than the first window's
    // slide of one requires: the host then decides the second batch
    // from two finished iterations (the mean stride) while a third
    // still runs, instead of draining the stream and leaving the GPU
    // idle; it is wasted only when the loop ends within two iterations.
    const int in_flight = issued - k;
    int need = (T - t + p - 1) / p;
    if (issued == 0 && T > 1) need = 2 + (T - 1 + p - 1) / p;
    if (k >= 2 && t > first_stride) {
        const double mean = (double)(t - first_stride) / (double)(k - 1);
        int est = (int)std::ceil((double)(T - t) / mean);
        est = est < issued ? est : issued;
        need = need > est ? need : est;
    }
    // the chain's last point (sigma = 0) is held to no change at all and so
    // takes an iteration of its own: while more than that point is left,
    // one in flight does not end the loop
    if (need <= in_flight && T - t > 1) need = in_flight + 1;
    need = need < T - t ? need : T - t;   // stride >= 1 bounds the rest
    need -= in_flight;
    if (issued + need > T) need = T - issued;
    if (need > 0) return {PicardNext::QUEUE, need};
    return {drained ? PicardNext::STUCK : PicardNext::DRAIN, 0};
}

}  // namespace pd
