// Completion of store / retrieve calls.
//
// One event per call, complete when everything the call enqueued is, tells
// whoever has to wait (a later store of the same blocks, the next call on the
// host link, a work-list buffer's next user, release, destroy) that the call is
// done.  Everybody names the call by its number, and a number below the oldest
// call still in flight needs no wait at all.  One record and not one per
// purpose: each is a packet between this call's kernel and the next one's (a
// 2 MiB store over the link left 13.4 us of gap with three records, a retrieve 8
// with two, an HBM-only retrieve 2.4 with one).  Given to the launch as its stop
// event it would cost the stream nothing (that store: 40.7 us a pass instead of
// 43.8, back to back), but then every wait behind such a launch takes longer, up
// to twice as long (33 MB out of HBM, each call waited for: 64.9 us instead of
// 33.7), so it is recorded.

#include "internal.hpp"

namespace kvp {

namespace {

constexpr size_t kMaxFlight = 4096;   // calls in flight from which on no event is created

// Beside a capture of another stream the runtime refuses an event query, and
// ends that capture too, unless the querying thread's capture mode is relaxed.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { check_hip(hipThreadExchangeStreamCaptureMode(&mode), "hipThreadExchangeStreamCaptureMode"); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

bool query(hipEvent_t e)
{
    const hipError_t q = hipEventQuery(e);
    if (q != hipSuccess) clear_hip_error();   // "not ready" is the answer, not an error to leave behind
    if (q != hipErrorNotReady) check_hip(q, "hipEventQuery");
    return q == hipSuccess;
}

void land(Pool &p)   // the oldest call is done
{
    if (p.flight.front().owned) p.idle.push_back(p.flight.front().done);   // room reserved with the event
    p.flight.pop_front();
    ++p.flight_first;
}

}  // namespace

void add_idle_event(Pool &p)
{
    p.idle.reserve(p.events + 1);
    hipEvent_t e = nullptr;
    check_hip(hipEventCreateWithFlags(&e, hipEventDisableTiming), "hipEventCreate");
    ++p.events;
    p.idle.push_back(e);
}

hipEvent_t take_request_event(Pool &p)
{
    if (p.idle.size() <= kIdleEvents) add_idle_event(p);
    const hipEvent_t e = p.idle.back();
    p.idle.pop_back();
    return e;
}

void give_request_event(Pool &p, hipEvent_t e) noexcept
{
    forget_event(p, e);
    p.idle.push_back(e);
}

void forget_event(Pool &p, hipEvent_t e) noexcept
{
    for (auto &f : p.flight)
        if (f.done == e) f.done = nullptr;
}

const FlightRec *in_flight(const Pool &p, uint64_t call)
{
    if (call < p.flight_first) return nullptr;
    const FlightRec &f = p.flight[call - p.flight_first];
    return f.done ? &f : nullptr;
}

void wait_call(const Pool &p, uint64_t call)
{
    if (const FlightRec *f = in_flight(p, call)) check_hip(hipEventSynchronize(f->done), "hipEventSynchronize");
}

bool event_done(hipEvent_t e)
{
    const RelaxedCapture scope;
    return query(e);
}

void land_done_calls(Pool &p)
{
    if (p.flight.empty() || hipPeekAtLastError() != hipSuccess) return;
    const RelaxedCapture scope;
    while (!p.flight.empty() && (!p.flight.front().done || query(p.flight.front().done))) land(p);
}

hipEvent_t begin_call(Pool &p, hipStream_t s, hipEvent_t lent, hipEvent_t own, bool may_create)
{
    if (!lent && p.idle.empty() && may_create && p.flight.size() < kMaxFlight) {
        try {
            add_idle_event(p);
        } catch (const Error &) {   // the request's event will do
        }
    }
    if (!lent && p.idle.empty() && !(lent = own)) return nullptr;
    p.flight.push_back(FlightRec{lent ? lent : p.idle.back(), s, !lent});
    if (!lent) p.idle.pop_back();
    return p.flight.back().done;
}

void cancel_call(Pool &p) noexcept
{
    if (p.flight.back().owned) p.idle.push_back(p.flight.back().done);
    p.flight.pop_back();
}

uint64_t last_call(const Pool &p) { return p.flight_first + p.flight.size() - 1; }

void drain_calls(Pool &p) noexcept
{
    for (auto &f : p.flight)
        if (f.done) (void)hipEventSynchronize(f.done);
    for (auto &f : p.flight)
        if (f.owned) (void)hipEventDestroy(f.done);
    for (auto &r : p.requests)
        if (r.second->event) (void)hipEventDestroy(r.second->event);
    for (auto e : p.idle) (void)hipEventDestroy(e);
    p.flight.clear();
    p.idle.clear();
}

}  // namespace kvp
