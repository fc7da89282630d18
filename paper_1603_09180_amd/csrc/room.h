// room.h -- admission of kernels whose blocks wait for each other.  Host code
// that needs no GPU to run.
#pragma once

#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace thin {

// Room on a device for such kernels (k_flow, k_coop), held from before the
// launch until the kernel has ended: two that are each partly resident would
// keep one another waiting.  Kernels run together if all their blocks become
// resident wherever each one goes: with no more blocks than the device has
// compute units (a block not yet resident then finds a unit without any of
// them, and takes it when whatever else runs there ends), or, all of one
// kernel, no more than the device holds of it.  The dispatcher deals a
// kernel's blocks to the XCDs in turn, so what counts is the fullest XCD: a
// kernel's blocks are rounded up to a whole turn (three kernels of 85 blocks
// leave 33 to one XCD's 32 units).  First come, first served, but a kernel that
// fits goes past those that wait for more room, each of which lets kPasses
// pass (128x128 from 8 threads, one image each: 25 us an image, 100 if launches
// run one by one).  A kernel that could run another way waits only while room
// is being given back: it leaves without when nobody has left for `patience`
// microseconds (a cooperative run of seconds, or a stream that has not come to
// its kernel yet).
class Room {
public:
    // which: the kernel; holds: how many of its blocks the device holds;
    // patience: < 0 without end
    Room(int device, int which, int blocks, int holds, int num_cus, int64_t patience)
        : gate_(gate_of(device)), blocks_((blocks + kXcds - 1) / kXcds * kXcds)
    {
        std::unique_lock<std::mutex> lock(gate_.m);
        Waiter me;
        Waiter** at = &gate_.first;
        while (*at) at = &(*at)->next;
        *at = &me;
        auto may = [&] {
            const int all = gate_.used + blocks_;
            if (gate_.used != 0 && all > num_cus && !(gate_.which == which && all <= holds)) return false;
            for (const Waiter* w = gate_.first; w != &me; w = w->next)
                if (w->passed >= kPasses) return false;
            return true;
        };
        while (!(held_ = may())) {
            gate_.sought = std::chrono::steady_clock::now();
            if (patience < 0) {
                gate_.freed.wait(lock);
                continue;
            }
            const uint64_t left = gate_.left;
            const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(patience);
            if (!gate_.freed.wait_until(lock, until, [&] { return gate_.left != left || may(); })) break;
        }
        for (at = &gate_.first; *at != &me; at = &(*at)->next)
            if (held_) ++(*at)->passed;
        *at = me.next;
        if (gate_.first) gate_.freed.notify_all();
        if (!held_) return;
        gate_.which = gate_.used == 0 || gate_.which == which ? which : kMixed;
        gate_.used += blocks_;
    }
    ~Room()
    {
        if (!held_) return;
        const std::lock_guard<std::mutex> lock(gate_.m);
        gate_.used -= blocks_;
        ++gate_.left;
        if (gate_.first) gate_.freed.notify_all();
    }
    Room(const Room&) = delete;
    Room& operator=(const Room&) = delete;

    bool held() const { return held_; }

    // Whether somebody found no room within the last 10 seconds: then a caller
    // asks for room only once its stream has come to the kernel (some
    // microseconds more of a call), so that nobody waits for what the stream has
    // to do before.
    static bool sought(int device)
    {
        Gate& gate = gate_of(device);
        const std::lock_guard<std::mutex> lock(gate.m);
        return std::chrono::steady_clock::now() - gate.sought < std::chrono::seconds(10);
    }

    static constexpr int kCoop = -1;  // which: k_coop; k_flow's are its shapes from 0 on
    static constexpr int kXcds = 8;
    static constexpr int kPasses = 8;

private:
    static constexpr int kMixed = -2;
    struct Waiter {
        Waiter* next = nullptr;
        int passed = 0;      // later ones that went in before it
    };
    struct Gate {
        std::mutex m;
        std::condition_variable freed;
        Waiter* first = nullptr;  // those that wait, in the order they came
        uint64_t left = 0;   // how many have given room back
        std::chrono::steady_clock::time_point sought{};  // somebody waited last (or never)
        int used = 0;        // blocks of all that hold room
        int which = kMixed;  // the kernel they all are
    };
    static Gate& gate_of(int device)
    {
        static Gate gates[64];
        return gates[device & 63];
    }
    Gate& gate_;
    const int blocks_;
    bool held_ = false;
};

}  // namespace thin
