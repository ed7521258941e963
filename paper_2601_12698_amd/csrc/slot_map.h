// Who may use which piece of the device memory in which workgroups of one launch meet (addrms_split_body, the gate).  Host
// code only, no HIP.
//
// Such memory belongs to the loaded code object and is cut into units.  A launch has units of its own, from before it is
// queued until it is reported as done in host memory (slot_pool.h); only then are they another launch's.  Nothing else is asked: not
// which stream a launch is on (a stream's handle may come back as another stream's while the first one's work is in flight).
// Each GPU has a copy of the memory, and a map of its own.
#pragma once
#include <stdint.h>

namespace addrms_host {

// The launches with units from one place on are numbered from 1, and never with the same number again: what one of them leaves in
// memory is told from what another has written there by the number (the gate).  After 2^32 - 1 of them, which take months, the
// place is not used any more.
template <int UNITS, typename Number = uint32_t>
class SlotMap {
public:
    // The first of `units` adjacent units that are free now; -1: none found.  Calls are serialised by the caller.
    // done[u]: the number of the last launch with units from u on that has been reported.
    int take(int units, const volatile uint32_t* done)
    {
        // Once around from behind the units taken last, where those longest in flight are.  No launch's units begin before u
        // and end behind it: u is 0 or where some launch's units end, and those that begin in what is taken are free.
        for (int u = next_, left = UNITS + units; left > 0;) {
            if (u + units > UNITS) {
                left -= UNITS - u;
                u = 0;
            }
            const int busy = busy_end(u, units, done);
            if (busy == 0) {
                for (int i = u; i < u + units; ++i) unit_[i].span = 0;
                unit_[u].span = units;
                ++unit_[u].number;
                next_ = u + units;
                return u;
            }
            left -= busy - u;
            u = busy;
        }
        return -1;
    }
    // The number by which the launch with these units is reported.
    uint32_t number(int first) const { return unit_[first].number; }
    // There is no such launch after all.
    void give_back(int first) { unit_[first].span = 0; }

private:
    struct Unit {
        Number number;                                       // of the last launch with units from here on
        int span;                                            // its units; 0: none, or free
    };
    // 0: units [u, u + n) are free.  Else where to look on: the end of the first launch's in flight.
    int busy_end(int u, int n, const volatile uint32_t* done) const
    {
        for (int i = u; i < u + n; i += unit_[i].span ? unit_[i].span : 1)
            if (unit_[i].span && done[i] != unit_[i].number) return i + unit_[i].span;
        return unit_[u].number == static_cast<Number>(-1) ? u + 1 : 0;       // no more launches from here on
    }
    Unit unit_[UNITS] = {};
    int next_ = 0;
};

}  // namespace addrms_host
