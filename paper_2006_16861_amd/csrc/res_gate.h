// Which resident launches of a process may run side by side on one device.
//
// The tiles of a resident launch wait for each other, so all workgroups of all
// such launches that may overlap must fit the device.  Launches form epochs:
// those of one epoch need no more than the device has and do not wait for each
// other; a launch of the next one waits for every operator of the epoch before,
// on its own stream (and so, through them, for all earlier epochs).  An
// operator's own launches are ordered by its stream and count once.
//
// The unit is 32 workgroups for 32 compute units, each workgroup counted as if it
// took a compute unit: workgroups are dealt out to the 8 XCDs, and there to 4
// shader engines, in turn, so that n of them put at most ceil(n / 32) on one of
// these.  A launch of more than the device has by this count (two workgroups
// share a compute unit in large runs) runs alone.
#pragma once

namespace tdp {

class ResGateBook {
public:
    static constexpr int kMax = 64;
    struct Entry {
        unsigned long long op;
        int need;
        void *event;               // recorded behind the operator's latest launch
    };

    static int units(int workgroups) { return workgroups <= 32 ? 1 : (workgroups + 31) / 32; }

    // Admits a launch of `op`; wait receives the events that it has to wait for
    // (at most kMax), the result is their number.
    int admit(unsigned long long op, void *event, int need, int cap, void **wait)
    {
        if (cap > kMax) cap = kMax;
        int at = 0;
        while (at < nnow_ && now_[at].op != op) ++at;
        const bool in = at < nnow_;
        const int rest = sum_ - (in ? now_[at].need : 0);
        if (in && now_[at].need > need) need = now_[at].need;
        if (rest == 0 || rest + need <= cap) {
            now_[at] = {op, need, event};
            sum_ = rest + need;
            if (in) return 0;      // has waited when it joined
            ++nnow_;
        } else {
            for (int i = 0; i < nnow_; ++i) before_[i] = now_[i];
            nbefore_ = nnow_;
            now_[0] = {op, need, event};
            nnow_ = 1;
            sum_ = need;
        }
        int n = 0;
        for (int i = 0; i < nbefore_; ++i)
            if (before_[i].op != op) wait[n++] = before_[i].event;
        return n;
    }

    // op's waits could not be issued: its launch does not take place
    void withdraw(unsigned long long op) { sum_ -= drop(now_, nnow_, op); }

    // op's launches are over and its event goes
    void forget(unsigned long long op)
    {
        withdraw(op);
        drop(before_, nbefore_, op);
    }

private:
    static int drop(Entry *e, int &n, unsigned long long op)
    {
        int need = 0, k = 0;
        for (int i = 0; i < n; ++i) {
            if (e[i].op == op) need = e[i].need;
            else e[k++] = e[i];
        }
        n = k;
        return need;
    }

    // every entry but a lone one needs at least 1 of at most kMax
    Entry now_[kMax] = {}, before_[kMax] = {};
    int nnow_ = 0, nbefore_ = 0, sum_ = 0;
};

}  // namespace tdp
