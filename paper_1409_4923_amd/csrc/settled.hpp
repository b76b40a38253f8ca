// settled.hpp -- a question about the built code whose answer cannot change, asked until it
// has been answered: a call that failed says nothing about the code and is made again.
#pragma once

#include <atomic>

namespace bm {

class Settled {
    std::atomic<int> known{0};           // 0 not answered, 1 no, 2 yes

public:
    // ask(bool &yes) returns 0 if it could answer, else an error.  Returns that error, or 0
    // with the answer in `yes`.
    template <typename Ask> auto operator()(bool &yes, Ask ask) -> decltype(ask(yes))
    {
        int k = known.load(std::memory_order_relaxed);
        if (k == 0) {
            bool y = false;
            const auto e = ask(y);
            if (e) return e;
            k = y ? 2 : 1;
            known.store(k, std::memory_order_relaxed);
        }
        yes = k == 2;
        return decltype(ask(yes))(0);
    }
};

} // namespace bm
