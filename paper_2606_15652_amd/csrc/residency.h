// Resident workgroups per CU of a kernel by its dynamic LDS, asked of the runtime
// as seldom as possible.  More LDS never lets more workgroups in, so between two
// sizes of the same answer every size has that answer: a kernel keeps, per
// answer, the smallest and the largest size that got it.  A few queries settle
// the range that a program uses (a slot per size ran full after 64 shapes, and
// every further shape asked on each call).  Not safe for several threads by itself.
#pragma once

#include <stddef.h>

namespace mq_host {

class ResidencyTable {
    static constexpr int kKernels = 32, kMost = 8;
    struct Row {
        const void* kernel;
        struct {
            bool known;
            size_t least, most;
        } of[kMost + 1];
    };
    Row rows_[kKernels] = {};
    int used_ = 0;

public:
    // query(): workgroups per CU, or 0 if the runtime could not say (then 1, and
    // nothing is remembered).
    template <typename Query>
    int get(const void* kernel, size_t lds, Query&& query) {
        Row* row = nullptr;
        for (int i = 0; i < used_ && !row; ++i)
            if (rows_[i].kernel == kernel) row = &rows_[i];
        if (row)
            for (int occ = 1; occ <= kMost; ++occ)
                if (row->of[occ].known && row->of[occ].least <= lds && lds <= row->of[occ].most) return occ;
        const int occ = query();
        if (occ < 1) return 1;
        if (!row && used_ < kKernels) {
            row = &rows_[used_++];
            row->kernel = kernel;
        }
        if (row && occ <= kMost) {
            auto& o = row->of[occ];
            o.least = o.known && o.least < lds ? o.least : lds;
            o.most = o.known && o.most > lds ? o.most : lds;
            o.known = true;
        }
        return occ;
    }
};

}  // namespace mq_host
