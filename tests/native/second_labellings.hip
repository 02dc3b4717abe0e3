// Host check (no GPU): blocks that end while another thread gives up the second
// labellings.  Meant for a build with AddressSanitizer on the host side.
#include "basis.hip"

#include <cstdio>
#include <thread>

int main() {
    using namespace xdg;
    int bad = 0;
    for (int round = 0; round < 8; ++round) {
        const int n = 4000;
        std::vector<xdg_basis_s *> blocks(n);
        for (auto &b : blocks) {
            b = new xdg_basis_s;
            auto rel = std::make_shared<Relabelled>();
            rel->bytes = 1;
            offer_relabelled(b, std::move(rel));
        }
        std::thread give([&] {
            set_device_memory_limit(device_memory_in_use() + 1);
            DevBuf d;
            bad += d.alloc(2) != XDG_ENOMEM;   // one byte short
            bad += !give_up_relabelled();
            set_device_memory_limit(0);
        });
        while (blocks[0]->has_inner) {}
        for (auto *b : blocks) {
            while (b->has_inner) {}
            forget_relabelled(b);
            delete b;
        }
        give.join();
        auto *later = new xdg_basis_s;   // the list holds no block that ended
        offer_relabelled(later, std::make_shared<Relabelled>());
        forget_relabelled(later);
        delete later;
        bad += give_up_relabelled();     // nothing was missing
    }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
