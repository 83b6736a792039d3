// The plan's rules that need no device (lgf_host.h), for tests/test_host_rules.py.  Reads one
// query per line from stdin and prints one answer per line:
//   fields items chunks bytes        near_fields_fit
//   items targets                    field_items
//   runs n copies height...          of a batch of `copies` layouts, each a row of 2x2-block towers of
//                                    these heights: the level-0 runs of the first layout (their groups),
//                                    then 0, all runs, and the 4-wave workgroups that march in lockstep
//                                    (4 equal runs of 8 and more), the others
//   solve overlap eager_only lattice beside graph plan_eager plan_graph
//                                    solve_schedule
//   m2l parents S F n                m2l_default: children per lane, parents per workgroup
//   schedule n p levels prec edge ex ey ez step
//                                    default_schedule, eager and graph, of the cube of edge^3 blocks;
//                                    ex > 0: f on every step-th block of its corner of ex x ey x ez
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "lgf_host.h"

using namespace lgfdev;

int main() {
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string kind;
        in >> kind;
        if (kind == "fields") {
            long long items = 0;
            int chunks = 0, bytes = 0;
            in >> items >> chunks >> bytes;
            std::cout << near_fields_fit(items, chunks, bytes) << "\n";
        } else if (kind == "items") {
            long long n = 0;
            in >> n;
            std::cout << field_items(n) << "\n";
        } else if (kind == "runs") {
            int n = 0, copies = 0, h = 0;
            in >> n >> copies;
            std::vector<int32_t> b;
            for (int x = 0; in >> h; x += 2)
                for (int z = 0; z < h; ++z) b.insert(b.end(), {x, 0, z, x + 1, 0, z, x, 1, z, x + 1, 1, z});
            std::vector<HostPlan> parts(copies);
            for (HostPlan& P : parts)
                if (build_host(b.data(), (int64_t)b.size() / 3, n, 4, 0, P) != LGF_OK) return 3;
            const HostPlan H = concat(parts);
            if (check_host(H) != LGF_OK) return 3;
            // parts left in the order of their blocks give the same union
            for (HostPlan& P : parts)
                if (build_host(b.data(), (int64_t)b.size() / 3, n, 4, 0, P = HostPlan(), nullptr, 0, true) != LGF_OK)
                    return 3;
            const HostPlan U = concat(parts);
            bool same_lists = U.g0_runs == H.g0_runs && U.g0_src64 == H.g0_src64 && U.g0_tgt8 == H.g0_tgt8 &&
                              U.g0_flags == H.g0_flags;
            for (int l = 1; l <= H.L; ++l)
                same_lists = same_lists && U.lv[l].m2l_ord == H.lv[l].m2l_ord && U.lv[l].m2l_mask == H.lv[l].m2l_mask &&
                             U.lv[l].src216 == H.lv[l].src216 && U.lv[l].par == H.lv[l].par;
            if (!same_lists) return 4;
            const std::vector<int32_t>& r = H.g0_runs;
            for (size_t k = 0; k < r.size() && H.g0_coord[4 * r[k] + 3] == 0; k += 2) std::cout << r[k + 1] << " ";
            int lock = 0, other = 0;
            for (size_t k = 0; k < r.size(); k += 8) {
                bool same = k + 8 <= r.size() && r[k + 1] >= 8;
                for (size_t j = k; same && j < k + 8; j += 2) same = r[j + 1] == r[k + 1];
                ++(same ? lock : other);
            }
            std::cout << "0 " << r.size() / 2 << " " << lock << " " << other << "\n";
        } else if (kind == "solve") {
            int v[7] = {};
            for (int& x : v) in >> x;
            std::cout << solve_schedule(v[0], v[1] != 0, v[2] != 0, v[3] != 0, v[4] != 0, v[5], v[6]) << "\n";
        } else if (kind == "m2l") {
            long long parents = 0, S = 0;
            int F = 0, n = 0;
            in >> parents >> S >> F >> n;
            const M2LVariant v = m2l_default(parents, S, F, n);
            std::cout << v.children << " " << v.parents << "\n";
        } else if (kind == "schedule") {
            int n = 0, p = 0, levels = 0, prec = 0, edge = 0, ex = 0, ey = 0, ez = 0, step = 1;
            in >> n >> p >> levels >> prec >> edge >> ex >> ey >> ez >> step;
            std::vector<int32_t> all, src;
            int k = 0;
            for (int z = 0; z < edge; ++z)
                for (int y = 0; y < edge; ++y)
                    for (int x = 0; x < edge; ++x) {
                        all.insert(all.end(), {x, y, z});
                        if (x < ex && y < ey && z < ez && k++ % step == 0) src.insert(src.end(), {x, y, z});
                    }
            HostPlan H;
            const lgf_status st = src.empty() ? build_host(all.data(), (int64_t)all.size() / 3, n, p, levels, H)
                                              : build_host(src.data(), (int64_t)src.size() / 3, n, p, levels, H,
                                                           all.data(), (int64_t)all.size() / 3);
            if (st != LGF_OK) return 3;
            const lgf_precision pr = prec == 64 ? LGF_F64 : LGF_F32;
            std::cout << default_schedule(H, pr, false) << " " << default_schedule(H, pr, true) << "\n";
        } else {
            std::cerr << "unknown query " << kind << "\n";
            return 2;
        }
    }
    return 0;
}
