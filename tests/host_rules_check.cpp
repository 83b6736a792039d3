// The plan's rules that need no device (lgf_host.h), for tests/test_host_rules.py.  Reads one
// query per line from stdin and prints one answer per line:
//   fields items chunks bytes        near_fields_fit
#include <iostream>
#include <sstream>
#include <string>

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
        } else {
            std::cerr << "unknown query " << kind << "\n";
            return 2;
        }
    }
    return 0;
}
