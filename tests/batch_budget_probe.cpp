// Prints what a batch may take for operands and stored rows at each free size.
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

int main(int argc, char **argv) {
    for (int i = 1; i < argc; ++i) {
        const knn::BatchBudget b = knn::batch_budget(std::strtoull(argv[i], nullptr, 10));
        std::printf("%zu %zu\n", b.split, b.rows);
    }
    return 0;
}
