// What the workgroups of a launch in two sets of column tiles (strips) compute: every one of every panel (group) once, the first
// set's before the second's.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "spmm_places.h"

#define REQUIRE(x) do { if (!(x)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); std::exit(1); } } while (0)

static void check(uint32_t rows, uint32_t columns, uint32_t set)
{
    std::vector<int> seen((size_t)rows * columns, 0);
    for (uint32_t place = 0; place < rows * columns; ++place) {
        const set_place at = place_in_sets(place, rows, columns, set);
        REQUIRE(at.row < rows && at.column < columns && (at.column < set) == (place < rows * set));
        ++seen[(size_t)at.row * columns + at.column];
    }
    for (int n : seen) REQUIRE(n == 1);
    for (uint32_t behind = 0; behind < 16; ++behind) REQUIRE(place_in_sets(rows * columns + behind, rows, columns, set).row >= rows);  // padding
}

int main()
{
    for (uint32_t rows = 1; rows <= 40; ++rows)
        for (uint32_t columns = 1; columns <= 36; ++columns)
            for (uint32_t set = 1; set <= columns; ++set) check(rows, columns, set);
    check(5000, 260, 132);
    const uint32_t rows = 1u << 20, columns = 4095, set = 2048;  // nearly 2^32 places
    const set_place last = place_in_sets(rows * columns - 1, rows, columns, set), first = place_in_sets(rows * set, rows, columns, set);
    REQUIRE(last.row == rows - 1 && last.column == columns - 1 && first.row == 0 && first.column == set);
    std::printf("ok\n");
    return 0;
}
