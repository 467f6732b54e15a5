// How much of the free device memory a plan's optional parts take (plain C++: the host's arithmetic, without HIP).
#pragma once
#include <cstddef>

namespace spg {

struct PlanRoom {
  double list;     // structure list of the dense rows
  double shorts;   // order of the products of short rows
  bool desc;       // whether the descriptions of A's entries stay
};

// free_b: bytes free now, the descriptions (desc bytes) already taken; list_want / short_want: what the other two could use;
// c_most: what C can take at most; asked: the caller's limit, of the list and of what short rows have (descriptions included).
// The list has a third of the free memory at most, whatever C takes (the caller's choice since there is a list).  The short rows
// come after C: what they take leaves room for the largest C beside the list, or comes out of the list's own share (a sixteenth
// of it: a few hundred bytes for every short row between the dense ones of a graph).
inline PlanRoom plan_room(double free_b, double list_want, double short_want, double desc, double c_most, double asked) {
  auto least = [](double a, double b) { return a < b ? a : b; };
  PlanRoom r{};
  r.desc = desc > 0.0 && desc <= least((free_b + desc) / 4.0, asked) && free_b - least(list_want, least(free_b / 3.0, asked)) >= c_most;
  if (!r.desc) { free_b += desc; desc = 0.0; }
  r.list = least(list_want, least(free_b / 3.0, asked));
  const double room = free_b - r.list - c_most > 0.0 ? free_b - r.list - c_most : 0.0;
  r.shorts = least(short_want, least((free_b + desc) / 4.0, asked) - desc);
  if (r.shorts > room) {
    const double share = r.list / 16.0;
    r.shorts = least(r.shorts, room > share ? room : share);
    r.list -= r.shorts > room ? r.shorts - room : 0.0;
  }
  return r;
}

}  // namespace spg
