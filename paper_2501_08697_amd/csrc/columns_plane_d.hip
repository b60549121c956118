#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<45>(const ColumnsCall &);
template int columns_plane_n1<48>(const ColumnsCall &);
template int columns_plane_n1<54>(const ColumnsCall &);
}  // namespace apw
